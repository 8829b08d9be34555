"""The streaming product behind the three projections at the edges of its tiles: 16-row blocks, the 64- and 128-row forms, k ranges
that end in half a stage, single strips and groups of four."""
import numpy as np
import pytest
import torch

import paper_2507_19427_amd as mfa
from oracle import mfa_oracle as O

import gpu_util as U

pytestmark = pytest.mark.gpu

# bf16 result: 2^-9 of an element; the query path rounds its normalised row as well, the output projection its activations.  Sums in 32 bits.
TOL = 1e-2


@pytest.mark.parametrize("d_model", [64, 192, 256, 1088])      # 1 and 3 units of 64 k; groups of four strips; 17 units over 8 strips
@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 65, 112, 127, 128, 129, 200])
def test_products_at_tile_edges(B, d_model):
    print(f"\n[case] products B={B} d_model={d_model}", flush=True)
    rank = 128 if d_model < 1088 else 384
    ctx = U.get_ctx(max_batch=256, max_seq_len=1024, d_model=d_model, q_rank=rank)
    g = torch.Generator().manual_seed(1000 * d_model + B)
    x = torch.full((B + 3, d_model), float("nan"), dtype=torch.bfloat16)      # rows past B must not be seen
    x[:B] = torch.randn(B, d_model, generator=g).to(torch.bfloat16)
    attn = torch.full((B + 3, 64, 256), float("nan"))
    attn[:B] = torch.randn(B, 64, 256, generator=g) * 0.05
    w_kv, w_qa, w_qb, w_o = ((torch.randn(k, n, generator=g) * 0.05).to(torch.bfloat16)
                             for k, n in ((d_model, 512), (d_model, rank), (rank, 16384), (16384, d_model)))
    ctx.workspace.fill_(0xFF)                                                # nor anything a former call has left
    k = torch.zeros(B, 2, 256, dtype=torch.bfloat16, device="cuda")
    v = torch.zeros_like(k)
    lens = torch.ones(B, dtype=torch.int32, device="cuda")
    mfa.mfa_kv_append(ctx, x.cuda()[:B], w_kv.cuda(), k, v, lens)
    ctx.workspace.fill_(0xFF)
    q = mfa.mfa_query_proj(ctx, x.cuda()[:B], w_qa.cuda(), w_qb.cuda())
    ctx.workspace.fill_(0xFF)
    y = mfa.mfa_out_proj(ctx, attn.cuda()[:B], w_o.cuda())
    torch.cuda.synchronize()
    b = O.bits_of
    ref = O.linear(b(x[:B]), b(w_kv))
    assert U.row_normalised_error(torch.cat([k[:, 1], v[:, 1]], 1).float().cpu().numpy(), ref) <= TOL
    assert not k[:, 0].any() and not v[:, 0].any()
    rows = sorted({0, B - 1, B // 2, min(15, B - 1), min(16, B - 1), min(64, B - 1)})
    _, q64, _ = O.query_proj(b(x[rows]), b(w_qa), b(w_qb), 1e-6, want_f64=True)
    assert torch.isfinite(q).all() and torch.isfinite(y).all()
    assert U.row_normalised_error(q[rows].float().cpu().numpy().reshape(-1, 256), np.asarray(q64).reshape(-1, 256)) <= TOL
    assert U.row_normalised_error(y[rows].float().cpu().numpy(), O.linear(attn[rows].reshape(len(rows), -1).numpy(), b(w_o))) <= TOL


@pytest.mark.parametrize("B", [5, 40, 100])
def test_a_row_that_is_not_finite_stays_alone(B):
    """Rows share the matrix instructions' other operand only: infinities and NaN of one row reach no other."""
    ctx = U.get_ctx(max_batch=256, max_seq_len=1024, d_model=256, q_rank=128)
    g = torch.Generator().manual_seed(77 + B)
    attn = torch.randn(B, 64, 256, generator=g) * 0.05
    w_o = (torch.randn(16384, 256, generator=g) * 0.05).to(torch.bfloat16).cuda()
    clean = mfa.mfa_out_proj(ctx, attn.cuda(), w_o).cpu()
    attn[B // 2, 3, 7], attn[B // 2, 60, 200] = float("inf"), float("nan")
    got = mfa.mfa_out_proj(ctx, attn.cuda(), w_o).cpu()
    assert torch.isnan(got[B // 2]).all()
    others = [i for i in range(B) if i != B // 2]
    assert torch.equal(got[others].view(torch.int16), clean[others].view(torch.int16))


def test_rank_beyond_a_thread_group():
    """A rank above four columns for each of 512 threads: the rows' further columns pass through LDS."""
    B, d_model, rank = 3, 128, 2176
    ctx = U.get_ctx(max_batch=256, max_seq_len=1024, d_model=d_model, q_rank=rank)
    g = torch.Generator().manual_seed(5)
    x = torch.randn(B, d_model, generator=g).to(torch.bfloat16)
    w_qa, w_qb = ((torch.randn(k, n, generator=g) * 0.05).to(torch.bfloat16) for k, n in ((d_model, rank), (rank, 16384)))
    gain = 1.0 + 0.1 * torch.randn(rank, generator=g)
    q = mfa.mfa_query_proj(ctx, x.cuda(), w_qa.cuda(), w_qb.cuda(), rms_gain=gain.cuda()).float().cpu().numpy()
    b = O.bits_of
    _, q64, _ = O.query_proj(b(x), b(w_qa), b(w_qb), 1e-6, gain=gain.numpy(), want_f64=True)
    assert U.row_normalised_error(q.reshape(-1, 256), np.asarray(q64).reshape(-1, 256)) <= TOL


def test_rows_more_than_two_gib_apart():
    """32 rows of x that lie more than 2 GiB apart from first to last, as one wave reads them; all of x and w_qa but five k are zeros."""
    B, d_model, rank = 65, 35 << 20, 128
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("takes 33 GB of device memory")
    ctx = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=B, max_seq_len=1024, d_model=d_model, q_rank=rank))
    g = torch.Generator().manual_seed(6)
    ks = torch.tensor([0, 1003, d_model // 2 + 70, d_model - 64, d_model - 1])
    some_x = torch.randn(B, 5, generator=g).to(torch.bfloat16)
    some_w, w_qb = ((torch.randn(k, n, generator=g) * 0.05).to(torch.bfloat16) for k, n in ((5, rank), (rank, 16384)))
    x = torch.zeros(B, d_model, dtype=torch.bfloat16, device="cuda")
    w_qa = torch.zeros(d_model, rank, dtype=torch.bfloat16, device="cuda")
    x[:, ks.cuda()], w_qa[ks.cuda()] = some_x.cuda(), some_w.cuda()
    q = mfa.mfa_query_proj(ctx, x, w_qa, w_qb.cuda()).float().cpu().numpy()
    ctx.close()
    del x, w_qa, ctx
    torch.cuda.empty_cache()
    c = some_x.double() @ some_w.double()
    c = c / torch.sqrt(c.square().mean(-1, keepdim=True) + 1e-6)
    assert U.row_normalised_error(q.reshape(-1, 256), (c @ w_qb.double()).numpy().reshape(-1, 256)) <= TOL
