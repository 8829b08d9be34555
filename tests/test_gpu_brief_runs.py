"""Few rows of longer contexts, whose units of 32 tokens are dealt out to runs that leave partial results: numbers of runs and lengths around units, runs and
rounds of waves, every cache type, layout and number of query tokens, against 64 bits, the kernels that cut the cache and the oracle."""
import numpy as np
import pytest
import torch

import paper_2507_19427_amd as mfa
from paper_2507_19427_amd import workloads as W

import gpu_util as U

pytestmark = pytest.mark.gpu


# (lengths, query tokens, hint): 16 to 64 runs of one row, 32 of two, 9 of five (a hint that is no multiple of anything), 4 of sixteen, 3 of twenty; more runs than
# units, lengths of 0, 1 and less than the query tokens; 16, 4, 2 runs with several tokens, 2 of 24 rows with two
SIZES = [
    ([1025], 1, 1025), ([8200], 1, 8200), ([33], 1, 5000), ([4096, 2047], 1, 4096), ([1300, 0, 1, 289, 1057], 1, 1301), ([0, 31, 32, 2000] * 4, 1, 2000),
    ([1600, 1, 513] * 6 + [96, 97], 1, 1600), ([3000, 2], 2, 3000), ([2100], 4, 2100), ([1, 2, 3, 2500], 4, 2500), ([4, 0, 2049, 33, 700, 2500, 65, 1], 4, 2500), ([1500, 700, 2, 64, 1499], 3, 1500)]

RUNS = [(*size, kv) for size in SIZES for kv in ("bf16", "fp8", "fp4")]
RUNS += [([2048, 1, 33, 700] * 3, 2, 2048, "bf16"), ([2600, 1, 33, 700] * 3, 2, 2600, "fp8"), ([2600, 1, 33, 700] * 3, 2, 2600, "fp4")]


@pytest.mark.parametrize("lens,q_len,hint,kv", RUNS)
def test_runs(lens, q_len, hint, kv):
    print(f"\n[case] runs {len(lens)} x {max(lens)} under {hint}, {q_len} query tokens, {kv}", flush=True)
    B, ctx = len(lens), U.get_ctx()
    paged = W.make_paged_case("runs", 60 + B, lens, kv_dtype=kv, spare_pages=3, poison=True, max_blocks=(hint + 63) // 64)
    case = W.paged_to_contiguous(paged, hint)
    q = W.make_multi_query(case, q_len, 7) if q_len > 1 else case.q.view(B, 1, 64, 256)
    got = U.attend(ctx, case, q, hint)
    assert torch.equal(got, U.attend(ctx, paged, q, hint))
    # the accuracy of little work: weights of 16 bits
    err = U.weight_error(case, q, got)
    print(f"   error {err:.2e} of sum w |v|", flush=True)
    assert err <= U.WEIGHT_ERROR
    tol = U.TOL_BF16 if kv == "bf16" else U.TOL_FP8
    assert U.row_normalised_error(got.numpy(), U.attend(U.get_ctx(target_workgroups=256), case, q, hint).numpy()) <= tol
    # the oracle on some rows: query token j attends to the first L - (q_len - 1 - j) tokens
    full, worst = case.seq_lens, 0.0
    for j in range(q_len):
        case.q, case.seq_lens = q[:, j].contiguous(), (full - (q_len - 1 - j)).clamp(min=0).to(torch.int32)
        rows = U.sample_rows(case, 10, seed=j)
        worst = max(worst, U.row_normalised_error(np.stack([got[b, j, h].numpy() for b, h in rows]), U.run_oracle(case, rows=rows)))
    print(f"   error {worst:.2e}", flush=True)
    assert worst <= tol


@pytest.mark.parametrize("kv", ["bf16", "fp4"])
def test_runs_replayed(kv):
    """In a captured graph: other lengths under the same hint, with eager calls of other sizes (the same scratch memory) between the replays."""
    hint = 2500
    case = W.make_contiguous_case("runs graph", 31, B=3, S=hint, kv_dtype=kv, poison=False)
    d, ctx = U.to_dev, U.get_ctx()
    t = [d(case.q.view(3, 1, 64, 256)), d(case.k), d(case.v), d(case.seq_lens), hint, d(case.k_scale), d(case.v_scale)]
    out = torch.empty(3, 1, 64, 256, device="cuda")
    mfa.mfa_decode_attn_multi(ctx, *t, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mfa.mfa_decode_attn_multi(ctx, *t, out=out)
    for lens in ([2500, 2500, 2500], [1, 0, 2049], [700, 2500, 31], [0, 0, 0]):
        t[3].copy_(torch.tensor(lens, dtype=torch.int32))
        eager = mfa.mfa_decode_attn_multi(ctx, *t).cpu()
        mfa.mfa_decode_attn_multi(ctx, t[0][:1].contiguous(), t[1][:1], t[2][:1], torch.tensor([hint], dtype=torch.int32, device="cuda"), hint, *[x if x is None else x[:1] for x in t[5:]])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.cpu(), eager), lens


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_runs_of_minus_infinity(kv):
    """Tokens 0 .. 199 have scores of -inf: all that some of the runs have under a length of 230, and the first units of every run under 1500.  The rows are
    those of the same cache without them."""
    S, skip = 1500, 200
    case = W.make_contiguous_case("runs inf", 93, B=2, S=S, kv_dtype=kv, seq_lens=[S, 230], poison=False)
    case.q[..., 0] = 1.0
    if kv == "bf16":
        case.k[:, :skip, 0] = float("-inf")
    else:
        case.k.view(torch.uint8)[:, :skip] = 0
        case.k.view(torch.uint8)[:, :skip, 0] = 0xB8                    # -1 in dim 0, 0 elsewhere
        case.k_scale[:, :skip] = float("inf")
    got = U.attend(U.get_ctx(), case, case.q.view(2, 1, 64, 256), S)
    for name in ("k", "v", "k_scale", "v_scale"):
        t = getattr(case, name)
        setattr(case, name, None if t is None else t[:, skip:].contiguous())
    case.seq_lens = case.seq_lens - skip
    rows = U.sample_rows(case, 16)
    err = U.row_normalised_error(np.stack([got[b, 0, h].numpy() for b, h in rows]), U.run_oracle(case, rows=rows))
    print(f"\n[case] runs of -inf, {kv}: error {err:.2e}", flush=True)
    assert err <= (U.TOL_BF16 if kv == "bf16" else U.TOL_FP8)
