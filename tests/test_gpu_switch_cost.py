"""The schedule's allowance for starting on another sequence: ranges that end inside the allowance, ranges without a tile of their own, sequences
without tiles in between, batches beyond one group of 64 lengths, equal lengths that do not divide evenly."""
import pytest
import torch

import paper_2507_19427_amd as mfa
from paper_2507_19427_amd import workloads as W
from oracle import mfa_oracle as O

import gpu_util as U

pytestmark = pytest.mark.gpu


def _lens(kind):
    g = torch.Generator().manual_seed(len(kind))
    if kind == "odd equal":                                   # 37 x 8 tiles over 256 workgroups: boundaries in mid-range
        return [512] * 37
    if kind == "one past":                                    # a tile more than workgroups: every range but one is a tile
        return [64] * 200 + [0] * 20 + [57 * 64]
    if kind == "short among empty":
        return [0, 1, 0, 0, 65, 0] * 45 + [9000, 0]
    if kind == "three groups":                                # the search goes back over groups of 64 lengths
        return [9000] + torch.randint(0, 700, (140,), generator=g).tolist()
    return [1] * 70 + [12000, 11999, 64, 4000]                # "long tail"


@pytest.mark.parametrize("q_len", [1, 2, 3, 4])
@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("kind", ["odd equal", "one past", "short among empty", "three groups", "long tail"])
def test_against_the_oracle(get_ctx, kind, kv, q_len):
    lens = _lens(kind)
    print(f"\n[case] switch cost {kind} {kv} q_len={q_len} B={len(lens)}", flush=True)
    case = W.make_paged_case("sw", 60 + q_len, lens, kv_dtype=kv, spare_pages=3, poison=True)
    ctx = get_ctx(max_batch=512)
    qm = W.make_multi_query(case, q_len, 61) if q_len > 1 else case.q.unsqueeze(1)
    dev = [U.to_dev(t) for t in (case.k_pool, case.v_pool, case.block_table, case.seq_lens)]
    scales = (U.to_dev(case.k_scale_pool), U.to_dev(case.v_scale_pool))
    ctx.workspace.fill_(0xFF)
    got = mfa.mfa_decode_attn_paged_multi(ctx, qm.cuda(), *dev, max(lens), *scales).cpu().numpy()
    again = mfa.mfa_decode_attn_paged_multi(ctx, qm.cuda(), *dev, max(lens), *scales).cpu().numpy()
    assert (got.view("uint32") == again.view("uint32")).all()
    assert torch.isfinite(torch.from_numpy(got)).all()
    # every sequence, by one head or another; more heads of the longest and of a few others
    longest = sorted(range(len(lens)), key=lambda b: -lens[b])[:2]
    picks = set(longest + [0, 1, len(lens) // 2, len(lens) - 1])
    rows = sorted({(b, (5 * b + 3) % 64) for b in range(len(lens))} | {(b, h) for b in picks for h in (0, 17, 63)})
    b_ = O.bits_of
    kd = {"bf16": O.KV_BF16, "fp8": O.KV_E4M3, "fp4": O.KV_E2M1}[kv]
    opt = lambda t: None if t is None else b_(t)
    for j in range(q_len):
        ref = O.decode_attn_paged(b_(qm[:, j].contiguous()), b_(case.k_pool), b_(case.v_pool), case.block_table.numpy(),
                                  (case.seq_lens - (q_len - 1 - j)).clamp(min=0).numpy(), case.scale,
                                  k_scale_pool=opt(case.k_scale_pool), v_scale_pool=opt(case.v_scale_pool), kv_dtype=kd, rows=rows)
        err = U.row_normalised_error(torch.stack([torch.from_numpy(got[b, j, h]) for b, h in rows]).numpy(), ref)
        assert err <= (U.TOL_BF16 if kv == "bf16" else U.TOL_FP8), (j, err)
