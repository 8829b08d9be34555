"""Few rows of many partial results each, which several waves of a block merge: numbers of partial results around the waves and their batches of
eight, equal and ragged lengths, one to four query tokens, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2507_19427_amd as mfa
from paper_2507_19427_amd import workloads as W

import gpu_util as U

pytestmark = pytest.mark.gpu


# (lengths, query tokens, workgroups): a row's partial results are about tiles * workgroups / all tiles
@pytest.mark.parametrize("lens,q_len,n_wgs", [
    ([768], 1, 12), ([64 * 63], 1, 63), ([64 * 65 + 1], 2, 65), ([16384], 1, 256), ([4096, 0, 5], 1, 256), ([64 * 12] * 2, 1, 24),
    ([2000, 3000, 1], 3, 200), ([1500] * 8, 1, 256), ([900, 64, 5000, 1, 2, 700, 3000, 65, 4000], 1, 256), ([1400, 3], 4, 40), ([800] * 16, 1, 208),
    ([2000, 1, 1300, 64, 3000, 2, 900], 2, 256), ([900] * 6, 2, 256), ([1200, 1, 1300, 64, 2000, 2], 4, 256), ([700] * 7, 3, 256)])
@pytest.mark.parametrize("kv", ["bf16", "fp4"])
def test_few_rows(lens, q_len, n_wgs, kv):
    print(f"\n[case] few rows {len(lens)} x {max(lens)}, {q_len} query tokens, {n_wgs} workgroups, {kv}", flush=True)
    B, hint = len(lens), max(lens)
    ctx = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=16, max_seq_len=32768, target_workgroups=n_wgs))
    case = W.make_contiguous_case("few", 70 + B, B=B, S=hint, seq_lens=lens, kv_dtype=kv, poison=True)
    q = W.make_multi_query(case, q_len, 5) if q_len > 1 else case.q.view(B, 1, 64, 256)
    d = U.to_dev
    args = (ctx, d(q), d(case.k), d(case.v), d(case.seq_lens), hint, d(case.k_scale), d(case.v_scale))
    got = mfa.mfa_decode_attn_multi(*args)
    assert torch.equal(got, mfa.mfa_decode_attn_multi(*args))
    got = got.cpu()
    full, worst = case.seq_lens, 0.0
    for j in range(q_len):
        case.q, case.seq_lens = q[:, j].contiguous(), (full - (q_len - 1 - j)).clamp(min=0).to(torch.int32)
        rows = U.sample_rows(case, 10, seed=j)
        worst = max(worst, U.row_normalised_error(np.stack([got[b, j, h].numpy() for b, h in rows]), U.run_oracle(case, rows=rows)))
    print(f"   error {worst:.2e}", flush=True)
    assert worst <= (U.TOL_BF16 if kv == "bf16" else U.TOL_FP8)
