"""Three and four query tokens over a bf16 cache at the edges of the kernels' tiles and units.  A context of few workgroups gives
three tokens to decode_bf16_multi_kernel where one of 256 takes short_bf16_multi_kernel; four tokens always take the former, in
long and in short segments.  Tolerance: TOL_BF16, as for every bf16 case (weights rounded to bf16, 2^-9 each)."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2507_19427_amd as mfa
import paper_2507_19427_amd.workloads as W

import gpu_util as U

pytestmark = pytest.mark.gpu

# every remainder of a 32-token unit and a 64-token tile, sequences shorter than the new tokens, runs long enough for the steady loop
LENS = [4133, 1, 0, 2, 3, 31, 32, 33, 34, 63, 64, 65, 66, 67, 95, 97, 128, 130, 640, 1501]


def _run(ctx, case, qm):
    d = U.to_dev
    hint = int(case.seq_lens.max())
    if case.paged:
        out = mfa.mfa_decode_attn_paged_multi(ctx, d(qm), d(case.k_pool), d(case.v_pool), d(case.block_table), d(case.seq_lens), hint)
    else:
        out = mfa.mfa_decode_attn_multi(ctx, d(qm), d(case.k), d(case.v), d(case.seq_lens), hint)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _compare(case, q_len, mask_dim=None):
    qm = W.make_multi_query(case, q_len, 43)
    if mask_dim is not None:
        qm[..., mask_dim] = 1.0
    ref = []
    for j in range(q_len):
        lens = torch.clamp(case.seq_lens - (q_len - 1 - j), min=0).to(torch.int32)
        ref.append(U.run_oracle(dataclasses.replace(case, q=qm[:, j].contiguous(), seq_lens=lens)))
    ref = np.stack(ref, axis=1)
    for n in (256, 5, 1):
        print(f"[case] {q_len} query tokens, {n} workgroups", flush=True)
        ctx = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=32, max_seq_len=8192, target_workgroups=n))
        got = _run(ctx, case, qm)
        err = U.row_normalised_error(got, ref)
        print(f"   row-normalised max error {err:.3e}", flush=True)
        assert err <= U.TOL_BF16
        assert np.array_equal(got, _run(ctx, case, qm))
        ctx.close()


@pytest.mark.parametrize("q_len", [3, 4])
@pytest.mark.parametrize("paged", [False, True])
def test_both_kernels_at_the_edges_of_units_and_tiles(q_len, paged):
    if paged:
        case = W.make_paged_case("multi", 71, seq_lens=LENS)
    else:
        case = W.make_contiguous_case("multi", 71, B=len(LENS), S=max(LENS), seq_lens=LENS, poison=True)
    _compare(case, q_len)


@pytest.mark.parametrize("q_len", [3, 4])
def test_scores_that_outrun_the_reference_exponent(q_len):
    """Keys scaled until their scores lie far above (and below) the rest: late in a run, twice in a row, in the last unit."""
    lens = [4000, 900, 130, 2000]
    case = W.make_contiguous_case("multirestart", 72, B=len(lens), S=4000, seq_lens=lens, poison=True)
    for b, pos, gain in ((0, 3333, 256.0), (1, 77, 64.0), (1, 500, 512.0), (3, 1999, 256.0)):
        case.k[b, pos] = case.k[b, pos] * gain
    _compare(case, q_len)


@pytest.mark.parametrize("q_len", [3, 4])
@pytest.mark.parametrize("n_masked", [31, 32, 33, 200, 4000])
def test_scores_of_minus_infinity_ahead_of_finite_ones(q_len, n_masked):
    """Keys whose scores are -inf for every head (dimension 0 used as a mask: -inf in the key, positive in the query) at the start of a
    sequence: their weight is 0, whatever unit, segment or kernel they begin."""
    lens = [4100, 900, 300, 2000]
    case = W.make_contiguous_case("multimask", 73, B=len(lens), S=max(lens), seq_lens=lens, poison=True)
    case.k[:, :n_masked, 0] = torch.where(torch.arange(n_masked) < case.seq_lens[:, None] - 4, float("-inf"), case.k[:, :n_masked, 0].float()).to(case.k.dtype)
    _compare(case, q_len, mask_dim=0)
