"""Short contexts, which one launch works off without cutting them: every form of that kernel (by the number of rows) at the edges of its
units of 32 tokens and rounds of waves, for every cache type, layout and number of query tokens.  Weights meet the values as two bf16 terms and sums are in single
precision: against 64 bits the results are held to that (U.WEIGHT_ERROR).  The kernels that cut the cache round weights to 8 bits: against those, and against the oracle, the tolerances
of the other attention tests."""
import numpy as np
import pytest
import torch

import paper_2507_19427_amd as mfa
from paper_2507_19427_amd import workloads as W

import gpu_util as U

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 3, 31, 32, 33, 64, 65, 127, 160, 161, 255, 256, 257, 320]
# (sequences, query tokens, longest): 1 .. 16, 17 .. 32, 33 .. 64 and more rows; a hint of less than a unit; several rounds of every wave
CASES = [(1, 1, 20), (5, 3, 700), (7, 4, 321), (16, 1, 1152), (30, 1, 600), (21, 2, 330), (20, 3, 90), (60, 1, 896), (90, 1, 384), (35, 2, 257)]


@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("B,q_len,longest", CASES)
def test_short_contexts(B, q_len, longest, kv):
    print(f"\n[case] short contexts {B} x {longest}, {q_len} query tokens, {kv}", flush=True)
    lens = [min(EDGES[(3 * b + 1) % len(EDGES)], longest) for b in range(B)]
    lens[-1] = longest
    ctx = U.get_ctx()
    paged = W.make_paged_case("brief", 40 + B, lens, kv_dtype=kv, spare_pages=3, poison=True)
    case = W.paged_to_contiguous(paged, longest)
    q = W.make_multi_query(case, q_len, 7) if q_len > 1 else case.q.view(B, 1, 64, 256)
    got = U.attend(ctx, case, q, longest)
    assert torch.equal(got, U.attend(ctx, paged, q, longest))
    # the accuracy of little work: weights of 16 bits
    err = U.weight_error(case, q, got)
    print(f"   error {err:.2e} of sum w |v|", flush=True)
    assert err <= U.WEIGHT_ERROR
    # the kernels that cut the cache, which have tests of their own
    tol = U.TOL_BF16 if kv == "bf16" else U.TOL_FP8
    assert U.row_normalised_error(got.numpy(), U.attend(U.get_ctx(target_workgroups=256), case, q, longest).numpy()) <= tol
    # the oracle on some rows: query token j attends to the first L - (q_len - 1 - j) tokens
    full, worst = case.seq_lens, 0.0
    for j in range(q_len):
        case.q, case.seq_lens = q[:, j].contiguous(), (full - (q_len - 1 - j)).clamp(min=0).to(torch.int32)
        rows = U.sample_rows(case, 12, seed=j)
        worst = max(worst, U.row_normalised_error(np.stack([got[b, j, h].numpy() for b, h in rows]), U.run_oracle(case, rows=rows)))
    print(f"   error {worst:.2e}", flush=True)
    assert worst <= tol


@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("B", [2, 20, 40, 70])
def test_scores_of_minus_infinity_and_growing_ones(B, kv):
    """Tokens 0 .. 39 (a unit and part of one) have scores of -inf and count for nothing; later scores grow by hundreds, so that every wave's reference
    moves.  The rows are those of the same cache without its first 40 tokens."""
    S, skip = 300, 40
    case = W.make_contiguous_case("brief inf", 90 + B, B=B, S=S, kv_dtype=kv, poison=False)
    case.q[..., 0] = 1.0
    if kv == "bf16":
        case.k[:, skip:] *= (1 + torch.arange(S - skip) / 20).to(torch.bfloat16)[None, :, None]
        case.k[:, :skip, 0] = float("-inf")
    else:
        case.k_scale[:, skip:] *= 1 + torch.arange(S - skip)[None, :] / 20
        case.k.view(torch.uint8)[:, :skip] = 0
        case.k.view(torch.uint8)[:, :skip, 0] = 0xB8 if kv == "fp8" else 0x0A            # -1 in dim 0, 0 elsewhere
        case.k_scale[:, :skip] = float("inf")
    got = U.attend(U.get_ctx(), case, case.q.view(B, 1, 64, 256), S)
    for name in ("k", "v", "k_scale", "v_scale"):
        t = getattr(case, name)
        setattr(case, name, None if t is None else t[:, skip:].contiguous())
    case.seq_lens = case.seq_lens - skip
    rows = U.sample_rows(case, 16)
    err = U.row_normalised_error(np.stack([got[b, 0, h].numpy() for b, h in rows]), U.run_oracle(case, rows=rows))
    print(f"\n[case] -inf and growing scores, {B} sequences, {kv}: error {err:.2e}", flush=True)
    assert err <= (U.TOL_BF16 if kv == "bf16" else U.TOL_FP8)


# (sequences, longest): each form of the uncut kernel, and runs
INFINITIES = [(3, 300), (20, 300), (40, 300), (70, 300), (3, 2500)]


@pytest.mark.parametrize("B,S", INFINITIES)
@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp4"])
def test_infinite_values(B, S, kv):
    """An infinite value (or value scale) makes the elements it meets infinite, not NaN, as in the plain sum of weights times values; NaN is only what
    that has too (infinities of both signs, an infinite scale over a code of 0).  The rest of such a row keeps 16 bits of every weight."""
    print(f"\n[case] infinite values, {B} x {S}, {kv}", flush=True)
    lens = [S, 1, S - 1] + [40] * (B - 3)
    case = W.make_contiguous_case("inf values", 50 + B, B=B, S=S, seq_lens=lens, kv_dtype=kv, poison=True)
    inf = float("inf")
    if kv == "bf16":
        case.v[0, 7, 5] = inf                                           # once; of either sign; of both; at the end of the sequence, and in its first unit and another
        case.v[0, 40, 6] = -inf
        case.v[0, 7, 100], case.v[0, S - 1, 100] = inf, -inf
        case.v[0, S - 1, 255], case.v[0, 33, 9], case.v[0, 3, 9] = inf, inf, inf
        case.v[1, 0, 77], case.v[1, 0, 78] = inf, -inf                  # the only token
    else:
        case.v_scale[0, S - 1] = inf
        case.v_scale[1, 0] = inf
    case.q[0] *= 0.25                                                   # (no weight underflows)
    got = U.attend(U.get_ctx(), case, case.q.view(B, 1, 64, 256), S)[:, 0].double()
    worst = 0.0
    for b, n in enumerate(lens):
        want, magnitude = U.exact_heads(case, b, case.q[b], n)
        same = torch.isnan(got[b]) == torch.isnan(want)
        assert same.all(), (b, int((~same).sum()))
        infinite, finite = torch.isinf(want), torch.isfinite(want)
        assert torch.equal(torch.isinf(got[b]), infinite) and torch.equal(got[b][infinite], want[infinite])
        if n == 1 and kv == "bf16":
            assert torch.equal(got[b][finite], want[finite])            # a row of one token is that token's value row
        if finite.any():
            worst = max(worst, float(((got[b] - want).abs() / magnitude)[finite].max()))
    print(f"   error {worst:.2e} of sum w |v|", flush=True)
    # a weight loses 2^-16 of itself at most in two terms that are both positive; as much again for its score, its exponential and the sums
    assert worst <= 2.0 ** -15


@pytest.mark.parametrize("q_len,lens,hint", [(1, [70, 0, 1, 64, 300], 900), (1, [2100, 1, 65], 4096), (3, [2, 500, 64], 1000)])
def test_block_table_entries_past_the_length_do_not_matter(q_len, lens, hint):
    """Those below the hint may be looked up before the length is known; whatever they hold, the result is the same."""
    case = W.make_paged_case("garbage", 77, lens, spare_pages=3, poison=True, max_blocks=(hint + 63) // 64)
    q = W.make_multi_query(case, q_len, 7) if q_len > 1 else case.q.view(len(lens), 1, 64, 256)
    want = U.attend(U.get_ctx(), case, q, hint)
    for b, n in enumerate(lens):
        past = case.block_table[b, (n + 63) // 64:]
        past.copy_(torch.arange(len(past)) * 99991 - (1 << 30))
    assert torch.isfinite(want).all() and torch.equal(want, U.attend(U.get_ctx(), case, q, hint))
