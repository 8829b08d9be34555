"""The two kernels over the 8-bit and 4-bit caches.  Which one a call takes follows from the tiles per workgroup at the length of
the hint: a context of few workgroups takes decode_lowbit_kernel for what a context of 256 gives to short_lowbit_kernel.

Tolerance: TOL_FP8 as for every low-bit case; both kernels are also held to 4e-3, from their operands: a weight carries 8
significant bits (relative error at most 2^-8 = 3.9e-3, which many tokens average out and a single one shows in full), the query 8 as
well down to 2^-17 of its largest element."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2507_19427_amd as mfa
import paper_2507_19427_amd.workloads as W

import gpu_util as U

pytestmark = pytest.mark.gpu

TOL = 4e-3


def _run(ctx, case, qm, hint):
    d = U.to_dev
    if case.paged:
        out = mfa.mfa_decode_attn_paged_multi(ctx, d(qm), d(case.k_pool), d(case.v_pool), d(case.block_table), d(case.seq_lens), hint,
                                              d(case.k_scale_pool), d(case.v_scale_pool))
    else:
        out = mfa.mfa_decode_attn_multi(ctx, d(qm), d(case.k), d(case.v), d(case.seq_lens), hint, d(case.k_scale), d(case.v_scale))
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _oracle(case, qm):
    q_len = qm.shape[1]
    outs = []
    for j in range(q_len):
        lens = torch.clamp(case.seq_lens - (q_len - 1 - j), min=0).to(torch.int32)
        outs.append(U.run_oracle(dataclasses.replace(case, q=qm[:, j].contiguous(), seq_lens=lens)))
    return np.stack(outs, axis=1)


def _compare(case, q_len, hint, workgroups, schedule=None, mask_dim=None, tol=TOL):
    qm = W.make_multi_query(case, q_len, 41) if q_len > 1 else case.q.unsqueeze(1).contiguous()
    if mask_dim is not None:
        qm[..., mask_dim] = 1.0
    ref = _oracle(case, qm)
    kw = {} if schedule is None else {"schedule": schedule}
    for n in workgroups:
        ctx = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=max(16, case.B), max_seq_len=32768, target_workgroups=n, **kw))
        print(f"[case] {case.kv_dtype} {q_len} query tokens, {n} workgroups", flush=True)
        got = _run(ctx, case, qm, hint)
        err = U.row_normalised_error(got, ref)
        print(f"   row-normalised max error {err:.3e}", flush=True)
        assert err <= tol
        assert np.array_equal(got, _run(ctx, case, qm, hint))
        ctx.close()


# every remainder of a tile and of a pair of tiles, empty and one-token sequences, and runs long enough for the steady loop
LENS = [4133, 1, 0, 63, 64, 65, 127, 128, 129, 640, 1500, 2]


@pytest.mark.parametrize("q_len", [1, 2, 3])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("paged", [False, True])
def test_both_kernels_at_the_edges_of_tiles_and_stages(kv_dtype, q_len, paged):
    if paged:
        case = W.make_paged_case("lowbit", 61, seq_lens=LENS, kv_dtype=kv_dtype)
    else:
        case = W.make_contiguous_case("lowbit", 61, B=len(LENS), S=max(LENS), seq_lens=LENS, kv_dtype=kv_dtype, poison=True)
    _compare(case, q_len, max(LENS), (256, 7, 1))


@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
def test_both_kernels_under_the_fixed_schedule(kv_dtype):
    case = W.make_contiguous_case("lowbitfixed", 62, B=len(LENS), S=max(LENS), seq_lens=LENS, kv_dtype=kv_dtype, poison=True)
    _compare(case, 1, max(LENS), (256, 12), mfa.MFA_SCHEDULE_FIXED)


@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
def test_long_chunks_of_the_fixed_schedule(kv_dtype):
    """Two chunks of 55 tiles per sequence, enough for decode_lowbit_kernel: partial results by item, workgroups whose chunk lies past the
    sequence's end, sequences that end just before, at and after the first chunk's end."""
    lens = [7000, 100, 0, 3519, 3520, 3521, 3584, 1]
    case = W.make_contiguous_case("lowbitchunks", 67, B=len(lens), S=7000, seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    _compare(case, 1, 7000, (16,), mfa.MFA_SCHEDULE_FIXED)


@pytest.mark.parametrize("q_len", [1, 2])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("paged", [False, True])
def test_more_sequences_than_one_wave_scans(kv_dtype, q_len, paged):
    """Above 512 sequences the workgroup works the schedule out together; few workgroups, so decode_lowbit_kernel, and all of them
    for the other kernel.  Empty sequences in front, in runs and at the end.  Tolerance: a row of a few tokens shows a weight's
    rounding, 2^-8, in full, and where their values cancel twice of it."""
    rng = np.random.default_rng(68)
    lens = [0, 0] + [int(x) for x in rng.integers(1, 150, 636)] + [0, 0]
    lens[100:170] = [0] * 70
    lens[639 - 64:639] = [65] * 64
    if paged:
        case = W.make_paged_case("lowbit640", 68, seq_lens=lens, kv_dtype=kv_dtype)
    else:
        case = W.make_contiguous_case("lowbit640", 68, B=len(lens), S=150, seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    _compare(case, q_len, 150, (8, 256), tol=2 * 2.0 ** -8)


@pytest.mark.parametrize("q_len", [1, 2])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
def test_scores_that_outrun_the_reference_exponent(kv_dtype, q_len):
    """Tokens whose key scale is raised until their scores lie hundreds above (and below) the rest, so that the segment is streamed
    again with the maxima it has seen: late in a run of tiles, twice in a row, in the last tile, for one sequence only."""
    lens = [4000, 900, 130, 2000]
    case = W.make_contiguous_case("lowbitrestart", 63, B=len(lens), S=4000, seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    for b, pos, gain in ((0, 3333, 300.0), (1, 77, 100.0), (1, 500, 400.0), (3, 1999, 300.0)):
        case.k_scale[b, pos] *= gain
    _compare(case, q_len, 4000, (256, 3, 1))


def _mask_tokens(case, b, n):
    """Scores of -inf in fp32 for the first n tokens of sequence b and every head whose query element 0 is positive: codes of 0 but
    for the lowest in dimension 0, and a scale near the largest fp32 number."""
    codes = case.k.view(torch.uint8)[b, :n]
    codes.zero_()
    codes[:, 0] = 0xFE if case.kv_dtype == "fp8" else 0x0F
    case.k_scale[b, :n] = 3e38


@pytest.mark.parametrize("q_len", [1, 2])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("n_masked", [63, 64, 65, 128, 200, 4000])
def test_scores_of_minus_infinity_ahead_of_finite_ones(kv_dtype, q_len, n_masked):
    """Their weight is 0, whatever wave, segment or kernel they begin.  Tolerance: some 40 tokens stay at the least; over
    so few a row's largest output can be half of the sum of its weighted magnitudes, and the weights' rounding, at most 2^-8 each, then
    twice that of the result."""
    lens = [4100, 900, 300, 2000, 65]
    case = W.make_contiguous_case("lowbitmask", 64, B=len(lens), S=max(lens), seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    for b, n in enumerate(lens):
        _mask_tokens(case, b, min(n_masked, n - 40))
    _compare(case, q_len, 4100, (256, 7, 3, 1), mask_dim=0, tol=2 * 2.0 ** -8)


@pytest.mark.parametrize("q_len", [1, 2])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("k_scale", [1e3, 3e5, 3e7])
@pytest.mark.parametrize("n_low", [64, 200, 4000])
def test_far_lower_scores_ahead(kv_dtype, q_len, k_scale, n_low):
    """Finite scores far below the rest begin every segment, to either side of 2^24 (where the rounding of an exponent reaches 1): their size
    must not show in what follows.  Tolerance: as for scores of -inf."""
    lens = [4100, 900, 300, 2000, 65]
    case = W.make_contiguous_case("lowbitlow", 69, B=len(lens), S=max(lens), seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    for b, n in enumerate(lens):
        n_here = min(n_low, n - 40)
        _mask_tokens(case, b, n_here)
        case.k_scale[b, :n_here] = k_scale if kv_dtype == "fp4" else k_scale / 64
    _compare(case, q_len, 4100, (256, 7, 1), mask_dim=0, tol=2 * 2.0 ** -8)


@pytest.mark.parametrize("q_len", [1, 2])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("size_log2", [10, 20, 25, 28])
def test_equal_scores_of_any_size_weigh_the_same(kv_dtype, q_len, size_log2):
    """One key for all tokens, scores of either sign up to about 2^size: the result is the mean of the values, as it is for scores of 0, whether
    a token's weight comes from the first tile of a segment or from a later one.  Tolerance: TOL, since a weight's rounding is that of all others."""
    lens = [4100, 900, 300, 65]
    case = W.make_contiguous_case("lowbitequal", 70, B=len(lens), S=max(lens), seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    for b, n in enumerate(lens):
        case.k.view(torch.uint8)[b, :n] = 0x38 if kv_dtype == "fp8" else 0x22               # codes of 1
        case.k_scale[b, :n] = 0.0
    qm = W.make_multi_query(case, q_len, 41) if q_len > 1 else case.q.unsqueeze(1).contiguous()
    ref = _oracle(case, qm)
    for b, n in enumerate(lens):
        case.k_scale[b, :n] = 1.1 * 2.0 ** size_log2 / 4                 # (the elements of a query sum to about 16, the softmax scale is 1/16)
    for n_wgs in (7, 3, 1):
        ctx = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=16, max_seq_len=32768, target_workgroups=n_wgs))
        err = U.row_normalised_error(_run(ctx, case, qm, max(lens)), ref)
        print(f"[case] {kv_dtype} {q_len} query tokens, 2^{size_log2}, {n_wgs} workgroups: {err:.3e}", flush=True)
        assert err <= TOL
        ctx.close()


@pytest.mark.parametrize("q_len", [1, 2])
@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("vscale_log2", [40, 100, 110])
def test_large_values_under_scores_that_grow(kv_dtype, q_len, vscale_log2):
    """Value scales far above 1 and a late token whose score lies some 2^36 above the first ones, which the reference exponent allows: the
    weights, or their sums with the codes, would leave fp32, while the result (2^120 at most) does not.  Tolerance: as above, a row is
    about one token's value."""
    lens = [4000, 900, 130, 2000]
    case = W.make_contiguous_case("lowbitlarge", 65, B=len(lens), S=4000, seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    case.v_scale *= 2.0 ** vscale_log2
    for b, pos in ((0, 3333), (1, 500), (3, 1998)):
        codes = case.k.view(torch.uint8)[b, pos]
        codes.zero_()
        codes[0] = 0x38 if kv_dtype == "fp8" else 0x02                 # 1.0 in dimension 0, where every query holds 1
        case.k_scale[b, pos] = 36 * 16 / 1.4427
    _compare(case, q_len, 4000, (256, 3, 1), mask_dim=0, tol=2 * 2.0 ** -8)


def _weight_rounding_bound(case, row_q, b, n):
    """Per element of the [64, 256] output of sequence b: what the rounding of the weights may cost, from exact weights.  Weight times value
    scale w of token t is held to 2^-8 of itself or to 2^-22 of the largest of its head and 64-token tile, whichever is larger (two e4m3
    terms under one power of two).  Beside it: 2^-9 of each weight for the scores, and 2^-12 of the largest product of a
    tile for the matrix instruction's sums, which keep 2^-13 of it."""
    codes = {"fp8": lambda x: x.double(), "fp4": _e2m1}[case.kv_dtype]
    k, v = codes(case.k[b, :n]), codes(case.v[b, :n])
    s = (row_q.double() @ k.T) * case.k_scale[b, :n].double() * case.scale
    p = torch.softmax(s, dim=-1)
    w = p * case.v_scale[b, :n].double().abs()
    tiles = torch.nn.functional.pad(w, (0, -n % 64)).view(64, -1, 64)
    top = tiles.amax(-1).repeat_interleave(64, dim=-1)[:, :n]
    rounding = torch.maximum(2.0 ** -8 * w, 2.0 ** -22 * top) + 2.0 ** -9 * w
    product = w.unsqueeze(-1) * v.abs().unsqueeze(0)                                    # [64, n, 256]
    largest = torch.nn.functional.pad(product, (0, 0, 0, -n % 64)).view(64, -1, 64, 256).amax(2).sum(1)
    return ((p * case.v_scale[b, :n].double()) @ v).numpy(), (rounding @ v.abs() + 2.0 ** -12 * largest).numpy()


def _e2m1(rows):
    grid = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)
    return torch.stack([grid[(rows & 15).long()], grid[(rows >> 4).long()]], dim=-1).flatten(-2)


@pytest.mark.parametrize("kv_dtype", ["fp8", "fp4"])
@pytest.mark.parametrize("by", ["value scale", "attention"])
@pytest.mark.parametrize("log2", [10, 13, 16, 20, 26])
def test_light_tokens_beside_a_heavy_one(kv_dtype, by, log2):
    """One token of a tile is 2^log2 heavier than the rest, by its value scale or by its weight, and its codes are 0 in half of the
    dimensions: those hold the light tokens' sum alone, to the precision the header states.  Both kernels."""
    lens = [700, 130]
    case = W.make_contiguous_case("lowbitheavy", 66, B=len(lens), S=3200, seq_lens=lens, kv_dtype=kv_dtype, poison=True)
    case.q[..., 0] = 1.0
    for b, pos in ((0, 333), (1, 17)):
        case.v.view(torch.uint8)[b, pos, case.v.shape[-1] // 2:] = 0
        if by == "value scale":
            case.v_scale[b, pos] *= 2.0 ** log2
        else:
            codes = case.k.view(torch.uint8)[b, pos]
            codes.zero_()
            codes[0] = 0x38 if kv_dtype == "fp8" else 0x02             # 1.0 in dimension 0
            case.k_scale[b, pos] = log2 * 16 / 1.4427
    for n in (256, 1):
        ctx = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=16, max_seq_len=8192, target_workgroups=n))
        got = _run(ctx, case, case.q.unsqueeze(1).contiguous(), 3200)[:, 0]
        ctx.close()
        for b, length in enumerate(lens):
            ref, bound = _weight_rounding_bound(case, case.q[b], b, length)
            share = np.abs(got[b] - ref) / bound
            zero_half = np.abs(got[b] - ref)[:, 128:] / np.abs(ref[:, 128:]).max()
            print(f"[case] {n} workgroups, {length} tokens: {share.max():.2f} of the bound, zero half {zero_half.max():.1e} of its largest", flush=True)
            assert share.max() <= 1.0
