"""Helpers shared by the GPU parity tests: move a host case to the device, run the library through
its binding, run the oracle on the same bytes, and compare with the row-normalised error."""
import numpy as np
import torch

import paper_2507_19427_amd as mfa
from oracle import mfa_oracle as O

TOL_BF16 = 1e-2      # max over rows of max_d|gpu-ref| / max_d|ref|, bf16 cache
TOL_FP8 = 3e-2       # same, fp8 and fp4 caches (the arithmetic after the codes is the same)

_ctx_cache = {}


def get_ctx(max_batch=128, max_seq_len=32768, **kw):
    key = (max_batch, max_seq_len, tuple(sorted(kw.items())))
    if key not in _ctx_cache:
        _ctx_cache[key] = mfa.mfa_decode_init(mfa.MfaConfig(max_batch=max_batch, max_seq_len=max_seq_len, **kw))
    return _ctx_cache[key]


def to_dev(t):
    return None if t is None else t.cuda()


def run_gpu(ctx, case, hint=None):
    """Run one AttnCase through the C boundary; returns the fp32 output as a host numpy array."""
    hint = int(hint if hint is not None else max(int(case.seq_lens.max()), 1))
    q, lens = to_dev(case.q), to_dev(case.seq_lens)
    if case.paged:
        out = mfa.mfa_decode_attn_paged(ctx, q, to_dev(case.k_pool), to_dev(case.v_pool), to_dev(case.block_table),
                                        lens, hint, to_dev(case.k_scale_pool), to_dev(case.v_scale_pool))
    else:
        out = mfa.mfa_decode_attn(ctx, q, to_dev(case.k), to_dev(case.v), lens, hint, to_dev(case.k_scale),
                                  to_dev(case.v_scale))
    torch.cuda.synchronize()
    return out.cpu().numpy()


def run_oracle(case, rows=None):
    b = O.bits_of
    kd = {"bf16": O.KV_BF16, "fp8": O.KV_E4M3, "fp4": O.KV_E2M1}[case.kv_dtype]
    opt = lambda t: None if t is None else b(t)
    if case.paged:
        return O.decode_attn_paged(b(case.q), b(case.k_pool), b(case.v_pool), case.block_table.numpy(),
                                   case.seq_lens.numpy(), case.scale, k_scale_pool=opt(case.k_scale_pool),
                                   v_scale_pool=opt(case.v_scale_pool), kv_dtype=kd, rows=rows)
    return O.decode_attn(b(case.q), b(case.k), b(case.v), case.seq_lens.numpy(), case.scale,
                         k_scale=opt(case.k_scale), v_scale=opt(case.v_scale), kv_dtype=kd, rows=rows)


_E2M1 = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)


def _rows64(codes, scales):
    """Cache rows of a sequence in 64 bits."""
    if codes.dtype == torch.uint8:
        x = torch.stack([_E2M1[(codes & 15).long()], _E2M1[(codes >> 4).long()]], dim=-1).flatten(-2)
    else:
        x = codes.float().double()
    return x if scales is None else x * scales.double()[..., None]


def exact_heads(case, b, q, n):
    """Attention of the queries q [heads, D] over the first n tokens of sequence b (contiguous cache), in 64 bits: the rows (a plain sum of weights times
    values, with its infinities and NaN) and sum_t w_t |v_t|, which is what rounding errors of the weights are relative to."""
    k, v = [_rows64(t[b, :n], None if sc is None else sc[b, :n]) for t, sc in ((case.k, case.k_scale), (case.v, case.v_scale))]
    w = torch.softmax(q.double() @ k.T * case.scale, dim=-1)
    rows = torch.stack([(w[h][:, None] * v).sum(0) for h in range(len(w))])
    return rows, w @ torch.where(torch.isfinite(v), v, torch.zeros_like(v)).abs()


WEIGHT_ERROR = 2.0 ** -16
# of sum_t w_t |v_t|: what a result may differ by where weights meet the values as two bf16 terms.  The terms lose 2^-17 of a weight; scores (256 exact
# products summed in 32 bits, about 10 in size), exponentials and sums as much again.  One bf16 term would lose 2^-9: 3e-4 .. 2e-3
# of that sum in the worst of some thousand elements, at 1152 .. 20 tokens.


def weight_error(case, q, got, n_heads=8, n_seqs=4):
    """Largest error of got [B, q_len, H, D] relative to sum_t w_t |v_t|, over some heads of the longest, the first, the last and other sequences of a contiguous case."""
    B, q_len = q.shape[:2]
    worst = 0.0
    for b in sorted({int(case.seq_lens.argmax()), 0, B - 1, *range(0, B, max(1, B // n_seqs))}):
        for j in range(q_len):
            n = int(case.seq_lens[b]) - (q_len - 1 - j)
            if n <= 0:
                assert (got[b, j] == 0).all()
                continue
            heads = torch.arange(n_heads) * (64 // n_heads) + b % (64 // n_heads)
            want, magnitude = exact_heads(case, b, q[b, j, heads], n)
            worst = max(worst, float(((got[b, j, heads].double() - want).abs() / magnitude).max()))
    return worst


def attend(ctx, case, q, hint):
    """Queries q [B, q_len, H, D] through the multi-token entry point of the case's layout; the result on the host."""
    d = to_dev
    f = mfa.mfa_decode_attn_paged_multi if case.paged else mfa.mfa_decode_attn_multi
    cache = (case.k_pool, case.v_pool, case.block_table) if case.paged else (case.k, case.v)
    scales = (case.k_scale_pool, case.v_scale_pool) if case.paged else (case.k_scale, case.v_scale)
    out = f(ctx, d(q), *[d(t) for t in cache], d(case.seq_lens), hint, *[d(t) for t in scales])
    torch.cuda.synchronize()
    return out.cpu()


def row_normalised_error(got, ref):
    """max over rows of max_d|got-ref| / max_d|ref| (rows whose reference is all zero must match exactly)."""
    got = np.asarray(got, dtype=np.float64).reshape(-1, got.shape[-1])
    ref = np.asarray(ref, dtype=np.float64).reshape(-1, ref.shape[-1])
    assert np.isfinite(got).all(), "non-finite values in the GPU result"
    num = np.abs(got - ref).max(axis=1)
    den = np.abs(ref).max(axis=1)
    zero = den == 0
    assert (num[zero] == 0).all()
    return float((num[~zero] / den[~zero]).max()) if (~zero).any() else 0.0


def sample_rows(case, n, seed=0, H=64):
    """n distinct (b,h) pairs, always including the first and last sequence and the longest one."""
    rng = np.random.default_rng(seed)
    B = case.B
    rows = {(0, 0), (B - 1, H - 1), (int(case.seq_lens.argmax()), 17), (int(case.seq_lens.argmin()), 40)}
    while len(rows) < n:
        rows.add((int(rng.integers(B)), int(rng.integers(H))))
    return sorted(rows)
