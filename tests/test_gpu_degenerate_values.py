"""Degenerate operand values, HIP path vs the CPU oracle and vs closed forms: all-zero
queries and keys (uniform attention inside each group), all-zero everything, and strongly
peaked softmax rows (large logits), in both precisions and on aligned and unaligned groups."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu

# (dtype, B, N, H, Hkv, D, G)
FEW_ROWS = [
    ("f32", 1, 300, 4, 2, 64, 100),
    ("bf16", 1, 1024, 4, 2, 128, 256),
    ("bf16", 1, 600, 4, 4, 128, 200),      # tiles that are not full
]
MANY_ROWS = [
    ("f32", 1, 3300, 4, 2, 64, 100),
    ("bf16", 1, 2304, 4, 2, 128, 256),     # tile-aligned kernels
    ("bf16", 1, 2000, 4, 4, 128, 200),     # partial tiles
    ("bf16", 1, 6144, 2, 2, 128, 2048),    # eight-wave forward
]
CASES = FEW_ROWS + MANY_ROWS


def test_which_kernels_the_cases_reach():
    from gpu_util import beyond_few_rows
    assert all(beyond_few_rows(B, N, H, G, dtype) == (case in MANY_ROWS) for case in CASES for dtype, B, N, H, _, _, G in [case])


def scaled_inputs(dtype, B, N, H, Hkv, D, seed, **factor):
    """Seeded inputs with whole tensors multiplied by a power of two (exact in bf16)."""
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=seed, dtype=dtype)
    for name, f in factor.items():
        inp[name] = (inp[name] * np.float32(f)).astype(np.float32)
        if dtype == "bf16":
            inp[name + "_bits"] = inputs.round_to_bf16_bits(inp[name])
            assert np.array_equal(inputs.bf16_bits_to_f32(inp[name + "_bits"]), inp[name])
    return inp


def compare(dtype, out, ref):
    if dtype == "f32":
        from test_gpu_parity_f32 import compare as cmp
    else:
        from test_gpu_parity_bf16 import compare as cmp
    return cmp(out, ref)


def visible_counts(N, G, H, shift):
    """Number of keys each token attends to, per head, for the default pattern with the
    wrap group kept whole (position p of a group sees p + 1 keys)."""
    cnt = np.empty((H, N), dtype=np.float64)
    t = np.arange(N)
    for h in range(H):
        s = shift if h >= H // 2 else 0
        cnt[h] = ((t - s) % N) % G + 1
    return cnt


@pytest.mark.parametrize("case", CASES)
def test_zero_queries_and_keys_give_uniform_attention(case):
    from gpu_util import run_hip
    dtype, B, N, H, Hkv, D, G = case
    inp = scaled_inputs(dtype, B, N, H, Hkv, D, seed=900, q=0.0, k=0.0)
    out = run_hip(inp, G, dtype)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G)
    compare(dtype, out, ref)
    # closed form: every visible key has weight 1/count, so lse = log(count)
    want = np.log(visible_counts(N, G, H, G // 2))
    assert np.abs(out["lse"][0] - want).max() <= 2e-5
    # the scores do not depend on q or k, but dS is not zero: dq = scale * dS K = 0 (K = 0), dk = 0 (Q = 0)
    assert not out["dq"].any() and not out["dk"].any()
    assert np.abs(out["dv"]).max() > 0


@pytest.mark.parametrize("case", CASES)
def test_all_zero_operands_give_zeros(case):
    from gpu_util import run_hip
    dtype, B, N, H, Hkv, D, G = case
    inp = scaled_inputs(dtype, B, N, H, Hkv, D, seed=901, q=0.0, k=0.0, v=0.0, do=0.0)
    out = run_hip(inp, G, dtype)
    for name in ("o", "dq", "dk", "dv"):
        assert not out[name].any(), name
    assert np.abs(out["lse"][0] - np.log(visible_counts(N, G, H, G // 2))).max() <= 2e-5


@pytest.mark.parametrize("case", CASES)
def test_peaked_softmax_rows(case):
    """q and k four times larger: logits of standard deviation 16, so most rows put nearly
    all their weight on one key and exp() of the raw scores would overflow.

    v is made eight times smaller.  On a peaked row dS = P * (dP - delta) is a difference of
    two nearly equal numbers, and the backward pass forms delta from the output it is handed,
    which in bf16 mode carries that format's rounding (the oracle's delta does not); the
    resulting error of dq and dk is proportional to |K| |V| resp. |Q| |V|, which this choice
    keeps at or below its usual size, so the usual tolerances apply unchanged."""
    from gpu_util import run_hip
    dtype, B, N, H, Hkv, D, G = case
    inp = scaled_inputs(dtype, B, N, H, Hkv, D, seed=902, q=4.0, k=4.0, v=0.125)
    out = run_hip(inp, G, dtype)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G)
    assert np.abs(ref[1]).max() > 40.0          # the case is what it claims: lse far above exp's comfort
    if dtype == "f32":
        compare(dtype, out, ref)
        return
    # bf16: the usual bound (2e-2 plus the rounding of the stored output) plus 2^-8 |ref| for the
    # bf16 rounding of the P and dS operands: entries of P near 1 each err by up to 2^-9, and so
    # do the matching dS entries, with nothing to average over when one query dominates a key's
    # column (on N(0,1) operands thousands of small entries share a column and this term vanishes)
    from gpu_util import bf16_tol
    o, lse, dq, dk, dv = ref
    assert np.abs(out["lse"] - lse).max() <= 2e-3
    for name, r in (("o", o), ("dq", dq), ("dk", dk), ("dv", dv)):
        err = np.abs(out[name].astype(np.float64) - r)
        tol = bf16_tol(r) + 2.0 ** -8 * np.abs(r)
        assert np.all(np.isfinite(out[name])) and np.all(err <= tol), (name, float(err.max()), float((err / tol).max()))
