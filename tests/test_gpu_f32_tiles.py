"""fp32 kernels at the edges of their tiles (16 rows a wave, 32 a staged tile, 64 a workgroup; few rows: 16 a tile), on
grids that the kernels for few rows take and on the fewest groups beyond:
group sizes one step below, at and above each, the smallest group, several heads per kv head
and the wrap-around group cut off any tile boundary, against the oracle.  Bound: the 1e-4
max-abs of the fp32 mode (products and sums are fp32, so single elements err by some 1e-6)."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [2, 14, 16, 18, 30, 32, 34, 62, 64, 66, 126, 130, 322])
@pytest.mark.parametrize("few", [True, False])
def test_group_sizes_around_the_tiles(G, D, few):
    from gpu_util import beyond_few_rows, max_abs, run_hip
    B, H, Hkv = 1, 4, 2
    N = G * (3 if few else 256 // (H * -(-G // 64)) + 1)
    assert beyond_few_rows(B, N, H, G, "f32") != few
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=500 + G + D, dtype="f32")
    for kw, okw in ((dict(), dict()), (dict(wrap_variant=2, shift=G // 2 + 1), dict(variant2=True, shift=G // 2 + 1))):
        if kw and G // 2 + 1 >= G:
            continue
        out = run_hip(inp, G, "f32", **kw)
        ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, **okw)
        for name, r in zip(("o", "lse", "dq", "dk", "dv"), ref):
            assert np.all(np.isfinite(out[name])) and max_abs(out[name], r) <= 1e-4, (name, kw)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("low", [-np.inf, -3e38])
@pytest.mark.parametrize("n_low", [8, 32, 40])
@pytest.mark.parametrize("H", [2, 66])     # few rows (tiles of 16 keys), and the kernels beyond (32)
def test_first_scores_of_a_row_minus_infinity(D, low, n_low, H):
    """The first keys of every group score -inf (or the lowest finite numbers): rows that see any
    other key are softmax over the others, whether the low keys are part of their first tile,
    all of it, or reach into the second."""
    import torch
    from gpu_util import beyond_few_rows, to_dev, to_np
    from paper_2309_12307_amd import binding
    N, G = 256, 128
    assert beyond_few_rows(1, N, H, G, "f32") == (H > 2)
    rng = np.random.default_rng(77)
    q, k, v = (rng.standard_normal((1, N, H, D)).astype(np.float32) for _ in range(3))
    q[..., 0] = np.abs(q[..., 0]) + 0.5
    dead = np.arange(N) % G < n_low
    k[:, dead, :, 0] = low
    qt, kt, vt = (to_dev(x) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    binding.s2attn_fwd_ex(binding.make_params(qt, kt, vt, o, lse, G, shift_rule=binding.SHIFT_NONE))
    o, lse = to_np(o), to_np(lse)
    for g in range(N // G):
        rows = slice(g * G + n_low, (g + 1) * G)     # these rows and these keys only
        for h in range(H):
            s = q[0, rows, h].astype(np.float64) @ k[0, rows, h].astype(np.float64).T / np.sqrt(D)
            s = np.where(np.tril(np.ones_like(s)) > 0, s, -np.inf)
            m = s.max(axis=1, keepdims=True)
            e = np.exp(s - m)
            ref = e / e.sum(axis=1, keepdims=True) @ v[0, rows, h].astype(np.float64)
            assert np.abs(o[0, rows, h] - ref).max() <= 1e-4
            assert np.abs(lse[0, h, rows] - (m[:, 0] + np.log(e.sum(axis=1)))).max() <= 1e-4
