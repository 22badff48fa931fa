"""fp32 kernels at the edges of their tiles (16 rows a wave, 32 a staged tile, 64 a workgroup):
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
def test_group_sizes_around_the_tiles(G, D):
    from gpu_util import max_abs, run_hip
    B, N, H, Hkv = 1, 3 * G, 4, 2
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=500 + G + D, dtype="f32")
    for kw, okw in ((dict(), dict()), (dict(wrap_variant=2, shift=G // 2 + 1), dict(variant2=True, shift=G // 2 + 1))):
        if kw and G // 2 + 1 >= G:
            continue
        out = run_hip(inp, G, "f32", **kw)
        ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, **okw)
        for name, r in zip(("o", "lse", "dq", "dk", "dv"), ref):
            assert np.all(np.isfinite(out[name])) and max_abs(out[name], r) <= 1e-4, (name, kw)
