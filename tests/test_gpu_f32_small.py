"""fp32: the kernels for few rows (16 rows to a workgroup, its four waves on different tiles) and the
lines between them and those of 64 rows to a workgroup, against the oracle.  Bound: the 1e-4 max-abs of
the fp32 mode (products and sums are fp32; the order of the sums differs between the two)."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


def check(B, N, H, Hkv, D, G, okw=None, **kw):
    from gpu_util import max_abs, run_hip
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=N + G + D, dtype="f32")
    out = run_hip(inp, G, "f32", **kw)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, **(okw or {}))
    for name, r in zip(("o", "lse", "dq", "dk", "dv"), ref):
        assert np.all(np.isfinite(out[name])) and max_abs(out[name], r) <= 1e-4, name


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,N,H,Hkv,G", [
    (1, 512, 2, 2, 512),       # one long chain per workgroup
    (2, 300, 4, 1, 100),       # heads of both classes on one kv head: partial sums; two batches
    (1, 288, 6, 2, 72),        # three query heads per kv head, tiles of 16 not filled
    (1, 80, 4, 4, 16), (1, 90, 4, 2, 18),   # one tile a group, one and a rest
])
def test_few_rows(B, N, H, Hkv, G, D):
    check(B, N, H, Hkv, D, G)
    check(B, N, H, Hkv, D, G, dict(variant2=True, shift=G // 2 - 1), wrap_variant=2, shift=G // 2 - 1)


# (forward line, backward line): workgroups of 64 rows on and one step above it
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,N,H,Hkv,G", [
    (1, 1024, 4, 4, 64), (1, 1088, 4, 4, 64),       # forward 64 | 68
    (1, 512, 4, 4, 64), (1, 576, 4, 4, 64),         # backward 32 | 36
    (1, 2048, 8, 8, 128), (1, 2176, 8, 8, 128),     # forward 256 | 272
    (1, 2048, 4, 4, 256), (1, 2304, 4, 4, 256),     # two sizes beyond the backward's
    (1, 1536, 4, 4, 256), (1, 1792, 4, 4, 256),     # backward 96 | 112
    (1, 1920, 4, 4, 320), (1, 2240, 4, 4, 320),     # backward 120 | 140
    (1, 3072, 4, 4, 128), (1, 3328, 4, 4, 128),     # forward, D = 128: 12 | 13 sequences of an XCD, 96 | 104 workgroups of 16 rows
    (1, 1024, 8, 2, 128), (1, 1152, 8, 2, 128),     # the same, four query heads per kv head
    (1, 8000, 2, 2, 1000), (1, 9000, 2, 2, 1000),   # both 256 | 288
    (1, 2048, 2, 2, 2048), (1, 2080, 2, 2, 2080),   # backward, one group: 32 | 33 workgroups of an XCD
])
def test_on_the_lines(B, N, H, Hkv, G, D):
    check(B, N, H, Hkv, D, G)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [2, 14, 18, 30, 34, 62, 66, 130])
def test_many_rows_at_the_edges_of_tiles(G, D):
    """The kernels of 64 rows to a workgroup at partial tiles (small N goes to the others)."""
    groups = 34 if G <= 64 else 18
    check(1, groups * G, 8, 4, D, G)
    check(1, groups * G, 8, 4, D, G, dict(variant2=True, shift=G // 2), wrap_variant=2, shift=G // 2)
