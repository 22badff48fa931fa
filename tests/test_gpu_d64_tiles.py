"""Head dimension 64 at the edges of its tiles (32 rows a wave, 64 a staged tile, 128 a workgroup):
group sizes one step below, at and above each, with the wrap point of the roll at a tile's edge and
inside one, and the wrap-around group cut at its seam, against the oracle.  Bounds: those of the
parity tests."""
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [2, 30, 32, 34, 62, 64, 66, 126, 128, 130, 190, 192, 194, 256, 258, 322])
@pytest.mark.parametrize("shift", ["half", "odd", "tile"])
def test_group_sizes_around_the_tiles(G, shift):
    from gpu_util import run_hip
    from test_gpu_parity_bf16 import compare
    B, N, H, Hkv, D = 1, 3 * G, 4, 2, 64
    s = {"half": G // 2, "odd": G // 2 + 1, "tile": 64}[shift]
    if s >= G:
        pytest.skip("the shift is smaller than the group")
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=900 + G + s, dtype="bf16")
    for split in (False, True):
        out = run_hip(inp, G, "bf16", shift=s, wrap_variant=2 if split else 0)
        ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, shift=s, variant2=split)
        compare(out, ref)
