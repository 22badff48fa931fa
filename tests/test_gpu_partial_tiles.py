"""Head dimension 128, runs that no tile divides: dK/dV (64 query rows a tile, 128 keys a workgroup)
at group sizes one step below, at and above each edge, and all kernels at the group sizes around 2048 where
larger grids take the eight-wave forward, with the wrap point of the roll at a tile's edge and
inside one, and the wrap-around group cut at its seam, against the oracle.  Bounds: those of the
parity tests."""
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


def check(G, groups, shift, split, many=False):
    from bf16_rounding_model import compare_or_model
    from gpu_util import run_hip
    from test_gpu_parity_bf16 import compare
    inp = inputs.make_inputs(1, groups * G, 4, 2, 128, seed=700 + G + shift, dtype="bf16")
    out = run_hip(inp, G, "bf16", shift=shift, wrap_variant=2 if split else 0)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, shift=shift, variant2=split)
    if many:
        compare_or_model(out, inp, ref, G, shift, "second_half", split)
    else:
        compare(out, ref)


@pytest.mark.parametrize("G", [2, 62, 64, 66, 126, 128, 130, 190, 192, 194, 258, 322])
@pytest.mark.parametrize("shift", ["half", "odd", "tile"])
def test_dkdv_group_sizes_around_the_tiles(G, shift):
    """The fewest groups that are beyond the kernels for few rows: up to 65 of them, and so more first keys of a run than
    in the parity tests; bounds of the random sweep."""
    from gpu_util import beyond_few_rows
    s = {"half": G // 2, "odd": G // 2 + 1, "tile": 64}[shift]
    if s >= G:
        pytest.skip("the shift is smaller than the group")
    groups = 256 // (4 * -(-G // 32)) + 1
    assert beyond_few_rows(1, groups * G, 4, G, "bf16")
    for split in (False, True):
        check(G, groups, s, split, many=True)


@pytest.mark.parametrize("G", [2046, 2048, 2050, 2078, 2082, 2110, 2112, 2114, 2176, 2302, 2306])
@pytest.mark.parametrize("shift,split", [("half", False), ("odd", False), ("odd", True), (128, True)])
def test_group_sizes_from_2048_on(G, shift, split):
    check(G, 2, {"half": G // 2, "odd": G // 2 + 1}.get(shift, shift), split)
