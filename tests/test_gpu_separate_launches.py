"""dK/dV and dQ launched one by one on small problems: grids just beyond those that share a launch, so that
the kernels of the large layers meet partial tiles, a wrap-around group cut at its seam, odd shifts, views
of a packed projection, grouped heads, a kv head of both classes and heads cut into parts (the shared
launch, which small problems otherwise take, is compiled from the same parts with other wave counts and
launch bounds).  Against the oracle, bounds of the random sweep."""
import math

import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    # (B, N, H, Hkv, D, G), shift, variant2, packed
    ((2, 40 * 322, 8, 2, 128, 322), None, False, False),
    ((2, 40 * 322, 8, 2, 128, 322), 161, True, False),       # two runs of 161 rows
    ((1, 37 * 322, 12, 3, 128, 322), 65, True, False),       # the middle kv head serves both classes: two parts
    ((2, 20 * 322, 8, 8, 128, 322), 7, False, True),
    ((1, 37 * 322, 16, 4, 128, 322), None, True, True),
    ((1, 8 * 642, 64, 1, 128, 642), None, False, False),     # eight parts
    ((1, 8 * 640, 64, 1, 128, 640), 321, True, True),
    ((1, 8 * 640, 64, 1, 128, 640), None, False, False),     # aligned, eight parts
    ((2, 41 * 256, 16, 16, 64, 256), None, False, False),    # interior query tiles of the D = 64 dK/dV
    ((2, 41 * 256, 16, 16, 64, 256), 129, True, True),
    ((2, 43 * 322, 16, 4, 64, 322), None, False, False),
    ((2, 43 * 322, 16, 4, 64, 322), 161, True, False),
    ((1, 45 * 512, 32, 1, 64, 512), None, False, False),     # parts
    ((1, 46 * 322, 36, 3, 64, 322), 65, True, True),         # a kv head of both classes
]


@pytest.mark.parametrize("shape,shift,variant2,packed", CASES)
def test_grids_beyond_one_launch(shape, shift, variant2, packed):
    from bf16_rounding_model import compare_or_model
    from gpu_util import run_hip, run_hip_packed
    from paper_2309_12307_amd import binding
    B, N, H, Hkv, D, G = shape
    partials = binding.bwd_workspace_bytes(B, N, H, Hkv, D, G) - 2 * ((B * H * N * 4 + 255) // 256 * 256)
    parts = max(1, partials // (2 * B * N * Hkv * D * 4))
    # one launch takes up to 1536 workgroups (5120)
    assert B * (N // G) * (Hkv * parts * -(-G // 128) + H * -(-G // (256 if D == 128 else 128))) > (1536 if D == 128 else 5120)
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=1100 + N + H + (shift or 0), dtype="bf16")
    # do smaller by the root of the heads that share a kv head (as a power of two, exact in bf16): dk and dv,
    # sums over them, and the roundings in them are then of the size that the bound is stated for
    small = 2.0 ** -round(math.log2(H // Hkv) / 2)
    inp["do"] = inp["do"] * np.float32(small)
    inp["do_bits"] = inputs.round_to_bf16_bits(inp["do"])
    kw = dict(wrap_variant=2 if variant2 else 0, shift=-1 if shift is None else shift)
    out = (run_hip_packed if packed else run_hip)(inp, G, "bf16", **kw)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, shift=shift, variant2=variant2)
    compare_or_model(out, inp, ref, G, shift, "second_half", variant2)
