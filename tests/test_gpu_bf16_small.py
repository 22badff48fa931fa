"""bf16, D = 128: the kernels for few rows (32 rows to a workgroup, its four waves on different tiles) and the
lines between them and the others, against the oracle with the element-wise bound of the bf16 mode."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


def check(B, N, H, Hkv, G, okw=None, **kw):
    from gpu_util import bf16_tol, max_abs, run_hip
    inp = inputs.make_inputs(B, N, H, Hkv, 128, seed=N + G, dtype="bf16")
    out = run_hip(inp, G, "bf16", **kw)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, **(okw or {}))
    for name, r in zip(("o", "lse", "dq", "dk", "dv"), ref):
        assert np.all(np.isfinite(out[name])), name
        if name == "lse":
            assert max_abs(out[name], r) <= 2e-3
        else:
            assert np.all(np.abs(out[name] - r) <= bf16_tol(r)), name


@pytest.mark.parametrize("B,N,H,Hkv,G", [
    (1, 64, 2, 2, 32), (1, 60, 2, 1, 30), (1, 68, 4, 2, 34),   # a tile a group, one below, one and a rest
    (1, 8, 2, 2, 2),                                           # the smallest group
    (1, 512, 2, 2, 512),                                       # four tiles a wave
    (2, 396, 6, 2, 132),                                       # tiles dealt unevenly, three heads per kv head
    (2, 300, 4, 1, 100),                                       # heads of both classes on one kv head: partial sums
])
def test_few_rows(B, N, H, Hkv, G):
    check(B, N, H, Hkv, G)
    s = max(1, G // 2 - 1)
    check(B, N, H, Hkv, G, dict(variant2=True, shift=s), wrap_variant=2, shift=s)


# workgroups of 32 rows on and one step above each line
@pytest.mark.parametrize("B,N,H,Hkv,G", [
    (1, 1024, 8, 4, 64), (1, 512, 8, 4, 64), (1, 576, 8, 4, 64),   # forward 256, backward 128 | 144
    (1, 1024, 8, 4, 128), (1, 1152, 8, 4, 128),     # both 256 | 288
    (1, 1280, 4, 4, 256), (1, 1536, 4, 4, 256),     # backward, one head per kv head 160 | 192
    (1, 512, 16, 16, 512), (1, 576, 16, 16, 576),   # the same, long chains 256 | 288
    (1, 1536, 2, 2, 1536), (1, 1664, 2, 2, 1664),   # backward, group size
    (1, 2048, 2, 2, 2048), (1, 2304, 2, 2, 2304),   # forward, group size
    (1, 960, 8, 4, 96), (1, 1056, 8, 4, 96),        # forward, 30 | 33 workgroups of an XCD
    (1, 480, 8, 8, 96), (1, 576, 8, 8, 96),         # backward, one head per kv head, 30 | 36 of both kernels
    (1, 576, 8, 8, 192), (1, 768, 8, 8, 192),       # the same, longer chains 36 | 48
    (1, 1280, 4, 4, 320), (1, 1600, 4, 4, 320),     # the same, ten workgroups to a sequence 40 | 60
    (1, 768, 8, 8, 768), (1, 1536, 6, 6, 768),      # the same, one sequence of an XCD | two
    (1, 960, 6, 3, 160), (1, 1120, 6, 3, 160),      # the same, a kv head of both classes 50 | 60
])
def test_on_the_lines(B, N, H, Hkv, G):
    check(B, N, H, Hkv, G)


@pytest.mark.parametrize("G", [2, 62, 64, 66, 126, 128, 130, 190, 194, 254, 256, 258, 322, 384, 512, 514])
@pytest.mark.parametrize("shift", ["half", "odd"])
@pytest.mark.parametrize("split", [False, True])
def test_many_rows_at_the_edges_of_tiles(G, shift, split):
    """The other kernels at the edges of their tiles of 64, 128 and 256 rows."""
    H = 8
    groups = 257 // (H * -(-G // 32)) + 1
    s = G // 2 + (shift == "odd" and G > 2)
    check(1, groups * G, H, 4, G, dict(shift=s, variant2=split), shift=s, wrap_variant=2 if split else 0)


@pytest.mark.parametrize("H", [66, 67])
@pytest.mark.parametrize("N", [2, 30, 34, 62, 66, 126, 130])
def test_row_terms_of_many_heads(N, H):
    """The pass that forms the row terms, at token counts around its tiles, even and odd numbers of heads."""
    from gpu_util import bf16_tol, run_hip
    layer = inputs.make_inputs(2, N, H + H % 2, H + H % 2, 128, seed=1300 + N + H, dtype="bf16")
    inp = {n: np.ascontiguousarray(x[:, :, :H]) for n, x in layer.items()}
    out = run_hip(inp, N, "bf16", shift_rule=1, **(dict(heads_total=H + 1) if H % 2 else {}))
    ref = orc.s2attn_fwd_bwd(layer["q"], layer["k"], layer["v"], layer["do"], N, shift_heads="none")
    for name, r in zip(("dq", "dk", "dv"), (ref[2], ref[3], ref[4])):
        assert np.all(np.abs(out[name] - r[:, :, :H]) <= bf16_tol(r[:, :, :H])), name
