"""dK/dV with the query heads of a kv head cut into parts (fp32 partial sums, combined): parts
of several heads and of one, a kv head that serves shifted and unshifted heads with the class
boundary in the middle and off it, aligned, partial-tile, D = 64 and fp32 kernels, and a
workspace with room for the fewest parts only.  Bounds: those of the parity tests."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, (B, N, H, Hkv, D, G), parts wanted (2 * parts * B * N * Hkv * D floats beyond the row terms)
    ("bf16", (1, 2048, 8, 1, 128, 1024), 8),      # MQA, both classes: one head each
    ("bf16", (1, 1536, 12, 1, 128, 768), 6),      # two heads each
    ("bf16", (1, 2048, 8, 2, 128, 1024), 4),      # no shared kv head: cut for the chip's sake only
    ("bf16", (2, 1024, 12, 3, 128, 512), 2),      # the middle kv head serves both classes
    ("bf16", (1, 2000, 8, 1, 128, 1000), 4),      # partial tiles
    ("bf16", (1, 2048, 8, 1, 64, 1024), 8),       # head dimension 64
    ("f32", (1, 512, 8, 1, 64, 256), 8),
    ("f32", (1, 600, 6, 1, 128, 300), 6),
]


@pytest.mark.parametrize("dtype,shape,parts", CASES)
@pytest.mark.parametrize("least", [False, True])
def test_parts(dtype, shape, parts, least):
    from gpu_util import run_hip
    from paper_2309_12307_amd import binding
    from test_gpu_parity_bf16 import compare as compare_bf16
    from test_gpu_parity_f32 import compare as compare_f32
    B, N, H, Hkv, D, G = shape
    rows = 2 * ((B * H * N * 4 + 255) // 256 * 256)     # delta and lse * log2(e)
    wanted = binding.bwd_workspace_bytes(B, N, H, Hkv, D, G, binding.BF16 if dtype == "bf16" else binding.F32)
    assert wanted == rows + 2 * parts * B * N * Hkv * D * 4
    mixed = (H // 2) % (H // Hkv) != 0
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=600 + sum(shape), dtype=dtype)
    ws = rows + (4 * B * N * Hkv * D * 4 if mixed else 0) if least else None
    out = run_hip(inp, G, dtype, ws_bytes=ws)
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, dtype=np.float64)
    (compare_bf16 if dtype == "bf16" else compare_f32)(out, ref)


@pytest.mark.parametrize("dtype,shape,room,parts", [("bf16", (1, 2048, 8, 1, 128, 1024), 7, 4),
                                                    ("bf16", (1, 1536, 12, 1, 128, 768), 5, 4),
                                                    ("f32", (1, 512, 8, 1, 64, 256), 4, 4)])
def test_a_workspace_between_the_least_and_the_wanted(dtype, shape, room, parts):
    """Room for some of the parts: the largest number of them that divides the query heads and fits, with
    the partials ending where the workspace of that many ends."""
    from gpu_util import run_hip
    from paper_2309_12307_amd import binding
    from test_gpu_parity_bf16 import compare as compare_bf16
    from test_gpu_parity_f32 import compare as compare_f32
    B, N, H, Hkv, D, G = shape
    rows = 2 * ((B * H * N * 4 + 255) // 256 * 256)
    each = 2 * B * N * Hkv * D * 4
    assert binding.bwd_workspace_bytes(B, N, H, Hkv, D, G, binding.BF16 if dtype == "bf16" else binding.F32) > rows + room * each
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=620 + N, dtype=dtype)
    out = run_hip(inp, G, dtype, ws_bytes=rows + room * each)
    exact = run_hip(inp, G, dtype, ws_bytes=rows + parts * each)
    for name in ("dq", "dk", "dv"):
        assert np.array_equal(out[name], exact[name]), name
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, dtype=np.float64)
    (compare_bf16 if dtype == "bf16" else compare_f32)(out, ref)


def test_static_scratch_with_room_for_fewer_parts():
    """The library's own scratch holds two parts where the workspace query asks for more: dk and dv add up
    in another order, within the bounds."""
    import torch
    from gpu_util import run_hip, to_dev, to_np
    from paper_2309_12307_amd import binding
    from test_gpu_parity_bf16 import compare
    B, N, H, Hkv, D, G = 1, 4096, 8, 1, 128, 1024
    assert binding.bwd_workspace_bytes(B, N, H, Hkv, D, G) > binding.STATIC_SCRATCH_BYTES
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=630, dtype="bf16")
    q, k, v, do = (to_dev(inp[n], inp[n + "_bits"]) for n in ("q", "k", "v", "do"))
    o, dq, dk, dv = (torch.full_like(t, float("nan")) for t in (q, q, k, v))
    lse = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    binding.s2attn_fwd(q, k, v, o, lse, G)
    binding.s2attn_bwd_ex_static(binding.make_params(q, k, v, o, lse, G, dout=do, dq=dq, dk=dk, dv=dv))
    torch.cuda.synchronize()
    out = {n: to_np(t) for n, t in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv))}
    compare(out, orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G))
    assert np.array_equal(out["dq"], run_hip(inp, G, "bf16")["dq"])     # dq does not depend on the parts


def test_class_boundary_off_the_middle_of_a_kv_head():
    """A shard whose first kv head has two unshifted and six shifted query heads."""
    from gpu_util import run_hip
    from test_gpu_parity_bf16 import compare
    B, N, H, Hkv, D, G = 1, 2048, 16, 2, 128, 1024
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=611, dtype="bf16")
    out = run_hip(inp, G, "bf16", heads_total=36, head_offset=16)
    halves = [orc.s2attn_fwd_bwd(inp["q"][:, :, a:b], np.repeat(inp["k"], 8, axis=2)[:, :, a:b],
                                 np.repeat(inp["v"], 8, axis=2)[:, :, a:b], inp["do"][:, :, a:b], G, shift_heads=name)
              for a, b, name in ((0, 2, "none"), (2, 16, "all"))]
    o, dq, dk, dv = (np.concatenate([x[i] for x in halves], axis=2) for i in (0, 2, 3, 4))
    lse = np.concatenate([x[1] for x in halves], axis=1)
    dk, dv = (x.reshape(B, N, Hkv, 8, D).sum(axis=3) for x in (dk, dv))
    compare(out, (o, lse, dq, dk, dv))
