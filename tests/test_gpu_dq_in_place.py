"""dq stored over q, o or dout (the tensor is no longer needed once its gradient is there): the sizes
are those whose dK/dV and dQ otherwise share a launch, where dK/dV would read rows that dQ has
already replaced.  Against the oracle, bounds of the parity tests."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("Hkv,G", [(8, 512), (2, 250)])
@pytest.mark.parametrize("over", ["q", "o", "do"])
@pytest.mark.parametrize("static", [False, True])
def test_dq_over_an_input(dtype, D, Hkv, G, over, static):
    import torch
    from gpu_util import to_dev, to_np
    from paper_2309_12307_amd import binding
    from test_gpu_parity_bf16 import compare as compare_bf16
    from test_gpu_parity_f32 import compare as compare_f32
    B, N, H = 1, 4 * G, 8
    bf = dtype == "bf16"
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=400 + G + D, dtype=dtype)
    t = {n: to_dev(inp[n], inp.get(n + "_bits") if bf else None) for n in ("q", "k", "v", "do")}
    t["o"] = torch.full_like(t["q"], float("nan"))
    lse = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    binding.s2attn_fwd(t["q"], t["k"], t["v"], t["o"], lse, G)
    out = dict(o=to_np(t["o"]), lse=to_np(lse))
    dk, dv = torch.full_like(t["k"], float("nan")), torch.full_like(t["v"], float("nan"))
    kw = dict(dout=t["do"], dq=t[over], dk=dk, dv=dv)
    p = binding.make_params(t["q"], t["k"], t["v"], t["o"], lse, G, **kw)
    if static:
        binding.s2attn_bwd_ex_static(p)
    else:
        ws = torch.empty(binding.bwd_workspace_bytes_ex(p), dtype=torch.uint8, device="cuda")
        binding.s2attn_bwd_ex(binding.make_params(t["q"], t["k"], t["v"], t["o"], lse, G, workspace=ws, **kw))
    torch.cuda.synchronize()
    out.update(dq=to_np(t[over]), dk=to_np(dk), dv=to_np(dv))
    ref = orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, dtype=np.float64)
    (compare_bf16 if bf else compare_f32)(out, ref)
