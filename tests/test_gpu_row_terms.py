"""The pass that forms the row terms of the bf16 backward (two heads and 32 or 64 tokens a workgroup; one
head and twice the tokens where the number of heads is odd): token counts one step below, at and above
its tiles, two sequences and more, even and odd numbers of heads (a shard), against the oracle.  Bounds: those of
the random sweep."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("H", [1, 2, 3, 6])
@pytest.mark.parametrize("N", [2, 30, 32, 34, 62, 64, 66, 126, 128, 130])
def test_token_counts_around_the_tiles(N, H, D):
    from bf16_rounding_model import compare_or_model
    from gpu_util import beyond_few_rows, run_hip
    # D = 128: the fewest sequences beyond the kernels for few rows, which form the row terms themselves
    B = 2 if D == 64 else 256 // (H * -(-N // 32)) + 1
    assert D == 64 or beyond_few_rows(B, N, H, N, "bf16")
    layer = inputs.make_inputs(B, N, H + H % 2, H + H % 2, D, seed=1000 + N + H, dtype="bf16")
    inp = {n: np.ascontiguousarray(x[:, :, :H]) for n, x in layer.items()}
    out = run_hip(inp, N, "bf16", shift_rule=1, **(dict(heads_total=H + 1) if H % 2 else {}))
    o, lse, dq, dk, dv = orc.s2attn_fwd_bwd(layer["q"], layer["k"], layer["v"], layer["do"], N, shift_heads="none",
                                            dtype=np.float64)
    compare_or_model(out, inp, (o[:, :, :H], lse[:, :H], dq[:, :, :H], dk[:, :, :H], dv[:, :, :H]), N, None, "none")
