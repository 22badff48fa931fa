"""dK/dV and dQ in one launch (few workgroups) and one by one: group sizes at the edges of the 256-row
dQ tile, dK/dV first and dQ first (one or several query heads to a kv head), the largest grid that
takes one launch (1536 workgroups of 512 threads; fewer where groups are short) and the next one, against
the oracle.  Bounds: those of the parity tests for the group sizes, those of the random sweep for the
larger tensors of the grids."""
import numpy as np
import pytest

from oracle import s2attn_oracle as orc
from paper_2309_12307_amd import inputs

pytestmark = pytest.mark.gpu


def run(B, N, H, Hkv, G, D=128, **kw):
    from gpu_util import run_hip
    inp = inputs.make_inputs(B, N, H, Hkv, D, seed=800 + N + H + Hkv, dtype="bf16")
    out = run_hip(inp, G, "bf16", **kw)
    return inp, out, orc.s2attn_fwd_bwd(inp["q"], inp["k"], inp["v"], inp["do"], G, variant2=bool(kw))


def check_grid(*shape, **kw):
    """Element by element 2e-2 and the rounding of the value to its bf16 output.  Up to 16 elements of a
    tensor may be beyond it (of 16.8 million of N(0,1) data in short groups a few are: P sits on few keys
    there and delta carries the rounding of single elements of o), if they are what the fp64 model of those
    roundings gives."""
    from bf16_rounding_model import bf16_backward_model, to_bf16
    from gpu_util import bf16_tol, check_bf16_tensor, half_ulp_bf16, max_abs
    inp, out, (o, lse, *grads) = run(*shape, **kw)
    assert max_abs(out["lse"], lse) <= 2e-3
    check_bf16_tensor("o", out["o"], o)
    model = None
    for i, (name, r) in enumerate(zip(("dq", "dk", "dv"), grads)):
        assert np.all(np.isfinite(out[name])), name
        over = np.abs(out[name].astype(np.float64) - r) > bf16_tol(r)
        if over.any():
            assert over.sum() <= 16, (name, int(over.sum()))
            if model is None:
                model = bf16_backward_model(inp["q"], inp["k"], inp["v"], inp["do"], shape[4], None, "second_half", False)
            m = model[i][over]
            assert np.all(np.abs(out[name][over] - to_bf16(m)) <= 6e-3 + 2 * half_ulp_bf16(m)), (name, np.argwhere(over))


@pytest.mark.parametrize("Hkv", [4, 1])
@pytest.mark.parametrize("G", [128, 254, 256, 258, 384, 512, 514, 640])
@pytest.mark.parametrize("split", [False, True])
def test_group_sizes_around_the_dq_tile(G, Hkv, split):
    from test_gpu_parity_bf16 import compare
    _, out, ref = run(1, 3 * G, 4, Hkv, G, **(dict(wrap_variant=2) if split else {}))
    compare(out, ref)


# 256 keys and 256 query rows a group: two workgroups of dK/dV and one of dQ per group and head
@pytest.mark.parametrize("groups", [16, 17])
def test_largest_grid_of_one_launch_and_the_next(groups):
    check_grid(4, 256 * groups, 8, 8, 256)


# groups of 128: a workgroup of dK/dV to each group and kv head (two parts where it serves both classes of
# heads), one of dQ to each group and head; 700 workgroups in one launch, 1100 with eight heads to a kv head
@pytest.mark.parametrize("Hkv,groups", [(2, 70), (2, 71), (1, 110), (1, 111)])
def test_largest_grid_of_one_launch_and_the_next_short_groups(Hkv, groups):
    check_grid(1, 128 * groups, 8, Hkv, 128)


# D = 64: one workgroup of each kernel per group and head, 5120 in one launch
@pytest.mark.parametrize("groups", [40, 41])
def test_largest_grid_of_one_launch_and_the_next_d64(groups):
    check_grid(4, 128 * groups, 16, 16, 128, D=64)
