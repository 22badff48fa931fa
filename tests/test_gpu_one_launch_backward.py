"""dK/dV and dQ in one launch (few workgroups) and one by one: group sizes at the edges of the 256-row
dQ tile, dK/dV first and dQ first (one or several query heads to a kv head), the largest grid that
takes one launch (1536 workgroups of 512 threads; fewer where groups are short) and the next one, against
the oracle.  Bounds: those of the random sweep."""
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
    from bf16_rounding_model import compare_or_model
    inp, out, ref = run(*shape, **kw)
    compare_or_model(out, inp, ref, shape[4])


@pytest.mark.parametrize("Hkv", [4, 1])
@pytest.mark.parametrize("G", [128, 254, 256, 258, 384, 512, 514, 640])
@pytest.mark.parametrize("split", [False, True])
def test_group_sizes_around_the_dq_tile(G, Hkv, split):
    """The fewest groups that are beyond the kernels for few rows: 1.7 workgroups to a CU at most, one launch."""
    from bf16_rounding_model import compare_or_model
    from gpu_util import beyond_few_rows
    groups = 256 // (4 * -(-G // 32)) + 1
    assert beyond_few_rows(1, groups * G, 4, G, "bf16")
    parts = 4 if Hkv == 1 else 1
    assert groups * (Hkv * parts * (-(-G // 128) + split) + 4 * (-(-G // 256) + split)) <= 440
    inp, out, ref = run(1, groups * G, 4, Hkv, G, **(dict(wrap_variant=2) if split else {}))
    compare_or_model(out, inp, ref, G, None, "second_half", split)


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
