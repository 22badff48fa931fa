"""bf16 forward where the scores of a row change by orders of magnitude from tile to tile: the running maximum
rises many times, or never again, and keys of the lowest finite numbers come first.  The three forward kernels of D = 128
against fp64 on the GPU.  Bounds: o 2e-2 plus the rounding to bf16 (a weighted mean of v), lse 2e-3 plus what
fp32 scores of its size are off by (2^-20 of the largest)."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,G", [(8192, 4, 2048), (8192, 8, 1024), (1024, 4, 1024)])   # eight waves, four, few rows
@pytest.mark.parametrize("kind", ["rising", "falling", "steps", "low"])
@pytest.mark.parametrize("scale", [0.0, 1.5])
def test_scores_that_grow(N, H, G, kind, scale):
    import torch
    from paper_2309_12307_amd import binding
    D, n_low = 128, 40
    gen = torch.Generator(device="cuda").manual_seed(N + G)
    q, k, v = (torch.randn((1, N, H, D), generator=gen, device="cuda") for _ in range(3))
    pos = torch.arange(N, device="cuda") % G
    x = pos / G
    factor = {"rising": 0.05 + 8 * x * x, "falling": 8 * (1 - x) ** 4, "steps": 2.0 ** (pos // 128 % 6 - 2.0), "low": torch.ones_like(x)}[kind]
    k = k * factor[None, :, None, None]
    if kind == "low":
        q[..., 0] = q[..., 0].abs() + 0.5
        k[:, pos < n_low, :, 0] = -3e38
    q, k, v = (t.bfloat16() for t in (q, k, v))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, H, N), float("nan"), device="cuda")
    binding.s2attn_fwd_ex(binding.make_params(q, k, v, o, lse, G, shift_rule=binding.SHIFT_NONE, scale=scale))
    lo = n_low if kind == "low" else 0     # these rows and these keys only
    causal = torch.ones(G - lo, G - lo, dtype=torch.bool, device="cuda").tril()
    for h in range(H):
        for g in range(N // G):
            at = slice(g * G + lo, (g + 1) * G)
            s = q[0, at, h].double() @ k[0, at, h].double().T * (scale or 1 / math.sqrt(D))
            s = s.masked_fill(~causal, -math.inf)
            ref = torch.softmax(s, 1) @ v[0, at, h].double()
            err = (o[0, at, h].double() - ref).abs()
            assert torch.isfinite(o[0, at, h]).all() and (err <= 2e-2 + ref.abs() * 2.0 ** -8).all(), float(err.max())
            want = torch.logsumexp(s, 1)
            assert ((lse[0, h, at].double() - want).abs() <= 2e-3 + want.abs() * 2.0 ** -20).all()


@pytest.mark.parametrize("factor", [4.0, 16.0])
def test_peaked_rows_are_as_exact_as_with_the_four_wave_kernel(factor):
    """Few keys carry a row, and its largest probability is exactly 1 if the running maximum was raised for it: O of
    the eight-wave kernel is no further from 64 bits than that of the four-wave kernel, which a shift that no head
    uses and 64 does not divide selects.  (2 %: the same roundings, in sums of another order.)"""
    import torch
    from paper_2309_12307_amd import binding
    N, H, G, D = 12288, 4, 2048, 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, N, H, D), generator=gen, device="cuda") for _ in range(3))
    q, k, v = (q * factor).bfloat16(), k.bfloat16(), v.bfloat16()
    causal = torch.ones(G, G, dtype=torch.bool, device="cuda").tril()
    ref = torch.empty(1, N, H, D, dtype=torch.float64, device="cuda")
    for h in range(H):
        for at in (slice(g, g + G) for g in range(0, N, G)):
            s = (q[0, at, h].double() @ k[0, at, h].double().T / math.sqrt(D)).masked_fill(~causal, -math.inf)
            ref[0, at, h] = torch.softmax(s, 1) @ v[0, at, h].double()
    err = []
    for shift in (0, 1):
        o, lse = torch.empty_like(q), torch.empty((1, H, N), device="cuda")
        binding.s2attn_fwd_ex(binding.make_params(q, k, v, o, lse, G, shift_rule=binding.SHIFT_NONE, shift=shift))
        err.append((o.double() - ref).norm().item())
    assert err[0] <= 1.02 * err[1], err
