"""Sums over tokens keep their bits: tokens that are all alike, so that the sum of their
terms is known exactly and a long chain of 32-bit additions would show."""
import pytest

pytestmark = pytest.mark.gpu

# (dtype, d): both bf16 tilings with few tokens, the exact forms, the fp32 kernels
FORMS = [("bf16", 256), ("bf16", 1024), ("bf16", 2048), ("bf16", 2560), ("bf16", 48), ("bf16", 72), ("bf16", 640),
         ("bf16", 1160), ("bf16", 1800), ("bf16", 3080), ("f32", 24), ("f32", 264), ("f32", 2056)]


def _inputs(K, T, d, V, dtype, seed=5):
    import torch

    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(seed)
    row = torch.randn(d, generator=g, device="cuda").to(dt)
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).to(dt)
    h = row.expand(K, T, d).contiguous()
    return h, torch.ones(d, dtype=dt, device="cuda"), W, torch.full((K, T), 3, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("dtype,d", FORMS, ids=[f"{a}-{b}" for a, b in FORMS])
def test_gain_gradient(dtype, d):
    """64 equal terms x in module 0, 8 in module 1 (its other rows are zero, and so are their
    terms): sums of 8 x and 64 x by doubling or in 64 bits are exact, a chain x, 2 x, 3 x, .. is not."""
    import torch

    from paper_2609_35440_amd import binding

    h, gain, W, y = _inputs(2, 64, d, 4001, dtype)
    h[1, 8:] = 0
    r = binding.readout_general(h, gain.repeat(2, 1), W, y)
    assert torch.isfinite(r.dgain).all() and float(r.dgain.abs().max()) > 0
    assert torch.equal(r.dgain[0], 8 * r.dgain[1])
