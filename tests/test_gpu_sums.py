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


@pytest.mark.parametrize("T,V", [(4096, 600), (100, 40)], ids=["many", "few"])
@pytest.mark.parametrize("dtype,d", FORMS, ids=[f"{a}-{b}" for a, b in FORMS])
def test_bias_gradient(dtype, d, T, V):
    """T equal tokens: db_v = p_v (less one at the target), of the head (the bias-gradient
    pass) and, outside the bf16 families, of the terminal (the readout-gradient pass).  A chain of n equal terms in fp32
    is off by up to n 2^-25; what is allowed is the error of one p: its log-sum-exp, about
    9 + log2(8) in base 2, stored with 24 bits (2^-21 ln 2 at most), and the rounding and
    sums of logits below 1 in magnitude, 2^-24 each over up to d / 16 steps of one sum."""
    import torch

    from paper_2609_35440_amd import binding

    h, gain, W, y = _inputs(2, T, d, V, dtype)
    r = binding.readout_general(h, gain, W, y, want_dbias=True)
    z = (h[0, 0].double() * torch.rsqrt(h[0, 0].double().square().mean() + 1e-6)) @ W.double().t()
    p = torch.softmax(z, 0)
    p[3] -= 1.0
    tol = 2.0**-21 + (8 + d / 16) * 2.0**-24
    for k in range(1 if dtype == "bf16" and d % 256 == 0 else 2):
        err = ((r.dbias[k].double() - p) / p).abs().max()
        assert float(err) <= tol, (k, float(err), tol)


def _row_losses(op, dtype, d, T=1024, V=2001, bias=None):
    """The calls' row losses of 2 x T rows, and the same in 64 bits."""
    import torch

    from paper_2609_35440_amd import binding

    K = 2
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(6)
    h = torch.randn(K, T, d, generator=g, device="cuda").to(dt)
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).to(dt)
    y = torch.randint(0, V, (K, T), generator=g, device="cuda", dtype=torch.int32)
    gain = (1 + 0.1 * torch.randn(d, generator=g, device="cuda")).to(dt)
    b = 0.1 * torch.randn(K, V, generator=g, device="cuda") if bias else None
    if op == "train":
        got = binding.readout_general(h, gain, W, y, bias=b, row_loss=True).row_loss
    else:
        got = binding.exit_eval(h, gain, W, y, bias=b).row_loss
    n = h.double() * torch.rsqrt(h.double().square().mean(2, keepdim=True) + 1e-6)
    z = (n * gain.double()) @ W.double().t()
    if bias:
        z = z + b.double()[:, None, :]
    return got.double(), torch.logsumexp(z, 2) - z.gather(2, y.long()[..., None])[..., 0]


@pytest.mark.parametrize("op", ["train", "eval"])
@pytest.mark.parametrize("dtype,d", [("bf16", 48), ("bf16", 200), ("bf16", 640), ("bf16", 1800), ("f32", 264)],
                         ids=["bf16-48", "bf16-200", "bf16-640", "bf16-1800", "f32-264"])
def test_row_losses_are_not_biased(op, dtype, d):
    """Calls defined in fp32: a row loss near 8 rounds by at most 2.4e-7, the sums before it by
    as much, to either side.  The mean over 2048 rows is then within 5e-7 / sqrt(2048) = 1.1e-8
    of the truth, one standard error; ten are allowed (a logarithm that reads half a unit low
    is off by 3e-7)."""
    got, ref = _row_losses(op, dtype, d)
    assert abs(float((got - ref).mean())) <= 1.1e-7


@pytest.mark.parametrize("bias", [False, True], ids=["", "bias"])
@pytest.mark.parametrize("T,V", [(1024, 2001), (130, 120)], ids=["many", "few"])
@pytest.mark.parametrize("d", [200, 1496, 2040, 2552, 2568, 3080, 4096])
def test_row_losses_of_wide_rows(d, T, V, bias):
    """Exit evaluation of the bf16 widths defined in fp32.  The target's logit has a deviation of
    s = 0.02 sqrt(d); summed 16 products at a time in n steps its partial sums round by 2^-25
    (rms, about) of sqrt(k / n) s each, together sqrt(n / 2) 2^-25 s, with n = d / 16 up to d = 2560
    and 32 past it, where sixteen such pieces at most add to as much again.  The row's end rounds
    by 3e-7 at most.  (A chain of both planes was off by 9.3e-7 at d = 4096.)"""
    got, ref = _row_losses("eval", "bf16", d, T, V, bias)
    n = d / 16 if d <= 2560 else 2 * 32
    tol = 3e-7 + (n / 2) ** 0.5 * 2.0**-25 * 0.02 * d**0.5
    err = (got - ref).square().mean().sqrt()
    assert float(err) <= tol, (float(err), tol)


@pytest.mark.parametrize("bias", [False, True], ids=["", "bias"])
@pytest.mark.parametrize("d", [200, 504, 640, 904, 1160, 1528, 1800, 3080, 4096])
def test_gain_gradient_over_a_long_vocabulary(d, bias):
    """The exact forms, unsplit, over 2000 chunks of readout rows.  A term e n of dgain takes about
    six roundings of 2.5e-8 (rms) of itself; their signs and the terms' are random, so the sum is
    as close, 6e-8 of its norm.  (Accumulated chunk by chunk in the matrix instruction,
    which cuts instead of rounding, e was off by enough for 9e-8.)"""
    import torch

    from paper_2609_35440_amd import binding
    from tests.routes import route

    T, V = 16384, 32000
    assert route(False, 1, T, d, V)[0] == 1
    g = torch.Generator(device="cuda").manual_seed(8)
    h = torch.randn(1, T, d, generator=g, device="cuda").bfloat16()
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).bfloat16()
    y = torch.randint(0, V, (1, T), generator=g, device="cuda", dtype=torch.int32)
    gain = (1 + 0.1 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    b = 0.5 * torch.randn(1, V, generator=g, device="cuda") if bias else None
    got = binding.readout_general(h, gain, W, y, bias=b).dgain
    W8, b8 = W.double(), b.double() if bias else 0.0
    want = torch.zeros(d, dtype=torch.float64, device="cuda")
    for t in range(0, T, 2048):
        n = h[0, t:t + 2048].double()
        n = n * torch.rsqrt(n.square().mean(1, keepdim=True) + 1e-6)
        p = torch.softmax((n * gain.double()) @ W8.t() + b8, 1)
        p.scatter_add_(1, y[0, t:t + 2048].long()[:, None], torch.full((2048, 1), -1.0, dtype=torch.float64, device="cuda"))
        want += ((p @ W8) * n).sum(0) / T
    err = float((got.double() - want).norm() / want.norm())
    assert err <= 6e-8, err
