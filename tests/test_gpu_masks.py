"""Vocabulary entries masked by a bias of -inf or of the type's lowest value (times
log2 e it overflows to -inf): a padded tail, a leading block, and an allowed set in the
middle, so that whole chunks at the start of a call and at the start of the parts it is
split into hold no finite logit.  Every kernel form, against the oracle."""
import dataclasses

import numpy as np
import pytest

from solo_inputs import make_extras, make_inputs
from tests.routes import FUSED, PROD, SPLIT, route_of
from tests.test_gpu_general import check_exit_eval, compare, oracle_general, run_exit_eval, run_general

pytestmark = pytest.mark.gpu

LOW = {"inf": -np.inf, "lowest": np.finfo(np.float32).min}
# allowed columns as shares of the vocabulary
KEEP = {"head": (0.0, 0.45), "middle": (0.4, 0.6), "most": (0.2, 1.0), "tail": (0.7, 1.0)}


def masked(cfg, K, T, d, V, keep, low, **extras):
    """The inputs, and the same call over the allowed columns [lo, hi) alone."""
    x = make_extras(make_inputs(cfg, seed=31, K=K, T=T, d=d, V=V), seed=31, bias=True, **extras)
    lo, hi = (int(V * f) for f in KEEP[keep])
    x["targets"] = (lo + x["targets"].astype(np.int64) % (hi - lo)).astype(x["targets"].dtype)
    few = dict(x, W=x["W"][lo:hi], bias=x["bias"][:, lo:hi].copy(), targets=x["targets"] - np.int32(lo),
               cfg=dataclasses.replace(x["cfg"], V=hi - lo))
    if "W_bits" in x:
        few["W_bits"] = x["W_bits"][lo:hi]
    x["bias"][:, :lo] = LOW[low]
    x["bias"][:, hi:] = LOW[low]
    return x, few, lo, hi


def check(x, few, lo, hi, flags, what):
    g = run_general(x, flags)
    for name, axis in (("dW", 0), ("dbias", 1)):
        if g[name] is not None:  # a masked entry has no gradient at all
            out = np.delete(g[name], np.s_[lo:hi], axis=axis)
            assert not out.any(), (what, name)
            g[name] = g[name][lo:hi] if axis == 0 else g[name][:, lo:hi]
    compare(g, oracle_general(few, flags), x["cfg"].dtype, flags, what)


# (splits beyond one are asserted, so that parts start inside a mask)
# few tokens (split) of both bf16 tilings, the exact forms and the fp32 kernels; the last ones are not split
TRAIN = [("1b", 2, 40, 1024, 4001), ("1b", 3, 20, 2048, 3000), ("2b", 2, 20, 2560, 3001), ("1b", 2, 40, 640, 3001),
         ("1b", 2, 20, 1800, 2001), ("1b", 2, 40, 48, 3001), ("tiny", 2, 40, 264, 3001),
         ("1b", 1, 9, 640, 100), ("1b", 1, 9, 256, 100), ("2b", 1, 9, 2560, 100)]


@pytest.mark.parametrize("low", list(LOW))
@pytest.mark.parametrize("keep", list(KEEP))
@pytest.mark.parametrize("cfg,K,T,d,V", TRAIN, ids=["-".join(map(str, c)) for c in TRAIN])
def test_train(cfg, K, T, d, V, keep, low):
    m = masked(cfg, K, T, d, V, keep, low, tau=True)
    flags = dict(final_module_dW=True, want_dtau=True, want_dbias=True)
    assert (route_of(m[0], False, **flags)[0] > 4) == (V > 100)
    check(*m, flags, f"masked {keep} {low} d={d}")


@pytest.mark.parametrize("keep", list(KEEP))
def test_rot(keep):
    check(*masked("1b", 3, 30, 512, 4001, keep, "inf", rot=True), dict(final_module_dW=True), f"masked rot {keep}")


# the split form (few rows) of both bf16 tilings, the whole fused form, planes and fp32
EVAL = [("1b", 3, 30, 512, 8003), ("1b", 2, 16, 2048, 8000), ("2b", 2, 30, 2560, 8003), ("1b", 2, 9, 1024, 40),
        ("1b", 2, 300, 72, 4097), ("tiny", 2, 30, 64, 3001)]


@pytest.mark.parametrize("low", list(LOW))
@pytest.mark.parametrize("keep", list(KEEP))
@pytest.mark.parametrize("cfg,K,T,d,V", EVAL, ids=["-".join(map(str, c)) for c in EVAL])
def test_eval(cfg, K, T, d, V, keep, low):
    x, few, lo, hi = masked(cfg, K, T, d, V, keep, low)
    form = PROD if d == 72 else (SPLIT if cfg != "tiny" and V > 100 else FUSED)
    assert route_of(x, True)[0] == form
    losses, row_loss, top1 = run_exit_eval(x)
    check_exit_eval(few, losses, row_loss, top1 - lo, f"masked eval {keep} {low} d={d}", min_rows_for_agreement=100)


@pytest.mark.parametrize("dtype,T,d,V", [("bf16", 40, 48, 3001), ("bf16", 40, 640, 3001), ("bf16", 9, 640, 100),
                                         ("bf16", 20, 1800, 2001), ("bf16", 300, 72, 4097), ("bf16", 9, 3080, 600),
                                         ("f32", 40, 264, 3001)])
def test_lowest_value_everywhere_or_at_the_target(dtype, T, d, V):
    """Calls defined in fp32: the type's lowest value is finite, and so is the loss of a row whose
    every entry is masked by it (all alike: log V), or whose target is (the mask itself,
    short of what base 2 can hold)."""
    import torch

    from paper_2609_35440_amd import binding

    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(7)
    h = torch.randn(2, T, d, generator=g, device="cuda").to(dt)
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).to(dt)
    gain = torch.ones(d, dtype=dt, device="cuda")
    y = torch.full((2, T), V // 2, dtype=torch.int32, device="cuda")
    low = torch.finfo(torch.float32).min
    bias = torch.zeros(2, V, device="cuda")
    bias[0] = low
    bias[1, V // 2] = low
    for r in (binding.readout_general(h, gain, W, y, bias=bias, row_loss=True), binding.exit_eval(h, gain, W, y, bias=bias)):
        assert float((r.row_loss[0] - np.log(V)).abs().max()) <= 1e-5
        assert bool((r.row_loss[1] > 2e38).all()) and bool(torch.isfinite(r.row_loss[1]).all())
    assert bool((r.top1[0] == 0).all())
