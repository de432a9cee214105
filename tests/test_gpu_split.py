"""Calls of few tokens, whose row tiles are split over the vocabulary: every
family and tiling, against the oracle, with vocabularies that end inside a
chunk or leave splits of unequal length; exit evaluation over the rows of all
modules as one list (per-module gains and temperatures), with one readout per
head (not one list), and ties whose columns lie in different splits."""
import numpy as np
import pytest

import oracle
from solo_inputs import make_extras, make_inputs
from tests.gpu_helpers import check_close, log, run_gpu
from tests.routes import SPLIT, route, route_of
from tests.test_gpu_general import check_exit_eval, compare, oracle_general, run_exit_eval, run_general

pytestmark = pytest.mark.gpu

TRAIN = [("1b", 4, 3, 256, 2065), ("1b", 2, 65, 1024, 1999), ("1b", 3, 33, 2048, 1040), ("2b", 2, 17, 2560, 1041),
         ("1b", 2, 5, 3072, 2050), ("tiny", 3, 9, 200, 4100)]


@pytest.mark.parametrize("cfg,K,T,d,V", TRAIN, ids=["-".join(map(str, c)) for c in TRAIN])
def test_train(cfg, K, T, d, V):
    x = make_inputs(cfg, seed=8, K=K, T=T, d=d, V=V)
    log(f"split {cfg} {K} {T} {d} {V}")
    assert route_of(x, False)[0] > 1
    check_close(run_gpu(x, True), oracle.readout_fwd_bwd(x["h"], x["gain"], x["W"], x["targets"], True),
                x["cfg"].dtype, what=f"split d={d}")


@pytest.mark.parametrize("cfg,d", [("1b", 1024), ("2b", 2560), ("tiny", 72)])
def test_general(cfg, d):
    x = make_extras(make_inputs(cfg, seed=9, K=3, T=37, d=d, V=1500), seed=9, per_module_gain=True, tau=True,
                    bias=True)
    flags = dict(final_module_dW=True, want_dtau=True, want_dbias=True)
    assert route_of(x, False, **flags)[0] > 1
    compare(run_general(x, flags), oracle_general(x, flags), x["cfg"].dtype, flags, f"split general d={d}")


@pytest.mark.parametrize("extras", [dict(per_module_gain=True, tau=True), dict(wbar="per_head", tau=True),
                                    dict(bias=True)], ids=["one-list", "per-head", "bias"])
@pytest.mark.parametrize("cfg,d", [("1b", 512), ("1b", 2048), ("2b", 2560)])
def test_eval(cfg, d, extras):
    x = make_extras(make_inputs(cfg, seed=10, K=3, T=30, d=d, V=2003), seed=10, **extras)
    assert route_of(x, True)[0] == SPLIT
    losses, row_loss, top1 = run_exit_eval(x)
    check_exit_eval(x, losses, row_loss, top1, f"split eval d={d}", min_rows_for_agreement=60)


def test_eval_ties_across_splits():
    import torch

    from paper_2609_35440_amd import binding

    K, T, d, V = 2, 3, 1024, 4000
    assert route(True, K, T, d, V)[:2] == [SPLIT, 250]
    g = torch.Generator().manual_seed(3)
    h = torch.randn(K, T, d, generator=g).to(torch.bfloat16).cuda()
    W = (0.02 * torch.randn(V, d, generator=g)).to(torch.bfloat16)
    W[3999] = W[70] = W[2500] = (0.1 * h[0, 0].cpu().float()).to(torch.bfloat16)  # far above the rest for that row
    r = binding.exit_eval(h, torch.ones(d, dtype=torch.bfloat16, device="cuda"), W.cuda(),
                          torch.zeros(K, T, dtype=torch.int32, device="cuda"))
    assert int(r.top1[0, 0]) == 70
    assert np.isfinite(r.losses.cpu().numpy()).all()


@pytest.mark.parametrize("K,T,d,V", [(3, 2048, 2048, 25600), (1, 2900, 2560, 12000)], ids=["mfma", "wide"])
def test_more_tiles_than_half_the_chip(K, T, d, V):
    """Row tiles between half the chip and the whole of it are cut too (192 and 182 tiles, 4 ways).  Against the
    same rows without a readout gradient, which has no room for parts and is not cut."""
    import torch

    from paper_2609_35440_amd import binding

    g = torch.Generator(device="cuda").manual_seed(5)
    h = torch.randn(K, T, d, generator=g, device="cuda").to(torch.bfloat16)
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).to(torch.bfloat16)
    y = torch.randint(0, V, (K, T), generator=g, device="cuda", dtype=torch.int32)
    gain = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    assert route(False, K, T, d, V)[0] == 4 and route(False, K, T, d, V, final_module_dW=0)[0] == 1
    cut = binding.readout_fwd_bwd(h, gain, W, y, final_module_dW=True, row_loss=True)
    whole = binding.readout_fwd_bwd(h, gain, W, y, final_module_dW=False, row_loss=True)
    # the same fp32 logits; sums of up to 1600 chunks in another order: 2 x 1600 x 2^-24
    assert float((cut.row_loss - whole.row_loss).abs().max()) <= 2 * 1600 * 2.0**-24
    # one rounding of each output (2^-8 relative)
    a, b = cut.dh.float(), whole.dh.float()
    assert float((a - b).norm() / b.norm()) <= 2.0**-7
