"""The forward-only passes as a tiled product (exit evaluation over many rows, the
bias gradient over many tokens) at the edges of their 256 x 256 tiles: a last
tile of one row of either operand, rows in one list over modules with
their own gains and temperatures, one list per module (biases, one readout per
head), more rows than one pass holds, invalid targets, vocabulary entries masked
by a bias of -inf, the largest negative bias, and ties across tiles.

Every test asserts that the product form is the one taken (tests/routes.py)."""
import numpy as np
import pytest

import oracle
from solo_inputs import make_extras, make_inputs
from tests.gpu_helpers import rel_max_err
from tests.routes import FUSED, PROD, P, route, route_of
from tests.test_gpu_general import check_exit_eval, compare, oracle_general, run_exit_eval, run_general

pytestmark = pytest.mark.gpu


# a last tile of one row of either operand; two passes of rows; more than two modules per tile
EVAL = [("plain", 2, 1537, 16129, dict()), ("one-list", 2, 1537, 16129, dict(per_module_gain=True, tau=True)),
        ("bias", 2, 1537, 16129, dict(bias=True)),
        ("per-head", 2, 1537, 16129, dict(wbar="per_head", bias=True, tau=True)),
        ("two-passes", 2, 6017, 12289, dict(per_module_gain=True)),
        ("many-modules", 70, 45, 12289, dict(per_module_gain=True))]


@pytest.mark.parametrize("name,K,T,V,extras", EVAL, ids=[c[0] for c in EVAL])
def test_eval(name, K, T, V, extras):
    x = make_extras(make_inputs("1b", seed=12, K=K, T=T, d=256, V=V), seed=12, **extras)
    form, _, rows = route_of(x, True)
    assert form == PROD and (rows < K * T) == (name in ("two-passes", "bias", "per-head"))
    losses, row_loss, top1 = run_exit_eval(x)
    check_exit_eval(x, losses, row_loss, top1, f"product eval {name}", min_rows_for_agreement=100)


@pytest.mark.parametrize("d,V", [(1024, 16129), (2048, 4097)])
def test_eval_wide(d, V):
    x = make_inputs("1b", seed=12, K=2, T=1537, d=d, V=V)
    assert route_of(x, True)[0] == PROD
    losses, row_loss, top1 = run_exit_eval(x)
    check_exit_eval(x, losses, row_loss, top1, f"product eval d={d}", min_rows_for_agreement=100)


def _device(K, T, d, V, seed=4):
    import torch

    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randn(K, T, d, generator=g, device="cuda").to(torch.bfloat16)
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).to(torch.bfloat16)
    y = torch.randint(0, V, (K, T), generator=g, device="cuda", dtype=torch.int32)
    return h, torch.ones(d, dtype=torch.bfloat16, device="cuda"), W, y


def test_eval_masks_ties_and_invalid_targets():
    import torch

    from paper_2609_35440_amd import binding

    K, T, d, V = 1, 3073, 256, 12289
    assert route(True, K, T, d, V)[0] == PROD and route(True, K, T, d, V, bias=P)[0] == PROD
    h, gain, W, y = _device(K, T, d, V)
    W[12288] = W[70] = W[2500] = (0.1 * h[0, 7].float()).to(torch.bfloat16)
    y[0, 11] = V + 5
    y[0, 12] = -1
    plain = binding.exit_eval(h, gain, W, y)
    assert int(plain.top1[0, 7]) == 70
    bad = torch.isnan(plain.row_loss[0])
    assert bad[11] and bad[12] and int(bad.sum()) == 2
    # half the vocabulary masked, by -inf and by the type's lowest value, the target kept
    y = (y.clamp(0, V - 1) // 2 * 2).clamp(max=V - 1)
    for low in (-float("inf"), torch.finfo(torch.float32).min):
        bias = torch.zeros(K, V, device="cuda")
        bias[:, 1::2] = low
        r = binding.exit_eval(h, gain, W, y, bias=bias)
        z = (h[0].double() * torch.rsqrt(h[0].double().square().mean(1, keepdim=True) + 1e-6)) @ W.double().t()
        z[:, 1::2] = -float("inf")
        ref = torch.logsumexp(z, 1) - z.gather(1, y[0].long()[:, None])[:, 0]
        assert float((r.row_loss[0].double() - ref).abs().max()) < 2e-2
        assert int((r.top1 % 2).sum()) == 0
    # everything but the target masked: no loss
    bias = torch.full((K, V), -float("inf"), device="cuda")
    bias[:, 12288] = 0.0
    r = binding.exit_eval(h, gain, W, torch.full_like(y, 12288), bias=bias)
    assert torch.equal(r.row_loss, torch.zeros_like(r.row_loss)) and bool((r.top1 == 12288).all())


@pytest.mark.parametrize("T,V,extras,final", [(2049, 1025, dict(bias=True, tau=True), True),
                                              (1800, 513, dict(wbar="per_head", bias=True), False),
                                              (2304, 769, dict(per_module_gain=True), True),
                                              (1500, 600, dict(rot=True, tau=True), True)],
                         ids=["heads", "all-per-head", "no-bias", "rot"])
def test_bias_gradient(T, V, extras, final):
    x = make_extras(make_inputs("1b", seed=13, K=3, T=T, d=256, V=V), seed=13, **extras)
    flags = dict(final_module_dW=final, want_dtau=True, want_dbias=True)
    assert route_of(x, False, **flags)[2] > 1
    g = run_general(x, flags)
    ref = oracle_general(x, flags)
    compare(g, ref, "bf16", flags, f"product bias gradient {T} {V}")
    for k in range(3):
        assert rel_max_err(g["dbias"][k], ref["dbias"][k]) <= 2e-2


# bf16 widths defined in fp32: the product on two planes of g * h; the last ones
# up to d = 64, where a tile has two stages, with several tiles per split, and past 2560
PLANES = [("plain", 2, 300, 72, 1025, dict()), ("one-list", 3, 9, 640, 5000, dict(per_module_gain=True, tau=True)),
          ("bias", 2, 257, 1000, 700, dict(bias=True)), ("per-head", 2, 300, 136, 2049, dict(wbar="per_head")),
          ("many-modules", 40, 33, 136, 2049, dict(per_module_gain=True, tau=True)),
          ("wide", 1, 33, 3080, 513, dict()), ("wide-bias", 2, 130, 3080, 1500, dict(bias=True)),
          ("widest", 2, 5, 4096, 300, dict(tau=True)), ("narrow", 1, 700, 8, 7000, dict()),
          ("two-stages", 1, 4100, 64, 9000, dict(bias=True))]


@pytest.mark.parametrize("name,K,T,d,V,extras", PLANES, ids=[c[0] for c in PLANES])
def test_eval_planes(name, K, T, d, V, extras):
    from tests.gpu_helpers import row_loss_error_bound

    x = make_extras(make_inputs("1b", seed=14, K=K, T=T, d=d, V=V), seed=14, **extras)
    form, splits, _ = route_of(x, True)
    assert form == PROD and (name != "two-stages" or 2 * splits <= V // 256)
    losses, row_loss, top1 = run_exit_eval(x)
    check_exit_eval(x, losses, row_loss, top1, f"planes {name}", min_rows_for_agreement=100)
    # fp32 logits: within the bound of fp32 operands and sums
    ref = oracle.exit_eval(x["h"], x["gain"], x["W"], x["targets"], Wbar=x.get("Wbar"), tau=x.get("tau"),
                           bias=x.get("bias"))
    for k in range(K):
        R = oracle.solo_oracle_general.readout_matrix(k, K, x["W"], x.get("Wbar"))
        gk = x["gain"][k] if x["gain"].ndim == 2 else x["gain"]
        tk = 1.0 if x.get("tau") is None else float(x["tau"][k])
        bk = None if x.get("bias") is None else x["bias"][k]
        bound = row_loss_error_bound(x["h"][k], gk, R, x["targets"][k], tk, "f32", bk)
        assert np.all(np.abs(row_loss[k] - ref["row_loss"][k]) <= bound), (name, k)


@pytest.mark.parametrize("T,d,V,extras,final", [(1025, 136, 1025, dict(bias=True, tau=True), True),
                                                (700, 640, 513, dict(wbar="per_head", bias=True), False),
                                                (513, 1800, 600, dict(rot=True), True)], ids=["heads", "all", "rot"])
def test_bias_gradient_planes(T, d, V, extras, final):
    x = make_extras(make_inputs("1b", seed=15, K=3, T=T, d=d, V=V), seed=15, **extras)
    flags = dict(final_module_dW=final, want_dtau=True, want_dbias=True)
    assert route_of(x, False, **flags)[2] > 1
    g = run_general(x, flags)
    ref = oracle_general(x, flags)
    compare(g, ref, "bf16", flags, f"bias gradient on planes {T} {d} {V}")
    if "rot" not in extras:  # (rotated rows are rounded to bf16)
        for k in range(3):
            assert rel_max_err(g["dbias"][k], ref["dbias"][k]) <= 1e-5, k


def test_workspace_without_plane_copies(monkeypatch):
    """The plane copies are a matter of speed: a workspace of the statistics alone serves too,
    within the same fp32 bounds, and one byte less is refused."""
    from paper_2609_35440_amd import binding

    al = lambda n: -(-n // 256) * 256
    K, T, d, V = 2, 300, 72, 4097
    x = make_extras(make_inputs("1b", seed=14, K=K, T=T, d=d, V=V), seed=14, bias=True)
    assert route_of(x, True)[0] == PROD
    assert route_of(x, True, workspace_bytes=3 * al(K * T * 4))[0] == FUSED
    full = run_exit_eval(x)
    monkeypatch.setattr(binding, "exit_eval_workspace_size", lambda a: 3 * al(K * T * 4))
    losses, row_loss, top1 = run_exit_eval(x)
    check_exit_eval(x, losses, row_loss, top1, "eval without copies", min_rows_for_agreement=100)
    assert np.abs(row_loss - full[1]).max() <= 1e-4 and np.array_equal(top1, full[2])
    monkeypatch.setattr(binding, "exit_eval_workspace_size", lambda a: 3 * al(K * T * 4) - 1)
    with pytest.raises(Exception, match="(?i)workspace"):
        run_exit_eval(x)

    T, d, V = 1025, 136, 1025
    x = make_extras(make_inputs("1b", seed=15, K=3, T=T, d=d, V=V), seed=15, bias=True, tau=True)
    flags = dict(final_module_dW=True, want_dtau=True, want_dbias=True)
    size = binding.general_workspace_size

    def least(a):  # the terminal's bias gradient is free: without dbias there are no copies
        kept, a.dbias = a.dbias, None
        n = size(a)
        a.dbias = kept
        return n

    kt = 3 * T
    least_bytes = 3 * al(kt * 4) + al(kt * 16) + al(kt * 4) + al(-(-T // 8) * d * 4)
    assert route_of(x, False, **flags)[2] > 0
    assert route_of(x, False, workspace_bytes=least_bytes, **flags)[2] == 0
    monkeypatch.setattr(binding, "general_workspace_size", least)
    g = run_general(x, flags)
    ref = oracle_general(x, flags)
    compare(g, ref, "bf16", flags, "bias gradient without copies")
    for k in range(3):
        assert rel_max_err(g["dbias"][k], ref["dbias"][k]) <= 1e-5, k
