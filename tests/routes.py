"""Which kernel form a call takes, from the library's own rules (host only), for tests
that are about one form: a changed rule then fails them instead of emptying them."""
import ctypes

FUSED, SPLIT, PROD = 0, 1, 2
P = 0x10000  # stands for a pointer that is given; never dereferenced


def route(exit_eval: bool, K, T, d, V, dtype="bf16", workspace_bytes=1 << 50, **fields):
    """[form, splits, rows per pass] of exit evaluation, or [splits of the local-loss
    pass, of the terminal's own under ROT, splits of the bias gradient's product]."""
    from paper_2609_35440_amd import binding

    a = binding.SoloReadoutArgs()
    a.K, a.T, a.d, a.V, a.eps = K, T, d, V, 1e-6
    a.dtype = binding.SOLO_BF16 if dtype == "bf16" else binding.SOLO_F32
    a.final_module_dW = 1
    a.workspace_bytes = workspace_bytes
    for name, v in fields.items():
        setattr(a, name, v)
    out = (ctypes.c_longlong * 3)()
    assert binding.load_library().solo_readout_route(ctypes.byref(a), int(exit_eval), out) == 0
    return list(out)


def route_of(x: dict, exit_eval: bool, **flags):
    """The same for a test's inputs and flags."""
    K, T, d = x["h"].shape
    f = {}
    if x.get("Wbar") is not None:
        f["Wbar"] = P
        f["readout_per_head"] = int(x["Wbar"].ndim == 3)
    for name in ("tau", "bias", "rot"):
        if x.get(name) is not None:
            f[name] = P
    f["gain_per_module"] = int(x["gain"].ndim == 2)
    f["final_module_dW"] = int(flags.get("final_module_dW", True))
    f["heads_train_readout"] = int(flags.get("heads_train_readout", False))
    for name in ("dtau", "dbias"):
        if flags.get("want_" + name):
            f[name] = P
    if "workspace_bytes" in flags:
        f["workspace_bytes"] = flags["workspace_bytes"]
    return route(exit_eval, K, T, d, x["W"].shape[0], x["cfg"].dtype, **f)
