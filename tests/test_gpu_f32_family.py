"""The fp32 matrix-core family (fp32 storage, and the bf16 widths outside the
bf16 kernels) at the edges of its tilings: every column split, widths just past
one (a ragged last slab), one row past a tile, one readout row past a chunk,
and calls whose vocabulary is split over workgroups.

Products and sums are fp32 on either storage, so the fp32 outputs (losses,
dW, dgain) meet the fp32 tolerance for bf16 storage too; a bf16 dh adds its own
rounding to nearest at 8 significant bits, at most 2^-8 of each entry (unit
roundoff 2^-p for p bits)."""
import numpy as np
import pytest

import oracle
from solo_inputs import make_inputs
from tests.gpu_helpers import log, rel_max_err, run_gpu

pytestmark = pytest.mark.gpu

# (config, K, T, d, V); bf16 widths that are multiples of 256 up to 2048, and 2560, run on other kernels
CASES = [("tiny", 1, 1, 8, 1), ("tiny", 2, 33, 24, 257), ("tiny", 1, 31, 32, 256), ("tiny", 2, 32, 40, 511),
         ("tiny", 1, 65, 64, 513), ("tiny", 2, 17, 136, 1000), ("tiny", 1, 40, 264, 255), ("tiny", 1, 33, 520, 300),
         ("tiny", 2, 35, 768, 777), ("tiny", 1, 33, 776, 300), ("tiny", 1, 40, 1032, 300), ("tiny", 1, 34, 1544, 300),
         ("tiny", 1, 33, 2048, 300), ("tiny", 1, 17, 2056, 300), ("tiny", 1, 18, 3080, 260), ("tiny", 1, 17, 4096, 260),
         ("tiny", 2, 5, 64, 9000), ("tiny", 3, 70, 208, 5000),
         ("1b", 1, 33, 8, 257), ("1b", 2, 40, 72, 513), ("1b", 1, 31, 128, 256), ("1b", 2, 37, 640, 2000),
         ("1b", 2, 65, 200, 1030), ("1b", 1, 33, 904, 300), ("1b", 1, 33, 1160, 300), ("1b", 2, 34, 1528, 500), ("1b", 1, 33, 1800, 300),
         ("1b", 1, 18, 2304, 300), ("1b", 1, 17, 3072, 600), ("1b", 2, 19, 4088, 520)]


@pytest.mark.parametrize("final", [True, False], ids=["dW", "frozen"])
@pytest.mark.parametrize("cfg,K,T,d,V", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_edges(cfg, K, T, d, V, final):
    x = make_inputs(cfg, seed=5, K=K, T=T, d=d, V=V)
    log(f"f32 family {cfg} K={K} T={T} d={d} V={V} dW={final}")
    got = run_gpu(x, final)
    ref = oracle.readout_fwd_bwd(x["h"], x["gain"], x["W"], x["targets"], final)
    for k in range(K):
        # (V = 1: every loss is zero)
        assert abs(got["losses"][k] - ref["losses"][k]) <= 1e-5 * max(abs(ref["losses"][k]), 1e-2)
        e = np.abs(got["dh"][k] - ref["dh"][k])
        scale = np.abs(ref["dh"][k]).max()
        store = 2.0 ** -8 * np.abs(ref["dh"][k]) if x["cfg"].dtype == "bf16" else 0.0
        assert np.all(e <= 1e-5 * scale + store), (k, (e - store).max(), scale)
    if final:
        assert rel_max_err(got["dW"], ref["dW"]) <= 1e-5
        assert rel_max_err(got["dgain"], ref["dgain"]) <= 1e-5
