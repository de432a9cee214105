"""The rules that choose a call's kernel form (host only)."""
import os

import pytest

from paper_2609_35440_amd import binding as B
from tests.routes import FUSED, PROD, SPLIT, P, route

pytestmark = pytest.mark.skipif(not os.path.exists(B.library_path()), reason="library not built")


def test_exit_evaluation_forms():
    assert route(True, 4, 16, 2048, 32000)[0] == SPLIT       # a decode step
    assert route(True, 4, 16384, 2048, 32000)[0] == PROD     # a validation batch
    assert route(True, 2, 9, 1024, 40)[0] == FUSED           # a toy vocabulary
    assert route(True, 2, 300, 64, 8000, "f32") == [FUSED, 1, 0]  # fp32 has one form


@pytest.mark.parametrize("K,T,d,V", [(2, 300, 72, 1025), (1, 961, 1520, 4777), (2, 364, 800, 366), (40, 29, 1392, 2216)])
def test_copies_that_just_fit_take_one_pass(K, T, d, V):
    """The workspace holds copies of up to 16384 rows next to the parts of the most splits, so a
    list of that many rows is one pass whatever the splits: 32 us for the first call, 43 in
    the form taken when the least number of passes was counted one too high."""
    form, splits, rows = route(True, K, T, d, V)
    assert form == PROD and rows >= K * T
    assert splits == -(-V // 256)  # few row tiles: as many parts as readout tiles


def test_workspace_short_of_copies_takes_the_form_without():
    a = B.SoloReadoutArgs()
    a.K, a.T, a.d, a.V, a.dtype, a.eps = 2, 300, 72, 4097, B.SOLO_BF16, 1e-6
    full = B.exit_eval_workspace_size(a)
    assert route(True, 2, 300, 72, 4097, workspace_bytes=full)[0] == PROD
    assert route(True, 2, 300, 72, 4097, workspace_bytes=full - 1)[0] == FUSED


def test_local_loss_splits():
    # tiles that leave most of the chip idle are cut, at most 64 ways; a full chip is not
    assert 1 < route(False, 2, 8, 1024, 32000)[0] <= 64
    assert route(False, 4, 16384, 2048, 32000)[0] == 1
    # the parts live in a readout gradient: a call without one is not cut
    assert route(False, 2, 8, 1024, 32000, final_module_dW=0)[0] == 1
    assert route(False, 3, 8, 1024, 32000, final_module_dW=0, heads_train_readout=1, readout_per_head=1, Wbar=P)[0] > 1
    # and never larger than it: (T rows) x (d + 4) floats per part
    for T in (1, 7, 100, 1000):
        s = route(False, 1, T, 64, 300, "f32")[0]
        assert s == 1 or s * T * (64 + 4) <= 300 * 64
