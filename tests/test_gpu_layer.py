"""One layer without a projection through ql_lstm_layer_forward: on the whole
chip it runs as a stack of one, with the input product in the step.  Every tap,
h and the final state against the oracle bit for bit at the edges between that
layout's kernels (one row; groups of four on up to eight XCDs; units of 16, in
32- and 64-cell tiles, over one launch and two), with and without an initial
state, for narrow cells, which take a launch per layer where several launches of
units would be slower, and for an input too wide for any of it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1607_04683_amd import qlstm
    qlstm.load()
    return qlstm


@pytest.mark.parametrize("n_in,H,T,B", [(512, 500, 5, 1), (24, 17, 3, 2), (40, 100, 4, 32), (40, 36, 3, 33),
                                        (320, 500, 2, 257), (24, 500, 6, 600), (7, 20, 2, 530),
                                        (520, 64, 3, 20)])
def test_single_layer_equals_oracle(ql, orc, n_in, H, T, B):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, 1, seed=H + B)["layers"][0]
    rng = np.random.default_rng(B)
    x = rng.standard_normal((T, B, n_in)).astype(np.float32)
    h0 = c0 = None
    if B % 2:
        h0 = (np.tanh(rng.standard_normal((B, H))) * 0.7).astype(np.float32)
        c0 = rng.standard_normal((B, H)).astype(np.float32)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    g = ql.lstm_layer_forward(ql.quantize_layer(w), dev(x), dev(h0), dev(c0), taps=True)
    o = orc.lstm_layer_forward(orc.quantize_layer(w), x, h0, c0, taps=True)
    for k in ("h", "hT", "cT", "acc_x", "acc_h", "gates", "c"):
        if k in g and k in o:
            got, want = g[k].cpu().numpy().reshape(-1), np.asarray(o[k]).reshape(-1)
            assert np.array_equal(got.view(np.uint32), want.astype(got.dtype).view(np.uint32)), k


def test_single_layer_refuses_more_rows_than_the_spread_tiles_hold(ql):
    """2048 rows of 500 cells have no tiling that leaves room for the codes."""
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(24, 500, 1, seed=1)["layers"][0]
    with pytest.raises(ql.QLError, match="not supported"):
        ql.lstm_layer_forward(ql.quantize_layer(w), torch.zeros(1, 2048, 24, device="cuda"))
