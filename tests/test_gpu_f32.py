"""The unquantized fp32 model path against the oracle's float model.

The GPU accumulates products in fp32 (MFMA), the oracle in fp64, so results
agree to rounding rather than bit for bit: the bar is 1e-4 absolute on h, the
final state and the posteriors.  The GEMM alone is held to the standard
worst-case bound of fp32 summation, K * 2^-24 * sum_k |x_k w_k|."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.fixture(scope="module")
def ql():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1607_04683_amd import qlstm
    qlstm.load()
    return qlstm


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("m,rows,cols", [(1, 1, 1), (5, 33, 7), (130, 257, 129), (300, 2000, 320),
                                         (64, 8192, 500), (129, 130, 1023)])
def test_f32_matmul(ql, m, rows, cols):
    rng = np.random.default_rng(m + rows + cols)
    W = rng.normal(0, 0.05, (rows, cols)).astype(np.float32)
    X = rng.standard_normal((m, cols)).astype(np.float32)
    b = rng.normal(0, 0.1, rows).astype(np.float32)
    Y = ql.f32_matmul(dev(W), dev(X), dev(b)).cpu().numpy().astype(np.float64)
    ref = X.astype(np.float64) @ W.astype(np.float64).T + b
    mag = np.abs(X.astype(np.float64)) @ np.abs(W.astype(np.float64)).T + np.abs(b)
    bound = (cols + 2) * 2.0 ** -24 * mag
    assert np.all(np.abs(Y - ref) <= bound)


def _layer(ql, orc, n_in, H, P, T, B, seed, h0c0=False):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, 1, proj=P, seed=seed)["layers"][0]
    rng = np.random.default_rng(seed + 7)
    x = rng.standard_normal((T, B, n_in)).astype(np.float32)
    R = P if P else H
    h0 = c0 = None
    if h0c0:
        h0 = (np.tanh(rng.standard_normal((B, R))) * 0.5).astype(np.float32)
        c0 = rng.standard_normal((B, H)).astype(np.float32)
    g = ql.f32_lstm_layer_forward(ql.f32_layer(w), dev(x), dev(h0), dev(c0))
    o = orc.lstm_layer_forward_f32(w, x, h0, c0)
    for k in ("h", "hT", "cT"):
        assert np.max(np.abs(g[k].cpu().numpy() - o[k])) <= TOL, k


@pytest.mark.parametrize("n_in,H,P,T,B,h0c0", [
    (40, 37, 0, 7, 3, False),        # one batch row per tile, ragged units
    (320, 500, 0, 40, 64, True),     # 16-row MFMA tiles, W_h slice in LDS
    (64, 96, 32, 12, 20, True),      # projection, MFMA, ragged batch slice
    (48, 64, 16, 9, 2, False),       # projection, one batch row per tile
    (640, 2048, 512, 3, 16, False),  # the LSTMP layer's shapes
    (64, 2048, 512, 2, 256, False),  # batch 256: W_h slice read from L2
])
def test_f32_layer_shapes(ql, orc, n_in, H, P, T, B, h0c0):
    _layer(ql, orc, n_in, H, P, T, B, seed=n_in + H + P + B, h0c0=h0c0)


def test_f32_layer_500_T300_B1(ql, orc):
    """One 500-cell layer, 320-dim stacked features, T = 300, batch 1."""
    from paper_1607_04683_amd import workloads as wl
    w, _ = wl.model_weights(wl.LSTM1x500_T300_B1)
    x = wl.features(wl.LSTM1x500_T300_B1)
    L = w["layers"][0]
    g = ql.f32_lstm_layer_forward(ql.f32_layer(L), dev(x))
    o = orc.lstm_layer_forward_f32(L, x)
    for k in ("h", "hT", "cT"):
        assert np.max(np.abs(g[k].cpu().numpy() - o[k])) <= TOL, k


def test_f32_model_small(ql, orc):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(40, 48, 2, states=100, seed=3)
    x = np.random.default_rng(4).standard_normal((11, 5, 40)).astype(np.float32)
    g = ql.f32_acoustic_model_forward(ql.f32_model(w), dev(x))["post"].cpu().numpy()
    o = orc.acoustic_model_forward_f32(w, x)["post"]
    assert np.max(np.abs(g - o)) <= TOL
    assert np.allclose(g.sum(-1), 1.0, atol=1e-5)


def test_f32_model_5x500_B1(ql, orc):
    """The 5-layer 500-cell model with the 8192-way softmax, T = 500, batch 1."""
    from paper_1607_04683_amd import workloads as wl
    W = wl.LSTM5x500_S8192_T500_B1
    w, _ = wl.model_weights(W)
    x = wl.features(W)
    g = ql.f32_acoustic_model_forward(ql.f32_model(w), dev(x))["post"].cpu().numpy()
    o = orc.acoustic_model_forward_f32(w, x)["post"]
    assert np.max(np.abs(g - o)) <= TOL


def test_f32_model_B64_sampled_utterance(ql, orc):
    """Batch 64 x T = 1000 on the GPU; utterance 45 against the oracle
    (utterances are independent)."""
    from paper_1607_04683_amd import workloads as wl
    W = wl.LSTM5x500_S8192_T1000_B64
    w, _ = wl.model_weights(W)
    x = wl.features(W)
    g = ql.f32_acoustic_model_forward(ql.f32_model(w), dev(x))["post"][:, 45].cpu().numpy()
    o = orc.acoustic_model_forward_f32(w, x[:, 45:46])["post"][:, 0]
    assert np.max(np.abs(g - o)) <= TOL


# The last column: launches of the layout with an eighth of the batch per XCD (0: the
# batch in tiles over the chip, where several launches of narrow layers are slower).
@pytest.mark.parametrize("H,T,B,launches", [
    (1, 3, 1, 1),       # one cell, one row
    (15, 2, 8, 1),      # a tile one cell short; one row on every XCD
    (17, 4, 9, 1),      # a second tile of one cell; 2 rows, the last XCDs without
    (512, 2, 33, 1),    # every tile full; 5 rows: a second row group of one
    (500, 3, 64, 1),    # 8 rows per XCD
    (487, 3, 20, 1),    # rows of W_h off the 16-byte boundaries
    (96, 1, 65, 1),     # 9 rows: the 16-row form; one frame
    (260, 3, 128, 1),   # a full launch
    (36, 3, 129, 0),    # one row more than a launch holds
    (200, 2, 129, 0),
    (201, 3, 129, 2),   # launches of 65 and 64 rows
    (256, 2, 257, 0),
    (257, 2, 257, 3),
])
def test_f32_layer_xcd_rows(ql, orc, H, T, B, launches):
    """The layout with an eighth of the batch per XCD at its edges."""
    assert ql.float_layout(H, T, B) == launches
    _layer(ql, orc, 24, H, 0, T, B, seed=H + T + B, h0c0=B % 2 == 1)


@pytest.mark.parametrize("H,B", [(500, 3), (300, 140), (64, 140)])
def test_f32_layer_chunks_chain_bit_for_bit(ql, H, B):
    from paper_1607_04683_amd.workloads import random_model
    L = ql.f32_layer(random_model(24, H, 1, seed=H)["layers"][0])
    x = torch.randn(9, B, 24, device="cuda")
    whole, h, c, parts = ql.f32_lstm_layer_forward(L, x), None, None, []
    for a, b in [(0, 1), (1, 3), (3, 9)]:
        g = ql.f32_lstm_layer_forward(L, x[a:b].contiguous(), h, c)
        h, c = g["hT"], g["cT"]
        parts.append(g["h"])
    assert torch.equal(torch.cat(parts), whole["h"]) and torch.equal(c, whole["cT"])


# Row softmax: states around the registers per thread it is built for, and the
# first width beyond them all.
@pytest.mark.parametrize("S", [1, 63, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193])
def test_f32_posteriors_at_the_softmax_widths(ql, orc, S):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(8, 8, 1, states=S, seed=S)
    x = np.random.default_rng(S).standard_normal((3, 2, 8)).astype(np.float32)
    g = ql.f32_acoustic_model_forward(ql.f32_model(w), dev(x))["post"].cpu().numpy().astype(np.float64)
    o = orc.acoustic_model_forward_f32(w, x)["post"]
    # exp of a difference of logits |z| < 8 and fp32 sums of S terms
    assert np.max(np.abs(g - o)) <= TOL * np.max(o)
    assert np.max(np.abs(g.sum(-1) - 1.0)) < 1e-5
