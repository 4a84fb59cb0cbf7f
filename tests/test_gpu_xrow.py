"""Stacked layers at one batch row on the whole chip (one XCD per layer, 16
cells and 16 projection outputs per workgroup): every tap of every layer
against the oracle bit for bit where the layout has edges -- cell counts and
projection widths around a tile, tiles with cells but no outputs and the other
way round, the widest input, cells and projection, the most layers of a
launch, and sequences of one to three frames (the exchange's two step
parities)."""
import numpy as np
import pytest
import torch
from model_parity import assert_model_taps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1607_04683_amd import qlstm
    qlstm.load()
    return qlstm


@pytest.mark.parametrize("layers,n_in,H,P,T", [
    (2, 7, 15, 0, 3),
    (2, 9, 17, 0, 1),
    (3, 64, 16, 0, 2),
    (8, 40, 33, 0, 9),
    (2, 512, 512, 0, 3),
    (5, 320, 500, 0, 40),
    (2, 40, 16, 5, 1),
    (3, 24, 17, 16, 2),
    (2, 24, 20, 130, 5),     # more tiles with outputs than with cells
    (8, 40, 100, 17, 6),
    (2, 512, 512, 512, 3),
    (5, 320, 500, 200, 20),
    (3, 12, 40, 1, 4),       # one output
    (3, 12, 30, 1, 1),       # its words are two more a layer than k_pstack's scratch, which runs
])
def test_one_row_stack_equals_oracle(ql, orc, layers, n_in, H, P, T):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, layers, proj=P, states=24, seed=layers * 1000 + H + P)
    x = np.random.default_rng(H + T).standard_normal((T, 1, n_in)).astype(np.float32)
    M = ql.quantize_model(w)
    assert ql.model_layout(M, T, 1) == ("spread" if (H, P, T) == (30, 1, 1) else "xrow", 1)
    g = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda(), taps=True)
    o = orc.acoustic_model_forward(orc.quantize_model(w), x, taps=True)
    assert_model_taps(g, o, None, names=ql.TAP_NAMES)
    plain = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda())  # the build without taps
    assert torch.equal(plain["post"], g["post"])
