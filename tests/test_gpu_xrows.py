"""Stacked layers at a few batch rows per group (one XCD per layer and group,
four or eight rows): every tap of every layer against the oracle bit for bit
at the edges of the layout -- groups of one row short and full, one and several
groups, several launches, cell counts and projection widths around a tile,
tiles with cells but no outputs and the other way round, the widest layers,
the most layers, sequences of one to four frames; and the state carried
between calls."""
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


@pytest.mark.parametrize("layers,n_in,H,P,T,B", [
    (2, 7, 15, 0, 3, 2),
    (5, 320, 500, 0, 9, 4),
    (5, 40, 100, 0, 1, 5),
    (5, 40, 33, 0, 6, 8),
    (4, 24, 17, 0, 2, 9),      # two groups, of 5 and 4 rows
    (8, 24, 36, 0, 4, 3),
    (2, 512, 512, 0, 3, 31),   # four groups of 8, the last one short
    (2, 40, 16, 5, 1, 2),
    (3, 24, 20, 130, 4, 4),    # more tiles with outputs than with cells
    (5, 320, 500, 200, 8, 6),
    (2, 512, 512, 512, 3, 8),
    (8, 40, 33, 17, 5, 20),    # three launches
    (4, 16, 100, 40, 2, 33),   # three launches of two groups
])
def test_rows_equal_oracle(ql, orc, layers, n_in, H, P, T, B):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, layers, proj=P, states=24, seed=layers * 1000 + H + P + B)
    x = np.random.default_rng(H + B).standard_normal((T, B, n_in)).astype(np.float32)
    M = ql.quantize_model(w)
    g = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda(), taps=True)
    o = orc.acoustic_model_forward(orc.quantize_model(w), x, taps=True)
    assert_model_taps(g, o, None, names=ql.TAP_NAMES)
    plain = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda())  # the build without taps
    assert torch.equal(plain["post"], g["post"])


@pytest.mark.parametrize("P,B", [(0, 3), (24, 7), (24, 40)])
def test_rows_carry_state(ql, P, B):
    """Chunks of a sequence with the state carried give the whole call's bits."""
    from paper_1607_04683_amd.workloads import random_model
    M = ql.quantize_model(random_model(40, 100, 5, proj=P, states=32, seed=B))
    x = torch.randn(9, B, 40, device="cuda")
    whole = ql.acoustic_model_forward(M, x)["post"]
    state, parts = None, []
    for a, b in [(0, 1), (1, 5), (5, 9)]:
        out = ql.empty_state(M, B)
        parts.append(ql.acoustic_model_forward(M, x[a:b].contiguous(), state_in=state,
                                               state_out=out)["post"])
        state = out
    assert torch.equal(torch.cat(parts), whole)
