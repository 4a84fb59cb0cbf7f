"""Stacked layers at a few batch rows per group (one XCD per layer and group,
four or eight rows): every tap of every layer against the oracle bit for bit
at the edges of the layout -- groups one row short and full, one and several
groups, several launches, cell counts and projection widths around a tile,
tiles with cells but no outputs and the other way round, the widest layers,
the most layers, short sequences; which kernel each case runs; and the state
carried between calls."""
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


# The last columns: the kernel that runs (over how many launches).  The layout is
# there for up to four rows a group without a projection, and with one where the
# exchange words fit the space of W_x x + b, which takes about ten frames; the
# other cases compare what such batches fall back to.
@pytest.mark.parametrize("layers,n_in,H,P,T,B,layout,launches", [
    (2, 7, 15, 0, 3, 2, "xrows4", 1),
    (5, 320, 500, 0, 9, 4, "xrows4", 1),
    (4, 24, 17, 0, 2, 5, "xrows4", 1),       # two groups, of 3 and 2 rows
    (3, 24, 17, 0, 5, 7, "xrows4", 1),       # two groups, of 4 and 3 rows
    (8, 24, 36, 0, 4, 3, "xrows4", 1),
    (2, 512, 512, 0, 3, 15, "xrows4", 1),    # four groups, the last one short
    (2, 40, 48, 0, 9, 16, "xrows4", 1),      # four full groups
    (2, 40, 16, 5, 12, 2, "xrows4", 1),
    (5, 320, 500, 200, 12, 4, "xrows4", 1),
    (3, 24, 100, 130, 20, 4, "xrows4", 1),   # more tiles with outputs than with cells
    (2, 40, 200, 512, 40, 5, "xrows4", 1),   # 13 tiles with cells, 32 with outputs
    (2, 40, 512, 1, 12, 5, "xrows4", 1),     # 31 tiles without outputs; groups of 3 and 2 rows
    (5, 320, 500, 200, 12, 6, "xrows8", 1),
    (5, 40, 100, 24, 9, 7, "xrows8", 1),     # one row short; tiles without outputs
    (3, 24, 100, 130, 20, 13, "xrows8", 1),  # more outputs than cells; groups of 7 and 6 rows
    (2, 512, 512, 512, 20, 27, "xrows8", 1),  # every tile full; groups of 7, 7, 7 and 6 rows
    (8, 40, 33, 17, 12, 20, "xrows8", 3),    # launches of 7, 7 and 6 rows
    (4, 16, 100, 40, 12, 31, "xrows8", 2),   # launches of 16 and 15 rows, two groups each
    # elsewhere: more rows than a launch holds without a projection; too little
    # space for the words; too few frames for several launches
    (5, 40, 100, 0, 1, 5, "xstack32", 1),
    (5, 40, 33, 0, 6, 8, "xstack32", 1),
    (4, 24, 17, 0, 2, 9, "xstack32", 1),
    (2, 512, 512, 0, 3, 31, "xstack32", 1),
    (2, 40, 16, 5, 1, 2, "layers", 2),
    (3, 24, 20, 130, 4, 4, "layers", 3),
    (5, 320, 500, 200, 8, 6, "layers", 5),
    (2, 512, 512, 512, 3, 8, "layers", 2),
    (8, 40, 33, 17, 5, 20, "layers", 8),
    (4, 16, 100, 40, 2, 33, "layers", 4),
    (5, 40, 100, 24, 12, 40, "layers", 5),
])
def test_rows_equal_oracle(ql, orc, layers, n_in, H, P, T, B, layout, launches):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, layers, proj=P, states=24, seed=layers * 1000 + H + P + B)
    x = np.random.default_rng(H + B).standard_normal((T, B, n_in)).astype(np.float32)
    M = ql.quantize_model(w)
    assert ql.model_layout(M, T, B) == (layout, launches)
    g = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda(), taps=True)
    o = orc.acoustic_model_forward(orc.quantize_model(w), x, taps=True)
    assert_model_taps(g, o, None, names=ql.TAP_NAMES)
    plain = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda())  # the build without taps
    assert torch.equal(plain["post"], g["post"])


@pytest.mark.parametrize("P,B,cuts,layouts", [
    (0, 3, (0, 1, 5, 9), ("xrows4", "xrows4", "xrows4")),
    (24, 7, (0, 1, 5, 9), ("layers", "layers", "layers")),
    (24, 40, (0, 1, 5, 9), ("layers", "layers", "layers")),
    (24, 40, (0, 64, 65, 140), ("xrows8", "layers", "xrows8")),
    (24, 3, (0, 1, 13, 30), ("layers", "xrows4", "xrows4")),
    (24, 7, (0, 12, 13, 30), ("xrows8", "layers", "xrows8")),
])
def test_rows_carry_state(ql, P, B, cuts, layouts):
    """Chunks of a sequence with the state carried give the whole call's bits."""
    from paper_1607_04683_amd.workloads import random_model
    M = ql.quantize_model(random_model(40, 100, 5, proj=P, states=32, seed=B))
    x = torch.randn(cuts[-1], B, 40, device="cuda")
    whole = ql.acoustic_model_forward(M, x)["post"]
    state, parts = None, []
    for a, b, layout in zip(cuts, cuts[1:], layouts):
        assert ql.model_layout(M, b - a, B)[0] == layout
        out = ql.empty_state(M, B)
        parts.append(ql.acoustic_model_forward(M, x[a:b].contiguous(), state_in=state,
                                               state_out=out)["post"])
        state = out
    assert torch.equal(torch.cat(parts), whole)
