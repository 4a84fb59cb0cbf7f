"""Stacked layers without a projection (Section 4) on the whole chip: units of
up to 16 batch rows of one layer, on 16 workgroups of 32 cells or 8 of 64 that
share an XCD, hand the codes of h_t and the rows' min / max to each other through
its L2, and each layer's quantized output crosses to the next XCD.  Every tap of
every layer (input and recurrent sums, codes, row params, fp32 h, gates, c)
is compared with the oracle bit for bit on ragged shapes: the smallest batch and
full units, units one row short, cell counts that leave tiles without cells, the
widest input and cell count, the most layers one launch holds, several launches,
what other batches fall back to, and sequences of one and two frames; each case
asserts the kernel that ran."""
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


# layers, n_in, H, T, B
CASES = [
    (2, 40, 48, 9, 16),      # (two layers: four groups of four rows of the few-row layout)
    (3, 40, 48, 9, 16),      # the smallest batch: one full 16-row MFMA tile
    (2, 40, 48, 9, 17),      # two groups, of 9 and 8 rows
    (3, 24, 100, 6, 33),     # three groups of 11 rows; 100 cells: tiles 4..15 of a group hold none
    (8, 40, 64, 5, 21),      # the most layers of one launch; 11 + 10 rows
    (2, 512, 512, 4, 64),    # the widest input and cell count at full batch
    (3, 320, 500, 4, 64),    # the 5 x 500 model's widths
    (4, 70, 36, 7, 47),      # 36 cells: one full tile and one with 4 cells
    (3, 40, 48, 1, 20),      # one frame: x_1 never loaded, the last output at once
    (2, 24, 64, 2, 64),      # two frames: x_2 never loaded
]


@pytest.mark.parametrize("layers,n_in,H,T,B", CASES)
def test_xcd_stack_equals_oracle(ql, orc, layers, n_in, H, T, B):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, layers, states=40, seed=layers * 1000 + H + B)
    x = np.random.default_rng(B + H).standard_normal((T, B, n_in)).astype(np.float32)
    M = ql.quantize_model(w)
    assert ql.stack_layers_per_launch(M, T, B) == layers
    assert ql.stack_layout(M, T, B) == 1
    kernel = ql.model_layout(M, T, B)[0]
    assert kernel == "xrows4" if (layers, B) == (2, 16) else kernel.startswith("xstack")
    g = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda(), taps=True)
    o = orc.acoustic_model_forward(orc.quantize_model(w), x, taps=True)
    assert_model_taps(g, o, None, names=ql.TAP_NAMES)


def test_layout_choice(ql):
    """Batches 16 to 64 of 2 or more stacked layers take the XCD layout; one
    row, batch 15 or 65, a single layer or a layer with a projection do not."""
    from paper_1607_04683_amd.workloads import random_model
    M = lambda n, H=48, P=0: ql.quantize_model(random_model(40, H, n, proj=P, states=20, seed=3))
    assert ql.stack_layout(M(3), 10, 16) == 1
    assert ql.stack_layout(M(3), 10, 64) == 1
    assert ql.stack_layout(M(3), 10, 15) == 0
    assert ql.stack_layout(M(3), 10, 65) == 0
    assert ql.stack_layout(M(3), 10, 1) == 0
    assert ql.stack_layout(M(1), 10, 32) == 0
    assert ql.stack_layout(M(3, 64, 24), 10, 32) == 0


def test_xcd_stack_repeats_bit_for_bit(ql):
    """The 5 x 500 model's stack at batch 64, 60 frames: the build without taps
    twice and the build with taps once give the same codes."""
    from paper_1607_04683_amd.workloads import random_model
    M = ql.quantize_model(random_model(320, 500, 5, states=64, seed=4))
    x = torch.randn(60, 64, 320, device="cuda")
    assert ql.stack_layout(M, 60, 64) == 1
    ref = ql.acoustic_model_forward(M, x, taps=True)
    for _ in range(2):
        got = ql.acoustic_model_forward(M, x, taps=("h_codes",))
        for l in range(5):
            assert torch.equal(got["layers"][l]["h_codes"], ref["layers"][l]["h_codes"]), l
        assert torch.equal(got["post"], ref["post"])


# Row groups of up to 16 rows: 16 of them share the chip with 32-cell tiles, 32
# with 64-cell tiles, several launches beyond.  Batches at the edges of these.
# The last columns: the kernel that runs, and over how many launches.
GROUP_CASES = [
    (2, 40, 48, 6, 2, "xrows4", 1),      # (two rows: the few-row layout)
    (5, 40, 36, 3, 5, "xstack32", 1),    # the smallest batch of five layers
    (5, 40, 36, 5, 15, "xstack32", 1),   # one group per layer, one row short
    (5, 40, 36, 2, 48, "xstack32", 1),   # the most rows of 5 layers in 32-cell tiles
    (5, 40, 48, 4, 49, "xstack64", 1),   # one row more: 64-cell tiles, 4 groups of 13
    (8, 24, 64, 5, 33, "xstack64", 1),   # 2 groups of 16 at most: 64-cell tiles, 3 of 11
    (3, 24, 100, 3, 48, "xstack32", 1),  # three full groups; tiles without cells
    (5, 40, 500, 3, 97, "xstack64", 2),  # one row more than a launch holds: 49 + 48
    (4, 512, 512, 2, 128, "xstack64", 1),  # a full launch at the widest
    (4, 24, 300, 3, 200, "xstack64", 2),  # two launches of 7 groups
    (5, 40, 400, 3, 200, "xstack64", 3),  # three launches: 67 + 67 + 66 rows
    # several launches of narrow layers, or of few frames, lose to k_stack
    (3, 24, 100, 4, 65, "spread", 1),
    (3, 320, 260, 3, 190, "spread", 1),
    (5, 24, 16, 3, 150, "spread", 1),
    (2, 24, 48, 3, 300, "spread", 1),
    (9, 24, 32, 3, 20, "xstack32", 1),   # more layers than one launch holds: 5 + 4
    (3, 40, 130, 1, 60, "xstack32", 1),  # one frame
    (5, 40, 130, 1, 60, "xstack64", 1),  # one frame in 64-cell tiles
]


@pytest.mark.parametrize("layers,n_in,H,T,B,layout,launches", GROUP_CASES)
def test_row_groups_equal_oracle(ql, orc, layers, n_in, H, T, B, layout, launches):
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, layers, states=40, seed=layers * 1000 + H + B)
    x = np.random.default_rng(B + H).standard_normal((T, B, n_in)).astype(np.float32)
    M = ql.quantize_model(w)
    assert ql.model_layout(M, T, B) == (layout, launches)
    g = ql.acoustic_model_forward(M, torch.from_numpy(x).cuda(), taps=True)
    o = orc.acoustic_model_forward(orc.quantize_model(w), x, taps=True)
    assert_model_taps(g, o, None, names=ql.TAP_NAMES)


@pytest.mark.parametrize("B,H,layout", [(3, 100, "xrows4"), (20, 100, "xstack32"), (100, 100, "spread"),
                                        (100, 500, "xstack64")])
def test_row_groups_carry_state(ql, B, H, layout):
    """Chunks of a sequence with the state carried give the whole call's bits."""
    from paper_1607_04683_amd.workloads import random_model
    M = ql.quantize_model(random_model(40, H, 5, states=32, seed=B))
    x = torch.randn(9, B, 40, device="cuda")
    whole = ql.acoustic_model_forward(M, x)["post"]
    state, parts = None, []
    for a, b in [(0, 1), (1, 5), (5, 9)]:
        assert ql.model_layout(M, b - a, B)[0] == layout
        out = ql.empty_state(M, B)
        parts.append(ql.acoustic_model_forward(M, x[a:b].contiguous(), state_in=state,
                                               state_out=out)["post"])
        state = out
    assert torch.equal(torch.cat(parts), whole)


def test_stack_forward_still_takes_one_launch_only(ql):
    """ql_lstm_stack_forward runs its layers and rows in one launch or says
    that it cannot; only the model forward splits the batch."""
    from paper_1607_04683_amd.workloads import random_model
    M = ql.quantize_model(random_model(40, 500, 5, states=32, seed=1))
    x = torch.randn(2, 150, 40, device="cuda")
    assert ql.stack_layers_per_launch(M, 2, 150) < 5
    with pytest.raises(ql.QLError, match="not supported"):
        ql.lstm_stack_forward(M.layers, ql.quantize_activations(x.reshape(300, 40)), 2, 150)


@pytest.mark.parametrize("layers,n_in,H,T,B", [
    (3, 512, 512, 2, 48),    # 32-cell tiles
    (5, 320, 500, 3, 96),    # 64-cell tiles
])
def test_first_frame_is_read_before_the_second_replaces_it(ql, orc, layers, n_in, H, T, B):
    """x_0 and x_1 share a buffer, and their values, zero points and recovery
    factors are far apart here, so a wave that multiplied or recovered x_0 after
    another had put x_1 there would change acc_x or the gates of frame 0."""
    from paper_1607_04683_amd.workloads import random_model
    w = random_model(n_in, H, layers, states=24, seed=layers + B)
    x = np.random.default_rng(B).standard_normal((T, B, n_in)).astype(np.float32)
    x[0] = 5.0 + 1e-3 * x[0]
    x[1] = -40.0 + 30.0 * x[1]
    M, xd = ql.quantize_model(w), torch.from_numpy(x).cuda()
    o = orc.acoustic_model_forward(orc.quantize_model(w), x, taps=True)
    for _ in range(4):
        assert_model_taps(ql.acoustic_model_forward(M, xd, taps=True), o, None,
                          names=("acc_x", "gates", "h_codes"))
