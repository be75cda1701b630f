"""The general kernel of the quantised backbone (5 and more tokens, and the shapes the decode kernel does not take) where
its tiling can go wrong: ragged last row groups, contractions that do not divide over a workgroup's ranges or over the
parts of a cut contraction, every number of token blocks and their remainders, coarse groups, several adapters, and a
workspace too small for a cut contraction.  Against the CPU oracle; the bound is the one of every forward kernel here
(fp32 accumulation and one fp16 rounding of y, 2^-11 of the larger of |y| and rms(y), with room for a sum's order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2410_21271_amd as eora
    return eora


def _check(y, ref):
    from oracle import linear
    assert np.isfinite(y).all()
    assert linear.y_error(y, ref) <= TOL


# w_bits, ab_bits, r, M, d_in, d_out, group
SHAPES = [
    (4, 16, 128, 5, 128, 16, 128),          # one tile, one row block, most ranges of a workgroup empty
    (3, 16, 32, 17, 384, 48, 128),          # two token blocks, the second with one token; three row blocks
    (4, 4, 64, 33, 640, 208, 128),          # third token block with one token; 13 row blocks: a ragged last group of every size
    (2, 16, 96, 64, 1152, 1040, 384),       # coarse groups that do not divide over the ranges
    (4, 16, 160, 65, 2688, 336, 2688),      # channel-wise, a second group of token blocks with one token
    (3, 3, 128, 127, 896, 144, 128),
    (4, 16, 512, 24, 14336, 4096, 128),     # contraction cut into parts, B's sixteen tiles shared out
    (3, 16, 96, 37, 7296, 2688, 128),       # parts of unequal length, fewer tiles of B than parts
    (4, 16, 0, 48, 8320, 1024, 128),        # bare, cut
    (4, 16, 128, 2, 2176, 1536, 128),       # few tokens, a shape the decode kernel does not take
    (2, 4, 256, 16, 11008, 272, 128),
    (4, 16, 96, 300, 1024, 256, 128),       # many tokens with a rank the GEMM path does not take: two launches
]


@pytest.mark.parametrize("w_bits,ab_bits,r,M,d_in,d_out,group", SHAPES)
def test_wide_edges(gpu, w_bits, ab_bits, r, M, d_in, d_out, group):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9000 + M + d_out, d_in, d_out, M, r, w_bits, group=group, ab_bits=ab_bits, packer=gpu)
    ws = gpu.new_workspace(M, d_in, d_out, r)
    y = run_linear_q(c, ws=ws)
    assert gpu.debug_last_launch().startswith(("wide_q", "resident")), gpu.debug_last_launch()
    _check(y, c.oracle_y())
    assert np.array_equal(y, run_linear_q(c, ws=ws))            # same workspace again: the same bits
    assert gpu.workspace_error(ws) == 0


def test_wide_group_of_four_ragged_members(gpu):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9200 + i, 2688, d, 39, 96, 3, packer=gpu) for i, d in enumerate((2688, 16, 528, 896))]
    for c, y in zip(cs, run_linear_q_group(cs, cs[0].x)):
        _check(y, c.oracle_y(x=cs[0].x))


def test_wide_group_cut_contraction(gpu):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9300 + i, 14336, d, 20, 64, 4, packer=gpu) for i, d in enumerate((1024, 1040))]
    for c, y in zip(cs, run_linear_q_group(cs, cs[0].x)):
        _check(y, c.oracle_y(x=cs[0].x))


def test_smaller_workspace_still_serves(gpu):
    """A buffer without room for partial outputs: the contraction stays whole; everything below that is refused."""
    import torch
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9400, 14336, 256, 40, 128, 4, packer=gpu)
    full = gpu.workspace_bytes(40, 14336, 256, 128)
    small = full - (12 << 20)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    gpu.workspace_init(ws)
    _check(run_linear_q(c, ws=ws), c.oracle_y())
    with pytest.raises(gpu.EoraError) as e:
        run_linear_q(c, ws=ws[: small - 256])
    assert e.value.status == -5


def test_infinities_stay_in_their_token(gpu):
    """A token with an infinite activation does not disturb the others, whatever ranges and token blocks they share."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9500, 1152, 144, 21, 32, 4, packer=gpu)
    ref = c.oracle_y()
    x = c.x.copy()
    x[7, 300] = np.inf
    y = run_linear_q(c, x=x)
    keep = np.arange(21) != 7
    _check(y[keep], ref[keep])
    assert not np.isfinite(y[7]).any()
