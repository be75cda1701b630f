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
    (4, 16, 512, 24, 14336, 4096, 128),     # whole contraction at the largest rank: t of two token blocks fills the LDS
    (3, 16, 96, 37, 7296, 2688, 128),       # three token blocks, the last ragged
    (4, 16, 0, 48, 8320, 1024, 128),        # bare
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


def _parts(gpu):
    """(parts of the contraction in different workgroups, segments of the longest part) of the last launch."""
    s = gpu.debug_last_launch()
    assert s.startswith("wide_q "), s
    if "parts=" not in s:
        return 1, 1
    return int(s.split("parts=")[1].split()[0]), int(s.split("segments=")[1].split()[0])


# w_bits, ab_bits, r, M, d_in, d_out, group
CUT = [
    (3, 16, 96, 37, 17024, 784, 128),       # parts of unequal length, fewer tiles of B than parts
    (4, 16, 0, 48, 16768, 1024, 128),       # bare
    (4, 16, 512, 24, 16640, 512, 128),      # sixteen tiles of B shared out over the parts
    (4, 4, 512, 40, 16640, 272, 128),       # 4-bit factors: four tiles of B, some parts without one; a ragged row group
    (2, 4, 64, 24, 16640, 512, 16640),      # rank 64 in 4 bits: a single tile of B; channel-wise
    (3, 3, 128, 33, 17408, 80, 128),        # 3-bit factors
    (4, 16, 64, 12, 16384, 64, 256),        # one token block
    (2, 3, 128, 9, 17920, 96, 128),
    (3, 4, 256, 5, 28672, 48, 256),
    (4, 16, 128, 70, 16640, 256, 128),      # a second group of token blocks, ragged
]


@pytest.mark.parametrize("w_bits,ab_bits,r,M,d_in,d_out,group", CUT)
def test_wide_cut_contraction(gpu, w_bits, ab_bits, r, M, d_in, d_out, group):
    """The contraction in parts in different workgroups, summed by a second kernel: every share [g0, g1) of B's tiles."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9600 + M + d_out, d_in, d_out, M, r, w_bits, group=group, ab_bits=ab_bits, packer=gpu)
    ws = gpu.new_workspace(M, d_in, d_out, r)
    y = run_linear_q(c, ws=ws)
    assert _parts(gpu)[0] > 1, gpu.debug_last_launch()
    _check(y, c.oracle_y())
    assert np.array_equal(y, run_linear_q(c, ws=ws))
    assert gpu.workspace_error(ws) == 0


def test_wide_cut_contraction_several_adapters(gpu):
    from oracle import linear
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_multi
    M, n, r = 24, 4, 64
    c = QCase(9650, 16640, 512, M, n * r, 4, packer=gpu)
    sel = (np.arange(M) % (n + 1) - 1).astype(np.int32)
    y = run_linear_q_multi(c, sel, r)
    assert _parts(gpu)[0] > 1, gpu.debug_last_launch()
    _check(y, linear.eora_linear_q_multi(c.x, c.o_qw, c.o_sc, c.o_qz, c.o_A, c.o_B, c.o_As, c.o_Bs, sel, M, c.d_in, c.d_out, r, n,
                                         c.w_bits, c.group, c.ab_bits))


@pytest.mark.parametrize("w_bits,r,M,d_in,group", [
    (4, 32, 40, 53632, 128),                # 400 + 19 tiles; an odd number of groups: scales one by one
    (3, 0, 35, 57344, 256),                 # 400 + 48 tiles of coarse groups, eight scales at a time
    (2, 32, 64, 54272, 53 * 128),           # a group of 53 tiles across the border of the segments
])
def test_wide_scales_in_segments(gpu, w_bits, r, M, d_in, group):
    """A contraction longer than the scales that fit the LDS (and a workspace without room for parts, which would be
    shorter): segment after segment."""
    import torch
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9700 + M, d_in, 48, M, r, w_bits, group=group, packer=gpu)
    need = gpu.workspace_bytes(M, d_in, 48, r) - (12 << 20) + 4 * 4 * M * 48      # (a 2:4 call of that shape would put its parts there)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    gpu.workspace_init(ws)
    y = run_linear_q(c, ws=ws)
    assert _parts(gpu) == (1, 2), gpu.debug_last_launch()
    _check(y, c.oracle_y())
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
    ys = run_linear_q_group(cs, cs[0].x)
    assert _parts(gpu)[0] > 1, gpu.debug_last_launch()
    for c, y in zip(cs, ys):
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


def test_smaller_workspace_leaves_the_contraction_whole(gpu):
    """The same linear with and without room for partial outputs: in parts, and whole."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9420, 14336, 1024, 40, 128, 4, packer=gpu)
    ws = gpu.new_workspace(40, 14336, 1024, 128)
    _check(run_linear_q(c, ws=ws), c.oracle_y())
    assert _parts(gpu)[0] > 1
    _check(run_linear_q(c, ws=ws[: ws.numel() - 256]), c.oracle_y())
    assert _parts(gpu)[0] == 1


@pytest.mark.parametrize("M,d_in,d_out,r,w_bits,ab_bits", [
    (33, 640, 9216, 32, 3, 16),             # one group, its last block with one token
    (48, 256, 20480, 64, 4, 4),             # full; two row blocks per wavefront; a single tile per range
    (65, 384, 6160, 96, 2, 16),             # two groups, the second with two blocks; an odd number of chunks, a ragged last row group
    (96, 16640, 2048, 0, 4, 16),            # parts of a long contraction
    (48, 14336, 4096, 64, 4, 16),           # ... with factors: seven, of eight row blocks each
    (144, 256, 4112, 32, 4, 16),            # three groups, the most tokens that take three blocks
    (40, 384, 9232, 128, 3, 3),             # 3-bit factors; a ragged last row group
])
def test_wide_three_token_blocks(gpu, M, d_in, d_out, r, w_bits, ab_bits):
    """33..48, 65..96 and 129..144 tokens: three token blocks per workgroup."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9460 + M, d_in, d_out, M, r, w_bits, ab_bits=ab_bits, packer=gpu)
    ws = gpu.new_workspace(M, d_in, d_out, r)
    y = run_linear_q(c, ws=ws)
    assert " TB=3 " in gpu.debug_last_launch(), gpu.debug_last_launch()
    assert (M, d_in) != (48, 14336) or " parts=7 " in gpu.debug_last_launch(), gpu.debug_last_launch()
    _check(y, c.oracle_y())
    assert np.array_equal(y, run_linear_q(c, ws=ws))


@pytest.mark.parametrize("M,d_in,d_outs,r,w_bits,ab_bits", [
    (37, 512, (4096, 4112, 1040), 32, 4, 16),            # ragged members
    (96, 256, (2048, 4096, 2064), 128, 3, 3),            # two groups of token blocks
    (48, 384, (8192, 8208), 0, 2, 16),
])
def test_wide_three_token_blocks_in_a_group(gpu, M, d_in, d_outs, r, w_bits, ab_bits):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cases = [QCase(9500 + M + i, d_in, d, M, r, w_bits, ab_bits=ab_bits, packer=gpu) for i, d in enumerate(d_outs)]
    ys = run_linear_q_group(cases, cases[0].x)
    launch = gpu.debug_last_launch()
    assert launch.startswith("wide_q ") and " TB=3 " in launch and launch.endswith(" n=%d" % len(cases)), launch
    for c, y in zip(cases, ys):
        _check(y, c.oracle_y(x=cases[0].x))


@pytest.mark.parametrize("M,d_in,d_out,r,n", [(40, 512, 9216, 32, 4), (90, 256, 6160, 64, 3)])
def test_wide_three_token_blocks_with_several_adapters(gpu, M, d_in, d_out, r, n):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_multi
    from tests.test_gpu_multi import _oracle
    c = QCase(9540 + M, d_in, d_out, M, r * n, 4, packer=gpu)
    sel = np.random.default_rng(M).integers(-1, n, M).astype(np.int32)
    y = run_linear_q_multi(c, sel, r)
    assert " TB=3 " in gpu.debug_last_launch(), gpu.debug_last_launch()
    _check(y, _oracle(c, sel, r))


# M, d_in, d_outs, r, w_bits, ab_bits, token blocks and row groups of a workgroup
FEWER_BLOCKS = [
    (33, 4096, (1024,), 64, 4, 16, 1, 1),                # three groups of one token block, the last with one token
    (24, 1152, (272,), 0, 3, 16, 1, 1),                  # two groups
    (48, 2688, (2688,), 0, 4, 16, 1, 2),                 # two row blocks
    (40, 2048, (4080,), 32, 2, 16, 1, 4),                # four, the last row group ragged
    (127, 2048, (528,), 128, 4, 4, 1, 2),                # eight groups
    (100, 2048, (2688,), 128, 4, 3, 2, 4),               # four groups of two token blocks, one token block in the last
    (64, 4096, (4096, 1024, 1024), 128, 4, 16, 2, 4),    # a group of members
    (256, 1024, (528,), 96, 4, 16, 1, 4),                # sixteen groups: the most of a launch
]


@pytest.mark.parametrize("M,d_in,d_outs,r,w_bits,ab_bits,tb,nwr", FEWER_BLOCKS)
def test_wide_small_launches_take_fewer_token_blocks(gpu, M, d_in, d_outs, r, w_bits, ab_bits, tb, nwr):
    """Small launches: several groups of one or two token blocks, each with workgroups and producers of its own."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9430 + i + M, d_in, d, M, r, w_bits, ab_bits=ab_bits, packer=gpu) for i, d in enumerate(d_outs)]
    ws = gpu.new_workspace(M, d_in, max(d_outs), r, n_members=len(cs))
    ys = run_linear_q_group(cs, cs[0].x, ws=ws)
    assert " NWR=%d " % nwr in gpu.debug_last_launch() and " TB=%d " % tb in gpu.debug_last_launch(), gpu.debug_last_launch()
    for c, y, y2 in zip(cs, ys, run_linear_q_group(cs, cs[0].x, ws=ws)):
        _check(y, c.oracle_y(x=cs[0].x))
        assert np.array_equal(y, y2)
    assert gpu.workspace_error(ws) == 0


@pytest.mark.parametrize("w_bits,ab_bits,r,M,d_in,d_out,group,nwr", [
    (4, 4, 64, 1, 1024, 1024, 128, 1),
    (3, 16, 32, 4, 128, 48, 128, 4),                     # a single tile: one range without one
    (2, 3, 128, 3, 1664, 1040, 128, 1),
    (4, 16, 0, 3, 1152, 16, 1152, 1),                    # bare, channel-wise
    (4, 16, 96, 2, 1152, 9232, 128, 2),                  # two row blocks, the last row group ragged
    (3, 4, 128, 4, 640, 9216, 128, 2),
    (2, 16, 0, 1, 384, 9232, 128, 2),
    (4, 16, 32, 2, 384, 24592, 128, 4),                  # four, the last row group ragged
    (3, 3, 128, 4, 256, 24576, 128, 4),
    (4, 16, 64, 3, 34816, 32, 128, 1),                   # longer than one order is kept for
])
def test_wide_few_tokens(gpu, w_bits, ab_bits, r, M, d_in, d_out, group, nwr):
    """One to four tokens: four of a token block's sixteen rows are all that is read, with every split of a workgroup."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9900 + M + d_out, d_in, d_out, M, r, w_bits, group=group, ab_bits=ab_bits, packer=gpu)
    ws = gpu.new_workspace(M, d_in, d_out, r)
    y = run_linear_q(c, ws=ws)
    assert " NWR=%d " % nwr in gpu.debug_last_launch() and _parts(gpu) == (1, 1), gpu.debug_last_launch()
    _check(y, c.oracle_y())
    assert np.array_equal(y, run_linear_q(c, ws=ws))
    assert gpu.workspace_error(ws) == 0


@pytest.mark.parametrize("M,d_outs,r", [(257, (272,), 96), (259, (272, 144, 16), 96), (515, (48, 32), 160)])
def test_wide_last_launch_of_few_tokens(gpu, M, d_outs, r):
    """Ranks the GEMM path does not take: launches of 256 tokens, the last with one to three."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9990 + i, 640, d, M, r, 4, packer=gpu) for i, d in enumerate(d_outs)]
    for c, y in zip(cs, run_linear_q_group(cs, cs[0].x)):
        _check(y, c.oracle_y(x=cs[0].x))


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
