"""Prompts whose contraction is cut into parts in different workgroups (few output tiles): parts of unequal length, the
low-rank columns in the last part, ragged tokens and rows, groups, several adapters, and a workspace without room for the
parts.  Against the CPU oracle with the bound of the many-token path (2e-3: t and the dequantised weight are rounded to
fp16 once, y once)."""
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


def _parts(gpu):
    s = gpu.debug_last_launch()
    assert s.startswith("prefill "), s
    return int(s.split("ksplit=")[1].split()[0])


# w_bits, ab_bits, r, M, d_in, d_out, group
@pytest.mark.parametrize("w_bits,ab_bits,r,M,d_in,d_out,group", [
    (4, 16, 128, 128, 1152, 272, 128),       # nine steps over two parts, a ragged row tile
    (3, 4, 256, 129, 2688, 1040, 128),       # one token in the last tile, 21 steps
    (2, 3, 128, 300, 4096, 48, 4096),        # channel-wise, three row blocks
    (4, 16, 0, 200, 7296, 512, 128),         # bare
    (4, 16, 512, 140, 3072, 256, 384),       # as many low-rank columns as a part has
])
def test_prefill_in_parts(gpu, w_bits, ab_bits, r, M, d_in, d_out, group):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9700 + M, d_in, d_out, M, r, w_bits, group=group, ab_bits=ab_bits, packer=gpu)
    ws = gpu.new_workspace(M, d_in, d_out, r)
    y = run_linear_q(c, ws=ws)
    assert _parts(gpu) > 1
    _check(y, c.oracle_y())
    assert np.array_equal(y, run_linear_q(c, ws=ws))
    # a workspace without room for the parts: whole contraction
    small = ws[: ws.numel() - (48 << 20)]
    y1 = run_linear_q(c, ws=small)
    assert _parts(gpu) == 1
    _check(y1, c.oracle_y())


def test_prefill_group_in_parts(gpu):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9800 + i, 2176, d, 131, 128, 4, packer=gpu) for i, d in enumerate((528, 16, 272))]
    ys = run_linear_q_group(cs, cs[0].x)
    assert _parts(gpu) > 1
    for c, y in zip(cs, ys):
        _check(y, c.oracle_y(x=cs[0].x))


def test_few_token_group_of_a_general_shape_is_one_launch(gpu):
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9900 + i, 1152, d, 3, 96, 3, packer=gpu) for i, d in enumerate((528, 2064))]
    ys = run_linear_q_group(cs, cs[0].x)
    assert gpu.debug_last_launch().endswith("n=2"), gpu.debug_last_launch()
    for c, y in zip(cs, ys):
        _check(y, c.oracle_y(x=cs[0].x))


def test_workspace_of_a_long_prompt_serves_short_ones_alike(gpu):
    """A workspace sized for the longest prompt gives shorter calls what one of their own size gives them: parts, and the
    same bits.  Also for a group, and from 5 to 127 tokens."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q, run_linear_q_group
    big = gpu.new_workspace(5000, 4096, 272, 128, n_members=2)
    c = QCase(9950, 4096, 272, 333, 128, 4, packer=gpu)
    y = run_linear_q(c, ws=big)
    assert _parts(gpu) > 1
    assert np.array_equal(y, run_linear_q(c))
    _check(y, c.oracle_y())
    cs = [QCase(9960 + i, 4096, d, 140, 128, 3, packer=gpu) for i, d in enumerate((272, 80))]
    ys = run_linear_q_group(cs, cs[0].x, ws=big)
    assert _parts(gpu) > 1
    for a, b, q in zip(ys, run_linear_q_group(cs, cs[0].x), cs):
        assert np.array_equal(a, b)
        _check(a, q.oracle_y(x=cs[0].x))
    w = [QCase(9970 + i, 16640, d, 40, 128, 4, packer=gpu) for i, d in enumerate((272, 80))]
    import torch
    only = torch.empty(gpu.workspace_bytes_group(40, 16640, 128, 2) + 4 * 4 * 40 * 272, dtype=torch.uint8, device="cuda")      # (and what a 2:4 call of a member would ask for)
    gpu.workspace_init(only)
    for ws in (only, big):
        ys = run_linear_q_group(w, w[0].x, ws=ws)
        assert "parts=" in gpu.debug_last_launch(), gpu.debug_last_launch()
        for y, q in zip(ys, w):
            _check(y, q.oracle_y(x=w[0].x))


@pytest.mark.parametrize("groups", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 17, 18, 33])
def test_parts_of_the_down_projection_add_up(gpu, groups):
    """The sum of t's parts takes three or eight of them at a time: every remainder, with one part per quantisation group."""
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q
    c = QCase(9990 + groups, 128 * groups, 16, 130, 128, 4, packer=gpu)
    ws = gpu.new_workspace(130, 128 * groups, 16, 128)
    assert gpu.debug_prefill_plan(130, 128 * groups, [16], 128, ws.numel())[2] == groups
    _check(run_linear_q(c, ws=ws), c.oracle_y())
