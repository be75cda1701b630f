"""The GEMM for many tokens where its tiles and its requests end: workgroups of 128, 192 and 256 tokens (the rule takes the
larger ones for launches of many row tiles), every instance of them, contractions of one and two quantisation groups, scales
read eight groups at a time and one by one, groups of several tiles, parts that begin within eight groups.  Every row names the
kernel that it is meant for (the one for launches of few tiles is "prefill128"), and the launch has to have taken it.  Against
the CPU oracle on sampled token rows with the bound of the many-token path (2e-3: t and the dequantised weight are rounded to
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


def _check(gpu, w_bits, ab_bits, r, M, d_in, d_outs, group, kernel, tokens, parts):
    from oracle import linear
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9900 + M + i, d_in, d, M, r, w_bits, group=group, ab_bits=ab_bits, packer=gpu) for i, d in enumerate(d_outs)]
    ys = run_linear_q_group(cs, cs[0].x)
    assert gpu.debug_last_prefill() == "%s tokens=%d" % (kernel, tokens)
    assert "ksplit=%d " % parts in gpu.debug_last_launch(), gpu.debug_last_launch()
    rows = np.unique(np.concatenate([np.array([0, 15, 16, 63, 64, 127, M // 2, M - 2, M - 1]), np.random.default_rng(M).integers(0, M, 16)]))
    for c, y in zip(cs, ys):
        assert np.isfinite(y).all()
        assert linear.y_error(y[rows], c.oracle_y(rows=rows, x=cs[0].x)) <= TOL


# w_bits, ab_bits, r, M, d_in, d_outs, group, kernel, its tokens, parts
@pytest.mark.parametrize("w_bits,ab_bits,r,M,d_in,d_outs,group,kernel,tokens,parts", [
    (4, 16, 128, 1300, 512, (14336, 14288), 128, "prefill", 256, 1),      # the last token tile has 20, the last row tile 208 rows
    (3, 4, 128, 1281, 1024, (28656,), 128, "prefill", 256, 1),            # one token in the last tile, scales of eight groups at once
    (2, 16, 128, 250, 128, (32752, 32768), 128, "prefill", 256, 1),       # one group: no step of the main loop
    (2, 16, 0, 1537, 128, (16384, 12288), 128, "prefill", 192, 1),        # the same, one token in the last tile
    (4, 3, 256, 379, 384, (14336, 14320), 384, "prefill", 192, 1),        # channel-wise
    (3, 16, 128, 1281, 1536, (14320,), 384, "prefill", 192, 1),           # four groups of three tiles
    (3, 16, 128, 1281, 4096, (2064,), 512, "prefill", 192, 4),            # the same in parts: two groups of four tiles each
    (4, 4, 128, 1700, 7168, (1040,), 1024, "prefill", 256, 7),            # one group of eight tiles a part
    (3, 16, 128, 1700, 4096, (2560,), 128, "prefill", 256, 3),            # parts that begin at groups 10 and 21, eight groups at a time
    (4, 16, 0, 1000, 5120, (3088,), 128, "prefill", 256, 4),              # at groups 10, 20 and 30
    (2, 16, 0, 1000, 6656, (2064,), 128, "prefill", 256, 6),              # 52 groups one by one, parts of eight and nine
    (3, 16, 256, 193, 1024, (28672, 16), 128, "prefill128", 128, 1),      # a member of one row block
    (4, 16, 128, 128, 128, (16,), 128, "prefill128", 128, 1),             # the smallest launch
    (2, 4, 128, 255, 2048, (272, 16), 1024, "prefill128", 128, 4),        # groups of eight tiles in parts
    (3, 3, 128, 130, 3072, (528,), 128, "prefill128", 128, 6),
    (4, 16, 128, 200, 14336, (272,), 128, "prefill128", 128, 8),          # t in many parts, the last of them shorter
    (3, 4, 256, 131, 8320, (16, 272), 128, "prefill128", 128, 8),         # the same for two members, 65 groups
    (4, 16, 128, 1500, 2048, (528,), 128, "prefill128", 128, 4),          # parts beyond 1024 tokens
    (4, 16, 256, 1700, 8192, (4112,), 128, "prefill", 256, 2),            # parts that take the room of t's parts as well
    (2, 16, 128, 2047, 256, (4096,), 128, "prefill", 128, 1),             # every compute unit busy, the last token missing
])
def test_prefill_tiles(gpu, w_bits, ab_bits, r, M, d_in, d_outs, group, kernel, tokens, parts):
    _check(gpu, w_bits, ab_bits, r, M, d_in, d_outs, group, kernel, tokens, parts)


@pytest.mark.parametrize("tokens,M,d_out", [(128, 2047, 4096), (192, 300, 28656), (256, 385, 28656)])
@pytest.mark.parametrize("ab_bits", [None, 16, 4, 3])
@pytest.mark.parametrize("w_bits", [4, 3, 2])
def test_every_instance(gpu, w_bits, ab_bits, tokens, M, d_out):
    _check(gpu, w_bits, ab_bits or 16, 128 if ab_bits else 0, M, 256, (d_out,), 128, "prefill", tokens, 1)
