"""The GEMM for many tokens where its tiles and its requests end: workgroups of 128, 192 and 256 tokens (the rule takes the
larger ones for launches of many row tiles), contractions of one and two quantisation groups, scales read eight groups at a
time and one by one, parts that begin within eight groups.  Against the CPU oracle on sampled token rows with the bound of
the many-token path (2e-3: t and the dequantised weight are rounded to fp16 once, y once)."""
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


# w_bits, ab_bits, r, M, d_in, d_outs, group
@pytest.mark.parametrize("w_bits,ab_bits,r,M,d_in,d_outs,group", [
    (4, 16, 128, 1300, 256, (14336, 14288), 128),     # 256 tokens: the last token tile has 20, the last row tile 208 rows
    (3, 4, 128, 1281, 1024, (28656,), 128),           # 256 tokens, one in the last tile
    (2, 16, 0, 1537, 128, (16384, 12288), 128),       # 256 tokens, one group: no step of the main loop
    (4, 3, 256, 379, 384, (14336, 14320), 384),       # 192 tokens, channel-wise
    (3, 16, 256, 193, 1024, (28672, 16), 128),        # 192 tokens, one in the last tile; a member of one row block
    (4, 16, 128, 128, 128, (16,), 128),               # 128 tokens, the smallest launch
    (2, 4, 128, 255, 2048, (272, 16), 1024),          # 128 tokens, groups of eight tiles
    (3, 3, 128, 130, 3072, (528,), 128),              # parts that begin within eight groups
    (4, 16, 128, 200, 14336, (272,), 128),            # t in many parts, the last of them shorter
    (3, 4, 256, 131, 8320, (16, 272), 128),           # the same for two members, 65 groups
    (4, 16, 128, 1500, 2048, (528,), 128),            # parts beyond 1024 tokens
    (4, 16, 256, 1700, 8192, (4112,), 128),           # parts that take the room of t's parts as well
    (2, 16, 128, 2047, 256, (4096,), 128),            # 128 tokens, every compute unit busy, the last token missing
])
def test_prefill_tiles(gpu, w_bits, ab_bits, r, M, d_in, d_outs, group):
    from oracle import linear
    from tests.cases import QCase
    from tests.gpu_util import run_linear_q_group
    cs = [QCase(9900 + M + i, d_in, d, M, r, w_bits, group=group, ab_bits=ab_bits, packer=gpu) for i, d in enumerate(d_outs)]
    ys = run_linear_q_group(cs, cs[0].x)
    assert gpu.debug_last_launch().startswith("prefill "), gpu.debug_last_launch()
    rows = np.unique(np.concatenate([np.array([0, 15, 16, 63, 64, 127, M // 2, M - 2, M - 1]), np.random.default_rng(M).integers(0, M, 16)]))
    for c, y in zip(cs, ys):
        assert np.isfinite(y).all()
        assert linear.y_error(y[rows], c.oracle_y(rows=rows, x=cs[0].x)) <= TOL
