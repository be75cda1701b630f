"""Algorithm 1 steps 1-6 where the fp64 products and the factorisation end: rows, columns and contractions that are no multiples
of the 64 x 64 tile, of its stages of 32 and of the 16 x 16 blocks of a diagonal block, on both sides of each; contractions cut
into parts (long ones with few tiles: the block of vectors of a subspace iteration).  Against the numpy oracle with the
bounds of the other calibration tests (1e-9 on the singular values, 1e-8 on the product: fp64 on both sides, condition of
the Gram matrix up to 2e6)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2410_21271_amd as eora
    return eora


@pytest.mark.parametrize("d_in,d_out,n_tokens,r", [
    (62, 66, 131, 3),           # below and above one tile; contraction of one stage less two, more than four stages by three
    (66, 62, 129, 5),
    (64, 80, 127, 7),           # one block of 64, a multiple of 16 behind it
    (98, 34, 193, 4),           # 98 = 64 + 34: a diagonal block of two blocks of 16 and two rows
    (130, 418, 261, 9),
    (210, 142, 417, 11),
    (578, 578, 1025, 13),       # subspace iteration over a ragged T (blocks of 128 vectors)
    (514, 770, 1031, 16),
])
def test_factors_of_ragged_shapes(gpu, d_in, d_out, n_tokens, r):
    from tests.test_gpu_calibrate import _compare, _inputs, _run
    W, W_hat, Xt = _inputs(7100 + d_in + d_out, d_in, d_out, n_tokens, group=d_in)
    B, A, sig = _run(gpu, W, W_hat, Xt, r)
    _compare(W, W_hat, Xt, r, B, A, sig)
