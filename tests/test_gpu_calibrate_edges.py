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


@pytest.mark.parametrize("n_tokens", [17_043_000, 17_100_008])
def test_factors_of_more_tokens_than_32_bit_offsets_reach(gpu, n_tokens):
    """64 channels x some 17 million tokens on both sides of the limit: row 63 of the activations begins 4.3 GB behind row 0.  Against
    the same factors from a Gram matrix that torch sums in fp64 (4096 partial sums of the same products: relative error some
    1e-14, the bound 1e-9 on the singular values as above)."""
    import torch
    d, r = 64, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X = torch.empty(d, n_tokens, dtype=torch.float32, device="cuda")
    for i in range(d):
        X[i].normal_(generator=g)
        X[i] *= 1.0 + 0.1 * i
    W = torch.randn(d, d, generator=g, device="cuda") * 0.02
    W_hat = (W * 16).round() / 16
    G = torch.zeros(d, d, dtype=torch.float64, device="cuda")
    for part in X.split(n_tokens // 64 + 1, dim=1):
        P = part.double()
        G += P @ P.T.contiguous()
    L = np.linalg.cholesky(G.cpu().numpy())
    dW = (W.double() - W_hat.double()).cpu().numpy()
    U, s, _ = np.linalg.svd(dW @ L)
    f64 = dict(dtype=torch.float64, device="cuda")
    B, A, sig = torch.empty(d, r, **f64), torch.empty(r, d, **f64), torch.empty(r, **f64)
    ws = torch.empty(gpu.factors_workspace_bytes(d, d, r), dtype=torch.uint8, device="cuda")
    gpu.factors(W, W_hat, X, B, A, sig, n_tokens, d, d, r, 1e-12, ws)
    assert np.allclose(sig.cpu().numpy(), s[:r], rtol=1e-9, atol=0)
    want = U[:, :r] @ (U[:, :r].T @ dW)                      # B'A = U' U'^T dW
    got = (B @ A).cpu().numpy()
    assert np.linalg.norm(got - want) <= 1e-8 * np.linalg.norm(want)


@pytest.mark.parametrize("route", [0, 1])
@pytest.mark.parametrize("d_in,d_out,r", [(256, 320, 40), (320, 192, 24), (640, 768, 32)])
def test_factors_of_a_well_conditioned_gram_to_rounding(gpu, d_in, d_out, r, route):
    """Roots, reciprocals and rotations to the last bits on either route: with independent channels (condition of the Gram matrix
    below 3) nothing amplifies an error.  Cholesky: the singular values agree to the rounding of the Gram matrix's sums of 16 d_in
    products, 16 * 640 * 1.1e-16 = 1.1e-12 at most.  Eigendecomposition: a row is replaced in each of some 80 rounds of up to 25
    sweeps by a sum of 16 products, 80 * 25 * 16 * 1.1e-16 = 3.5e-12 at most.  A root good to 1e-11 only would show."""
    import torch
    from oracle import calibrate
    rng = np.random.default_rng(d_in + d_out)
    W = rng.standard_normal((d_out, d_in)).astype(np.float32)
    W_hat = (np.round(W * 8) / 8).astype(np.float32)
    Xt = rng.standard_normal((d_in, 16 * d_in)).astype(np.float32)
    Wd, Whd, Xd = (torch.from_numpy(a).cuda() for a in (W, W_hat, Xt))
    f64 = dict(dtype=torch.float64, device="cuda")
    B, A, sig = torch.empty(d_out, r, **f64), torch.empty(r, d_in, **f64), torch.empty(r, **f64)
    ws = torch.empty(gpu.factors_workspace_bytes(d_in, d_out, r), dtype=torch.uint8, device="cuda")
    gpu.debug_set_factors_route(route)
    try:
        gpu.factors(Wd, Whd, Xd, B, A, sig, Xt.shape[1], d_in, d_out, r, 1e-12, ws)
    finally:
        gpu.debug_set_factors_route(0)
    Bo, _ = calibrate.eora_factors(W, W_hat, Xt, r)
    want = np.linalg.norm(Bo, axis=0)
    off = np.abs(sig.cpu().numpy() / want - 1).max()
    assert off <= (3.5e-12 if route else 1.1e-12)


@pytest.mark.parametrize("d,r,block", [(1024, 128, 256), (1536, 192, 384), (2048, 256, 512)])
def test_ritz_rotations_of_every_short_row(gpu, d, r, block):
    """Subspace iterations whose blocks are 256, 384 and 512 vectors (128: the shapes above): one instance each of the rounds over short
    rows.  The singular values and the correction against LAPACK on the Cholesky factor of the same Gram matrix (any square root gives
    the same factors); the bounds of the other calibration tests."""
    from tests.test_gpu_calibrate import _factors_with_stats, _inputs
    W, W_hat, Xt = _inputs(7700 + d, d, d, 2 * d)
    B, A, sig, st = _factors_with_stats(gpu, W, W_hat, Xt, r)
    assert 0 < st["subspace_cycles"] <= 6, st
    X = Xt.astype(np.float64)
    L = np.linalg.cholesky(X @ X.T)
    dW = W.astype(np.float64) - W_hat
    U, s, _ = np.linalg.svd(dW @ L, full_matrices=False)
    assert np.allclose(sig, s[:r], rtol=1e-9, atol=0), np.abs(sig / s[:r] - 1).max()
    want = U[:, :r] @ (U[:, :r].T @ dW)
    assert np.abs(B @ A - want).max() <= 1e-8 * np.abs(want).max()


@pytest.mark.parametrize("route", [0, 1])
@pytest.mark.parametrize("m,L", [
    (66, 98), (210, 386),                # pair rounds: lengths that are no multiples of 128
    (96, 128), (160, 256), (224, 384), (320, 512),       # block rounds over short rows
    (336, 640), (528, 1024),             # block rounds
])
def test_rows_the_sweeps_leave_are_orthogonal(gpu, m, L, route):
    """The sweeps end after one whose rotations were all small, without another that finds nothing left.  With more rows than columns in W
    and every component asked for, the columns of B' are the rows that the sweeps rotated, all of them.  Their cosines: a pair
    left alone is at most tol = sqrt(L) 1.1e-16 and later rotations of the sweep add 0.81 tol; the rounding of the product that was compared
    with tol is the rest of 2 tol."""
    import torch
    rng = np.random.default_rng(m + L)
    W = rng.standard_normal((L, m)).astype(np.float32)
    W_hat = (np.round(W * 8) / 8).astype(np.float32)
    Xt = rng.standard_normal((m, 16 * m)).astype(np.float32)
    Wd, Whd, Xd = (torch.from_numpy(a).cuda() for a in (W, W_hat, Xt))
    f64 = dict(dtype=torch.float64, device="cuda")
    B, A, sig = torch.empty(L, m, **f64), torch.empty(m, m, **f64), torch.empty(m, **f64)
    ws = torch.empty(gpu.factors_workspace_bytes(m, L, m), dtype=torch.uint8, device="cuda")
    gpu.debug_set_factors_route(route)
    try:
        st = gpu.factors(Wd, Whd, Xd, B, A, sig, Xt.shape[1], m, L, m, 1e-12, ws, stats=True)
    finally:
        gpu.debug_set_factors_route(0)
    rows = B.cpu().numpy().astype(np.longdouble)
    rows /= np.sqrt((rows * rows).sum(0))
    left = float(np.abs(rows.T @ rows - np.eye(m)).max())
    tol = np.sqrt(L) * 1.1102230246251565e-16
    assert st["svd_rows"] == (16 if m % 16 == 0 and L % 128 == 0 else 2)
    assert left <= 2 * tol, left / tol


@pytest.mark.parametrize("m,r,large", [(512, 32, 8), (768, 64, 8), (768, 64, 100), (1024, 64, 100)])
def test_leading_subspace_where_the_first_products_are_nearly_dependent(gpu, m, r, large):
    """Rows of the error a factor 1e4 larger than the rest, fewer of them than the block has vectors: the Gram matrix of a random block's first product
    with S (spread of its Ritz values 1e8) has no Cholesky factor in 64 bits.  The products after it mend that, and the iteration is
    not given up for the sweeps over all rows.  Bounds of the other calibration tests."""
    import torch
    rng = np.random.default_rng(m + r)
    W = rng.standard_normal((m, m)).astype(np.float32)
    Xt = rng.standard_normal((m, 2 * m)).astype(np.float32)
    W[:large] *= 1e4
    Wd, Xd = torch.from_numpy(W).cuda(), torch.from_numpy(Xt).cuda()
    f64 = dict(dtype=torch.float64, device="cuda")
    B, A, sig = torch.empty(m, r, **f64), torch.empty(r, m, **f64), torch.empty(r, **f64)
    ws = torch.empty(gpu.factors_workspace_bytes(m, m, r), dtype=torch.uint8, device="cuda")
    st = gpu.factors(Wd, torch.zeros_like(Wd), Xd, B, A, sig, Xt.shape[1], m, m, r, 1e-12, ws, stats=True)
    assert 0 < st["subspace_cycles"] <= 6, st
    X = Xt.astype(np.float64)
    U, s, _ = np.linalg.svd(W.astype(np.float64) @ np.linalg.cholesky(X @ X.T), full_matrices=False)
    assert np.allclose(sig.cpu().numpy(), s[:r], rtol=1e-9, atol=0)
    want = U[:, :r] @ (U[:, :r].T @ W.astype(np.float64))
    assert np.abs((B @ A).cpu().numpy() - want).max() <= 1e-8 * np.abs(want).max()


@pytest.mark.parametrize("d_in,d_out,r,parts", [
    (2176, 2176, 160, 2),        # 204 tiles, of the parts that fit the cheapest
    (2170, 2170, 160, 2),        # ragged rows, columns and contraction
    (2816, 2816, 192, 3),        # 264 tiles: more than one round of a workgroup a compute unit
])
def test_products_with_s_in_parts(gpu, d_in, d_out, r, parts):
    """Products of the subspace iteration's block with S of 65 tiles and more whose contraction is cut into parts, those that add to their output among
    them (the filter's): singular values and correction against LAPACK, the bounds of the other calibration tests."""
    from tests.test_gpu_calibrate import _factors_with_stats, _inputs
    m, p = min(d_in, d_out), (max(2 * r, r + 64) + 127) // 128 * 128
    assert gpu.debug_factors_parts(p, m, m, d_in * d_in - 2 * p * m - 3 * p * p) == parts
    W, W_hat, Xt = _inputs(7900 + d_in, d_in, d_out, 2 * d_in, group=d_in)
    B, A, sig, st = _factors_with_stats(gpu, W, W_hat, Xt, r)
    assert 0 < st["subspace_cycles"] <= 6, st
    X = Xt.astype(np.float64)
    dW = W.astype(np.float64) - W_hat
    T = dW @ np.linalg.cholesky(X @ X.T)
    lam, U = np.linalg.eigh(T @ T.T)                          # (fifty times faster than the SVD; good to 1e-16 lam_1 / lam_r)
    s, U = np.sqrt(lam[::-1][:r]), U[:, ::-1][:, :r]
    assert np.allclose(sig, s, rtol=1e-9, atol=0), np.abs(sig / s - 1).max()
    want = U @ (U.T @ dW)
    assert np.abs(B @ A - want).max() <= 1e-8 * np.abs(want).max()
