"""The eigensolver over spectra where a tridiagonal solver can go wrong: multiple and nearly multiple eigenvalues,
matrices that fall apart, dead channels, rank-deficient Keys, entries near the ends of the fp32 range; and the
Jacobi solver (plain kernels) on the same matrices.

Bounds: the eigenvectors come out of double arithmetic and are rounded once to fp32, so R^T R and R^T C R carry at most
128 rounded entries per element: 2^-24 * 2 * sqrt(128) in the Frobenius sense, times sqrt(128) for the largest element
of R^T R; eigenvalues 2^-24 of the largest (their own rounding) plus the 6.4e-11 that the solver may shift them by.
Jacobi in fp32 is held to the solver's documented 1e-5."""
import numpy as np
import pytest
import torch

import paper_2605_19218_amd as rk

from gpu_util import D, DEV, Pipeline, to_dev, to_host

pytestmark = pytest.mark.gpu
rng = np.random.default_rng(77)


def recipe(L, noise=0.1, hot=10.0):
    K = rng.standard_normal((L, 16)) @ rng.standard_normal((16, D)) + noise * rng.standard_normal((L, D))
    K[:, [5, 90]] *= hot
    return K


def root(C):
    """Keys whose scatter is C."""
    w, v = np.linalg.eigh((C + C.T) / 2)
    return (v * np.sqrt(np.maximum(w, 0.0))).T


def dead_channels():
    K = recipe(600)
    K[:, 40:90] = 0.0
    return K


def glued():
    m = np.abs(np.arange(D) % 21 - 10.0)
    e = np.ones(D - 1)
    e[20::21] = 1e-6
    return root(np.diag(m) + np.diag(e, 1) + np.diag(e, -1) + 2 * np.eye(D))


def hadamard():
    h = np.ones((1, 1))
    while h.shape[0] < D:
        h = np.block([[h, h], [h, -h]])
    return np.vstack([h + 12 * np.eye(D)])


KEYS = {
    "recipe": lambda: recipe(3000),
    "fewer_rows_than_channels": lambda: recipe(64),
    "one_row": lambda: recipe(1),
    "two_rows": lambda: recipe(2),
    "rank_16": lambda: recipe(500, noise=0.0),
    "dead_channels": dead_channels,
    "one_live_pair": lambda: np.eye(D)[[3, 100]] * 2.0 + np.eye(D)[[100, 3]],
    "identity_plus_rank_one": lambda: np.vstack([10 * np.eye(D), rng.integers(-3, 4, D).astype(float)]),
    "all_ones": lambda: np.ones((3, D)),
    "equal_blocks": lambda: np.kron(np.eye(8), rng.standard_normal((16, 16))),
    "hadamard_clusters": hadamard,
    "glued_wilkinson": glued,
    "toeplitz": lambda: root(0.95 ** np.abs(np.subtract.outer(np.arange(D), np.arange(D)))),
    "flat": lambda: rng.standard_normal((20000, D)),
    "graded": lambda: np.diag(2.0 ** -np.arange(0, 32, 0.25)) @ np.linalg.qr(rng.standard_normal((D, D)))[0],
    "large_entries": lambda: recipe(200) * 1e15,
    "small_entries": lambda: recipe(200) * 1e-15,
}


@pytest.fixture(scope="module")
def ctx():
    c = rk.rk_create(0)
    yield c
    rk.rk_destroy(c)


def solve(ctx, K, sigma=None):
    K = K.astype(np.float32)[None, None]
    p = Pipeline(ctx, 1, 1, 1, 24, "f32", K.shape[2])
    sg = None if sigma is None else to_dev(sigma[None, None], "f32")
    p.fit(to_dev(K, "f32"), K.shape[2], sigma=sg, center=False)
    C = to_host(p.cov)[0, 0]
    if sigma is not None:
        C = C * np.outer(sigma, sigma)
    return to_host(p.R)[0, 0], to_host(p.lam)[0, 0], C, int(p.sweeps.cpu()[0, 0]), p


@pytest.mark.parametrize("name", list(KEYS))
def test_spectra(ctx, name):
    sigma = None
    if name == "recipe":
        sigma = (np.abs(rng.standard_normal(D)) + 0.25).astype(np.float32).astype(np.float64)
    K = KEYS[name]()
    R, lam, C, sweeps, p = solve(ctx, K, sigma)
    eps = 2.0 ** -24
    assert sweeps == 1
    assert np.abs(R.T @ R - np.eye(D)).max() <= 2 * eps * np.sqrt(D)
    assert np.linalg.norm(R.T @ C @ R - np.diag(lam)) <= 4 * eps * np.sqrt(D) * np.linalg.norm(C)
    want = np.linalg.eigvalsh(C)
    assert np.abs(np.sort(lam) - want).max() <= 1.5 * eps * np.abs(want).max() + 2e-10 * np.linalg.norm(C)
    keep, mask = p.keep_idx.cpu().numpy()[0, 0], p.mask.cpu().numpy()[0, 0]
    order = np.lexsort((np.arange(D), -lam))[:24]
    assert np.array_equal(keep, order) and np.array_equal(np.flatnonzero(mask), np.sort(order))


@pytest.mark.parametrize("name", ["recipe", "dead_channels", "equal_blocks", "one_live_pair"])
def test_jacobi(ctx, name):
    rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, 1)
    try:
        R, lam, C, sweeps, _ = solve(ctx, KEYS[name]())
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, 0)
    assert 1 <= sweeps < 20
    assert np.abs(R.T @ R - np.eye(D)).max() <= 1e-5
    assert np.linalg.norm(R.T @ C @ R - np.diag(lam)) <= 1e-5 * np.linalg.norm(C)


# A matrix whose tridiagonal form takes the solver's own shift of its diagonal back: a dense 4 x 4 block, and diagonal entries
# that the shift brings to within `gap` of each other.  Vectors of equal eigenvalues become one, which only the check behind
# the reduction can see; the matrix then goes to Jacobi.
@pytest.mark.parametrize("gap", [0.0, 1e-15, 4e-15, 1e-14, 1e-13, 1e-12])
def test_coinciding_eigenvalues(ctx, gap):
    block = np.random.default_rng(5).standard_normal((6, D))
    block[:, 4:] = 0.0
    block *= np.sqrt(0.7 / np.linalg.norm(block.T @ block))           # Frobenius norm in [1/2, 1): the solver's scale is 1
    i = np.arange(4, D)
    single = np.zeros((D - 4, D))
    single[i - 4, i] = np.sqrt(7e-11 - 5e-13 * (37 * i % D) + gap * (i - 4))
    R, lam, C, sweeps, p = solve(ctx, np.vstack([block, single]))
    if gap == 0.0:
        assert 1 < sweeps < 20
    assert np.abs(R.T @ R - np.eye(D)).max() <= 1e-5
    assert np.linalg.norm(R.T @ C @ R - np.diag(lam)) <= 1e-5 * np.linalg.norm(C)
    keep = p.keep_idx.cpu().numpy()[0, 0]
    assert np.array_equal(keep, np.lexsort((np.arange(D), -lam))[:24])
    assert np.array_equal(to_host(p.Rr)[0, 0], R[:, keep])


# Neighbours on both sides of the distance below which a vector takes a second round, in a chain beside a dense block.  The chain's
# entries are squares of fp32 numbers, 2e-6 and up: rounded by 2e-13 of the norm, a twentieth of the smallest gap.
@pytest.mark.parametrize("gap", [3e-9, 1e-10, 2e-11, 7e-12, 4e-12])
def test_close_eigenvalues(ctx, gap):
    block = np.random.default_rng(6).standard_normal((6, D))
    block[:, 4:] = 0.0
    block *= np.sqrt(0.7 / np.linalg.norm(block.T @ block))
    i = np.arange(4, D)
    single = np.zeros((D - 4, D))
    single[i - 4, i] = np.sqrt(2e-6 - 5e-13 * (37 * i % D) + gap * (i - 4))
    R, lam, C, sweeps, p = solve(ctx, np.vstack([block, single]))
    eps = 2.0 ** -24
    assert sweeps == 1
    assert np.abs(R.T @ R - np.eye(D)).max() <= 2 * eps * np.sqrt(D)
    assert np.linalg.norm(R.T @ C @ R - np.diag(lam)) <= 4 * eps * np.sqrt(D) * np.linalg.norm(C)


# Blocks of equal tridiagonal matrices joined by weak links: neighbours whose vectors spread over all blocks.  Entries are dyadic, so the
# reduction is handed the matrix as it is, and the solver's shift of its diagonal leaves many gaps just above the distance of the test before
# (second case: on both sides of it).
@pytest.mark.parametrize("block,link,slope,off", [(16, 18, 32, 0.125), (43, 26, 0, 0.5), (16, 28, 0, 0.5), (12, 14, 8, 0.25), (3, 28, 32, 0.125)])
def test_glued_blocks(ctx, block, link, slope, off):
    i = np.arange(D)
    K = np.diag(1.0 + (np.abs(i % block - (block - 1) // 2) / slope if slope else 0.0 * i))
    K[i[:-1], i[1:]] = np.where(i[:-1] % block == block - 1, 2.0 ** -link, off)
    R, lam, C, sweeps, p = solve(ctx, K)
    eps = 2.0 ** -24
    assert np.array_equal(C, np.triu(np.tril(C, 1), -1))
    assert sweeps == 1
    assert np.abs(R.T @ R - np.eye(D)).max() <= 2 * eps * np.sqrt(D)
    assert np.linalg.norm(R.T @ C @ R - np.diag(lam)) <= 4 * eps * np.sqrt(D) * np.linalg.norm(C)


def test_non_finite_keys(ctx):
    """A head with an infinity or a NaN in its Keys: no eigenproblem to solve; the call ends, the other heads are as ever."""
    K = np.stack([recipe(100), recipe(100), recipe(100)]).astype(np.float32)[None]
    K[0, 1, 7, 3] = np.inf
    K[0, 2, 9, 4] = np.nan
    p = Pipeline(ctx, 1, 3, 3, 8, "f32", 100)
    p.fit(to_dev(K, "f32"), 100, center=False)
    R = to_host(p.R)
    assert np.abs(R[0, 0].T @ R[0, 0] - np.eye(D)).max() <= 1e-5
    assert p.sweeps.cpu().numpy()[0, 0] == 1
    assert np.array_equal(R[0, 1], np.eye(D)) and np.array_equal(R[0, 2], np.eye(D))
