"""The covariance products and the check of C^LC at the sizes where their
kernels change (GPU, against numpy and LAPACK): tiles and parts of the products; rows per block of the resident tridiagonalisation (8 per block, 512
columns per thread slot), the launch-per-column one past 2048 rows, panels of
the Cholesky factorisation, and degenerate blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(C, n_split):
    """The report on C, reached through lc_covariance_general: vectors whose
    covariances give A = C and B = 0 (M infinite)."""
    import torch

    from paper_2205_11852_amd import lc

    # any symmetric C = 2 C^b - C^a: C^a = L^T L over the positive part of -C,
    # C^b over half the positive part of C
    P = C.shape[0]
    w, Q = np.linalg.eigh(C)
    up, dn = np.sqrt(np.maximum(w, 0.0) / 2.0), np.sqrt(np.maximum(-w, 0.0))
    # +-sqrt(P) rows: mean 0, N - 1 = 2P - 1
    f = np.sqrt((2 * P - 1) / 2.0)
    rows = lambda s: np.concatenate([f * s[:, None] * Q.T, -f * s[:, None] * Q.T])  # noqa: E731
    xi = torch.as_tensor(np.stack([rows(dn), rows(dn), rows(up)], axis=1)).cuda().contiguous()
    A, B, Co = (torch.empty((P, P), dtype=torch.float64, device="cuda") for _ in range(3))
    rep = lc.lc_covariance_general(xi, 2 * P, P, n_split, 1.0, 2.0, float("inf"), lc.LC_FP64, A, B, Co, report=True)
    torch.cuda.synchronize()
    return rep, Co.cpu().numpy()


def _assert_report(rep, C, n_split):
    for blk, sl in enumerate((slice(0, n_split), slice(n_split, C.shape[0]))):
        if sl.stop == sl.start:
            continue
        w = np.linalg.eigvalsh(C[sl, sl])
        n, size = len(w), max(abs(w[0]), abs(w[-1]))
        # backward stable: an error of a few n eps of the largest
        tol = 20 * n * 2.3e-16 * size + 1e-300
        assert abs(rep["min_eig"][blk] - w[0]) <= tol and abs(rep["max_eig"][blk] - w[-1]) <= tol
        assert (w < -tol).sum() <= rep["n_neg_eig"][blk] <= (w <= tol).sum()
        if w[0] > tol:
            assert rep["chol_ok"][blk] == 1
        if w[0] < -tol:
            assert rep["chol_ok"][blk] == 0


def _matrix(n, seed, positive):
    rng = np.random.default_rng(seed)
    X = rng.normal(size=(n, n + 50)) * rng.uniform(0.1, 3.0, size=(n, 1))
    C = X @ X.T / n
    if not positive:
        C -= np.diag(rng.uniform(0.0, 1.0, size=n) * C.diagonal())
    return 0.5 * (C + C.T)


@pytest.mark.parametrize("positive", [True, False])
@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 16, 17, 31, 32, 33, 63, 65, 96, 129, 511, 512, 513, 1024, 1025])
def test_check_sizes(n, positive):
    rep, C = _check(_matrix(n, n, positive), 0)
    _assert_report(rep, C, 0)


@pytest.mark.parametrize("n", [2047, 2048, 2049])
def test_check_large_sizes(n):
    rep, C = _check(_matrix(n, n, True), 5)
    _assert_report(rep, C, 5)


@pytest.mark.parametrize("n", [5, 40, 600])
def test_check_degenerate_blocks(n):
    rng = np.random.default_rng(n)
    d = rng.uniform(1.0, 2.0, size=n)
    for C in (np.zeros((n, n)), np.diag(d), np.diag(-d), 1e-200 * np.diag(d), 1e150 * _matrix(n, n, False),
              np.outer(d, d), np.diag(np.where(np.arange(n) % 3 == 0, 0.0, d))):
        rep, Co = _check(C, 0)
        _assert_report(rep, Co, 0)


# one row, edges of the 64- and 128-wide tiles; mocks below a slab, past the
# first split, a last part shorter than the others
@pytest.mark.parametrize("P", [1, 16, 63, 65, 129, 260])
@pytest.mark.parametrize("n_mock", [2, 15, 17, 64, 127, 130, 1025, 2309])
def test_sample_covariance_tiles_and_parts(P, n_mock):
    import torch

    from paper_2205_11852_amd import lc

    rng = np.random.default_rng(P * 10000 + n_mock)
    x = rng.normal(size=(n_mock, P)) * rng.uniform(0.01, 10.0, size=P) + rng.normal(size=P)
    ref = np.cov(x, rowvar=False).reshape(P, P)
    d = np.abs(x - x.mean(0))
    size = d.T @ d / (n_mock - 1)
    xd = torch.as_tensor(x).cuda()
    C = torch.full((P, P), float("nan"), dtype=torch.float64, device="cuda")
    # float64: the sums' rounding; float32: rounded deviations and 256 rows
    # summed in float32 (with LC_ACC32 all of them)
    u = 2.0 ** -24
    for prec, tol in ((lc.LC_FP64, 4.0 * (n_mock + 4) * 2.3e-16), (lc.LC_FP32_MFMA, (256 + 4) * u),
                      (lc.LC_FP32_MFMA | lc.LC_ACC32, (n_mock + 4) * u)):
        lc.lc_sample_covariance(xd, n_mock, P, prec, C)
        got = C.cpu().numpy()
        shift = 4.0 * 2.3e-16 * np.abs(x).max() * np.sqrt(np.outer(size.diagonal(), size.diagonal()))
        assert np.all(np.abs(got - ref) <= tol * size + n_mock * shift + 1e-300), prec
        assert np.array_equal(got, got.T)
