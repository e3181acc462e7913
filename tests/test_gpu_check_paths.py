"""Both ways of the check's tridiagonalisation, and the way from one to the
other (GPU, against LAPACK): matrices handed to the check as they are, with the
wait bound of the resident kernel given, or a launch per column."""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEFAULT, COLUMNS = -1, -2


def check(C, n_split=0, spin=DEFAULT, stream=None):
    """Report and the blocks' give-up marks; C is a device matrix."""
    import torch

    from paper_2205_11852_amd import lc

    rep, gave = lc.lc_cov_report(), (ctypes.c_int32 * 2)()
    s = stream if stream is not None else torch.cuda.current_stream()
    rc = lc.lib().lc_testing_check(ctypes.c_void_p(C.data_ptr()), C.shape[0], n_split, spin, ctypes.byref(rep), gave,
                                   ctypes.c_void_p(s.cuda_stream))
    assert rc == 0, lc.last_error()
    return rep.as_dict(), list(gave)


def device(C):
    import torch

    return torch.as_tensor(np.ascontiguousarray(C)).cuda()


def assert_spectrum(rep, C, blk=1):
    w = np.linalg.eigvalsh(C)
    # backward stable: an error of a few n eps of the largest
    tol = 20 * len(w) * 2.3e-16 * max(abs(w[0]), abs(w[-1]))
    assert abs(rep["min_eig"][blk] - w[0]) <= tol and abs(rep["max_eig"][blk] - w[-1]) <= tol
    assert (w < -tol).sum() <= rep["n_neg_eig"][blk] <= (w <= tol).sum()
    if w[0] > tol:
        assert rep["chol_ok"][blk] == 1
    if w[0] < -tol:
        assert rep["chol_ok"][blk] == 0


def dense(n, seed, shift):
    rng = np.random.default_rng(seed)
    X = rng.normal(size=(n, n + 50)) * rng.uniform(0.1, 3.0, size=(n, 1))
    C = X @ X.T / n
    return 0.5 * (C + C.T) - shift * np.eye(n)


# the column kernel's switches: 256 trailing rows, 512 and 1024 held elements;
# the resident one's: rows per block, 512 and 1024 columns
SIZES = [1, 2, 3, 4, 5, 8, 9, 17, 65, 256, 258, 259, 298, 513, 514, 1025, 1083]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("shift", [0.0, 1.0])
def test_launch_per_column(n, shift):
    C = dense(n, n, shift)
    rep, gave = check(device(C), spin=COLUMNS)
    assert gave == [0, 0]
    assert_spectrum(rep, C)


@pytest.mark.parametrize("n", SIZES + [2000, 2048])
def test_resident_gives_up(n):
    """Bound 0: every block gives up at its first column (a block of one row
    has none) and the columns take over."""
    C = dense(n, n, 0.5)
    rep, gave = check(device(C), spin=0)
    assert gave == [0, int(n > 1)]
    assert_spectrum(rep, C)


@pytest.mark.parametrize("spin", [1, 2, 5, 40])
@pytest.mark.parametrize("n", [9, 65, 600, 2000])
def test_short_waits(n, spin):
    """Some blocks may give up in the middle while others still wait."""
    C = dense(n, n, 0.5)
    d = device(C)
    for _ in range(3):
        rep, _ = check(d, spin=spin)
        assert_spectrum(rep, C)


def test_two_blocks_through_both():
    C = dense(700, 7, 0.3)
    d = device(C)
    for spin in (DEFAULT, COLUMNS, 0):
        rep, gave = check(d, 130, spin)
        assert gave == ([1, 1] if spin == 0 else [0, 0])
        assert_spectrum(rep, C[:130, :130], 0)
        assert_spectrum(rep, C[130:, 130:], 1)


def test_checks_of_several_threads():
    """Their resident blocks do not fit on the card together."""
    import torch

    C = dense(2000, 11, 0.5)
    d = device(C)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    out, bar = [None] * 4, threading.Barrier(4)

    def work(i):
        torch.cuda.set_device(0)
        bar.wait()
        out[i] = [check(d, stream=streams[i])[0] for _ in range(2)]

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert_spectrum(out[0][0], C)
    for o in out:
        for rep in o:
            for k in ("chol_ok", "n_neg_eig"):
                assert rep[k] == out[0][0][k]
            assert np.allclose(rep["min_eig"][1], out[0][0]["min_eig"][1], atol=1e-11)
            assert np.allclose(rep["max_eig"][1], out[0][0]["max_eig"][1], rtol=1e-11)


def weakly_coupled(n, eps, seed):
    """Next neighbours coupled by 1, all others by eps: a row's other elements
    are far below its first one, yet above the tolerance."""
    rng = np.random.default_rng(seed)
    E = rng.uniform(-1.0, 1.0, size=(n, n)) * eps
    return 2.0 * np.eye(n) + np.diag(np.ones(n - 1), 1) + np.diag(np.ones(n - 1), -1) + 0.5 * (E + E.T)


@pytest.mark.parametrize("spin", [DEFAULT, COLUMNS])
@pytest.mark.parametrize("eps", [1e-7, 9e-9, 1e-9, 1e-10, 1e-11, 1e-12])
@pytest.mark.parametrize("n", [3, 4, 9, 30, 70, 300])
def test_weakly_coupled_rows(n, eps, spin):
    """No element of a row may be dropped for being small beside the first
    (their squares are below its square's rounding from 1e-8 on)."""
    C = weakly_coupled(n, eps, n)
    rep, _ = check(device(C), spin=spin)
    assert_spectrum(rep, C)


@pytest.mark.parametrize("spin", [DEFAULT, COLUMNS])
def test_weak_coupling_decides_the_sign(spin):
    C = np.array([[2.0, 1.0, 9e-9], [1.0, 2.0, 1.0], [9e-9, 1.0, 2.0]]) - (2.0 - np.sqrt(2.0) + 2e-9) * np.eye(3)
    rep, _ = check(device(C), spin=spin)
    assert np.linalg.eigvalsh(C)[0] > 2e-9
    assert_spectrum(rep, C)
    assert rep["n_neg_eig"][1] == 0 and rep["chol_ok"][1] == 1


@pytest.mark.parametrize("spin", [DEFAULT, COLUMNS])
@pytest.mark.parametrize("n", [2, 5, 40, 600])
def test_infinities_are_reported(n, spin):
    """An infinite entry (an overflowed product) leaves no finite extremes."""
    for i, j in ((0, 0), (n - 1, n - 1), (0, n - 1), (n // 2, n // 2)):
        C = dense(n, n, 0.0)
        C[i, j] = C[j, i] = np.inf
        rep, _ = check(device(C), spin=spin)
        assert np.isnan(rep["min_eig"][1]) and np.isnan(rep["max_eig"][1]) and rep["n_neg_eig"][1] == -1, (i, j)


@pytest.mark.parametrize("small", [1e-20, 1e-31, 1e-36, 1e-60, 1e-120, 1e-250])
@pytest.mark.parametrize("scale", [1.0, 1e-30, 1e60])
def test_graded_blocks(small, scale):
    """Eigenvalues far below the largest, uncoupled from it: their signs, and
    the extreme one to its own precision."""
    for d in ([1.0, small], [small, 1.0], [1.0, small, 2.0 * small, 1.0], [small] * 3 + [1.0] + [small] * 3):
        rep, _ = check(device(np.diag(d) * scale))
        assert rep["n_neg_eig"][1] == 0 and rep["chol_ok"][1] == 1
        assert abs(rep["min_eig"][1] - small * scale) <= 1e-15 * small * scale
        rep, _ = check(device(-np.diag(d) * scale))
        assert rep["n_neg_eig"][1] == len(d) and rep["chol_ok"][1] == 0
        assert abs(rep["max_eig"][1] + small * scale) <= 1e-15 * small * scale
    d = np.diag([1.0, -small, small, 0.0]) * scale
    rep, _ = check(device(d))
    assert rep["n_neg_eig"][1] == 2  # a zero counts as below zero
    assert abs(rep["min_eig"][1] + small * scale) <= 1e-15 * small * scale


@pytest.mark.parametrize("n", [2, 9, 100, 700, 3100])
def test_graded_dense_blocks(n):
    """The same with a dense block 1e-33 of the other's size (3100 rows: counts
    from global memory)."""
    T = dense(n // 2, n, -0.1)
    C = np.zeros((n, n))
    C[: n - n // 2, : n - n // 2] = np.diag(np.linspace(1.0, 2.0, n - n // 2))
    C[n - n // 2:, n - n // 2:] = 1e-33 * T
    w = np.linalg.eigvalsh(T)
    tol = 20 * n * 2.3e-16 * w[-1]
    rep, _ = check(device(C))
    assert rep["n_neg_eig"][1] == 0 and rep["chol_ok"][1] == 1
    assert abs(rep["min_eig"][1] - 1e-33 * w[0]) <= 1e-33 * tol
    rep, _ = check(device(-C))
    assert rep["n_neg_eig"][1] == n and abs(rep["max_eig"][1] + 1e-33 * w[0]) <= 1e-33 * tol


def test_zero_rows_in_a_block():
    """Constant elements: zero eigenvalues among the others."""
    C = dense(300, 5, 0.0)
    z = [0, 7, 150, 299]
    C[z, :] = 0.0
    C[:, z] = 0.0
    rep, _ = check(device(C))
    assert rep["chol_ok"][1] == 0
    assert_spectrum(rep, C)  # (the reflections carry rounding into the zeros)


@pytest.mark.parametrize("n", [2, 5, 31, 32, 33, 64, 70, 200])
def test_cholesky_of_integer_factors(n):
    """C = L L^T with whole numbers in L: correctly rounded square roots and
    quotients make every step exact, so a last pivot of exactly zero is seen as
    zero, and one of 1 beside entries of millions as 1."""
    for seed in range(12):
        rng = np.random.default_rng(1000 * n + seed)
        L = np.tril(rng.integers(-60, 61, (n, n)).astype(float))
        np.fill_diagonal(L, rng.integers(1, 1000, n))
        for last, ok in ((0.0, 0), (1.0, 1)):
            L[-1, -1] = last
            rep, _ = check(device(L @ L.T))
            assert rep["chol_ok"][1] == ok, (seed, last)


@pytest.mark.parametrize("n", [2, 33, 70])
def test_cholesky_infinite_pivots(n):
    """An infinite diagonal entry is a positive pivot; its column is zero."""
    for i in (0, n // 2, n - 1):
        d = np.arange(1.0, n + 1.0)
        d[i] = np.inf
        rep, _ = check(device(np.diag(d)))
        assert rep["chol_ok"][1] == 1
        rep, _ = check(device(np.diag(-d)))
        assert rep["chol_ok"][1] == 0
