"""The check of C^LC beside other work on the card (GPU): its report may not
depend on when its blocks start."""
import dataclasses

import numpy as np
import pytest

import mockgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def counting():
    """A batch whose count holds every CU for some 80 ms, on a stream of its own."""
    import torch

    from paper_2205_11852_amd import lc
    from paper_2205_11852_amd.pipeline import Pipeline

    lc.lib()
    wl = dataclasses.replace(mockgen.WORKLOADS["c2"], cfg_id=78, n_mock=64, n_subsets=50)
    pl = Pipeline(mockgen.make_catalogues(wl))
    pl.build_cells()
    pl.count()
    torch.cuda.synchronize()
    return pl, torch.cuda.Stream()


def _positive(P, n_mock, seed):
    """Vectors whose C = A (M infinite) is the sample covariance of one set."""
    import torch

    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn(n_mock, P, generator=g, dtype=torch.float64, device="cuda")
    return x[:, None].expand(n_mock, 3, P).contiguous()


@pytest.mark.parametrize("P,n_split", [(2000, 0), (700, 120)])
def test_report_beside_a_count(counting, P, n_split):
    """A panel of the Cholesky factorisation is many blocks that factor the
    same diagonal block.  Beside a count they start one by one as its blocks
    end, some after others have finished."""
    import torch

    from paper_2205_11852_amd import lc

    pl, side = counting
    n_mock = 2 * P
    xi = _positive(P, n_mock, P)
    A, B, C = (torch.empty((P, P), dtype=torch.float64, device="cuda") for _ in range(3))

    def check():
        return lc.lc_covariance_general(xi, n_mock, P, n_split, 1.0, 2.0, float("inf"), lc.LC_FP64, A, B, C,
                                        report=True)

    alone = check()
    torch.cuda.synchronize()
    full = C.cpu().numpy()
    w = [np.linalg.eigvalsh(full[s, s]) if s.stop > s.start else np.zeros(0)
         for s in (slice(0, n_split), slice(n_split, P))]
    for _ in range(3):
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(3):
                pl.count()
        beside = check()
        for rep in (alone, beside):
            for blk in range(2):
                assert rep["chol_ok"][blk] == 1 and rep["n_neg_eig"][blk] == 0
                if len(w[blk]):
                    tol = 20 * len(w[blk]) * 2.3e-16 * w[blk][-1]
                    assert abs(rep["min_eig"][blk] - w[blk][0]) <= tol
                    assert abs(rep["max_eig"][blk] - w[blk][-1]) <= tol
    torch.cuda.synchronize()
