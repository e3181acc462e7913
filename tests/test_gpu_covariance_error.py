"""Rounding error of the float64 covariance products (GPU, against extended
precision): no larger than that of one float64 chain over the mocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# mocks in one part and in several (few tiles), and whole (17 x 18 / 2 tiles)
@pytest.mark.parametrize("P,n_mock", [(63, 700), (129, 3000), (540, 1200), (1080, 600)])
def test_float64_products_against_extended_precision(P, n_mock):
    import torch

    from paper_2205_11852_amd import lc

    rng = np.random.default_rng(P)
    x = rng.normal(size=(n_mock, P)) * rng.uniform(0.01, 10.0, size=P) + rng.normal(size=P)
    C = torch.empty((P, P), dtype=torch.float64, device="cuda")
    lc.lc_sample_covariance(torch.as_tensor(x).cuda(), n_mock, P, lc.LC_FP64, C)
    got = C.cpu().numpy()
    cols = rng.choice(P, size=min(P, 40), replace=False)
    xl = x[:, cols].astype(np.longdouble)
    dl = xl - xl.mean(0)
    ref = np.zeros((len(cols), len(cols)), dtype=np.longdouble)
    chain = np.zeros((len(cols), len(cols)))
    d = x[:, cols] - x[:, cols].mean(0)
    for n in range(n_mock):
        ref += np.outer(dl[n], dl[n])
        chain += np.outer(d[n], d[n])
    ref /= n_mock - 1
    chain /= n_mock - 1
    size = np.sqrt(np.outer(ref.diagonal(), ref.diagonal()))

    def error(v):
        return float(np.sqrt(np.mean(((v - ref) / size) ** 2)))

    assert error(got[np.ix_(cols, cols)]) <= error(chain)
