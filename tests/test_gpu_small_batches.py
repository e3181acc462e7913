"""Counts of batches too small to fill the card with whole cells per work
item: few tasks, cells cut into slices of their stencil, and queues whose
ranges end inside a task (GPU, bit-exact against the oracle)."""
import dataclasses

import numpy as np
import pytest

import mockgen
import oracle

pytestmark = pytest.mark.gpu


# (workload, points, r_max, mocks, randoms pool): the plan cuts cells into
# 8, 3 and 2 slices, leaves cells whole, or (few points) joins them in rows
CASES = [("c1", 20011, 100.0, 1, 1), ("c1", 9001, 60.0, 1, 2), ("c1", 15013, 200.0, 2, 2), ("c1", 301, 100.0, 1, 2),
         ("c4", 20011, 150.0, 1, 1), ("slab", 20011, 90.0, 1, 1), ("c1", 2999, 20.0, 3, 2)]


@pytest.mark.parametrize("los", ["z", "mid", "rppi"])
@pytest.mark.parametrize("name,points,r_max,n_mock,pool", CASES)
def test_small_batches_bit_exact(name, points, r_max, n_mock, pool, los):
    import torch

    from paper_2205_11852_amd.pipeline import Pipeline

    wl = mockgen.WORKLOADS[name]
    if wl.periodic and los == "mid":
        pytest.skip("the midpoint line of sight needs open geometry")
    wl = dataclasses.replace(wl, cfg_id=77, n_mock=n_mock, n_mean=float(points), n_parents=max(4, points // 25),
                             n_subsets=pool, subset_size=points, per_mock_randoms=False, n_r=10, r_max_mpc=r_max,
                             n_mu=7, los=los, pi_max_mpc=0.7 * r_max if los == "rppi" else 0.0)
    cats = mockgen.make_catalogues(wl)
    pl = Pipeline(cats)
    pl.build_cells()
    pl.count()
    torch.cuda.synchronize()
    got = pl.counts_host()
    for t, (a, b) in enumerate(pl.tasks):
        ref = oracle.count_pairs(cats.cat(a), None if a == b else cats.cat(b), wl.r_edges_units, wl.n_mu,
                                 wl.box_units, los, pi_max=wl.pi_max_units)
        assert np.array_equal(got[t], ref), (t, a, b)
