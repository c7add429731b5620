"""The OMP kernel at the edges of its blocks of eight selections, and with more
nodes than workers (nodes come from queues), against the oracle."""
import numpy as np
import pytest

from oracle import aqmp_oracle as O
from tests.test_gpu_omp import A, _run, _say, dic   # noqa: F401  (fixtures and the parity helper)
from workloads import piecewise_image

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 7, 8, 9, 17])
def test_omp_factor_blocks(A, dic, k):
    img = piecewise_image(64, 128, seed=40)
    p = dict(tol=1e-4, max_atoms=k, n_min=8, n_max=64)
    _say("omp k", k)
    rep = _run(A, dic, [img], [p], [(0, 0)], 1, dtype="f64")
    _say(rep.summary())
    assert rep.ok(), rep.summary()


@pytest.mark.parametrize("n", [8, 32, 64])
def test_omp_more_nodes_than_workers(A, dic, n):
    side = {8: 640, 32: 1536, 64: 2048}[n]
    img = piecewise_image(side, side, seed=41)
    p = dict(tol=0.02, max_atoms=10, n_min=n, n_max=n)
    tops = O.top_blocks(side, side, n)
    rng = np.random.default_rng(42)
    sample = [tops[i] for i in sorted(rng.choice(len(tops), size=12, replace=False))] + [tops[-1]]
    _say("omp nodes", len(tops))
    rep = _run(A, dic, [img], [p], [(0, 0)], 1, dtype="f64", blocks_per_job=[sample])
    _say(rep.summary())
    assert rep.ok(), rep.summary()
