"""The OMP kernel at the edges of its blocks of eight selections, and with more
nodes than workers (nodes come from queues), against the oracle; the Gram
kernel's arg-max among exact ties and undefined values."""
import numpy as np
import pytest

from oracle import aqmp_oracle as O
from tests.test_gpu_gram import _run as _run_gram
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


@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("fam", [1, 2, 3])
def test_gram_ties_and_undefined_pixels(A, n, fam):
    """One pixel per block, where whole rows of atoms have one correlation up
    to rounding: an atom with the largest is taken first.  A plane with an
    undefined pixel goes on until k in its block (undefined correlations are
    the largest) and leaves the other blocks alone."""
    import torch
    d = A.Dictionary(16, 64, families=fam)
    one = np.zeros((64, 64))
    one[::n, ::n] = 1.0                       # one pixel of every block
    nan = piecewise_image(64, 128, seed=43)
    nan[5, 7] = np.nan
    clean = piecewise_image(64, 128, seed=43)
    imgs = [torch.from_numpy(a).cuda() for a in (one, nan, clean)]
    p = dict(tol=1e-3, max_atoms=6, n_min=n, n_max=n)
    code = A.Code(d, imgs, [p], [(0, 0), (1, 0), (2, 0)], schedule=1, solver=A.SOLVER_GRAM)
    e = code.export_nodes()
    code.free()
    d.free()
    print("n", n, "fam", fam, "nodes", len(e.leaves), flush=True)
    dd = O.get_dict(n, fam).D if n < 64 else None
    for leaf in e.leaves:
        at = int(leaf["atom_off"])
        if leaf["job"] == 0 and dd is not None:
            c = np.abs(dd.T[:, 0])            # the pixel's values of every atom
            first = int(e.atom_idx[at])
            assert c[first] >= c.max() * (1 - 2.0 ** -50)
        if leaf["job"] == 1 and leaf["x0"] == 0 and leaf["y0"] == 0:
            assert leaf["n_atoms"] == 6 and np.isnan(leaf["resid_sq"])
    by = {(int(x["job"]), int(x["x0"]), int(x["y0"])): x for x in e.leaves}
    for (j, x0, y0), leaf in by.items():
        if j == 1 and (x0, y0) != (0, 0):
            other = by[(2, x0, y0)]
            na = int(leaf["n_atoms"])
            assert na == int(other["n_atoms"]) and leaf["resid_sq"] == other["resid_sq"]
            a, b = int(leaf["atom_off"]), int(other["atom_off"])
            assert (e.atom_idx[a:a + na] == e.atom_idx[b:b + na]).all() and (e.coef[a:a + na] == e.coef[b:b + na]).all()


@pytest.mark.parametrize("fam", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_gram_nodes_of_8(A, fam, dtype):
    """N = 8 of the Gram form, four nodes to a wave: more nodes than slots
    (16 384 on 256 CUs), a last wave with one node, step limits at the edges
    of the records' 16, blocks that end before the first step."""
    d = A.Dictionary(8, 8, families=fam)
    big = piecewise_image(1032, 1040, seed=51)          # 129 x 130 = 16 770 nodes
    small = np.ascontiguousarray(piecewise_image(64, 136, seed=52)[:8])   # 17 nodes, two of them zero
    small[:, 8:24] = 0
    imgs = [big, small, small, small, small]
    params = [dict(tol=0.02, max_atoms=k, n_min=8, n_max=8) for k in (9, 16, 17, 33, 1)]
    tops = O.top_blocks(1032, 1040, 8)
    rng = np.random.default_rng(53)
    sample = [tops[i] for i in sorted(rng.choice(len(tops), size=24, replace=False))] + [tops[-1]]
    rep = _run_gram(A, d, imgs, params, [(i, i) for i in range(5)], 1, dtype=dtype, families=fam,
                    blocks_per_job=[sample, None, None, None, None])
    d.free()
    _say("gram 8", fam, dtype, rep.summary())
    assert rep.ok(), rep.summary()
