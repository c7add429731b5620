"""Samples at the ends of their types in the dense solver's whole-level
pursuits: FP32 planes whose block norms FP32 cannot hold."""
import sys

import numpy as np
import pytest

from workloads import piecewise_image

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_09190_amd import aqmp
    return aqmp


@pytest.fixture(scope="module")
def dic(A):
    d = A.Dictionary(8, 64)
    yield d
    d.free()


def _nodes(A, dic, img, prm, prec, f64=False):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(img)).to(torch.float64 if f64 else torch.float32).cuda()
    code = A.Code(dic, [t], [prm], [(0, 0)], precision=prec, schedule=A.SCHED_BATCHED)
    e = code.export_nodes()
    code.free()
    return e


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [8, 16, 32, 64])
def test_norm_beyond_fp32(A, dic, n, prec):
    """FP32 planes up to 2^128, whose block norms are past FP32's largest
    value, ordinary blocks, noise and bright ones (all of the norm in a row's
    first product): the atoms and, times the power of two, the coefficients of
    the plane at its usual scale."""
    rng = np.random.default_rng(43)
    plane = piecewise_image(n, 4 * n, seed=44)
    img = np.concatenate([plane, rng.uniform(-1, 1, (n, 4 * n)), 1.8 + 0.19 * plane])
    img = img.astype(np.float32).astype(np.float64)
    prm = dict(tol=0.01, max_atoms=12, n_min=n, n_max=n)
    s = 2.0 ** 127
    _say("n", n, "prec", prec)
    want = _nodes(A, dic, img, prm, prec)
    got = _nodes(A, dic, img * s, dict(prm, tol=0.01 * s), prec)
    assert got.atom_idx.tobytes() == want.atom_idx.tobytes()
    assert (got.coef == want.coef * s).all()
    assert (got.leaves["resid_sq"] == want.leaves["resid_sq"] * s * s).all()
