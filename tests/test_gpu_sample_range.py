"""Samples at the ends of their types in the dense solver's whole-level
pursuits: an FP64 sample that FP32 cannot hold, and FP32 planes whose block
norms FP32 cannot hold."""
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


def _others_unchanged(got, want, bad, n, ends):
    """The nodes without a bad sample are those of the clean plane; the others
    select nothing if `ends`."""
    assert len(got.leaves) == len(want.leaves)
    for u, v in zip(want.leaves, got.leaves):
        assert (u["x0"], u["y0"]) == (v["x0"], v["y0"])
        if bad[u["y0"]:u["y0"] + n, u["x0"]:u["x0"] + n].any():
            assert v["n_atoms"] == 0 or not ends
            continue
        su, sv = (slice(w["atom_off"], w["atom_off"] + w["n_atoms"]) for w in (u, v))
        assert u["n_atoms"] == v["n_atoms"] and u["resid_sq"] == v["resid_sq"], (u["x0"], u["y0"])
        assert (want.atom_idx[su] == got.atom_idx[sv]).all() and (want.coef[su] == got.coef[sv]).all()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [8, 16, 32, 64])
def test_sample_beyond_fp32(A, dic, n, prec):
    """One FP64 sample of 1e39 in some blocks: a form with an FP32 residual
    selects nothing there (the FP32 form's N = 8 keeps it in FP64), and the
    blocks beside them, nodes of the same wave, keep their atoms."""
    img = piecewise_image(2 * n, 8 * n, seed=41)
    bad = np.zeros(img.shape, bool)
    bad[3, 5] = bad[n + 2, 2 * n + 1] = bad[n - 1, 6 * n + 3] = True
    prm = dict(tol=0.01, max_atoms=9, n_min=n, n_max=n)
    _say("n", n, "prec", prec)
    want = _nodes(A, dic, img, prm, prec, True)
    assert want.leaves["n_atoms"].max() == 9
    got = _nodes(A, dic, np.where(bad, 1e39, img), prm, prec, True)
    _others_unchanged(got, want, bad, n, not (n == 8 and prec == 0))


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_undefined_sample_exact_form(A, dic, value):
    """N = 8 of the FP32 form beside an infinite or undefined sample."""
    img = piecewise_image(16, 64, seed=42)
    bad = np.zeros(img.shape, bool)
    bad[3, 5] = bad[10, 41] = True
    prm = dict(tol=0.01, max_atoms=9, n_min=8, n_max=8)
    want = _nodes(A, dic, img, prm, 0)
    _others_unchanged(_nodes(A, dic, np.where(bad, value, img), prm, 0), want, bad, 8, True)


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
