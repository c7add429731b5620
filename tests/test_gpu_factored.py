"""The whole-level pursuits with the factored correlation against the
step-by-step form (``stepwise``: the unfactored correlation and a select
launch per MP step).  Both re-score in FP64 in the same order and store the
same FP32 residual, so trees, atoms, coefficients and norms are equal bit for
bit; only the ranking that proposes candidates differs."""
import sys

import numpy as np
import pytest

from oracle import aqmp_oracle as O
from tests import parity_util as PU
from workloads import gradient_edges_image, piecewise_image, workload

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
def dics(A):
    made = {}

    def get(fam):
        if fam not in made:
            made[fam] = A.Dictionary(8, 64, families=fam)
        return made[fam]
    yield get
    for d in made.values():
        d.free()


def _dev(img, f64=False):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(img))
    return t.to(torch.float64 if f64 else torch.float32).cuda()


def _nodes(A, dic, imgs, params, jobs, prec, **kw):
    code = A.Code(dic, imgs, params, jobs, precision=prec, schedule=kw.pop("schedule", 1), **kw)
    e = code.export_nodes()
    code.free()
    return e


def _same(a, b):
    assert a.leaves.tobytes() == b.leaves.tobytes()
    assert a.atom_idx.tobytes() == b.atom_idx.tobytes()
    assert a.coef.tobytes() == b.coef.tobytes()


def _both(A, dic, imgs, params, jobs, prec, **kw):
    step = _nodes(A, dic, imgs, params, jobs, prec, stepwise=True, **kw)
    whole = _nodes(A, dic, imgs, params, jobs, prec, **kw)
    _say("nodes", len(whole.leaves), "atoms", len(whole.atom_idx))
    _same(whole, step)
    return whole


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("fam", [1, 2, 3])
def test_matches_stepwise(A, dics, prec, fam):
    """Both block sizes, an odd plane, FP64 samples, both split rules, one and
    two families, k beyond one record window."""
    chans = [_dev(piecewise_image(200, 331, seed=5)), _dev(gradient_edges_image(150, 97, seed=6), True)]
    params = [dict(tol=0.02, max_atoms=32, n_min=32, n_max=64), dict(tol=0.01, max_atoms=12, n_min=32, n_max=64, split_rule="r2"),
              dict(tol=0.004, max_atoms=70, n_min=32, n_max=32), dict(tol=0.6, tol_mode="abs", max_atoms=5, n_min=64, n_max=64)]
    jobs = [(i, p) for p in range(len(params)) for i in range(2)]
    _say("stepwise", prec, fam)
    _both(A, dics(fam), chans, params, jobs, prec)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("scale", [1e-30, 1e-12, 1e15, 1e30])
def test_sample_scales(A, dics, prec, scale):
    """Planes far from the usual range: the ranking neither underflows nor
    overflows, and the atoms are those of the plane at its usual scale (a
    power of two times it, so every product scales exactly)."""
    s = 2.0 ** round(np.log2(scale))
    img = piecewise_image(64, 128, seed=8)
    p = dict(tol=0.03, max_atoms=10, n_min=32, n_max=64)
    ref = _nodes(A, dics(3), [_dev(img)], [p], [(0, 0)], prec)
    got = _nodes(A, dics(3), [_dev(img * s)], [dict(p, tol=0.03 * s)], [(0, 0)], prec)
    _say("scale", s)
    assert got.atom_idx.tobytes() == ref.atom_idx.tobytes()
    assert (got.coef == ref.coef * s).all()


@pytest.mark.parametrize("prec", [0, 1])
def test_exact_ties(A, dics, prec):
    """Planes of zeros and ones, where many atoms tie at a step and the FP64
    re-score decides among all of them; a constant and an all-zero plane;
    k = 0.  The reference is the FP32 step-by-step form: the BF16 one keeps
    eight candidates by BF16 correlation, and more than eight atoms that tie
    differ there by BF16 rounding alone."""
    rng = np.random.default_rng(9)
    dots = (rng.random((64, 64)) < 0.02).astype(np.float64)
    chk = np.zeros((64, 64))
    chk[::2, ::2] = 1.0
    one = np.zeros((64, 64))
    one[17, 40] = 1.0
    planes = [_dev(dots), _dev(chk), _dev(one), _dev(np.full((64, 64), 0.37)), _dev(np.zeros((64, 64)))]
    params = [dict(tol=1e-4, max_atoms=12, n_min=32, n_max=64), dict(tol=0.0, max_atoms=3, n_min=64, n_max=64),
              dict(tol=0.01, max_atoms=0, n_min=32, n_max=64)]
    jobs = [(i, p) for p in range(len(params)) for i in range(len(planes))]
    want = _nodes(A, dics(3), planes, params, jobs, 0, stepwise=True)
    _same(_nodes(A, dics(3), planes, params, jobs, prec), want)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("fam", [1, 2, 3])
@pytest.mark.parametrize("n", [32, 64])
def test_carried_correlations(A, dics, n, fam, prec):
    """Pursuits past the steps that a product serves: 100 steps without a stop
    on a noise block (its norm halves late), and a smooth one under a bright
    mean, whose norm falls by orders of magnitude within them.  The reference
    is the FP32 step-by-step form, a product per step."""
    rng = np.random.default_rng(31)
    y, x = np.mgrid[0:n, 0:n] / n
    planes = [_dev(0.5 + 0.2 * rng.standard_normal((n, n))), _dev(0.9 + 0.05 * np.sin(5 * x + 2 * y) + 0.01 * y ** 3)]
    p = dict(tol=1e-9, tol_mode="abs", max_atoms=100, n_min=n, n_max=n)
    jobs = [(0, 0), (1, 0)]
    want = _nodes(A, dics(fam), planes, [p], jobs, 0, stepwise=True)
    _same(_nodes(A, dics(fam), planes, [p], jobs, prec), want)
    assert (want.leaves["n_atoms"] == 100).all()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("fam", [1, 2, 3])
def test_carried_correlations_16(A, dics, fam, prec):
    """The same at N = 16, where a wave of the BF16 form carries two nodes that
    want a product at different steps (a noise block beside smooth ones).  The
    reference takes the FP64 arg-max over all atoms at every step and stores
    the FP32 residual (the step-by-step form's eight FP32 keys miss it by
    2.5e-8 ||r|| at one step of one block).  Coefficients: sums of 256 products
    of pixels below 1 with atoms of unit norm, within 256 2^-53 16."""
    rng = np.random.default_rng(32)
    y, x = np.mgrid[0:64, 0:64] / 64
    img = 0.9 + 0.05 * np.sin(5 * x + 2 * y) + 0.01 * y ** 3
    img[::, 16:32] += 0.02 * rng.standard_normal((64, 16))
    p = dict(tol=1e-4, tol_mode="abs", max_atoms=90, n_min=16, n_max=16)
    got = _nodes(A, dics(fam), [_dev(img)], [p], [(0, 0)], prec)
    tabs = [t for t, f in ((O.dct_matrix(16), 1), (O.haar_matrix(16), 2)) if fam & f]
    ends = np.cumsum(got.leaves["n_atoms"])
    _say("atoms", ends[-1], got.leaves["n_atoms"].max())
    assert got.leaves["n_atoms"].max() > 64
    for leaf, end in zip(got.leaves, ends):
        na = int(leaf["n_atoms"])
        r = img[leaf["y0"]:leaf["y0"] + 16, leaf["x0"]:leaf["x0"] + 16].astype(np.float32).astype(np.float64)
        for t in range(na):
            c = np.stack([t_ @ r @ t_.T for t_ in tabs])          # [f][p][q]
            flat = np.abs(c.transpose(0, 2, 1)).ravel()            # f K + q N + p
            if fam == 3:
                flat[256] = 0.0                                    # the second constant atom
            a = int(flat.argmax())
            f, q, pp = a // 256, a % 256 // 16, a % 16
            assert got.atom_idx[end - na + t] == a, (leaf["x0"], leaf["y0"], t)
            coef = got.coef[end - na + t]
            assert abs(coef - c[f, pp, q]) <= 256 * 2.0 ** -53 * 16
            # the stored residual, of the encoder's own coefficient and as one
            # rounding: Haar products fall on FP32's midpoints
            phi = np.outer(tabs[f][pp], tabs[f][q]) if a else np.full((16, 16), 1 / 16)
            r = (r - np.longdouble(coef) * phi).astype(np.float64).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("fam", [1, 2, 3])
@pytest.mark.parametrize("exp", [-560, -440, 0, 440, 500])
def test_exact_form_8(A, dics, fam, exp):
    """N = 8 of the FP32 form (FP64 residual, ranked by the FP16 split): the
    atoms are arg-maxima of the oracle's dictionary at every scale of an FP64
    plane, also where the norm underflows to zero or passes the ranking's
    range; coefficients scale exactly with a power of two."""
    img = piecewise_image(40, 64, seed=23)
    dots = (np.random.default_rng(24).random((16, 64)) < 0.1).astype(np.float64)
    img = np.concatenate([img, dots])
    p = dict(tol=0.0, max_atoms=12, n_min=8, n_max=8)
    s = 2.0 ** exp
    got = _nodes(A, dics(fam), [_dev(img * s, True)], [p], [(0, 0)], 0)
    _say("fam", fam, "2^", exp, "atoms", len(got.atom_idx))
    dic = O.get_dict(8, fam)
    at = 0
    for leaf in got.leaves:
        blk = img[leaf["y0"]:leaf["y0"] + 8, leaf["x0"]:leaf["x0"] + 8]
        r, na = O.unravel(blk), int(leaf["n_atoms"])
        tol = 64 * 2.0 ** -52 * np.linalg.norm(blk)   # 64 products, and the roundings of the residual
        for t in range(na):
            c = dic.D.T @ r
            a = int(got.atom_idx[at + t])
            assert abs(c[a]) >= np.abs(c).max() - tol, (leaf["x0"], leaf["y0"], t)
            assert abs(got.coef[at + t] / s - c[a]) <= tol
            r = r - got.coef[at + t] / s * dic.D[:, a]
        assert na == 12 or np.linalg.norm(r) <= tol
        at += na


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("fam", [1, 3])
def test_undefined_pixels(A, dics, prec, fam):
    """A plane with an infinite and one with an undefined pixel: their blocks
    stop as in the step-by-step form, and the other blocks are untouched."""
    base = piecewise_image(128, 128, seed=11)
    planes = []
    for v in (np.inf, np.nan):
        a = base.copy()
        a[70, 30] = v
        planes.append(_dev(a))
    p = dict(tol=0.02, max_atoms=8, n_min=64, n_max=64)
    step = _nodes(A, dics(fam), planes, [p], [(0, 0), (1, 0)], prec, stepwise=True)
    whole = _nodes(A, dics(fam), planes, [p], [(0, 0), (1, 0)], prec)
    assert (whole.leaves["n_atoms"] == step.leaves["n_atoms"]).all()
    assert whole.atom_idx.tobytes() == step.atom_idx.tobytes()
    np.testing.assert_array_equal(whole.coef, step.coef)
    np.testing.assert_array_equal(whole.leaves["resid_sq"], step.leaves["resid_sq"])


@pytest.mark.parametrize("prec,sched", [(1, 0), (1, 2), (0, 0), (0, 2)])
def test_schedules_and_replays(A, dics, prec, sched):
    """Every schedule gives the batched result, and replays on other planes
    and back reproduce it (nodes are handed out by a counter)."""
    w = workload("c1")
    p = dict(w["params"][0], n_min=32)
    a, b = _dev(w["channels"][0]), _dev(piecewise_image(512, 512, seed=21))
    ref = _nodes(A, dics(3), [a, b], [p], [(0, 0), (1, 0)], prec, stepwise=True)
    code = A.Code(dics(3), [a, b], [p], [(0, 0), (1, 0)], precision=prec, schedule=sched)
    for i in range(4):
        _same(code.export_nodes(), ref)
        code.reencode([b, a])
        code.export_nodes()
        code.reencode([a, b])
    code.free()


@pytest.mark.parametrize("fam", [1, 2, 3])
def test_small_blocks_fp32_match_stepwise(A, dics, fam):
    """N = 16 of the FP32 form: a node per wave, k across record windows."""
    chans = [_dev(piecewise_image(75, 133, seed=15)), _dev(gradient_edges_image(40, 210, seed=16), True)]
    params = [dict(tol=0.02, max_atoms=32, n_min=16, n_max=64), dict(tol=0.002, max_atoms=70, n_min=16, n_max=16),
              dict(tol=0.03, max_atoms=7, n_min=8, n_max=16, split_rule="r2")]
    jobs = [(i, p) for p in range(len(params)) for i in range(2)]
    _both(A, dics(fam), chans, params, jobs, 0)


@pytest.mark.parametrize("fam", [1, 2, 3])
def test_small_blocks_bf16_match_fp32(A, dics, fam):
    """N = 16 and 8 of the BF16 form (two and four nodes per wave) choose the
    FP32 form's trees and atoms; the coefficients differ by the order of
    FP64 sums and the FP32 roundings of the residual that it moves: at most
    2^-24 of the plane's range per pixel and step, over a unit atom."""
    chans = [_dev(piecewise_image(75, 133, seed=17)), _dev(gradient_edges_image(200, 150, seed=18), True)]
    params = [dict(tol=0.02, max_atoms=32, n_min=8, n_max=16), dict(tol=0.006, max_atoms=40, n_min=8, n_max=8),
              dict(tol=0.01, max_atoms=20, n_min=16, n_max=16, split_rule="r2"), dict(tol=0.2, tol_mode="abs", max_atoms=3, n_min=8, n_max=16)]
    jobs = [(i, p) for p in range(len(params)) for i in range(2)]
    want = _nodes(A, dics(fam), chans, params, jobs, 0, stepwise=True)
    got = _nodes(A, dics(fam), chans, params, jobs, 1)
    _say("nodes", len(got.leaves), "atoms", len(got.atom_idx))
    for f in ("job", "x0", "y0", "n", "n_atoms", "flags"):
        assert (got.leaves[f] == want.leaves[f]).all(), f
    assert got.atom_idx.tobytes() == want.atom_idx.tobytes()
    tol = 2.0 ** -24 * 16 * np.sqrt(40)          # N <= 16 pixels a side, 40 steps of independent roundings
    assert np.abs(got.coef - want.coef).max() <= tol
    assert np.abs(got.leaves["resid_sq"] - want.leaves["resid_sq"]).max() <= 16 * tol


@pytest.mark.parametrize("prec", [0, 1])
def test_small_blocks_edges(A, dics, prec):
    """Small blocks that end at once or tie: zero and constant planes, k = 0,
    exact ties of binary dots, one node."""
    rng = np.random.default_rng(19)
    dots = (rng.random((32, 48)) < 0.05).astype(np.float64)
    planes = [dots, np.full((33, 17), 0.3), np.zeros((16, 16)), dots[:5, :7]]
    params = [dict(tol=1e-4, max_atoms=10, n_min=8, n_max=16), dict(tol=0.0, max_atoms=3, n_min=16, n_max=16),
              dict(tol=0.01, max_atoms=0, n_min=8, n_max=16), dict(tol=1e-5, max_atoms=20, n_min=8, n_max=8)]
    jobs = [(i, p) for p in range(len(params)) for i in range(len(planes))]
    got = _nodes(A, dics(3), [_dev(x) for x in planes], params, jobs, prec)
    if prec == 0:
        _same(got, _nodes(A, dics(3), [_dev(x) for x in planes], params, jobs, 0, stepwise=True))
        return
    # the BF16 form sums in another order, which decides exact ties: the oracle's tie rules
    rep = PU.Report()
    for j, (i, p) in enumerate(jobs):
        on = O.encode_channel(planes[i].astype(np.float32).astype(np.float64), O.Params.from_dict(params[p]))
        PU.compare_job(planes[i], on, PU.gpu_nodes_by_key(got, j), 2e-3, params[p]["n_max"], rep=rep)
    _say(rep.summary())
    assert rep.ok(), rep.summary()


@pytest.mark.parametrize("prec,n", [(0, 16), (1, 16), (1, 8)])
def test_small_blocks_undefined_pixels(A, dics, prec, n):
    """A block with an infinite or undefined pixel selects nothing; the others
    are those of the plane without it."""
    good = piecewise_image(48, 32, seed=20)
    bad = good.copy()
    bad[3, 5], bad[40, 9] = np.inf, np.nan
    p = dict(tol=0.01, max_atoms=9, n_min=n, n_max=n)
    g = _nodes(A, dics(3), [_dev(good)], [p], [(0, 0)], prec)
    b = _nodes(A, dics(3), [_dev(bad)], [p], [(0, 0)], prec)
    for i in range(len(g.leaves)):
        u, v = g.leaves[i], b.leaves[i]
        assert (u["x0"], u["y0"]) == (v["x0"], v["y0"])
        if not np.isfinite(bad[u["y0"]:u["y0"] + n, u["x0"]:u["x0"] + n]).all():
            assert v["n_atoms"] == 0
            continue
        su, sv = slice(u["atom_off"], u["atom_off"] + u["n_atoms"]), slice(v["atom_off"], v["atom_off"] + v["n_atoms"])
        assert (g.atom_idx[su] == b.atom_idx[sv]).all() and (g.coef[su] == b.coef[sv]).all()
