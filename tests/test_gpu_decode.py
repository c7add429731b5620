"""The decoder of a job of a many-job code against the sum of its exported
leaves' atoms, formed from the FP64 dictionary on the host: mixed block
ranges, schedules, sample types, unaligned and odd-strided outputs, quantised
coefficients, and a re-encode that leaves fewer levels than the one before."""
import sys

import numpy as np
import pytest

from workloads import gradient_edges_image, piecewise_image

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_09190_amd import aqmp
    return aqmp


@pytest.fixture(scope="module")
def dic(A):
    d = A.Dictionary(4, 64)
    yield d
    d.free()


def _dev(img, f64=False):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(img))
    return t.to(torch.float64 if f64 else torch.float32).cuda()


_D: dict = {}


def _reference(dic, e, job, shape, step=0.0):
    """sum_t c_t phi_{i_t} of every leaf of the job, clipped to the plane."""
    h, w = shape
    out = np.full((-(-h // 64) * 64, -(-w // 64) * 64), np.nan)
    for r in e.leaves[e.leaves["job"] == job]:
        n, o, k = int(r["n"]), int(r["atom_off"]), int(r["n_atoms"])
        if n not in _D:
            _D[n] = dic.copy(n)
        c = e.coef[o:o + k]
        if step > 0:
            d = float(np.float32(step))
            c = np.rint(c / d) * d
        b = (_D[n][:, e.atom_idx[o:o + k]] @ c).reshape(n, n).T if k else np.zeros((n, n))
        out[r["y0"]:r["y0"] + n, r["x0"]:r["x0"] + n] = b
    return out[:h, :w]


def _check(A, code, dic, job, shape, dtype, pad, step=0.0):
    """Decodes into the middle of a buffer of NaN whose rows start `pad`
    samples further than the plane is wide."""
    import torch
    h, w = shape
    buf = torch.full((h + 2, w + pad), float("nan"), dtype=dtype, device="cuda")
    off = min(pad, 3)
    view = buf[1:1 + h, off:off + w] if off else buf[1:1 + h, :w]
    code.decode(job, view, step=step)
    torch.cuda.synchronize()
    got = buf.cpu().numpy().astype(np.float64)
    want = _reference(dic, code.export(), job, shape, step)
    inner = got[1:1 + h, off:off + w]
    # at most 40 terms of size <= 64 in another order, then the output's rounding
    tol = 1e-12 if dtype == torch.float64 else 2.0 ** -24 * max(1.0, np.abs(want).max()) * 1.01
    assert np.abs(inner - want).max() <= tol
    got[1:1 + h, off:off + w] = np.nan
    assert np.isnan(got).all()


@pytest.mark.parametrize("sched", [0, 1, 2])
@pytest.mark.parametrize("prec", [0, 1])
def test_decode_of_every_job(A, dic, prec, sched):
    import torch
    chans = [piecewise_image(100, 150, seed=41), gradient_edges_image(77, 70, seed=42), piecewise_image(64, 64, seed=43)]
    params = [dict(tol=0.02, max_atoms=24, n_min=4, n_max=64), dict(tol=0.02, max_atoms=16, n_min=8, n_max=32),
              dict(tol=0.5, tol_mode="abs", max_atoms=40, n_min=4, n_max=16), dict(tol=0.03, max_atoms=10, n_min=64, n_max=64),
              dict(tol=5.0, max_atoms=10, n_min=4, n_max=8)]
    jobs = [(i, p) for p in range(len(params)) for i in range(3)]
    code = A.Code(dic, [_dev(c, i == 1) for i, c in enumerate(chans)], params, jobs, precision=prec, schedule=sched)
    for j, (ci, _) in enumerate(jobs):
        for dtype, pad in ((torch.float32, 0), (torch.float64, 7), (torch.float32, 4)):
            _check(A, code, dic, j, chans[ci].shape, dtype, pad, step=0.01 if (j + pad) % 3 == 0 else 0.0)
    code.free()


def test_decode_after_a_shallower_reencode(A, dic):
    """The second image stops at the largest blocks: ranges of the lower levels
    left by the first encode are not used; then back again."""
    import torch
    rng = np.random.default_rng(44)
    deep = np.clip(piecewise_image(128, 192, seed=45) + rng.normal(0, 0.05, (128, 192)), 0, 1)
    flat = np.full((128, 192), 0.25)
    half = flat.copy()
    half[64:, :64] = deep[64:, :64]
    p = dict(tol=0.02, max_atoms=8, n_min=4, n_max=64)
    code = A.Code(dic, [_dev(deep), _dev(deep)], [p], [(0, 0), (1, 0)], precision=1, schedule=1)
    for a, b in ((deep, flat), (flat, half), (half, deep), (flat, flat), (deep, deep)):
        code.reencode([_dev(a), _dev(b)])
        for j in range(2):
            _check(A, code, dic, j, (128, 192), torch.float64, 4)
    code.free()


@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("k", [1, 3, 4, 5, 64, 65, 130])
def test_decode_of_list_lengths(A, dic, n, k):
    """Lists around the four atoms in flight and the 64 records of a wave.  The
    plane is noise: every list has k atoms, and partial sums stay below 2, so
    that 130 terms of three roundings differ by less than 1e-13."""
    import torch
    img = np.random.default_rng(46).random((n + 3, 2 * n - 1))
    p = dict(tol=1e-6, max_atoms=k, n_min=n, n_max=n)
    code = A.Code(dic, [_dev(img, True)], [p], [(0, 0)], precision=1, schedule=1)
    assert (code.export().leaves["n_atoms"] == k).all()
    for dtype, pad in ((torch.float32, 4), (torch.float64, 1)):
        _check(A, code, dic, 0, img.shape, dtype, pad)
    code.free()
