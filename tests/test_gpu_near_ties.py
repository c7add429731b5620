"""Checkered planes with a little noise, in the Haar basis alone: a quarter of
all atoms within the ranking's window of the largest, one of which it is."""
import numpy as np
import pytest

from oracle import aqmp_oracle as O
from tests import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_09190_amd import aqmp
    return aqmp


@pytest.fixture(scope="module")
def haar(A):
    d = A.Dictionary(8, 64, families=A.HAAR)
    yield d
    d.free()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("noise", [1e-6, 1e-4])
@pytest.mark.parametrize("n_min,n_max", [(8, 8), (16, 16), (32, 32), (64, 64), (8, 64)])
def test_near_ties_take_the_arg_max(A, haar, n_min, n_max, noise, prec):
    """Coefficients that differ in their sixth or fourth digit: the oracle's
    atoms, but for what lies within its own tolerance of a tie."""
    import torch
    y, x = np.mgrid[0:64, 0:128]
    img = ((x + y) & 1) + noise * np.random.default_rng(5).standard_normal((64, 128))
    img = img.astype(np.float32).astype(np.float64)
    prm = dict(tol=0.02, max_atoms=24, n_min=n_min, n_max=n_max)
    ref = O.encode_channel(img, O.Params.from_dict(dict(prm, families=O.HAAR)))
    code = A.Code(haar, [torch.from_numpy(img).float().cuda()], [prm], [(0, 0)], precision=prec)
    e = code.export_nodes()
    code.free()
    rep = PU.compare_job(img, ref, PU.gpu_nodes_by_key(e, 0), 2e-3, n_max, families=O.HAAR)
    print((n_min, n_max), noise, "prec", prec, rep.summary()[:300], flush=True)
    assert rep.ok()
