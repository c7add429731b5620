"""The windowed SSIM kernel at the edges of its tiling (64 columns a wave, rows
in groups of seven, four waves a workgroup, the number of groups by the plane's
size) against the oracle."""
import numpy as np
import pytest

from oracle import aqmp_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_09190_amd import aqmp
    return aqmp


# one window; a row and a column of windows; 64 and 65 columns of windows; 32
# and 33 rows (a workgroup of two groups); three and four groups
@pytest.mark.parametrize("shape", [(7, 7), (7, 75), (75, 7), (38, 70), (39, 71), (14, 69), (1500, 1100), (1533, 2053)])
@pytest.mark.parametrize("f64", [False, True])
def test_window_edges(A, shape, f64):
    import torch
    h, w = shape
    rng = np.random.default_rng(h * 3000 + w)
    dt = np.float64 if f64 else np.float32
    x = rng.random((h, w)).astype(dt)
    y = np.clip(x + 0.1 * rng.standard_normal((h, w)), 0, 1).astype(dt)
    # rows further apart than their length
    tx, ty = (torch.zeros((h, w + pad), dtype=torch.float64 if f64 else torch.float32, device="cuda") for pad in (3, 8))
    tx[:, :w], ty[:, :w] = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    print("shape", shape, "f64", f64, flush=True)
    got = A.ssim(tx[:, :w], ty[:, :w], A.SSIM_WINDOW7)
    want = O.ssim(x, y, "window7")
    # sums of 49 values up to 1 are within 49 2^-53 49 / 2 of exact, twice in a
    # (co)variance over 48, against C2 = 9e-4 in numerator and denominator
    assert abs(got - want) <= 4 * (49 * 49 * 2.0 ** -53 / 48) / 9e-4
