"""Which groups of grouped ICD run as moments: large ones with long windows.
Short windows (a 2 MHz pulse) and groups of which few members lie in the record
keep the window dots, which the FP32-product tuning (products = 1) runs always:
there the two tunings give the same numbers, elsewhere they differ in rounding
(1e-5, the bar of the parity tests of grouped ICD)."""
import numpy as np
import pytest

from synth import random_vector
from test_gpu_moments import card

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
umbir = pytest.importorskip("paper_2202_09703_amd.umbir")


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("kw, group, moments", [
    (dict(nx=56, nz=56, scans=4, rx=4, samples=600, f_c=2), (2, 2), False),        # 784 members, windows of 60
    (dict(nx=128, nz=100, scans=4, rx=4, samples=1200, f_c=2), (2, 2), True),      # 3200 members, windows of 60
    (dict(nx=64, nz=200, scans=2, rx=4, samples=230, mhz=10), (3, 3), False),      # 1474, a third in the record
    (dict(nx=64, nz=200, scans=2, rx=4, samples=900, mhz=10), (3, 3), True),       # 1474, all in the record
], ids=["short-window", "short-window-large", "short-record", "long-record"])
def test_route_of_groups(kw, group, moments):
    c = card(**kw)
    geom = umbir.build_geometry(c)
    x_true = torch.tensor(random_vector(geom.image_shape, seed=31), dtype=torch.float32).cuda()
    y = umbir.forward(geom, x_true)
    sigma = 0.05 * float(y.square().mean().sqrt())
    y = y + sigma * torch.tensor(random_vector(geom.trace_shape, seed=32), dtype=torch.float32).cuda()
    a = umbir.reconstruct_icd(geom, c.prior, sigma, y, 2, group=group)
    geom.set_tuning(products=1)
    b = umbir.reconstruct_icd(geom, c.prior, sigma, y, 2, group=group)
    assert torch.equal(a[0], b[0]) != moments
    assert max(rel(u.cpu(), v.cpu()) for u, v in zip(a, b)) <= 1e-5
    geom.free()
