"""The moment form's dense kernels with two and four sample tiles a block (from
256 blocks on), with traces and samples left over in the last ones: 60 scan
positions x 17 receivers are 31 whole tiles of 32 traces and one of 28.

Tolerances: 2e-6 relative L2 for FP32 results, as for the other tests of the
moment form; half a unit of the last place of a 16-bit trace (its one rounding);
1e-5 for grouped ICD, whose steps divide by a group's curvature."""
import dataclasses

import numpy as np
import pytest

from synth import random_vector
from oracle import operator as oo
from test_gpu_moments import card

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
umbir = pytest.importorskip("paper_2202_09703_amd.umbir")

TOL = 2e-6
MANY = dict(nx=13, nz=9, scans=60, rx=17)


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def tiles(c):
    tt, m = (c.n_traces + 31) // 32, c.acq.n_samples
    return 4 if tt * ((m + 127) // 128) >= 256 else 2 if tt * ((m + 63) // 64) >= 256 else 1


@pytest.mark.parametrize("samples, n", [(1100, 4), (550, 2)])
@pytest.mark.parametrize("kw", [dict(), dict(mhz=10), dict(f_c=2)], ids=["r5", "r6", "r8"])
def test_ragged_tiles(kw, samples, n):
    c = card(samples=samples, **MANY, **kw)
    assert tiles(c) == n
    geom = umbir.build_geometry(c)
    x = torch.tensor(random_vector(geom.image_shape, seed=5), dtype=torch.float32)
    r = torch.tensor(random_vector(geom.trace_shape, seed=6), dtype=torch.float32)
    y, xa = umbir.forward(geom, x.cuda()).cpu(), umbir.adjoint(geom, r.cuda()).cpu()
    acc = umbir.forward(geom, x.cuda(), r.cuda(), accumulate=True).cpu()
    yo = oo.forward(c, x.numpy().astype(np.float64))
    es = rel(y, yo), rel(xa, oo.adjoint(c, r.numpy().astype(np.float64))), rel(acc, r.numpy() + yo)
    print("forward, adjoint, accumulated rel L2 %.2e %.2e %.2e" % es)
    assert max(es) <= TOL
    geom.set_tuning(products=1)
    assert not torch.equal(y, umbir.forward(geom, x.cuda()).cpu())  # the moments did run
    geom.free()


@pytest.mark.parametrize("samples, n", [(2200, 4), (1100, 4), (550, 2)])
def test_ragged_tiles_with_templates(samples, n):
    """Four tiles in the convolution too from 512 blocks on (2200 samples).
    Against the fine grid, which picks the same template for every pair."""
    c = card(samples=samples, templates=4, **MANY)
    assert tiles(c) == n
    geom = umbir.build_geometry(c)
    assert geom.n_gamma == 4
    x = torch.tensor(random_vector(geom.image_shape, seed=5), dtype=torch.float32).cuda()
    r = torch.tensor(random_vector(geom.trace_shape, seed=6), dtype=torch.float32).cuda()
    y, xa = umbir.forward(geom, x), umbir.adjoint(geom, r)
    geom.set_tuning(products=1)
    y1, xa1 = umbir.forward(geom, x), umbir.adjoint(geom, r)
    assert not torch.equal(y, y1)
    es = rel(y.cpu(), y1.cpu()), rel(xa.cpu(), xa1.cpu())
    print("forward, adjoint against the fine grid: rel L2 %.2e %.2e" % es)
    assert max(es) <= TOL
    geom.free()


@pytest.mark.parametrize("samples", [1100, 550])
@pytest.mark.parametrize("storage, u", [(1, 2.0 ** -11), (2, 2.0 ** -8)])
def test_ragged_tiles_of_16bit_traces(storage, u, samples):
    c = card(samples=samples, storage=storage, **MANY)
    geom = umbir.build_geometry(c)
    x = torch.tensor(random_vector(geom.image_shape, seed=9), dtype=torch.float32)
    yo = oo.forward(c, x.numpy().astype(np.float64))
    assert rel(umbir.forward(geom, x.cuda()).float().cpu(), yo) <= u
    base = torch.tensor(random_vector(geom.trace_shape, seed=10), dtype=torch.float32).to(geom.trace_dtype)
    ref = base.double().numpy() + yo
    assert rel(umbir.forward(geom, x.cuda(), base.cuda(), accumulate=True).float().cpu(), ref) <= u
    geom.free()


def test_icd_groups_with_two_tiles():
    c = card(nx=56, nz=56, scans=60, rx=17, samples=550)
    assert tiles(c) == 2
    geom = umbir.build_geometry(c)
    x_true = torch.tensor(random_vector(geom.image_shape, seed=31), dtype=torch.float32).cuda()
    y = umbir.forward(geom, x_true)
    sigma = 0.05 * float(y.square().mean().sqrt())
    y = y + sigma * torch.tensor(random_vector(geom.trace_shape, seed=32), dtype=torch.float32).cuda()
    a = umbir.reconstruct_icd(geom, c.prior, sigma, y, 2, group=(2, 2))  # 784 members
    geom.set_tuning(products=1)
    b = umbir.reconstruct_icd(geom, c.prior, sigma, y, 2, group=(2, 2))
    assert not torch.equal(a[0], b[0])
    errs = [rel(u.cpu(), v.cpu()) for u, v in zip(a, b)]
    print("image, direct weights, cost against window dots: rel L2 %.2e %.2e %.2e" % tuple(errs))
    assert max(errs) <= 1e-5
    geom.free()
