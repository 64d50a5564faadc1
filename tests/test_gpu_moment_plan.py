"""The moment form's tables: built in parts where their histograms are large,
and left out, with the fine grid in their place, where they find no memory or a
sample has too many records.

Tolerance: as for the other tests of the moment form, 2e-6 relative L2."""
import dataclasses

import numpy as np
import pytest

from synth import tiny_card, random_vector
from synth.cards import Acquisition, Array, Grid, MM, MHZ, US
from oracle import operator as oo

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
umbir = pytest.importorskip("paper_2202_09703_amd.umbir")

TOL = 2e-6


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def card(nx, nz, scans, rx, samples, step=1, dx=MM, dz=0.5 * MM, spread=2):
    """`scans` positions `step` voxels apart, receivers `spread` voxels apart."""
    c = tiny_card(n_layers=3)
    return dataclasses.replace(
        c, grid=Grid(nx=nx, nz=nz, dx=dx, dz=dz, x0=-nx * dx / 2),
        array=Array(tx_x=tuple(step * i * dx for i in range(scans)),
                    rx_offset=tuple((j - rx // 2) * spread * dx for j in range(rx)), beta=8),
        acq=Acquisition(n_samples=samples, fs=20 * MHZ, f_c=0.5 * MHZ, sigma_t=1.25 * US, t_win=12 * US, oversample=32))


def pair(geom):
    x = torch.tensor(random_vector(geom.image_shape, seed=91), dtype=torch.float32)
    r = torch.tensor(random_vector(geom.trace_shape, seed=92), dtype=torch.float32)
    return x, r, umbir.forward(geom, x.cuda()).cpu(), umbir.adjoint(geom, r.cuda()).cpu()


def test_histograms_in_parts():
    """64 receivers, 65 chunks of relative columns, 16384 samples: 273 MB of
    histograms, so 63 receivers and then one."""
    geom = umbir.build_geometry(card(64, 6, 2, 64, 16384, step=4040))
    _, _, y, xa = pair(geom)
    geom.set_tuning(products=1)
    _, _, y1, xa1 = pair(geom)
    assert not torch.equal(y, y1)  # the moments did run
    assert rel(y, y1) <= TOL and rel(xa, xa1) <= TOL
    # the last receiver, alone in its part
    assert float(y1[:, 63].abs().sum()) > 0 and rel(y[:, 63], y1[:, 63]) <= TOL
    geom.free()


def test_too_many_records_of_a_sample():
    """Voxels of 1 um: some 40 rows of 512 lie in one sample."""
    c = card(512, 512, 1, 1, 40, dx=1e-6, dz=1e-6)
    geom = umbir.build_geometry(c)
    assert geom.bytes < umbir.estimate_bytes(c)  # no moment tables
    x, r, y, xa = pair(geom)
    vox = np.arange(0, 512 * 512, 3001)
    assert rel(y, oo.forward(c, x.numpy().astype(np.float64))) <= TOL
    assert rel(xa.reshape(-1)[vox], oo.adjoint_voxels(c, r.numpy().astype(np.float64), vox)) <= TOL
    geom.free()


def test_no_memory_for_the_tables():
    """A device with 1 GiB left: the tables (1.6 GB) do not fit, the rest of the
    geometry (0.1 GB) does, so it is built, on the fine grid."""
    c = card(512, 512, 64, 128, 64, step=8, spread=4)
    full = umbir.build_geometry(c)
    assert full.bytes - 1.2e9 < 0.5e9 < 1.2e9 < full.bytes
    x, r, y, xa = pair(full)
    full.free()
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    free, _ = torch.cuda.mem_get_info()
    filler = torch.empty(free - (1 << 30), dtype=torch.uint8, device="cuda")
    try:
        geom = umbir.build_geometry(c)
    finally:
        del filler
        torch.cuda.empty_cache()
    assert geom.bytes < 0.5e9 and umbir.estimate_bytes(c) > 1.2e9
    _, _, y1, xa1 = pair(geom)
    assert not torch.equal(y, y1)
    assert rel(y1, y) <= TOL and rel(xa1, xa) <= TOL
    geom.free()


def test_sessions_of_moments_hold_no_fine_grid():
    """A session that runs wholly as moments and its geometry's tables together
    need less than the same problem on the fine grid (an uneven scan), so a
    memory budget admits no fewer sessions; it gives umbir_reconstruct's
    result."""
    c = dataclasses.replace(card(96, 80, 6, 8, 1100, step=4), n_iter=4)
    uneven = dataclasses.replace(c, array=dataclasses.replace(c.array, tx_x=c.array.tx_x[:-1] + (19 * MM,)))
    need = []
    for cc in (c, uneven):
        geom = umbir.build_geometry(cc)
        need.append(geom.bytes + umbir.solver_bytes(geom, 4))
        y = torch.tensor(random_vector(geom.trace_shape, seed=93), dtype=torch.float32, device="cuda")
        x, g, cost = umbir.reconstruct(geom, cc.prior, 0.5, y, 4)
        s = umbir.Solver(geom, cc.prior, 0.5, y, 4)
        assert s.bytes == umbir.solver_bytes(geom, 4)
        s.step(4)
        xs, gs, cs = s.read()
        assert torch.equal(xs, x) and torch.equal(gs, g) and torch.equal(cs, cost)
        s.free()
        geom.free()
    assert need[0] < need[1]


def test_workspace_does_not_outgrow_the_fine_grid():
    """64 scan positions 120 voxels apart with one receiver and 64 samples: the
    fine grid takes 0.5 MB, the image by phase 36 MB.  The fine grid serves, in
    the workspace of the same problem with an uneven scan."""
    c = card(32, 600, 64, 1, 64, step=120)
    uneven = dataclasses.replace(c, array=dataclasses.replace(c.array, tx_x=c.array.tx_x[:-1] +
                                                              (c.array.tx_x[-1] - MM,)))
    a, b = umbir.build_geometry(c), umbir.build_geometry(uneven)
    for kind in (umbir.WORK_FORWARD, umbir.WORK_ADJOINT, umbir.WORK_RECONSTRUCT):
        assert a.workspace_bytes(kind) == b.workspace_bytes(kind)
    x, r, y, xa = pair(a)
    assert rel(y[:2], oo.forward(c, x.numpy().astype(np.float64), traces=[(0, 0), (1, 0)])[:2]) <= TOL
    a.free()
    b.free()
