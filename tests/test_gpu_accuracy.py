"""Error of the FP32 operators against the FP64 oracle where roundings that all
lean to one side would show: sums over many traces and over many templates.

Bounds.  A result carries a handful of independent FP32 roundings of at most
u = 2^-24 relative to its own size (moments, tables and weights, the running
sums of the dense products, the partial sums over traces), of RMS size
u / sqrt(3) each.  They average out over the terms of a sum, so the relative L2
error stays near sqrt(6 / 3) u and 2.5 u is allowed for a trace (the sums over
the traces of an image add as much again: 5 u).  Errors that lean to one side
do not average out and grow with the number of terms."""
import dataclasses

import numpy as np
import pytest

from synth import card_c2, card_c3, phantom, random_vector
from synth.cards import ALPHA_CEMENT, ALPHA_WATER
from oracle import operator as oo

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
umbir = pytest.importorskip("paper_2202_09703_amd.umbir")

U = 2.0 ** -24


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def test_adjoint_over_2048_traces(dev):
    card = card_c3()
    geom = umbir.build_geometry(card)
    r = torch.tensor(random_vector(geom.trace_shape, seed=71), dtype=torch.float32)
    x = umbir.adjoint(geom, r.to(dev)).cpu().numpy().reshape(-1)
    vox = np.random.default_rng(72).choice(card.n_voxels, 96, replace=False)
    ref = oo.adjoint_voxels(card, r.numpy().astype(np.float64), vox, workers=None)
    e = rel(x[vox], ref)
    print(f"adjoint of {card.n_traces} traces, 96 voxels: rel L2 {e:.2e}")
    assert e <= 5 * U
    geom.free()


def test_forward_over_16_templates(dev):
    card = card_c2()
    card = dataclasses.replace(card, medium=dataclasses.replace(card.medium, atten=(ALPHA_WATER, 0.0, ALPHA_CEMENT)))
    geom = umbir.build_geometry(card)
    x = torch.tensor(phantom(card) + 0.02 * random_vector((256, 256), seed=73), dtype=torch.float32)
    y = umbir.forward(geom, x.to(dev)).cpu().numpy()
    traces = [(i, j) for i in (0, 7, 15, 31) for j in (0, 6, 15)]
    ref = oo.forward(card, x.numpy().astype(np.float64), traces=traces, workers=None)
    e = rel([y[t] for t in traces], [ref[t] for t in traces])
    print(f"attenuated forward, {len(traces)} traces: rel L2 {e:.2e}")
    assert e <= 2.5 * U
    geom.free()


def test_forward_is_no_further_off_than_the_fine_grid(dev):
    """Interfaces and point reflectors only, where a sample is a few coherent
    terms that partly cancel: the moment form against the fine grid that it
    stands in for, on the same traces.  Moving the last scan position makes the
    geometry keep the fine grid and leaves the other positions' traces as they
    are.  A quarter is allowed for the choice of traces."""
    card = card_c3()
    tx = card.array.tx_x
    moved = dataclasses.replace(card, array=dataclasses.replace(card.array, tx_x=tx[:-1] + (tx[-1] + card.grid.dx,)))
    x = torch.tensor(phantom(card), dtype=torch.float32)
    traces = [(i, j) for i in (0, 12, 24, 36, 48, 62) for j in (0, 11, 20, 31)]
    ref = oo.forward(card, x.numpy().astype(np.float64), traces=traces, workers=None)
    e = []
    for c in (card, moved):
        geom = umbir.build_geometry(c)
        y = umbir.forward(geom, x.to(dev)).cpu().numpy()
        e.append(rel([y[t] for t in traces], [ref[t] for t in traces]))
        geom.free()
    print(f"forward of the phantom, {len(traces)} traces: rel L2 {e[0]:.2e}, fine grid {e[1]:.2e}")
    assert e[0] != e[1] and e[0] <= 1.25 * e[1]
