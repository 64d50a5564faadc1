"""The fine-grid form with products formed from bf16 pieces (the default where
the scan positions are uneven or half a voxel apart, and then the only form):
launch shapes, both gathers and the work-list batch.  The cards are those of the
tests that hold these on evenly spaced scans, with one scan position moved or
all of them half a voxel apart.

That the fine grid runs is shown by the geometry's bytes: it holds no tables of
the moment form, those of the even card do."""
import dataclasses

import numpy as np
import pytest

from synth import card_c1, card_c2, tiny_card, random_vector
from synth.cards import MM
from oracle import data as odata, operator as oo, solver as osv
from test_gpu_gather import WIN_FLOATS, host_windows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
umbir = pytest.importorskip("paper_2202_09703_amd.umbir")
batch = pytest.importorskip("paper_2202_09703_amd.batch")


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def uneven(card):
    """The last of three scan positions or more a voxel further; two of them
    half a voxel further apart; one joined by another half a voxel away."""
    tx = card.array.tx_x
    dx = card.grid.dx
    tx = tx[:-1] + (tx[-1] + dx,) if len(tx) > 2 else tx[:1] + ((tx[1] if len(tx) > 1 else tx[0]) + 0.5 * dx,)
    return dataclasses.replace(card, array=dataclasses.replace(card.array, tx_x=tx))


def on_fine_grid(card):
    """The geometry of the uneven card, checked to hold no moment tables."""
    c = uneven(card)
    even = dataclasses.replace(c, array=dataclasses.replace(
        c.array, tx_x=tuple(c.array.tx_x[0] + i * c.grid.dx for i in range(c.array.n_scans))))
    geom = umbir.build_geometry(c)
    # a record takes at least 24 bytes, one per receiver and voxel or more
    assert geom.bytes < umbir.estimate_bytes(even) - 10 * c.array.n_rx * c.n_voxels
    return c, geom


def f32(a):
    return torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("card", [
    tiny_card(n_layers=3, nx=17, nz=13, n_scans=3, n_rx=13, n_samples=700, oversample=32), card_c1()],
    ids=["tiny-q32", "c1"])
def test_launch_shapes_change_no_result(card):
    c, geom = on_fine_grid(card)
    x, r = f32(random_vector(geom.image_shape, seed=3)), f32(random_vector(geom.trace_shape, seed=4))
    y0, a0 = umbir.forward(geom, x), umbir.adjoint(geom, r)
    t0 = geom.tuning()
    assert t0["products"] == 2
    assert rel(y0.cpu(), oo.forward(c, x.cpu().numpy().astype(np.float64))) <= 1e-5
    assert rel(a0.cpu(), oo.adjoint(c, r.cpu().numpy().astype(np.float64))) <= 1e-5
    geom.set_tuning(products=1)
    y1, a1 = umbir.forward(geom, x), umbir.adjoint(geom, r)
    assert not torch.equal(y0, y1) and rel(y1.cpu(), y0.cpu()) <= 1e-6 and rel(a1.cpu(), a0.cpu()) <= 1e-6
    geom.set_tuning(products=2)
    for cg, rows, nb in [(2, 32, 1), (1, 64, 100000), (2, 128, 7)]:
        geom.set_tuning(conv_grid=cg, corr_tile_rows=rows, corr_blocks=nb)
        assert torch.equal(umbir.forward(geom, x), y0) and torch.equal(umbir.adjoint(geom, r), a0)
    for ct in (32, 64, 128, t0["conv_tile_rows"]):
        geom.set_tuning(conv_tile_rows=ct)
        y = umbir.forward(geom, x)
        assert torch.allclose(y, y0, rtol=1e-6, atol=1e-6 * float(y0.abs().max()))
        for cg in (1, 2):
            geom.set_tuning(conv_grid=cg)
            assert torch.equal(umbir.forward(geom, x), y)
    for blocks, kb in [(1, 1), (geom.n_scans * geom.n_rx * 4, 64), (100000, 1 << 20)]:
        geom.set_tuning(splat_blocks=blocks, gather_batch_kb=kb)
        assert torch.equal(umbir.forward(geom, x), y0)
        a = umbir.adjoint(geom, r)
        assert torch.allclose(a, a0, rtol=1e-6, atol=1e-6 * float(a0.abs().max()))
    geom.free()


GATHER = {
    "ragged-q16": tiny_card(n_layers=3, nx=17, nz=13, n_scans=3, n_rx=4, n_samples=300, oversample=16),
    "short-record": tiny_card(n_layers=3, nz=70, n_samples=40, oversample=32),
    "wide-q64": tiny_card(n_layers=3, nx=70, nz=40, n_scans=2, n_rx=3, n_samples=600, oversample=64),
    "c1": card_c1(),
}


@pytest.mark.parametrize("name", GATHER)
def test_windowed_gather_matches_rowwise_and_oracle(name):
    c, geom = on_fine_grid(GATHER[name])
    w = host_windows(c)
    if name == "short-record":  # empty windows and others
        assert (w == 0).any() and (w > 0).any()
    if name == "wide-q64":      # windows that do not fit LDS and others
        assert (w > 1.25 * WIN_FLOATS).any() and ((w > 0) & (w < WIN_FLOATS)).any()
    r = f32(random_vector(geom.trace_shape, seed=41))
    out = []
    for form in (1, 2):
        geom.set_tuning(gather_form=form)
        out.append((umbir.adjoint(geom, r), umbir.sqs_denominator(geom, 1.0)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    e = rel(out[1][0].cpu(), oo.adjoint(c, r.cpu().numpy().astype(np.float64)))
    print(f"{name}: adjoint rel L2 {e:.2e}")
    assert e <= 1e-5
    geom.free()


@pytest.mark.parametrize("q", [32, 64])
def test_worklist_batch(q):
    """Bitwise each problem's one-at-a-time result, and that matches the oracle:
    several splat chunks and one-trace gather batches in one problem, 32-, 64-
    and 128-sample convolution tiles, both gathers, problems that leave early."""
    cards = [dataclasses.replace(tiny_card(n_layers=3, nx=12, nz=10, n_scans=2, n_rx=3, n_samples=200,
                                           oversample=q), n_iter=7),
             dataclasses.replace(tiny_card(n_layers=2, nx=40, nz=30, n_scans=3, n_rx=4, n_samples=300,
                                           oversample=q), n_iter=4),
             dataclasses.replace(tiny_card(n_layers=4, nx=20, nz=14, n_scans=3, n_rx=2, n_samples=256,
                                           oversample=q), n_iter=6)]
    cards += [dataclasses.replace(card_c1(), n_iter=5)] if q == 64 else []
    cards = [uneven(c) for c in cards]
    data = [odata.synthesize(c)[1:] for c in cards]
    probs = batch.prepare(umbir, cards, device="cuda", log=lambda *a, **k: None, data=data)
    probs[2]["geom"].set_tuning(splat_blocks=probs[2]["geom"].n_scans * probs[2]["geom"].n_rx * 4, gather_batch_kb=1)
    probs[0]["geom"].set_tuning(conv_tile_rows=64, gather_form=1)
    probs[1]["geom"].set_tuning(conv_tile_rows=128, conv_grid=2)
    for i in (1, 2):
        probs[i]["geom"].set_tuning(gather_form=2)
    _, plain = batch.run_plain(umbir, probs)
    _, wl, n_batches = batch.run_batched(umbir, probs, umbir.BATCH_WORKLIST)
    assert n_batches == 1
    for c, (y, sigma), a, b in zip(cards, data, plain, wl):
        assert all(torch.equal(u, v) for u, v in zip(a, b)), c.name
        xo, go, co = osv.sqs(c, y, sigma, c.prior, c.n_iter)
        xe = rel(b[0].cpu(), xo)
        ce = float(np.max(np.abs(b[2].cpu().numpy() - co) / np.abs(co)))
        print(f"{c.name} ({c.n_iter} iterations): x {xe:.2e}, cost {ce:.2e}")
        assert xe <= 1e-5 and ce <= 1e-6
    for p in probs:
        p["geom"].free()


def test_products_of_bf16_pieces_at_full_size():
    """512 traces of 2048 samples, 256 x 256 voxels, the last scan moved: FP32
    products and bf16 pieces both within 2e-6 of the oracle on sampled traces
    and voxels, and not the same numbers."""
    c, geom = on_fine_grid(card_c2())
    x, r = f32(random_vector(geom.image_shape, seed=53)), f32(random_vector(geom.trace_shape, seed=54))
    traces = [(3, 7), (31, 12)]
    vox = np.random.default_rng(8).choice(c.n_voxels, 24, replace=False)
    fref = oo.forward(c, x.cpu().numpy().astype(np.float64), traces=traces)
    aref = oo.adjoint_voxels(c, r.cpu().numpy().astype(np.float64), vox)
    got = []
    for prod in (1, 2):
        geom.set_tuning(products=prod)
        y, xa = umbir.forward(geom, x).cpu().numpy(), umbir.adjoint(geom, r).cpu().numpy().reshape(-1)
        fe, ae = max(rel(y[t], fref[t]) for t in traces), rel(xa[vox], aref)
        print(f"products {prod}: forward {fe:.2e}, adjoint {ae:.2e}")
        assert fe <= 2e-6 and ae <= 2e-6
        got.append((y, xa))
    assert not np.array_equal(got[0][0], got[1][0]) and not np.array_equal(got[0][1], got[1][1])
    geom.free()
