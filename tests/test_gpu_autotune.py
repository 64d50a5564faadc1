"""What umbir_autotune times.  A geometry that runs wholly as moments has no
use for the fine grid's launch shapes: they stay as they were.  One whose
curvature keeps the fine grid (|A| of an odd apodization power) has its shapes
timed there, not on the moment kernels, which ignore them."""
import dataclasses

import pytest

from synth import tiny_card
from synth.cards import Acquisition, Array, Grid, MM, MHZ, US

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
umbir = pytest.importorskip("paper_2202_09703_amd.umbir")


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def card(beta=8, shift=0.0, scans=32):
    """512 traces over 128 x 128 voxels: 64 trace groups of 8 traces, 4 MiB of
    fine grid per group, so that a row-wise gather at 2 MiB takes two launches."""
    c = tiny_card(n_layers=3)
    tx = [(i - scans // 2 - 0.5) * MM for i in range(scans)]
    tx[-1] += shift
    return dataclasses.replace(
        c, grid=Grid(nx=128, nz=128, dx=MM, dz=0.5 * MM, x0=-64 * MM),
        array=Array(tx_x=tuple(tx), rx_offset=tuple((j - 7.5) * 2 * MM for j in range(16)), beta=beta),
        acq=Acquisition(n_samples=4096, fs=20 * MHZ, f_c=0.5 * MHZ, sigma_t=1.25 * US, t_win=12 * US, oversample=32))


def launches_of_autotune(geom):
    umbir.profile_collect()
    umbir.profile_enable(True)
    chosen = geom.autotune()
    umbir.profile_enable(False)
    return chosen, {k: v[0] for k, v in umbir.profile_collect().items()}


def test_shapes_stay_where_all_runs_as_moments():
    geom = umbir.build_geometry(card())
    before = geom.tuning()
    chosen, n = launches_of_autotune(geom)
    assert {k: v for k, v in chosen.items() if k != "operator_form"} == \
           {k: v for k, v in before.items() if k != "operator_form"}
    # at most the two forms' pairs, four times each
    assert n.get("conv", 0) <= 8 and n.get("corr", 0) <= 8
    geom.free()


def test_shapes_of_a_fine_grid_curvature_are_timed_on_the_fine_grid():
    geom = umbir.build_geometry(card(beta=7))
    chosen, n = launches_of_autotune(geom)
    if chosen["operator_form"] == 1:
        assert n["gather"] > n["reduce_groups"] > 8  # the moment gather is one launch
    geom.free()


def test_a_cache_tells_the_routes_apart():
    keys = set()
    for kw in (dict(), dict(beta=7), dict(shift=MM)):
        geom = umbir.build_geometry(card(**kw))
        keys.add(geom.shape_key)
        geom.free()
    assert len(keys) == 3
