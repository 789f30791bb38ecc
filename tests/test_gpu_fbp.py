"""GPU parity of the fan-beam filtered back-projection (dect_fbp) against the
FP64 oracle's FBP, on the tiny and ragged geometries and the full 512 x 512,
360-view workload; pairs equal single calls bit for bit; a uniform disk
comes back at its attenuation; ADM started from the FBP image matches the
oracle started from the same image; unsupported geometries are refused.

Tolerance: rel-L2 <= 1e-5.  The GPU evaluates each pixel's detector
position in FP32 (an error of ~1e-5 bin at 256 mm from the centre), which
moves the interpolated value by that fraction of the step between
neighbouring filtered bins.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1607_01650_amd import configs as C
from paper_1607_01650_amd import phantom as P

from helpers import f32, need_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

RAGGED = C.Geometry(nx=67, ny=45, pixel_mm=1.0, n_views=37, n_bins=101, bin_mm=1.3,
                    sod_mm=300.0, sdd_mm=600.0, det_offset_mm=0.7)


@pytest.fixture(scope="module")
def torch():
    return need_gpu()


def _dect():
    from paper_1607_01650_amd import dect
    return dect


@pytest.mark.parametrize("geom,seed", [(C.TINY, 0), (RAGGED, 1), (C.METRIC, 2)],
                         ids=["tiny", "ragged", "metric"])
def test_fbp_parity(torch, geom, seed):
    dect = _dect()
    s = P.make_slice(geom, seed, n_inserts=3, r_obj=18.0) \
        if geom is RAGGED else P.make_slice(geom, seed)
    for e in (0, 1):
        y = f32(s.sino[e])
        got = to_np(dect.fbp(to_dev(torch, y), geom))
        ref = O.fbp(geom, y)
        err = rel_l2(got, ref)
        print(f"fbp {geom.nx}x{geom.ny} V={geom.n_views} energy {e}: rel-L2 {err:.2e}", flush=True)
        assert err <= 1e-5


# Edges of the filter's 64-bin chunks, 512-bin stages and 8-view groups and of the
# back-projection's 16- and 32-column tiles and view eighths.
EDGES = {
    "1bin": dict(n_bins=1, bin_mm=90.0), "2bins": dict(n_bins=2, bin_mm=60.0),
    "63": dict(n_bins=63, bin_mm=2.1), "65": dict(n_bins=65, n_views=7),
    "511": dict(n_bins=511, bin_mm=0.5, n_views=8), "513": dict(n_bins=513, bin_mm=0.5, n_views=9),
    "1100": dict(n_bins=1100, bin_mm=0.31, n_views=17), "1view": dict(n_views=1),
    "tile": dict(nx=17, ny=33, n_views=64),
    "wide": dict(nx=545, ny=491, n_bins=640, bin_mm=2.4, sod_mm=1000.0, sdd_mm=2000.0),
}


@pytest.mark.parametrize("name", list(EDGES))
def test_fbp_edges(torch, name):
    dect = _dect()
    g = C.Geometry(**{**RAGGED.__dict__, **EDGES[name]})
    y = f32(P.random_sino(g, 5))
    got = to_np(dect.fbp(to_dev(torch, np.stack([y, 2.0 * y, y])), g))
    assert rel_l2(got[0], O.fbp(g, y)) <= 1e-5
    assert np.array_equal(got[1], 2.0 * got[0]) and np.array_equal(got[2], got[0])


def test_fbp_fine_bins(torch):
    # Bins so fine that a tile sees more of them than a window holds (the general kernel).
    # White noise: a position rounded to half the detector times 3 * 2^-24, times a
    # neighbour difference of at most 2.5 of the value.
    dect = _dect()
    g = C.Geometry(**{**RAGGED.__dict__, "n_bins": 900, "bin_mm": 0.2, "n_views": 21})
    y = f32(P.random_sino(g, 5))
    got = to_np(dect.fbp(to_dev(torch, y), g))
    assert rel_l2(got, O.fbp(g, y)) <= 450 * 3 * 2.5 * 2.0 ** -24


# Images whose last tiles lie mostly outside them: an orbit close to the image, so that such
# a tile's own centre would be at (15.5 mm) or beyond the source, and a windowed size whose
# tile sees as many bins as a window takes.
@pytest.mark.parametrize("n,sod,bin_mm", [(17, 15.5, 1.3), (17, 12.1, 1.0), (33, 24.0, 1.6), (17, 60.0, 1.65)])
def test_fbp_tiles_past_the_image(torch, n, sod, bin_mm):
    # Positions are FP32 sums relative to the centre of the tile's part of the image: three
    # roundings of the bins between it and its corners, times a neighbour difference of at
    # most 2.5 of the value (white noise); the distance's rounding enters its square.
    dect = _dect()
    g = C.Geometry(nx=n, ny=n, pixel_mm=1.0, n_views=24, n_bins=int(1.9 * sod / bin_mm) * 2 + 1,
                   bin_mm=bin_mm, sod_mm=sod, sdd_mm=2.0 * sod)
    r = 0.5 * np.hypot(n - 1, n - 1)
    bins = np.hypot(7.5, 7.5) * 2.0 * sod / (sod - r) / bin_mm / np.sqrt(1.0 - (r / sod) ** 2)
    y = f32(P.random_sino(g, 5))
    got = to_np(dect.fbp(to_dev(torch, y), g))
    assert rel_l2(got, O.fbp(g, y)) <= (3 * 2.5 * max(bins, 16.0) + 4 * sod / (sod - r)) * 2.0 ** -24


# The general kernel's split over the views (a quarter of them per wavefront up to 400 tiles):
# fewer views than parts, remainders of parts, groups and chunks, both sides of the line.
@pytest.mark.parametrize("n,views", [(17, 1), (17, 3), (17, 4), (17, 5), (33, 35), (33, 67), (17, 261), (321, 10),
                                     (320, 10)])
def test_fbp_general_parts(torch, n, views):
    # White noise; a position is the sum of at most 60 bins within a tile and the tile's FP64
    # position: three roundings of 2^-24 of that, times a neighbour difference of at most 2.5
    # of the value, rms below half of it: 60 * 3 * 2.5 * 2^-25
    dect = _dect()
    g = C.Geometry(nx=n, ny=n, pixel_mm=1.0, n_views=views, n_bins=6 * n, bin_mm=0.4, sod_mm=4.0 * n, sdd_mm=8.0 * n)
    y = f32(P.random_sino(g, 6))
    got = to_np(dect.fbp(to_dev(torch, y), g))
    assert rel_l2(got, O.fbp(g, y)) <= 60 * 3 * 2.5 * 2.0 ** -25


def test_fbp_fine_bins_from_the_tile(torch):
    # The general kernel at 900 bins, with the bound of the other parity tests: offsets from the
    # tile's centre of 47 bins rms, three roundings of 0.3 * 2^-23 of which, times neighbour
    # differences of 1.4 of the value, are 4e-6.  (Positions rounded to the detector's 260 bins
    # rms give five times that.)
    dect = _dect()
    g = C.Geometry(**{**RAGGED.__dict__, "n_bins": 900, "bin_mm": 0.2, "n_views": 21})
    y = f32(P.random_sino(g, 5))
    assert rel_l2(to_np(dect.fbp(to_dev(torch, y), g)), O.fbp(g, y)) <= 1e-5


def test_fbp_pairs_equal_single_calls(torch):
    dect = _dect()
    g = RAGGED
    ys = np.stack([f32(P.random_sino(g, 30 + i)) for i in range(3)])
    got = to_np(dect.fbp(to_dev(torch, ys), g))
    for i in range(3):
        assert np.array_equal(got[i], to_np(dect.fbp(to_dev(torch, ys[i]), g)))


def test_fbp_uniform_disk(torch):
    dect = _dect()
    g = C.Geometry(nx=128, ny=128, pixel_mm=1.0, n_views=360, n_bins=300, bin_mm=1.0,
                   sod_mm=300.0, sdd_mm=600.0)
    el = [P.Ellipse(20.0, -10.0, 15.0, 15.0, 0.0, 0.02, 0.03, 1)]
    img = to_np(dect.fbp(to_dev(torch, P.analytic_sinogram(el, g, 0)), g))
    r, c = int(round(-10 + 63.5)), int(round(20 + 63.5))
    assert np.abs(img[r - 5:r + 6, c - 5:c + 6] - 0.02).max() <= 2e-3 * 0.02


def test_adm_from_fbp_start(torch):
    """ADM-TV started from the FBP images (DECT_WARM_START) vs the oracle
    started from the same images."""
    dect = _dect()
    g = C.TINY
    s = P.make_slice(g, 0)
    x0 = [to_np(dect.fbp(to_dev(torch, s.sino[e]), g)) for e in (0, 1)]
    p = C.default_adm_params(g, 30)
    r = dect.adm_tv(to_dev(torch, s.sino[0]), to_dev(torch, s.sino[1]), g, p,
                    x0=(to_dev(torch, x0[0]), to_dev(torch, x0[1])))
    for e, (xe, beta) in enumerate(((r.x_high, p.beta_high), (r.x_low, p.beta_low))):
        ref = O.adm(g, f32(s.sino[e]), beta, p.mu, p.rho, p.xi, 30, x0=f32(x0[e]))
        err = rel_l2(to_np(xe), ref.x)
        print(f"ADM from FBP energy {e}: rel-L2 {err:.2e}", flush=True)
        assert err <= 1e-4


def test_fbp_refusals(torch):
    dect = _dect()
    g = C.Geometry(**{**C.TINY.__dict__,
                      "angles_rad": [2 * np.pi * v / C.TINY.n_views for v in range(C.TINY.n_views)]})
    with pytest.raises(dect.DectError):
        dect.fbp(torch.zeros((g.n_views, g.n_bins), device="cuda"), g)
    wide = C.Geometry(nx=32, ny=32, pixel_mm=1.0, n_views=8, n_bins=7000, bin_mm=0.01,
                      sod_mm=100.0, sdd_mm=200.0)
    with pytest.raises(dect.DectError):
        dect.fbp(torch.zeros((wide.n_views, wide.n_bins), device="cuda"), wide)
