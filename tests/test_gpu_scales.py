"""Rows of patterns at every scale of intensity: a power of 2 over the polar
image and its norm changes no sum, so that the rows of every route have to be
those of the exhaustive scan (per-template outputs asked for), bit for bit,
from patterns near the smallest float32 to the largest."""
import numpy as np
import pytest

from conftest import small_library
from test_gpu_search import _patterns, _same

pytestmark = pytest.mark.gpu

# down to the smallest norms with a finite inverse, up to one with a subnormal
# inverse
SCALES = (0, -95, -100, -104, -110, -122, 100, 122)


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2111_07347_amd as tm
    return tm


# sparse (searched by itself), dense (bounds refined for small batches,
# certified rescoring for the others), small enough to be scanned by the
# plain path (the bound and Fourier routes still bound it)
@pytest.mark.parametrize("T,max_spots,n_theta,Bs", [(2500, 8, 360, (1, 40)),
                                                    (4200, 70, 180, (1, 6, 140)),
                                                    (60, 30, 128, (9,))])
def test_rows_at_every_scale(tm, T, max_spots, n_theta, Bs):
    import torch
    R = 60 if max_spots > 40 else 34     # the dense library's rows: not crowded
    lib_np = small_library(T, seed=T, max_spots=max_spots, g_min=0.08, g_max=1.1)
    grid = tm.PolarGrid(R=R, n_theta=n_theta, cx=33.0, cy=35.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"],
                     (R - 4) / 1.2, grid, fft=True)
    for B in Bs:
        x = torch.from_numpy(_patterns(lib_np, (R - 4) / 1.2, R, B, seed=B)).cuda()
        for k in SCALES:
            print("[case] scales", T, n_theta, "B", B, "2^", k, flush=True)
            polar, norms, prof = tm.polar_transform(x, grid, lib=lib)
            full = tm.polar_transform(x, grid)[0] * 2.0 ** k
            polar, norms, prof = polar * 2.0 ** k, norms * 2.0 ** k, prof * 2.0 ** k
            assert bool(polar.isfinite().all()) and float(polar.abs().max()) > 0
            for N in (1, 5):
                ref = tm.match_batch(lib, polar, norms, N, with_best=True)[:3]
                nr = torch.zeros(B, dtype=torch.int32, device="cuda")
                routes = dict(plain={}, bound=dict(coarse="bound"), fft=dict(coarse="fft"),
                              certified=dict(coarse="bound", n_rescored=nr),
                              whole=dict(coarse="bound", n_rescored=nr, rescore_keep=1.0),
                              fourier=dict(coarse="fft", n_rescored=nr))
                for name, kw in routes.items():
                    assert _same(tm.match_batch(lib, polar, norms, N, **kw), ref), (name, N)
                for keep in (0.2, 0.9):
                    kept = tm.prefilter(lib, prof, int(np.ceil(keep * T - 1e-9)), "fp32")
                    cand = torch.cat([kept, kept + T], 1).contiguous()
                    want = tm.match_batch(lib, polar, norms, N, profiles=prof, prefilter_keep=keep)
                    assert _same(want, tm.match_candidates(lib, full, norms, cand, N)), (keep, N)
            b = tm.bound_scores(lib, polar, norms)
            best = tm.match_batch(lib, polar, norms, 1, with_best=True)[3]
            assert bool((b >= best).all())
    lib.free()



# norms that are not the patterns' own, either side of where the window bounds
# stop
@pytest.mark.parametrize("k", (-110, -90, 30, 45, 110))
def test_rows_with_norms_of_another_scale(tm, k):
    import torch
    R, T, B = 34, 2500, 9
    lib_np = small_library(T, seed=T, max_spots=8, g_min=0.08, g_max=1.1)
    grid = tm.PolarGrid(R=R, n_theta=360, cx=33.0, cy=35.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"],
                     (R - 4) / 1.2, grid)
    x = torch.from_numpy(_patterns(lib_np, (R - 4) / 1.2, R, B, seed=B)).cuda()
    polar, norms, _ = tm.polar_transform(x, grid, lib=lib)
    norms = norms * 2.0 ** k
    ref = tm.match_batch(lib, polar, norms, 5, with_best=True)
    assert _same(tm.match_batch(lib, polar, norms, 5), ref[:3])
    assert _same(tm.match_batch(lib, polar, norms, 5, coarse="bound"), ref[:3])
    assert bool((tm.bound_scores(lib, polar, norms) >= ref[3]).all())
    lib.free()
