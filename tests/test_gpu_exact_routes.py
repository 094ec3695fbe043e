"""Every route that promises the plain path's top-N against the exhaustive
scan of the allocation-free entry point, bit for bit, at sizes that reach the
route: refinement of the bounds of dense libraries, their certified
rescoring, and the Fourier kernels' certified rescoring (which run when the
number of templates scored is asked for)."""
import numpy as np
import pytest

from conftest import exhaustive, same_rows, small_library
from test_gpu_search import _patterns

pytestmark = pytest.mark.gpu

R = 34
PX = (R - 4) / 1.2


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2111_07347_amd as tm
    return tm


def _library(tm, n_theta, T, max_spots, **kw):
    lib_np = small_library(T, seed=n_theta + T, max_spots=max_spots, g_min=0.08, g_max=1.1)
    grid = tm.PolarGrid(R=R, n_theta=n_theta, cx=33.0, cy=35.0)
    return tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"], PX, grid,
                      **kw), lib_np, grid


# widths at the ends of what is refined (129 to 384 columns), with and without
# 8 | n_theta; batches of one workgroup per pattern and of several, and the
# first that is not refined (49; 9 of crowded templates, those with more than
# about a pixel per row); templates below and above the least number
@pytest.mark.parametrize("n_theta,rows,T,max_spots,refined", [
    (129, 60, 4200, 60, True), (180, 60, 4200, 70, True), (361, 64, 4100, 70, True),
    (384, 60, 4500, 70, True), (385, 60, 4200, 70, False), (360, 60, 1500, 70, False),
    (180, 34, 4200, 80, False)])
def test_dense_libraries(tm, n_theta, rows, T, max_spots, refined):
    import torch
    lib_np = small_library(T, seed=n_theta + T, max_spots=max_spots, g_min=0.08, g_max=1.1)
    px = (rows - 4) / 1.2
    grid = tm.PolarGrid(R=rows, n_theta=n_theta, cx=62.0, cy=64.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"], px, grid)
    pixels = lib.info()["n_spots"] / lib.n_total
    assert pixels > 24                           # dense, and as the route wants them or not
    assert refined == (lib.n_total >= 8192 and 128 < n_theta <= 384 and pixels < 1.08 * lib.rows()[0])
    for B in (1, 3, 8, 9, 40, 48, 49, 129):
        print("[case] dense", n_theta, rows, T, max_spots, "B", B, flush=True)
        x = torch.from_numpy(_patterns(lib_np, px, rows, B, seed=B, H=128, W=124)).cuda()
        for touched in (lib, None):
            polar, norms, _ = tm.polar_transform(x, grid, lib=touched)
            if B > 4:
                norms[4] = float("nan")
                polar[4, 0, 0] = float("nan")
            for N in (1, 5, 64):
                want = exhaustive(tm, lib, polar, norms, N)
                nr = torch.zeros(B, dtype=torch.int32, device="cuda")
                for kw in ({}, dict(coarse="bound"), dict(coarse="bound", n_rescored=nr)):
                    assert same_rows(tm.match_batch(lib, polar, norms, N, **kw), want), (B, N, kw)
                assert int(nr.min()) >= 0
    lib.free()


@pytest.mark.parametrize("n_theta,T,max_spots", [(90, 40, 25), (180, 300, 12), (360, 600, 8),
                                                 (720, 40, 25)])
def test_fourier_kernels_certified(tm, n_theta, T, max_spots):
    import torch
    lib, lib_np, grid = _library(tm, n_theta, T, max_spots, fft=True)
    for B in (1, 5, 65, 130):
        print("[case] fourier", n_theta, T, max_spots, "B", B, flush=True)
        x = torch.from_numpy(_patterns(lib_np, PX, R, B, seed=B)).cuda()
        for rows in (lib, None):
            polar, norms, _ = tm.polar_transform(x, grid, lib=rows)
            if B > 4:
                norms[4] = float("nan")
                polar[4, 0, 0] = float("nan")
            for N in (1, 5):
                want = exhaustive(tm, lib, polar, norms, N)
                nr = torch.full((B,), -1, dtype=torch.int32, device="cuda")
                got = tm.match_batch(lib, polar, norms, N, coarse="fft", n_rescored=nr)
                assert same_rows(got, want), (B, N)
                live = torch.isfinite(norms)
                assert int(nr[live].min()) >= N and int(nr.max()) <= lib.n_total
    lib.free()


@pytest.mark.parametrize("share", [1, 3])
def test_patterns_without_structure(tm, share):
    """Patterns of which most templates' bounds reach the best scores are given
    up and scanned in full: each in several tasks, or, from 1025 of them on,
    in one."""
    import torch
    lib, lib_np, grid = _library(tm, 360, 1300, 8)
    for B in (1, 40, 1024, 1025, 2049):
        print("[case] noise", share, "B", B, flush=True)
        x = np.resize(_patterns(lib_np, PX, R, min(B, 128), seed=B), (B, 70, 66)).astype(np.float32)
        x[::share] = np.random.default_rng(B).standard_normal(x[::share].shape)
        polar, norms, prof = tm.polar_transform(torch.from_numpy(x).cuda(), grid)
        for N in (1, 5, 64):
            want = exhaustive(tm, lib, polar, norms, N)
            for kw in ({}, dict(coarse="bound"),
                       dict(coarse="bound", n_rescored=torch.zeros(B, dtype=torch.int32, device="cuda"))):
                assert same_rows(tm.match_batch(lib, polar, norms, N, **kw), want), (B, N, kw)
        kept = tm.prefilter(lib, prof, 650, "fp32")
        cand = torch.cat([kept, kept + 1300], 1).contiguous()
        got = tm.match_batch(lib, polar, norms, 5, profiles=prof, prefilter_keep=0.5)
        assert same_rows(got, tm.match_candidates(lib, polar, norms, cand, 5)), B
    lib.free()


# batches around a workgroup per compute unit (256), half and one and a half
# of that, and what a compute unit's LDS holds; libraries whose rows leave room
# for several workgroups or fill it, short scans and long ones
@pytest.mark.parametrize("n_theta,rows,T,max_spots", [(360, 34, 200, 12), (180, 34, 1500, 12),
                                                      (360, 48, 70, 60), (361, 60, 400, 90)])
def test_scans_split_over_workgroups(tm, n_theta, rows, T, max_spots):
    import torch
    lib_np = small_library(T, seed=n_theta + T, max_spots=max_spots, g_min=0.08, g_max=1.1)
    px = (rows - 4) / 1.2
    grid = tm.PolarGrid(R=rows, n_theta=n_theta, cx=33.0, cy=35.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"], px, grid)
    x = torch.from_numpy(_patterns(lib_np, px, rows, 96, seed=7)).cuda()
    every, nall, _ = tm.polar_transform(x, grid, lib=lib)
    nall[4] = float("nan")
    every[4, 0, 0] = float("nan")
    for B in (1, 2, 44, 100, 128, 129, 256, 257, 384, 385, 448, 449, 513, 1025):
        print("[case] split", n_theta, rows, T, "B", B, flush=True)
        at = torch.arange(B, device="cuda") % 96
        polar, norms = every[at].contiguous(), nall[at].contiguous()
        N = min(7, 2 * T)
        want = exhaustive(tm, lib, polar, norms, N)
        got = tm.match_batch(lib, polar, norms, N, with_best=True)
        assert same_rows(got[:3], want), B
        assert same_rows(tm.match_batch(lib, polar, norms, N), want), B
        live = torch.isfinite(norms)
        assert torch.equal(got[3][live].amax(1), want[2][live][:, 0]), B
        assert torch.equal(got[3][live].gather(1, want[0][live].long()), want[2][live]), B
        assert torch.equal(got[4][live].gather(1, want[0][live].long()).int(), want[1][live]), B
        assert bool(got[3][~live].isnan().all()) and bool((got[4][~live] == -1).all())
    lib.free()


# on either side of the rule that sends the plain path of a sparse library to
# its search, and of those that leave the search for the certified passes (few
# columns over a multiple of the windows, many pixels per template)
@pytest.mark.parametrize("n_theta,T,max_spots,Bs", [
    (90, 2200, 8, (64, 127, 128, 700, 1500)), (72, 2200, 8, (128, 1500)), (180, 1500, 8, (300, 700, 1400)),
    (220, 900, 34, (500, 2047, 2048)), (240, 170, 34, (1024, 4096)),
    (360, 700, 8, (60, 300, 900, 1700)), (720, 600, 34, (100, 300, 900))])
def test_sparse_libraries_by_scan_search_or_certified(tm, n_theta, T, max_spots, Bs):
    import torch
    lib, lib_np, grid = _library(tm, n_theta, T, max_spots)
    assert lib.info()["n_spots"] <= 24 * lib.n_total
    x = torch.from_numpy(_patterns(lib_np, PX, R, 96, seed=3)).cuda()
    every, nall, _ = tm.polar_transform(x, grid, lib=lib)
    for B in Bs:
        print("[case] sparse", n_theta, T, max_spots, "B", B, flush=True)
        at = torch.arange(B, device="cuda") % 96
        polar, norms = every[at].contiguous(), nall[at].contiguous()
        for N in (1, 6):
            want = exhaustive(tm, lib, polar, norms, N)
            for kw in ({}, dict(coarse="bound")):
                assert same_rows(tm.match_batch(lib, polar, norms, N, **kw), want), (B, N, kw)
    lib.free()


# crowded libraries, one with about a pixel per row and template and one with
# fewer; patterns on either side of the rules that choose between scan, search
# and, for certified Fourier calls without counts, the Fourier kernels
@pytest.mark.parametrize("n_theta,rows,T,max_spots", [(180, 34, 4200, 80), (360, 34, 2600, 80),
                                                      (180, 34, 3900, 51), (180, 60, 2600, 70),
                                                      (386, 34, 2000, 80)])
def test_dense_libraries_by_scan_search_or_fourier(tm, n_theta, rows, T, max_spots):
    import torch
    lib_np = small_library(T, seed=n_theta + T, max_spots=max_spots, g_min=0.08, g_max=1.1)
    px = (rows - 4) / 1.2
    grid = tm.PolarGrid(R=rows, n_theta=n_theta, cx=62.0, cy=64.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"], px, grid, fft=True)
    info = lib.info()
    print("pixels per row and template", info["n_spots"] / lib.n_total / lib.rows()[0], lib.layout(), flush=True)
    assert info["n_spots"] > 24 * lib.n_total and lib.layout()["n_records"] >= 131072
    x = torch.from_numpy(_patterns(lib_np, px, rows, 512, seed=5, H=128, W=124)).cuda()
    every, nall, _ = tm.polar_transform(x, grid, lib=lib)
    for B in (1, 9, 24, 25, 49, 100, 200, 512):
        print("[case] dense", n_theta, rows, T, max_spots, "B", B, flush=True)
        polar, norms = every[:B], nall[:B]
        for N in (1, 5):
            want = exhaustive(tm, lib, polar, norms, N)
            for kw in ({}, dict(coarse="bound"), dict(coarse="fft")):
                assert same_rows(tm.match_batch(lib, polar, norms, N, **kw), want), (B, N, kw)
    lib.free()
