"""The plain path's top-N by search (tm_match_batch without per-template
outputs), the window-bound route and the pre-filter's rescoring against the
exhaustive kernel on the same polar images (per-template outputs asked for,
the allocation-free entry point, explicit candidate lists): the same rows bit
for bit, at the sizes where the routes and their layouts change."""
import ctypes

import numpy as np
import pytest

from conftest import small_library

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2111_07347_amd as tm
    return tm


def _patterns(lib, px, R, B, seed, H=70, W=66):
    """Rendered templates with noise; among them a blank, a constant and a
    noise pattern (which many templates' bounds reach)."""
    rng = np.random.default_rng(seed)
    yy, xx = np.mgrid[0:H, 0:W]
    imgs = 0.02 * rng.standard_normal((B, H, W)).astype(np.float32)
    for b in range(B):
        t = int(rng.integers(0, len(lib["offsets"]) - 1))
        a, e = lib["offsets"][t], lib["offsets"][t + 1]
        phi = rng.uniform(0, 2 * np.pi)
        x = W / 2 + px * (np.cos(phi) * lib["kx"][a:e] - np.sin(phi) * lib["ky"][a:e])
        y = H / 2 + px * (np.sin(phi) * lib["kx"][a:e] + np.cos(phi) * lib["ky"][a:e])
        for xc, yc, w in zip(x, y, lib["intensity"][a:e]):
            imgs[b] += w * np.exp(-((xx - xc) ** 2 + (yy - yc) ** 2) / 4.5)
    if B > 3:
        imgs[1] = 0.0
        imgs[2] = 0.25
        imgs[3] = rng.standard_normal((H, W))
    return imgs


def _same(a, b):
    import torch
    return all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))


# sparse libraries of few and of many templates (16 bits hold a bound's
# column), dense ones below and above the sizes that are refined, widths with
# and without 8 | n_theta, more than one window per wave (n_theta > 512)
CASES = [(64, 2500, 8), (65, 2600, 6), (127, 2200, 8), (360, 2500, 8), (361, 900, 20),
         (720, 2300, 8), (768, 2100, 5), (360, 9000, 4), (360, 700, 40), (180, 4200, 40)]


@pytest.mark.parametrize("n_theta,T,max_spots", CASES)
def test_search_equals_exhaustive_kernel(tm, n_theta, T, max_spots):
    import torch
    R = 34
    lib_np = small_library(T, seed=n_theta + T, max_spots=max_spots, g_min=0.08, g_max=1.1)
    px = (R - 4) / 1.2
    grid = tm.PolarGrid(R=R, n_theta=n_theta, cx=33.0, cy=35.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"], px, grid)
    for B in (1, 40, 300):
        print("[case] search", n_theta, T, max_spots, "B", B, flush=True)
        x = torch.from_numpy(_patterns(lib_np, px, R, B, seed=B)).cuda()
        for rows in (lib, None):
            polar, norms, prof = tm.polar_transform(x, grid, lib=rows)
            if B > 4:
                norms[4] = float("nan")
                polar[4, 0, 0] = float("nan")
            for N in (1, 5, 64):
                ref = tm.match_batch(lib, polar, norms, N, with_best=True)[:3]
                assert _same(tm.match_batch(lib, polar, norms, N), ref)
                assert _same(tm.match_batch(lib, polar, norms, N, coarse="bound"), ref)
        # the pre-filter's kept templates (and their mirrors)
        for keep in (0.15, 0.9):
            n_keep = int(np.ceil(keep * T - 1e-9))
            kept = tm.prefilter(lib, prof, n_keep, "fp16")
            cand = torch.cat([kept, kept + T], 1).contiguous()
            got = tm.match_batch(lib, polar, norms, 5, profiles=prof, prefilter_keep=keep,
                                 prefilter_prec="fp16")
            assert _same(got, tm.match_candidates(lib, polar, norms, cand, 5))
    lib.free()


def test_search_equals_allocation_free_scan_and_replays(tm):
    """The allocation-free entry scans; a captured call scans, too, and its
    replays equal the eager result."""
    import torch
    R, n_theta, T, B, N = 34, 360, 2500, 24, 5
    lib_np = small_library(T, seed=5, max_spots=8, g_min=0.08, g_max=1.1)
    px = (R - 4) / 1.2
    grid = tm.PolarGrid(R=R, n_theta=n_theta, cx=33.0, cy=35.0)
    lib = tm.Library(lib_np["kx"], lib_np["ky"], lib_np["intensity"], lib_np["offsets"], px, grid)
    x = torch.from_numpy(_patterns(lib_np, px, R, B, seed=9)).cuda()
    polar, norms, _ = tm.polar_transform(x, grid, lib=lib)
    eager = tm.match_batch(lib, polar, norms, N)
    out = [torch.zeros_like(o) for o in eager]
    o = tm._Opts(compact_rows=1)
    print("[case] allocation-free scan", flush=True)
    r = tm._lib.tm_match_batch_static(lib._h, polar.data_ptr(), norms.data_ptr(), None, B,
                                      ctypes.byref(o), N, *(v.data_ptr() for v in out), None, None,
                                      torch.cuda.current_stream().cuda_stream)
    assert r == tm.TM_OK, tm.last_error()
    assert _same(out, eager)
    print("[case] captured plain path", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        tm.match_batch(lib, polar, norms, N, out=tuple(out))
    for k in range(3):
        polar.copy_(torch.roll(polar, 1, dims=0))
        norms.copy_(torch.roll(norms, 1))
        g.replay()
        torch.cuda.synchronize()
        assert _same(out, tm.match_batch(lib, polar, norms, N)), k
    lib.free()
