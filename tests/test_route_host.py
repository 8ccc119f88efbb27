"""us_spmm_route, us_gemm_i8_route: what a call launches (host only; 256 compute units when no GPU is visible)."""
import argparse
import ctypes
import os
import random
import re
import time

import pytest

import bench
import test_gpu_gemm
import test_gpu_tile
from paper_2608_09291_amd import binding, build, synth

FORMS = [(4, False), (4, True), (2, False)]


@pytest.mark.parametrize("M,K,N,kernel,launches", [
    (4096, 11008, 8, "us_spmm_kernel", 1),             # a narrow call in one chunk per wavefront
    (28672, 8192, 1, "us_spmm_tile_kernel", 1),
    (28672, 8192, 32, "us_spmm_tile_kernel", 1),
    (12288, 4096, 1024, "us_spmm_tile_kernel", 1),
    # Narrow calls that the tile kernel splits no further, or hardly, than the chunked one does ...
    (7536, 2496, 16, "us_spmm_kernel", 1),
    (5120, 2432, 11, "us_spmm_kernel", 1),
    (3296, 4800, 12, "us_spmm_kernel", 1),
    (10832, 1536, 4, "us_spmm_kernel", 1),
    (23184, 896, 3, "us_spmm_kernel", 1),
    # ... and some that it does, or with fewer row blocks, or wider
    (5040, 1216, 12, "us_spmm_tile_kernel", 1),
    (880, 4992, 15, "us_spmm_tile_kernel", 1),
    (10832, 1536, 5, "us_spmm_tile_kernel", 1),
    (26640, 768, 3, "us_spmm_tile_kernel", 1),
    (4096, 11008, 12, "us_spmm_tile_kernel", 1),
    # Many row blocks of few LTs, and some that the tile kernel runs faster
    (1048576, 128, 1, "us_spmm_kernel", 1),
    (1048576, 128, 32, "us_spmm_kernel", 1),
    (49152, 256, 16, "us_spmm_kernel", 1),
    (262144, 768, 1, "us_spmm_kernel", 1),
    (131072, 320, 32, "us_spmm_kernel", 1),
    (34816, 128, 32, "us_spmm_kernel", 1),
    (38912, 256, 8, "us_spmm_kernel", 1),
    (45056, 768, 4, "us_spmm_kernel", 1),
    (49136, 512, 8, "us_spmm_kernel", 1),
    (28672, 256, 16, "us_spmm_tile_kernel", 1),
    (32768, 128, 32, "us_spmm_tile_kernel", 1),
    (34816, 256, 8, "us_spmm_tile_kernel", 1),
    (40960, 512, 1, "us_spmm_tile_kernel", 1),
    (262144, 512, 8, "us_spmm_tile_kernel", 1),
    (262144, 320, 16, "us_spmm_tile_kernel", 1),
    (262144, 768, 24, "us_spmm_tile_kernel", 1),
    (262144, 256, 100, "us_spmm_tile_kernel", 1),
    (4096, 64, 40, "us_spmm_kernel", 2),               # one LT per row block: no tile of that width
    (4096, 64, 49, "us_spmm_tile_kernel", 1),
    ((1 << 22) + 16, 64, 1024, "us_spmm_kernel", 32),  # Y beyond the tile kernel's offsets
])
def test_kernel_of_automatic_calls(M, K, N, kernel, launches):
    r = binding.spmm_route(M, K, N)
    assert (binding.KERNELS[r["kernel"]], r["launches"]) == (kernel, launches)


@pytest.mark.parametrize("bits,reordered", FORMS)
def test_agrees_with_the_plan_off_the_tile_kernel(bits, reordered):
    chunked = 0
    for M, K in ((16, 64), (512, 512), (1024, 4096), (4096, 11008), (12288, 4096), (48, 130048)):
        for N in (1, 4, 8, 12, 16, 17, 32, 33):
            for opts in ({}, {"split_k": 2, "chunk_lts": 4}, {"variant": 1}, {"split_k": 4, "variant": 3}):
                try:
                    plan = binding.spmm_plan(M, K, N, bits=bits, reordered=reordered, **opts)
                except binding.UsError as e:
                    with pytest.raises(binding.UsError) as e2:
                        binding.spmm_route(M, K, N, bits=bits, reordered=reordered, **opts)
                    assert e2.value.status == e.status
                    continue
                r = binding.spmm_route(M, K, N, bits=bits, reordered=reordered, **opts)
                if binding.KERNELS[r["kernel"]] == "us_spmm_tile_kernel":
                    assert not opts and r["launches"] == 1 and r["split_k"] <= K // 64
                    continue
                chunked += 1
                assert (r["split_k"], r["chunk_lts"]) == plan[:2]
                assert (binding.KERNELS[r["kernel"]] == "us_spmm_burst_kernel") == (plan[2] == 3)
                assert r["launches"] == -(-N // 32) and r["col_blocks"] == (2 if N > 16 else 1)
    assert chunked > 0


def test_argument_errors():
    L, ok, out = binding.lib(), ctypes.byref(binding.SpmmOpts()), ctypes.byref(binding.RouteInfo())
    assert L.us_spmm_route(32, 128, 8, 4, 0, None, out) == 0
    assert L.us_spmm_route(32, 128, 8, 4, 0, ok, None) == -1
    assert L.us_spmm_route(32, 128, 8, 3, 0, ok, out) == -1
    assert L.us_spmm_route(32, 128, 8, 2, 1, ok, out) == -1
    assert L.us_spmm_route(40, 128, 8, 4, 0, ok, out) == -2
    assert L.us_spmm_route(32, 128, 1025, 4, 0, ok, out) == -2
    assert L.us_spmm_route(32, 128, 8, 4, 0, ctypes.byref(binding.SpmmOpts(3)), out) == -1


@pytest.mark.parametrize("workload,N,kernel", [("ffn_down_4096x11008_s50", 8, "us_spmm_kernel"),
                                               ("ffn_28672x8192_s70", 32, "us_spmm_tile_kernel")])
def test_bench_reports_the_kernel_it_times(workload, N, kernel):
    args = argparse.Namespace(split_k=0, variant=0, reorder=False, bits=4, chunk_lts=0, k_blocks=0)
    w = synth.WORKLOADS[workload]
    out = bench.launched(w, N, args)
    r = binding.spmm_route(w.M, w.K, N)
    assert out["kernel"] == kernel and out["split_k"] == r["split_k"] and out["chunk_lts"] == r["chunk_lts"]
    assert (out["staging"] == "tile") == (kernel == "us_spmm_tile_kernel")


def built(header, macro, fields):
    """The configurations a header lists, cut to `fields` of their columns."""
    text = open(os.path.join(build.CSRC, header)).read()
    body = re.search(r"#define " + macro + r"\(X\)(.*?)\n\n", text, re.S).group(1)
    return [tuple(int(row.split(",")[k]) for k in fields) for row in re.findall(r"X\(([^)]*)\)", body)]


@pytest.mark.parametrize("form", ["plain", "reordered", "w2"])
def test_tile_tests_run_every_configuration(form):
    cfgs = built("us_spmm_tile.h", "US_TILE_CFGS", range(4))
    assert len(set(cfgs)) == len(cfgs) == 17
    for M, K, N, cfg in test_gpu_tile.SHAPES:
        assert test_gpu_tile.tile_config(M, K, N, form) == cfg, (M, K, N)
    assert {s[3] for s in test_gpu_tile.SHAPES} == set(cfgs)
    # The long-slice cases: more than 64 chunks of four LTs, and a last chunk that is empty for one slice.
    for M, K, N in ((8208, 16704, 1000), (4112, 66304, 500)):
        assert -(-(K // 64 // test_gpu_tile.tile_config(M, K, N, form)[3]) // 4) > 64
    assert test_gpu_tile.tile_config(15408, 8256, 200, form) == (4, 4, 2, 2)


def test_gemm_tests_run_every_configuration():
    cfgs = built("us_gemm.h", "US_GEMM_CFGS", range(5))
    assert len(set(cfgs)) == len(cfgs) == 13
    for M, K, N, cfg in test_gpu_gemm.SHAPES:
        assert tuple(binding.gemm_i8_route(M, K, N).values()) == cfg, (M, K, N)
    assert {s[3] for s in test_gpu_gemm.SHAPES} == set(cfgs)


@pytest.mark.parametrize("M,K,N,row_blocks,split_k", [
    # Large matrices at few columns: slower than the kernel before this one without K slices, or with four long ones
    (28672, 4096, 1, 1, 4), (28672, 8192, 8, 1, 4), (53248, 4096, 1, 1, 4), (28672, 1536, 1, 1, 4),
    (28688, 1024, 1, 1, 4), (32752, 2048, 8, 1, 4),
    (28672, 11008, 1, 2, 8), (16384, 16384, 1, 2, 8),
    # or with more than one generation of eight
    (12288, 8192, 1, 1, 4), (11280, 8192, 8, 1, 4),
    # and those that it keeps
    (28672, 768, 1, 1, 1), (32768, 2048, 1, 1, 1), (49152, 2048, 1, 1, 1), (12288, 256, 1, 1, 1), (28672, 2048, 16, 1, 1), (8192, 8192, 1, 2, 8),
    (4096, 11008, 8, 1, 8),
])
def test_gemm_choice_of_large_narrow_products(M, K, N, row_blocks, split_k):
    r = binding.gemm_i8_route(M, K, N)
    assert (r["row_blocks"], r["split_k"]) == (row_blocks, split_k)


def test_gemm_grids_can_be_launched():
    # A grid holds fewer than 2^32 threads. Every product that fits 288 GB of
    # HBM, for M below 2^30, as with one row block per 64 threads.
    rng = random.Random(1)
    shapes = [(1 << 28, 64, 49), (1 << 29, 64, 17), ((1 << 30) - 16, 64, 1), (1 << 27, 256, 32)]
    while len(shapes) < 20000:
        M, K, N = (int(2 ** rng.uniform(a, b)) for a, b in ((14, 26), (0, 11), (0, 10)))
        M, K = 16 * M, 64 * K
        if K <= 130048 and M * K + 4 * M * N + K * N <= 288e9:
            shapes.append((M, K, N))
    for M, K, N in shapes:
        r = binding.gemm_i8_route(M, K, N)
        groups, tiles = -(-M // (16 * r["row_blocks"] * r["waves_m"])), -(-N // (16 * r["col_blocks"] * r["waves_n"]))
        threads = 64 * r["waves_m"] * r["waves_n"] * r["split_k"]
        assert 8 * -(-groups // 8) * tiles * threads < 1 << 32, (M, K, N, r)


def test_gemm_argument_errors():
    L, out = binding.lib(), ctypes.byref(binding.GemmRouteInfo())
    assert L.us_gemm_i8_route(32, 128, 8, None) == -1
    for M, K, N in ((40, 128, 8), (32, 96, 8), (32, 128, 0), (32, 128, 1025), (0, 64, 1), (16, 130048 + 64, 1)):
        assert L.us_gemm_i8_route(M, K, N, out) == -2
    assert L.us_gemm_i8_route(16, 130048, 1024, out) == 0


def test_narrow_calls_search_for_a_plan_once():
    """Routing a narrow call and planning its launch share one search over
    the chunked configurations: the route costs about what us_spmm_plan
    (one search) does, not two or three times as much."""
    L, out = binding.lib(), binding.RouteInfo()
    a, b, c = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
    ra, rb, rc, ro = ctypes.byref(a), ctypes.byref(b), ctypes.byref(c), ctypes.byref(out)

    def best(call):
        times = []
        for _ in range(30):
            t = time.perf_counter()
            for _ in range(200):
                call()
            times.append(time.perf_counter() - t)
        return min(times)

    for M, K, N in ((4096, 11008, 8), (2048, 8192, 4)):
        assert binding.KERNELS[binding.spmm_route(M, K, N)["kernel"]] == "us_spmm_kernel"
        ratios = []
        for _ in range(8):                                 # (one quiet attempt shows it on a busy host)
            search, route = (best(lambda: f(M)) - best(lambda: f(40))      # M = 40 is refused before the search
                             for f in (lambda m: L.us_spmm_plan(m, K, N, 4, 0, None, ra, rb, rc, None),
                                       lambda m: L.us_spmm_route(m, K, N, 4, 0, None, ro)))
            ratios.append(route / search if search > 0 else float("inf"))
            if ratios[-1] < 1.5:
                break
        assert ratios[-1] < 1.5, (M, K, N, ratios)
