"""GPU parity of the tile kernel (most automatic calls).

At least one shape per built configuration, in every weight form, with ragged
ends where the configuration has an edge: rows that do not fill a wavefront's
row blocks or the workgroup, LTs that do not fill a chunk of four or split
unevenly over the K slices, columns that do not fill a block or a tile. The
shapes are chosen so that the automatic choice takes the configuration given
with them on a 256-CU GPU (test_route_host.py and, on such a GPU, the test
below assert it). INT32 results are exact and the dequantised ones are
compared bit for bit with the oracle.
"""
import numpy as np
import pytest

from paper_2608_09291_amd import binding, synth
from test_gpu_spmm import announce, check, run_spmm, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# M, K, N, (row blocks, column blocks per wavefront, wavefronts along M, K slices)
SHAPES = [
    (16, 192, 7, (1, 1, 1, 2)),             # a single row block, one LT in one slice
    (12448, 2112, 1, (1, 1, 1, 2)),
    (16, 320, 3, (1, 1, 1, 4)),
    (48, 1088, 9, (1, 1, 1, 8)),
    (80, 6848, 12, (1, 1, 1, 16)),
    (12400, 3008, 9, (2, 1, 1, 4)),
    (16, 320, 17, (1, 1, 1, 4)),            # two column tiles
    (80, 1088, 29, (1, 1, 1, 8)),
    (16, 128, 17, (1, 1, 1, 2)),
    (4112, 320, 17, (1, 1, 1, 2)),
    (9152, 1088, 18, (1, 2, 1, 2)),
    (4352, 1408, 17, (1, 2, 1, 4)),
    (1616, 1088, 33, (1, 2, 1, 8)),
    (13136, 1728, 17, (2, 2, 1, 4)),
    (9872, 1088, 65, (2, 3, 1, 2)),
    (12304, 576, 33, (2, 3, 1, 4)),
    (6416, 1088, 33, (1, 1, 1, 2)),         # three column tiles
    (16, 64, 50, (2, 4, 1, 1)),             # one LT, half a row group
    (11056, 320, 121, (2, 4, 1, 1)),
    (12304, 704, 200, (2, 4, 1, 1)),
    (12304, 1984, 250, (2, 4, 1, 1)),
    (6416, 576, 100, (2, 4, 1, 4)),
    (4112, 8320, 50, (2, 4, 1, 8)),
    (6448, 4928, 521, (4, 4, 2, 2)),        # shared activations and split K; uneven slices
    (12320, 320, 195, (2, 8, 4, 1)),
    (4112, 64, 1021, (2, 8, 4, 1)),         # one LT
    (14000, 128, 778, (3, 8, 4, 1)),        # one chunk, half empty
    (13968, 320, 845, (3, 8, 4, 1)),
]
# Shapes on which the weight forms take different configurations.
MIXED = [(12592, 2688, 9), (12304, 320, 65)]


@pytest.mark.parametrize("form", ["plain", "reordered", "w2"])
@pytest.mark.parametrize("M,K,N,cfg", SHAPES + [(*s, None) for s in MIXED])
def test_every_configuration(torch_cuda, M, K, N, cfg, form):
    announce(f"tile {form} M={M} K={K} N={N}")
    bits = 2 if form == "w2" else 4
    if cfg and torch_cuda.cuda.get_device_properties(0).multi_processor_count == 256:
        assert tile_config(M, K, N, form) == cfg
    W, Xt, sc = synth.random_problem(M, K, N, 0.5, M + K + N, bits=bits)
    Y, Yf = run_spmm(torch_cuda, W, Xt, sc, reorder=form == "reordered", bits=bits)
    check(Y, Yf, W, Xt, sc)


def tile_config(M, K, N, form):
    """The tile configuration of an automatic call, None if it takes another kernel."""
    r = binding.spmm_route(M, K, N, reordered=form == "reordered", bits=2 if form == "w2" else 4)
    tile = binding.KERNELS[r["kernel"]] == "us_spmm_tile_kernel"
    return (r["row_blocks"], r["col_blocks"], r["waves_m"], r["split_k"]) if tile else None


@pytest.mark.parametrize("form", ["plain", "reordered", "w2"])
@pytest.mark.parametrize("s", [0.0, 0.02, 0.97, 1.0])
def test_extreme_densities(torch_cuda, form, s):
    """Full chunks (whose payload takes one more load) down to no payload at all."""
    bits = 2 if form == "w2" else 4
    for M, K, N in ((80, 1088, 29), (12304, 192, 70), (208, 704, 300)):
        announce(f"tile {form} s={s} M={M} K={K} N={N}")
        W, Xt, sc = synth.random_problem(M, K, N, s, 7 + N, bits=bits)
        Y, Yf = run_spmm(torch_cuda, W, Xt, sc, reorder=form == "reordered", bits=bits)
        check(Y, Yf, W, Xt, sc)


@pytest.mark.parametrize("M,K,N,form", [
    (8208, 16704, 1000, "plain"), (4112, 66304, 500, "plain"),
    # 129 LTs in two slices of 4 x 4 blocks: 17 chunks, of which one slice's last is empty
    (15408, 8256, 200, "plain"), (15408, 8256, 200, "reordered"), (15408, 8256, 200, "w2"),
])
def test_long_slices(torch_cuda, M, K, N, form):
    """Slices of many chunks (above 64 their payload ranges are worked out in
    several steps) against a forced chunked configuration (which the other
    tests compare with the oracle) on the same encoded matrix."""
    torch = torch_cuda
    announce(f"tile long {form} M={M} K={K} N={N}")
    bits = 2 if form == "w2" else 4
    if K == 8256 and torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert tile_config(M, K, N, form) == (4, 4, 2, 2)
    W, Xt, _ = synth.random_problem(M, 1024, N, 0.5, 11, bits=bits)
    W = np.ascontiguousarray(np.tile(W, (1, K // 1024 + 1))[:, :K])
    Xt = synth.random_problem(16, K, N, 0.5, 12)[1]
    dev = binding.to_device(binding.encode(W, reorder=form == "reordered", bits=bits))
    xp = torch.from_numpy(binding.pack_int4(Xt)).cuda()
    y = torch.full((N, M), -1, dtype=torch.int32, device="cuda")
    y0 = torch.full((N, M), -2, dtype=torch.int32, device="cuda")
    binding.spmm(dev, xp, N, y)
    binding.spmm(dev, xp, N, y0, variant=1)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)


def test_most_rows(torch_cuda):
    """The most rows the tile kernel takes: a column tile of Y is 2^31 bytes.
    The matrix repeats 4096 rows, and so do the columns of Y."""
    torch = torch_cuda
    M, K, N, rep = 1 << 22, 64, 150, 4096
    announce(f"tile M={M} K={K} N={N}")
    assert tile_config(M, K, N, "plain") and not tile_config(M + 16, K, N, "plain")
    W, Xt, sc = synth.random_problem(rep, K, N, 0.5, 13)
    dev = binding.to_device(binding.encode(np.tile(W, (M // rep, 1))))
    xp, scale = torch.from_numpy(binding.pack_int4(Xt)).cuda(), torch.from_numpy(np.tile(sc, M // rep)).cuda()
    y = torch.full((N, M), -1, dtype=torch.int32, device="cuda")
    yf = torch.full((N, M), float("nan"), dtype=torch.float32, device="cuda")
    binding.spmm(dev, xp, N, y, scale, yf)
    torch.cuda.synchronize()
    check(y[:, :rep].cpu().numpy().T, yf[:, :rep].cpu().numpy().T, W, Xt, sc)
    for v in (y, yf):
        v = v.view(N, M // rep, rep)
        assert bool((v == v[:, :1]).all())


@pytest.mark.parametrize("form", ["plain", "reordered", "w2"])
@pytest.mark.parametrize("M,K,N", [
    (7536, 2496, 16), (3312, 4800, 12),                 # one 11-LT chunk per wavefront
    (10832, 1536, 4), (23184, 896, 3),                  # short slices, two row blocks
    (41008, 128, 17), (49168, 192, 32), (49168, 256, 1),            # row blocks of few LTs
    (81936, 704, 3), (49168, 384, 7), (131088, 384, 25), (34816, 128, 29), (45072, 768, 2),
])
def test_calls_the_chunked_kernel_keeps(torch_cuda, M, K, N, form):
    """Both sides of the rules that keep narrow calls off the tile kernel."""
    announce(f"route {form} M={M} K={K} N={N}")
    if form == "plain" and torch_cuda.cuda.get_device_properties(0).multi_processor_count == 256:
        assert tile_config(M, K, N, form) is None
    bits = 2 if form == "w2" else 4
    W, Xt, sc = synth.random_problem(M, K, N, 0.5, M + K + N, bits=bits)
    Y, Yf = run_spmm(torch_cuda, W, Xt, sc, reorder=form == "reordered", bits=bits)
    check(Y, Yf, W, Xt, sc)
