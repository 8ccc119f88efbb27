"""GPU parity of the tile kernel (most automatic calls).

One shape per built configuration, each with ragged ends where the
configuration has an edge: rows that do not fill a wavefront's row blocks or
the workgroup, LTs that do not fill a chunk of four or split unevenly over the
K slices, columns that do not fill a block or a tile. The shapes are chosen so
that the automatic choice takes the configuration named beside them on a
256-CU GPU. INT32 results are exact and the dequantised ones are compared bit
for bit with the oracle.
"""
import numpy as np
import pytest

from paper_2608_09291_amd import binding, synth
from test_gpu_spmm import announce, check, run_spmm, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# (M, K, N): row blocks x column blocks, wavefronts along M, K slices
SHAPES = [
    (16, 192, 7),           # 1 x 1, 1, 2; a single row block, one LT in one slice
    (16, 320, 3),           # 1 x 1, 1, 4
    (48, 1088, 9),          # 1 x 1, 1, 8
    (80, 6848, 12),         # 1 x 1, 1, 16
    (12592, 2688, 9),       # 2 x 1, 1, 4
    (16, 320, 17),          # 1 x 1, 1, 4; two column tiles
    (80, 1088, 29),         # 1 x 1, 1, 8
    (16, 128, 17),          # 1 x 2, 1, 2
    (4112, 320, 17),        # 1 x 2, 1, 4
    (1616, 1088, 33),       # 1 x 2, 1, 8
    (12304, 576, 33),       # 2 x 2, 1, 4
    (12304, 320, 65),       # 2 x 3, 1, 2
    (6416, 1088, 33),       # 2 x 3, 1, 4
    (16, 64, 50),           # 2 x 4, 1, 1; one LT, half a row group
    (6416, 576, 100),       # 2 x 4, 1, 4
    (4112, 8320, 50),       # 2 x 4, 1, 8
    (12304, 1984, 250),     # 4 x 4, 2, 2
    (12304, 704, 200),      # 2 x 8, 4, 1
    (4112, 64, 1021),       # 3 x 8, 4, 1
]


@pytest.mark.parametrize("form", ["plain", "reordered", "w2"])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_every_configuration(torch_cuda, M, K, N, form):
    announce(f"tile {form} M={M} K={K} N={N}")
    bits = 2 if form == "w2" else 4
    W, Xt, sc = synth.random_problem(M, K, N, 0.5, M + K + N, bits=bits)
    Y, Yf = run_spmm(torch_cuda, W, Xt, sc, reorder=form == "reordered", bits=bits)
    check(Y, Yf, W, Xt, sc)


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


@pytest.mark.parametrize("M,K,N", [(8208, 16704, 1000), (4112, 66304, 500)])
def test_long_slices(torch_cuda, M, K, N):
    """Slices of more than 64 chunks, whose payload ranges are worked out in
    several steps, against a forced chunked configuration (which the other
    tests compare with the oracle) on the same encoded matrix."""
    torch = torch_cuda
    announce(f"tile long M={M} K={K} N={N}")
    W, Xt, _ = synth.random_problem(M, 1024, N, 0.5, 11)
    W = np.ascontiguousarray(np.tile(W, (1, K // 1024 + 1))[:, :K])
    Xt = synth.random_problem(16, K, N, 0.5, 12)[1]
    dev = binding.to_device(binding.encode(W))
    xp = torch.from_numpy(binding.pack_int4(Xt)).cuda()
    y = torch.full((N, M), -1, dtype=torch.int32, device="cuda")
    y0 = torch.full((N, M), -2, dtype=torch.int32, device="cuda")
    binding.spmm(dev, xp, N, y)
    binding.spmm(dev, xp, N, y0, variant=1)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)
