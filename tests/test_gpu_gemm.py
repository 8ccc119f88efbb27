"""GPU parity of every built configuration of the dense INT8 GEMM.

The shapes are chosen so that the automatic choice takes the configuration
given with them on a 256-CU GPU (test_route_host.py and, on such a GPU, the
test below assert it), with rows, columns and k that do not fill its tiles,
chunks or slices. Results are exact.
"""
import numpy as np
import pytest

from oracle import product
from paper_2608_09291_amd import binding
from test_gpu_spmm import announce, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# M, K, N, (row blocks, column blocks, wavefronts along M, along N, K slices)
SHAPES = [
    (48, 64, 4, (1, 1, 1, 1, 1)),
    (16, 576, 4, (1, 1, 1, 1, 8)),
    (16, 320, 21, (1, 1, 1, 1, 4)),
    (4528, 320, 1, (2, 1, 1, 1, 4)),
    (5584, 2752, 1, (2, 1, 1, 1, 8)),
    (4112, 320, 17, (2, 2, 1, 1, 4)),
    (4208, 576, 18, (2, 2, 1, 1, 8)),
    (8880, 832, 17, (4, 2, 1, 1, 4)),
    (9808, 1600, 17, (4, 2, 1, 1, 8)),
    (10032, 448, 132, (4, 4, 1, 1, 4)),
    (7024, 704, 100, (4, 4, 1, 1, 8)),
    (10704, 64, 98, (2, 4, 2, 2, 1)),
    (8464, 64, 652, (4, 4, 2, 2, 1)),
    (8208, 704, 200, (2, 4, 2, 2, 1)),      # several chunks
    (12304, 704, 500, (4, 4, 2, 2, 1)),     # several chunks
    (48, 130048, 3, (1, 1, 1, 1, 8)),       # the longest k
    # large matrices at up to 8 columns
    (28688, 1600, 1, (1, 1, 1, 1, 4)),
    (8720, 8128, 5, (1, 1, 1, 1, 4)),
    (16400, 8256, 3, (2, 1, 1, 1, 8)),
]


# More than 64 KB of LDS (4 x 4 blocks, 8 slices; its limit is set by the
# first call), less of it, and several wavefronts sharing it.
CAPTURED = [(7024, 704, 100), (16, 320, 21), (8208, 704, 200)]


def test_captured(torch_cuda):
    """Calls captured in a graph before any other call of their shapes, and
    replayed on changed activations, with eager calls between the replays."""
    torch = torch_cuda
    rng = np.random.default_rng(5)
    calls, ref = [], []
    for M, K, N in CAPTURED:
        announce(f"gemm captured M={M} K={K} N={N}")
        W = rng.integers(-128, 128, size=(M, K), dtype=np.int8)
        Xts = [rng.integers(-128, 128, size=(N, K), dtype=np.int8) for _ in range(3)]
        w, x = torch.from_numpy(W).cuda(), torch.from_numpy(Xts[0]).cuda()
        calls.append((w, x, M, K, N, torch.full((N, M), -7, dtype=torch.int32, device="cuda"), Xts))
        ref.append([product.to_int32(product.matmul_c(W, Xt)) for Xt in Xts])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for w, x, M, K, N, y, _ in calls:
            binding.gemm_i8(w, x, M, K, N, y)
    for i in range(3):
        for _, x, _, _, _, y, Xts in calls:
            x.copy_(torch.from_numpy(Xts[i]))
            y.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        for (w, x, M, K, N, y, _), r in zip(calls, ref):
            assert np.array_equal(y.cpu().numpy().T, r[i]), (i, M, K, N)
            y.fill_(-7)
            binding.gemm_i8(w, x, M, K, N, y)
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy().T, r[i]), (i, M, K, N)


@pytest.mark.parametrize("M,K,N,cfg", SHAPES)
def test_every_configuration(torch_cuda, M, K, N, cfg):
    torch = torch_cuda
    announce(f"gemm M={M} K={K} N={N}")
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert tuple(binding.gemm_i8_route(M, K, N).values()) == cfg
    rng = np.random.default_rng(M + K + N)
    W = rng.integers(-128, 128, size=(M, K), dtype=np.int8)
    Xt = rng.integers(-128, 128, size=(N, K), dtype=np.int8)
    y = torch.full((N + 1, M), -7, dtype=torch.int32, device="cuda")
    binding.gemm_i8(torch.from_numpy(W).cuda(), torch.from_numpy(Xt).cuda(), M, K, N, y)
    torch.cuda.synchronize()
    out = y.cpu().numpy()
    assert np.array_equal(out[:N].T, product.to_int32(product.matmul_c(W, Xt)))
    assert (out[N] == -7).all()                       # nothing past the last column
