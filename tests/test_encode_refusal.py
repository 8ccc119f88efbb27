"""A matrix with a weight out of range is refused without the work of encoding it."""
import ctypes
import time

import numpy as np
import pytest

from paper_2608_09291_amd import binding, synth


@pytest.mark.parametrize("position", [(0, 0), (1023, 2047), (520, 77)])
def test_reordered_refusal_does_not_reorder(position):
    M, K = 1024, 2048
    W = synth.random_problem(M, K, 1, 0.5, 3)[0]
    bad = W.copy()
    bad[position] = 8

    def run(w):
        out, t = binding.IEBME(), time.perf_counter()
        rc = binding.lib().us_encode_reordered(w.ctypes.data, M, K, K, ctypes.byref(out))
        t = time.perf_counter() - t
        binding.lib().us_iebme_free(ctypes.byref(out))
        return rc, t

    ok = [run(W) for _ in range(3)]
    refused = [run(bad) for _ in range(3)]
    assert {r[0] for r in ok} == {0} and {r[0] for r in refused} == {-3}
    assert min(t for _, t in refused) < 0.3 * min(t for _, t in ok)
