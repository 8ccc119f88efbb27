"""The encoder's plain loops (US_ENCODE_PORTABLE) give the bytes of the built library."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2608_09291_amd import binding, build, synth


@pytest.fixture(scope="module")
def portable(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("enc") / "enc.so")
    subprocess.run(["g++", *build.CXX_FLAGS, "-DUS_ENCODE_PORTABLE", "-shared", os.path.join(build.CSRC, "us_encode.cpp"),
                    "-o", so, "-lpthread"], check=True)
    L = ctypes.CDLL(so)
    for name in ("us_encode", "us_encode_w2", "us_encode_reordered"):
        getattr(L, name).argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int64,
                                     ctypes.POINTER(binding.IEBME)]
    L.us_iebme_free.argtypes = [ctypes.POINTER(binding.IEBME)]
    return L


@pytest.mark.parametrize("form", ["us_encode", "us_encode_w2", "us_encode_reordered"])
@pytest.mark.parametrize("M,K,s,pad", [(16, 64, 0.5, 0), (48, 640, 0.3, 7), (64, 1024, 0.95, 64), (32, 192, 0.0, 0),
                                       (32, 192, 1.0, 1)])
def test_same_bytes(portable, form, M, K, s, pad):
    bits = 2 if form == "us_encode_w2" else 4
    W = synth.random_problem(M, K, 1, s, M + K, bits=bits)[0]
    buf = np.full((M, K + pad), 99, dtype=np.int8)          # the row padding is never read
    buf[:, :K] = W
    a, b = binding.IEBME(), binding.IEBME()
    for L, out in ((portable, a), (binding.lib(), b)):
        assert getattr(L, form)(buf.ctypes.data, M, K, K + pad, ctypes.byref(out)) == 0
    ea, eb = binding.Encoded(a), binding.Encoded(b)
    try:
        assert (ea.nnz, ea.n_payload, ea.n_lt) == (eb.nnz, eb.n_payload, eb.n_lt)
        assert np.array_equal(ea.bitmaps, eb.bitmaps) and np.array_equal(ea.offsets, eb.offsets)
        assert np.array_equal(ea.payload, eb.payload)
        assert (ea.perm is None) == (eb.perm is None)
        assert ea.perm is None or np.array_equal(ea.perm, eb.perm)
    finally:
        portable.us_iebme_free(ctypes.byref(a))
        a.bitmaps = None


@pytest.mark.parametrize("form,value", [("us_encode", 8), ("us_encode", -9), ("us_encode_w2", 2), ("us_encode_w2", -3),
                                        ("us_encode_reordered", 127)])
def test_range_errors_everywhere(portable, form, value):
    for m, k in ((0, 0), (31, 127), (17, 63), (16, 64)):
        W = np.zeros((32, 128), dtype=np.int8)
        W[m, k] = value
        for L in (portable, binding.lib()):
            out = binding.IEBME()
            assert getattr(L, form)(W.ctypes.data, 32, 128, 128, ctypes.byref(out)) == -3
            assert not out.bitmaps
