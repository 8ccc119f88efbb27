"""The 32-bit payload range of the tile kernel, compiled for the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#define __host__
#define __device__
#include "us_range.h"
#include <cstdio>
#include <initializer_list>
using namespace us_range;
template <int BITS> int run() {
    long bad = 0, n = 0;
    const uint32_t top = 0xFFFFFFFCu;
    for (uint32_t pay : {0u, 16u, 4096u, 1u << 20, 0x7FFFFFF0u, 0x80000000u})
        for (uint32_t ob : {0u, 4u, 60u, 1020u, 8192u, 1u << 21, top})
            for (uint32_t len : {0u, 4u, 28u, 1024u, 4096u, 1u << 20, top})
                for (uint32_t most : {66u, 130u}) {
                    const uint32_t oe = ob + len, a0 = first_byte<BITS>(ob, pay);
                    const uint32_t got = value_bytes<BITS>(oe, a0, pay, most);
                    // Whole pieces up to the run's last value, at most `most`
                    // of them, and never past the payload.
                    const uint64_t end = (uint64_t)oe * BITS / 8;
                    uint64_t want = end > a0 ? (end - a0 + 15) / 16 * 16 : 0;
                    if (want > 16 * most) want = 16 * most;
                    if (want > pay - a0) want = pay - a0;
                    if (got != want || (uint64_t)a0 + got > pay || got % 16) ++bad;
                    ++n;
                }
    printf("%ld of %ld bad\n", bad, n);
    return bad != 0;
}
int main() { return run<4>() | run<2>(); }
'''


def test_value_bytes_saturates(tmp_path):
    src = tmp_path / "r.cpp"
    src.write_text(SRC)
    exe = tmp_path / "r"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2608_09291_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
