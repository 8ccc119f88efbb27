"""Register budget and M0 use of the built tile and dense GEMM kernels (host only: compiles to gfx950 assembly)."""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2608_09291_amd import build

CSRC = build.CSRC
UNITS = ("us_spmm_tile_plain", "us_spmm_tile_perm", "us_spmm_tile_w2", "us_gemm")


@pytest.fixture(scope="module")
def texts(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    tmp = tmp_path_factory.mktemp("tile_res")

    def compile_unit(u):
        out = str(tmp / (u + ".s"))
        flags = [f for f in build.hip_flags(u + ".hip") if f != "-fPIC"]
        r = subprocess.run([build.HIPCC, *flags, "-I", CSRC, "--cuda-device-only", "-S",
                            os.path.join(CSRC, u + ".hip"), "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(out).read()

    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        return list(ex.map(compile_unit, UNITS))


def test_registers_fit_and_nothing_spills(texts):
    n = 0
    for text in texts:
        for m in re.finditer(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", text, re.S):
            g = re.search(r"us_spmm_tile_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)", m.group(1))
            d = re.search(r"us_gemm_i8_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", m.group(1))
            if not g and not d:
                continue
            lw = int(g.group(6) if g else d.group(7))
            lw = 7 if g and g.group(8) == "1" and lw == 8 else lw
            vgpr = int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", m.group(2)).group(1))
            scratch = int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", m.group(2)).group(1))
            assert vgpr <= (512 // lw) // 8 * 8, (m.group(1), vgpr, lw)
            assert scratch == 0, m.group(1)
            n += 1
    assert n == 3 * 17 + 13, n


def test_m0_is_only_the_direct_loads(texts):
    # The direct-to-LDS loads set M0 in assembly, which is only sound while
    # the compiler itself keeps nothing in it.
    n = 0
    for text in texts:
        lines = [ln.strip() for ln in text.splitlines()]
        for i, ln in enumerate(lines):
            if "m0" in ln and not ln.startswith((";", ".")):
                assert re.fullmatch(r"s_mov_b32 m0, s\d+", ln), ln
                assert lines[i + 1] == "s_nop 0" and re.match(r"buffer_load_dwordx4 v\d+, s\[\d+:\d+\], (s\d+|0) offen",
                                                              lines[i + 2]) and lines[i + 2].endswith(" lds"), lines[i:i + 3]
                n += 1
    assert n
