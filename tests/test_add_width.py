"""The width of the adding passes (csrc/nz_width.hpp) is a rule on the message and its frames: 256 threads only where that
puts more workgroups on the chip than 512 do, or leaves a thread less to take element by element.  The rule is compiled here
and held to that over sizes and frames."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12396_amd", "csrc")
CUS, BLOCK = 256, 65536                                   # compute units; elements of a 256-thread workgroup


@pytest.fixture(scope="module")
def width(tmp_path_factory):
    d = tmp_path_factory.mktemp("width")
    src, lib = d / "w.cpp", d / "libw.so"
    src.write_text('#include "nz_width.hpp"\nextern "C" uint32_t w(uint64_t n, uint32_t chunk) { return nz::add_pass_threads(n, chunk); }\n')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    f = C.CDLL(str(lib)).w
    f.argtypes, f.restype = [C.c_uint64, C.c_uint32], C.c_uint32
    return f


def _grid(n, chunk, threads):
    block, frames = threads * 256, -(-n // chunk)
    return (frames - 1) * -(-chunk // block) + -(-(n - (frames - 1) * chunk) // block)


SIZES = [1, 16384, 300007, 917504, 917505, 1 << 20, 1114109, 2500001, 1 << 22, 4259843, 11000003, 1 << 24, (1 << 24) + 49157, 18000000,
         20000000, 3 << 23, 30000000, 32554433, 33423360, 33423361, 1 << 26]


@pytest.mark.parametrize("n", SIZES)
def test_frames_that_fit_one_workgroup(width, n):
    """Both widths launch one workgroup per frame: 256 threads put nothing on idle compute units and build a frame's tables
    with half as many threads, so they have to be worth it: the frame fills them, or 512 need one more round of workgroups."""
    for chunk in (1, 1000, 2048, 4096, 8192, 10003, 16384, 24577, 32768, 49152, 57344, 65535):
        frames = -(-n // chunk)
        assert _grid(n, chunk, 256) == _grid(n, chunk, 512) == frames
        if -(-frames // (3 * CUS)) >= -(-frames // (2 * CUS)):
            assert width(n, chunk) == 512, (n, chunk)


@pytest.mark.parametrize("n", SIZES)
def test_second_workgroup_of_a_frame_nearly_empty(width, n):
    for chunk in (65537, 70000, 98303):
        assert width(n, chunk) == 512, (n, chunk)


@pytest.mark.parametrize("chunk", [262144, 524288, 1 << 20])
def test_long_ragged_end(width, chunk):
    """More 256-thread workgroups than compute units: the ragged end decides, which 512 threads take twice as fast."""
    for n in ((1 << 24) + 32773, (1 << 24) + 65533, 18000000, (3 << 23) + 49157, 32554433):
        assert _grid(n, chunk, 256) > CUS and width(n, chunk) == 512, n
    for n in (1 << 24, (1 << 24) + 70536, 20000000, 3 << 23, 30000000):       # no ragged end to speak of, or one that 512 take whole
        assert width(n, chunk) == 256, n


def test_range(width):
    for chunk in (65536, 131072, 262144, 1 << 20):
        assert [width(n, chunk) for n in (1, 917504, 917505, 1 << 20, 11000003, 1 << 24, 33423361, 1 << 26)] == \
            [512, 512, 256, 256, 256, 256, 512, 512], chunk
    # whole frames of 65536: equal grids, but a 512-thread workgroup is never filled
    assert width(1 << 22, 65536) == 256 and width(1 << 24, 98304) == 256
    # odd frames: nothing is taken by vectors, 512 threads leave a thread less once the compute units are busy
    assert width(1 << 20, 100003) == 256 and width(1 << 24, 100003) == 512
    # 512-thread workgroups in four rounds, 256-thread ones in three
    assert width(32554433, 16384) == 256 and width(1 << 24, 16384) == 512


def test_gpu_parity_shapes_reach_both_widths(width):
    from test_gpu_add_width import LARGE, SMALL
    assert [width(*s) for s in SMALL] == [256] * len(SMALL)
    assert [width(*s) for s in LARGE] == [512] * len(LARGE)
