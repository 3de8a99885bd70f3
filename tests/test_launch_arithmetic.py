"""Grid and index arithmetic of launches at sizes that no test runs (plain C++ headers, compiled here)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_04670_amd", "csrc")


@pytest.fixture(scope="module")
def builder(tmp_path_factory):
    d = tmp_path_factory.mktemp("builder_grid")
    (d / "g.cpp").write_text(
        '#include "builder_grid.h"\n'
        'extern "C" long long groups(int h, int w) { return evk::builder_wide_groups(h, w); }\n'
        'extern "C" int ls(int w) { return evk::builder_wide_ls(w); }\n'
        'extern "C" void share(unsigned gx, unsigned gy, unsigned nt, unsigned bx, unsigned by, unsigned t, long long* out) {\n'
        '  const evk::ClearShare s = evk::clear_share(gx, gy, nt, bx, by, t);\n  out[0] = s.first; out[1] = s.step;\n}\n')
    so = d / "g.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(d / "g.cpp")], check=True)
    lib = ctypes.CDLL(str(so))
    lib.groups.restype = ctypes.c_longlong
    return lib


@pytest.mark.parametrize("gx,gy", [(1, 1), (20, 90), (704, 2), (1, 1 << 22), (1 << 22, 1), (1 << 18, 16), (1 << 23, 1), (1, 1 << 27),
                                   ((1 << 23) - 1, 32)])
def test_builder_clears_its_own_words(builder, gx, gy):
    """The words that a thread of the increment builder clears start and advance at the global thread number and
    count, without a wrap: tall inputs make launches of 2^31 threads and more."""
    out = (ctypes.c_longlong * 2)()
    for bx in {0, gx // 2, gx - 1}:
        for by in {0, gy // 2, gy - 1}:
            for t in (0, 1, 511):
                builder.share(gx, gy, 512, bx, by, t, out)
                assert list(out) == [(by * gx + bx) * 512 + t, gx * gy * 512]


@pytest.mark.parametrize("w", [1, 6, 8, 9, 16, 17, 20, 32, 33, 64, 65, 96, 129, 346, 4096])
def test_wide_builder_launches_hold_what_tiles_held(builder, w):
    """Increment builder for more than 8 channels: on an input of few columns about as many workgroups of 64
    sites as 8 x 8 tiles, and a launch that fits (fewer than 2^32 threads along x) for every number of
    rows that a workgroup per tile fitted, up to 2^31 elements of 9 channels."""
    cols = 1 << builder.ls(w)
    for h in (1, 7, 8, 9, 1000, 4194304, min(((1 << 31) - 1) // (9 * w), (((1 << 23) - 1) // -(-w // 8)) * 8, 1 << 30)):
        groups, tiles = builder.groups(h, w), -(-h // 8) * -(-w // 8)
        assert groups == -(-h // 8) * 8 // (64 // cols) * -(-w // cols)
        assert groups <= tiles if w <= 8 else groups <= 2 * tiles
        if tiles < 1 << 23 and 9 * h * w < 1 << 31:
            assert groups * 512 < 1 << 32, (h, w, groups)
