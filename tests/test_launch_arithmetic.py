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
        'extern "C" void share(unsigned gx, unsigned gy, unsigned nt, unsigned bx, unsigned by, unsigned t, long long* out) {\n'
        '  const evk::ClearShare s = evk::clear_share(gx, gy, nt, bx, by, t);\n  out[0] = s.first; out[1] = s.step;\n}\n')
    so = d / "g.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(d / "g.cpp")], check=True)
    return ctypes.CDLL(str(so))


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
