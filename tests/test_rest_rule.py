"""The rule that splits a fused network's batch (csrc/rest.h, plain C++),
compiled for the host: what runs layer by layer is a rest behind whole rounds,
never more than the activation buffers hold, and the limit falls with the
device's compute units (the layer kernels' time per cell rises with fewer)."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "%s"
extern "C" int64_t limit(int64_t cells, int n_cu) { return chemdnn::rest_limit(cells, n_cu); }
extern "C" int64_t rest(int64_t n, int64_t round, int64_t lim, int fp32) {
  return chemdnn::rest_cells(n, round, lim, fp32 != 0);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rest")
    (d / "rest.cpp").write_text(SRC % os.path.join(ROOT, "paper_2508_18969_amd", "csrc", "rest.h"))
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-o", str(d / "rest.so"), str(d / "rest.cpp")], check=True)
    lib = C.CDLL(str(d / "rest.so"))
    for f in (lib.limit, lib.rest):
        f.restype = C.c_int64
    lib.limit.argtypes = [C.c_int64, C.c_int]
    lib.rest.argtypes = [C.c_int64, C.c_int64, C.c_int64, C.c_int]
    return lib


@pytest.mark.parametrize("cells,fp32,tile", [(6144, 1, 32), (4096, 0, 64), (256, 0, 64)])
def test_rests(rule, cells, fp32, tile):
    assert rule.limit(cells, 256) == cells and rule.limit(cells, 304) == cells
    last = 0
    for n_cu in (1, 31, 32, 64, 128, 255, 256):
        lim = rule.limit(cells, n_cu)
        assert last <= lim <= cells * n_cu / 256 and lim % 16 == 0
        last = lim
        rnd = n_cu * tile
        for n in (1, 15, 16, 17, lim - 1, lim, lim + 1, rnd - 1, rnd, rnd + 1, rnd + lim // 2, rnd + lim // 2 + 1,
                  3 * rnd + 5, 10 * rnd):
            if n < 1:
                continue
            r = rule.rest(n, rnd, lim, fp32)
            assert 0 <= r <= lim and (n - r) % rnd == 0 or r == 0
            if n < rnd and n <= lim:
                assert r == n
            if n >= rnd:
                assert r <= (lim * 2 // 3 if fp32 else lim // 2)
