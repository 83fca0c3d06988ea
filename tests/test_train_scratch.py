"""The allocation-free training step takes every batch whose layer-by-layer
scratch fits the static array: the tile path's scratch (read off the workspace
sizes, no GPU needed) fits it too, for every species count and chunk, at the
largest batch and at the most chunks."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIDDEN = (400, 200, 100)


@pytest.fixture(scope="module")
def L():
    from paper_2508_18969_amd import binding
    if not os.path.exists(binding.LIB):
        pytest.skip("library not built")
    return binding


def _layered_bytes(S, cap, chunk):
    """Scratch of the layer-by-layer training kernels (bytes)."""
    w = (S + 2,) + HIDDEN + (S,)
    ld = min(chunk, cap) if chunk else cap
    f = ld * (w[0] + sum(HIDDEN) + S + 2 * max(w[1:])) + 32 * max(a * b for a, b in zip(w[:-1], w[1:]))
    return 4 * (f + 256 * max(w[1:]) + 1024) + 8 * (-(-cap // ld)) + 2560


def _tile_bytes(L, S, cap, chunk):
    def ws(max_batch):
        d, keep = L.make_desc((S + 2,) + HIDDEN + (S,), "fp32", np.zeros(S + 2), np.ones(S + 2),
                              max_batch=max_batch, recompute_chunk=chunk)
        return L.workspace_bytes(d)
    r = [(a + 15) // 16 for a in HIDDEN]               # row-blocks; k-steps of 32
    q = [(a + 31) // 32 for a in HIDDEN]
    pack = r[0] + r[1] * q[0] + r[2] * q[1] + 2 * q[2] + r[2] + r[1] * q[2] + r[0] * q[1] + 2 * q[0]
    return ws(cap) - ws(0) + pack * 3072


@pytest.mark.parametrize("S", range(1, 31))
def test_the_static_scratch_takes_what_the_layered_path_takes(L, S):
    header = open(os.path.join(ROOT, "include", "chem_dnn.h")).read()
    m, e = re.search(r"CHEM_DNN_NOALLOC_SCRATCH_BYTES \((\d+)u << (\d+)\)", header).groups()
    limit = int(m) << int(e)
    largest = max(c for c in range(16, 1 << 14, 16) if _layered_bytes(S, c, 0) <= limit)
    assert 9000 < largest < 9400
    for cap in range(9000 // 16 * 16, largest + 1, 16):
        assert _tile_bytes(L, S, cap, 0) <= limit, cap
    for chunk in list(range(16, 1024, 16)) + list(range(1024, largest + 1, 256)) + [largest]:
        cap = chunk * ((limit - _layered_bytes(S, chunk, 0)) // 8 + 1)     # the most chunks
        assert _layered_bytes(S, cap, chunk) <= limit
        assert _tile_bytes(L, S, cap, chunk) <= limit, chunk
