"""The order in which the workgroups of the large-d kernels take their tiles (csrc/attn_tiles.hpp), on the CPU: every tile that is
needed once and no other, and what the order is there for."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_09397_amd", "csrc")
SOURCE = """
#include "attn_tiles.hpp"
extern "C" int count_scores(int nb, int causal) { return attn::score_tiles(nb, causal != 0); }
extern "C" void scores(int blocks, int nb, int bhs, int causal, int* out) {
    for (int i = 0; i < blocks; ++i) {
        const attn::ScoreTile t = attn::score_tile(i, nb, bhs, causal != 0);
        out[3 * i] = t.bh, out[3 * i + 1] = t.qb, out[3 * i + 2] = t.kb;
    }
}
extern "C" void products(int blocks, int count, int mbs, int nbs, int bhs, int causal, int* out) {
    for (int i = 0; i < blocks; ++i) {
        const attn::ProductTile t = attn::product_tile(i, count, mbs, nbs, bhs, causal != 0);
        out[4 * i] = t.bh, out[4 * i + 1] = t.which, out[4 * i + 2] = t.mb, out[4 * i + 3] = t.nb;
    }
}
"""
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    folder = tmp_path_factory.mktemp("tiles")
    (folder / "tiles.cpp").write_text(SOURCE)
    out = str(folder / "tiles.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(folder / "tiles.cpp"), "-o", out])
    return ctypes.CDLL(out)


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("nb", list(range(1, 18)) + [31, 64, 127, 128])
def test_score_tiles(lib, nb, causal):
    for bhs in (1, 3, 7, 8, 16):
        n = bhs * lib.count_scores(nb, causal)
        out = np.empty((n, 3), np.int32)
        lib.scores(n, nb, bhs, causal, out.ctypes.data_as(ctypes.c_void_p))
        bh, qb, kb = out.T
        assert out.min() >= 0 and bh.max() < bhs and qb.max() < nb and kb.max() < nb
        assert len(np.unique((bh * nb + qb) * nb + kb)) == n
        # nothing that the causal rule hides is launched: one such workgroup holds a CU's LDS and those behind it wait
        assert not causal or (kb <= qb).all()
        assert n == bhs * (nb * (nb + 1) // 2 if causal else nb * nb)
        # workgroups go to the 8 XCDs in turn: each has a contiguous run of the heads' tiles, as many as any other or one less
        first = [out[x::8] for x in range(min(8, n))]
        assert np.array_equal(np.concatenate(first), np.concatenate([out[x::8] for x in range(8)])) and max(map(len, first)) - min(map(len, first)) <= 1
        heads = np.concatenate(first)[:, 0]
        assert (np.diff(heads) >= 0).all()


@pytest.mark.parametrize("count", [1, 3])
@pytest.mark.parametrize("causal", [0, 1])
def test_product_tiles(lib, count, causal):
    for mbs, nbs, bhs in ((1, 1, 1), (1, 4, 3), (3, 2, 1), (7, 4, 7), (8, 2, 5), (16, 8, 4), (5, 4, 8), (9, 2, 16), (128, 4, 2)):
        n = count * mbs * nbs * bhs
        out = np.empty((n, 4), np.int32)
        lib.products(n, count, mbs, nbs, bhs, causal, out.ctypes.data_as(ctypes.c_void_p))
        bh, which, mb, nb = out.T
        assert out.min() >= 0 and bh.max() < bhs and which.max() < count and mb.max() < mbs and nb.max() < nbs
        row = (bh * count + which) * mbs + mb
        assert len(np.unique(row * nbs + nb)) == n
        if not causal:
            continue
        # rows that a tile sums over; longest first, but for the row blocks that are dealt to the XCDs together
        length = np.where((count == 3) & (which < 2), mbs - mb, mb + 1)
        assert (length[8 * nbs:] <= length[:-8 * nbs]).all()
        # the column tiles of a row block on one XCD (workgroups go to the 8 of them in turn), but for what is left at the end
        units = count * mbs * bhs
        for r in np.unique(row[: (units & ~7) * nbs]):
            at = np.nonzero(row == r)[0]
            assert len(set(at % 8)) == 1 and (np.diff(at) == 8).all()
