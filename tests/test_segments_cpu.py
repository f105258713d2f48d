"""The segment walk and the partial slots of segments.h, compiled for the host, against the
work list's reference: every token of every (user, head) pair once, in order, and a slot of
its own for every segment of a split pair, found again by the merge's numbering."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "segments.h"
using namespace sa;
extern "C" int64_t walk(const int64_t* off, int64_t B, int64_t T, int32_t H, int64_t C, int64_t n, int64_t range, int64_t* out) {
    SegmentWalk w(off, B, T, H, C, n, range);
    Segment s;
    int64_t k = 0;
    for (; w.next(s); ++k, out += 6) {
        out[0] = s.b; out[1] = s.h; out[2] = s.t0; out[3] = s.t1; out[4] = s.split; out[5] = s.slot;
    }
    return k;
}
extern "C" int64_t slots(int64_t lo, int64_t hi, int64_t b, int64_t h, int64_t B, int64_t T, int64_t C, int64_t n, int64_t* out) {
    PairSlots p(lo, hi, b, h, B, T, C, n);
    for (int64_t i = 0; i < p.count; ++i) out[i] = p.slot(i);
    return p.count;
}
extern "C" int64_t after(const int64_t* off, int64_t b, int64_t B, int64_t T, int64_t t) { return next_user_after(off, b, B, T, t); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("segments")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#define __device__\n")
    (d / "walk.cpp").write_text(SOURCE)
    so = d / "walk.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", str(d), "-I",
                    os.path.join(ROOT, "paper_2609_08443_amd", "csrc"), str(d / "walk.cpp"), "-o", str(so)], check=True)
    L = ctypes.CDLL(str(so))
    for f in (L.walk, L.slots, L.after):
        f.restype = ctypes.c_int64
    return L


def i64(*xs):
    return [ctypes.c_int64(x) for x in xs]


LENGTHS = [[0], [5], [0, 0, 0, 40], [40, 0, 0, 0], [33, 0, 1, 64], [100] + [0] * 37 + [1, 0, 200] + [0] * 64,
           [0] * 9 + [31, 32, 33] + [0] * 16 + [64], [1] * 50, [0, 1] * 40]


@pytest.mark.parametrize("lengths", LENGTHS)
@pytest.mark.parametrize("H,C", [(1, 32), (2, 32), (3, 96), (2, 1024)])
def test_walk_covers_every_token_once(lib, lengths, H, C):
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    p, B, T = off.ctypes.data_as(ctypes.c_void_p), len(lengths), int(off[-1])
    n = (H * T + C - 1) // C
    seen, used = [], {}
    for r in range(n):
        out = np.zeros((len(lengths) * H + 1, 6), np.int64)
        k = lib.walk(p, *i64(B, T), ctypes.c_int32(H), *i64(C, n, r), out.ctypes.data_as(ctypes.c_void_p))
        for b, h, t0, t1, split, slot in out[:k].tolist():
            assert off[b] <= t0 < t1 <= off[b + 1] and r * C <= h * T + t0 and h * T + t1 <= (r + 1) * C
            assert split == (t0 > off[b] or t1 < off[b + 1])
            seen += [(h, t) for t in range(t0, t1)]
            if split:
                assert 0 <= slot < n + H * B and slot not in used.values()
                used[(b, h, t0)] = slot
    assert seen == [(h, t) for h in range(H) for t in range(T)]
    for b in range(B):
        for h in range(H):
            out = np.zeros(n + 1, np.int64)
            k = lib.slots(*i64(off[b], off[b + 1], b, h, B, T, C, n), out.ctypes.data_as(ctypes.c_void_p))
            mine = [used[key] for key in sorted(used) if key[:2] == (b, h)]
            assert k == (max(len(mine), 1) if lengths[b] else 0)
            if mine:
                assert out[:k].tolist() == mine


@pytest.mark.parametrize("lengths", LENGTHS)
def test_next_user_after(lib, lengths):
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    p, B, T = off.ctypes.data_as(ctypes.c_void_p), len(lengths), int(off[-1])
    for b in range(B + 1):
        for t in range(T + 1):
            want = next((u for u in range(b, B) if off[u + 1] > t), B)
            assert lib.after(p, *i64(b, B, T, t)) == want
