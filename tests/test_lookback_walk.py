"""CPU test of the look-back's index arithmetic (csrc/pm_lookback.h, compiled for
the host): walks over segments of one tile to several rounds of 1024, from every
kind of position, with blocks that have handed on in part or not at all, tiles
that publish only when they are read again, and neighbouring segments' statuses
in the same words.  Every walk must add up its tiles exactly and read nothing but
its own segment's words and blocks."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2604_11008_amd", "csrc")

# One wave's walk, lane by lane; statuses are published one field at a time, each
# time a lane finds one missing.  Returns the sum, or -1 on a read out of range.
SRC = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include "pm_lookback.h"
using namespace pm;
extern "C" int64_t walk(int q0, int q, const uint16_t *known, uint16_t *status,
                        const uint32_t *handed, int *rounds)
{
    uint32_t sum = 0, excl = 0;
    int end = q;
    bool more = q > q0;
    *rounds = 0;
    auto word = [&](int w) {
        uint64_t x = 0;
        for (int f = 0; f < 4; ++f)
            x |= (uint64_t)status[4 * w + f] << (16 * f);
        return x;
    };
    while (more) {
        ++*rounds;
        int k = 63;
        bool found = false;
        uint32_t h = 0;
        for (int lane = 0; lane < 64 && !found; ++lane) {
            const int b = walk_block(q0, end, lane);
            if (b >= (q - q0) >> 6)
                return -1;
            const uint32_t v = b >= 0 ? handed[b] : (b == -1 ? 1u : 0u);
            if (v) {
                found = true;
                k = lane;
                h = v;
            }
        }
        const int from = walk_from(q0, end, k), low = walk_low(end);
        for (int lane = 0; lane < 64; ++lane)
            for (int i = 0; i < kWalkWords; ++i) {
                const int w = walk_word(end, lane, i);
                uint64_t v = 0;
                if (walk_reads(q0, w)) {
                    if (w < q0 >> 2 || w > (q - 1) >> 2)
                        return -1;
                    v = word(w);
                }
                const uint64_t mask = walk_mask(w, from, end);
                if (mask && !walk_reads(q0, w))
                    return -1;
                while (mask && walk_missing(v, mask)) {
                    for (int f = 0; f < 4; ++f)
                        if (!status[4 * w + f] && (mask >> (16 * f) & 0xffff)) {
                            status[4 * w + f] = known[4 * w + f];
                            break;
                        }
                    v = word(w);
                }
                if (mask)
                    sum += walk_sum(v, mask);
            }
        if (low > from) {
            end = low;
        } else {
            excl = found ? h - 1u : 0u;
            more = !found && from > q0;
            end = from;
        }
    }
    return (int64_t)(uint32_t)(excl + sum);
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    src, so = str(d / "walk.cpp"), str(d / "walk.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", so, src],
                   check=True)
    fn = ctypes.CDLL(so).walk
    fn.restype = ctypes.c_int64
    fn.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p,
                   ctypes.c_void_p, ctypes.c_void_p]
    return fn


@pytest.mark.parametrize("tiles", [1, 2, 5, 63, 64, 65, 129, 1023, 1024, 1025, 1100, 2500, 5200])
def test_walks_add_up(walk, tiles):
    g = np.random.default_rng(tiles)
    most = 0
    for trial in range(40):
        q0 = int(g.integers(0, 200))
        top = 4096 if trial % 3 == 0 else 3
        size = (q0 + tiles + 8) // 4 * 4 + 4
        leavers = g.integers(0, top + 1, size)
        known = (leavers + 1).astype(np.uint16)
        pre = np.concatenate([[0], np.cumsum(leavers[q0:q0 + tiles])])
        for q in {q0, q0 + tiles - 1, q0 + int(g.integers(0, tiles))}:
            j = q - q0
            handed = (pre[64:(j // 64) * 64 + 1:64] + 1).astype(np.uint32)
            p = [0.0, 0.02, 0.5, 1.0][trial % 4]
            handed[g.random(len(handed)) >= p] = 0
            status = known.copy()
            # what later tiles and the neighbours hold is of no account
            status[g.random(size) < [0.0, 0.3, 1.0][trial % 3]] = 0
            status[:q0] = g.integers(0, 4097, q0)
            rounds = ctypes.c_int()
            handed = np.append(handed, np.uint32(0))
            got = walk(q0, q, known.ctypes.data, status.ctypes.data, handed.ctypes.data,
                       ctypes.addressof(rounds))
            assert got == pre[j], (trial, q0, q, got, pre[j])
            most = max(most, rounds.value)
    assert most >= (2 if tiles > 1100 else 0), most
