"""Workgroup -> tile maps of the large kernels (csrc/tile_order.h, compiled
here for the CPU): every tile, and every k chunk of a cut tile, must be run
exactly once for any number of groups, m-tiles, column tiles and sequences, and
the cut tiles' partial sums must fit the bound that the allocation-free entry
point's array has."""
import ctypes
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2607_28418_amd" / "csrc"

SHIM = r"""
#include "tile_order.h"
using namespace wide;
extern "C" {
int mb_share(int cols, int m_tiles) { return mblock_share(cols, m_tiles); }
void mb_place(int cols, int m_tiles, int ntpg, int halves, int shift, int id, int* out) {
  mblock_place(cols, m_tiles, ntpg, halves != 0, shift != 0, id % 8, id / 8, out[0], out[1]);
}
void kd_tail(long long M, int N, int K, int ng, unsigned long long avail, long long* out) {
  const Kd256Tail t = kd256_tail(M, N, K, ng, avail);
  out[0] = t.base, out[1] = t.split, out[2] = t.m0;
}
void kd_coords(int id, int n_tiles, int total, int* out) { kd256_coords(id, n_tiles, total, out[0], out[1]); }
void kd_chunk(int id, int m_tiles, int n_tiles, int base, int split, int* out) {
  kd256_chunk(id, m_tiles, n_tiles, base, split, out[0], out[1], out[2]);
}
void kd_steps(int K, int c, int split, int* out) { kd256_steps(K, c, split, out[0], out[1]); }
unsigned long long part_max() { return kKd256PartMaxFloats; }
int pattern_groups() { return kPatternMaxGroups; }
int remap(int id, int n) { return xcd_remap(id, n); }
void at_place(int rem, int n_seq, int n_slots, int block, int* out) {
  attn_place(rem, n_seq, n_slots, block, out[0], out[1]);
}
}
"""


@pytest.fixture(scope="module")
def maps(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_order")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", str(CSRC),
                           str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.part_max.restype = ctypes.c_uint64
    lib.kd_tail.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3 + [ctypes.c_uint64, ctypes.c_void_p]
    return lib


def call(fn, n, *args, ctype=ctypes.c_int):
    out = (ctype * n)()
    fn(*args, out)
    return tuple(out)


def test_gate_up_walk_covers_every_tile_once(maps):
    """The m-blocked walk, in a launch of its own size and in the larger one
    that serves tiles of either width (unused workgroups take padding)."""
    g = np.random.default_rng(1)
    shapes = [(1, 1, 1), (3, 2, 1), (8, 4, 4), (86, 17, 1), (112, 32, 1), (224, 2, 2), (4096, 1, 1)]
    shapes += [(int(g.integers(1, 300)) * n, int(g.integers(1, 40)), n) for n in (1, 2, 4) for _ in range(60)]
    for cols, m_tiles, ntpg in shapes:
        want = [(c, m) for c in range(cols) for m in range(m_tiles)]
        own = maps.mb_share(cols, m_tiles)
        for halves, shift, share in ((0, 1, own), (1, 1, own), (0, 0, maps.mb_share(2 * cols, m_tiles))):
            got = [call(maps.mb_place, 2, cols, m_tiles, ntpg, halves, shift, i) for i in range(8 * share)]
            assert sorted(p for p in got if p[1] < m_tiles) == want, (cols, m_tiles, ntpg, halves)
            assert all(m == m_tiles for c, m in got if not 0 <= m < m_tiles)


def test_gate_up_walk_deals_exact_eighths(maps):
    """No XCD holds more tiles than its eighth, up to what a column cannot be cut into."""
    for cols, m_tiles, ntpg in [(108, 7, 2), (86, 13, 1), (4, 33, 4), (43, 5, 1), (112, 32, 1), (54, 3, 2), (1, 40, 1)]:
        tiles = [0] * 8
        for i in range(8 * maps.mb_share(cols, m_tiles)):
            tiles[i % 8] += call(maps.mb_place, 2, cols, m_tiles, ntpg, 1, 1, i)[1] < m_tiles
        assert max(tiles) <= cols * m_tiles / 8 + 1.5, (cols, m_tiles, tiles)


def test_gate_up_walk_uses_every_shader_engine(maps):
    """An XCD's four shader engines, eight CUs each, take its workgroups in turn.
    In rows of an even number of columns, every other group of them empty, the
    real tiles must not meet in one or two of the engines."""
    for cols, m_tiles, ntpg in [(64, 9, 1), (96, 13, 1), (128, 16, 1), (48, 33, 2), (64, 13, 2)]:
        for xcd in range(8):
            got = [(i, *call(maps.mb_place, 2, cols, m_tiles, ntpg, 1, 1, 8 * i + xcd))
                   for i in range(maps.mb_share(cols, m_tiles))]
            real = np.bincount([i % 4 for i, c, m in got if m < m_tiles and c // ntpg % 2 == 0], minlength=4)
            assert real.max() <= max(8, 0.375 * real.sum()), (cols, m_tiles, real)


def test_cut_tiles_cover_every_chunk_once_and_fit(maps):
    g = np.random.default_rng(2)
    pattern = maps.pattern_groups()
    cases = [(int(np.exp(g.uniform(0, np.log(20000)))), 256 * int(g.integers(1, 40)), 64 * int(g.integers(1, 300)),
              int(g.choice([1, 4, pattern, pattern + 1, 112]))) for _ in range(400)]
    cases += [(256, 65536, 4096, 112), (1, 256, 64, 1), (300, 65792, 4096, 112)]
    cut = 0
    for M, N, K, ng in cases:
        n_tiles, m_tiles = N // 256, -(-M // 256)
        total = m_tiles * n_tiles
        avail = int(g.choice([0, M * N, 3 * M * N, 1 << 40]))
        base, split, m0 = call(maps.kd_tail, 3, M, N, K, ng, avail, ctype=ctypes.c_int64)
        rem = total - base
        whole = [call(maps.kd_coords, 2, i, n_tiles, base) for i in range(base)]
        want = [(m, n) for m in range(m_tiles) for n in range(n_tiles)]
        if split == 1:
            assert rem == 0 and m0 == M and sorted(whole) == want
            continue
        cut += 1
        rows = M - m0
        assert base % n_tiles == 0 and m0 == base // n_tiles * 256 and rows > 0
        assert m0 == 0 or ng == 1 or ng > pattern
        assert split * rows * N <= min(avail, maps.part_max()) and rem * split <= 256
        chunks = [call(maps.kd_chunk, 3, i, m_tiles, n_tiles, base, split) for i in range(rem * split)]
        assert sorted(whole + [(m, n) for c, m, n in chunks if c == 0]) == want
        assert len(set(chunks)) == len(chunks)
        assert {c for c, _, _ in chunks} == set(range(split))
        steps = [call(maps.kd_steps, 2, K, c, split) for c in range(split)]
        assert steps[0][0] == 0 and steps[-1][1] == K // 64
        assert all(b > a for a, b in steps) and all(x[1] == y[0] for x, y in zip(steps, steps[1:]))
    assert cut > 50


@pytest.mark.parametrize("M,N,K,ng,cut", [
    (2000, 2048, 1024, 8, False), (5000, 1024, 1024, 4, False), (1000, 4096, 1024, 4, False),
    (2000, 4096, 2048, 8, False), (3500, 2048, 2048, 8, False),
    (1000, 256, 512, 8, True), (200, 1024, 1024, 8, True), (2000, 2048, 2048, 16, True), (777, 4096, 4096, 8, True), (300, 4096, 14336, 112, True),
])
def test_tiles_are_cut_where_it_pays(maps, M, N, K, ng, cut):
    """Measured both ways: few steps to share do not pay for the partial sums."""
    assert (call(maps.kd_tail, 3, M, N, K, ng, 1 << 40, ctype=ctypes.c_int64)[1] > 1) == cut


def test_attention_places_cover_every_tile_once(maps):
    for n_seq, n_slots, block in [(1, 1, 1), (1, 7, 8), (9, 3, 8), (11, 4, 4), (32, 8, 4), (64, 1, 8), (5, 6, 1)]:
        for b in (block, n_seq):
            got = [call(maps.at_place, 2, i, n_seq, n_slots, b) for i in range(n_seq * n_slots)]
            assert sorted(got) == [(s, q) for s in range(n_slots) for q in range(n_seq)], (n_seq, n_slots, b)
            lengths = [s for s, q in got if q // max(b, 1) == 0]
            assert lengths == sorted(lengths, reverse=True)   # long key ranges first within a block


def test_xcd_remap_is_a_permutation(maps):
    for n in (1, 7, 8, 9, 255, 256, 513):
        ids = [maps.remap(i, n) for i in range(n)]
        assert sorted(ids) == list(range(n))
        for x in range(8):   # an XCD's workgroups take consecutive ids
            own = ids[x::8]
            assert own == list(range(own[0], own[0] + len(own))) if own else True
