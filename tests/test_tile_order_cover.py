"""Workgroup -> tile maps of the 256-row kernels, restated (no GPU): every
tile, and every k chunk of a cut tile, must be run exactly once for any number
of groups, m-tiles and column tiles, and the cut tiles' partial sums must fit
the bound that the allocation-free entry point's array has."""
import re
from pathlib import Path

import numpy as np

CSRC = Path(__file__).resolve().parents[1] / "paper_2607_28418_amd" / "csrc"


def _const(name, text):
    return int(re.search(r"%s = (\d+)" % name, text).group(1))


KD = (CSRC / "gemm256.hip").read_text()
MAX_SPLIT, MIN_STEPS = _const("kKdMaxSplit", KD), _const("kKdMinSteps", KD)


def mblocked(cols, m_tiles, ntpg, halves):
    """Column tile and m-tile of every workgroup (xcd = id % 8)."""
    share = (cols + 7) // 8 * m_tiles
    for b in range(8 * share):
        xcd, l = b % 8, b // 8
        c0 = cols * xcd // 8
        n = cols * (xcd + 1) // 8 - c0
        if halves and n >= 4 * ntpg:
            h = n // 2
            if l < h * m_tiles:
                n = h
            else:
                l, c0, n = l - h * m_tiles, c0 + h, n - h
        m = min(l // n, m_tiles) if n else m_tiles
        if m < m_tiles:
            yield c0 + l % n, m


def test_gate_up_walk_covers_every_tile_once():
    g = np.random.default_rng(1)
    shapes = [(1, 1, 1), (3, 2, 1), (8, 4, 4), (86, 17, 1), (112, 32, 1), (224, 2, 2), (4096, 1, 1)]
    shapes += [(int(g.integers(1, 300)) * n, int(g.integers(1, 40)), n) for n in (1, 2, 4) for _ in range(60)]
    for cols, m_tiles, ntpg in shapes:
        for halves in (False, True):
            seen = sorted(mblocked(cols, m_tiles, ntpg, halves))
            assert seen == [(c, m) for c in range(cols) for m in range(m_tiles)], (cols, m_tiles, ntpg, halves)


def kd_tail(M, N, K, ng, avail):
    n_tiles, m_tiles = N // 256, -(-M // 256)
    total = m_tiles * n_tiles
    if total == 0 or n_tiles > 256:
        return total, 1, M
    mr = 256 // n_tiles
    mb = m_tiles // mr * mr
    rem, rows = total - mb * n_tiles, M - mb * 256
    if rem == 0 or (mb > 0 and 2 <= ng <= 8):
        return total, 1, M
    split = min(256 // rem, MAX_SPLIT, K // 64 // MIN_STEPS, avail // (rows * N))
    return (mb * n_tiles, split, mb * 256) if split >= 2 else (total, 1, M)


def xcd_remap(i, n):
    q, r = divmod(n, 8)
    xcd, local = i % 8, i // 8
    return xcd * (q + 1) + local if xcd < r else r * (q + 1) + (xcd - r) * q + local


def test_cut_tiles_cover_every_chunk_once_and_fit():
    g = np.random.default_rng(2)
    cases = [(int(np.exp(g.uniform(0, np.log(20000)))), 256 * int(g.integers(1, 40)), 64 * int(g.integers(1, 300)),
              int(g.choice([1, 4, 8, 9, 112]))) for _ in range(400)] + [(256, 65536, 4096, 112), (1, 256, 64, 1)]
    cut = 0
    for M, N, K, ng in cases:
        avail = int(g.choice([0, M * N, 3 * M * N, 1 << 40]))
        base, split, m0 = kd_tail(M, N, K, ng, avail)
        n_tiles, m_tiles = N // 256, -(-M // 256)
        total = m_tiles * n_tiles
        rem = total - base
        if split == 1:
            assert rem == 0 and m0 == M
            continue
        cut += 1
        rows = M - m0
        assert base % n_tiles == 0 and m0 == base // n_tiles * 256 and rows > 0
        assert split * rows * N <= min(avail, 256 * 256 * 256) and rem * split <= 256
        mt, seen = rem // n_tiles, set()
        for i in range(rem * split):
            j = xcd_remap(i, rem * split)
            seen.add((j // rem, base // n_tiles + j % rem % mt, j % rem // mt))
        assert seen == {(c, m, n) for c in range(split) for m in range(m_tiles - mt, m_tiles) for n in range(n_tiles)}
        steps = [(K // 64 * c // split, K // 64 * (c + 1) // split) for c in range(split)]
        assert steps[0][0] == 0 and steps[-1][1] == K // 64
        assert all(b > a for a, b in steps) and all(x[1] == y[0] for x, y in zip(steps, steps[1:]))
    assert cut > 50
