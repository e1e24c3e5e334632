"""CPU model of the state-vector reverse mode's work split (test-side only).

The kernel numbers psi's entries by items of 64 (in tiles of the trailing
modes), hands each XCD a contiguous eighth of the chunks of eight items, shares
the sums of six to eight modes between two wavefronts, adds up 16 items at a time
and folds the sums over the lanes by halving.  The model walks the same items in
the same order on small chunks, checks that every half visits every entry once and
takes every sum once, that the fold leaves each value in exactly one lane, and
compares the result with the oracle's closed-form adjoint."""
import math

import numpy as np
import pytest

import oracle as O


def tiles(C, tmax=2048):
    sp, T = len(C), 1
    while sp > 0 and T * C[sp - 1] <= tmax:
        sp -= 1
        T *= C[sp]
    return T, math.prod(C) // T


def walk(items, grid, chunk, halves, waves=4):
    """(half, items in visiting order) of every wavefront."""
    chunks = -(-items // chunk)
    per, groups = -(-chunks // 8), waves // halves
    for block in range(grid):
        xcd = block & 7
        for wave in range(waves):
            c, mine = xcd * per + (block >> 3), []
            while c < min((xcd + 1) * per, chunks):
                mine += [c * chunk + j for j in range(wave // halves, chunk, groups) if c * chunk + j < items]
                c += grid >> 3
            yield wave % halves, mine


def split(M):
    """Per half: its rows (b terms) and the pairs (row, column) it takes."""
    halves = 2 if M > 5 else 1
    half = lambda i: 1 if halves == 2 and i >= (M + 1) // 2 else 0
    out = [[[], []] for _ in range(halves)]
    for i in range(M):
        out[half(i)][0].append(i)
        for l in range(i, M):
            row = l if half(i) != half(l) and (i + l) & 1 else i
            out[half(row)][1].append((row, i + l - row))
    return out


def fold_index(n, lane, bit=32):
    if bit == 0:
        return 0
    h = (n + 1) // 2
    i = fold_index(h, lane, bit // 2)
    j = i + (h if lane & bit else 0)
    return -1 if i < 0 or j >= n else j


def fold(v):
    """v[value][lane] by halving: the partner of a lane differs in the step's bit."""
    v = [list(x) for x in v]
    for bit, partner in ((32, lambda l: l ^ 32), (16, lambda l: l ^ 16), (8, lambda l: l ^ 15), (4, lambda l: l ^ 7),
                         (2, lambda l: l ^ 2), (1, lambda l: l ^ 1)):
        n, h = len(v), (len(v) + 1) // 2
        get = lambda j, l: v[j][l] if j < n else 0
        v = [[get(j + h if l & bit else j, l) + get(j + h if l & bit else j, partner(l)) for l in range(64)]
             for j in range(h)]
    assert len(v) == 1
    return v[0]


@pytest.mark.parametrize("n", [2, 4, 10, 18, 28, 30, 36, 42, 46, 64])
def test_fold_by_halving(n):
    rng = np.random.default_rng(n)
    v = rng.integers(-1000, 1000, size=(n, 64))
    got = fold(v.tolist())
    at = [fold_index(n, lane) for lane in range(64)]
    assert sorted(i for i in at if i >= 0) == list(range(n))
    for lane, i in enumerate(at):
        if i >= 0:
            assert got[lane] == v[i].sum()


@pytest.mark.parametrize("M", range(0, 9))
def test_halves_take_every_sum_once(M):
    parts = split(M)
    rows = sorted(i for p in parts for i in p[0])
    pairs = sorted(tuple(sorted(x)) for p in parts for x in p[1])
    assert rows == list(range(M))
    assert pairs == [(i, l) for i in range(M) for l in range(i, M)]
    values = [2 * (len(p[0]) + len(p[1]) + (h == 0)) for h, p in enumerate(parts)]
    assert max(values) <= 64   # one value to a lane after the fold


@pytest.mark.parametrize("items,grid", [(1, 8), (7, 8), (64, 8), (65, 16), (513, 24), (4097, 512), (262144, 512)])
@pytest.mark.parametrize("halves", [1, 2])
def test_items_visited_once(items, grid, halves):
    seen = [[] for _ in range(halves)]
    for half, mine in walk(items, grid, 8, halves):
        seen[half] += mine
    for s in seen:
        assert sorted(s) == list(range(items))


@pytest.mark.parametrize("C,tmax,grid,chunk", [([5], 8, 8, 2), ([6, 5], 8, 8, 2), ([4, 3, 5], 16, 8, 1),
                                               ([3, 2, 3, 2, 3, 2], 10, 16, 2), ([2, 3, 2, 2, 3, 2, 2], 6, 8, 8)])
def test_sums_against_the_adjoint(C, tmax, grid, chunk):
    rng = np.random.default_rng(sum(C))
    M = len(C)
    X = rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))
    A, b, c = 0.2 * (X + X.T), 0.3 * (rng.standard_normal(M) + 1j * rng.standard_normal(M)), 0.8 - 0.1j
    psi = O.state_vector(A, b, c, C)
    g = rng.standard_normal(C) + 1j * rng.standard_normal(C)
    T, nt = tiles(C, tmax)
    ept = -(-T // 64)
    Ab, bb, cs = np.zeros((M, M), complex), np.zeros(M, complex), 0j
    parts = split(M)
    for half, mine in walk(nt * ept, grid, chunk, len(parts)):
        for q in mine:
            tile, f0 = q // ept, q % ept * 64
            for f in range(f0, min(f0 + 64, T)):
                m = np.unravel_index(tile * T + f, C)
                step = lambda i, s: tuple(x + s * (d == i) for d, x in enumerate(m))
                p = np.conj(psi[m])
                if half == 0:
                    cs += g[m] * p
                u = {i: math.sqrt(m[i] + 1) * g[step(i, 1)] if m[i] + 1 < C[i] else 0 for i in range(M)}
                v = {l: math.sqrt(m[l]) * np.conj(psi[step(l, -1)]) if m[l] > 0 else 0 for l in range(M)}
                for i in parts[half][0]:
                    bb[i] += u[i] * p
                for row, col in parts[half][1]:
                    Ab[min(row, col), max(row, col)] += 0.5 * u[row] * v[col]
    rA, rb, rc = O.adjoint_closed_form(A, b, c, psi, g)
    got = np.concatenate([(Ab + Ab.T - np.diag(np.diag(Ab))).ravel(), bb, [cs / np.conj(c)]])
    ref = np.concatenate([np.asarray(rA).ravel(), rb, [rc]])
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
