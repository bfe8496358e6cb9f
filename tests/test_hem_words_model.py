"""CPU model of the node-based matching pass: facts about edges spread through words.

A vertex has one word: a bit per lower edge ("not taken"), and a top bit that
says one of them is taken, when every other bit is set too.  The lower edges of
a vertex with more than a word holds ("wide") have their bits in extension
words, its own word the top bit and "all dead".  A vertex walks its list of
higher edge-neighbours, heaviest first, lowest index on ties:

* a neighbour is available once the bits below the vertex's own edge are all
  set, and unavailable if its top bit is set without that;
* an available one makes the vertex's later edges dead at once;
* the vertex takes it once its own lower edges are all dead;
* a taken vertex makes all its edges dead.

Every word is read late, each reading tile on its own: of the ORs a word has
had it sees as many first ones as chance has it, in no order between words.  A
choice in a higher tile is looked up by another wave, which leaves "known" and
"available" bits for the vertex, in one word or, to show why one, in two.  The
result is compared with the oracle's sequential matching.  A vertex whose
choice is wide is visited by several lanes that hold its entries in turn: they
act on one lane's reading, or, to show why, each on its own.  This model shares
no code with the kernel or the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import problems as P


class Word:
    """A word that is only ORed into; each reader sees a prefix of the ORs."""

    def __init__(self, rng, readers):
        self.rng, self.ors, self.seen = rng, [0], [0] * readers

    def set(self, bits):
        self.ors.append(self.ors[-1] | bits)

    def read(self, reader):
        last = len(self.ors) - 1
        self.seen[reader] = int(self.rng.integers(self.seen[reader], last + 1))
        return self.ors[self.seen[reader]]


def words_model(a, T, rng, bits=31, packed=True, one_reading=True):
    """T rows a tile, `bits` lower edges a word; packed: "known" and "available" in one word; one_reading: the lanes
    that visit a vertex act on one lane's reading of its choice."""
    n, rp, ci, v = a.n, a.row_ptr, a.col, a.val
    lower = [[] for _ in range(n)]  # stored entries below the diagonal: the bits' order
    for y in range(n):
        lower[y] = [int(x) for x in ci[rp[y]:rp[y + 1]] if x < y]
    value = {(u, int(ci[e])): v[e] for u in range(n) for e in range(rp[u], rp[u + 1])}
    higher = []
    for u in range(n):
        hs = sorted((-abs(v[e]), int(ci[e])) for e in range(rp[u], rp[u + 1]) if ci[e] > u and v[e] != 0.0)
        higher.append([(j, lower[j].index(u)) for _, j in hs])
    nt = (n + T - 1) // T
    top, alld = 1 << bits, (1 << bits) - 1
    wide = [len(lower[y]) > bits for y in range(n)]
    word = [Word(rng, nt) for _ in range(n)]
    ext = [[Word(rng, nt) for _ in range((len(lower[y]) + bits - 1) // bits)] if wide[y] else [] for y in range(n)]
    for y in range(n):
        if not wide[y]:
            word[y].set(alld & ~((1 << len(lower[y])) - 1))
        for k, x in enumerate(ext[y]):
            x.set(alld & ~((1 << max(0, min(bits, len(lower[y]) - bits * k))) - 1))
    # what the other wave leaves: (entry known, entry available) of a vertex's list
    left = [(Word(rng, 1), Word(rng, 1)) for _ in range(n)]

    def dead(j, pos):
        if wide[j]:
            ext[j][pos // bits].set(1 << (pos % bits))
        else:
            word[j].set(1 << pos)

    def taken(j, pos):
        if not wide[j]:
            word[j].set(top | alld & ~(1 << pos))
            return
        steps = [(x, alld if k != pos // bits else alld & ~(1 << (pos % bits))) for k, x in enumerate(ext[j])]
        for k in rng.permutation(len(steps)):
            steps[k][0].set(steps[k][1])
        word[j].set(top)

    def full(j, pos, t, w):
        if not wide[j]:
            return w & ((1 << pos) - 1) == (1 << pos) - 1
        for k, x in enumerate(ext[j]):
            need = (1 << max(0, min(bits, pos - bits * k))) - 1
            if x.read(t) & need != need:
                return False
        return True

    for u in range(n):  # stored zeros are no edges
        for x in lower[u]:
            if value[x, u] == 0.0:
                dead(u, lower[u].index(x))
    mate = np.full(n, -1)
    done, conf, at, waits = [False] * n, [False] * n, [0] * n, [None] * n
    todo = list(range(n))
    for step in range(1000 * n + 4000):
        if not todo:
            break
        u = todo[int(rng.integers(len(todo)))]
        t, hs = u // T, higher[u]
        if rng.random() < 0.5 and waits[u] is not None:  # the other wave's turn
            j, pos = hs[waits[u]]
            w = word[j].read(t)
            av = full(j, pos, t, w)
            bit = 1 << waits[u]
            if av or w & top:
                if packed:  # one OR of both
                    left[u][0].set(bit | (bit << len(hs) if av else 0))
                else:
                    if av:
                        left[u][1].set(bit)
                    left[u][0].set(bit)
            continue
        own = word[u].read(t)
        if wide[u] and all(x.read(t) == alld for x in ext[u]):
            own |= alld
        if own & top:
            for j, pos in hs:
                dead(j, pos)
            done[u] = True
        else:
            while not conf[u]:
                if at[u] == len(hs):
                    conf[u] = True
                    break
                j, pos = hs[at[u]]
                if j // T == t or wide[j]:
                    w = word[j].read(t)
                    av = full(j, pos, t, w)
                    gone = not av and bool(w & top)
                else:
                    kn = left[u][0].read(0)
                    av = bool((kn >> len(hs) if packed else left[u][1].read(0)) >> at[u] & 1)
                    av, gone = av and bool(kn >> at[u] & 1), not av and bool(kn >> at[u] & 1)
                    if not (av or gone):
                        waits[u] = at[u]
                if wide[j] and not one_reading:
                    w = word[j].read(t)  # the other of two lanes
                    other = not full(j, pos, t, w) and bool(w & top)
                    if gone != other:  # one goes on alone, among the entries that it holds itself
                        at[u], waits[u] = min(at[u] + 2, len(hs)), None
                        continue
                if gone:
                    at[u], waits[u] = at[u] + 1, None
                    continue
                if not av:
                    break
                conf[u] = True
                for i, q in hs[at[u] + 1:]:
                    dead(i, q)
            if conf[u] and own & alld == alld:
                if at[u] < len(hs):
                    j, pos = hs[at[u]]
                    mate[u], mate[j] = j, u
                    taken(j, pos)
                    if rng.random() < 0.5:  # whoever takes a vertex may make its edges dead, before it knows itself
                        for i, q in higher[j]:
                            dead(i, q)
                done[u] = True
        if done[u]:
            todo.remove(u)
    return mate if not todo else None  # None: did not finish


def random_case(seed):
    rng = np.random.default_rng(1700 + seed)
    n = int(rng.integers(2, 60))
    a = P.random_symmetric_pattern(n, float(rng.uniform(0.03, 0.4)), seed, weights=(1, 2, 3)[: 1 + seed % 3],
                                   nonsym_values=seed % 2 == 1, explicit_zeros=0.15 * (seed % 4 == 0))
    return a, rng


@pytest.mark.parametrize("seed", range(30))
def test_words_equal_sequential_random(seed):
    a, rng = random_case(seed)
    want = oracle.hem_pass(a)
    for T in (1, 3, int(rng.integers(2, a.n + 1)), a.n):
        for bits in (31, 2, 5):
            got = words_model(a, T, rng, bits=bits)
            np.testing.assert_array_equal(got, want, err_msg=f"n={a.n} T={T} bits={bits}")


@pytest.mark.parametrize("make", [lambda: P.poisson3d(5, 4, 4), lambda: P.convdiff3d(4),
                                  lambda: P.lognormal_diffusion3d(4, 2), lambda: P.poisson2d(10, 7)])
def test_words_equal_sequential_grids_all_levels(make):
    a = make()
    rng = np.random.default_rng(7)
    for _ in range(4):  # follow the passes down the hierarchy
        want = oracle.hem_pass(a)
        for T in (7, 30, max(1, a.n // 3)):
            for bits in (31, 3):
                np.testing.assert_array_equal(words_model(a, T, rng, bits=bits), want,
                                              err_msg=f"n={a.n} T={T} bits={bits}")
        agg, nc = oracle.number(want)
        if nc == a.n or nc < 2:
            break
        rp, ci, cv = oracle.rap(a, agg, nc)
        a = P.CSR(nc, rp, ci, cv)


def test_known_and_available_belong_in_one_word():
    """In two words read in no order, an entry can look known and not available before the second arrives, and the
    vertex passes its choice by: the matching is then another one, or none."""
    wrong = 0
    for seed in range(10):
        a, rng = random_case(seed)
        wrong += not np.array_equal(words_model(a, 3, rng, packed=False), oracle.hem_pass(a))
    assert wrong > 0


def test_lanes_act_on_one_reading():
    """Where lanes read a changing word apart, some may pass a choice by alone and miss the entries of the others."""
    wrong = 0
    for seed in range(10):
        a, rng = random_case(seed)
        wrong += not np.array_equal(words_model(a, 3, rng, bits=2, one_reading=False), oracle.hem_pass(a))
    assert wrong > 0
