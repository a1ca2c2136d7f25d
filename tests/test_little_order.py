"""Order of the single-source little solvers' exchanges.

Their workgroups exchange vectors and partial sums through barriers that mostly
wait for neighbours only. The waits are enumerated here with vector clocks: every
read of an exchanged value must come after its write, and every later write of the
same place after all its reads. The slots of the first Gram-Schmidt passes come
from the kernel's own rule, compiled for the host.
"""
import itertools
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0706_2298_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include "little_slots.h"
using namespace dfl::little;
int main()
{
    std::printf("%d %d\n", kPairAllRead, NK);
    const int range[6] = {SA, SB, SC, SA1, NSLOT, NSLOT_PAIR};
    for (int r : range)
        std::printf("%d ", r);
    std::printf("\n");
    for (int k = 0; k < NK; ++k)
        std::printf("%d ", pair_first_slot(k));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    lines = subprocess.run([str(d / "p")], check=True, capture_output=True, text=True).stdout.split("\n")
    all_read, nk = (int(v) for v in lines[0].split())
    SA, SB, SC, SA1, nslot, nslot_pair = (int(v) for v in lines[1].split())
    first = [int(v) for v in lines[2].split()]
    assert len(first) == nk and SB - SA == SC - SB == nslot_pair - SA1
    # the passes' slots lie in ranges of their own
    assert set(first) <= {SA, SA1} and SA1 >= nslot
    return dict(all_read=all_read, nk=nk, first=first)


def neighbours(nb):
    """For every block the owners (block // 2) of its eight neighbours, and the colours."""
    coords = list(itertools.product(*(range(n) for n in nb)))
    index = {c: i for i, c in enumerate(coords)}
    own = []
    for c in coords:
        o = set()
        for mu in range(4):
            for s in (1, -1):
                d = list(c)
                d[mu] = (d[mu] + s) % nb[mu]
                o.add(index[tuple(d)] // 2)
        own.append(o)
    return own, [sum(c) % 2 for c in coords]


class Machine:
    """Workgroups in lockstep; ``clock[b][a]``: the last operation of a that b knows to be over."""

    def __init__(self, G):
        self.G, self.now = G, 0
        self.clock = [[-1] * G for _ in range(G)]
        self.writes, self.reads, self.bad = {}, {}, set()

    def write(self, res, who=None):
        for a in range(self.G) if who is None else who:
            for b, j in self.reads.get((res, a), {}).items():
                if b != a and self.clock[a][b] < j:
                    self.bad.add((res, a, b))
            self.writes[res, a] = self.now
        self.now += 1

    def read(self, res, who, of):
        for b in who:
            for a in of(b):
                if a != b and self.clock[b][a] < self.writes[res, a]:
                    self.bad.add((res, a, b))
                self.reads.setdefault((res, a), {})[b] = self.now
        self.now += 1

    def barrier(self, waits, raisers=None):
        for g in range(self.G):
            self.clock[g][g] = self.now
        at_raise = [list(c) for c in self.clock]
        self.now += 1
        for g in range(self.G):
            for q in waits(g):
                if raisers is None or q in raisers:
                    self.clock[g] = [max(x, y) for x, y in zip(self.clock[g], at_raise[q])]

    def reduce(self, slot, ns, all_read):
        everyone, owners = range(self.G), range(min(ns, self.G))
        if all_read:
            self.barrier(lambda g: everyone)
            self.read(slot, everyone, lambda b: everyone)
            return
        self.barrier(lambda g: everyone if g in owners else ())
        self.read(slot, owners, lambda b: everyone)
        self.write("pub", owners)
        self.barrier(lambda g: owners, set(owners))
        self.read("pub", everyone, lambda b: owners)


def unordered(nb, rule, first, steps, rng):
    """(slot, writer, reader) whose order no barrier of the block-pair solver gives, over a solve of random decisions."""
    own, colour = neighbours(nb)
    G = len(own) // 2
    odd = [own[2 * g + (1 - colour[2 * g])] for g in range(G)]   # owners that the odd block's neighbours have
    even = [own[2 * g + colour[2 * g]] for g in range(G)]
    m = Machine(G)
    write, read, barrier = m.write, m.read, m.barrier
    everyone = range(G)

    def reduce(slot, ns):
        m.reduce(slot, ns, G <= rule["all_read"])

    def operator():
        read("even", everyone, lambda b: odd[b])
        write("odd")
        barrier(lambda g: even[g])
        read("odd", everyone, lambda b: even[b])

    nq = rng.choice([0, 20])
    write("odd")
    barrier(lambda g: even[g])
    read("odd", everyone, lambda b: even[b])
    write("SW")
    reduce("SW", 1 + nq)
    done = 0
    while done < steps:
        nkv = rng.choice([1, 2, 5, 16, rule["nk"]])
        for k in range(nkv):
            write("even")
            if k == 0 or rng.random() < 0.8:
                barrier(lambda g: odd[g])
            else:
                write("SC")
                reduce("SC", 1)
                if rng.random() < 0.1:
                    break
            operator()
            write(first[k])
            reduce(first[k], 2 * k + 2 + nq)
            if rng.random() < 0.2:
                write("SB")
                reduce("SB", 2 * k + 2 + nq)
            done += 1
        write("even")
        barrier(lambda g: odd[g])
        operator()
        write("SW")
        reduce("SW", 1 + nq)
    write("even")
    barrier(lambda g: odd[g])
    read("even", everyone, lambda b: odd[b])
    return m.bad


SHAPES = [nb for nb in itertools.product((2, 4, 6, 8), repeat=4) if nb[0] * nb[1] * nb[2] * nb[3] <= 64]


@pytest.mark.parametrize("nb", SHAPES, ids=lambda nb: "x".join(map(str, nb)))
def test_pair_solver_order(nb, rule):
    rng = random.Random(sum(n * 10 ** i for i, n in enumerate(nb)))
    for _ in range(2):
        assert not unordered(nb, rule, rule["first"], 30, rng)


def test_one_slot_range_would_race(rule):
    """The model sees the race of first passes that all use one range of slots."""
    bad = unordered((2, 2, 2, 2), rule, [0] * rule["nk"], 60, random.Random(1))
    assert len(bad) == 8 and {r for r, _, _ in bad} == {0}


def unordered_general(nb, G, eo, fp64, steps, rng):
    """The same for the solver of any number of blocks a workgroup: pair p of blocks belongs to workgroup p % G."""
    own, colour = neighbours(nb)
    blocks = [[b for p in range(g, len(own) // 2, G) for b in (2 * p, 2 * p + 1)] for g in range(G)]
    everyone = range(G)
    few = 8 * max(len(b) for b in blocks) <= 512

    def owners_of(sel):
        return [{p % G for b in blocks[g] if sel(colour[b]) for p in own[b]} for g in range(G)]

    first = owners_of((lambda c: c == 1) if eo else (lambda c: True))
    second = owners_of(lambda c: c == 0)
    m = Machine(G)

    def sync(half):
        m.barrier(lambda g: half[g] if few else everyone)

    def operator(u):
        m.read(u, everyone, lambda b: first[b])
        if eo:
            m.write("w2 odd")
            sync(second)
            m.read("w2 odd", everyone, lambda b: second[b])

    nq = rng.choice([0, 20]) if eo else 0
    if eo:
        m.write("w1")
        sync(second)
        m.read("w1", everyone, lambda b: second[b])
    m.write("x")
    m.write("SW")
    m.reduce("SW", 1 + nq, False)
    if nq:
        m.write("x")
    done, skipped = 0, False
    while done < steps:
        nkv = rng.choice([1, 2, 5, 16])
        skipped = False
        for k in range(nkv):
            far = fp64 and k > 0 and rng.random() < 0.8
            if not far:
                m.write(("xi", k))
            if k == 0 or far:
                sync(first)
            else:
                m.write("SC")
                m.reduce("SC", 1, False)
                if rng.random() < 0.1:
                    skipped = fp64 and rng.random() < 0.5
                    break
            operator(("xi", k))
            for slot in ("SA", "SB")[:1 if rng.random() < 0.8 else 2]:
                m.write(slot)
                m.reduce(slot, 2 * k + 2 + nq, False)
            if fp64 and k + 1 < nkv:
                m.write(("xi", k + 1))
            done += 1
        m.write("x")
        if skipped:
            break
        sync(first)
        operator("x")
        m.write("SR")
        m.reduce("SR", 2 + nq, False)
        if nq:
            m.write("x")
    if eo:
        if nq or skipped:
            sync(first)
        m.read("x", everyone, lambda b: first[b])
    return m.bad


@pytest.mark.parametrize("nb,G", [((2, 2, 2, 2), 1), ((2, 2, 2, 2), 4), ((4, 2, 2, 4), 5), ((4, 4, 2, 4), 32),
                                  ((4, 4, 4, 4), 24), ((6, 4, 2, 4), 7), ((2, 2, 2, 8), 16), ((4, 4, 4, 6), 2)])
@pytest.mark.parametrize("eo", [True, False])
def test_general_solver_order(nb, G, eo):
    rng = random.Random(G)
    for fp64 in (True, False):
        for _ in range(2):
            assert not unordered_general(nb, G, eo, fp64, 30, rng)
