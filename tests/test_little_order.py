"""Order of the block-pair little solver's exchanges.

Its workgroups exchange vectors and partial sums through barriers that mostly
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


def unordered(nb, rule, first, steps, rng):
    """(writer, reader) pairs whose order no barrier gives, over a solve of random decisions."""
    own, colour = neighbours(nb)
    G = len(own) // 2
    odd = [own[2 * g + (1 - colour[2 * g])] for g in range(G)]   # owners that the odd block's neighbours have
    even = [own[2 * g + colour[2 * g]] for g in range(G)]
    clock = [[-1] * G for _ in range(G)]  # last operation of every workgroup known to be over
    writes, reads, bad = {}, {}, set()
    now = [0]

    def write(res, who=None):
        for a in range(G) if who is None else who:
            for b, j in reads.get((res, a), {}).items():
                if b != a and clock[a][b] < j:
                    bad.add((res, a, b))
            writes[res, a] = now[0]
        now[0] += 1

    def read(res, who, of):
        for b in who:
            for a in of(b):
                if a != b and clock[b][a] < writes[res, a]:
                    bad.add((res, a, b))
                reads.setdefault((res, a), {})[b] = now[0]
        now[0] += 1

    def barrier(waits, raisers=None):
        for g in range(G):
            clock[g][g] = now[0]
        at_raise = [list(c) for c in clock]
        now[0] += 1
        for g in range(G):
            for q in waits(g):
                if raisers is None or q in raisers:
                    clock[g] = [max(x, y) for x, y in zip(clock[g], at_raise[q])]

    everyone = range(G)

    def reduce(slot, ns):
        owners = range(min(ns, G))
        if G <= rule["all_read"]:
            barrier(lambda g: everyone)
            read(slot, everyone, lambda b: everyone)
            return
        barrier(lambda g: everyone if g in owners else ())
        read(slot, owners, lambda b: everyone)
        write("pub", owners)
        barrier(lambda g: owners, set(owners))
        read("pub", everyone, lambda b: owners)

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
    return bad


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
