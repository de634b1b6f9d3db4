"""The single-sweep encoder's look-back entries: a workgroup first publishes its own size, then replaces it by
the running total (or the stalled mark).  Both are relaxed stores to one address, so nothing but the program
order of one lane makes the second the last.  This file takes from the kernel's source which wavefront issues
each store, runs every interleaving that leaves the device and checks, without a GPU, that an entry ends as its
final mark.  (tests/test_gpu_parity.py looks at the entries a launch leaves behind.)"""
import itertools
import os
import re

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "..", "paper_2204_08211_amd", "csrc", "k_fused.hip")
STORE = "__hip_atomic_store(&state[b]"


def publishers(team):
    """Wavefront of every store to the workgroup's own entry, in the order of the source, for teams of that size."""
    body = open(SOURCE).read()
    body = body[body.index("void k_encode_fused("):body.index("k_zero_fused(")]
    look = re.search(r"kLbWave = kTeam > 1 \? (\d+) : (\d+);", body)
    lb_wave = int(look.group(1) if team > 1 else look.group(2))
    out = []
    for at in (m.start() for m in re.finditer(re.escape(STORE), body)):
        guards = re.findall(r"if \((t == [^)\n]*|wv == kLbWave)\)", body[:at])
        g = guards[-1]
        if g == "t == 0":
            out.append(0)
        else:
            assert g in ("t == 64u * kLbWave", "wv == kLbWave"), g
            out.append(lb_wave)
    return out


def final_entries(first, second):
    """What an entry can end as: stores of one wavefront land in order, of two in any."""
    stores = [(first, "size"), (second, "final")]
    ends = set()
    for order in itertools.permutations(stores):
        if first == second and order[0][1] != "size":
            continue
        ends.add(order[-1][1])
    return ends


@pytest.mark.parametrize("team", [1, 4])
def test_an_entry_ends_as_its_final_mark(team):
    who = publishers(team)
    assert len(who) == 3          # the size, the stalled mark, the running total
    for final in who[1:]:
        assert final_entries(who[0], final) == {"final"}


def test_two_writers_would_lose_the_final_mark():
    assert final_entries(0, 1) == {"size", "final"}
