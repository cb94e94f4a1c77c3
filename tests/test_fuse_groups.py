"""How many workgroups an object gets in one launch of the one-kernel fusion over several objects, which of them begin with tiles of their
own, and where tickets are counted, on the CPU: the launch must not end in a last round that is a small part of what the machine holds,
and no count may lie on another's place."""
import ctypes
import heapq
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2511_03126_amd" / "csrc"


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    d = tmp_path_factory.mktemp("groups")
    (d / "g.cpp").write_text('#include "fuse_tile_groups.hpp"\n'
                             'extern "C" int groups(int s, int np, int n, int resident, int tiles) {\n'
                             '  return aura::fused_groups_per_object(s, np, n, resident, tiles);\n}\n'
                             'extern "C" int given(int all, int resident) {\n'
                             '  return aura::given_groups(all, resident);\n}\n'
                             'extern "C" int counter_words(int n) { return aura::counter_words(n); }\n'
                             'extern "C" int ticket_word(int xcd, int n) { return aura::launch_ticket_word(xcd, n); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "g.so"), str(d / "g.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "g.so"))
    lib.groups.given, lib.groups.counter_words, lib.groups.ticket_word = lib.given, lib.counter_words, lib.ticket_word
    return lib.groups


# (channels / 256, producers, resident workgroups) of the forms that store rows
@pytest.mark.parametrize("s,np,resident", [(1, 1, 1024), (2, 1, 512), (2, 4, 256), (3, 4, 256), (4, 4, 256)])
def test_few_objects_keep_the_larger_number(groups, s, np, resident):
    for n in range(2, 65):
        got = groups(s, np, n, resident, 6250)
        assert got in (128, 256)
        if s > 1 and n * 128 < (4 if np == 1 else 6) * resident:      # (256 channels: 128 measured faster from five objects on)
            assert got == 256
        for tiles in (1, 63, 64, 153, 1000, 1500):     # at least eight tiles per workgroup, whole rounds of the XCDs
            got = groups(s, np, n, resident, tiles)
            assert got * 8 <= tiles and got % 8 == 0 and got <= 256


def _end_of_launch(groups, n, resident, tiles, given):
    """When the last tile of a launch is done, in tiles: workgroups start in order as places become free; the first `given` of them
    begin with four tiles of their own, the others and the rest of an object's tiles find each other by asking."""
    free = [(0, i) for i in range(resident)]
    waiting = [(o, k) for o in range(n) for k in range(groups)]
    begins = [max(0, min(groups, given - o * groups)) for o in range(n)]   # workgroups of each object that begin with tiles
    left = [max(0, tiles - 4 * b) for b in begins]
    events, end = [], 0
    while waiting or events:
        while waiting and free:
            t, place = heapq.heappop(free)
            o, k = waiting.pop(0)
            own = sum(k + q * begins[o] < tiles for q in range(4)) if k < begins[o] else 0
            heapq.heappush(events, (t, place, o, own))
        t, place, o, own = heapq.heappop(events)
        if own > 0:
            heapq.heappush(events, (t + 1, place, o, own - 1))
        elif left[o] > 0:
            left[o] -= 1
            heapq.heappush(events, (t + 1, place, o, 0))
        else:
            heapq.heappush(free, (t, place))
            end = max(end, t)
    return end


# workgroups per object, objects, resident workgroups.  No later than if every tile were asked for, by more than a turn (given to all, 9
# turns were 6).
@pytest.mark.parametrize("g,n,resident", [(88, 3, 256), (56, 5, 256), (40, 7, 256), (24, 11, 256), (104, 5, 512), (88, 6, 512), (48, 6, 256),
                                          (128, 2, 256), (64, 4, 256), (64, 64, 512), (128, 64, 512), (48, 40, 512)])
@pytest.mark.parametrize("per_group", [1, 2, 3, 5, 8, 15, 16, 40])
def test_given_tiles_do_not_wait_for_workgroups_that_begin_last(groups, g, n, resident, per_group):
    tiles, given = g * per_group - 3, groups.given(g * n, resident)
    assert given in (resident, g * n) and (given == g * n or resident < g * n)
    assert _end_of_launch(g, n, resident, tiles, given) <= _end_of_launch(g, n, resident, tiles, 0) + 1


SEEN_WORD = 7   # of an object's eight words: the length of its list of seen tiles


@pytest.mark.parametrize("B", [1, 2, 7, 8, 9, 57, 63, 64, 65, 71, 72, 73, 128, 129, 130, 200, 4096])
def test_every_count_of_a_call_has_a_word_of_its_own_in_front_of_the_status_words(groups, B):
    """Launches of up to 64 objects of a call, one after the other: words that a launch counts in belong to no other launch of the call, to
    no object's list, and lie within what the workspace has for the counters."""
    size, taken = groups.counter_words(B), set()
    assert 8 * B <= size < 8 * B + 64 and size % 64 == 0   # (256 bytes each, as the workspace is divided)
    for first in range(0, B, 64):
        n = min(64, B - first)
        objects = set(range(8 * first, 8 * (first + n)))
        launch = [8 * first + groups.ticket_word(x, n) for x in range(8)]
        lists = {8 * (first + b) + SEEN_WORD for b in range(n)}
        assert len(set(launch)) == 8 and all(b - a >= 8 for a, b in zip(launch, launch[1:])) and max(launch) < size
        assert not lists & set(launch) and not taken & (objects | set(launch))
        taken |= objects | set(launch)
