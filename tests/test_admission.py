"""Admission of launches whose workgroups wait for each other (CPU): whatever
their sizes and streams, the launches that can run at the same time never want
more compute units than the device has."""
import ctypes
import itertools
import random

import pytest

from paper_1107_2157_amd import sw


def admit(cus, nwg, stream):
    """Ancestors of each launch (a bit set): what it is ordered behind, by event waits or by its stream."""
    n = len(nwg)
    f = sw.lib().sw_internal_admission
    ints = ctypes.c_int * n
    f.argtypes = [ctypes.c_int, ctypes.c_int, ints, ints, ctypes.c_char_p]
    waits = ctypes.create_string_buffer(n * n)
    most = f(cus, n, ints(*nwg), ints(*stream), waits)
    assert 0 < most <= cus
    before = []
    for i in range(n):
        b = 0
        for k in range(i):
            if waits.raw[i * n + k] or stream[i] == stream[k]:
                b |= 1 << k | before[k]
        before.append(b)
    return before


def together(before):
    """All sets of launches no two of which are ordered."""
    n = len(before)
    for r in range(1, n + 1):
        for c in itertools.combinations(range(n), r):
            if all(not before[j] >> i & 1 for i, j in itertools.combinations(c, 2)):
                yield c


CASES = [([200, 56, 10, 100], [0, 1, 2, 3]),        # the third takes over from the first, which still runs
         ([256, 100, 100], [0, 1, 2]),               # the second waits for the first, the third must not pass it
         ([240, 240, 240, 240], [0, 1, 2, 3]),
         ([1] * 9, list(range(9))),
         ([2160, 16, 300, 16], [0, 1, 0, 1])]        # more workgroups than fit at once
RNG = random.Random(11)
CASES += [([RNG.choice([1, 9, 30, 64, 100, 200, 256, 700]) + RNG.randint(0, 12) for _ in range(9)],
           [RNG.randint(0, 4) for _ in range(9)]) for _ in range(60)]


@pytest.mark.parametrize("nwg,stream", CASES)
def test_concurrent_launches_fit(nwg, stream):
    before = admit(256, nwg, stream)
    for c in together(before):
        assert sum(min(nwg[i], 256) for i in c) <= 256, (c, [nwg[i] for i in c])


def test_small_launches_do_not_wait():
    """Launches that fit together, on streams of their own, are not ordered."""
    assert admit(256, [64, 64, 64, 64], [0, 1, 2, 3]) == [0, 0, 0, 0]
    # a stream takes over from its own launches before it takes over from another's
    assert admit(256, [128, 128, 128, 128], [0, 1, 0, 1]) == [0, 0, 1, 2]


def test_shares_stay_bounded():
    rng = random.Random(5)
    n = 400
    nwg = [rng.choice([1, 2, 3, 40]) for _ in range(n)]
    admit(64, nwg, [rng.randint(0, 99) for _ in range(n)])


@pytest.mark.parametrize("nwg,stream", CASES + [([12, 244], [0, 1]), ([9, 247], [0, 1])])
def test_concurrent_launches_fit_each_xcd(nwg, stream):
    """Workgroup i of a launch runs on XCD i % 8, of 32 compute units each."""
    before = admit(256, nwg, stream)
    for c in together(before):
        for x in range(8):
            assert sum((min(nwg[i], 256) - x + 7) // 8 for i in c) <= 32, (c, [nwg[i] for i in c], x)
