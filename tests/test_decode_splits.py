"""How the attention of a decode step over several sequences is dealt out to workgroups (host side: no kernel runs here)."""
import ctypes as C
import os
import random

import pytest

from paper_2601_13155_amd import binding

FLOATS = 8 * 130   # scratch of one split of one kv head at d = 128


class Splits(C.Structure):
    _fields_ = [("first", C.c_int * 17)]


def batch_splits(pairs, Hkv, scratch_splits):
    f = getattr(binding.load(), "_ZN4spts24decode_attn_batch_splitsEPKliiim")
    f.restype, f.argtypes = Splits, [C.POINTER(C.c_int64), C.c_int, C.c_int, C.c_int, C.c_size_t]
    n = len(pairs)
    first = f((C.c_int64 * n)(*pairs), n, Hkv, 128, scratch_splits * Hkv * FLOATS).first[:n + 1]
    return [b - a for a, b in zip(first, first[1:])]


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__ as g
        g.build()


@pytest.mark.parametrize("Hkv", [1, 4, 8, 64, 600])
def test_every_sequence_has_its_share_within_the_scratch(Hkv):
    rng = random.Random(Hkv)
    for _ in range(200):
        n = rng.randint(1, 16)
        pairs = [int(2 ** rng.uniform(0, 15)) for _ in range(n)]
        room = rng.choice([n, n + 3, 4096])
        ns = batch_splits(pairs, Hkv, room)
        total = max(n, min(512 // Hkv, room))
        assert all(1 <= s <= 256 for s in ns) and sum(ns) <= total
        longest = max(-(-p // s) for p, s in zip(pairs, ns))
        # what is left over would not shorten the longest split; and no other deal of `total` splits has a shorter one
        if sum(ns) < total:
            assert longest <= 64 or any(s == 256 for s in ns)
        elif longest > 64 and max(ns) < 256:
            assert sum(-(-p // (longest - 1)) for p in pairs) > total


def test_equal_sequences_have_equal_shares():
    assert batch_splits([8300] * 8, 8, 4096) == [8] * 8
    assert batch_splits([100, 100], 8, 4096) == [2, 2]
