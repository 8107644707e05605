"""The launch order of attention items (attn_order.h, through the host-only
build): every item appears exactly once whatever the batch, no-op entries never
outnumber the items, the eight queues are balanced wherever single items allow
it, each queue runs its longest items first, and the row groups of one chunk
share a queue where bundles can be balanced."""

import ctypes
import os

import numpy as np
import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_01019_amd")


@pytest.fixture(scope="module")
def lib():
    path = os.path.join(PKG, "libhvd_host.so")
    if not os.path.exists(path):
        from paper_2606_01019_amd.build import build
        build()
    return ctypes.CDLL(path)


def order(lib, pieces, how="order"):
    a = np.ascontiguousarray(pieces, np.int32)
    out = np.zeros((2 * len(a) + 8, 4), np.int32)
    n = getattr(lib, "hvdh_attn_" + how)(len(a), a.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p), len(out))
    assert n <= 2 * len(a)
    return out[:n]


def pieces_of(seqs, heads, chunk):
    """seqs: (row groups' key counts) per sequence -> (stream, unit, chunk, keys)."""
    out, unit = [], 0
    for b, groups in enumerate(seqs):
        for g in range(heads):
            for keys in groups:
                out += [(b * heads + g, unit, c, min(keys, (c + 1) * chunk) - c * chunk) for c in range(-(-keys // chunk))]
                unit += 1
    return out


CASES = {
    "prefill": ([[64 * (i + 1) for i in range(32)]], 8, 1024),
    "prefill, 4 heads": ([[64 * (i + 1) for i in range(32)]], 4, 1024),
    "prefill, 1 head": ([[777 + 64 * i for i in range(32)]], 1, 512),
    "mixed batch": ([[int(n)] for n in np.random.default_rng(0).integers(1024, 8192, 16)], 8, 1024),
    "two row groups": ([[int(n), int(n) + 7] for n in np.random.default_rng(1).integers(64, 9000, 11)], 8, 512),
    "one long, many short": ([[16384]] + [[70]] * 31, 8, 1024),
    "few": ([[100]], 3, 32),
    "one": ([[5]], 1, 64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_order(lib, name):
    pieces = pieces_of(*CASES[name])
    out = order(lib, pieces)
    real = [tuple(int(v) for v in r) for r in out if r[1] >= 0]
    assert sorted(real) == sorted(pieces)
    if len(out) == len(pieces) and len(out) % 8 and all(out[i][3] >= out[i + 1][3] for i in range(len(out) - 1)):
        return  # plain length order: queues too uneven to interleave
    queues = [[tuple(int(v) for v in r) for r in out[x::8] if r[1] >= 0] for x in range(8)]
    loads = [sum(p[3] for p in q) for q in queues]
    assert max(loads) * 8 <= sum(loads) * 9 // 8 + 8 * max(p[3] for p in pieces)
    for q in queues:
        assert all(q[i][3] >= q[i + 1][3] for i in range(len(q) - 1))
    if name in ("prefill", "mixed batch", "two row groups"):
        home = {}
        for x, q in enumerate(queues):
            for s, _, c, _ in q:
                assert home.setdefault((s, c), x) == x


@pytest.mark.parametrize("name", list(CASES))
def test_interleave(lib, name):
    """Unit order: every item once, and the row groups that read a chunk of one
    stream on one XCD (positions 8 apart), next to each other."""
    pieces = pieces_of(*CASES[name])
    out = [tuple(int(v) for v in r) for r in order(lib, pieces, "interleave")]
    real = [p for p in out if p[1] >= 0]
    assert sorted(real) == sorted(pieces) and len(out) <= 2 * len(pieces)
    assert [p[0] for p in real] == sorted(p[0] for p in real)  # stream after stream
    groups, at = {}, {}
    for i, (s, u, c, _) in enumerate(out):
        if u >= 0:
            groups.setdefault(s, set()).add(u)
            at.setdefault((s, c), []).append((u, i))
    most = {s: 1 + max(c for r, c in at if r == s) for s in groups}
    for (s, c), members in at.items():
        members.sort()
        assert members[-1][1] - members[0][1] <= 8 * (len(groups[s]) - 1)
        if c // 8 < most[s] // 8:  # (a stream's last run may be shorter)
            assert len({i % 8 for _, i in members}) == 1
    if all(len(g) == 1 for g in groups.values()):
        assert out == pieces  # one row group each: the order is the units'



def model_order(pieces):
    """attn_order by comparison sorts."""
    pieces = sorted(pieces, key=lambda p: (p[0], p[2], p[1]))

    def deal(bundles):
        load, queues = [0] * 8, [[] for _ in range(8)]
        for b in sorted(bundles, key=lambda b: -sum(p[3] for p in b)):
            x = load.index(min(load))
            load[x] += sum(p[3] for p in b)
            queues[x] += b
        return queues, max(load) * 8 <= sum(load) + sum(load) // 8

    bundles = {}
    for p in pieces:
        bundles.setdefault((p[0], p[2]), []).append(p)
    queues, even = deal(list(bundles.values()))
    if not even:
        queues, _ = deal([[p] for p in pieces])
    by_length = lambda ps: sorted(ps, key=lambda p: (-p[3], p[0], p[2], p[1]))
    queues = [by_length(q) for q in queues]
    longest = max(len(q) for q in queues)
    if longest * 8 > 2 * len(pieces):
        return by_length(pieces)
    out = [q[i] if i < len(q) else (-1, -1, 0, 0) for i in range(longest) for q in queues]
    while out[-1][1] < 0:
        out.pop()
    return out


@pytest.mark.parametrize("seed", range(40))
def test_order_equals_the_model(lib, seed):
    r = np.random.default_rng(seed)
    chunk, heads = int(r.choice([32, 64, 256, 1024])), int(r.choice([1, 2, 3, 8]))
    seqs = []
    for _ in range(int(r.integers(1, 9))):
        first, groups = int(r.choice([r.integers(1, 90), r.integers(90, 9000)])), int(r.choice([1, 1, 2, 3, 32]))
        seqs.append([first + 64 * i for i in range(groups)])
    pieces = pieces_of(seqs, heads, chunk)
    assert [tuple(int(v) for v in p) for p in order(lib, pieces)] == model_order(pieces)


@pytest.mark.parametrize("seqs, heads, chunk, pays", [
    ([[4096]] * 8, 8, 512, False),                                       # two full rounds of equal items
    ([[600]] * 40, 8, 1024, False),                                      # equal items, none of a chunk's length
    ([[530, 562]] * 2, 4, 32, False),                                    # two 64-row drafts, 288 items of 32 keys
    ([[100]] * 16, 8, 32, False),                                        # two rounds whatever the order
    ([[1500]] * 8, 8, 512, False),                                       # less than a round
    ([[16449]] * 2, 8, 512, True),                                       # a third round for 16 items of 65 keys
    ([[int(n)] for n in np.random.default_rng(0).integers(1024, 8192, 16)], 8, 1024, True),
    ([[64 * (i + 1) for i in range(32)]], 8, 1024, True),                # a 2048-row prefill chunk
    ([[14336 + 64 * (i + 1) for i in range(32)]], 8, 2048, False),       # one deep in a prompt
])
def test_longest_first_only_where_it_shortens_the_launch(lib, seqs, heads, chunk, pays):
    a = np.ascontiguousarray(pieces_of(seqs, heads, chunk), np.int32)
    assert bool(lib.hvdh_attn_order_pays(len(a), a.ctypes.data_as(ctypes.c_void_p), 256)) == pays
