"""The work plan of the large-batch GEMMs (tiled_plan.h, through the host-only
build): whatever the shape and the scratch it may use, the plan keeps what the
kernel relies on -- every K step of a shared tile has exactly one worker, no
run spans more than two tiles, partial slots are distinct and consecutive per
tile, and the partial tiles fit the scratch."""

import ctypes
import os

import numpy as np
import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_01019_amd")
BM, BN = [128, 128, 256, 256, 128], [128, 256, 256, 256, 256]
SHAPES = [(6144, 4096), (4096, 4096), (28672, 4096), (4096, 14336), (128256, 4096), (10240, 5120), (5120, 8192),
          (55296, 5120), (5120, 27648), (152064, 5120), (768, 256), (256, 1024), (2048, 256), (128, 32), (384, 2048)]


@pytest.fixture(scope="module")
def lib():
    path = os.path.join(PKG, "libhvd_host.so")
    if not os.path.exists(path):
        from paper_2606_01019_amd.build import build
        build()
    return ctypes.CDLL(path)


@pytest.mark.parametrize("part_bytes", [0, 8 << 20, 128 << 20])
@pytest.mark.parametrize("single", [0, 1])
def test_plan_covers_every_k_step_once(lib, single, part_bytes):
    out = (ctypes.c_int32 * 4)()
    for N, K in SHAPES:
        KT = K // 32
        for mtiles in (9, 16, 17, 24, 32, 54, 128, 130):
            lib.hvdh_tiled_plan(mtiles, N, KT, single, 256, ctypes.c_int64(part_bytes), out)
            tile, n_wg, shared, n_sk = out
            case = (N, K, mtiles, tile, n_wg, shared, n_sk)
            assert N % BN[tile] == 0, case
            T = -(-mtiles * 16 // BM[tile]) * (N // BN[tile])
            assert lib.hvdh_tiled_plan_ok(tile, n_wg, shared, n_sk, T, KT), case
            assert 1 <= n_wg and 0 <= shared <= T and n_sk <= n_wg and (shared > 0) == (n_sk > 0), case
            if not shared:
                continue
            assert shared < n_sk <= shared * KT, case
            n_slots = n_sk + (shared if n_sk % shared else 0)
            assert n_slots * BM[tile] * BN[tile] * 4 <= part_bytes, case
            done = np.zeros(shared * KT, dtype=np.int32)
            workers, slots = set(), {}
            for w in range(n_sk):
                lib.hvdh_tiled_run(shared, KT, n_sk, w, out)
                lo, hi, worker, holder = out
                assert lo < hi < lo + KT and holder == w, case  # a part, never a whole tile
                workers.add(worker)
                done[lo:hi] += 1
                tiles = range(lo // KT, (hi - 1) // KT + 1)
                assert len(tiles) <= 2, case
                for t in tiles:
                    slot = lib.hvdh_tiled_slot(shared, KT, n_sk, w, t)
                    assert 0 <= slot < n_slots and slot not in slots, case
                    slots[slot] = t
                if n_sk % shared == 0:  # an even split: one tile per worker, cut alike
                    i = w % (n_sk // shared)
                    assert len(tiles) == 1 and lo % KT == i * KT // (n_sk // shared), case
            assert (done == 1).all() and workers == set(range(n_sk)), case
            for t in range(shared):  # consecutive per tile, as the finishing kernel reads them
                mine = sorted(s for s, u in slots.items() if u == t)
                assert mine == list(range(mine[0], mine[0] + len(mine))), case
            assert len(slots) == sum((out_hi(lib, shared, KT, n_sk, w) for w in range(n_sk))), case


def out_hi(lib, shared, KT, n_sk, w):
    """Tiles that worker w's run touches."""
    out = (ctypes.c_int32 * 4)()
    lib.hvdh_tiled_run(shared, KT, n_sk, w, out)
    return (out[1] - 1) // KT - out[0] // KT + 1


@pytest.mark.parametrize("plan, T, KT, ok", [
    ((4, 192, 96, 192), 96, 128, True),
    ((4, 256, 128, 256), 896, 128, True),
    ((4, 256, 140, 256), 140, 256, True),
    ((4, 300, 0, 0), 300, 16, True),
    ((4, 40, 40, 40), 40, 64, False),      # one worker per shared tile
    ((4, 256, 255, 256), 511, 128, False),  # 127.5 steps per worker: the first 128 runs are whole tiles
    ((4, 256, 254, 256), 510, 128, True),   # 127 steps each
    ((4, 8, 1, 8), 1, 7, False),            # more workers than steps
    ((4, 8, 2, 16), 2, 64, False),          # more workers than workgroups
    ((4, 8, 3, 8), 2, 64, False),           # more shared tiles than tiles
    ((4, 8, 2, 0), 2, 64, False),
])
def test_plans_the_kernels_cannot_run_are_refused(lib, plan, T, KT, ok):
    """A run that covers a whole tile would be finished twice, once from a partial
    slot that nothing wrote: the launcher refuses such plans."""
    assert bool(lib.hvdh_tiled_plan_ok(*plan, T, KT)) == ok
    if ok and plan[2]:
        out = (ctypes.c_int32 * 4)()
        for w in range(plan[3]):
            lib.hvdh_tiled_run(plan[2], KT, plan[3], w, out)
            assert out[1] - out[0] < KT


@pytest.mark.parametrize("rows", [144, 192, 256])
@pytest.mark.parametrize("N, K", [(4096, 4096), (4096, 14336), (5120, 27648), (4096, 4128)])
def test_small_scratch_still_splits_narrow_gemms(lib, rows, N, K):
    """8 MiB of partial tiles (the static scratch) hold a two-way split of any
    256 x 4096 product: one slot per worker, whether or not the split divides K."""
    out = (ctypes.c_int32 * 4)()
    lib.hvdh_tiled_plan(rows // 16, N, K // 32, 0, 256, ctypes.c_int64(8 << 20), out)
    tile, n_wg, shared, n_sk = out
    T = -(-rows // BM[tile]) * (N // BN[tile])
    if T * 2 * BM[tile] * BN[tile] * 4 <= 8 << 20:
        assert shared == T and n_sk >= 2 * T, (tile, n_wg, shared, n_sk)
    else:
        assert n_wg >= 40, (tile, n_wg, shared, n_sk)
