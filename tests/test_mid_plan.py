"""The work plan of the GEMMs of 33 to 128 rows (mid_plan.h, through the host-only
build): whole column blocks, row blocks that cover the rows, partial tiles and
splits within their bounds, and column blocks chosen together with the splits
that the scratch allows."""

import ctypes
import os

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_01019_amd")
SHAPES = [(6144, 4096), (4096, 4096), (28672, 4096), (4096, 14336), (128256, 4096), (10240, 5120), (5120, 8192),
          (55296, 5120), (5120, 27648), (152064, 5120), (4160, 4160), (4096, 4128)]
MB = 1 << 20


@pytest.fixture(scope="module")
def lib():
    path = os.path.join(PKG, "libhvd_host.so")
    if not os.path.exists(path):
        from paper_2606_01019_amd.build import build
        build()
    return ctypes.CDLL(path)


def plan(lib, mtiles, N, K, part_bytes, wide=1, force=(0, 0)):
    out = (ctypes.c_int32 * 4)()
    takes = lib.hvdh_mid_plan(mtiles, N, K, wide, ctypes.c_int64(part_bytes), *force, out)
    return bool(takes), tuple(out)


@pytest.mark.parametrize("part_bytes", [0, 8 * MB, 128 * MB])
@pytest.mark.parametrize("force", [(0, 0), (1, 3), (4, 16), (8, 8)])
def test_plan_keeps_the_kernels_bounds(lib, part_bytes, force):
    for N, K in SHAPES:
        for mtiles in list(range(3, 9)) + [9, 17, 25, 64]:
            takes, (strips, splits, mb, mtb) = plan(lib, mtiles, N, K, part_bytes, force=force)
            case = (N, K, mtiles, strips, splits, mb, mtb)
            assert takes and strips in (4, 8) and N // 16 % strips == 0, case
            assert 3 <= mtb <= 8 and mb * mtb >= mtiles > (mb - 1) * mtb, case
            units = N // 16 // strips * mb
            assert 1 <= splits <= 16 and 8 * splits <= max(8, K // 32), case
            assert splits == 1 or units * splits * mtb * 16 * strips * 16 * 4 <= part_bytes, case
            if not force[0]:
                assert units * splits <= max(units, 256), case
    assert not plan(lib, 2, 4096, 4096, 128 * MB)[0] and not plan(lib, 3, 4032, 4096, 128 * MB)[0]


@pytest.mark.parametrize("mtiles", [3, 5, 6, 7, 8])
def test_small_scratch_does_not_halve_the_workgroups(lib, mtiles):
    """8 MiB of partial tiles (the static scratch): down of the 8B shape keeps 64
    columns and four splits where 128 columns would be cut to half the CUs."""
    for N, K in SHAPES:
        _, (strips, splits, mb, _) = plan(lib, mtiles, N, K, 8 * MB)
        fewest = min(4, max(1, 8 * MB // (mb * 8 * 16 * N * 4)))  # splits that fit at 128 rows
        assert N // 16 // strips * mb * splits >= min(256, N // 64 * fewest) * 3 // 4, (N, K, strips, splits)
    if mtiles == 8:
        assert plan(lib, 8, 4096, 14336, 8 * MB)[1] == (4, 4, 1, 8)
    assert plan(lib, mtiles, 4096, 14336, 128 * MB)[1][:2] == (8, 8)


def test_operands_past_32_bit_offsets_are_left_to_the_general_kernel(lib):
    """launch_gemm_mid refuses them, so the dispatch must not send them there."""
    K = 14336
    most = (2 ** 31 - 1) // (K // 32 * 1024)
    assert plan(lib, most, 4160, K, 128 * MB)[0]
    assert not plan(lib, most + 1, 4160, K, 128 * MB)[0]
