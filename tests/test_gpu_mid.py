"""GPU parity of the one-launch slice GEMM and recomposition on 64 x 64 tiles (gemm_mid_kernel): edges of its tiles and 64s of k, one
and two workgroups to a CU, one to four groups of anti-diagonals, one stage in LDS and several.  Digits, leading words and C
are the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import ozaki as oz
from paper_2511_13778_amd import workloads as wl
from test_gpu_parity import check_against_oracle, lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


# calls on 64 x 64 tiles (tests/test_unit_walk_cpu.py holds them to it): two workgroups to a CU, and one
TWO = [
    (1030, 1290, 64, 1), (961, 1030, 300, 2), (1030, 1300, 70, 3), (1100, 1000, 200, 4), (1500, 1600, 50, 5), (1030, 1300, 450, 6),
    (65, 9000, 130, 5), (9000, 65, 130, 5), (1100, 1024, 129, 7), (1281, 1030, 65, 8),
]
ONE = [
    (700, 800, 64, 1), (700, 800, 64, 5), (640, 770, 300, 3), (900, 1000, 100, 8), (700, 800, 130, 9), (700, 810, 64, 10), (705, 800, 65, 12),
    (900, 1000, 100, 13), (700, 800, 190, 16), (520, 530, 1000, 3),
    (1500, 1300, 64, 14), (1490, 1310, 130, 13), (300, 1650, 64, 16),                                   # both groups of eight
    (2100, 2200, 700, 9), (1100, 1200, 2000, 9),                                                        # a long k
]


@pytest.mark.parametrize("m,n,k,S", TWO + ONE + [(600, 700, 3000, 12)])
def test_tiles_of_64(lib, m, n, k, S):
    g, h = lib
    A, B, Cin = wl.lognormal_spread(m, k, n, 0.5, seed=5000 + S + k, with_c=True)
    beta = 0.5 if (m + S) & 1 else 0.0
    check_against_oracle(g, h, A, B, -1.5, beta, Cin if beta else None, mode="unguarded", slices=S, bound=False, pad=3,
                         transa="NT"[S & 1], transb="NT"[k & 1])


@pytest.mark.parametrize("m,n,k", [(700, 800, 100), (900, 770, 60)])
def test_tiles_of_64_with_slice_counts_per_block(lib, m, n, k):
    g, h = lib
    A, B = wl.wide_rows(m, k, n, seed=k, row_lo=m // 2, row_hi=m // 2 + 10, spread=24)
    got, gm, res = run_gpu(g, h, A, B, 1.0, 0.0, None, "N", "T", mode=g.OZ_DYNAMIC, target_bits=53, max_bits=110, heuristic=0,
                           tile_slices=1)
    tr = oz.emulated_dgemm(A, B, 1.0, 0.0, None, mode=oz.MODE_DYNAMIC, target_bits=53, max_bits=110, per_tile=True)
    assert (res.slices_used, res.slices_min, res.pair_tiles) == (tr.verdict.slices_used, tr.verdict.slices_min, tr.verdict.pair_tiles)
    np.testing.assert_array_equal(got, tr.C)


CARRIES = [1, 2, 4, 5, 6, 7, 8, 9, 10, 13, 16]


def carries_size(S):
    return (1030, 1300, 96) if S <= 10 else (1100, 1400, 96)


@pytest.mark.parametrize("S", CARRIES)
def test_carries_at_their_extremes(lib, S):
    """Entries of all-ones digits with one sign (the largest sums and carries, either way), rows of C that are zero because a row of A
    is or because the halves of k cancel, and values of one low digit."""
    g, h = lib
    m, n, k = carries_size(S)
    A, B = np.full((m, k), 2.0 - 2.0 ** -52), np.full((k, n), -(2.0 - 2.0 ** -52))
    B[:, ::3] *= -1.0
    A[5::7] = 0.0
    A[6::7, k // 2:] *= -1.0
    A[1::7, 1:] = 2.0 ** -(8 * S - 4)
    B[1:, 1::5] = -2.0 ** -(8 * S - 4)
    check_against_oracle(g, h, A, B, mode="unguarded", slices=S, bound=False)
