"""GPU parity of the one-launch slice GEMM and recomposition of small calls (gemm_small_kernel) at the edges of its 32 x 32
tiles, its 64s of k and its slice counts, and of the routes that larger calls keep.  Digits, leading words and C are the
oracle's bit for bit."""
import numpy as np
import pytest

from oracle import ozaki as oz
from paper_2511_13778_amd import workloads as wl
from test_gpu_parity import check_against_oracle, lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


# calls on 32 x 32 tiles (tests/test_unit_walk_cpu.py holds them to it), each form of the kernel
TILES_32 = [
    (1, 1, 1, 1), (31, 33, 63, 2), (32, 32, 64, 8), (33, 31, 65, 9), (65, 96, 127, 16), (40, 70, 129, 17),      # one and two anti-diagonals per wave
    (100, 64, 300, 26), (64, 100, 320, 24),                         # the most slices: one 64 of k in LDS at a time
    (200, 300, 1030, 7), (129, 90, 1500, 12),                       # more 64s of k than fit in LDS
    (520, 640, 200, 6), (1000, 450, 130, 10), (300, 900, 65, 17),   # more tiles than CUs: two workgroups per CU
    (520, 530, 70, 18),                                             # and one
]


@pytest.mark.parametrize("m,n,k,S", TILES_32 + [(130, 90, 1500, 3), (700, 600, 200, 5), (1100, 1000, 130, 10)])
@pytest.mark.parametrize("beta", [0.0, 0.5])
def test_small_calls(lib, m, n, k, S, beta):
    g, h = lib
    A, B, Cin = wl.lognormal_spread(m, k, n, 0.5, seed=4000 + S + k, with_c=True)
    check_against_oracle(g, h, A, B, -1.5, beta, Cin if beta else None, mode="unguarded", slices=S, bound=False, pad=3,
                         transa="NT"[S & 1], transb="NT"[m & 1])


@pytest.mark.parametrize("m,n,k", [(300, 520, 200), (1000, 700, 100)])
def test_small_calls_with_slice_counts_per_block(lib, m, n, k):
    g, h = lib
    A, B = wl.wide_rows(m, k, n, seed=k, row_lo=m // 2, row_hi=m // 2 + 10, spread=24)
    got, gm, res = run_gpu(g, h, A, B, 1.0, 0.0, None, "N", "T", mode=g.OZ_DYNAMIC, target_bits=53, max_bits=200, heuristic=0,
                           tile_slices=1)
    tr = oz.emulated_dgemm(A, B, 1.0, 0.0, None, mode=oz.MODE_DYNAMIC, target_bits=53, max_bits=200, per_tile=True)
    assert (res.slices_used, res.slices_min, res.pair_tiles) == (tr.verdict.slices_used, tr.verdict.slices_min, tr.verdict.pair_tiles)
    np.testing.assert_array_equal(got, tr.C)


@pytest.mark.parametrize("m,n,k,S", [(2300, 2500, 200, 7), (2310, 2050, 190, 5), (1030, 1300, 900, 6), (1100, 1200, 2000, 9), (129, 300, 5000, 4)])
def test_calls_just_beyond_them(lib, m, n, k, S):
    # 64 x 64 tiles, and parts of units (129 x 300 x 5000)
    g, h = lib
    A, B = wl.lognormal_spread(m, k, n, 0.5, seed=4100 + S + k)
    check_against_oracle(g, h, A, B, 1.0, 0.0, None, mode="unguarded", slices=S, bound=False)


# calls on units, whatever the estimate of the tiles (tests/test_unit_walk_cpu.py holds them to it): whole, a split last round, parts put together by
# the recomposition, sums by atomics
UNITS = [(1500, 2200, 6000, 3), (2100, 2200, 9000, 3), (1500, 700, 9000, 3), (1500, 700, 3000, 8), (130, 65, 3000, 3), (130, 300, 9000, 12)]


@pytest.mark.parametrize("m,n,k,S", UNITS)
def test_calls_on_units(lib, m, n, k, S):
    g, h = lib
    A, B, Cin = wl.lognormal_spread(m, k, n, 0.5, seed=4200 + S + k, with_c=True)
    check_against_oracle(g, h, A, B, 1.5, 0.5, Cin, mode="unguarded", slices=S, bound=False, pad=1, transa="NT"[S & 1])
