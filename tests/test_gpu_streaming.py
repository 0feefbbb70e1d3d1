"""Scan and slicing where their kernels branch: entries at either end of what the FP64 unit cuts (far below their row's largest, of both
signs, exact and inexact), rows beyond its range, whole and ragged 64s of k in either storage order, and operands larger than
the Infinity Cache, read or written.  Exponents, slices and C are the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import ozaki as oz
from test_gpu_parity import lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


def operand(rng, rows, k, extreme):
    """Rows of magnitudes 2^-300 .. 2^300, entries down to 2^-200 below their row's largest; some whole numbers, halves and their
    negatives of the last digit, zeros; extreme: every 40th row, beyond a wave of 64 rows that has none, near either end of the exponents."""
    x = rng.uniform(-1.0, 1.0, (rows, k)) * np.exp2(rng.integers(-200, 1, (rows, k)).astype(float))
    x[:, ::7] = rng.integers(-128, 129, (rows, len(range(0, k, 7)))) * 2.0 ** -9
    x[::3, k // 2] = -2.0 ** -180
    x[1::3, k // 3] = 0.0
    x[:, 0] = rng.choice([-1.0, 1.0, 0.75, -0.5], rows)
    x = np.ldexp(x, rng.integers(-300, 300, (rows, 1)))
    if extreme:
        at = np.arange(70, rows, 40)
        x[at] = np.ldexp(rng.uniform(-1.0, 1.0, (len(at), k)), rng.choice([-1073, -1030, -1000, -950, 990, 1023], (len(at), 1)))
        x[at[::4]] = 0.0
    return x


@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 21, 26])
@pytest.mark.parametrize("rows,k,extreme", [(300, 70, True), (257, 128, False), (64, 15, True), (130, 64, True)])
def test_slices_of_either_storage_order(lib, S, rows, k, extreme):
    g, h = lib
    rng = np.random.default_rng(S * 1000 + rows)
    A, B = operand(rng, rows, k, extreme), operand(rng, rows + 9, k, extreme).T.copy()
    eA, eB = oz.row_exponents(A), oz.col_exponents(B)
    want = oz.slice_rows(A, eA, S), oz.slice_rows(np.ascontiguousarray(B.T), eB, S)
    for ta, tb in (("N", "N"), ("T", "T")):                   # either order of either operand
        for pad in (0, 3):
            _, gm, _ = run_gpu(g, h, A, B, 1.0, 0.0, None, ta, tb, pad, mode=g.OZ_FIXED_UNGUARDED, slices=S)
            for got, ref in zip(gm.slices(S), want):
                np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("ta", ["N", "T"])
def test_scan_of_an_operand_larger_than_the_cache(lib, ta):
    g, h = lib
    rng = np.random.default_rng(3)
    m, n, k = 760001, 3, 70                                   # 426 MB
    A = rng.standard_normal((m, k))
    A[::1001, 5] = 0.0
    A[7::5003, 66] = np.ldexp(1.0, -1050)
    A[11::7001] = 0.0
    B = rng.standard_normal((k, n))
    _, gm, res = run_gpu(g, h, A, B, 1.0, 0.0, None, ta, "N", mode=g.OZ_FORCED_GUARDED, slices=1)
    eA = oz.row_exponents(A)
    got, _ = gm.row_exponents()
    np.testing.assert_array_equal(got, np.where(eA > oz.NEG_INF_BELOW, eA, -12288))
    assert res.esc == min(oz.esc_coarse(A, B, 64), 4096)


# 256 x 256 blocks with one slice and with two, units (both: C at 16 bytes aligned and not), and 64 x 64 tiles, whose results are always streamed
LARGE = [(4801, 4810, 1500, 1, 0, 0.5), (5000, 4990, 2000, 2, 0, 0.0), (4802, 3904, 6000, 7, 0, -1.5), (4801, 3904, 6000, 7, 0, 0.5)]


@pytest.mark.parametrize("m,n,k,S,pad,beta", LARGE + [(4810, 4801, 1500, 2, 1, 0.0), (4801, 3902, 700, 7, 3, -1.5), (4802, 3902, 700, 7, 0, 0.0)])
def test_results_larger_than_the_cache(lib, m, n, k, S, pad, beta):
    """Rows of C at either edge and scattered over it, bit for bit."""
    g, h = lib
    rng = np.random.default_rng(S)
    A, B, Cin = rng.uniform(-1.0, 1.0, (m, k)), rng.uniform(-1.0, 1.0, (k, n)), rng.uniform(-1.0, 1.0, (m, n))
    got, _, _ = run_gpu(g, h, A, B, 0.75, beta, Cin if beta else None, "N", "N", pad, mode=g.OZ_FIXED_UNGUARDED, slices=S)
    at = np.r_[0:70, m // 2:m // 2 + 70, m - 70:m]
    tr = oz.emulated_dgemm(A[at], B, 0.75, beta, Cin[at] if beta else None, mode=oz.MODE_FIXED_UNGUARDED, slices=S)
    np.testing.assert_array_equal(got[at], tr.C)
