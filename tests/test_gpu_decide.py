"""Small guarded calls: scan and exponents in one launch, and ESC, verdict and slicing in one, at the edges of the sizes that take them (k, rows
and ESC blocks of the scan; blocks of pairs, table rows, workgroups of the other), against the oracle bit for bit: record,
exponents, slices, products, C.  Ordinary spans, spans beyond what the matrix unit holds, zeros that leave pairs without a
candidate, zero rows and columns, Inf and NaN."""
import numpy as np
import pytest

from oracle import ozaki as oz
from paper_2511_13778_amd import workloads as wl
from test_gpu_parity import check_against_oracle, lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


def operands(kind, m, k, n, seed):
    rng = np.random.default_rng(seed)
    A, B = wl.lognormal_spread(m, k, n, 0.5, seed=seed)
    if kind == "wide":                   # spans of 40 to 90 where one row of A meets any column of B
        i = int(rng.integers(m))
        A[i] = np.ldexp(A[i], rng.integers(-30, 1, k))
        B[:, n // 2] = np.ldexp(B[:, n // 2], rng.integers(-60, 1, k))
    elif kind == "zeros":
        A[rng.random(A.shape) < 0.02] = 0.0
        B[rng.random(B.shape) < 0.02] = 0.0
    elif kind == "zero row":
        A[m - 1] = 0.0
        B[:, 0] = 0.0
    elif kind == "inf":
        B[k - 1, n - 1] = np.inf
    elif kind == "nan":
        A[m - 1, 0] = np.nan
    return A, B


SIZES = [(1, 1, 1, 0), (64, 64, 64, 0), (65, 63, 129, 0), (96, 80, 112, 16), (300, 200, 260, 0), (512, 256, 64, 0), (513, 256, 64, 0),
         (60, 70, 1024, 32), (60, 70, 1025, 64), (100, 90, 513, 16), (100, 90, 512, 16), (256, 1000, 30, 0), (1024, 1000, 70, 48),
         (1025, 1000, 70, 0), (320, 300, 330, 128),
         # the largest tables in LDS, and one block of pairs more than it holds
         (64, 832, 320, 32), (832, 63, 192, 16), (64, 896, 320, 32), (833, 64, 190, 16)]


@pytest.mark.parametrize("m,n,k,b", SIZES)
@pytest.mark.parametrize("kind", ["plain", "wide", "zeros", "zero row", "inf"])
def test_small_calls_decide_as_the_oracle(lib, m, n, k, b, kind):
    g, h = lib
    A, B = operands(kind, m, k, n, m + n + k)
    ta, tb = "NT"[m % 2], "NT"[k % 2]
    for mode, max_bits in (("dynamic", 200), ("forced", 55)) if m * n < 10 ** 5 else (("dynamic", 200),):
        check_against_oracle(g, h, A, B, mode=mode, max_bits=max_bits, esc_block=b, transa=ta, transb=tb, pad=2, bound=False)


@pytest.mark.parametrize("kind", ["plain", "wide", "zeros", "zero row", "inf", "nan"])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "T")])
def test_every_mode_of_a_small_call(lib, kind, ta, tb):
    g, h = lib
    A, B = operands(kind, 130, 200, 150, 3)
    for mode in ("dynamic", "forced", "fixed_guarded", "unguarded"):
        if mode == "unguarded" and kind in ("inf", "nan"):
            continue
        for max_bits in (55, 91, 92, 200):
            check_against_oracle(g, h, A, B, mode=mode, max_bits=max_bits, transa=ta, transb=tb, bound=False)
    for mode, max_bits in (("dynamic", 30), ("dynamic", 54)):
        check_against_oracle(g, h, A, B, mode=mode, max_bits=max_bits, transa=ta, transb=tb, bound=False)


@pytest.mark.parametrize("m,n,k", [(300, 310, 200), (64, 1100, 90), (700, 60, 100)])
@pytest.mark.parametrize("kind", ["plain", "wide", "zeros", "zero row"])
@pytest.mark.parametrize("hz", [0, 1])
def test_per_block_counts_of_a_small_call(lib, m, n, k, kind, hz):
    g, h = lib
    A, B = operands(kind, m, k, n, m)
    hs = g.Handle(0)
    model = oz.HeuristicModel(int8_ops_per_ns=10 ** 9, fp64_flops_per_ns=1000, bytes_per_ns=10 ** 6, fixed_ns=0) if hz else None
    if hz:                               # a model by which a small call pays
        hs.set_heuristic(10 ** 9, 1000, 10 ** 6, 0)
    got, gm, res = run_gpu(g, hs, A, B, mode=g.OZ_DYNAMIC, target_bits=53, max_bits=200, heuristic=hz, tile_slices=1)
    tr = oz.emulated_dgemm(A, B, mode=oz.MODE_DYNAMIC, target_bits=53, max_bits=200, per_tile=True, heuristic=model)
    v = tr.verdict
    assert (res.fallback, res.reason, res.slices_used, res.esc, res.required_bits, res.slices_min, res.pair_tiles) == \
        (v.fallback, v.reason, v.slices_used, v.esc, v.required_bits, v.slices_min, v.pair_tiles)
    if not v.fallback:
        np.testing.assert_array_equal(gm.tile_slice_counts(), tr.S_tile)
        np.testing.assert_array_equal(gm.tile_order(), np.arange(tr.S_tile.size))
        np.testing.assert_array_equal(got, tr.C)
    hs.close()
