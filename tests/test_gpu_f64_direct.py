"""The FP64 GEMM on small tiles straight from memory (dgemm_f64_direct_kernel) at the edges of its tiles, of its 16s of k and of the
quarter of k each wave takes, alone and with k split over workgroups.  The oracle is the product in extended precision; an element
may be off by the forward bound of any summation order."""
import numpy as np
import pytest

from test_gpu_parity import lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [
    (1, 1, 1), (1, 17, 3), (16, 16, 4), (17, 15, 5), (33, 31, 13), (64, 48, 16), (47, 65, 17), (100, 90, 63), (81, 79, 65),
    (200, 300, 260), (512, 512, 512), (600, 700, 500), (530, 1290, 131),         # every tile form in turn
    (1000, 1300, 777), (1280, 1000, 301), (2000, 33, 90), (33, 2000, 90),
    (64, 64, 7001), (200, 300, 5000),                                           # k split over workgroups as well
])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")])
def test_small_tiles(lib, m, n, k, ta, tb):
    g, h = lib
    rng = np.random.default_rng(m + 7 * n + k)
    A, B, C = rng.standard_normal((m, k)), rng.standard_normal((k, n)), rng.standard_normal((m, n))
    got, _, res = run_gpu(g, h, A, B, -1.5, 0.5, C, ta, tb, pad=3, mode=g.OZ_NATIVE)
    assert res.fallback == 1
    L = np.longdouble
    ref = (L(-1.5) * (A.astype(L) @ B.astype(L)) + L(0.5) * C.astype(L)) if m * n * k < 2e7 else -1.5 * (A @ B) + 0.5 * C
    bound = (k + 3) * 2.0 ** -53 * (1.5 * (np.abs(A) @ np.abs(B)) + 0.5 * np.abs(C)) * (1 if m * n * k < 2e7 else 2)
    assert np.all(np.abs(got - ref) <= bound)


@pytest.mark.parametrize("m,n,k", [(705, 800, 1), (710, 801, 5), (768, 832, 15), (1900, 1700, 13)])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")])
def test_less_than_a_k_step_through_lds(lib, m, n, k, ta, tb):
    # outputs of this size and a k below 16 take, without beta, 64 x 64 tiles through LDS in the bounds-checked loop
    g, h = lib
    rng = np.random.default_rng(m + k)
    A, B = rng.standard_normal((m, k)), rng.standard_normal((k, n))
    got, _, res = run_gpu(g, h, A, B, -1.5, 0.0, None, ta, tb, pad=3, mode=g.OZ_NATIVE)
    assert res.fallback == 1
    bound = 2 * (k + 3) * 2.0 ** -53 * 1.5 * (np.abs(A) @ np.abs(B))
    assert np.all(np.abs(got + 1.5 * (A @ B)) <= bound)


@pytest.mark.parametrize("m,n,k", [(50, 70, 21), (130, 100, 66)])
def test_small_tiles_keep_inf_and_nan_in_their_row_and_column(lib, m, n, k):
    # rows past the end are read from the last row; of k past the end (a first 16 that is not full, the only such) nothing is kept.
    # Neither may reach another element.  That no load lies outside the operands is test_fp64_tiles_stay_inside_their_operands's.
    g, h = lib
    rng = np.random.default_rng(k)
    A, B = rng.standard_normal((m, k)), rng.standard_normal((k, n))
    A[m - 1, k - 1] = np.inf
    B[k - 1, n - 1] = np.nan
    for ta, tb in (("N", "N"), ("T", "T")):
        got, _, _ = run_gpu(g, h, A, B, 1.0, 0.0, None, ta, tb, mode=g.OZ_NATIVE)
        assert np.all(np.isfinite(got[:-1, :-1])) and np.all(np.isnan(got[:, -1])) and np.all(np.isinf(got[-1, :-1]))


@pytest.mark.parametrize("m,n,k,opts", [
    (1, 1, 1, dict(mode=1, max_bits=55)), (31, 33, 65, dict(mode=1, max_bits=55)), (200, 300, 261, dict(mode=0, heuristic=0)),
    (512, 512, 512, dict(mode=0, heuristic=0, max_bits=103)), (64, 1500, 130, dict(mode=1, slices=12)),       # 32 x 32 tiles
    (700, 800, 130, dict(mode=1, max_bits=55)), (705, 770, 66, dict(mode=0, heuristic=0, max_bits=103, tile_slices=1)),
    (1100, 1030, 129, dict(mode=1, max_bits=55)), (2300, 2500, 70, dict(mode=1, max_bits=55)),       # 64 x 64 (the second); launches of their own
    (700, 750, 100, dict(mode=1, max_bits=55)), (1127, 501, 18, dict(mode=1, slices=4)), (1180, 768, 236, dict(mode=1, slices=1)),     # 64 x 64, one and two to a CU
])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")])
def test_guarded_call_falls_back_in_its_last_launch(lib, m, n, k, opts, ta, tb):
    g, h = lib
    rng = np.random.default_rng(m + k)
    A, B, C = rng.standard_normal((m, k)), rng.standard_normal((k, n)), rng.standard_normal((m, n))
    A[m // 2, k // 2] = np.nan
    got, _, res = run_gpu(g, h, A, B, -1.5, 0.5, C, ta, tb, pad=3, **opts)
    assert (res.fallback, res.reason, res.infnan) == (1, 1, 1)
    rest = np.arange(m) != m // 2
    assert np.all(np.isnan(got[m // 2]))
    ref = -1.5 * (A[rest] @ B) + 0.5 * C[rest]
    bound = 2 * (k + 3) * 2.0 ** -53 * (1.5 * (np.abs(A[rest]) @ np.abs(B)) + 0.5 * np.abs(C[rest]))
    assert np.all(np.abs(got[rest] - ref) <= bound)
