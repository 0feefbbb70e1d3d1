"""Scan and exponents on the GPU at the edges of their blocks and batches: zeros and denormals in a batch that also holds normal
numbers, ESC blocks shorter and longer than a batch, one and four blocks per workgroup, row groups by the dozen.  Exponents, ESC
and everything that follows are the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import ozaki as oz
from test_gpu_parity import check_against_oracle, lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


def operand(rng, rows, k, along):
    """Entries of a few bits of spread; in every block some zeros, in every third row a denormal, one row of denormals alone."""
    x = rng.uniform(1.0, 2.0, (rows, k)) * np.exp2(rng.integers(-3, 3, (rows, k)))
    x[::3, rng.integers(0, k)] = 5e-324
    x[rows // 2] = rng.integers(1, 9, k) * 2.0 ** -1060
    x[:, along] = 0.0
    return x


@pytest.mark.parametrize("m,n,k,b", [(1, 1, 1, 16), (17, 65, 16, 16), (70, 33, 100, 48), (64, 80, 129, 64), (90, 130, 2100, 1024),
                                     (300, 200, 700, 128), (65, 300, 9000, 16), (2100, 2300, 530, 64),
                                     # blocks of two and four 64s of k on either side of where a workgroup takes 64 rows
                                     (600, 40, 1600, 128), (600, 40, 1700, 128), (40, 600, 3201, 256), (40, 600, 3301, 256)])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "T")])
def test_exponents_of_mixed_blocks(lib, m, n, k, b, ta, tb):
    g, h = lib
    rng = np.random.default_rng(m + k)
    A = operand(rng, m, k, slice(0, k // 2, 5))
    B = operand(rng, n, k, slice(k // 2 + 1, k, 7)).T.copy()
    big = m * n > 10 ** 6
    for mode in ("forced",) if big else ("forced", "unguarded"):
        check_against_oracle(g, h, A, B, mode=mode, slices=4, esc_block=b, transa=ta, transb=tb, bound=False, pad=3)
    esc = oz.esc_coarse(A, B, b)
    _, _, res = run_gpu(g, h, A, B, 1.0, 0.0, None, ta, tb, mode=g.OZ_FORCED_GUARDED, slices=4, esc_block=b)
    assert res.esc == min(esc, 4096)


@pytest.mark.parametrize("where", [(0, 0), (699, 1040), (255, 64)])
def test_one_inf_or_nan_is_seen_wherever_it_is(lib, where):
    g, h = lib
    rng = np.random.default_rng(5)
    for ta, tb in (("N", "N"), ("T", "T")):
        for second in (False, True):
            A, B = rng.standard_normal((700, 1041)), rng.standard_normal((1041, 700))
            X = B.T if second else A
            X[where] = [np.inf, -np.inf, np.nan][where[0] % 3]
            _, _, res = run_gpu(g, h, A, B, 1.0, 0.0, None, ta, tb, mode=g.OZ_FORCED_GUARDED, max_bits=55)
            assert (res.fallback, res.reason, res.infnan, res.esc) == (1, 1, 1, -1)
