"""Scan of operands larger than the Infinity Cache: exponents and ESC are the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import ozaki as oz
from test_gpu_parity import lib, run_gpu  # noqa: F401  (lib: fixture)

pytestmark = pytest.mark.gpu


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
