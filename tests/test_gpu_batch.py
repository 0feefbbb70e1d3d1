"""Problems that share their launches (batched calls with more than one workspace, the four products of a complex one): every
problem's C and record are those of the call for it alone, whatever route the others take."""
import numpy as np
import pytest

from paper_2511_13778_amd import workloads as wl
from test_gpu_parity import lib  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n,k,nb,lanes,opts", [
    (150, 120, 300, 7, 4, dict(mode=0, max_bits=200, heuristic=0)),                      # small calls, remainder of three
    (300, 520, 130, 5, 2, dict(mode=0, max_bits=103, heuristic=0, tile_slices=1)),       # slice counts per block, remainder of one
    (400, 300, 3000, 4, 4, dict(mode=1, max_bits=55)),                                   # 64 x 64 tiles, one and (the next but one) two to a CU
    (1000, 900, 2000, 3, 3, dict(mode=0, max_bits=103, heuristic=0)),
    (700, 800, 700, 4, 4, dict(mode=3, max_bits=55)),                                    # no guards
    (700, 600, 4000, 4, 3, dict(mode=0, max_bits=103, heuristic=0)),                     # units, k split into parts (tests/test_unit_walk_cpu.py
    (1000, 1000, 3000, 4, 4, dict(mode=0, max_bits=103, heuristic=0)),                   # holds them to it), and whole, one to a CU
    (96, 80, 112, 9, 4, dict(mode=0)), (200, 100, 5000, 6, 4, dict(mode=4)), (50, 60, 4000, 5, 2, dict(mode=4)),      # native: shared workspace, k split
    (600, 700, 10, 3, 2, dict(mode=4)), (100, 90, 0, 3, 2, dict(mode=0)),
    (1500, 1400, 600, 3, 3, dict(mode=1, max_bits=55)),                                  # too large to share: streams
])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "T")])
def test_batch_equals_single_calls(lib, m, n, k, nb, lanes, opts, ta, tb):
    g, h = lib
    opts = g.make_opts(**opts)
    rng = np.random.default_rng(m + n + k)
    pad = 3
    ra, ca = (m, k) if ta == "N" else (k, m)
    rb, cb = (k, n) if tb == "N" else (n, k)
    lda, ldb, ldc = max(1, ra) + pad, max(1, rb) + pad, m + pad
    A = rng.standard_normal((nb, max(1, ca), lda)) * np.exp2(rng.integers(-6, 7, (nb, max(1, ca), lda)) * (np.arange(nb) % 3)[:, None, None])
    B = rng.standard_normal((nb, max(1, cb), ldb))
    if k:
        A[nb - 2, 0, 0] = np.nan
    C = rng.standard_normal((nb, n, ldc))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    one = -(-h.workspace_bytes(ta, tb, m, n, k, opts) // 256) * 256
    ws = torch.full((one * lanes,), 0x5A, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    want, want_rec = [], []
    for b in range(nb):
        dC = torch.from_numpy(C[b]).cuda()
        rec = torch.zeros(g.RESULT_INT32_WORDS, dtype=torch.int32, device="cuda")
        h.dgemm(st, ta, tb, m, n, k, -1.5, dA[b].data_ptr(), lda, dB[b].data_ptr(), ldb, 0.5, dC.data_ptr(), ldc, opts, ws.data_ptr(),
                one, rec.data_ptr())
        want.append(dC.cpu().numpy())
        want_rec.append(rec.cpu().tolist())
    for _ in range(2):
        dC = torch.from_numpy(C).cuda()
        recs = torch.zeros((nb, g.RESULT_INT32_WORDS), dtype=torch.int32, device="cuda")
        ws.fill_(0x5A)
        h.dgemm_strided_batched(st, ta, tb, m, n, k, -1.5, dA.data_ptr(), lda, dA.stride(0), dB.data_ptr(), ldb, dB.stride(0), 0.5,
                                dC.data_ptr(), ldc, dC.stride(0), nb, opts, ws.data_ptr(), one * lanes, recs.data_ptr())
        got = dC.cpu().numpy()
        assert recs.cpu().tolist() == want_rec
        for b in range(nb):
            if want_rec[b][0] == 0:                # emulated: the same integers, one rounding order
                np.testing.assert_array_equal(got[b], want[b])
            else:                                  # native: tiles and parts may differ
                np.testing.assert_allclose(got[b], want[b], rtol=0, equal_nan=True, atol=2.0 ** -51 * (k + 2) * 1.5 *
                                           (np.nanmax(np.abs(A[b])) * np.abs(B[b]).max() * max(k, 1) ** 0.5 + 1))
    # operands that repeat
    if k:
        dC = torch.from_numpy(C).cuda()
        h.dgemm_strided_batched(st, ta, tb, m, n, k, -1.5, dA.data_ptr(), lda, 0, dB.data_ptr(), ldb, 0, 0.5, dC.data_ptr(), ldc,
                                dC.stride(0), nb, opts, ws.data_ptr(), one * lanes, 0)
        a = dC[1:2, :, :m] - 0.5 * torch.from_numpy(C).cuda()[1:2, :, :m]
        b = dC[:1, :, :m] - 0.5 * torch.from_numpy(C).cuda()[:1, :, :m]
        assert torch.allclose(a, b, rtol=1e-9, atol=1e-9 * b.abs().max().item())


@pytest.mark.parametrize("m,n,k,opts", [
    (150, 270, 333, dict(mode=0, max_bits=200, heuristic=0)), (500, 700, 900, dict(mode=1, max_bits=55)),
    (1000, 1000, 800, dict(mode=0, max_bits=103, heuristic=0, tile_slices=1)), (300, 200, 100, dict(mode=0)), (2000, 1900, 300, dict(mode=4)),
    (20, 30, 0, dict(mode=0)),
])
@pytest.mark.parametrize("ta,tb", [("N", "C"), ("T", "N")])
def test_complex_product_with_and_without_shared_launches(lib, m, n, k, opts, ta, tb):
    # the workspace of one product at a time, as it was before products could share launches, still serves
    g, h = lib
    opts = g.make_opts(**opts)
    rng = np.random.default_rng(k)
    cplx = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    A = cplx(*((k, m) if ta == "N" else (m, k)))
    B = cplx(*((n, k) if tb == "N" else (k, n)))
    C = cplx(n, m)
    if A.size:
        A.flat[3] = np.inf if m == 150 else A.flat[3]
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    full = h.zgemm_workspace_bytes(ta, tb, m, n, k, opts)
    up = lambda x: -(-x // 256) * 256
    least = 2 * up(8 * m * k) + 2 * up(8 * k * n) + 2 * up(8 * m * n) + up(h.workspace_bytes("N" if ta == "N" else "T", "N" if tb == "N" else "T", m, n, k, opts))
    assert least <= full and (k == 0 or least < full)
    st = torch.cuda.current_stream().cuda_stream
    out = []
    for size in (least, full):
        ws = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        dC = torch.from_numpy(C).cuda()
        recs = torch.zeros((4, g.RESULT_INT32_WORDS), dtype=torch.int32, device="cuda")
        h.zgemm(st, ta, tb, m, n, k, complex(1.25, -0.5), dA.data_ptr(), max(1, A.shape[1]), dB.data_ptr(), max(1, B.shape[1]), complex(0.5, 2.0),
                dC.data_ptr(), m, opts, ws.data_ptr(), size, recs.data_ptr())
        out.append((dC.cpu().numpy(), recs.cpu().tolist()))
    assert out[0][1] == out[1][1]
    if any(r[0] for r in out[0][1]):
        fin = np.isfinite(out[0][0])
        np.testing.assert_array_equal(fin, np.isfinite(out[1][0]))
        np.testing.assert_allclose(out[1][0][fin], out[0][0][fin], rtol=0, atol=2.0 ** -50 * (k + 2) * 20)
    else:
        np.testing.assert_array_equal(out[1][0], out[0][0])
    with pytest.raises(Exception):
        h.zgemm(st, ta, tb, m, n, k, 1.0 + 0j, dA.data_ptr(), max(1, A.shape[1]), dB.data_ptr(), max(1, B.shape[1]), 0j, dC.data_ptr(), m, opts,
                ws.data_ptr(), least - 256, 0)
