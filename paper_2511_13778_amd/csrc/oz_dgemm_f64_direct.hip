// Native FP64 GEMM for outputs that give the 128 x 128 tiles of dgemm_f64_kernel too few workgroups: small tiles, k split over the
// waves of a workgroup, operands straight from memory into registers.
// (paper: section "Heuristic run time Selection": what the guard falls back to.)
//
// What bounds such a product is the fullest CU's share of the tiles and everything around its K loop.  An FP64 MFMA takes 64
// cycles for 16 x 16 x 4, so operands need no LDS: a wave that owns the whole tile of the workgroup and a quarter of k reads
// (NI + NJ) fragments for NI x NJ MFMAs, 2 KB per 256 cycles at 2 x 2, 3.5 KB per 768 at 3 x 4.  So there is no barrier
// in the loop, the loads of a chunk have three MFMA steps to arrive, and the tile edges can be any multiples of 16: the form
// whose tiles come out even on the CUs is taken.  The four waves' sums meet in LDS at the end and are added in wave order
// (deterministic), so k is split four ways without a second launch and without a pass over partial products.
// Whole calls, against LDS tiles with k split over workgroups: 1000 x 1300 x 777 63 -> 44 us, 512^3 27 -> 10,
// 600 x 700 x 500 28 -> 15, 200 x 300 x 5000 45 -> 24, 64 x 64 x 7000 34 -> 11.  Large products stay on the LDS tiles (4096^3
// 1866 us, here 1918): an operand fragment is read by four waves there, here by one.
#include "oz_f64_direct.h"

namespace oz {

// Tile of 16 NI x 16 NJ; grid: tiles x zsplit, the parts of k as in dgemm_f64_kernel (f64_k_part).
template <bool AC, bool BC, int NI, int NJ>
__global__ __launch_bounds__(256, NI * NJ <= 4 ? 4 : 2) void dgemm_f64_direct_kernel(F64Call c, F64Plan p) {
    constexpr int TI = 16 * NI, TJ = 16 * NJ;
    __shared__ double sums[f64_direct_lds(NI, NJ, 4) / 8];
    f64_problem(c.batch, c.rec, c.A, c.B, c.C, p.partial);
    if (c.rec && !c.rec->res.fallback) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) write_known_record(c.known, c.batch, int(blockIdx.z));
    int ti, tj, z;
    f64_tile_of(int(blockIdx.x), p.ntm, p.ntn, p.zsplit, ti, tj, z);
    int64_t kb;
    f64_k_part(p.zsplit, z, p.kpart, c.k, kb);
    const int64_t ldp = int64_t(p.ntm) * TI;
    f64_direct_tile<AC, BC, NI, NJ, 4>(sums, c.m, c.n, c.k, kb, int64_t(ti) * TI, int64_t(tj) * TJ, c.alpha, c.A, c.a_sr, c.a_sl, c.B,
                                       c.b_sr, c.b_sl, c.beta, c.C, c.ldc,
                                       p.zsplit > 1 ? p.partial + int64_t(z) * p.ntn * TJ * ldp : nullptr, ldp);
}

void launch_dgemm_f64_direct(hipStream_t st, const F64Call& c, const F64Plan& p) {
    const dim3 grid(unsigned(p.ntm) * unsigned(p.ntn) * unsigned(p.zsplit), 1, unsigned(c.batch.count)), block(256);
#define OZ_DIRECT(AC, BC, NI, NJ)                                                                                        \
    hipLaunchKernelGGL((dgemm_f64_direct_kernel<AC, BC, NI, NJ>), grid, block, 0, st, c, p)
#define OZ_DIRECT_T(NI, NJ)                                                                                              \
    if (p.ti == 16 * NI && p.tj == 16 * NJ) {                                                                              \
        if (c.a_rows && c.b_rows) OZ_DIRECT(true, true, NI, NJ);                                                           \
        else if (c.a_rows) OZ_DIRECT(true, false, NI, NJ);                                                                 \
        else if (c.b_rows) OZ_DIRECT(false, true, NI, NJ);                                                                 \
        else OZ_DIRECT(false, false, NI, NJ);                                                                              \
        return;                                                                                                            \
    }
    OZ_DIRECT_T(1, 1)
    OZ_DIRECT_T(2, 2)
    OZ_DIRECT_T(2, 4)
    OZ_DIRECT_T(4, 2)
    OZ_DIRECT_T(3, 4)
    OZ_DIRECT_T(4, 3)
#undef OZ_DIRECT_T
#undef OZ_DIRECT
}

}  // namespace oz
