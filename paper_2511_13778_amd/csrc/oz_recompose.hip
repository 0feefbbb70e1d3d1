// FP64 recomposition of the aggregated anti-diagonal sums and the alpha/beta update.
// (paper: section "FP64 Emulation on Low-Precision Units": slice products are recombined;
//  section "Pre-processing and Safety Checks", second half: partial results are aggregated
//  before the terminal conversion to FP64, so an Inf can only appear in that last step.)
//
// The slice GEMM leaves, per k-block, the exact integer Z = sum_d P_d 256^(S-1-d) as a leading int32
// word T and balanced base-256 digits L_d in [-128,127]:  Z = T 256^(S-1) + sum_{d>=1} L_d 256^(S-1-d).
//
//   AB_ij = 2^(eA_i + eB_j - 10) * sum_kb ( T + sum_{d>=1} 256^-d L_d )
//   C_ij  = alpha * AB_ij + beta * C_ij           (C not read when beta == 0)
//
// Order (fixed, so results are reproducible): k-blocks ascending; inside a k-block from the least
// significant digit, R <- L_d + R * 2^-8, then R <- T + R * 2^-8 (up to seven slices every step but
// this last one is exact: the k-block's value is the exact integer rounded once); block results
// added unscaled; the power of two applied last with ldexp; alpha*AB and beta*C rounded separately,
// then added.
// HBM-bound: (4 + S - 1) * nkb bytes read and 8 (+8 when beta != 0) bytes moved per element of C.
#include <type_traits>

#include "oz_internal.h"

namespace oz {

constexpr int kRecI = 4;   // four consecutive i per thread: one 16-byte load of T per j, of L per digit
constexpr int kRecJ = 4;   // four consecutive j per thread: the four bytes of an L dword
constexpr int kVecC = 1, kStreamC = 2;       // c_flags

// KIND: where the sums of a k-block come from.  kNone: the planes T / L, complete.  kParts: the planes hold part 0 of a
// k split and the raw buffer the others, each with digits of its own; they are added digit by digit with the slice
// GEMM's carry chain.  kAtomic: the raw buffer holds the unaggregated sums of every anti-diagonal, which go through
// the same chain.  In both, the digits are those of the whole integer then; they are written back to T / L, and used
// at once.  (A kernel of its own in between, with a thread walking its digits one load at a time, took 30-44 us of
// a 1024^3 call's 180.)
template <KSplit KIND>
__global__ __launch_bounds__(256) void recompose_kernel(std::conditional_t<KIND == KSplit::kNone, const int32_t, int32_t>* __restrict__ T,
                                                        std::conditional_t<KIND == KSplit::kNone, const int8_t, int8_t>* __restrict__ L,
                                                        const int32_t* __restrict__ raw, SplitPlan split,
                                                        const int32_t* __restrict__ eA,
                                                        const int32_t* __restrict__ eB, int64_t m, int64_t n,
                                                        int64_t mp, int64_t np, int64_t kp, int s_cap,
                                                        double alpha, double beta,
                                                        double* __restrict__ C, int64_t ldc,
                                                        const Record* rec,
                                                        const int32_t* __restrict__ tile_S, int64_t j4_first,
                                                        int c_flags, Batch bt) {
    {
        const int64_t ws = bt.ws_at(blockIdx.z);
        T = at_bytes(T, ws); L = at_bytes(L, ws);
        raw = at_bytes(raw, ws);
        eA = at_bytes(eA, ws); eB = at_bytes(eB, ws);
        rec = at_bytes(rec, ws);
        if (tile_S) tile_S = at_bytes(tile_S, ws);
        C += int64_t(blockIdx.z) * bt.c;
    }
    if (rec->res.fallback) return;
    const int S_all = rec->res.slices_used;
    const int64_t kblk = k_block_length(S_all);             // k-blocks of the call's largest count
    const int nkb = int((kp + kblk - 1) / kblk);
    const int64_t j4 = j4_first + blockIdx.y;
    const int64_t j0 = j4 * kRecJ;
    const int64_t i0 = (int64_t(blockIdx.x) * 256 + threadIdx.x) * kRecI;
    if (i0 >= m) return;
    // per-tile mode: the block of C these elements lie in walked only its own anti-diagonals
    // (a 4 x 4 patch never straddles a block: kTile is a multiple of 4)
    const int S = tile_S ? min(tile_S[(j0 / kTile) * (mp / kTile) + i0 / kTile], S_all) : S_all;
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    typedef std::conditional_t<KIND == KSplit::kNone, const i32x4, i32x4> plane4;
    plane4* t4 = reinterpret_cast<plane4*>(T);
    plane4* l4 = reinterpret_cast<plane4*>(L);   // one dword = the four j of one i
    // the unit of the slice GEMM this patch lies in (a patch never straddles units), and the patch inside it
    int local = 0, units = 0;
    const int il = int(i0) & (kUnit - 1), jl = int(j0) & (kUnit - 1);
    if (KIND != KSplit::kNone) {
        const GemmGrid& g = split.g;
        const int ui = int(i0 / kUnit), uj = int(j0 / kUnit);
        if (tile_S) {      // per-block order of a split product: position = block, quadrants one after the other
            units = 4 * g.count;
            local = ((ui & 1) + 2 * (uj & 1)) * g.count + tile_to_lin(ui >> 1, uj >> 1, g.nti, g.ntj);
        } else {
            units = g.count;
            local = tile_to_lin(ui, uj, g.um, g.un);
        }
    }
    // C is requested first (when it is read at all), then the planes of each k-block in batches: all
    // loads of a batch are in flight together before the first digit is consumed
    double cin[kRecJ][kRecI];
    const bool rows_full = i0 + kRecI <= m;
    // kVecC: C and ldc allow 16-byte accesses (the host checked alignment); used for full groups of four rows
    const bool vec = (c_flags & kVecC) && rows_full;
    if (beta != 0.0) {
#pragma unroll
        for (int jj = 0; jj < kRecJ; ++jj) {
            if (vec && j0 + jj < n) {
                const double2* src = reinterpret_cast<const double2*>(C + (j0 + jj) * ldc + i0);
                const double2 lo2 = src[0], hi2 = src[1];
                cin[jj][0] = lo2.x; cin[jj][1] = lo2.y; cin[jj][2] = hi2.x; cin[jj][3] = hi2.y;
            } else {
#pragma unroll
                for (int q = 0; q < kRecI; ++q)
                    cin[jj][q] = (j0 + jj < n && (rows_full || i0 + q < m)) ? C[(j0 + jj) * ldc + i0 + q] : 0.0;
            }
        }
    }
    double R[kRecJ][kRecI];
#pragma unroll
    for (int jj = 0; jj < kRecJ; ++jj)
#pragma unroll
        for (int q = 0; q < kRecI; ++q) R[jj][q] = 0.0;
    constexpr int kBatch = 8;
    const int kt_total = split.g.kt_total, kt_per_block = int(kblk / kBK);
    for (int kb = 0; kb < nkb; ++kb) {
        // the planes are read once: streaming loads keep them out of the way of C
        const int64_t t_at = ((int64_t(kb) * np + j0) * mp + i0) / 4;                               // + jj * mp / 4
        const int64_t l_at = ((int64_t(kb) * (s_cap - 1) * (np / 4) + j4) * mp + i0) / 4;           // + (d-1) * l_step
        const int64_t l_step = (np / 4) * mp / 4;
        int z_lo = 0, z_hi = 0;
        if (KIND == KSplit::kParts) parts_of_block(kt_total, kt_per_block, split.g.zsplit, kb, z_lo, z_hi);
        auto slot_of = [&](int z) -> const i32x4* {     // part z's T of this patch's unit
            return reinterpret_cast<const i32x4*>(raw) +
                   ((int64_t(z - 1) * units + local) * split.g.nkb_part + (kb - part_first(kt_total, split.g.zsplit, z) / kt_per_block)) *
                       (part_slot_bytes(s_cap) / 16) + il / 4;
        };
        // raw sums of anti-diagonal d: element (j, i) of the unit's slot
        auto raw_of = [&](int d) -> const i32x4* {
            return reinterpret_cast<const i32x4*>(raw) +
                   ((int64_t(kb) * s_cap + d) * split.raw_units + local) * (kUnit * kUnit / 4) + (jl * kUnit + il) / 4;
        };
        i32x4 tv[kRecJ];
#pragma unroll
        for (int jj = 0; jj < kRecJ; ++jj) {
            if (KIND != KSplit::kNone) tv[jj] = i32x4{0, 0, 0, 0};
            if (KIND == KSplit::kAtomic) tv[jj] = raw_of(0)[jj * (kUnit / 4)];
            else if (KIND == KSplit::kNone || z_lo == 0)
                tv[jj] = __builtin_nontemporal_load(&t4[((int64_t(kb) * np + j0 + jj) * mp + i0) / 4]);
        }
        double Rb[kRecJ][kRecI];
        i32x4 carry[kRecJ];
#pragma unroll
        for (int jj = 0; jj < kRecJ; ++jj) {
            carry[jj] = i32x4{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < kRecI; ++q) Rb[jj][q] = 0.0;
        }
        if constexpr (KIND == KSplit::kAtomic) {
            for (int d = S - 1; d >= 1; --d) {
                i32x4 w = {0, 0, 0, 0};
#pragma unroll
                for (int jj = 0; jj < kRecJ; ++jj) {
                    const i32x4 v = raw_of(d)[jj * (kUnit / 4)] + carry[jj];
                    carry[jj] = (v + 128) >> 8;
                    w |= (v & 255) << (8 * jj);
#pragma unroll
                    for (int q = 0; q < kRecI; ++q) Rb[jj][q] = double((v[q] << 24) >> 24) + Rb[jj][q] * 0x1p-8;
                }
                l4[l_at + (d - 1) * l_step] = w;
            }
        } else {
            if (KIND == KSplit::kParts && S == 1)      // no digits: the leading words alone
                for (int z = max(z_lo, 1); z <= z_hi; ++z)
#pragma unroll
                    for (int jj = 0; jj < kRecJ; ++jj) tv[jj] += slot_of(z)[(jl + jj) * (kUnit / 4)];
            for (int d_hi = S - 1; d_hi >= 1; d_hi -= kBatch) {
                i32x4 w[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int d = d_hi - u;
                    if (KIND != KSplit::kNone) w[u] = i32x4{0, 0, 0, 0};
                    if (d >= 1 && (KIND == KSplit::kNone || z_lo == 0))
                        w[u] = __builtin_nontemporal_load(&l4[(((int64_t(kb) * (s_cap - 1) + (d - 1)) * (np / 4) + j4) * mp + i0) / 4]);
                }
                if constexpr (KIND == KSplit::kParts) {
                    // the four digits of a dword are added as two pairs of 16-bit fields, biased so that no field borrows:
                    // field = digit + 128 per part
                    i32x4 even[kBatch], odd[kBatch];
                    const bool main_counts = z_lo == 0;
#pragma unroll
                    for (int u = 0; u < kBatch; ++u) {
                        const i32x4 x = w[u] ^ int(0x80808080);
                        even[u] = main_counts ? x & 0x00FF00FF : i32x4{0, 0, 0, 0};
                        odd[u] = main_counts ? (x >> 8) & 0x00FF00FF : i32x4{0, 0, 0, 0};
                    }
                    // two parts at a time: their loads, and on the first round those of T, are in flight together (one at a
                    // time, T before all digits: 200x300x260 in five parts 21 us, now 14; each round trip counts there)
                    for (int z = max(z_lo, 1); z <= z_hi; z += 2) {
                        i32x4 y[2][kBatch], t2[2][kRecJ];
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            if (z + p > z_hi) continue;
                            const i32x4* top = slot_of(z + p);
                            const i32x4* src = top + kUnit * kUnit / 4 + (jl / 4) * (kUnit / 4);
#pragma unroll
                            for (int u = 0; u < kBatch; ++u)
                                if (d_hi - u >= 1) y[p][u] = src[(d_hi - u - 1) * (kUnit / 4) * (kUnit / 4)];
                            if (d_hi == S - 1) {
#pragma unroll
                                for (int jj = 0; jj < kRecJ; ++jj) t2[p][jj] = top[(jl + jj) * (kUnit / 4)];
                            }
                        }
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            if (z + p > z_hi) continue;
#pragma unroll
                            for (int u = 0; u < kBatch; ++u) {
                                if (d_hi - u < 1) continue;
                                const i32x4 x = y[p][u] ^ int(0x80808080);
                                even[u] += x & 0x00FF00FF;
                                odd[u] += (x >> 8) & 0x00FF00FF;
                            }
                            if (d_hi == S - 1) {
#pragma unroll
                                for (int jj = 0; jj < kRecJ; ++jj) tv[jj] += t2[p][jj];
                            }
                        }
                    }
                    const int bias = 128 * (z_hi - z_lo + 1);
#pragma unroll
                    for (int u = 0; u < kBatch; ++u) {
                        if (d_hi - u < 1) continue;
                        i32x4 out = {0, 0, 0, 0};
#pragma unroll
                        for (int jj = 0; jj < kRecJ; ++jj) {
                            const i32x4 f = (jj & 1) ? odd[u] : even[u];
                            const i32x4 v = ((jj & 2) ? (f >> 16) & 0xFFFF : f & 0xFFFF) - bias + carry[jj];
                            carry[jj] = (v + 128) >> 8;
                            out |= (v & 255) << (8 * jj);
                        }
                        w[u] = out;
                        l4[l_at + (d_hi - u - 1) * l_step] = out;
                    }
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if (d_hi - u >= 1) {
#pragma unroll
                        for (int q = 0; q < kRecI; ++q)
#pragma unroll
                            for (int jj = 0; jj < kRecJ; ++jj) {
                                const int digit = (w[u][q] << (24 - 8 * jj)) >> 24;       // sign-extended byte jj
                                Rb[jj][q] = double(digit) + Rb[jj][q] * 0x1p-8;
                            }
                    }
                }
            }
        }
#pragma unroll
        for (int jj = 0; jj < kRecJ; ++jj) {
            if constexpr (KIND != KSplit::kNone) {
                tv[jj] += carry[jj];
                t4[t_at + jj * (mp / 4)] = tv[jj];
            }
#pragma unroll
            for (int q = 0; q < kRecI; ++q) R[jj][q] = R[jj][q] + (double(tv[jj][q]) + Rb[jj][q] * 0x1p-8);
        }
    }
    const int4 ea4 = *reinterpret_cast<const int4*>(eA + i0);
    const int ea[4] = {ea4.x, ea4.y, ea4.z, ea4.w};
#pragma unroll
    for (int jj = 0; jj < kRecJ; ++jj) {
        const int64_t j = j0 + jj;
        if (j >= n) break;
        const int eb = eB[j];
        double out[kRecI];
#pragma unroll
        for (int q = 0; q < kRecI; ++q) {
            const int sc = (ea[q] > kExpAllZero ? ea[q] : 0) + (eb > kExpAllZero ? eb : 0) + (2 * kHeadroomBits - 12);
            const double ab = ldexp(R[jj][q], sc);
            out[q] = __dmul_rn(alpha, ab);
            if (beta != 0.0) out[q] = __dadd_rn(out[q], __dmul_rn(beta, cin[jj][q]));
        }
        if (vec) {
            typedef double f64x2 __attribute__((ext_vector_type(2)));
            f64x2* dst = reinterpret_cast<f64x2*>(C + j * ldc + i0);
            const f64x2 lo = {out[0], out[1]}, hi = {out[2], out[3]};
            if (c_flags & kStreamC) {
                __builtin_nontemporal_store(lo, dst);
                __builtin_nontemporal_store(hi, dst + 1);
            } else {
                dst[0] = lo;
                dst[1] = hi;
            }
        } else {
#pragma unroll
            for (int q = 0; q < kRecI; ++q)
                if (i0 + q < m) C[j * ldc + i0 + q] = out[q];
        }
    }
}

// C = beta * C (beta == 0 stores zeros without reading C)
__global__ __launch_bounds__(256) void scale_c_kernel(int64_t m, double beta, double* __restrict__ C,
                                                      int64_t ldc) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int64_t j = blockIdx.y;
    if (i >= m) return;
    C[j * ldc + i] = (beta == 0.0) ? 0.0 : __dmul_rn(beta, C[j * ldc + i]);
}

void launch_recompose(hipStream_t st, const Workspace& w, const Problem& p, const SplitPlan& split, double alpha, double beta,
                      double* C, int64_t ldc) {
    const unsigned gx = unsigned((p.m + 256 * kRecI - 1) / (256 * kRecI));
    const int64_t n4 = (p.n + kRecJ - 1) / kRecJ;
    const int c_flags = (reinterpret_cast<uintptr_t>(C) % 16 == 0 && ldc % 2 == 0 && p.batch.c % 2 == 0 ? kVecC : 0) |
                        (results_stream(p) ? kStreamC : 0);
    for (int64_t j4 = 0; j4 < n4; j4 += 65535) {
        const unsigned gy = unsigned(n4 - j4 < 65535 ? n4 - j4 : 65535);
        const int32_t* tile_S = p.tile_mode ? w.tile_S : nullptr;
        const dim3 grid(gx, gy, unsigned(p.batch.count)), block(256);
        if (split.kind == KSplit::kParts)
            hipLaunchKernelGGL(recompose_kernel<KSplit::kParts>, grid, block, 0, st, w.T, w.L, w.raw, split, w.eA, w.eB, p.m,
                               p.n, p.mp, p.np, p.kp, p.s_cap, alpha, beta, C, ldc, w.rec, tile_S, j4, c_flags, p.batch);
        else if (split.kind == KSplit::kAtomic)
            hipLaunchKernelGGL(recompose_kernel<KSplit::kAtomic>, grid, block, 0, st, w.T, w.L, w.raw, split, w.eA, w.eB, p.m,
                               p.n, p.mp, p.np, p.kp, p.s_cap, alpha, beta, C, ldc, w.rec, tile_S, j4, c_flags, p.batch);
        else
            hipLaunchKernelGGL(recompose_kernel<KSplit::kNone>, grid, block, 0, st, w.T, w.L, w.raw, split, w.eA, w.eB, p.m,
                               p.n, p.mp, p.np, p.kp, p.s_cap, alpha, beta, C, ldc, w.rec, tile_S, j4, c_flags, p.batch);
    }
}

void launch_scale_c(hipStream_t st, int64_t m, int64_t n, double beta, double* C, int64_t ldc) {
    const unsigned gx = unsigned((m + 255) / 256);
    for (int64_t j0 = 0; j0 < n; j0 += 65535) {
        const unsigned gy = unsigned(n - j0 < 65535 ? n - j0 : 65535);
        hipLaunchKernelGGL(scale_c_kernel, dim3(gx, gy), dim3(256), 0, st, m, beta, C + j0 * ldc, ldc);
    }
}

}  // namespace oz
