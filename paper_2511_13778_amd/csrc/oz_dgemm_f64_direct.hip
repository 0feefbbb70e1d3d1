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
// Whole calls, against LDS tiles of 64 with k split over workgroups: 1000 x 1300 x 777 53 -> 44 us, 512^3 17 -> 10,
// 600 x 700 x 500 29 -> 14, 200 x 300 x 5000 45 -> 29, 64 x 64 x 7000 35 -> 13.  Large products stay on the LDS tiles (4096^3
// 1866 us, here 1918): an operand fragment is read by four waves there, here by one.
#include "oz_f64.h"

namespace oz {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

constexpr int kChunkK = 16;          // k per loop iteration: four MFMA steps
constexpr int kSumBatch = 8;         // fragments whose sums are in LDS at a time

// One operand of a wave: NF fragments of 16 rows.  MFMA step s of a chunk multiplies k = 4g + s for lane group g (the same set for
// both operands), so a lane of a k-contiguous operand reads 16 bytes for two steps and four lanes 128 in a row.
// The address is a wave-uniform base plus a 32-bit lane offset that never changes.
template <bool ROWS_CONTIG, int NF>
struct DirectSide {
    const char* u;           // wave-uniform: row r0 of the operand at the k that is loaded next
    uint32_t off[NF];        // this lane's row of fragment f and its k inside a chunk, bytes
    int64_t sl;              // bytes from one k to the next
    double v[4][NF];         // fragments of the four MFMA steps of a chunk

    __device__ __forceinline__ void init(const double* X, int64_t stride_r, int64_t stride_l, int64_t r0, int64_t rows, int64_t k0) {
        u = reinterpret_cast<const char*>(X + r0 * stride_r + k0 * stride_l);
        sl = stride_l * 8;
        const int lane = threadIdx.x & 63, g = lane >> 4;
#pragma unroll
        for (int f = 0; f < NF; ++f) {         // rows past the end are read from the last one; what they give is never stored
            const int64_t r = min(int64_t(f * 16 + (lane & 15)), rows - 1 - r0);
            off[f] = uint32_t(r * stride_r + int64_t(4 * g) * stride_l) * 8u;
        }
    }
    // the first chunk: `len` (1..16) k, in the last ceil(len / 4) steps, four k a step
    __device__ __forceinline__ void load_first(int len) {
        const int g = (threadIdx.x & 63) >> 4, skip = 4 - (len + 3) / 4;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int kk = 4 * (s - skip) + g;                     // this lane's k, read at the nearest one there is
            const int64_t at = int64_t(min(max(kk, 0), len - 1) - 4 * g) * sl;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double x = *reinterpret_cast<const double*>(u + off[f] + at);
                v[s][f] = kk >= 0 && kk < len ? x : 0.0;
            }
        }
    }
    // step s of the chunk at u; k-contiguous operands come two steps at a time
    __device__ __forceinline__ void load(int s) {
        if (ROWS_CONTIG) {
            const char* us = u + s * sl;
#pragma unroll
            for (int f = 0; f < NF; ++f) v[s][f] = *reinterpret_cast<const double*>(us + off[f]);
        } else if (s & 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const f64x2u x = *reinterpret_cast<const f64x2u*>(u + (s - 1) * 8 + off[f]);
                v[s - 1][f] = x[0];
                v[s][f] = x[1];
            }
        }
    }
};

// Tile of 16 NI x 16 NJ; grid: tiles x zsplit, part 0 of k carries k mod kpart as in dgemm_f64_kernel.
template <bool AC, bool BC, int NI, int NJ>
__global__ __launch_bounds__(256, NI * NJ <= 4 ? 4 : 2) void dgemm_f64_direct_kernel(
    const Record* rec, KnownRecord known, int64_t m, int64_t n, int64_t k, double alpha, const double* __restrict__ A,
    int64_t a_sr, int64_t a_sl, const double* __restrict__ B, int64_t b_sr, int64_t b_sl, double beta,
    double* __restrict__ C, int64_t ldc, int ntm, int ntn, int zsplit, int64_t kpart, double* __restrict__ partial, Batch bt) {
    constexpr int TI = 16 * NI, TJ = 16 * NJ, NF = NI * NJ, NQ = (NF + 3) / 4;
    constexpr int kPerBatch = kSumBatch / 4;
    __shared__ double sums[3 * (NF < kSumBatch ? NQ * 4 : kSumBatch) * 4 * 64];
    f64_problem(bt, rec, A, B, C, partial);
    if (rec && !rec->res.fallback) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) write_known_record(known, bt, int(blockIdx.z));
    int ti, tj, z;
    f64_tile_of(int(blockIdx.x), ntm, ntn, zsplit, ti, tj, z);
    const int64_t i0 = int64_t(ti) * TI, j0 = int64_t(tj) * TJ;
    int64_t kb;
    f64_k_part(zsplit, z, kpart, k, kb);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // this wave's quarter of k, in units of four
    const int64_t quads = (k + 3) / 4;
    const int64_t k_lo = quads * wave / 4 * 4, k_hi = min(quads * (wave + 1) / 4 * 4, k);
    f64x4 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (k_lo < k_hi) {
        const int first = int((k_hi - k_lo - 1) % kChunkK) + 1;
        DirectSide<AC, NI> a;
        DirectSide<BC, NJ> b;
        a.init(A, a_sr, a_sl, i0, m, kb + k_lo);
        b.init(B, b_sr, b_sl, j0, n, kb + k_lo);
        a.load_first(first);
        b.load_first(first);
        int64_t adv = first;
        int skip = 4 - (first + 3) / 4;  // MFMA steps the first chunk does not need
        for (int left = int((k_hi - k_lo - first) / kChunkK);; --left) {
            if (left > 0) {              // otherwise the chunk is loaded again, for nobody
                a.u += adv * a.sl;
                b.u += adv * b.sl;
            }
            adv = kChunkK;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s >= skip) {
#pragma unroll
                    for (int fj = 0; fj < NJ; ++fj)
#pragma unroll
                        for (int fi = 0; fi < NI; ++fi)
                            acc[fj * NI + fi] = __builtin_amdgcn_mfma_f64_16x16x4f64(b.v[s][fj], a.v[s][fi], acc[fj * NI + fi], 0, 0, 0);
                }
                a.load(s);
                b.load(s);
                __builtin_amdgcn_sched_barrier(0);
            }
            skip = 0;
            if (left == 0) break;
        }
    }

    // result register r of fragment f: j = (f / NI) * 16 + 4r + lane / 16, i = (f % NI) * 16 + lane % 16.  Fragment f is finished by wave
    // f mod 4, which requests its part of C before it waits for the other waves.
    const int64_t jl = j0 + (lane >> 4), il = i0 + (lane & 15);
    double cin[NQ][4];
    if (beta != 0.0 && zsplit == 1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int f = min(4 * q + wave, NF - 1);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                cin[q][r] = C[min(jl + (f / NI) * 16 + 4 * r, n - 1) * ldc + min(il + (f % NI) * 16, m - 1)];
        }
    }
#pragma unroll
    for (int q0 = 0; q0 < NQ; q0 += kPerBatch) {
        if (q0 > 0) __syncthreads();
#pragma unroll
        for (int f = 4 * q0; f < 4 * (q0 + kPerBatch) && f < NF; ++f) {
            const int owner = f & 3;
            if (wave != owner) {
                double* dst = sums + ((f - 4 * q0) * 3 + (wave > owner ? wave - 1 : wave)) * 256 + lane;
#pragma unroll
                for (int r = 0; r < 4; ++r) dst[r * 64] = acc[f][r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int f = 4 * q0; f < 4 * (q0 + kPerBatch) && f < NF; ++f) {
            const int owner = f & 3, q = f >> 2;
            if (wave != owner) continue;
            const double* src = sums + (f - 4 * q0) * 3 * 256 + lane;
            const int64_t i = il + (f % NI) * 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double part[4];
#pragma unroll
                for (int w = 0, x = 0; w < 4; ++w) part[w] = w == owner ? acc[f][r] : src[(x++) * 256 + r * 64];
                const double sum = __dadd_rn(__dadd_rn(__dadd_rn(part[0], part[1]), part[2]), part[3]);
                const int64_t j = jl + (f / NI) * 16 + 4 * r;
                if (zsplit > 1) {
                    partial[(int64_t(z) * ntn * TJ + j) * (int64_t(ntm) * TI) + i] = sum;
                } else if (i < m && j < n) {
                    double out = __dmul_rn(alpha, sum);
                    if (beta != 0.0) out = __dadd_rn(out, __dmul_rn(beta, cin[q][r]));
                    C[j * ldc + i] = out;
                }
            }
        }
    }
}

void launch_dgemm_f64_direct(hipStream_t st, const F64Call& c, const F64Plan& p) {
    const dim3 grid(unsigned(p.ntm) * unsigned(p.ntn) * unsigned(p.zsplit), 1, unsigned(c.batch.count)), block(256);
#define OZ_DIRECT(AC, BC, NI, NJ)                                                                                        \
    hipLaunchKernelGGL((dgemm_f64_direct_kernel<AC, BC, NI, NJ>), grid, block, 0, st, c.rec, c.known, c.m, c.n, c.k,      \
                       c.alpha, c.A, c.a_sr, c.a_sl, c.B, c.b_sr, c.b_sl, c.beta, c.C, c.ldc, p.ntm, p.ntn, p.zsplit, \
                       p.kpart, p.partial, c.batch)
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
