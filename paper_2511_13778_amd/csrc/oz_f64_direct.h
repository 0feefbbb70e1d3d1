// A tile of the native FP64 GEMM straight from memory: the body of dgemm_f64_direct_kernel, and the fallback inside the launches of
// emulated calls on small tiles.
#pragma once

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

// bytes of LDS a tile needs
constexpr int f64_direct_lds(int ni, int nj, int waves) {
    return (ni * nj < kSumBatch ? ni * nj : kSumBatch) * (waves - 1) * 256 * 8;
}

// Tile of 16 NI x 16 NJ at (i0, j0) over k [kb, kb + k), by a workgroup of WAVES waves; partial: leave the sums there, the element
// (i, j) of C at partial[j * ldp + i], instead of finishing C.
template <bool AC, bool BC, int NI, int NJ, int WAVES>
__device__ __forceinline__ void f64_direct_tile(double* sums, int64_t m, int64_t n, int64_t k, int64_t kb, int64_t i0, int64_t j0,
                                                double alpha, const double* __restrict__ A, int64_t a_sr, int64_t a_sl,
                                                const double* __restrict__ B, int64_t b_sr, int64_t b_sl, double beta,
                                                double* __restrict__ C, int64_t ldc, double* __restrict__ partial, int64_t ldp) {
    constexpr int NF = NI * NJ, NQ = (NF + WAVES - 1) / WAVES;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // this wave's share of k, in units of four
    const int64_t quads = (k + 3) / 4;
    const int64_t k_lo = quads * wave / WAVES * 4, k_hi = min(quads * (wave + 1) / WAVES * 4, k);
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
    // f mod WAVES, which requests its part of C before it waits for the other waves.
    const int64_t jl = j0 + (lane >> 4), il = i0 + (lane & 15);
    double cin[NQ][4];
    if (beta != 0.0 && !partial) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int f = min(WAVES * q + wave, NF - 1);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                cin[q][r] = C[min(jl + (f / NI) * 16 + 4 * r, n - 1) * ldc + min(il + (f % NI) * 16, m - 1)];
        }
    }
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += kSumBatch) {
        if (f0 > 0) __syncthreads();
#pragma unroll
        for (int f = f0; f < f0 + kSumBatch && f < NF; ++f) {
            const int owner = f % WAVES;
            if (wave != owner) {
                double* dst = sums + ((f - f0) * (WAVES - 1) + (wave > owner ? wave - 1 : wave)) * 256 + lane;
#pragma unroll
                for (int r = 0; r < 4; ++r) dst[r * 64] = acc[f][r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int f = f0; f < f0 + kSumBatch && f < NF; ++f) {
            const int owner = f % WAVES, q = f / WAVES;
            if (wave != owner) continue;
            const double* src = sums + (f - f0) * (WAVES - 1) * 256 + lane;
            const int64_t i = il + (f % NI) * 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double sum = 0.0;
#pragma unroll
                for (int w = 0, x = 0; w < WAVES; ++w) {
                    const double part = w == owner ? acc[f][r] : src[(x++) * 256 + r * 64];
                    sum = w == 0 ? part : __dadd_rn(sum, part);
                }
                const int64_t j = jl + (f / NI) * 16 + 4 * r;
                if (partial) {
                    partial[j * ldp + i] = sum;
                } else if (i < m && j < n) {
                    double out = __dmul_rn(alpha, sum);
                    if (beta != 0.0) out = __dadd_rn(out, __dmul_rn(beta, cin[q][r]));
                    C[j * ldc + i] = out;
                }
            }
        }
    }
}

// What an emulated call's last launch needs to fall back by itself.  A == nullptr: it need not, the FP64 GEMM has its own launch.
struct Fallback {
    const double* A;
    int64_t a_sr, a_sl;
    const double* B;
    int64_t b_sr, b_sl;
    int64_t k;
    int32_t a_rows, b_rows;
};

// problem p of a batch, tile (i0, j0) of 16 NI x 16 NJ
template <int NI, int NJ, int WAVES>
__device__ __forceinline__ void fall_back(const Fallback& f, const Batch& bt, int p, double* lds, int64_t m, int64_t n, int64_t i0, int64_t j0,
                                          double alpha, double beta, double* __restrict__ C, int64_t ldc) {
    const double* const A = f.A + bt.a_at(p);
    const double* const B = f.B + bt.b_at(p);
#define OZ_FALL(AC, BC) f64_direct_tile<AC, BC, NI, NJ, WAVES>(lds, m, n, f.k, 0, i0, j0, alpha, A, f.a_sr, f.a_sl, B, f.b_sr, f.b_sl, beta, C, ldc, nullptr, 0)
    if (f.a_rows && f.b_rows) OZ_FALL(true, true);
    else if (f.a_rows) OZ_FALL(true, false);
    else if (f.b_rows) OZ_FALL(false, true);
    else OZ_FALL(false, false);
#undef OZ_FALL
}

}  // namespace oz
