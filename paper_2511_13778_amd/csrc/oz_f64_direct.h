// A tile of the native FP64 GEMM straight from memory: the body of dgemm_f64_direct_kernel, and the fallback inside the launches of
// emulated calls on small tiles.
#pragma once

#include "oz_f64.h"
#include "oz_f64_walk.h"

namespace oz {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kSumBatch = 8;         // fragments whose sums are in LDS at a time

// What walk_share asks of the compiler on the device.
struct KeepOrder {
    __device__ __forceinline__ void order() const { __builtin_amdgcn_sched_barrier(0); }
    __device__ __forceinline__ void scalar(int64_t& x) const { asm volatile("" : "+s"(x)); }
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
    f64x4 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = f64x4{0.0, 0.0, 0.0, 0.0};
    const WaveShare share = wave_share(k, wave, WAVES);
    if (share.first > 0) {
        DirectSide<AC, NI> a;
        DirectSide<BC, NJ> b;
        a.init(A, a_sr, a_sl, i0, m, kb + share.lo, lane);
        b.init(B, b_sr, b_sl, j0, n, kb + share.lo, lane);
        walk_share(share, a, b, lane, [&](int s) {
#pragma unroll
            for (int fj = 0; fj < NJ; ++fj)
#pragma unroll
                for (int fi = 0; fi < NI; ++fi)
                    acc[fj * NI + fi] = __builtin_amdgcn_mfma_f64_16x16x4f64(b.v[s][fj], a.v[s][fi], acc[fj * NI + fi], 0, 0, 0);
        }, KeepOrder{});
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
