// How a wave of the FP64 tiles straight from memory walks its share of k: which elements it loads and which MFMA step multiplies
// them.  Apart from the kernel so that a host program can run the same code over the operands (tests/host_f64_walk.cpp).
#pragma once

#include "oz_internal.h"

namespace oz {

typedef double f64x2u __attribute__((vector_size(16), aligned(8)));

constexpr int kChunkK = 16;          // k per loop iteration: four MFMA steps

// k range of one of `waves` waves, in units of four: [lo, lo + first + 16 * chunks), the remainder of 16 first.  first == 0: nothing.
struct WaveShare {
    int64_t lo;
    int first;           // 1 .. 16
    int chunks;          // full ones behind it
};
__host__ __device__ __forceinline__ WaveShare wave_share(int64_t k, int wave, int waves) {
    const int64_t quads = (k + 3) / 4;
    const int64_t lo = quads * wave / waves * 4, end = quads * (wave + 1) / waves * 4, hi = end < k ? end : k;
    if (lo >= hi) return WaveShare{lo, 0, 0};
    const int first = int((hi - lo - 1) % kChunkK) + 1;
    return WaveShare{lo, first, int((hi - lo - first) / kChunkK)};
}

// One operand of a wave: NF fragments of 16 rows.  MFMA step s of a chunk multiplies k = 4g + s for lane group g (the same set for
// both operands), so a lane of a k-contiguous operand reads 16 bytes for two steps and four lanes 128 in a row.
// The address is a wave-uniform base plus a 32-bit lane offset that never changes.
template <bool ROWS_CONTIG, int NF>
struct DirectSide {
    const char* u;           // wave-uniform: row r0 of the operand at the k that is loaded next
    uint32_t off[NF];        // this lane's row of fragment f and its k inside a chunk, bytes
    int64_t sl;              // bytes from one k to the next
    double v[4][NF];         // fragments of the four MFMA steps of a chunk

    __host__ __device__ __forceinline__ void init(const double* X, int64_t stride_r, int64_t stride_l, int64_t r0, int64_t rows, int64_t k0,
                                                  int lane) {
        u = reinterpret_cast<const char*>(X + r0 * stride_r + k0 * stride_l);
        sl = stride_l * 8;
        const int g = lane >> 4;
#pragma unroll
        for (int f = 0; f < NF; ++f) {         // rows past the end are read from the last one; what they give is never stored
            const int64_t row = f * 16 + (lane & 15), last = rows - 1 - r0, r = row < last ? row : last;
            off[f] = uint32_t(r * stride_r + int64_t(4 * g) * stride_l) * 8u;
        }
    }
    // the first chunk: `len` (1..16) k, in the last ceil(len / 4) steps, four k a step
    __host__ __device__ __forceinline__ void load_first(int len, int lane) {
        const int g = lane >> 4, skip = 4 - (len + 3) / 4;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int kk = 4 * (s - skip) + g, nearest = kk < 0 ? 0 : (kk < len ? kk : len - 1);     // this lane's k, read at the nearest one there is
            const int64_t at = int64_t(nearest - 4 * g) * sl;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double x = *reinterpret_cast<const double*>(u + off[f] + at);
                v[s][f] = kk >= 0 && kk < len ? x : 0.0;
            }
        }
    }
    // step s of the full chunk at u; k-contiguous operands come two steps at a time
    __host__ __device__ __forceinline__ void load(int s) {
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

// Loads and multiplies a share that is not empty; multiply(s): MFMA step s with the fragments a.v[s], b.v[s]; keep.order(): the loads
// of a step stay behind its products; keep.scalar(x): addresses are advanced in scalar registers.
template <class SideA, class SideB, class Multiply, class Keep>
__host__ __device__ __forceinline__ void walk_share(const WaveShare& w, SideA& a, SideB& b, int lane, Multiply&& multiply, const Keep& keep) {
    a.load_first(w.first, lane);
    b.load_first(w.first, lane);
    int64_t adv = w.first;
    int skip = 4 - (w.first + 3) / 4;    // MFMA steps the first chunk does not need
    for (int left = w.chunks; left > 0; --left) {
        int64_t step_a = adv * a.sl, step_b = adv * b.sl;
        keep.scalar(step_a);
        keep.scalar(step_b);
        a.u += step_a;
        b.u += step_b;
        adv = kChunkK;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= skip) multiply(s);
            a.load(s);
            b.load(s);
            keep.order();
        }
        skip = 0;
    }
    // The last chunk is multiplied without another load: load() reads 16 k, and where the share is one short chunk fewer are left
    // in the operand.
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (s >= skip) multiply(s);
}

}  // namespace oz
