// How a product of the native FP64 GEMM is cut into workgroups: tile, parts of k and form of the K loop, kept apart from the kernels
// so that a host program can follow the choice.
#pragma once

#include <algorithm>

#include "oz_internal.h"

namespace oz {

constexpr int kDK = 16;                         // K step of dgemm_f64_kernel

// What the choice depends on.  guarded: behind a verdict that may not select the product.
struct F64Size {
    int64_t m, n, k;
    int problems;
    bool guarded;
};

struct F64Plan {
    bool direct;           // dgemm_f64_direct_kernel, otherwise dgemm_f64_kernel
    int ti, tj;            // tile
    int ntm, ntn;          // tiles
    int zsplit;            // parts of k over workgroups
    int64_t kpart;         // length of every part but the first
    double* partial;       // [zsplit][ntn * tj][ntm * ti] partial products of a split
};

// Tiles a call can be cut into and what they cost, in us: a workgroup start + round per round of all CUs, and step per MFMA step of a
// round (16 k in dgemm_f64_kernel, 4 k of each of the four waves in dgemm_f64_direct_kernel); first: per step of the call, for
// the operands' way to the first workgroup of a CU.  Operands come out of the caches at 9 TB/s at most (4096^3 and 6144^3 on tiles of
// 64 and less).  Fitted to 5879 timings of 126 shapes (50 to 8000, k to 65000, all four transposes, every tile, 1 to 16 parts): the
// choice by these numbers is 3 % off the best one on average, 19 % at most, and 1.18 times as fast as the best choice among
// the two tiles of dgemm_f64_kernel (at most 10 % slower).
struct F64Tile {
    bool direct;
    int ti, tj;
    double start, round, step, first;
};
constexpr F64Tile kF64Tiles[] = {
    {false, 128, 128, 0.0, 7.42, 1.717, 0.167}, {false, 64, 64, 2.51, 1.69, 0.433, 0.336},
    {true, 16, 16, 3.26, 0.38, 0.075, 0.018},   {true, 32, 32, 3.53, 0.94, 0.169, 0.0},
    {true, 32, 64, 4.07, 2.00, 0.273, 0.0},     {true, 64, 32, 3.31, 2.56, 0.262, 0.008},
    {true, 48, 64, 3.10, 3.95, 0.341, 0.039},   {true, 64, 48, 3.46, 3.47, 0.361, 0.027},
};
constexpr double kF64CacheBytesPerUs = 9e6;

// Tile and number of parts of the k range.  With scratch memory at hand, k may be split over several workgroups per tile:
// they leave partial products in the scratch memory and a second kernel adds them in the order of the parts (deterministic)
// and applies alpha and beta: a launch of 4.5 us and zsplit + 2 passes over C at 4.5 TB/s.  A guarded call pays that launch
// whether it falls back or not: 20 there.
inline F64Plan choose_f64(const F64Size& c, int num_cu, void* scratch, size_t scratch_bytes, double* us_of = nullptr) {
    F64Plan best{};
    double best_us = 0.0;
    const uint32_t m = uint32_t(c.m), n = uint32_t(c.n), cus = uint32_t(num_cu), problems = uint32_t(c.problems);
    for (const F64Tile& t : kF64Tiles) {
        if (!t.direct && c.k < kDK) continue;                // whose fast loads always fetch a full K step
        const uint32_t ti = uint32_t(t.ti), tj = uint32_t(t.tj), ntm = (m + ti - 1) / ti, ntn = (n + tj - 1) / tj;
        const uint64_t tiles64 = uint64_t(ntm) * ntn;
        if (tiles64 > uint64_t(kMaxGridThreads) / 256) continue;
        const uint32_t tiles = uint32_t(tiles64);            // of a problem
        const uint64_t all = tiles64 * problems;
        const double cache_us = double(all) * double(ti + tj) * double(c.k) * 8.0 / kF64CacheBytesPerUs;
        const int64_t k_least = t.ti == 128 ? 256 : 64;      // what a part keeps at least
        for (uint32_t z : {1u, 2u, 3u, 4u, 6u, 8u, 12u, 16u}) {
            if (z > 1 && (scratch == nullptr || c.k < k_least * z || all * z > 4 * cus ||
                          uint64_t(tiles) * z * ti * tj * 8 > scratch_bytes))
                break;
            const double rounds = double((all * z + cus - 1) / cus), steps = double(uint32_t(c.k + z * kDK - 1) / (z * kDK));
            double us = std::max(t.start + rounds * (t.round + t.step * steps) + t.first * steps, cache_us);
            if (z > 1) us += (c.guarded ? 20.0 : 4.5) + double(z + 2) * double(m) * double(n) * double(problems) * 8.0 / 4.5e6;
            if (best_us == 0.0 || us < best_us) {
                best_us = us;
                best = F64Plan{t.direct, t.ti, t.tj, int(ntm), int(ntn), int(z), z > 1 ? c.k / z / kDK * kDK : 0,
                               static_cast<double*>(scratch)};
            }
        }
    }
    if (us_of) *us_of = best_us;
    return best;
}

// operands cut out of a very large parent matrix, or a size of 2^31 and more: offsets inside a tile may not fit 32 bits (a lane's
// own: at most 15 leading dimensions plus a row of the tile; its elements: up to 7 x 16 leading dimensions further on; in bytes)
inline bool wide_offsets(int64_t m, int64_t n, int64_t k, int64_t ld_max) {
    return (128 * ld_max + 256) * 8 >= (int64_t(1) << 32) || ((m | n | k) >> 31) != 0;
}

// Form of dgemm_f64_kernel's K loop: 0 and 1 load full K steps through 32-bit offsets (1: edge tiles, and a short first step),
// 2 checks bounds with 64-bit indexing in every step.  k < 16 has no full step to load.
inline int f64_mode(bool wide, int64_t m, int64_t n, int64_t k, int ti, int tj) {
    if (wide || k < kDK) return 2;
    return (m % ti || n % tj || k % kDK) ? 1 : 0;
}

}  // namespace oz
