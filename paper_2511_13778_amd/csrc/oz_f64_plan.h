// How a product of the native FP64 GEMM is cut into workgroups: tile, parts of k and form of the K loop, kept apart from the kernels
// so that a host program can follow the choice.
#pragma once

#include <algorithm>

#include "oz_internal.h"

namespace oz {

constexpr int kDK = 16;                         // K step of dgemm_f64_kernel

// What the choice depends on.
struct F64Size {
    int64_t m, n, k;
    int problems;
    bool guarded;          // behind a verdict that may not select the product
    bool beta;             // C is read
    int k_contig;          // operands with k contiguous (0 to 2), and how many of them have their rows at addresses that share the
    double near;           // caches' sets: 1 each for rows a multiple of 512 bytes apart, 0.7 of 128
};
inline F64Size f64_size(int64_t m, int64_t n, int64_t k, int problems, bool guarded, bool beta, bool a_rows, int64_t lda, bool b_rows, int64_t ldb) {
    auto near = [](bool rows, int64_t ld) { return rows ? 0.0 : (ld % 64 == 0 ? 1.0 : (ld % 16 == 0 ? 0.7 : 0.0)); };
    return F64Size{m, n, k, problems, guarded, beta, int(!a_rows) + int(!b_rows), near(a_rows, lda) + near(b_rows, ldb)};
}

struct F64Plan {
    bool direct;           // dgemm_f64_direct_kernel, otherwise dgemm_f64_kernel
    int ti, tj;            // tile
    int ntm, ntn;          // tiles
    int zsplit;            // parts of k over workgroups
    int64_t kpart;         // length of every part but the first
    double* partial;       // [zsplit][ntn * tj][ntm * ti] partial products of a split
};

// Tiles a call can be cut into and what they cost, in us: start, and per round of all CUs: round, more with beta, step per MFMA step
// (16 k in dgemm_f64_kernel, 4 k of each of the four waves in dgemm_f64_direct_kernel); first: per step of the call, for the operands'
// way to the first workgroup of a CU, and far, where they are more than an XCD's L2 holds; c per million elements of C, more with
// beta.  Tiles straight from memory: per step and round more for each operand with k contiguous, and for its rows near each other in
// the caches' sets, and so per round.  Tiles through LDS: more where an edge is ragged, and per round where k has a short first step.  Operands come out of the caches at 9 TB/s at most; of two
// cuts they bound alike, the one with less else to do.
// A split of k costs a launch and 0.31 us a part (the sums are added one after the other), and passes over C (2.6: with 2.0 the model takes
// eight parts for 256 x 7936 x 8192, 508 us, and four take 494).
// Fitted to 9406 calls (2 to 8000, k 1 to 50000, all four transposes, beta zero and not), each timed on every tile, from k = 64 on with
// 1 to 16 parts: the choice is 1.2 % off the best on average (a model without beta, layout and ragged edges, fitted to k of 50 and
// more, was 4.7 % off; 1261 x 2649 x 18 with beta took 31.9 us on 128 x 128 tiles, now 17; 7732 x 2885 x 14 66.9 us, now 36).
struct F64Tile {
    bool direct;
    int ti, tj;
    double start, round, round_beta, step, first, far, c, c_beta;
    double k_step, near_step, near_round;      // straight from memory
    double ragged, short_round;                // through LDS
};
constexpr F64Tile kF64Tiles[] = {
    {false, 128, 128, 4.68, 0.0, 0.812, 1.610, 0.280, 0.0, 1.42, 2.81, 0.0, 0.0, 0.0, 0.66, 0.451},
    {false, 64, 64, 4.13, 0.0, 0.790, 0.446, 0.225, 0.088, 0.96, 0.59, 0.0, 0.0, 0.0, 0.75, 0.204},
    {true, 16, 16, 4.08, 0.215, 0.065, 0.048, 0.0, 0.035, 2.03, 0.14, 0.005, 0.015, 0.051, 0.0, 0.0},
    {true, 32, 32, 4.39, 0.423, 0.080, 0.140, 0.0, 0.006, 0.18, 0.27, 0.001, 0.013, 0.280, 0.0, 0.0},
    {true, 32, 64, 4.61, 0.596, 0.153, 0.288, 0.0, 0.0, 1.33, 0.32, 0.0, 0.009, 0.408, 0.0, 0.0},
    {true, 64, 32, 4.59, 0.492, 0.189, 0.285, 0.0, 0.0, 1.22, 0.30, 0.0, 0.004, 0.604, 0.0, 0.0},
    {true, 48, 64, 5.11, 0.804, 0.557, 0.391, 0.0, 0.0, 1.33, 0.19, 0.0, 0.0, 0.449, 0.0, 0.0},
    {true, 64, 48, 5.06, 1.188, 0.361, 0.409, 0.0, 0.0, 1.66, 0.11, 0.0, 0.0, 0.540, 0.0, 0.0},
};
constexpr double kF64CacheBytesPerUs = 9e6;
constexpr double kF64NearBytes = 4e6;
constexpr double kGuardedSplitUs = 7.5;         // charged for a split where calls that do not fall back pay 3 to 4 for the launch that adds its parts
                                                // (at 15.5 58 x 32 x 4432 took 53.8 us falling back, now 33)

// Tile and number of parts of the k range.  With scratch memory at hand, k may be split over several workgroups per tile:
// they leave partial products in the scratch memory and a second kernel adds them in the order of the parts (deterministic)
// and applies alpha and beta.
// scratch_bytes 0: none.  The caller sets where the partial products go.
inline F64Plan choose_f64(const F64Size& c, int num_cu, size_t scratch_bytes, double* us_of = nullptr) {
    F64Plan best{};
    double best_us = 0.0;
    const uint32_t m = uint32_t(c.m), n = uint32_t(c.n), cus = uint32_t(num_cu), problems = uint32_t(c.problems);
    const double area = double(c.m) * double(c.n) * double(problems) * 1e-6;
    const bool far = double(c.m + c.n) * double(c.k) * double(c.problems) * 8.0 > kF64NearBytes;
    for (const F64Tile& t : kF64Tiles) {
        const double first = t.first + (far ? t.far : 0.0);
        const uint32_t ti = uint32_t(t.ti), tj = uint32_t(t.tj), ntm = (m + ti - 1) / ti, ntn = (n + tj - 1) / tj;
        const uint64_t tiles64 = uint64_t(ntm) * ntn;
        if (tiles64 > uint64_t(kMaxGridThreads) / 256) continue;
        const uint32_t tiles = uint32_t(tiles64);            // of a problem
        const uint64_t all = tiles64 * problems;
        const bool short_first = c.k % kDK != 0, ragged = short_first || m % ti != 0 || n % tj != 0;
        const double cache_us = double(all) * double(ti + tj) * double(c.k) * 8.0 / kF64CacheBytesPerUs;
        const double per_call = t.start + (ragged ? t.ragged : 0.0) + area * (t.c + (c.beta ? t.c_beta : 0.0));
        const double per_round = t.round + (c.beta ? t.round_beta : 0.0) + t.near_round * c.near + (short_first ? t.short_round : 0.0);
        const double per_step = t.step + t.k_step * c.k_contig + t.near_step * c.near;
        const int64_t k_least = t.ti == 128 ? 256 : 64;      // what a part keeps at least
        for (uint32_t z : {1u, 2u, 3u, 4u, 6u, 8u, 12u, 16u}) {
            if (z > 1 && (scratch_bytes == 0 || c.k < k_least * z || all * z > 4 * cus ||
                          uint64_t(tiles) * z * ti * tj * 8 > scratch_bytes))
                break;
            // 128 x 128, no operand with k contiguous: the two workgroups of a CU keep step, and where the last rounds are an odd one the
            // pairs that start together leave half of the CUs without any (513 to 768 tiles take as long as 1024: 2703 x 4171 x 3943 1842 us,
            // on 64 x 64 tiles 1560)
            uint64_t rounds_whole = (all * z + cus - 1) / cus;
            if (t.ti == 128 && c.k_contig == 0 && rounds_whole > 1) rounds_whole += rounds_whole & 1;
            const double rounds = double(rounds_whole), steps = double(uint32_t(c.k + z * kDK - 1) / (z * kDK));
            double us = per_call + rounds * (per_round + per_step * steps) + first * steps;
            if (z > 1) us += 1.4 + 0.31 * double(z) + 2.6 * double(z + 2) * area;
            us = std::max(us, 0.7 * cache_us + 0.3 * us);
            if (z > 1 && c.guarded) us += kGuardedSplitUs;
            // sums in four parts have half the error: tiles straight from memory where they are as fast
            if (!t.direct && z == 1 && c.k >= 128) us *= 1.03;
            if (best_us == 0.0 || us < best_us) {
                best_us = us;
                best = F64Plan{t.direct, t.ti, t.tj, int(ntm), int(ntn), int(z), z > 1 ? c.k / z / kDK * kDK : 0, nullptr};
            }
        }
    }
    if (us_of) *us_of = best_us;
    return best;
}

// operands cut out of a very large parent matrix, or a size of 2^31 and more: offsets inside a tile may not fit 32 bits, in bytes.
// Tiles through LDS: a lane's own is at most 15 leading dimensions plus a row of the tile, its elements lie up to 7 x 16 leading
// dimensions further on.  Tiles straight from memory: a lane's own is at most 63 leading dimensions (the last row of 64, k contiguous)
// plus 12 of k, or 12 leading dimensions plus a row; what a step adds is kept in 64 bits.
inline bool wide_offsets(int64_t m, int64_t n, int64_t k, int64_t ld_max) {
    return (128 * ld_max + 256) * 8 >= (int64_t(1) << 32) || ((m | n | k) >> 31) != 0;
}

// Whether the native product of a guarded call is as fast on square tiles of this edge (32: gemm_small_kernel, 64: gemm_mid_kernel) in the
// last launch of the emulated call as in launches of its own: whatever choose_f64 takes for it, with the call's scratch memory.
// alone: the emulated kernel's LDS leaves one workgroup to a CU.
// In us: launches of its own take 1.6, 0.9 of choose_f64's estimate and 4.6 for the sums of a split; tiles as below, and no less than the
// operands at the rate of the caches.  Fitted to 2250 calls that fall back (16 to 8000, k 20 to 6000), timed with either: half of
// them fold, 0.6 % slower than the better one on average, and sixteen by more than 5 % than in launches of their own.  (Against the
// unsplit product alone, without the layout and with two workgroups to a CU throughout, 519 x 123 x 4328 took 72 us, now 41, and
// 811 x 1516 x 101 36, now 26.)
inline bool f64_folds(const F64Size& c, int num_cu, size_t scratch_bytes, int edge, bool alone) {
    double own_us = 0.0;
    const F64Plan own = choose_f64(c, num_cu, scratch_bytes, &own_us);
    if (own.zsplit > 1) own_us -= kGuardedSplitUs;
    own_us = 1.6 + 0.9 * own_us + (own.zsplit > 1 ? 4.6 : 0.0);
    const int64_t tiles = ((c.m + edge - 1) / edge) * ((c.n + edge - 1) / edge) * c.problems;
    const int64_t per_round = edge == 64 || alone ? num_cu : 2 * num_cu;
    const double rounds = double((tiles + per_round - 1) / per_round), steps = double((c.k + kDK - 1) / kDK);
    const double area = double(c.m) * double(c.n) * double(c.problems) * 1e-6, beta = c.beta ? 1.0 : 0.0;
    double us;
    if (edge == 64) us = rounds * (4.87 + 0.458 * steps + 0.46 * beta + 1.01 * c.near) + 2.17 * area;
    else if (alone) us = 0.82 + rounds * (2.23 + (0.118 + 0.017 * c.k_contig) * steps + 0.30 * beta + 0.93 * c.near) + 2.82 * area;
    else us = 0.60 + 0.045 * steps + rounds * ((0.224 + 0.053 * c.k_contig) * steps + 0.42 * beta + 0.71 * c.near) + 5.90 * area;
    return std::max(us, double(tiles) * (2 * edge) * double(c.k) * 8.0 / kF64CacheBytesPerUs) <= own_us;
}

// Whether `all` products of one shape go into one launch, without scratch memory, or `at_once` at a time with a split of k for each
// where that pays.  A launch that cannot split has to be 3 % better: whole-k tiles of one workgroup each end far apart (524 x 591 x 27591,
// four products: 1799 us in one launch, estimated 1357; 1594 split, one after the other).
inline bool f64_together(F64Size c, int all, int at_once, int num_cu, size_t scratch_bytes) {
    double one_us = 0.0, group_us = 0.0;
    c.problems = all;
    choose_f64(c, num_cu, 0, &one_us);
    c.problems = at_once;
    const F64Plan group = choose_f64(c, num_cu, scratch_bytes, &group_us);
    return one_us <= group_us * double((all + at_once - 1) / at_once) * (group.zsplit > 1 ? 0.97 : 1.0);
}

// Form of dgemm_f64_kernel's K loop: 0 and 1 load full K steps through 32-bit offsets (1: edge tiles, and a short first step),
// 2 checks bounds with 64-bit indexing in every step.  k < 16 has no full step to load.
inline int f64_mode(bool wide, int64_t m, int64_t n, int64_t k, int ti, int tj) {
    if (wide || k < kDK) return 2;
    return (m % ti || n % tj || k % kDK) ? 1 : 0;
}

}  // namespace oz
