// Coarsened Exponent Span Capacity and the verdict.
// (paper: section "ESC", formula ESC = exp(x_p) + exp(y_q) - exp(z_r) maximised over the mn dot
//  products with z_r estimated from per-block Max/Min exponents, plus the +1 safety margin;
//  sections "Heuristic run time Selection" and "GPU-Resident Integration" for the verdict.)
//
// The estimate is a max-plus matrix product  zt = U (x) V  with inner length 2G:
//   zt_ij = max_h ( U[h][i] + V[h][j] ),  U = [Max(xb); Min(xb)],  V = [Min(yb); Max(yb)],
// followed by  span = max_ij ( eA_i + eB_j - zt_ij ).
//
// Two ways to compute it, in one kernel (esc_kernel), block of 128 x 128 pairs by block.
//  * On the BF16 matrix unit.
//    With u = U[h][i] - eA_i <= 0 and v = V[h][j] - eB_j <= 0 the table entries are encoded as
//    the powers of two 2^(5u+61) and 2^(5v+61) (exact in BF16; entries below -37 and the "zero"
//    sentinels become 0).  One MFMA sums 16 such products in FP32; all terms are non-negative, so
//    2^(5t+122) <= sum <= 16 * 2^(5t+122) with t = max_h (u+v) over the 16 steps, whatever the
//    order and rounding of the accumulation, and floor((exponent(sum) - 122) / 5) = t exactly.
//    The running maximum over the chunks of 16 is kept on the raw FP32 bit patterns.  A pair
//    whose result is below -37 (or has no candidate at all) may have lost candidates to the
//    clamping, so its block is computed again the other way.
//  * On the vector ALU with packed int16 add/max over the unencoded tables, one lane instruction per two
//    (i,j) pairs: exact for every span, 8 times slower.
// Both give the exact coarsened ESC; the first covers spans up to 37 bits at matrix-unit speed.
// The last workgroup of the kernel gives the verdict and, in per-block mode, the slice counts of the blocks and the order
// they are dealt in: what were up to four more launches of 4-5 us each, in which one workgroup did something or none.
#include <algorithm>

#include "oz_verdict.h"

namespace oz {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

struct ExponentSide {
    const int16_t* group_max;     // [groups][rows_p]
    int32_t* e;
    const int16_t* tab;           // [H2][rows_p]
    uint4* enc;
    int64_t rows_p;
};

constexpr int kExpRows = 64;      // rows per workgroup, one per lane
constexpr int kExpWaves = 16;

// Between scan and ESC.  e[r]: the largest exponent of a row over the scan's groups of blocks (every workgroup of a row block finds
// it for itself; 16 waves share the groups).  Then the encoded tables, 8 h of a row at a time (groups of 8 wave by wave,
// over gridDim.y workgroups):
//   enc[(h/8) * rows_p + r][h%8] = BF16 bits of 2^(5*(tab[h][r] - e[r]) + 61), or 0
// And the control record is cleared on the way, for the ESC kernel and the slice GEMM.
// Bound by latency (8192^3: 7.6 us, where clearing and encoding took 5 + 8 in launches of their own).
__global__ __launch_bounds__(kExpRows * kExpWaves) void exponents_kernel(ExponentSide a, ExponentSide b, int blocks_a, int groups, int H2,
                                                                         int chunks, Record* rec, int32_t* __restrict__ tile_span,
                                                                         int64_t tiles, KnownRecord known, Batch bt) {
    __shared__ int part[kExpWaves][kExpRows];
    const bool second = int(blockIdx.x) >= blocks_a;
    const int64_t ws = bt.ws_at(blockIdx.z);
    ExponentSide s = second ? b : a;
    s.group_max = at_bytes(s.group_max, ws);
    s.e = at_bytes(s.e, ws);
    s.tab = at_bytes(s.tab, ws);
    s.enc = at_bytes(s.enc, ws);
    rec = at_bytes(rec, ws);
    tile_span = at_bytes(tile_span, ws);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r = int64_t(int(blockIdx.x) - (second ? blocks_a : 0)) * kExpRows + lane;
    int e = kExpAllZero;
#pragma unroll 16
    for (int g = wave; g < groups; g += kExpWaves) e = max(e, int(s.group_max[int64_t(g) * s.rows_p + r]));
    part[wave][lane] = e;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        if (threadIdx.x == 0) {
            rec->span_max = 0;
            rec->esc_done = 0;
            write_known_record(known, bt, int(blockIdx.z));
        }
        if (threadIdx.x < 8) rec->tile_sync[threadIdx.x] = 0;
    }
    for (int64_t t = (int64_t(blockIdx.y) * gridDim.x + blockIdx.x) * (kExpRows * kExpWaves) + threadIdx.x; t < tiles;
         t += int64_t(gridDim.x) * gridDim.y * (kExpRows * kExpWaves))
        tile_span[t] = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kExpWaves; ++w) e = max(e, part[w][lane]);
    if (wave == 0 && blockIdx.y == 0) {
        s.e[r] = e;
        if (e == kExpInfNan) atomicOr(&rec->infnan, 1);      // the scan has cleared it
    }
    for (int hc = int(blockIdx.y) * kExpWaves + wave; hc < chunks; hc += int(gridDim.y) * kExpWaves) {
        int x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = s.tab[int64_t(min(hc * 8 + q, H2 - 1)) * s.rows_p + r];      // all in flight at once
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t bits = hc * 8 + q < H2 ? enc_bits(x[q], e) : 0u;
            w[q >> 1] |= bits << (16 * (q & 1));
        }
        s.enc[int64_t(hc) * s.rows_p + r] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

typedef short short2_t __attribute__((ext_vector_type(2)));
typedef short short8_t __attribute__((ext_vector_type(8)));

constexpr int kEscTile = 128;   // pairs (i,j) per workgroup and direction
constexpr int kEscHChunk = 32;  // inner steps staged in LDS at a time (int16 way)
constexpr short kEscPadValue = -16384;  // two of them add to the int16 minimum without wrapping
static_assert(kTile == 2 * kEscTile, "four ESC blocks per block of C");

struct EscLds {
    union {
        struct { short8_t Ut[kEscHChunk][kEscTile / 8], Vt[kEscHChunk][kEscTile / 8]; } exact;
        struct { int cnt[kMaxSlices + 1][256]; int base[kMaxSlices + 1]; } order;
    };
    uint32_t least[4];
    unsigned long long pairs[4];
    int smin[4];
    int last, stop;
};

// Largest span of a block of 128 x 128 pairs the exact way (16 x 16 threads of 8 x 8 pairs); of all threads.
__device__ __forceinline__ int exact_span(EscLds& lds, const int16_t* __restrict__ U, const int16_t* __restrict__ V,
                                          const int32_t* __restrict__ eA, const int32_t* __restrict__ eB, int64_t mp, int64_t np,
                                          int H2, int64_t i0, int64_t j0) {
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;

    short2_t acc[8][4];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = short2_t{-32768, -32768};

    for (int h0 = 0; h0 < H2; h0 += kEscHChunk) {
        __syncthreads();
        // 32 x 128 int16 per table = 512 vectors of 8; two per thread
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int v = threadIdx.x + t * 256;
            const int hh = v >> 4, col = v & 15;
            short8_t uu, vv;
            if (h0 + hh < H2) {
                uu = *reinterpret_cast<const short8_t*>(U + int64_t(h0 + hh) * mp + i0 + col * 8);
                vv = *reinterpret_cast<const short8_t*>(V + int64_t(h0 + hh) * np + j0 + col * 8);
            } else {
                uu = short8_t(kEscPadValue);
                vv = short8_t(kEscPadValue);
            }
            lds.exact.Ut[hh][col] = uu;
            lds.exact.Vt[hh][col] = vv;
        }
        __syncthreads();
#pragma unroll 4
        for (int hh = 0; hh < kEscHChunk; ++hh) {
            const short8_t u = lds.exact.Ut[hh][ty];
            const short8_t v = lds.exact.Vt[hh][tx];
            const short2_t v2[4] = {short2_t{v[0], v[1]}, short2_t{v[2], v[3]},
                                    short2_t{v[4], v[5]}, short2_t{v[6], v[7]}};
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const short2_t ua = short2_t{u[a], u[a]};
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[a][c] = __builtin_elementwise_max(acc[a][c], ua + v2[c]);
            }
        }
    }

    int best = 0;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const int ea = eA[i0 + ty * 8 + a];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int z = acc[a][c][q];
                const int eb = eB[j0 + tx * 8 + c * 2 + q];
                int span;
                if (z >= kSumRealFloor) span = ea + eb - z;          // a real exponent sum
                else if (z >= kSumDeadBelow) span = kEscCap;          // no candidate: unbounded
                else span = 0;                                        // identically zero product
                best = max(best, span);
            }
        }
    }
    return best;
}

// Per-tile mode: the order in which the tiles of C are dealt to the workgroups.  An XCD runs its tiles in
// rounds of 32 that keep in step to share panels in L2; a round that mixes tiles of different slice counts
// falls out of step when its light tiles finish (their successors wait in vain for the heavy ones and then
// run alone: measured 18.0 ms instead of 13.9 ms for 64 ten-slice tiles lying in one block column).  So the
// tiles are sorted by slice count, heaviest first and otherwise in the usual block order, and the sorted
// groups of 32 are dealt to the XCDs in turn: group g is round g / 8 of XCD g % 8.  Rounds are then uniform
// but for one per slice count, the heavy rounds are spread over the XCDs, and the lightest tiles end up in
// the partial last round or the k-split launch.  `first` = tiles of the first launch (its XCD ranges are what
// the groups are dealt into), of which the leading first / 256 * 256 sorted tiles are dealt; the others keep
// the sorted order in the positions that remain.  order[position] = index of the tile in the block order.
// One workgroup; a stable counting sort over the slice counts 0 .. kMaxSlices.
constexpr int kOrderRound = 32;
__device__ __forceinline__ void tile_order(EscLds& lds, const int32_t* tile_S, int32_t* order, int nti, int ntj, int first, int deal) {
    const int tiles = nti * ntj, tid = threadIdx.x;
    if (!deal) {
        for (int lin = tid; lin < tiles; lin += 256) order[lin] = lin;
        return;
    }
    int (*const cnt)[256] = lds.order.cnt;
    int* const base = lds.order.base;
    const int chunk = (tiles + 255) / 256;
    const int lo = min(tiles, tid * chunk), hi = min(tiles, lo + chunk);
    auto key_of = [&](int lin) -> int {
        int ti, tj;
        lin_to_tile(lin, nti, ntj, ti, tj);
        return min(max(tile_S[tj * nti + ti], 0), kMaxSlices);
    };
    for (int k = 0; k <= kMaxSlices; ++k) cnt[k][tid] = 0;
    for (int lin = lo; lin < hi; ++lin) ++cnt[key_of(lin)][tid];
    __syncthreads();
    if (tid <= kMaxSlices) {      // exclusive prefix over the threads' chunks, per key
        int run = 0;
        for (int t = 0; t < 256; ++t) {
            const int c = cnt[tid][t];
            cnt[tid][t] = run;
            run += c;
        }
        base[tid] = run;
    }
    __syncthreads();
    if (tid == 0) {               // keys in descending order
        int run = 0;
        for (int k = kMaxSlices; k >= 0; --k) {
            const int c = base[k];
            base[k] = run;
            run += c;
        }
    }
    __syncthreads();
    const int per = first >> 3, rem = first & 7, rounds = first / (8 * kOrderRound), dealt = rounds * 8 * kOrderRound;
    for (int lin = lo; lin < hi; ++lin) {
        const int k = key_of(lin);
        const int si = base[k] + cnt[k][tid]++;      // position in the sorted sequence
        int q = si;
        if (si < dealt) {
            const int g = si / kOrderRound, wpos = si % kOrderRound, r = g >> 3, x = g & 7;
            q = x * per + min(x, rem) + r * kOrderRound + wpos;
        } else if (si < first) {
            // what is left of the XCD ranges behind their dealt rounds, XCD by XCD
            int t = si - dealt;
            for (int x = 0; x < 8; ++x) {
                const int left = per + (x < rem ? 1 : 0) - rounds * kOrderRound;
                if (t < left) {
                    q = x * per + min(x, rem) + rounds * kOrderRound + t;
                    break;
                }
                t -= left;
            }
        }
        order[q] = lin;
    }
}

// Smallest of the block's chunk-maximum sums as FP32 bit patterns (0xFFFFFFFF: the block holds padding only); of
// all threads.  4 waves of 64x64 pairs, 2x2 MFMA tiles of 32x32 each.
__device__ __forceinline__ uint32_t least_sum(const uint4* __restrict__ EU, const uint4* __restrict__ EV, int64_t m,
                                              int64_t n, int64_t mp, int64_t np, int steps, int64_t bi, int64_t bj) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 31, lh = lane >> 5;
    const int64_t i0 = bi * kEscTile + (wave & 1) * 64;
    const int64_t j0 = bj * kEscTile + (wave >> 1) * 64;
    const uint4* pa = EU + int64_t(lh) * mp + i0 + lr;
    const uint4* pb = EV + int64_t(lh) * np + j0 + lr;

    uint32_t run[2][2][16];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) run[a][b][r] = 0;

    const f32x16_t zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    // Two chunks per step (the tables are zero-padded to a multiple of 32 inner steps).  The
    // operands of the next step are requested before the current step's arithmetic; the loads are
    // written as asm so that they stay where they are issued, and the explicit wait ties the
    // destination registers to the point where the data has arrived.
    u32x4_t X[8], Y[8];
    int loaded = 0;   // step the pointers address
#define OZ_ESC_ISSUE(buf)                                                                      \
    do {                                                                                       \
        const uint4* pa1_ = pa + 2 * mp;                                                       \
        const uint4* pb1_ = pb + 2 * np;                                                       \
        asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(buf[0]) : "v"(pa));             \
        asm volatile("global_load_dwordx4 %0, %1, off offset:512" : "=&v"(buf[1]) : "v"(pa));  \
        asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(buf[2]) : "v"(pa1_));           \
        asm volatile("global_load_dwordx4 %0, %1, off offset:512" : "=&v"(buf[3]) : "v"(pa1_));\
        asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(buf[4]) : "v"(pb));             \
        asm volatile("global_load_dwordx4 %0, %1, off offset:512" : "=&v"(buf[5]) : "v"(pb));  \
        asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(buf[6]) : "v"(pb1_));           \
        asm volatile("global_load_dwordx4 %0, %1, off offset:512" : "=&v"(buf[7]) : "v"(pb1_));\
        if (loaded + 1 < steps) { pa += 4 * mp; pb += 4 * np; ++loaded; }  /* else: re-read */   \
        __builtin_amdgcn_sched_barrier(0);   /* the arithmetic below must not move above the loads */ \
    } while (0)
#define OZ_ESC_WAIT(buf)                                                                       \
    __builtin_amdgcn_sched_barrier(0);       /* the arithmetic above stays above the wait */   \
    asm volatile("s_waitcnt vmcnt(0)"                                                          \
                 : "+v"(buf[0]), "+v"(buf[1]), "+v"(buf[2]), "+v"(buf[3]), "+v"(buf[4]),       \
                   "+v"(buf[5]), "+v"(buf[6]), "+v"(buf[7]));                                  \
    __builtin_amdgcn_sched_barrier(0)
#define OZ_ESC_COMPUTE(buf)                                                                    \
    _Pragma("unroll") for (int a = 0; a < 2; ++a) _Pragma("unroll") for (int b = 0; b < 2; ++b) { \
        const u32x16_t d0 = __builtin_bit_cast(u32x16_t, __builtin_amdgcn_mfma_f32_32x32x16_bf16( \
            __builtin_bit_cast(bf16x8_t, buf[a]), __builtin_bit_cast(bf16x8_t, buf[4 + b]), zero, 0, 0, 0)); \
        const u32x16_t d1 = __builtin_bit_cast(u32x16_t, __builtin_amdgcn_mfma_f32_32x32x16_bf16( \
            __builtin_bit_cast(bf16x8_t, buf[2 + a]), __builtin_bit_cast(bf16x8_t, buf[6 + b]), zero, 0, 0, 0)); \
        _Pragma("unroll") for (int r = 0; r < 16; ++r) /* sums are >= 0: unsigned order is numeric order */ \
            run[a][b][r] = max(run[a][b][r], max(d0[r], d1[r]));                                \
    }

    OZ_ESC_ISSUE(X);
    for (int c = 0; c < steps; c += 2) {
        OZ_ESC_WAIT(X);
        OZ_ESC_ISSUE(Y);
        OZ_ESC_COMPUTE(X);
        OZ_ESC_WAIT(Y);
        OZ_ESC_ISSUE(X);
        if (c + 1 < steps) { OZ_ESC_COMPUTE(Y); }
    }
    OZ_ESC_WAIT(X);   // nothing may be in flight when the wave ends
#undef OZ_ESC_ISSUE
#undef OZ_ESC_WAIT
#undef OZ_ESC_COMPUTE

    // The span of a pair decreases with its sum, so the largest span of the tile belongs to the
    // smallest sum: reduce the raw bit patterns first, convert once.
    uint32_t least = 0xFFFFFFFFu;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t i = i0 + a * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                const int64_t j = j0 + b * 32 + lr;
                if (i < m && j < n) least = min(least, run[a][b][r]);
            }
    return least;
}

// A workgroup takes every gridDim.x-th block of 128 x 128 pairs: few enough workgroups (two per CU) that their arrivals
// at one counter do not queue up (17 ns each: one per block took 70 us at 8192^3).
__global__ __launch_bounds__(256) void esc_kernel(const uint4* __restrict__ EU, const uint4* __restrict__ EV,
                                                  const int16_t* __restrict__ U, const int16_t* __restrict__ V,
                                                  const int32_t* __restrict__ eA, const int32_t* __restrict__ eB, int64_t m,
                                                  int64_t n, int64_t k, int64_t mp, int64_t np, int H2, int steps, Record* rec,
                                                  int32_t* __restrict__ tile_span, VerdictArgs v, Batch bt) {
    __shared__ EscLds lds;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    {
        const int64_t ws = bt.ws_at(blockIdx.z);
        EU = at_bytes(EU, ws); EV = at_bytes(EV, ws);
        U = at_bytes(U, ws); V = at_bytes(V, ws);
        eA = at_bytes(eA, ws); eB = at_bytes(eB, ws);
        rec = at_bytes(rec, ws);
        tile_span = at_bytes(tile_span, ws);
        v.tile_S = at_bytes(v.tile_S, ws);
    }
    const int infnan = any_infnan(rec, v.infnan_parts);
    if (infnan) {
        // the native path is decided: one workgroup says so, no span is needed
        if (blockIdx.x != 0) return;
    } else {
        const int64_t nbi = mp / kEscTile, blocks = nbi * (np / kEscTile);
        int widest = 0;
        for (int64_t block = blockIdx.x; block < blocks; block += gridDim.x) {
            int64_t bi, bj;
            esc_block_at(block, nbi, np / kEscTile, gridDim.x, bi, bj);
            uint32_t least = least_sum(EU, EV, m, n, mp, np, steps, bi, bj);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) least = min(least, uint32_t(__shfl_xor(int(least), off)));
            __syncthreads();
            if (lane == 0) lds.least[wave] = least;
            __syncthreads();
            least = min(min(lds.least[0], lds.least[1]), min(lds.least[2], lds.least[3]));
            if (least == 0xFFFFFFFFu) continue;              // padding only
            // exponent(sum) - 122 lies in [5t, 5t+4]; shifted by 5*64 so that the division is of a
            // non-negative number
            const int E = int(least >> 23) - 127 - 2 * kEncBias;
            const int t = (E + kEncScale * 64) / kEncScale - 64;
            int span = -t;
            if (t < -kEncRange) {
                // below the encodable range, or no candidate at all: this block once more, the exact way
                int best = exact_span(lds, U, V, eA, eB, mp, np, H2, bi * kEscTile, bj * kEscTile);
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) best = max(best, __shfl_xor(best, off));
                __syncthreads();
                if (lane == 0) lds.least[wave] = uint32_t(best);
                __syncthreads();
                span = max(max(int(lds.least[0]), int(lds.least[1])), max(int(lds.least[2]), int(lds.least[3])));
            }
            widest = max(widest, span);
            // the block's largest span goes to the C block it lies in (four such blocks per kTile x kTile block)
            if (v.tile_mode && threadIdx.x == 0) atomicMax(&tile_span[(bj >> 1) * (mp / kTile) + (bi >> 1)], span);
        }
        // the last workgroup to get here has everybody's spans before it
        if (threadIdx.x == 0) {
            // a stale read only costs a redundant atomic, the maximum is monotone
            if (widest > *reinterpret_cast<volatile int32_t*>(&rec->span_max)) atomicMax(&rec->span_max, widest);
            // The spans are atomics of this thread, carried out where all XCDs see them: once they are done, so is this
            // workgroup.  No fence: an agent-scope release writes the XCD's L2 back (150 us with one per block).
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds.last = __hip_atomic_fetch_add(&rec->esc_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == int(gridDim.x) - 1;
        }
        __syncthreads();
        if (!lds.last) return;
    }

    // ---- one workgroup from here on ----
    auto read = [](const int32_t* p) -> int { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    unsigned long long pairs = 0;
    int smin = kMaxSlices;
    if (v.tile_mode) {
        // slice count of every kTile x kTile block of C from the largest span inside it
        for (int64_t t = threadIdx.x; t < int64_t(v.nti) * v.ntj; t += 256) {
            const int S = span_slices(v.o, read(&tile_span[t]));
            v.tile_S[t] = S;
            pairs += (unsigned long long)(S) * (S + 1) / 2;
            smin = min(smin, S);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            pairs += __shfl_xor(pairs, off);
            smin = min(smin, __shfl_xor(smin, off));
        }
        if (lane == 0) { lds.pairs[wave] = pairs; lds.smin[wave] = smin; }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (v.tile_mode) {
            pairs = lds.pairs[0] + lds.pairs[1] + lds.pairs[2] + lds.pairs[3];
            smin = min(min(lds.smin[0], lds.smin[1]), min(lds.smin[2], lds.smin[3]));
        }
        const oz_result_t r = verdict(v, infnan, read(&rec->span_max), pairs, smin, m, n, k);
        rec->res = r;
        if (v.user) v.user[blockIdx.z] = r;
        lds.stop = r.fallback;
    }
    __threadfence_block();
    __syncthreads();
    if (!v.tile_mode || lds.stop) return;
    tile_order(lds, v.tile_S, v.tile_S + v.nti * v.ntj, v.nti, v.ntj, v.first, v.deal);
}

__global__ void known_record_kernel(KnownRecord known) {
    if (threadIdx.x == 0) write_known_record(known, Batch{}, 0);
}

oz_result_t known_verdict(const Problem& p, const oz_opts_t& o, int kind) {
    oz_result_t r = {};
    r.esc = -1;
    if (kind == 2) return r;
    if (kind == 3) {
        r.fallback = 1;
        r.reason = 3;
    } else if (o.mode == OZ_NATIVE) {
        r.fallback = 1;
        r.reason = 4;
    } else {
        r.slices_used = r.slices_min = fixed_slices(o);
        r.pair_tiles = ((p.m + kTile - 1) / kTile) * ((p.n + kTile - 1) / kTile) * (int64_t(r.slices_used) * (r.slices_used + 1) / 2);
    }
    return r;
}

void launch_known_record(hipStream_t st, const KnownRecord& known) {
    hipLaunchKernelGGL(known_record_kernel, dim3(1), dim3(64), 0, st, known);
}

void launch_exponents(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, bool encode,
                      const KnownRecord& known) {
    const ScanGrid g = scan_grid(p, a.stride_r == 1, b.stride_r == 1);
    const int H2 = 2 * p.G;
    const int chunks = encode ? (H2 + 2 * kEncChunk - 1) / (2 * kEncChunk) * 4 : 0;
    const int blocks_a = int(p.mp / kExpRows), blocks = int((p.mp + p.np) / kExpRows);
    // several workgroups per row block while the CUs are not filled and each still has a chunk for every wave
    const int y = std::max(1, std::min((p.num_cu + blocks * p.batch.count - 1) / (blocks * p.batch.count), chunks / kExpWaves));
    const ExponentSide sa{w.group_max_a(), w.eA, w.U, reinterpret_cast<uint4*>(w.EU), p.mp};
    const ExponentSide sb{w.group_max_b(), w.eB, w.V, reinterpret_cast<uint4*>(w.EV), p.np};
    hipLaunchKernelGGL(exponents_kernel, dim3(unsigned(blocks), unsigned(y), unsigned(p.batch.count)), dim3(kExpRows * kExpWaves), 0, st, sa, sb, blocks_a,
                       int(g.groups), H2, chunks, w.rec, w.tile_span, (p.mp / kTile) * (p.np / kTile), known, p.batch);
}

void launch_esc_verdict(hipStream_t st, const Workspace& w, const Problem& p, const oz_opts_t& o, const oz_heuristic_t& hm,
                        oz_result_t* user_result) {
    const int H2 = 2 * p.G;
    const int steps = (H2 + 2 * kEncChunk - 1) / (2 * kEncChunk);   // 32 inner steps (4 groups of 8) each
    uint4* const EU = reinterpret_cast<uint4*>(w.EU);
    uint4* const EV = reinterpret_cast<uint4*>(w.EV);
    const VerdictArgs v = verdict_args(w, p, o, hm, user_result);
    const int64_t blocks = (p.mp / kEscTile) * (p.np / kEscTile);
    hipLaunchKernelGGL(esc_kernel, dim3(unsigned(std::min<int64_t>(blocks, std::max(1, 2 * p.num_cu / p.batch.count))), 1, unsigned(p.batch.count)), dim3(256), 0, st, EU, EV, w.U,
                       w.V, w.eA, w.eB, p.m, p.n, p.k, p.mp, p.np, H2, steps, w.rec, w.tile_span, v, p.batch);
}

}  // namespace oz
