// Pre-pass over op(A) and op(B): Inf/NaN scan, per-block exponent Max/Min tables for the
// coarsened ESC, and what the row / column exponents the slicing aligns to are made of: the largest exponent of each row
// in every group of blocks a workgroup takes (exponents_kernel finishes them; with atomics on the exponents themselves, a
// launch of its own had to clear them and the control record first: 4.8 us a call).
// (paper: sections "Pre-processing and Safety Checks" and "Exponent Span Estimation";
//  block Max/Min: section "ESC", the paragraph on blocks of length b.)
//
// HBM-bound: every FP64 element is read once (8 B), two int16 are written per block of b.  Scan and exponents at 8192^3 (1.07 GB) 178 us
// with both operands' rows contiguous, 198 with k contiguous (231 and 276 with 128 bytes of a row per load there and without the streaming
// hint; a read of 1 GiB with the hint takes 154).
#include "oz_internal.h"

namespace oz {

// Exponents (floor(log2|x|)) of the entries that one thread has seen of a block, a batch of loaded entries at a time.  Kept on
// the high words: the exponent field grows with the magnitude, so the largest and smallest word have the largest and
// smallest exponent, and Inf and NaN come out as kExpInfNan.  Five instructions per entry and no branch, so the loads of a
// batch are all in flight before the first is looked at; zeros and denormals, whose exponent lies elsewhere, are looked
// for only in a batch that has one.  (Entry by entry, with branches for zeros, loads were waited for one by one: 200 x 300 x 260
// 5.3 us, then 3.6; 1024 x 1024 x 65536 219, then 196; 8192^3 254, then 238.)
struct BlockStat {
    uint32_t mx, mn;       // largest high word (without sign), smallest of the normal numbers less kMinNormal
    int mx_low, mn_low;    // exponents of the denormals: -32768 and 32767: none
    int any_zero;
    static constexpr uint32_t kMinNormal = 0x00100000u;
    __device__ __forceinline__ void reset() { mx = 0; mn = ~0u; mx_low = -32768; mn_low = 32767; any_zero = 0; }
    template <int N>
    __device__ __forceinline__ void add(const uint64_t (&x)[N]) {
        uint32_t least = ~0u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t hi = uint32_t(x[i] >> 32) & 0x7FFFFFFFu;
            mx = max(mx, hi);
            mn = min(mn, hi - kMinNormal);       // a word below kMinNormal wraps to more than any other
            least = min(least, hi);
        }
        if (least < kMinNormal) {
#pragma unroll 1
            for (int i = 0; i < N; ++i) {
                uint64_t mag = 0;
#pragma unroll
                for (int q = 0; q < N; ++q) mag = q == i ? x[q] & 0x7FFFFFFFFFFFFFFFull : mag;
                if (mag == 0) {
                    any_zero = 1;
                } else if (uint32_t(mag >> 32) < kMinNormal) {
                    const int e = (63 - __builtin_clzll(mag)) - 1074;
                    mx_low = max(mx_low, e);
                    mn_low = min(mn_low, e);
                }
            }
        }
    }
    // largest and smallest exponent of the non-zero entries; -32768 and 32767: none
    __device__ __forceinline__ int max_exp() const { return mx >= kMinNormal ? int(mx >> 20) - 1023 : mx_low; }
    __device__ __forceinline__ int min_exp() const { return min(mn_low, mn < 0x80000000u ? int((mn + kMinNormal) >> 20) - 1023 : 32767); }
};

__device__ __forceinline__ int table_max(int mx) { return mx == -32768 ? kExpAllZero : mx; }
__device__ __forceinline__ int table_min(int mx, int mn, int any_zero) {
    return mx == -32768 ? kExpAllZero : (any_zero ? kExpZeroInMin : mn);
}

struct ScanSide {
    Operand o;
    int16_t* tab;          // [2G][rows_p]
    int max_half;          // 1: Max in the first half of the table, Min in the second; 0: the other way round
    int16_t* group_max;    // [groups][rows_p] largest exponent of a row in a group of blocks
    int64_t row_blocks;    // workgroups along the rows
};

__device__ __forceinline__ void scan_store(const ScanSide& s, int G, int g, int64_t r, int mx, int mn) {
    s.tab[int64_t(s.max_half ? g : G + g) * s.o.rows_p + r] = int16_t(mx);
    s.tab[int64_t(s.max_half ? G + g : g) * s.o.rows_p + r] = int16_t(mn);
}

// NT: with the streaming hint (launch_scan)
template <bool NT>
__device__ __forceinline__ uint64_t load_entry(const uint64_t* p) {
    return NT ? __builtin_nontemporal_load(p) : *p;
}

// Rows contiguous in memory (stride_r == 1): lanes along 64 rows, so every load instruction of a wave reads 512
// contiguous bytes; the four waves take every fourth k of a block, which keeps a thread's chain of loads short (a
// thread per row for four whole blocks: 28 us for 2048 x 2048, now 10), and are combined through LDS.
template <bool NT>
__device__ __forceinline__ void scan_rows(const ScanSide& s, int64_t rb, int g0, int per, int64_t k, int b, int G) {
    __shared__ int2 part[kScanBlocksPerWg][4][64];     // max; min, with bit 16 set when the part holds a zero
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);        // addresses are scalar but for the lane
    const int64_t r = rb * 64 + lane;
#pragma unroll 1
    for (int u = 0; u < per; ++u) {
        const int g = g0 + u;
        BlockStat st;
        st.reset();
        if (g < G && r < s.o.rows) {
            // past the end of a block its last entry is read again: it changes neither maximum nor minimum
            const int64_t l0 = int64_t(g) * b;
            const int len = int(min(int64_t(b), k - l0));
            const uint64_t* src = reinterpret_cast<const uint64_t*>(s.o.X) + rb * 64 + l0 * s.o.stride_l;
            for (int l = wave; l < len; l += 64) {
                uint64_t x[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = load_entry<NT>(src + min(l + 4 * i, len - 1) * s.o.stride_l + lane);
                st.add(x);
            }
        }
        part[u][wave][lane] = make_int2(st.max_exp(), (st.min_exp() & 0xFFFF) | (st.any_zero << 16));
    }
    __syncthreads();
    // wave u finishes block g0 + u
    const bool mine = wave < per && g0 + wave < G;
    int mx = -32768, mn = 32767, any_zero = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int2 x = part[mine ? wave : 0][w][lane];
        mx = max(mx, x.x);
        mn = min(mn, int(int16_t(x.y & 0xFFFF)));
        any_zero |= x.y >> 16;
    }
    if (mine) scan_store(s, G, g0 + wave, r, table_max(mx), table_min(mx, mn, any_zero));
    __syncthreads();
    int* const row_max = reinterpret_cast<int*>(part);
    row_max[wave * 64 + lane] = mine ? table_max(mx) : kExpAllZero;
    __syncthreads();
    if (wave == 0) {
        const int e = max(max(row_max[lane], row_max[64 + lane]), max(row_max[128 + lane], row_max[192 + lane]));
        s.group_max[int64_t(g0 / per) * s.o.rows_p + r] = int16_t(e);
    }
}

// k contiguous in memory (stride_l == 1): 16 lanes share one row so that a load instruction
// reads 128 contiguous bytes per row; partial results are combined across the 16 lanes.
// A workgroup covers 16 rows.  For calls that do not take scan_k64 below (scan_grid).  The loads of two blocks are in flight together (of
// four: 77 registers, and six workgroups to a CU instead of eight: 4224 x 3008 x 1792 32 us against 25).
template <int PER>
__device__ __forceinline__ void scan_k(const ScanSide& s, int64_t rb, int g0, int64_t k, int b, int G) {
    constexpr int PAIR = PER < 2 ? PER : 2;
    const int q = threadIdx.x & 15;
    const int64_t r = rb * 16 + (threadIdx.x >> 4);
    const uint64_t* const row = reinterpret_cast<const uint64_t*>(s.o.X) + r * s.o.stride_r;
    int row_max = kExpAllZero;
#pragma unroll 1
    for (int g = g0; g < min(g0 + PER, G); g += PAIR) {
        BlockStat st[PAIR];
#pragma unroll
        for (int u = 0; u < PAIR; ++u) st[u].reset();
        if (r < s.o.rows) {
            for (int l = q; l < b; l += 64) {
                uint64_t x[PAIR][4];
#pragma unroll
                for (int u = 0; u < PAIR; ++u) {
                    // past the end of a block its last entry is read again, past the last block that block
                    const int64_t l0 = int64_t(min(g + u, G - 1)) * b;
                    const int len = int(min(int64_t(b), k - l0));
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[u][i] = (row + l0)[min(l + 16 * i, len - 1)];
                }
#pragma unroll
                for (int u = 0; u < PAIR; ++u) st[u].add(x[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < PAIR; ++u) {
            int mx = st[u].max_exp(), mn = st[u].min_exp(), any_zero = st[u].any_zero;
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) {
                mx = max(mx, __shfl_xor(mx, off));
                mn = min(mn, __shfl_xor(mn, off));
                any_zero |= __shfl_xor(any_zero, off);
            }
            if (q == 0 && g + u < G) {
                scan_store(s, G, g + u, r, table_max(mx), table_min(mx, mn, any_zero));
                row_max = max(row_max, table_max(mx));
            }
        }
    }
    if (q == 0) s.group_max[int64_t(g0 / PER) * s.o.rows_p + r] = int16_t(row_max);
}

// Blocks that are whole 64s of k: a load instruction of a wave reads 64 entries of one row, 512 contiguous bytes as in scan_rows,
// with 16 rows in flight; the rows' partial results, one per lane, then fold into each other across the lanes.  A wave covers 16
// rows, a workgroup 64.
// A code of 16 bits stands for an entry: the top 16 bits of its magnitude (exponent field and four bits of the significand) plus
// kLowCodes, the exponent of a denormal + 1075 (1 .. 52), 0 for a zero.  A word holds the largest code of a row and, in its high
// half, the inverse of the smallest, so that one packed maximum takes both.
constexpr uint32_t kLowCodes = 64;
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
template <int CTRL>
__device__ __forceinline__ uint32_t pk_max_dpp(uint32_t x) {
    return pk_max(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), CTRL, 0xF, 0xF, false)));
}
__device__ __forceinline__ int code_exp(uint32_t code) {     // of a non-zero entry
    return code >= kLowCodes ? int((code - kLowCodes) >> 4) - 1023 : int(code) - 1075;
}
// codes of 16 entries into 16 words
__device__ __forceinline__ void add_codes(const uint64_t (&x)[16], uint32_t (&stat)[16]) {
    uint32_t least = ~0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) least = min(least, uint32_t(x[i] >> 32) << 1);
    if (!__any(least < 2 * BlockStat::kMinNormal)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t hi = uint32_t(x[i] >> 32);
            const u16x2 top = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(hi, hi, 0x07060706u) & 0x7FFF7FFFu);
            stat[i] = pk_max(stat[i], __builtin_bit_cast(uint32_t, top * u16x2{1, 0xFFFF} + u16x2{kLowCodes, 0xFFFF - kLowCodes}));
        }
    } else {                             // a zero or a denormal among them
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            uint32_t hi = uint32_t(x[i] >> 32);
            asm volatile("" : "+v"(hi));             // one entry at a time: registers
            hi &= 0x7FFFFFFFu;
            const uint32_t lo = uint32_t(x[i]);
            const uint32_t low = hi ? 64 - __builtin_clz(hi) : (lo ? 32 - __builtin_clz(lo) : 0u);
            const uint32_t code = hi >= BlockStat::kMinNormal ? (hi >> 16) + kLowCodes : low;
            stat[i] = pk_max(stat[i], code | ((0xFFFFu - code) << 16));
        }
    }
}
// 16 words of 64 lanes, a row each, to one word per row: row 4 (lane / 16) + lane % 4
__device__ __forceinline__ uint32_t fold_rows(uint32_t (&stat)[16], int lane) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const auto p = __builtin_amdgcn_permlane32_swap(stat[i], stat[i + 8], false, false);
        stat[i] = pk_max(p[0], p[1]);                      // lanes 0 .. 31 row i, 32 .. 63 row i + 8
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto p = __builtin_amdgcn_permlane16_swap(stat[i], stat[i + 4], false, false);
        uint32_t x = pk_max(p[0], p[1]);                   // rows i, i + 4, i + 8, i + 12, in 16 lanes each
        x = pk_max_dpp<0x128>(x);                          // row_ror 8, 4, 2, 1
        x = pk_max_dpp<0x124>(x);
        x = pk_max_dpp<0x122>(x);
        stat[i] = pk_max_dpp<0x121>(x);
    }
    const uint32_t low = (lane & 1) ? stat[1] : stat[0], high = (lane & 1) ? stat[3] : stat[2];
    return (lane & 2) ? high : low;
}
template <bool NT>
__device__ __forceinline__ void scan_k64(const ScanSide& s, int64_t rb, int g0, int per, int64_t k, int b, int G) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r0 = rb * 64 + wave * 16;
    const char* const base = reinterpret_cast<const char*>(s.o.X + r0 * s.o.stride_r);
    const int64_t row_bytes = s.o.stride_r * 8;
    const int last_row = int(max(min(int64_t(15), s.o.rows - 1 - r0), int64_t(-1)));     // -1: padding only
    const int my_row = (lane >> 4) * 4 + (lane & 3);         // the row whose results this lane holds in the end
    uint32_t row_max = 0;
#pragma unroll 1
    for (int g = g0; g < min(g0 + per, G); ++g) {
        uint32_t stat[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) stat[i] = 0;
        const int64_t l0 = int64_t(g) * b;
        const int len = last_row < 0 ? 0 : int(min(int64_t(b), k - l0));
#pragma unroll 1
        for (int l = 0; l < len; l += 64) {
            // past the end of a block its last entry is read again, past the last row that row
            const uint32_t at = uint32_t(min(l + lane, len - 1)) * 8u;
            const char* row = base + l0 * 8;
            uint64_t x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                x[i] = load_entry<NT>(reinterpret_cast<const uint64_t*>(row + at));
                row += i < last_row ? row_bytes : 0;
            }
            add_codes(x, stat);
        }
        const uint32_t mine = fold_rows(stat, lane);
        const uint32_t largest = my_row <= last_row ? mine & 0xFFFFu : 0u, smallest = 0xFFFFu - (mine >> 16);
        if ((lane & 12) == 0)
            scan_store(s, G, g, r0 + my_row, largest ? code_exp(largest) : kExpAllZero,
                       largest ? (smallest ? code_exp(smallest) : kExpZeroInMin) : kExpAllZero);
        row_max = max(row_max, largest);
    }
    if ((lane & 12) == 0) s.group_max[int64_t(g0 / per) * s.o.rows_p + r0 + my_row] = int16_t(row_max ? code_exp(row_max) : kExpAllZero);
}

// Both operands in one launch: the first blocks_a workgroups scan op(A), the others op(B), from ESC block g_first on.
// K64: some operand takes scan_k64, which needs 78 registers for its 16 rows in flight, six workgroups to a CU; calls without such an operand
// have a kernel of 52 registers and eight to a CU (one kernel of 78 for all: ESC blocks of 16, 4096^3 with k contiguous 132 us, now 122, 2048^3 38,
// now 35; scan_k64 with 63 registers, each 64 of k folded by itself: ESC blocks of 256, 4096^3 72 and then 77).
template <bool NT, bool K64>
__global__ __launch_bounds__(256, K64 ? 6 : 8) void scan_kernel(ScanSide a, ScanSide b, int64_t blocks_a, int g_first, int per, int64_t k,
                                                   int bl, int G, Record* rec, Batch bt) {
    const int64_t ws = bt.ws_at(blockIdx.z);
    if (blockIdx.x == 0 && threadIdx.x == 0) at_bytes(rec, ws)->infnan = 0;        // the exponents tell (exponents_kernel)
    const bool second = int64_t(blockIdx.x) >= blocks_a;
    ScanSide s = second ? b : a;
    s.o.X += second ? bt.b_at(blockIdx.z) : bt.a_at(blockIdx.z);
    s.tab = at_bytes(s.tab, ws);
    s.group_max = at_bytes(s.group_max, ws);
    const int64_t id = int64_t(blockIdx.x) - (second ? blocks_a : 0);
    const int64_t rb = id % s.row_blocks;
    const int g0 = g_first + int(id / s.row_blocks) * per;
    if (s.o.stride_r == 1) scan_rows<NT>(s, rb, g0, per, k, bl, G);
    else if constexpr (K64) scan_k64<NT>(s, rb, g0, per, k, bl, G);
    else if (per == 1) scan_k<1>(s, rb, g0, k, bl, G);
    else scan_k<kScanBlocksPerWg>(s, rb, g0, k, bl, G);
}

constexpr double kStreamBytes = 400e6;

void launch_scan(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p) {
    const ScanGrid g = scan_grid(p, a.stride_r == 1, b.stride_r == 1);
    const ScanSide sa{a, w.U, 1, w.group_max_a(), g.row_blocks_a}, sb{b, w.V, 0, w.group_max_b(), g.row_blocks_b};
    // The streaming hint keeps the operands out of the 256 MB Infinity Cache.  What fits there the slicing reads from it; of more it finds
    // little, and the scan is the faster for it (scan and slicing, seven slices: 8192 x 8192 twice, 1.07 GB, 586 -> 543 us with rows
    // contiguous, 679 -> 629 with k; 4096 x 4096 twice, 268 MB, 171 -> 185)
    const bool stream = (double(p.m) + double(p.n)) * double(p.k) * 8.0 * p.batch.count > kStreamBytes;
    const auto kernel = stream ? (g.k64 ? scan_kernel<true, true> : scan_kernel<true, false>) : (g.k64 ? scan_kernel<false, true> : scan_kernel<false, false>);
    for (int64_t y = 0; y < g.groups; y += g.slab) {
        const int64_t gy = g.groups - y < g.slab ? g.groups - y : g.slab;
        hipLaunchKernelGGL(kernel, dim3(unsigned((g.row_blocks_a + g.row_blocks_b) * gy), 1, unsigned(p.batch.count)), dim3(256), 0, st, sa, sb,
                           g.row_blocks_a * gy, int(y) * g.per, g.per, p.k, p.esc_block, p.G, w.rec, p.batch);
    }
}

// ---- scan and exponents of a small call in one launch --------------------------------------
// A workgroup of 8 waves takes 16 rows and all of k.  Pieces of 64 k of a block, 16 loads a lane, go to the waves in turn and meet, as
// codes, in LDS; then row exponents, tables, and their encoding.  What a small call waits for is the chain of its launches, and
// this is one less.  16 rows, so that as many CUs read as there are: with 64 a call of 512 x 512 x 1024 had 16 workgroups and took
// 5 us more than in two launches.
constexpr int kOnceWaves = 8;
static_assert(kOnceRows == 16, "four groups of 16 lanes");

struct ScanOnceSide {
    ScanSide s;
    int32_t* e;
    uint4* enc;
};

__global__ __launch_bounds__(64 * kOnceWaves) void scan_exponents_kernel(ScanOnceSide a, ScanOnceSide b, int blocks_a, int64_t k, int bl, int G,
                                                                         int chunks, Record* rec, int32_t* __restrict__ tile_span, int64_t tiles,
                                                                         KnownRecord known, Batch bt) {
    __shared__ uint32_t most[kScanOnceBlocks][kOnceRows], least[kScanOnceBlocks][kOnceRows];       // largest and smallest code
    const bool second = int(blockIdx.x) >= blocks_a;
    const int64_t ws = bt.ws_at(blockIdx.z);
    ScanOnceSide t = second ? b : a;
    const Operand o = t.s.o;
    const double* const X = o.X + (second ? bt.b_at(blockIdx.z) : bt.a_at(blockIdx.z));
    rec = at_bytes(rec, ws);
    tile_span = at_bytes(tile_span, ws);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = threadIdx.x & (kOnceRows - 1), place = threadIdx.x / kOnceRows;          // what a thread finishes
    constexpr int kPlaces = 64 * kOnceWaves / kOnceRows;
    const int64_t r0 = int64_t(int(blockIdx.x) - (second ? blocks_a : 0)) * kOnceRows;
    for (int g = place; g < G; g += kPlaces) {
        most[g][row] = 0;
        least[g][row] = 0xFFFFu;
    }
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            rec->span_max = 0;
            rec->esc_done = 0;
            write_known_record(known, bt, int(blockIdx.z));
        }
        if (threadIdx.x < 8) rec->tile_sync[threadIdx.x] = 0;
        for (int64_t x = threadIdx.x; x < tiles; x += 64 * kOnceWaves) tile_span[x] = 0;
    }
    __syncthreads();
    const int last_row = int(max(min(int64_t(kOnceRows), o.rows - r0), int64_t(0))) - 1;     // -1: padding only
    const int per_block = (bl + 63) / 64, pieces = last_row < 0 ? 0 : G * per_block;
    for (int piece = wave; piece < pieces; piece += kOnceWaves) {
        const int g = piece / per_block, l = (piece - g * per_block) * 64;
        const int64_t l0 = int64_t(g) * bl;
        const int len = int(min(int64_t(bl), k - l0));
        if (l >= len) continue;
        // past the end of a block its last entry is read again, past the last row that row
        uint64_t x[16];
        uint32_t stat[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) stat[i] = 0;
        uint32_t mine;
        int my_row;
        bool holds;
        if (o.stride_r == 1) {           // a load: 16 rows of four k
            const uint32_t at = uint32_t(min(lane & 15, last_row)) * 8u;
            const char* const src = reinterpret_cast<const char*>(X + r0 + l0 * o.stride_l);
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = *reinterpret_cast<const uint64_t*>(src + min(l + 4 * i + (lane >> 4), len - 1) * o.stride_l * 8 + at);
            add_codes(x, stat);
#pragma unroll
            for (int i = 1; i < 16; ++i) stat[0] = pk_max(stat[0], stat[i]);
            mine = stat[0];
            my_row = lane & 15;
            holds = true;
        } else {                         // a load: 64 k of a row
            const uint32_t at = uint32_t(min(l + lane, len - 1)) * 8u;
            const char* const src = reinterpret_cast<const char*>(X + r0 * o.stride_r + l0);
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = *reinterpret_cast<const uint64_t*>(src + min(i, last_row) * o.stride_r * 8 + at);
            add_codes(x, stat);
            mine = fold_rows(stat, lane);
            my_row = (lane >> 4) * 4 + (lane & 3);
            holds = (lane & 12) == 0;
        }
        if (holds && my_row <= last_row) {
            atomicMax(&most[g][my_row], mine & 0xFFFFu);
            atomicMin(&least[g][my_row], 0xFFFFu - (mine >> 16));
        }
    }
    __syncthreads();
    auto table = [&](bool largest, int g) -> int {
        const uint32_t hi = most[g][row], lo = least[g][row];
        if (hi == 0) return kExpAllZero;
        return largest ? code_exp(hi) : (lo ? code_exp(lo) : kExpZeroInMin);
    };
    uint32_t top = 0;
    for (int g = 0; g < G; ++g) top = max(top, most[g][row]);
    const int e = top ? code_exp(top) : kExpAllZero;
    if (wave == 0) {
        if (place == 0) at_bytes(t.e, ws)[r0 + row] = e;
        const bool bad = __any(e == kExpInfNan);
        if (lane == 0) rec->infnan_part[blockIdx.x] = bad ? 1 : 0;
    }
    if (chunks == 0) return;                                 // no guards: nobody reads the tables
    int16_t* const tab = at_bytes(t.s.tab, ws);
    for (int h = place; h < 2 * G; h += kPlaces) {
        const bool half = h >= G;
        tab[int64_t(h) * o.rows_p + r0 + row] = int16_t(table(half != bool(t.s.max_half), half ? h - G : h));
    }
    uint4* const enc = at_bytes(t.enc, ws);
    for (int hc = place; hc < chunks; hc += kPlaces) {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int h = hc * 8 + q;
            if (h < 2 * G) {
                const bool half = h >= G;
                w[q >> 1] |= enc_bits(table(half != bool(t.s.max_half), half ? h - G : h), e) << (16 * (q & 1));
            }
        }
        enc[int64_t(hc) * o.rows_p + r0 + row] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

void launch_scan_exponents(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, bool encode,
                           const KnownRecord& known) {
    const int chunks = encode ? (2 * p.G + 2 * kEncChunk - 1) / (2 * kEncChunk) * 4 : 0;
    const int blocks_a = int(p.mp / kOnceRows), blocks = int((p.mp + p.np) / kOnceRows);
    const ScanOnceSide sa{ScanSide{a, w.U, 1, nullptr, blocks_a}, w.eA, reinterpret_cast<uint4*>(w.EU)};
    const ScanOnceSide sb{ScanSide{b, w.V, 0, nullptr, blocks - blocks_a}, w.eB, reinterpret_cast<uint4*>(w.EV)};
    hipLaunchKernelGGL(scan_exponents_kernel, dim3(unsigned(blocks), 1, unsigned(p.batch.count)), dim3(64 * kOnceWaves), 0, st, sa, sb, blocks_a, p.k,
                       p.esc_block, p.G, chunks, w.rec, w.tile_span, (p.mp / kTile) * (p.np / kTile), known, p.batch);
}

}  // namespace oz
