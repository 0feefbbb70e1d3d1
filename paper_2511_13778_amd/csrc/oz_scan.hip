// Pre-pass over op(A) and op(B): Inf/NaN scan, per-block exponent Max/Min tables for the
// coarsened ESC, and the row / column exponents the slicing aligns to (integer atomicMax over the
// block maxima: order-free, hence deterministic).
// (paper: sections "Pre-processing and Safety Checks" and "Exponent Span Estimation";
//  block Max/Min: section "ESC", the paragraph on blocks of length b.)
//
// HBM-bound: every FP64 element is read once (8 B), two int16 are written per block of b.
#include "oz_internal.h"

namespace oz {

// exp(x) = floor(log2|x|) from the bit pattern; zero -> is_zero; all-ones field -> bad.
__device__ __forceinline__ int exponent_of(uint64_t bits, bool& is_zero, bool& bad) {
    const uint64_t mag = bits & 0x7FFFFFFFFFFFFFFFull;
    const int field = int(mag >> 52);
    is_zero = (mag == 0);
    bad = (field == 0x7FF);
    if (field != 0) return field - 1023;
    // denormal: value = frac * 2^-1074, exponent = position of the leading one - 1074
    return is_zero ? 0 : (63 - __builtin_clzll(mag)) - 1074;
}

struct BlockStat {
    int mx;        // max exponent over non-zero entries
    int mn;        // min exponent over non-zero entries
    int any_nz;    // block has a non-zero entry
    int any_zero;  // block has a zero entry
    __device__ __forceinline__ void reset() { mx = -32768; mn = 32767; any_nz = 0; any_zero = 0; }
    __device__ __forceinline__ void add(uint64_t bits, int& bad_acc) {
        bool z, bad;
        const int e = exponent_of(bits, z, bad);
        bad_acc |= int(bad);
        if (z) { any_zero = 1; } else { any_nz = 1; mx = max(mx, e); mn = min(mn, e); }
    }
    __device__ __forceinline__ int16_t table_max() const { return int16_t(any_nz ? mx : kExpAllZero); }
    __device__ __forceinline__ int16_t table_min() const {
        return int16_t(!any_nz ? kExpAllZero : (any_zero ? kExpZeroInMin : mn));
    }
};

// resets the control record and the row / column exponents (targets of atomicMax in the scans)
__global__ __launch_bounds__(256) void init_kernel(Record* rec, int32_t* eA, int64_t mp, int32_t* eB, int64_t np,
                                                   int32_t* tile_span, int64_t tiles, KnownRecord known) {
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (t == 0) {
        rec->infnan = 0;
        rec->span_max = 0;
        rec->esc_done = 0;
        write_known_record(known);
    }
    if (t < tiles) tile_span[t] = 0;
    if (t < 8) {
        rec->tile_sync[t] = 0;
    }
    if (t < mp) eA[t] = kExpAllZero;
    if (t < np) eB[t] = kExpAllZero;
}

struct ScanSide {
    Operand o;
    int16_t* tab;          // [2G][rows_p]
    int max_half;          // 1: Max in the first half of the table, Min in the second; 0: the other way round
    int32_t* e_out;
    int64_t row_blocks;    // workgroups along the rows
};

__device__ __forceinline__ void scan_store(const ScanSide& s, int G, int g, int64_t r, int mx, int mn) {
    s.tab[int64_t(s.max_half ? g : G + g) * s.o.rows_p + r] = int16_t(mx);
    s.tab[int64_t(s.max_half ? G + g : g) * s.o.rows_p + r] = int16_t(mn);
}

// Rows contiguous in memory (stride_r == 1): lanes along 64 rows, so every load instruction of a wave reads 512
// contiguous bytes; the four waves take every fourth k of a block, which keeps a thread's chain of loads short (a
// thread per row for four whole blocks: 28 us for 2048 x 2048, now 10), and are combined through LDS.
__device__ __forceinline__ int scan_rows(const ScanSide& s, int64_t rb, int g0, int per, int64_t k, int b, int G) {
    __shared__ int2 part[kScanBlocksPerWg][4][64];     // max; min, with bit 16 set when the part holds a zero
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r = rb * 64 + lane;
    int bad = 0;
#pragma unroll 1
    for (int u = 0; u < per; ++u) {
        const int g = g0 + u;
        BlockStat st;
        st.reset();
        if (g < G && r < s.o.rows) {
            const int64_t l0 = int64_t(g) * b, l1 = min(k, l0 + b);
            const uint64_t* src = reinterpret_cast<const uint64_t*>(s.o.X) + r + (l0 + wave) * s.o.stride_l;
#pragma unroll 16
            for (int64_t l = l0 + wave; l < l1; l += 4, src += 4 * s.o.stride_l) st.add(*src, bad);
        }
        part[u][wave][lane] = make_int2(st.mx, (st.mn & 0xFFFF) | (st.any_zero << 16));
    }
    __syncthreads();
    // wave u finishes block g0 + u
    const bool mine = wave < per && g0 + wave < G;
    BlockStat st;
    st.reset();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int2 x = part[mine ? wave : 0][w][lane];
        st.mx = max(st.mx, x.x);
        st.mn = min(st.mn, int(int16_t(x.y & 0xFFFF)));
        st.any_zero |= x.y >> 16;
    }
    st.any_nz = st.mx != -32768;
    if (mine) scan_store(s, G, g0 + wave, r, st.table_max(), st.table_min());
    __syncthreads();
    int* const row_max = reinterpret_cast<int*>(part);
    row_max[wave * 64 + lane] = mine ? int(st.table_max()) : kExpAllZero;
    __syncthreads();
    if (wave == 0) {
        const int e = max(max(row_max[lane], row_max[64 + lane]), max(row_max[128 + lane], row_max[192 + lane]));
        if (e > kExpAllZero) atomicMax(&s.e_out[r], e);
    }
    return bad;
}

// k contiguous in memory (stride_l == 1): 16 lanes share one row so that a load instruction
// reads 128 contiguous bytes per row; partial results are combined across the 16 lanes.
// A workgroup covers 16 rows.
__device__ __forceinline__ int scan_k(const ScanSide& s, int64_t rb, int g0, int per, int64_t k, int b, int G) {
    int row_max = kExpAllZero;
    const int q = threadIdx.x & 15;
    const int64_t r = rb * 16 + (threadIdx.x >> 4);
    int bad = 0;
    for (int g = g0; g < min(G, g0 + per); ++g) {
        BlockStat st;
        st.reset();
        if (r < s.o.rows) {
            const int64_t l0 = int64_t(g) * b;
            const int64_t l1 = min(k, l0 + b);
            const uint64_t* src = reinterpret_cast<const uint64_t*>(s.o.X) + r * s.o.stride_r;
#pragma unroll 4
            for (int64_t l = l0 + q; l < l1; l += 16) st.add(src[l], bad);
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) {
            st.mx = max(st.mx, __shfl_xor(st.mx, off));
            st.mn = min(st.mn, __shfl_xor(st.mn, off));
            st.any_nz |= __shfl_xor(st.any_nz, off);
            st.any_zero |= __shfl_xor(st.any_zero, off);
        }
        if (q == 0) {
            scan_store(s, G, g, r, st.table_max(), st.table_min());
            row_max = max(row_max, int(st.table_max()));
        }
    }
    if (q == 0 && row_max > kExpAllZero) atomicMax(&s.e_out[r], row_max);
    return bad;
}

// Both operands in one launch: the first blocks_a workgroups scan op(A), the others op(B), from ESC block g_first on.
__global__ __launch_bounds__(256) void scan_kernel(ScanSide a, ScanSide b, int64_t blocks_a, int g_first, int per, int64_t k,
                                                   int bl, int G, Record* rec, int check) {
    const bool second = int64_t(blockIdx.x) >= blocks_a;
    const ScanSide& s = second ? b : a;
    const int64_t id = int64_t(blockIdx.x) - (second ? blocks_a : 0);
    const int64_t rb = id % s.row_blocks;
    const int g0 = g_first + int(id / s.row_blocks) * per;
    const int bad = s.o.stride_r == 1 ? scan_rows(s, rb, g0, per, k, bl, G) : scan_k(s, rb, g0, per, k, bl, G);
    if (check && bad) atomicOr(&rec->infnan, 1);
}

void launch_init(hipStream_t st, const Workspace& w, const Problem& p, const KnownRecord& known) {
    const int64_t tiles = (p.mp / kTile) * (p.np / kTile);
    int64_t nmax = p.mp > p.np ? p.mp : p.np;
    if (tiles > nmax) nmax = tiles;
    hipLaunchKernelGGL(init_kernel, dim3(unsigned((nmax + 255) / 256)), dim3(256), 0, st, w.rec, w.eA, p.mp, w.eB, p.np,
                       w.tile_span, tiles, known);
}

void launch_scan(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, bool check_infnan) {
    const ScanGrid g = scan_grid(p, a.stride_r == 1, b.stride_r == 1);
    const ScanSide sa{a, w.U, 1, w.eA, g.row_blocks_a}, sb{b, w.V, 0, w.eB, g.row_blocks_b};
    for (int64_t y = 0; y < g.groups; y += g.slab) {
        const int64_t gy = g.groups - y < g.slab ? g.groups - y : g.slab;
        hipLaunchKernelGGL(scan_kernel, dim3(unsigned((g.row_blocks_a + g.row_blocks_b) * gy)), dim3(256), 0, st, sa, sb,
                           g.row_blocks_a * gy, int(y) * g.per, g.per, p.k, p.esc_block, p.G, w.rec, int(check_infnan));
    }
}

}  // namespace oz
