// Exponent-aligned slicing of op(A) (per row) and op(B) (per column) into 8-bit two's-complement
// digits with the unsigned-slice encoding.
// (paper: section "ESC" on the per-row shift space; section "Unsigned Slice Encoding": the
//  leading slice is rounded toward -infinity so that the remainder is non-negative, and every
//  sub-leading u8 digit >= 128 is stored as digit-256 with a carry into the next higher digit.)
//
// For an entry a of a row with exponent e_row and S slices:
//   X = floor(a * 2^q),  q = 8S - 3 - e_row,  |X| < 2^(8S-2)   (one headroom bit)
//   X = sum_s d_s 256^(S-1-s),  d_s in [-128, 127].
// a = sgn * M * 2^(E-1075) with the integer significand M, so X = (sgn*M) shifted by
// E - 1075 + q: written here as a 64-bit window W at bit offset o (X = W * 2^o), which covers
// any S up to 26 without multi-word arithmetic (up to 8 and up to 16 slices take one word of 64 or 128 bits instead).
//
// Output layout (what the INT8 GEMM's tiles load with contiguous 16-byte pieces):
//   slices[s][l/16][r][l%16]  for row r (padded to rows_p), k index l (padded to kp); padding = 0.
// HBM-bound: 8 B read and S bytes written per element.  Operands and slices are touched once per call
// here, so loads and stores carry the streaming (non-temporal) hint: measured 11 % faster.
#include "oz_internal.h"

namespace oz {

struct Fixed {
    int64_t W;
    int o;
};

__device__ __forceinline__ Fixed fixed_point(uint64_t bits, int e_row, int S) {
    const uint64_t mag = bits & 0x7FFFFFFFFFFFFFFFull;
    Fixed f;
    f.W = 0;
    f.o = 0;
    if (mag == 0 || e_row <= kExpAllZero) return f;
    const int field = int(mag >> 52);
    const uint64_t frac = mag & 0x000FFFFFFFFFFFFFull;
    const int64_t M = int64_t(field ? (frac | 0x0010000000000000ull) : frac);
    const int64_t sM = (bits >> 63) ? -M : M;
    const int sh = max(field, 1) - 1075 + (8 * S - 2 - kHeadroomBits - e_row);
    if (sh >= 0) {
        f.W = sM;
        f.o = min(sh, 8 * S);   // only Inf/NaN input (unguarded mode) can reach the clamp
    } else {
        f.W = sM >> min(-sh, 63);   // arithmetic shift: rounds toward -infinity
    }
    return f;
}

// bits [8b, 8b+8) of W * 2^o (two's complement, sign-extended), b = 0 least significant
__device__ __forceinline__ uint32_t byte_of(const Fixed& f, int b) {
    const int p = 8 * b - f.o;
    if (p >= 0) return uint32_t(f.W >> min(p, 63)) & 0xFFu;
    if (p > -8) return (uint32_t(f.W) << (-p)) & 0xFFu;
    return 0u;
}

// Digits of 16 consecutive k of one row, least significant slice first; writes 16 bytes per slice.
__device__ __forceinline__ void emit_slices(const Fixed (&f)[16], int S, int8_t* dst,
                                            int64_t slice_stride) {
    uint32_t carry[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) carry[e] = 0;
    for (int s = S - 1; s >= 0; --s) {
        const int b = S - 1 - s;
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t u = byte_of(f[e], b) + carry[e];
            carry[e] = (u >= 128u) ? 1u : 0u;       // unused after the leading slice
            w[e >> 2] |= (u & 0xFFu) << (8 * (e & 3));
        }
        *reinterpret_cast<uint4*>(dst + int64_t(s) * slice_stride) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Up to 8 slices the whole fixed-point value fits one 64-bit word, and the carry chain of the remap
// collapses into one addition: with BIAS = 0x80 in every sub-leading byte, the digits are the bytes
// of X + BIAS with the top bit of every sub-leading byte flipped.
//
// X for S <= 8 without branches: with sh = max(field,1) - 1075 + q (q = 8S - 3 - e_row) it is
// sM << sh or sM >> -sh (arithmetic: rounds toward -infinity), both computed and one selected;
// shift counts are clamped to 63 (a left shift beyond the word only happens for Inf/NaN input in
// unguarded mode).  Zeros, all-zero rows and padding have sM = 0 and need no special case.
__device__ __forceinline__ uint64_t biased_fixed64(uint64_t bits, int q_minus_1075, uint64_t bias) {
    const uint64_t mag = bits & 0x7FFFFFFFFFFFFFFFull;
    const int field = int(mag >> 52);
    const uint64_t frac = mag & 0x000FFFFFFFFFFFFFull;
    const uint64_t M = field ? (frac | 0x0010000000000000ull) : frac;
    const uint64_t sgn = uint64_t(int64_t(bits) >> 63);              // all ones for negative entries
    const int64_t sM = int64_t((M ^ sgn) - sgn);
    const int sh = max(field, 1) + q_minus_1075;
    const int64_t left = sM << min(max(sh, 0), 63);
    const int64_t right = sM >> min(max(-sh, 0), 63);
    return uint64_t(sh >= 0 ? left : right) + bias;
}

// The same for 9 to 16 slices on 128 bits.  sh beyond the word leaves zeros (only Inf/NaN input in unguarded mode).
// (Digit by digit with a carry per element instead: 100 us for 4096 x 4096 with nine slices, now 58.)
__device__ __forceinline__ void biased_fixed128(uint64_t bits, int q_minus_1075, uint64_t bias_lo, uint64_t bias_hi,
                                                uint64_t& lo, uint64_t& hi) {
    const uint64_t mag = bits & 0x7FFFFFFFFFFFFFFFull;
    const int field = int(mag >> 52);
    const uint64_t frac = mag & 0x000FFFFFFFFFFFFFull;
    const uint64_t M = field ? (frac | 0x0010000000000000ull) : frac;
    const uint64_t sgn = uint64_t(int64_t(bits) >> 63);
    const int64_t sM = int64_t((M ^ sgn) - sgn);
    const int sh = max(field, 1) + q_minus_1075;
    const int up = min(max(sh, 0), 127), down = min(max(-sh, 0), 63);
    const int64_t low = up < 64 ? int64_t(uint64_t(sM) << (up & 63)) : 0;
    // bits 64.. of sM << up: for up < 64 what falls out at the top (with the sign above it)
    const int64_t high = up < 64 ? (sM >> 1) >> (63 - (up & 63)) : int64_t(uint64_t(sM) << (up & 63));
    const int64_t right = sM >> down;
    const bool out = sh > 127;
    const uint64_t x_lo = out ? 0ull : uint64_t(sh >= 0 ? low : right), x_hi = out ? 0ull : uint64_t(sh >= 0 ? high : right >> 63);
    lo = x_lo + bias_lo;
    hi = x_hi + bias_hi + (lo < x_lo ? 1ull : 0ull);
}

// Byte b of 16 values (NW dwords each, least significant first) is gathered into four dwords with byte permutes
// (three per dword).
template <int NW>
__device__ __forceinline__ void emit_words(const uint32_t (&y)[NW][16], int S, int8_t* dst, int64_t slice_stride) {
#pragma unroll
    for (int v = NW - 1; v >= 0; --v)
        for (int b = min(S - 1, 4 * v + 3); b >= 4 * v; --b) {
            const uint32_t k = uint32_t(b) & 3u;
            const uint32_t pick = k * 0x0101u + 0x0400u;            // result bytes: [second.k, first.k, -, -]
            const uint32_t flip = (b == S - 1) ? 0u : 0x80808080u;  // the leading digit keeps its sign bit
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t t1 = __builtin_amdgcn_perm(y[v][4 * j + 1], y[v][4 * j], pick);
                const uint32_t t2 = __builtin_amdgcn_perm(y[v][4 * j + 3], y[v][4 * j + 2], pick);
                w[j] = __builtin_amdgcn_perm(t2, t1, 0x05040100u) ^ flip;
            }
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            __builtin_nontemporal_store(u32x4{w[0], w[1], w[2], w[3]},
                                        reinterpret_cast<u32x4*>(dst + int64_t(S - 1 - b) * slice_stride));
        }
}

__device__ __forceinline__ void emit(const uint64_t (&bits)[16], int e_row, int S, int8_t* dst,
                                     int64_t slice_stride) {
    const int q = 8 * S - 2 - kHeadroomBits - (e_row > kExpAllZero ? e_row : 0) - 1075;
    if (S <= 8) {
        const uint64_t bias = S >= 2 ? (0x8080808080808080ull >> (8 * (9 - S))) : 0ull;
        uint32_t y[2][16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint64_t x = biased_fixed64(bits[e], q, bias);
            y[0][e] = uint32_t(x);
            y[1][e] = uint32_t(x >> 32);
        }
        emit_words<2>(y, S, dst, slice_stride);
    } else if (S <= 16) {
        const uint64_t bias_hi = S >= 10 ? (0x8080808080808080ull >> (8 * (17 - S))) : 0ull;
        uint32_t y[4][16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            uint64_t lo, hi;
            biased_fixed128(bits[e], q, 0x8080808080808080ull, bias_hi, lo, hi);
            y[0][e] = uint32_t(lo);
            y[1][e] = uint32_t(lo >> 32);
            y[2][e] = uint32_t(hi);
            y[3][e] = uint32_t(hi >> 32);
        }
        emit_words<4>(y, S, dst, slice_stride);
    } else {
        Fixed f[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) f[e] = fixed_point(bits[e], e_row, S);
        emit_slices(f, S, dst, slice_stride);
    }
}

// Rows contiguous in memory: thread = row, lanes along rows; loads coalesce across the wave.
// A workgroup cuts 256 rows x 16 k (chunk c).
__device__ __forceinline__ void slice_rows(const Operand& o, int64_t rb, int64_t c, int64_t k, int64_t kp, int er,
                                           int8_t* __restrict__ out, int S) {
    const int64_t r = rb * 256 + threadIdx.x;
    // loads are unconditional at clamped addresses (rows >= 1 and k >= 1 here); out-of-range
    // elements are then replaced by zero, so the loop has no divergent branches
    const bool row_ok = r < o.rows;
    const uint64_t* src = reinterpret_cast<const uint64_t*>(o.X) + (row_ok ? r : o.rows - 1);
    uint64_t bits[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int64_t l = c * 16 + e;
        const uint64_t x = __builtin_nontemporal_load(&src[(l < k ? l : k - 1) * o.stride_l]);
        bits[e] = (row_ok && l < k) ? x : 0ull;
    }
    emit(bits, er, S, out + (c * o.rows_p + r) * 16, kp * o.rows_p);
}

// k contiguous in memory: a 64-row x 64-k tile is read with lanes along k (512 contiguous bytes
// per wave load), transposed through LDS, then each thread owns (row, 16-k chunk).
__device__ __forceinline__ void slice_k(const Operand& o, int64_t rb, int64_t lb, int64_t k, int64_t kp,
                                        int er, int8_t* __restrict__ out, int S, uint64_t (*T)[65]) {
    const int64_t r0 = rb * 64, l0 = lb * 64;
    {
        const int ll = threadIdx.x & 63;
        const int rr0 = threadIdx.x >> 6;
        const uint64_t* src = reinterpret_cast<const uint64_t*>(o.X);
#pragma unroll
        for (int it = 0; it < 16; ++it) {
            const int rr = rr0 + it * 4;
            const int64_t r = r0 + rr, l = l0 + ll;
            const uint64_t x = __builtin_nontemporal_load(&src[(r < o.rows ? r : o.rows - 1) * o.stride_r + (l < k ? l : k - 1)]);
            T[rr][ll] = (r < o.rows && l < k) ? x : 0ull;
        }
    }
    __syncthreads();
    const int rr = threadIdx.x & 63, cc = threadIdx.x >> 6;
    const int64_t r = r0 + rr;
    uint64_t bits[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) bits[e] = T[rr][cc * 16 + e];
    const int64_t c = l0 / 16 + cc;
    emit(bits, er, S, out + (c * o.rows_p + r) * 16, kp * o.rows_p);
}

struct SliceSide {
    Operand o;
    const int32_t* e_row;
    int8_t* out;
    int64_t row_blocks, blocks;      // workgroups along the rows, in all
};

// workgroups [0, a.blocks) cut a, the others b (swapped: a is op(B)).  The LDS tile is dynamic: an operand with contiguous rows needs none
__global__ __launch_bounds__(256) void slice_kernel(SliceSide a, SliceSide b, int64_t k, int64_t kp, const Record* rec, Batch bt, int swapped) {
    extern __shared__ uint64_t slice_lds[];
    const bool second = int64_t(blockIdx.x) >= a.blocks;
    const int64_t ws = bt.ws_at(blockIdx.z);
    SliceSide s = second ? b : a;
    s.o.X += (second != bool(swapped)) ? bt.b_at(blockIdx.z) : bt.a_at(blockIdx.z);
    s.e_row = at_bytes(s.e_row, ws);
    s.out = at_bytes(s.out, ws);
    rec = at_bytes(rec, ws);
    const int64_t id = int64_t(blockIdx.x) - (second ? a.blocks : 0);
    const int64_t rb = id % s.row_blocks, cb = id / s.row_blocks;
    const bool rows = s.o.stride_r == 1;
    // the row's exponent is requested together with the record: two loads in a row before the operand's is what a small
    // call waits for
    const int er = s.e_row[rows ? rb * 256 + threadIdx.x : rb * 64 + (threadIdx.x & 63)];
    const int fallback = rec->res.fallback, S = rec->res.slices_used;
    if (fallback) return;
    if (rows) slice_rows(s.o, rb, cb, k, kp, er, s.out, S);
    else slice_k(s.o, rb, cb, k, kp, er, s.out, S, reinterpret_cast<uint64_t (*)[65]>(slice_lds));
}

void launch_slice(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p) {
    auto side = [&](const Operand& o, const int32_t* e, int8_t* out) {
        const bool rows = o.stride_r == 1;
        const int64_t rbs = o.rows_p / (rows ? 256 : 64);
        return SliceSide{o, e, out, rbs, rbs * (p.kp / (rows ? 16 : 64))};
    };
    const SliceSide sa = side(a, w.eA, w.As), sb = side(b, w.eB, w.Bs);
    constexpr size_t kLds = 64 * 65 * sizeof(uint64_t);
    const size_t lds_a = a.stride_r == 1 ? 0 : kLds, lds_b = b.stride_r == 1 ? 0 : kLds;
    // Both operands in one launch where they need the same LDS, or where the launch itself is what counts (fewer
    // workgroups than 16 per CU); otherwise the LDS tile of the one would halve the occupancy of the other.
    const unsigned z = unsigned(p.batch.count);
    if (lds_a == lds_b || (sa.blocks + sb.blocks) * z < int64_t(16) * p.num_cu) {
        hipLaunchKernelGGL(slice_kernel, dim3(unsigned(sa.blocks + sb.blocks), 1, z), dim3(256), lds_a > lds_b ? lds_a : lds_b, st, sa,
                           sb, p.k, p.kp, w.rec, p.batch, 0);
    } else {
        hipLaunchKernelGGL(slice_kernel, dim3(unsigned(sa.blocks), 1, z), dim3(256), lds_a, st, sa, sb, p.k, p.kp, w.rec, p.batch, 0);
        hipLaunchKernelGGL(slice_kernel, dim3(unsigned(sb.blocks), 1, z), dim3(256), lds_b, st, sb, sa, p.k, p.kp, w.rec, p.batch, 1);
    }
}

}  // namespace oz
