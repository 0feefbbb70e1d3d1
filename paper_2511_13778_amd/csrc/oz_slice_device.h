// Device code of the slicing, shared by its own kernel and by the one that decides a small call on the way (oz_esc_slice.hip): the
// digits of an entry, and the loads and stores of either storage order.
//
// For an entry a of a row with exponent e_row and S slices:
//   X = floor(a * 2^q),  q = 8S - 3 - e_row,  |X| < 2^(8S-2)   (one headroom bit)
//   X = sum_s d_s 256^(S-1-s),  d_s in [-128, 127].
// a = sgn * M * 2^(E-1075) with the integer significand M, so X = (sgn*M) shifted by
// E - 1075 + q: beyond 16 slices a word of 64 bits at a byte of its own holds all digits that are not zero, up to 8 and up to 16 slices
// one word of 64 or 128 bits holds all of X.
//
// Output layout (what the INT8 GEMM's tiles load with contiguous 16-byte pieces):
//   slices[s][l/16][r][l%16]  for row r (padded to rows_p), k index l (padded to kp); padding = 0.
#pragma once

#include "oz_internal.h"

namespace oz {


// Digits of an entry for any slice count: those of a 64-bit word, eight of them, from bit o (a multiple of eight) on; the others are zero.
// (53 bits shifted by at most seven: the leading one of the eight holds what is left with its sign, so no carry leaves them.  Byte
// by byte with a carry a register more an entry, and 20 slices of 3000 x 3000 twice 175 to 179 us, now 116 to 134.)
struct Fixed {
    uint64_t D;
    int o;
};

__device__ __forceinline__ Fixed fixed_point(uint64_t bits, int e_row, int S) {
    const uint64_t mag = bits & 0x7FFFFFFFFFFFFFFFull;
    Fixed f;
    f.D = 0;
    f.o = 0;
    if (mag == 0 || e_row <= kExpAllZero) return f;
    const int field = int(mag >> 52);
    const uint64_t frac = mag & 0x000FFFFFFFFFFFFFull;
    const int64_t M = int64_t(field ? (frac | 0x0010000000000000ull) : frac);
    const int64_t sM = (bits >> 63) ? -M : M;
    const int sh = min(max(field, 1) - 1075 + (8 * S - 2 - kHeadroomBits - e_row), 8 * S);   // only Inf/NaN input (unguarded mode) can reach the clamp
    constexpr uint64_t kBias = 0x0080808080808080ull;
    if (sh >= 0) {
        f.D = ((uint64_t(sM) << (sh & 7)) + kBias) ^ kBias;
        f.o = sh & ~7;
    } else {
        f.D = (uint64_t(sM >> min(-sh, 63)) + kBias) ^ kBias;   // arithmetic shift: rounds toward -infinity
    }
    return f;
}

// N = 4 or 16 consecutive k of one row leave N bytes per slice.
template <int N>
__device__ __forceinline__ void store_digits(const uint32_t (&w)[N / 4], int8_t* plane, uint32_t lane_off) {
    typedef uint32_t vec __attribute__((ext_vector_type(N / 4)));
    vec v;
    if constexpr (N == 4) v = w[0];
    else v = vec{w[0], w[1], w[2], w[3]};
    __builtin_nontemporal_store(v, reinterpret_cast<vec*>(plane + lane_off));
}

template <int N>
__device__ __forceinline__ void emit_slices(const Fixed (&f)[N], int S, int8_t* plane0, uint32_t lane_off, int64_t slice_stride) {
    for (int s = S - 1; s >= 0; --s) {
        uint32_t w[N / 4] = {};
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint32_t p = uint32_t(8 * (S - 1 - s) - f[e].o);
            w[e >> 2] |= (p < 64u ? uint32_t(f[e].D >> (p & 63u)) & 0xFFu : 0u) << (8 * (e & 3));
            if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        store_digits<N>(w, plane0 + int64_t(s) * slice_stride, lane_off);
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

// X + BIAS for S <= 8 on the FP64 unit, in five instructions instead of 24: with the unit rounding toward -infinity, adding
// 1.5 * 2^52 leaves floor(a * 2^(q-32)) in the low word, what that leaves over is in [0, 1), and 2^32 times that plus 2^52 leaves the
// low word of X in the low word.  Rounding the rest (an entry far below its row's largest, negative) downwards changes no floor.  The
// two constants carry the bias: its low word may carry into the upper word of the second sum, which is added to the first.
// (Both operands of 8192^3, seven slices, rows contiguous: 447 us in integer arithmetic at 128 registers, now 360.)
struct Fp64Cut {
    double scale, magic_hi, magic_lo;
    static constexpr uint32_t kTwo52 = 0x43300000u;          // upper word of 2^52
    // q_minus_32 within the exponents of normal numbers
    __device__ __forceinline__ Fp64Cut(int q_minus_32, uint64_t bias)
        : scale(__builtin_bit_cast(double, uint64_t(q_minus_32 + 1023) << 52)),
          magic_hi(__builtin_bit_cast(double, 0x4338000000000000ull | uint32_t(uint32_t(bias >> 32) - kTwo52))),
          magic_lo(__builtin_bit_cast(double, uint64_t(kTwo52) << 32 | uint32_t(bias))) {}
    __device__ __forceinline__ void cut(uint64_t bits, uint32_t& lo, uint32_t& hi) const {
        const double a = __builtin_bit_cast(double, bits);
        const double h = __builtin_fma(a, scale, magic_hi);
        const double rest = __builtin_fma(a, scale, -(h - magic_hi));
        const uint64_t l = __builtin_bit_cast(uint64_t, __builtin_fma(rest, 0x1p32, magic_lo));
        lo = uint32_t(l);
        hi = uint32_t(__builtin_bit_cast(uint64_t, h)) + uint32_t(l >> 32);
    }
};

// Byte b of N values (NW dwords each, least significant first) goes to plane S - 1 - b, four values to a dword: transposes of four
// dwords in two steps of byte permutes.
template <int NW, int N>
__device__ __forceinline__ void emit_words(const uint32_t (&y)[NW][N], int S, int8_t* plane0, uint32_t lane_off, int64_t slice_stride) {
#pragma unroll
    for (int v = NW - 1; v >= 0; --v) {
        if (4 * v >= S) continue;
#pragma unroll
        for (int half = 1; half >= 0; --half) {              // bytes 2, 3 and 0, 1
            if (4 * v + 2 * half >= S) continue;
            uint32_t w[2][N / 4];
#pragma unroll
            for (int j = 0; j < N / 4; ++j) {
                const uint32_t pick = half ? 0x07030602u : 0x05010400u;
                const uint32_t t01 = __builtin_amdgcn_perm(y[v][4 * j + 1], y[v][4 * j], pick);
                const uint32_t t23 = __builtin_amdgcn_perm(y[v][4 * j + 3], y[v][4 * j + 2], pick);
                w[0][j] = __builtin_amdgcn_perm(t23, t01, 0x05040100u);
                w[1][j] = __builtin_amdgcn_perm(t23, t01, 0x07060302u);
            }
#pragma unroll
            for (int q = 1; q >= 0; --q) {
                const int b = 4 * v + 2 * half + q;
                if (b >= S) continue;
                const uint32_t flip = b == S - 1 ? 0u : 0x80808080u;     // the leading digit keeps its sign bit
#pragma unroll
                for (int j = 0; j < N / 4; ++j) w[q][j] ^= flip;
                store_digits<N>(w[q], plane0 + int64_t(S - 1 - b) * slice_stride, lane_off);
            }
        }
    }
}

// plane0: where the first plane's entries of this wave lie (uniform), lane_off: bytes to this lane's
template <int MAXS, int N>
__device__ __forceinline__ void emit(const uint64_t (&bits)[N], int e_row, int S, int8_t* plane0, uint32_t lane_off,
                                     int64_t slice_stride) {
    const int q = 8 * S - 2 - kHeadroomBits - (e_row > kExpAllZero ? e_row : 0);
    if (S <= 8) {
        const uint64_t bias = S >= 2 ? (0x8080808080808080ull >> (8 * (9 - S))) : 0ull;
        uint32_t y[2][N];
        // Inf and NaN (unguarded mode), and rows of 2^-960 and less, whose factor is no normal number: integer arithmetic
        if (__all(e_row < kExpInfNan && q - 32 >= -1022 && q - 32 <= 1023)) {
            const Fp64Cut c(q - 32, bias);
#pragma unroll
            for (int e = 0; e < N; ++e) c.cut(bits[e], y[0][e], y[1][e]);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const uint64_t x = biased_fixed64(bits[e], q - 1075, bias);
                y[0][e] = uint32_t(x);
                y[1][e] = uint32_t(x >> 32);
                __builtin_amdgcn_sched_barrier(0);           // one at a time: registers
            }
        }
        emit_words<2, N>(y, S, plane0, lane_off, slice_stride);
        return;
    }
    if constexpr (MAXS > 8) {
        if (S <= 16) {
            const uint64_t bias_hi = S >= 10 ? (0x8080808080808080ull >> (8 * (17 - S))) : 0ull;
            uint32_t y[4][N];
#pragma unroll
            for (int e = 0; e < N; ++e) {
                uint64_t lo, hi;
                biased_fixed128(bits[e], q - 1075, 0x8080808080808080ull, bias_hi, lo, hi);
                y[0][e] = uint32_t(lo);
                y[1][e] = uint32_t(lo >> 32);
                y[2][e] = uint32_t(hi);
                y[3][e] = uint32_t(hi >> 32);
            }
            emit_words<4, N>(y, S, plane0, lane_off, slice_stride);
            return;
        }
    }
    if constexpr (MAXS > 16) {
        Fixed f[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            f[e] = fixed_point(bits[e], e_row, S);
            __builtin_amdgcn_sched_barrier(0);               // one at a time: registers
        }
        emit_slices<N>(f, S, plane0, lane_off, slice_stride);
    }
}

// FP64 rounds toward -infinity from here on (Fp64Cut).  As assembly, and before the loads that all FP64 arithmetic waits for: the
// compiler sets the mode back before such arithmetic where it knows of a change.
__device__ __forceinline__ void round_down_fp64() {
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 2\n\ts_nop 1" ::: "memory");
}

// Rows contiguous in memory: a thread takes 16 k (chunk c) of row rb * 256 + at, lanes along the rows, so loads coalesce across the wave.
__device__ __forceinline__ void load_rows(const Operand& o, int64_t rb, uint32_t at, int64_t c, int64_t k, uint64_t (&bits)[16]) {
    // loads are unconditional at clamped addresses (rows >= 1 and k >= 1 here, and every block of rows has one); out-of-range
    // elements are then replaced by zero, so the loop has no divergent branches
    const int64_t rows_here = o.rows - rb * 256;
    const bool row_ok = int64_t(at) < rows_here;
    const uint32_t lane = uint32_t(min(int64_t(at), rows_here - 1)) * 8u;
    const char* const src = reinterpret_cast<const char*>(o.X + rb * 256);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int64_t l = c * 16 + e;
        const uint64_t x = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(src + (l < k ? l : k - 1) * o.stride_l * 8 + lane));
        bits[e] = (row_ok && l < k) ? x : 0ull;
    }
}
template <int MAXS>
__device__ __forceinline__ void put_rows(const uint64_t (&bits)[16], const Operand& o, int64_t rb, uint32_t at, int64_t c, int64_t kp, int er,
                                         int8_t* __restrict__ out, int S) {
    emit<MAXS, 16>(bits, er, S, out + (c * o.rows_p + rb * 256) * 16, at * 16u, kp * o.rows_p);
}

// The same with four k (part p of chunk c) a thread, for calls of few entries: a quarter of the work in a row, four times the threads.
__device__ __forceinline__ void load_rows4(const Operand& o, int64_t r0, uint32_t at, int64_t c, int p, int64_t k, uint64_t (&bits)[4]) {
    const bool row_ok = r0 + at < o.rows;
    const uint64_t* const src = reinterpret_cast<const uint64_t*>(o.X) + min(r0 + at, o.rows - 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t l = c * 16 + p * 4 + e;
        const uint64_t x = src[(l < k ? l : k - 1) * o.stride_l];
        bits[e] = row_ok && l < k ? x : 0ull;
    }
}

// k contiguous in memory: four lanes share 16 consecutive k (chunk c) of a row (128 bytes, 16 per load and lane), a wave takes 16 rows from
// r0 on; a lane's four k are a dword of every plane, and the 64 lanes' dwords lie behind each other.  (A 64 x 64 tile transposed
// through LDS instead, so that a thread has 16 k: four workgroups to a CU that load and cut in turn, 8192 x 8192 with seven slices 255 us,
// now 210.)
__device__ __forceinline__ void load_k(const Operand& o, int64_t r0, int64_t c, int64_t k, uint64_t (&x)[4]) {
    typedef uint64_t pair __attribute__((ext_vector_type(2), aligned(8)));
    const int lane = threadIdx.x & 63;
    const bool row_ok = (lane >> 2) < o.rows - r0;
    const int64_t l0 = c * 16 + (lane & 3) * 4;
    // rows past the end read the last one, and count as zero
    const uint64_t* const src = reinterpret_cast<const uint64_t*>(o.X) + min(r0 + (lane >> 2), o.rows - 1) * o.stride_r;
    if (c * 16 + 16 <= k) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const pair p = __builtin_nontemporal_load(reinterpret_cast<const pair*>(src + l0 + h * 2));
            x[2 * h] = row_ok ? p[0] : 0ull;
            x[2 * h + 1] = row_ok ? p[1] : 0ull;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t y = src[min(l0 + e, k - 1)];
            x[e] = row_ok && l0 + e < k ? y : 0ull;
        }
    }
}
template <int MAXS>
__device__ __forceinline__ void put_k(const uint64_t (&x)[4], const Operand& o, int64_t r0, int64_t c, int64_t kp, int er, int8_t* __restrict__ out,
                                      int S) {
    emit<MAXS, 4>(x, er, S, out + (c * o.rows_p + r0) * 16, uint32_t(threadIdx.x & 63) * 4u, kp * o.rows_p);
}

}  // namespace oz
