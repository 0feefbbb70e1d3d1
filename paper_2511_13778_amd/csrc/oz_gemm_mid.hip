// Slice-pair GEMMs and FP64 recomposition in one kernel on 64 x 64 tiles of C: what gemm_i8_kernel and recompose_kernel compute,
// for calls whose k is short beside the size of C, and for mid-sized ones.
// (paper: section "FP64 Emulation on Low-Precision Units".)
//
// With units of 128 x 128 such a call spends its time around the products: a unit of a short k is mostly its start and its two or
// three ends of groups of anti-diagonals, nothing runs beside them (one wave per SIMD, all accumulators taken), the digits written
// are read again, and less than a round of units leaves CUs idle.  Here all S slices of a 64 of k lie in LDS (4 KB each), a wave
// owns 32 columns i and keeps all anti-diagonals of its part in registers, D of them side by side (a step reads one slice of A and
// one of B and multiplies it with the window of D, as in gemm_i8_kernel), so k is walked once, and carry chain, powers of two,
// alpha and beta follow in the same launch.
//   SETS = 1   4 waves of 32 rows j, D = 4, up to 8 slices, 80 KB: two workgroups to a CU, one ends or loads while the other multiplies
//   SETS = 2   8 waves of 16 rows j, D = 8, up to 16 slices, all of the LDS: more than one stage up to 10 slices
// Either way a step of a full window is 16 MFMAs of a wave, and all waves have the same share.  (Two sets of four waves with groups of
// four anti-diagonals dealt to the sets: with nine slices one set had 31 pairs of 45 and the other 14, and their sums met in LDS.  16
// problems of 512^3 205 us, now 202; 1024^3 75 -> 68, 1500x1300x900 124 -> 110, 3000x3000x700 on these tiles 362 -> 314.)
// The walk over k is compiled once per slice count: the same loops with the count in a register have a branch in front of every
// step, so that reads cannot be placed among products, and took 215 and 75 us for the first two of these, 225 and 79 with fewer LDS reads.
// Digits, leading words and C are 26 bytes per element, read and written once and streamed past L2, where the slices of the next tiles
// live (plain stores, which drive those out, cost 85 us of 690 at 7936 x 7936 x 256).  What bounds it at a short k is the end of a tile:
// memory, and the integer work of the carry chain, which the other workgroup's products only partly cover (7936 x 7936, seven
// slices: 325 us plus 82 per 64 of k); at a long one the transfers of slices into LDS (7936 x 7936 x 256: 650 us, 595 when
// all of them hit L2, 545 without any; 2048^3 with seven slices 235, 229, 198).  Stages of 32 of k, twice as deep, gain 5 percent where they
// save half a stage (k = 200) and lose 5 at 512; wave priorities gain nothing.
// Measured, whole calls, against units: 7936x7936x256 802 -> 650 us, 1500x1300x900 124 -> 79 with seven slices, 170 -> 110 with nine;
// 16 problems of 512^3, which also share their launches, 399 -> 202.
#include "oz_f64_direct.h"
#include "oz_gemm_device.h"

namespace oz {

constexpr int kMidSlice = kMidTile * kBK;                   // bytes of one slice of one operand for a 64 of k: [k chunk][row][16 B]
static_assert(kMidTile == 64 && kBK == 64, "a transfer moves one k chunk of 64 rows, a wave owns 32 columns of a tile");
static_assert(kMidMaxSlices * 2 * kMidSlice <= kSmallLdsMax, "one stage must fit");
static_assert(kMidPairSlices * 2 * kMidSlice <= kSmallLdsMax / 2, "one of two workgroups");

template <int N>
struct MidInt { static constexpr int v = N; };

// f(MidInt<1>) ... f(MidInt<N>)
template <int N, class F>
__device__ __forceinline__ void mid_each(F&& f) {
    if constexpr (N > 0) {
        mid_each<N - 1>(f);
        f(MidInt<N>{});
    }
}

template <int SETS>
__global__ __launch_bounds__(256 * SETS, 2) void gemm_mid_kernel(
    const int8_t* __restrict__ As, const int8_t* __restrict__ Bs, int32_t* __restrict__ T, int8_t* __restrict__ L,
    const int32_t* __restrict__ eA, const int32_t* __restrict__ eB, int64_t m, int64_t n, int64_t mp, int64_t np, int64_t kp,
    int ntm, int ntn, int kt_total, int lds_bytes, double alpha, double beta, double* __restrict__ C, int64_t ldc, const Record* rec,
    const int32_t* __restrict__ tile_S, Batch bt, Fallback fb) {
    constexpr int WAVES = 4 * SETS, D = 4 * SETS, FB = 2 / SETS;           // FB: tiles of 16 rows j of a wave
    constexpr int MAX_S = SETS == 1 ? kMidPairSlices : kMidMaxSlices, GROUPS = MAX_S / D;
    extern __shared__ __align__(16) uint8_t lds[];
    {
        const int64_t ws = bt.ws_at(blockIdx.z);
        As = at_bytes(As, ws); Bs = at_bytes(Bs, ws);
        T = at_bytes(T, ws); L = at_bytes(L, ws);
        eA = at_bytes(eA, ws); eB = at_bytes(eB, ws);
        rec = at_bytes(rec, ws);
        if (tile_S) tile_S = at_bytes(tile_S, ws);
        C += int64_t(blockIdx.z) * bt.c;
    }
    const int fallback = rec->res.fallback, S_all = rec->res.slices_used;
    int ti, tj;
    {
        const int total = ntm * ntn, xcd = int(blockIdx.x) & 7, slot = int(blockIdx.x) >> 3;
        const int per = total >> 3, rem = total & 7;
        lin_to_tile(xcd * per + min(xcd, rem) + slot, ntm, ntn, ti, tj);
    }
    const int64_t i0 = int64_t(ti) * kMidTile, j0 = int64_t(tj) * kMidTile;
    if (fallback) {
        if (fb.A) fall_back<4, 4, WAVES>(fb, bt, int(blockIdx.z), reinterpret_cast<double*>(lds), m, n, i0, j0, alpha, beta, C, ldc);
        return;
    }
    const int S = tile_S ? min(tile_S[(j0 / kTile) * (mp / kTile) + i0 / kTile], S_all) : S_all;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int set = wave >> 2, qi = wave & 1, qj = wave >> 1;

    // ---- elements this thread finishes: column i, and in each tile of 16 rows j two times four
    const int64_t i = i0 + qi * 32 + (lane & 31);
    auto row_of = [&](int b, int u) -> int64_t { return j0 + qj * (16 * FB) + b * 16 + (lane >> 5) * 8 + u * 4; };
    double cin[FB][2][4];
    if (beta != 0.0) {
#pragma unroll
        for (int b = 0; b < FB; ++b)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    cin[b][u][q] = C[min(row_of(b, u) + q, n - 1) * ldc + min(i, m - 1)];
    }

    // ---- transfers: a wave fetches k chunk (wave & 3) of every SETS-th slice, A's then B's
    const uint32_t lane_off = uint32_t(lane) * 16;
    const uint32_t lds_base = uint32_t(uintptr_t((__attribute__((address_space(3))) uint8_t*)lds));
    const uint32_t stage_bytes = uint32_t(2 * kMidSlice) * uint32_t(S);
    const int stages = min(kt_total, lds_bytes / int(stage_bytes));
    const int pieces = 2 * ((S - set + SETS - 1) / SETS);          // of this wave per 64 of k
    const uint8_t* nextA = reinterpret_cast<const uint8_t*>(As) + ((wave & 3) * mp + i0) * 16 + set * (kp * mp);
    const uint8_t* nextB = reinterpret_cast<const uint8_t*>(Bs) + ((wave & 3) * np + j0) * 16 + set * (kp * np);
    const int64_t planeA = SETS * kp * mp, planeB = SETS * kp * np;
    auto issue = [&](int stage) {
        uint32_t to = lds_base + uint32_t(stage) * stage_bytes + uint32_t(wave & 3) * 1024u + uint32_t(set) * kMidSlice;
        const uint8_t *a = nextA, *b = nextB;
        for (int q = set; q < S; q += SETS) {
            dma16<0>(a, lane_off, to);
            dma16<0>(b, lane_off, to + uint32_t(S) * kMidSlice);
            a += planeA;
            b += planeB;
            to += SETS * kMidSlice;
        }
        nextA += int64_t(kBK) * mp;
        nextB += int64_t(kBK) * np;
    };
    int issued = 0, put = 0;
    auto issue_next = [&](int limit) {
        if (issued >= limit) return;
        issue(put);
        ++issued;
        put = put + 1 == stages ? 0 : put + 1;
    };
    issue_next(1);
    issue_next(min(2, stages));

    // ---- anti-diagonals in groups of D side by side (as in gemm_i8_kernel, where D is 4)
    v4i acc[GROUPS][D][FB][2];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int j = 0; j < D; ++j)
#pragma unroll
            for (int b = 0; b < FB; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) acc[g][j][b][a] = v4i{0, 0, 0, 0};
    const uint32_t rd = uint32_t(lane >> 4) * 1024u + uint32_t(lane & 15) * 16u;
    const uint32_t rdA = rd + uint32_t(qi) * 512u, rdB = rd + uint32_t(qj) * (256u * FB) + uint32_t(S) * kMidSlice;
    // the walk over k for a slice count that the compiler knows: no branches between the products, and reads placed among them
    auto walk = [&](auto SS) {
        constexpr int NS = decltype(SS)::v;
        int stage = 0;
        for (int kt = 0; kt < kt_total; ++kt) {
            wait_transfers((issued - 1 - kt) * pieces);
            __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): this wave's reads of the stage before have returned
            asm volatile("s_barrier" ::: "memory");
            const int limit = min(min(kt + stages, issued + 1), kt_total);
            issue_next(limit);
            const uint8_t* const atA = lds + uint32_t(stage) * stage_bytes + rdA;
            const uint8_t* const atB = lds + uint32_t(stage) * stage_bytes + rdB;
            constexpr int USED = (NS + D - 1) / D;
            v4i fa[USED][2][2], fb[USED][D][FB];
            auto read_a = [&](int gg, int s) {
#pragma unroll
                for (int f = 0; f < 2; ++f) fa[gg][s & 1][f] = *reinterpret_cast<const v4i*>(atA + s * kMidSlice + f * 256);
            };
            auto read_b = [&](int gg, int t) {
#pragma unroll
                for (int f = 0; f < FB; ++f) fb[gg][t & (D - 1)][f] = *reinterpret_cast<const v4i*>(atB + t * kMidSlice + f * 256);
            };
            auto read_first = [&](int gg) {
                const int d_hi = NS - 1 - D * gg;
                read_a(gg, 0);
#pragma unroll
                for (int t = d_hi; t >= 0 && t > d_hi - D; --t) read_b(gg, t);
            };
            read_first(0);
#pragma unroll
            for (int gg = 0; gg < USED; ++gg) {
                const int d_hi = NS - 1 - D * gg;
                // step s multiplies A_s with B_(d_hi - s - j), j = 0 .. D - 1; slice t of B lies in slot t mod D.  What the next
                // step needs is read before its products (left to itself the compiler reads it after them and waits).
#pragma unroll
                for (int s = 0; s <= d_hi; ++s) {
                    const int r = d_hi - s;
                    __builtin_amdgcn_sched_barrier(0);
                    if (r > 0) read_a(gg, s + 1);
                    if (gg + 1 < USED && r == 1) read_first(gg + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        if (j > r) continue;
#pragma unroll
                        for (int b = 0; b < FB; ++b)
#pragma unroll
                            for (int a = 0; a < 2; ++a)
                                acc[gg][j][b][a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[gg][(r - j) & (D - 1)][b], fa[gg][s & 1][a], acc[gg][j][b][a], 0, 0, 0);
                        if (j == 0 && r >= D) read_b(gg, r - D);
                    }
                }
            }
            if (stages == 1) {
                __builtin_amdgcn_s_waitcnt(0xC07F);
                asm volatile("s_barrier" ::: "memory");
                issue_next(kt_total);
            }
            stage = stage + 1 == stages ? 0 : stage + 1;
        }
    };
    mid_each<MAX_S>([&](auto V) {
        if (S == decltype(V)::v) walk(V);
    });

    // ---- carry chain and recomposition of columns i and, four at a time, rows j .. j + 3 of C.
    const int ea = eA[i];
    const int64_t planeL = np * mp / 4;      // in words
    auto finish = [&](int t, double Rb, int eb, double c, int64_t j) {
        __builtin_nontemporal_store(t, T + j * mp + i);
        const double R = 0.0 + (double(t) + Rb * 0x1p-8);
        const int sc = (ea > kExpAllZero ? ea : 0) + (eb > kExpAllZero ? eb : 0) + (2 * kHeadroomBits - 12);
        double out = __dmul_rn(alpha, ldexp(R, sc));
        if (beta != 0.0) out = __dadd_rn(out, __dmul_rn(beta, c));
        if (i < m && j < n) __builtin_nontemporal_store(out, C + j * ldc + i);
    };
    // A wave holds every anti-diagonal of its part, so the sums stay in registers.  Rows of 16 lanes trade places so that 32 lanes
    // hold 32 neighbouring columns: a line of 128 bytes leaves in one store (64 bytes at a time cost 7 percent of the call).
    // VALU work bounds this part, so the chain runs on digits + 128: v = sum + 128 + (v before >> 8), the digit is its low byte less
    // 128.  The six least digits are 48 bits, exact in a double in any grouping, and are converted four and two at a time
    // (7936 x 7936 x 256: 724 us with a digit at a time, 675 so); the others follow one by one, each step rounded.  The exponents are
    // fetched first: behind stores a load is only there when those have been accepted.
    constexpr int EXACT = 6;
    int4 eb4[FB][2];
#pragma unroll
    for (int b = 0; b < FB; ++b)
#pragma unroll
        for (int u = 0; u < 2; ++u) eb4[b][u] = *reinterpret_cast<const int4*>(eB + row_of(b, u));
    const double unit = ldexp(1.0, -8 * (min(S - 1, EXACT) - 1));
#pragma unroll
    for (int b = 0; b < FB; ++b) {
        int v[2][4] = {}, top[2][4] = {};
        double Rb[2][4];
        uint32_t w[2][EXACT];
#pragma unroll
        for (int t = 0; t < MAX_S; ++t) {
            if (t < S) {
                int p[2][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const auto two = __builtin_amdgcn_permlane16_swap(uint32_t(acc[t / D][t % D][b][0][q]), uint32_t(acc[t / D][t % D][b][1][q]), false, false);
                    p[0][q] = int(two[0]);
                    p[1][q] = int(two[1]);
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (t == S - 1) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) top[u][q] = p[u][q] + (v[u][q] >> 8);
                        if (t < EXACT) w[u][t] = 0x80808080u;
                    } else if (t < MAX_S - 1) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[u][q] = p[u][q] + 128 + (v[u][q] >> 8);
                        const uint32_t digits = __builtin_amdgcn_perm(v[u][1], v[u][0], 0x0c0c0400u) | __builtin_amdgcn_perm(v[u][3], v[u][2], 0x04000c0cu);
                        __builtin_nontemporal_store(digits ^ 0x80808080u, reinterpret_cast<uint32_t*>(L + ((row_of(b, u) >> 2) * mp + i) * 4) + (S - 2 - t) * planeL);
                        if (t < EXACT) {
                            w[u][t] = digits;
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q) Rb[u][q] = double(int(digits >> (8 * q) & 255u) - 128) + Rb[u][q] * 0x1p-8;
                        }
                    }
                }
            } else if (t < EXACT) {
#pragma unroll
                for (int u = 0; u < 2; ++u) w[u][t] = 0x80808080u;
            }
            if (t != EXACT - 1) continue;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t lo01 = __builtin_amdgcn_perm(w[u][1], w[u][0], 0x05010400u), hi01 = __builtin_amdgcn_perm(w[u][1], w[u][0], 0x07030602u);
                const uint32_t lo23 = __builtin_amdgcn_perm(w[u][3], w[u][2], 0x05010400u), hi23 = __builtin_amdgcn_perm(w[u][3], w[u][2], 0x07030602u);
                const uint32_t x0[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                        __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    Rb[u][q] = (double(x0[q]) - 0x80808080p0) * unit;
                    if (S > 5) {
                        const uint32_t x1 = __builtin_amdgcn_perm(w[u][5], w[u][4], 0x0c0c0400u + 0x0101u * q);
                        Rb[u][q] = Rb[u][q] + (double(x1) - 0x8080p0) * (unit * 0x1p32);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int eb[4] = {eb4[b][u].x, eb4[b][u].y, eb4[b][u].z, eb4[b][u].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) finish(top[u][q], Rb[u][q], eb[q], cin[b][u][q], row_of(b, u) + q);
        }
    }
}

bool prepare_gemm_mid() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_mid_kernel<1>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kSmallLdsMax) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_mid_kernel<2>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kSmallLdsMax) == hipSuccess;
}

void launch_gemm_mid(hipStream_t st, const Workspace& w, const Problem& p, const LaunchPlan& lp, double alpha, double beta,
                     double* C, int64_t ldc, const Fallback& fb) {
    const int ntm = int((p.m + kMidTile - 1) / kMidTile), ntn = int((p.n + kMidTile - 1) / kMidTile);
    const int32_t* tile_S = p.tile_mode ? w.tile_S : nullptr;
    const dim3 grid(unsigned(ntm) * unsigned(ntn), 1, unsigned(p.batch.count));
    if (lp.mid_pair)
        hipLaunchKernelGGL(gemm_mid_kernel<1>, grid, dim3(256), kSmallLdsMax / 2, st, w.As, w.Bs, w.T, w.L, w.eA, w.eB, p.m, p.n, p.mp,
                           p.np, p.kp, ntm, ntn, lp.kt, kSmallLdsMax / 2, alpha, beta, C, ldc, w.rec, tile_S, p.batch, fb);
    else
        hipLaunchKernelGGL(gemm_mid_kernel<2>, grid, dim3(512), kSmallLdsMax, st, w.As, w.Bs, w.T, w.L, w.eA, w.eB, p.m, p.n, p.mp,
                           p.np, p.kp, ntm, ntn, lp.kt, kSmallLdsMax, alpha, beta, C, ldc, w.rec, tile_S, p.batch, fb);
}

}  // namespace oz
