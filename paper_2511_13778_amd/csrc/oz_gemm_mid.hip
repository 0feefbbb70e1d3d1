// Slice-pair GEMMs and FP64 recomposition in one kernel on 64 x 64 tiles of C: what gemm_i8_kernel and recompose_kernel compute,
// for calls whose k is short beside the size of C, and for mid-sized ones.
// (paper: section "FP64 Emulation on Low-Precision Units".)
//
// With units of 128 x 128 such a call spends its time around the products: a unit of a short k is mostly its start and its two or
// three ends of groups of anti-diagonals, nothing runs beside them (one wave per SIMD, all accumulators taken), the digits written
// are read again, and less than a round of units leaves CUs idle.  Here all S slices of a 64 of k lie in LDS (4 KB each), a wave
// owns a quadrant of 32 x 32 and keeps anti-diagonals in groups of four (a step reads one slice of A and one of B and multiplies
// it with the window of four, as in gemm_i8_kernel: 2 LDS reads per 8 MFMAs), so k is walked once, and carry chain, powers of two,
// alpha and beta follow in the same launch.
//   SETS = 1   4 waves, up to 8 slices, 80 KB: two workgroups to a CU, one ends or loads while the other multiplies
//   SETS = 2   8 waves (two sets share the groups), up to 16 slices, all of the LDS: more than one stage up to 10 slices
// Digits, leading words and C are 26 bytes per element, read and written once and streamed past L2, where the slices of the next tiles
// live (plain stores, which drive those out, cost 85 us of 690 at 7936 x 7936 x 256).  What bounds it at a short k is the end of a tile:
// memory, and the integer work of the carry chain, which the other workgroup's products only partly cover (7936 x 7936, seven
// slices: 270 us plus 83 per 64 of k); at a long one LDS, from which a quadrant reads 42 KB per 64 of k and seven slices beside the 56 KB
// that arrive (1750 cycles of 128 B for 1792 of MFMA).  Stages of 32 of k, twice as deep, gain 5 percent where they save half a stage (k = 200)
// and lose 5 at 512; the first reads of a group during the group before gain nothing; nor do wave priorities.
// Measured, whole calls, against units: 7936x7936x256 814 -> 600 us, 1000^3 (seven slices, no guards) 86 -> 51; 16 problems of 512^3, which
// also share their launches, 540 -> 168.  The sums of one set through LDS and plain stores, before: 690, 53, 174.
#include "oz_f64_direct.h"
#include "oz_gemm_device.h"

namespace oz {

constexpr int kMidSlice = kMidTile * kBK;                   // bytes of one slice of one operand for a 64 of k: [k chunk][row][16 B]
constexpr int kMidRow = kMidTile + 4;                       // words between rows of the sums
constexpr int kMidPlane = kMidTile / 2 * kMidRow * 4;       // bytes per anti-diagonal of half a tile's sums
static_assert(kMidTile == 64 && kBK == 64, "a transfer moves one k chunk of 64 rows, a wave owns a quadrant of 32 x 32");
static_assert(kMidMaxSlices * 2 * kMidSlice <= kSmallLdsMax && kMidMaxSlices * kMidPlane <= kSmallLdsMax, "one stage must fit");
static_assert(kMidPairSlices * 2 * kMidSlice <= kSmallLdsMax / 2, "one of two workgroups");

template <int N>
struct MidInt { static constexpr int v = N; };

template <int SETS>
__global__ __launch_bounds__(256 * SETS, 2) void gemm_mid_kernel(
    const int8_t* __restrict__ As, const int8_t* __restrict__ Bs, int32_t* __restrict__ T, int8_t* __restrict__ L,
    const int32_t* __restrict__ eA, const int32_t* __restrict__ eB, int64_t m, int64_t n, int64_t mp, int64_t np, int64_t kp,
    int ntm, int ntn, int kt_total, int lds_bytes, double alpha, double beta, double* __restrict__ C, int64_t ldc, const Record* rec,
    const int32_t* __restrict__ tile_S, Batch bt, Fallback fb) {
    constexpr int WAVES = 4 * SETS, D = 4;
    constexpr int GROUPS = (SETS == 1 ? kMidPairSlices : kMidMaxSlices) / D / SETS;     // of four anti-diagonals per wave
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
    const int set = wave >> 2, qi = wave & 1, qj = (wave >> 1) & 1;

    // ---- elements this thread finishes.  One set: column i of its quadrant, rows of four j.
    // Two sets: column i, in either half of the tile's rows 8 / WAVES times four j.
    constexpr int QUADS = 8 / WAVES;
    const int64_t i = SETS == 1 ? i0 + qi * 32 + (lane & 31) : i0 + lane;
    auto row_of = [&](int h, int u) -> int64_t { return SETS == 1 ? j0 + qj * 32 + h * 16 + (lane >> 5) * 8 + u * 4 : j0 + h * 32 + (u * WAVES + wave) * 4; };
    double cin[2][QUADS][4];
    if (beta != 0.0) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < QUADS; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    cin[h][u][q] = C[min(row_of(h, u) + q, n - 1) * ldc + min(i, m - 1)];
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

    // ---- anti-diagonals in groups of four side by side (as in gemm_i8_kernel); set x takes groups x, x + SETS, ...
    v4i acc[GROUPS][D][2][2];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int j = 0; j < D; ++j)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) acc[g][j][b][a] = v4i{0, 0, 0, 0};
    const uint32_t rd = uint32_t(lane >> 4) * 1024u + uint32_t(lane & 15) * 16u;
    const uint32_t rdA = rd + uint32_t(qi) * 512u, rdB = rd + uint32_t(qj) * 512u + uint32_t(S) * kMidSlice;
    int stage = 0;
    for (int kt = 0; kt < kt_total; ++kt) {
        wait_transfers((issued - 1 - kt) * pieces);
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): this wave's reads of the stage before have returned
        asm volatile("s_barrier" ::: "memory");
        const int limit = min(min(kt + stages, issued + 1), kt_total);
        issue_next(limit);
        const uint8_t* const atA = lds + uint32_t(stage) * stage_bytes + rdA;
        const uint8_t* const atB = lds + uint32_t(stage) * stage_bytes + rdB;
#pragma unroll
        for (int gg = 0; gg < GROUPS; ++gg) {
            const int d_hi = S - 1 - D * (set + SETS * gg);
            if (d_hi < 0) continue;
            v4i fa[2][2], fb[4][2];
            auto read_a = [&](int par, int s) {
#pragma unroll
                for (int f = 0; f < 2; ++f) fa[par][f] = *reinterpret_cast<const v4i*>(atA + s * kMidSlice + f * 256);
            };
            auto read_b = [&](int slot, int t) {
#pragma unroll
                for (int f = 0; f < 2; ++f) fb[slot][f] = *reinterpret_cast<const v4i*>(atB + t * kMidSlice + f * 256);
            };
            // step r multiplies A_(d_hi - r) with B_(r - j), j = 0 .. 3; slice t of B lies in slot t mod 4
            read_a(0, 0);
            read_a(1, 0);
#pragma unroll
            for (int sl = 0; sl < 4; ++sl) read_b(sl, max(d_hi - ((d_hi - sl) & 3), 0));
            auto step = [&](auto VV, auto NN, int r) {
                constexpr int v = decltype(VV)::v, sets = decltype(NN)::v;
                if (r > d_hi) return;
                if (r > 0) read_a((v + 1) & 1, d_hi - r + 1);
#pragma unroll
                for (int j = 0; j < sets; ++j) {
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int a = 0; a < 2; ++a)
                            acc[gg][j][b][a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[(v - j) & 3][b], fa[v & 1][a], acc[gg][j][b][a], 0, 0, 0);
                    if (j == 0 && sets == 4 && r >= 4) read_b(v, r - 4);
                }
            };
            for (int rb = d_hi & ~3; rb > 0; rb -= 4) {
                step(MidInt<3>{}, MidInt<4>{}, rb + 3);
                step(MidInt<2>{}, MidInt<4>{}, rb + 2);
                step(MidInt<1>{}, MidInt<4>{}, rb + 1);
                step(MidInt<0>{}, MidInt<4>{}, rb);
            }
            step(MidInt<3>{}, MidInt<4>{}, 3);
            step(MidInt<2>{}, MidInt<3>{}, 2);
            step(MidInt<1>{}, MidInt<2>{}, 1);
            step(MidInt<0>{}, MidInt<1>{}, 0);
        }
        if (stages == 1) {
            __builtin_amdgcn_s_waitcnt(0xC07F);
            asm volatile("s_barrier" ::: "memory");
            issue_next(kt_total);
        }
        stage = stage + 1 == stages ? 0 : stage + 1;
    }

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
    if constexpr (SETS == 1) {
        // A wave holds every anti-diagonal of its quadrant, so the sums stay in registers.  Rows of 16 lanes trade places so that 32 lanes
        // hold 32 neighbouring columns: a line of 128 bytes leaves in one store (64 bytes at a time cost 7 percent of the call).
        // VALU work bounds this part, so the chain runs on digits + 128: v = sum + 128 + (v before >> 8), the digit is its low byte less
        // 128.  The six least digits are 48 bits, exact in a double in any grouping, and are converted four and two at a time
        // (7936 x 7936 x 256: 724 us with a digit at a time, 675 so).  The exponents are fetched first: behind stores a load is only there
        // when those have been accepted.
        int4 eb4[2][QUADS];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int u = 0; u < QUADS; ++u) eb4[b][u] = *reinterpret_cast<const int4*>(eB + row_of(b, u));
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            int v[2][4] = {}, top[2][4] = {};
            uint32_t w[2][kMidPairSlices - 1];
#pragma unroll
            for (int t = 0; t < kMidPairSlices; ++t) {
                if (t > S - 1) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (t < kMidPairSlices - 1) w[u][t] = 0x80808080u;
                    continue;
                }
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
                        if (t < kMidPairSlices - 1) w[u][t] = 0x80808080u;
                    } else if (t < kMidPairSlices - 1) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[u][q] = p[u][q] + 128 + (v[u][q] >> 8);
                        w[u][t] = __builtin_amdgcn_perm(v[u][1], v[u][0], 0x0c0c0400u) | __builtin_amdgcn_perm(v[u][3], v[u][2], 0x04000c0cu);
                        __builtin_nontemporal_store(w[u][t] ^ 0x80808080u, reinterpret_cast<uint32_t*>(L + ((row_of(b, u) >> 2) * mp + i) * 4) + (S - 2 - t) * planeL);
                    }
                }
            }
            const double unit = ldexp(1.0, -8 * (min(S - 1, 6) - 1));
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t lo01 = __builtin_amdgcn_perm(w[u][1], w[u][0], 0x05010400u), hi01 = __builtin_amdgcn_perm(w[u][1], w[u][0], 0x07030602u);
                const uint32_t lo23 = __builtin_amdgcn_perm(w[u][3], w[u][2], 0x05010400u), hi23 = __builtin_amdgcn_perm(w[u][3], w[u][2], 0x07030602u);
                const uint32_t x0[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                        __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
                const int eb[4] = {eb4[b][u].x, eb4[b][u].y, eb4[b][u].z, eb4[b][u].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    double Rb = (double(x0[q]) - 0x80808080p0) * unit;
                    if (S > 5) {
                        const uint32_t x1 = __builtin_amdgcn_perm(w[u][5], w[u][4], 0x0c0c0400u + 0x0101u * q);
                        Rb = Rb + (double(x1) - 0x8080p0) * (unit * 0x1p32);
                        if (S > 7) Rb = double(int(w[u][6] >> (8 * q) & 255u) - 128) + Rb * 0x1p-8;
                    }
                    finish(top[u][q], Rb, eb[q], cin[b][u][q], row_of(b, u) + q);
                }
            }
        }
    } else {
        // half by half of the tile's columns j the sums of both sets meet in LDS
        int32_t* const sums = reinterpret_cast<int32_t*>(lds);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            __syncthreads();
            if (qj == h) {
#pragma unroll
                for (int gg = 0; gg < GROUPS; ++gg)
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        const int d = S - 1 - D * (set + SETS * gg) - j;
                        if (d < 0) continue;
#pragma unroll
                        for (int b = 0; b < 2; ++b)
#pragma unroll
                            for (int a = 0; a < 2; ++a)
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    sums[d * (kMidPlane / 4) + (b * 16 + 4 * (lane >> 4) + r) * kMidRow + qi * 32 + a * 16 + (lane & 15)] =
                                        acc[gg][j][b][a][r];
                    }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < QUADS; ++u) {
                const int64_t j = row_of(h, u);
                const int32_t* mine = sums + (u * WAVES + wave) * 4 * kMidRow + lane;
                uint32_t* const lw = reinterpret_cast<uint32_t*>(L + ((j >> 2) * mp + i) * 4);
                int carry[4] = {0, 0, 0, 0};
                double Rb[4] = {0.0, 0.0, 0.0, 0.0};
                int p[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) p[q] = mine[(S - 1) * (kMidPlane / 4) + q * kMidRow];
                for (int d = S - 1; d >= 1; --d) {
                    int next[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) next[q] = mine[(d - 1) * (kMidPlane / 4) + q * kMidRow];
                    uint32_t w = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int v = p[q] + carry[q];
                        carry[q] = (v + 128) >> 8;
                        w |= (uint32_t(v) & 255u) << (8 * q);
                        Rb[q] = double((v << 24) >> 24) + Rb[q] * 0x1p-8;
                        p[q] = next[q];
                    }
                    __builtin_nontemporal_store(w, lw + (d - 1) * planeL);
                }
                const int4 e4 = *reinterpret_cast<const int4*>(eB + j);
                const int eb[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) finish(p[q] + carry[q], Rb[q], eb[q], cin[h][u][q], j + q);
            }
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
