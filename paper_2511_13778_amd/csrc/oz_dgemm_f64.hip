// Native FP64 GEMM on the FP64 matrix instruction: the path the guard falls back to.
// (paper: sections "Pre-processing and Safety Checks" and "Heuristic run time Selection":
//  Inf/NaN in the inputs, an exponent span beyond the available bits, or a slice count outside
//  the efficient range route the call to the native FP64 GEMM.)
//
//   C = alpha * op(A) * op(B) + beta * C,  ordinary floating-point accumulation over k.
//
// v_mfma_f64_16x16x4_f64; 128x128 tile per workgroup, 4 waves of 64x64 (4x4 MFMA tiles),
// K step 16 through double-buffered LDS.  op(B) feeds the row operand and op(A) the column
// operand so that the result's lane index runs along i and stores to column-major C coalesce.
// LDS banks: a tile row (one k) is 130 doubles = 260 dwords, i.e. 4 banks further per k.  The MFMA
// operand reads pair lane groups whose k differ by 8 (= 32 banks): MFMA number kk of a K step
// multiplies k = {kk, kk+8, kk+4, kk+12}, the same set for both operands; they are conflict-free.
// Stores of a k-contiguous operand (16 lanes on 16 different k, same row index) keep a two-way conflict
// on the 32-bank store path (the counters show exactly 4 extra cycles per store); other row lengths
// (129, 131, 133) give the same run time, so it is left as it is.
// Tile loads go through a buffer descriptor (no vector address arithmetic in the K loop); ragged sizes
// run the same loop with clamped rows and a short first K step; where the caller provides scratch memory, k may be
// split over several workgroups per tile (partial products added in a fixed order by dgemm_f64_reduce_kernel).  The tile edge
// (128, or 64 with waves of 32x32), the small tiles of dgemm_f64_direct_kernel and the number of parts are chosen together by
// an estimated time (choose_f64).
// Behind a guarded call it is launched on every call and returns at once unless the verdict selected it; calls that are recomposed
// on small tiles hold a direct tile in that launch instead where it is as fast (f64_folds).
#include <algorithm>

#include "oz_f64.h"

namespace oz {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kDPad = 2;                        // doubles of padding per LDS row (see the bank note above)
// The tile is T x T with T = 128 (the fast path) or T = 64 (outputs too small to give 128-tiles to
// every CU).  Per thread and operand a K step has T/16 elements; a wave owns (T/2) x (T/2).

// tile loader: 16 (k) x 128 (r) elements of an operand whose element (r, l) is at
// base[r*stride_r + l*stride_l]; out-of-range elements are zero.  8 values per thread.
template <bool ROWS_CONTIG, int T>
__device__ __forceinline__ void dg_load(double (&v)[T / 16], const double* __restrict__ X, int64_t stride_r,
                                        int64_t stride_l, int64_t r0, int64_t rows, int64_t l0, int64_t k) {
#pragma unroll
    for (int q = 0; q < T / 16; ++q) {
        int rr, ll;
        if (ROWS_CONTIG) { rr = threadIdx.x & (T - 1); ll = threadIdx.x / T + (256 / T) * q; }
        else { ll = threadIdx.x & 15; rr = (threadIdx.x >> 4) + 16 * q; }
        const int64_t r = r0 + rr, l = l0 + ll;
        // clamped address + select: the load is unconditional, so the loop stays branch-free
        const int64_t rc = r < rows ? r : rows - 1, lc = l < k ? l : k - 1;
        const double x = X[rc * stride_r + lc * stride_l];
        v[q] = (r < rows && l < k) ? x : 0.0;
    }
}
// interior tiles (no bounds to check): `u` is the wave-uniform address of the K step of this tile,
// `vo` this thread's byte offset inside it (fixed for the whole kernel), the elements of a thread are
// qstep_bytes apart.  The loads go through a buffer descriptor built on `u` (48-bit base in scalar
// registers, element distance as the instruction's scalar offset, `vo` as its 32-bit lane offset), so a
// K step has no vector address arithmetic at all.  Written as plain loads from `u + q*qstep + vo` the
// compiler keeps a 64-bit per-lane address for every element and rebuilds all of them with 64-bit
// vector adds in every K step: some forty vector instructions that compete with the MFMAs for the
// issue slot (measured at 8192^3: 15.36 ms with those, 14.70 ms with the descriptor form).
// The descriptor covers 4 GiB from `u` (raw buffer, no swizzle); the launcher sends operands whose
// offsets could exceed that to the bounds-checked path.
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
// PER_Q: every element of a thread has a lane offset of its own (ragged tiles of a k-contiguous
// operand, whose rows are clamped one by one); otherwise one lane offset and q * qstep_bytes.
template <int T, bool PER_Q>
__device__ __forceinline__ void dg_load_fast(double (&v)[T / 16], const double* u, const uint32_t (&vo)[PER_Q ? T / 16 : 1],
                                             uint32_t qstep_bytes) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(u), 0, -1, 0x00020000);
#pragma unroll
    for (int q = 0; q < T / 16; ++q) {
        const v2u x = __builtin_amdgcn_raw_buffer_load_b64(r, int(vo[PER_Q ? q : 0]),
                                                           PER_Q ? 0 : int(uint32_t(q) * qstep_bytes), 0);
        v[q] = __builtin_bit_cast(double, x);
    }
}
// lane offsets (bytes) of a thread's elements inside a K step of a tile that has `vr` (1..T) valid rows:
// rows past the last valid one are read from the last valid one instead (their products land in rows
// or columns of C that are never stored), so every address stays inside the operand
template <bool ROWS_CONTIG, int T, bool PER_Q>
__device__ __forceinline__ void dg_lane_offsets(uint32_t (&vo)[PER_Q ? T / 16 : 1], int64_t stride_r, int64_t stride_l,
                                                int vr) {
    if (ROWS_CONTIG) {
        const int rr = min(int(threadIdx.x & (T - 1)), vr - 1);
        vo[0] = uint32_t(rr * stride_r + (threadIdx.x / T) * stride_l) * 8u;
    } else {
#pragma unroll
        for (int q = 0; q < (PER_Q ? T / 16 : 1); ++q) {
            const int rr = min(int(threadIdx.x >> 4) + 16 * q, vr - 1);
            vo[q] = uint32_t(rr * stride_r + (threadIdx.x & 15) * stride_l) * 8u;
        }
    }
}

template <bool ROWS_CONTIG, int T>
__device__ __forceinline__ void dg_store(const double (&v)[T / 16], double* lds) {
#pragma unroll
    for (int q = 0; q < T / 16; ++q) {
        int rr, ll;
        if (ROWS_CONTIG) { rr = threadIdx.x & (T - 1); ll = threadIdx.x / T + (256 / T) * q; }
        else { ll = threadIdx.x & 15; rr = (threadIdx.x >> 4) + 16 * q; }
        lds[ll * (T + kDPad) + rr] = v[q];
    }
}

// MODE 0: m, n multiples of the tile and k of the K step.  MODE 1: any m, n, k: edge tiles clamp their
// rows in the (loop-invariant) lane offsets and k % 16 is taken as a short first K step, loaded by the
// bounds-checked loader once per tile; the K loop itself is the same as in MODE 0.  MODE 2: the
// bounds-checked loader with 64-bit indexing everywhere (operands whose leading dimension does not
// fit the 32-bit offsets of the fast loads, and k < 16, which has no full K step).
template <bool A_ROWS_CONTIG, bool B_ROWS_CONTIG, int MODE, int T>
__global__ __launch_bounds__(256, 2) void dgemm_f64_kernel(
    const Record* rec, KnownRecord known, int64_t m, int64_t n, int64_t k, double alpha, const double* __restrict__ A,
    int64_t a_sr, int64_t a_sl, const double* __restrict__ B, int64_t b_sr, int64_t b_sl, double beta,
    double* __restrict__ C, int64_t ldc, int ntm, int ntn, int zsplit, int64_t kpart, double* __restrict__ partial, Batch bt) {
    constexpr bool EDGE = MODE == 2;                       // bounds-checked loads in the K loop
    constexpr bool RAGGED = MODE != 0;                     // bounds-checked stores of C
    constexpr bool A_PER_Q = MODE == 1 && !A_ROWS_CONTIG, B_PER_Q = MODE == 1 && !B_ROWS_CONTIG;
    constexpr int kDLd = T + kDPad;      // LDS row length
    constexpr int WT = T / 2;            // wave tile
    constexpr int MT = WT / 16;          // MFMA tiles per wave and direction
    constexpr int EPT = T / 16;          // elements per thread, operand and K step
    __shared__ double At[2][kDK * kDLd];
    __shared__ double Bt[2][kDK * kDLd];
    f64_problem(bt, rec, A, B, C, partial);
    if (rec && !rec->res.fallback) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) write_known_record(known, bt, int(blockIdx.z));

    int ti, tj, z;
    f64_tile_of(int(blockIdx.x), ntm, ntn, zsplit, ti, tj, z);
    const int64_t i0 = int64_t(ti) * T, j0 = int64_t(tj) * T;
    // from here on A, B and k describe this unit's k range alone
    int64_t kb;
    f64_k_part(zsplit, z, kpart, k, kb);
    A += kb * a_sl;
    B += kb * b_sl;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = wave & 1, wj = wave >> 1;

    v4d acc[MT][MT];   // [fj][fi]
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};

    double va[EPT], vb[EPT];
    const double* ua = A + i0 * a_sr;   // wave-uniform: start of this tile's rows at k = 0
    const double* ub = B + j0 * b_sr;
    uint32_t voa[A_PER_Q ? EPT : 1], vob[B_PER_Q ? EPT : 1];
    dg_lane_offsets<A_ROWS_CONTIG, T, A_PER_Q>(voa, a_sr, a_sl, MODE == 1 ? int(min(int64_t(T), m - i0)) : T);
    dg_lane_offsets<B_ROWS_CONTIG, T, B_PER_Q>(vob, b_sr, b_sl, MODE == 1 ? int(min(int64_t(T), n - j0)) : T);
    const uint32_t qa = uint32_t(A_ROWS_CONTIG ? (256 / T) * a_sl : 16 * a_sr) * 8u;   // bytes between a thread's elements
    const uint32_t qb = uint32_t(B_ROWS_CONTIG ? (256 / T) * b_sl : 16 * b_sr) * 8u;
    // length of the first K step: k % 16 (a full step when that is zero); only MODE 1 has a short one
    const int kfirst = (MODE == 1 && (k & (kDK - 1))) ? int(k & (kDK - 1)) : kDK;
    if (EDGE || kfirst != kDK) {
        dg_load<A_ROWS_CONTIG, T>(va, A, a_sr, a_sl, i0, m, 0, EDGE ? k : kfirst);
        dg_load<B_ROWS_CONTIG, T>(vb, B, b_sr, b_sl, j0, n, 0, EDGE ? k : kfirst);
    } else {
        dg_load_fast<T, A_PER_Q>(va, ua, voa, qa);
        dg_load_fast<T, B_PER_Q>(vb, ub, vob, qb);
    }
    dg_store<A_ROWS_CONTIG, T>(va, At[0]);
    dg_store<B_ROWS_CONTIG, T>(vb, Bt[0]);
    __syncthreads();

    // fragments of MFMA step kk of the K step in LDS buffer `b`: lane group g = lane/16 multiplies
    // k = kk + 8*(g&1) + 4*(g>>1) (see the bank note at the top)
    const int g = lane >> 4;
    const int krow = (8 * (g & 1) + 4 * (g >> 1)) * kDLd;
    const int la_off = wi * WT + (lane & 15) + krow, lb_off = wj * WT + (lane & 15) + krow;
#define OZ_DG_READ(fa, fb, b, kk)                                                              \
    _Pragma("unroll") for (int f = 0; f < MT; ++f) {                                           \
        fa[f] = At[b][la_off + (kk) * kDLd + f * 16];                                          \
        fb[f] = Bt[b][lb_off + (kk) * kDLd + f * 16];                                          \
    }
#define OZ_DG_MFMA(fa, fb)                                                                     \
    _Pragma("unroll") for (int fj = 0; fj < MT; ++fj) _Pragma("unroll") for (int fi = 0; fi < MT; ++fi) \
        acc[fj][fi] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[fj], fa[fi], acc[fj][fi], 0, 0, 0);

    // Software pipeline of one K step (16 k = 4 MFMA steps of 16 MFMAs), arranged so that the matrix
    // unit always has work.  Interior tiles run it branch-free (the last K step loads its own tile
    // again and stores it where nobody reads it), which leaves one scheduling region per half, and
    // the group barriers below fix the interleave inside it:
    //   step 0: one global load of the next tile per MFMA          (fragments of step 1 are read first)
    //   step 1: MFMAs only                                         (fragments of step 2 are read first)
    //   step 2: one LDS store of the next tile per MFMA            (fragments of step 3 are read first)
    //   barrier: next tile visible, nobody reads this buffer any more (step 3 is in registers)
    //   step 3: MFMAs; they cover the barrier and the first fragment read of the next tile
    double xa[MT], xb[MT], ya[MT], yb[MT];
    int buf = 0;
    OZ_DG_READ(xa, xb, 0, 0);
    // K steps: [0, kfirst), then full steps of 16.  l0 is where the current step ends = the next one starts
    int64_t adv = kfirst;               // distance from the current step's start to the next one's
    for (int64_t l0 = kfirst;; l0 += kDK) {
        const bool have_next = l0 < k;
        if (EDGE) {
            if (have_next) {
                dg_load<A_ROWS_CONTIG, T>(va, A, a_sr, a_sl, i0, m, l0, k);
                dg_load<B_ROWS_CONTIG, T>(vb, B, b_sr, b_sl, j0, n, l0, k);
            }
        } else {
            // the last K step loads its own tile again (valid addresses, stored where nobody reads it)
            ua += have_next ? adv * a_sl : 0;
            ub += have_next ? adv * b_sl : 0;
            adv = kDK;
            dg_load_fast<T, A_PER_Q>(va, ua, voa, qa);
            dg_load_fast<T, B_PER_Q>(vb, ub, vob, qb);
        }
        OZ_DG_READ(ya, yb, buf, 1);
        OZ_DG_MFMA(xa, xb);
        OZ_DG_READ(xa, xb, buf, 2);
        OZ_DG_MFMA(ya, yb);
        OZ_DG_READ(ya, yb, buf, 3);
        if (!EDGE || have_next) {
            dg_store<A_ROWS_CONTIG, T>(va, At[buf ^ 1]);
            dg_store<B_ROWS_CONTIG, T>(vb, Bt[buf ^ 1]);
        }
        OZ_DG_MFMA(xa, xb);
        if (!EDGE && T == 128) {
            // masks: 0x008 MFMA, 0x020 global load, 0x100 LDS read, 0x200 LDS write
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            }
        }
        __syncthreads();
        buf ^= 1;
        if (!EDGE || have_next) { OZ_DG_READ(xa, xb, buf, 0); }
        OZ_DG_MFMA(ya, yb);
        if (!EDGE && T == 128) {
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
        }
        if (!have_next) break;
    }
#undef OZ_DG_READ
#undef OZ_DG_MFMA

    // result register r of tile (fj, fi): j = fj*16 + 4*r + lane/16, i = fi*16 + lane%16
    if (zsplit > 1) {
        // partial product of this part of the k range, at its place in a matrix of whole tiles
        const int64_t ldp = int64_t(ntm) * T;
        double* dst = partial + (int64_t(z) * ntn * T + j0) * ldp + i0;
#pragma unroll
        for (int fj = 0; fj < MT; ++fj)
#pragma unroll
            for (int fi = 0; fi < MT; ++fi)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    dst[(wj * WT + fj * 16 + 4 * r + (lane >> 4)) * ldp + wi * WT + fi * 16 + (lane & 15)] = acc[fj][fi][r];
        return;
    }
#pragma unroll
    for (int fj = 0; fj < MT; ++fj)
#pragma unroll
        for (int fi = 0; fi < MT; ++fi)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j = j0 + wj * WT + fj * 16 + 4 * r + (lane >> 4);
                const int64_t i = i0 + wi * WT + fi * 16 + (lane & 15);
                if (!RAGGED || (i < m && j < n)) {
                    double out = __dmul_rn(alpha, acc[fj][fi][r]);
                    if (beta != 0.0) out = __dadd_rn(out, __dmul_rn(beta, C[j * ldc + i]));
                    C[j * ldc + i] = out;
                }
            }
}

// C = alpha * (sum of the parts' partial products, in the order of the parts) + beta * C
__global__ __launch_bounds__(256) void dgemm_f64_reduce_kernel(const Record* rec, int64_t m, int64_t n, double alpha,
                                                               double beta, double* __restrict__ C, int64_t ldc, int zsplit,
                                                               const double* __restrict__ partial, int64_t ldp,
                                                               int64_t part_stride, int64_t j_first, Batch bt) {
    if (rec) rec = at_bytes(rec, bt.ws_at(blockIdx.z));
    partial = at_bytes(partial, bt.ws_at(blockIdx.z));
    C += blockIdx.z * bt.c;
    if (rec && !rec->res.fallback) return;
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int64_t j = j_first + blockIdx.y;
    if (i >= m) return;
    const double* src = partial + j * ldp + i;
    double sum = src[0];
    for (int z = 1; z < zsplit; ++z) sum = __dadd_rn(sum, src[z * part_stride]);
    double out = __dmul_rn(alpha, sum);
    if (beta != 0.0) out = __dadd_rn(out, __dmul_rn(beta, C[j * ldc + i]));
    C[j * ldc + i] = out;
}

void launch_dgemm_f64(hipStream_t st, const Record* rec, const KnownRecord& known, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                      double alpha, const double* A, int64_t lda, const double* B, int64_t ldb, double beta,
                      double* C, int64_t ldc, int num_cu, const Batch& batch, void* scratch, size_t scratch_bytes) {
    // op(A)(i,l): N -> A[i + l*lda] (rows contiguous), T -> A[l + i*lda]
    // op(B)(l,j): N -> B[l + j*ldb] (k contiguous),    T -> B[j + l*ldb] (rows contiguous)
    const F64Call c{rec, known, m, n, k, alpha, A, ta ? lda : 1, ta ? 1 : lda, B, tb ? 1 : ldb, tb ? ldb : 1, beta, C, ldc, !ta, tb, batch};
    // the fast loads keep every offset inside a K step of a tile in 32 bits; where they may not fit, the bounds-checked path indexes in 64
    const bool wide = wide_offsets(m, n, k, lda > ldb ? lda : ldb);
    F64Plan p{};
    if (!wide) p = choose_f64(f64_size(m, n, k, batch.count, rec != nullptr, beta != 0.0, !ta, lda, tb, ldb), num_cu, scratch ? scratch_bytes : 0);
    if (p.ti == 0) {
        const int T = ((m + 127) / 128) * ((n + 127) / 128) < num_cu ? 64 : 128;
        p = F64Plan{false, T, T, int((m + T - 1) / T), int((n + T - 1) / T), 1, 0, nullptr};
    }
    p.partial = static_cast<double*>(scratch);
    if (p.direct) {
        launch_dgemm_f64_direct(st, c, p);
    } else {
        const bool ac = c.a_rows, bc = c.b_rows;
        const dim3 grid(unsigned(p.ntm) * unsigned(p.ntn) * unsigned(p.zsplit), 1, unsigned(batch.count)), block(256);
        const int mode = f64_mode(wide, m, n, k, p.ti, p.tj);
#define OZ_DG_M(AC, BC, MODE, TT)                                                                              \
    hipLaunchKernelGGL((dgemm_f64_kernel<AC, BC, MODE, TT>), grid, block, 0, st, rec, known, m, n, k, alpha, A, c.a_sr, \
                       c.a_sl, B, c.b_sr, c.b_sl, beta, C, ldc, p.ntm, p.ntn, p.zsplit, p.kpart, p.partial, batch)
#define OZ_DG_T(AC, BC, TT)                                                                                    \
    {                                                                                                          \
        if (mode == 2) OZ_DG_M(AC, BC, 2, TT);                                                                 \
        else if (mode == 1) OZ_DG_M(AC, BC, 1, TT);                                                            \
        else OZ_DG_M(AC, BC, 0, TT);                                                                           \
    }
#define OZ_DG(AC, BC)                                                                                          \
    {                                                                                                          \
        if (p.ti == 64) OZ_DG_T(AC, BC, 64) else OZ_DG_T(AC, BC, 128)                                          \
    }
        if (ac && bc) OZ_DG(true, true)
        else if (ac && !bc) OZ_DG(true, false)
        else if (!ac && bc) OZ_DG(false, true)
        else OZ_DG(false, false)
#undef OZ_DG_T
#undef OZ_DG_M
#undef OZ_DG
    }
    if (p.zsplit > 1) {
        const unsigned gx = unsigned((m + 255) / 256);
        const int64_t ldp = int64_t(p.ntm) * p.ti, part_stride = ldp * p.ntn * p.tj;
        for (int64_t j = 0; j < n; j += 65535) {
            const dim3 rgrid(gx, unsigned(n - j < 65535 ? n - j : 65535), unsigned(batch.count));
            hipLaunchKernelGGL(dgemm_f64_reduce_kernel, rgrid, dim3(256), 0, st, rec, m, n, alpha, beta, C, ldc, p.zsplit,
                               p.partial, ldp, part_stride, j, batch);
        }
    }
}

}  // namespace oz
