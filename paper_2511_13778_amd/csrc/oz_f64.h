// What the kernels of the native FP64 GEMM share: the call, how it is cut into workgroups, and which of them a workgroup is.
#pragma once

#include "oz_f64_plan.h"

namespace oz {

struct F64Call {
    const Record* rec;     // nullptr: run unconditionally
    KnownRecord known;
    int64_t m, n, k;
    double alpha;
    const double* A;       // element (i, l) of op(A) at A[i * a_sr + l * a_sl]
    int64_t a_sr, a_sl;
    const double* B;       // element (l, j) of op(B) at B[j * b_sr + l * b_sl]
    int64_t b_sr, b_sl;
    double beta;
    double* C;
    int64_t ldc;
    bool a_rows, b_rows;   // rows (not k) contiguous
    Batch batch;
};

// Workgroup ids are dealt round-robin to the 8 XCDs; each XCD gets a contiguous range of a tile order in which 64 consecutive
// tiles form an 8 x 8 block, so they share 16 panels in that XCD's L2.  With a k split a work unit is (tile, part of k),
// ordered part by part.
__device__ __forceinline__ void f64_tile_of(int id, int ntm, int ntn, int zsplit, int& ti, int& tj, int& z) {
    const int tiles = ntm * ntn, total = tiles * zsplit;
    const int xcd = id & 7, slot = id >> 3;
    const int per = total >> 3, rem = total & 7;
    const int unit = xcd * per + min(xcd, rem) + slot;
    z = unit / tiles;
    const int lin = unit - z * tiles;
    constexpr int GW = 8;
    const int panel = lin / (GW * ntm);
    const int in_panel = lin - panel * GW * ntm;
    const int w = min(GW, ntn - panel * GW);
    ti = in_panel / w;
    tj = panel * GW + in_panel % w;
}

// part z of k: [kb, kb + k) of the whole.  Part 0 is [0, k - (zsplit-1)*kpart) and carries k mod 16, the others have kpart (a
// multiple of 16) each
__device__ __forceinline__ void f64_k_part(int zsplit, int z, int64_t kpart, int64_t& k, int64_t& kb) {
    kb = 0;
    if (zsplit > 1) {
        const int64_t k0 = k - int64_t(zsplit - 1) * kpart;
        kb = z == 0 ? 0 : k0 + int64_t(z - 1) * kpart;
        k = z == 0 ? k0 : kpart;
    }
}

// problem p = blockIdx.z of a batch
template <class Rec, class In, class Out>
__device__ __forceinline__ void f64_problem(const Batch& bt, Rec& rec, In& A, In& B, Out& C, Out& partial) {
    const int p = int(blockIdx.z);
    const int64_t ws = bt.ws_at(p);        // not used by problems beyond the workspaces: no verdict to read, no partial products
    if (rec) rec = at_bytes(rec, ws);
    A += bt.a_at(p);
    B += bt.b_at(p);
    C += p * bt.c;
    partial = at_bytes(partial, ws);
}

void launch_dgemm_f64_direct(hipStream_t st, const F64Call& c, const F64Plan& p);

}  // namespace oz
