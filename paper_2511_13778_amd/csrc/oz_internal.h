// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ozdgemm.h"

namespace oz {

// ---- constants of the method -----------------------------------------------------------
constexpr int kHeadroomBits = 1;      // spare bit in the leading digit: |X| < 2^(8S-2)
constexpr int kMaxSlices = 26;        // 200 mantissa bits
constexpr int kEscCap = 4096;         // reported ESC is clamped to this
constexpr int kDefaultEscBlock = 64;
constexpr int64_t kMaxRows = int64_t(1) << 22;   // largest m, n
constexpr int64_t kMaxK = int64_t(1) << 21;      // largest k
constexpr int64_t kMaxMnk = int64_t(1) << 52;    // largest m*n*k: the cost model multiplies 2mnk by up to 351 pairs in int64

// Exponents are kept as int16 in the block tables.  Real exponents lie in [-1074, 1023].
// kExpZeroInMin: Min of a block that holds a zero (exp(0) = -infinity).
// kExpAllZero  : Max and Min of a block without any non-zero entry.
// Sums of two table entries classify a candidate: >= -4096 a real exponent sum,
// [-10000, -4096) "no information", < -10000 "this block contributes nothing to the product".
constexpr int kExpZeroInMin = -6144;
constexpr int kExpAllZero = -12288;
constexpr int kExpInfNan = 1024;      // exponent of Inf and NaN: their field is all ones, that of a number at most 1023 + 1023
constexpr int kSumRealFloor = -4096;
constexpr int kSumDeadBelow = -10000;

// ---- tiling constants shared between kernels and the workspace layout --------------------
constexpr int kRowPad = 256;          // rows of the slice panels are padded to this
constexpr int kKPad = 128;            // k is padded to this (a multiple of the slice GEMM's step of kBK)
constexpr int kTile = 256;            // edge of the blocks of C that can take their own slice count (kRowPad is a multiple):
                                      // two by two units of gemm_i8_kernel, one workgroup's share in gemm_i8_few_kernel

// ---- a scan whose workgroups hold all of k (scan_exponents_kernel) ----------------------
constexpr int kOnceRows = 16;         // rows of a workgroup
constexpr int kScanOnceParts = 128;   // most workgroups
constexpr int kScanOnceBlocks = 32;   // most ESC blocks

// ---- encoding of the block tables for the ESC on the matrix unit (oz_esc.hip) --------------
constexpr int kEncScale = 5;     // exponent units per bit of span; 16 equal terms stay below 2^5
constexpr int kEncBias = 61;     // 2*61 + 4 < 128: a chunk sum cannot overflow FP32
constexpr int kEncRange = 37;    // 5*(-37) + 61 >= -126: smallest encodable entry (BF16 normal)
constexpr int kEncChunk = 16;    // inner steps per MFMA (K of v_mfma_f32_32x32x16_bf16)
// BF16 bits of 2^(5 (x - e) + 61), 0 for what the code does not hold
__device__ __forceinline__ uint32_t enc_bits(int x, int e) {
    const int d = x - e;
    return x > kSumRealFloor / 2 && d >= -kEncRange && d <= 0 ? uint32_t(kEncScale * d + kEncBias + 127) << 7 : 0u;
}

// ---- device-resident control record ---------------------------------------------------
struct Record {
    int32_t infnan;        // cleared by the scan, set by exponents_kernel for a row or column exponent of kExpInfNan
    int32_t span_max;      // max_ij (eA_i + eB_j - zt_ij), set by the ESC kernels (atomicMax)
    int32_t esc_done;      // workgroups of the ESC kernel that have left their span (atomicAdd): the last one gives the verdict
    int32_t pad_;
    int32_t tile_sync[8];  // per-XCD arrival counters of the slice GEMM's workgroups
    oz_result_t res;       // the verdict, read by every later kernel
    uint8_t infnan_part[kScanOnceParts];   // of a call that is scanned in one launch: the flag of every workgroup, instead of infnan
};

// A record that the host knows before anything runs (no guards, or the native GEMM chosen by the cost model), written
// by the first kernel of the call.  rec == nullptr: nothing to write.
struct KnownRecord {
    Record* rec;
    oz_result_t* user;     // may be nullptr
    oz_result_t value;
};

// Problems of one shape that share every launch of a call: problem p = blockIdx.z finds its workspace p * ws bytes further on, its
// operands and result p * a, b, c elements.  A chain of dependent launches costs 4 to 5 us a launch, whatever it computes,
// so several small problems take little more than one.
struct Batch {
    int32_t count = 1;
    int32_t four = 0;      // the four real products of a complex one: A of problem p is number p & 1, B number (p & 1) ^ (p >> 1)
    int32_t lanes = 1;     // workspaces; only native products without a k split, which need none, may be more
    int32_t pad_ = 0;
    int64_t ws = 0, a = 0, b = 0, c = 0;
    __device__ int64_t ws_at(int p) const { return p * ws; }
    __device__ int64_t a_at(int p) const { return (four ? p & 1 : p) * a; }
    __device__ int64_t b_at(int p) const { return (four ? (p & 1) ^ (p >> 1) : p) * b; }
};
template <class T>
__device__ inline T* at_bytes(T* x, int64_t bytes) {
    return (T*)((const char*)x + bytes);
}
__device__ inline void write_known_record(const KnownRecord& k, const Batch& bt, int p) {
    if (!k.rec) return;
    if (p < bt.lanes) at_bytes(k.rec, bt.ws_at(p))->res = k.value;
    if (k.user) k.user[p] = k.value;
}

struct Problem {
    int64_t m, n, k;
    int64_t mp, np, kp;    // padded sizes
    int32_t s_cap;         // slice planes the workspace holds
    int32_t s_min;         // fewest slices an emulated block of C can come out with
    int32_t nkb;           // number of k-blocks (int32 accumulator headroom)
    int64_t kblk;          // k-block length (multiple of kKPad)
    int32_t esc_block;     // b
    int32_t G;             // ceil(k / b)
    int32_t num_cu;        // compute units of the device
    int32_t tile_mode;     // 1: every kTile x kTile block of C takes its own slice count (OZ_DYNAMIC + tile_slices)
    Batch batch;           // problems that share the launches
    int32_t raw_slots;     // kTile blocks the raw buffer holds, four units each (a launch of fewer units than CUs may split k)
};

struct Workspace {
    Record* rec;
    int32_t* eA;           // [mp]
    int32_t* eB;           // [np]
    int16_t* U;            // [2G][mp]  h <  G: Max exponent of block h of row i of op(A)
                           //           h >= G: Min exponent of block h-G
    int16_t* V;            // [2G][np]  h <  G: Min exponent of block h of column j of op(B)
                           //           h >= G: Max exponent of block h-G
    uint16_t* EU;          // [ceil(2G/32)*4][mp][8] BF16 encoding of U relative to eA
    uint16_t* EV;          // [ceil(2G/32)*4][np][8] BF16 encoding of V relative to eB
    int8_t* As;            // [s_cap][kp/16][mp][16]
    int8_t* Bs;            // [s_cap][kp/16][np][16]
    // aggregated anti-diagonal sums of a k-block: Z = sum_d P_d 256^(S-1-d) = T * 256^(S-1) + sum_{d>=1} L_d 256^(S-1-d)
    int32_t* T;            // [nkb][np][mp]                   leading word (anti-diagonal 0 plus the carry from below)
    int8_t* L;             // [nkb][s_cap-1][np/4][mp][4]     balanced digit of anti-diagonal d >= 1 at plane d-1; four
                           //                                 consecutive j of one i share a dword
    int32_t* raw;          // [nkb][s_cap][raw_slots][kTile][kTile]  what the parts of a k split leave (see KSplit), in
                           //                                 slots of one 128 x 128 unit
    int32_t* tile_span;    // [np/kTile][mp/kTile] largest coarsened span of the block's dot products (atomicMax)
    int32_t* tile_S;       // [np/kTile][mp/kTile] slice count of the block (per-tile mode), followed by as many
                           // entries again: the order in which the slice GEMM deals the tiles to its workgroups

    // largest exponent of every row in each group of blocks of the scan: in the slice planes, not yet written then and
    // always larger (two bytes per row and at least one block of 16 k)
    int16_t* group_max_a() const { return reinterpret_cast<int16_t*>(As); }
    int16_t* group_max_b() const { return reinterpret_cast<int16_t*>(Bs); }
};

// ---- geometry of the slice GEMM's launches, shared with the recomposition ----------------
constexpr int kUnit = 128;            // edge of the unit of C a workgroup of the slice GEMM owns (four per kTile block)
constexpr int kBK = 64;               // k per step (kKPad is a multiple)

// What a launch of the slice GEMM covers.
struct GemmGrid {
    int nti, ntj;      // kTile x kTile blocks of the padded C
    int um, un;        // units with at least one row / column of C
    int begin, count;  // plain order: units [begin, begin + count); per-block order: as many positions of the order table
    int kt_total;      // 64s of k, the last one possibly part padding
    int zsplit;        // parts of the k range per unit
    int nkb_part;      // k-blocks a part's slot has room for (parts other than the first)
    int full_chip;     // 8 XCDs of 32 CUs: the in-step waits make sense
    int persistent;    // a workgroup takes several units, and every unit has at least kMinUnitItems items
};

// How the whole product was split along k, for the recomposition to put together: not at all (the planes T / L are
// complete), into parts that hold their own aggregated sums, or with integer atomics into raw sums.  kDone: nothing is left to
// do, C is written.
enum class KSplit { kNone, kParts, kAtomic, kDone };
struct SplitPlan {
    KSplit kind;
    GemmGrid g;        // of the one launch that covered the product
    int raw_units;     // 128 x 128 slots per plane of the raw buffer
};

// Where part z > 0 of unit `local` of a launch leaves its aggregated sums: a slot of the raw buffer holding, per
// k-block the part touches, T [128 j][128 i] int32 and L [s_cap-1][32][128 i][4 j] int8 of the unit alone.
__host__ __device__ inline int64_t part_slot_bytes(int s_cap) { return int64_t(kUnit) * kUnit * (4 + (s_cap - 1)); }

// Position `lin` of the tile order -> tile coordinates, and back: panels of 8 tile columns, inside a panel row by row,
// so 32 consecutive tiles form a 4 (i) x 8 (j) block.
constexpr int kPanelTiles = 8;
__host__ __device__ inline void lin_to_tile(int lin, int nti, int ntj, int& ti, int& tj) {
    const int panel = lin / (kPanelTiles * nti);
    const int in_panel = lin - panel * kPanelTiles * nti;
    const int w = ntj - panel * kPanelTiles < kPanelTiles ? ntj - panel * kPanelTiles : kPanelTiles;
    ti = in_panel / w;
    tj = panel * kPanelTiles + in_panel % w;
}
__host__ __device__ inline int tile_to_lin(int ti, int tj, int nti, int ntj) {
    const int panel = tj / kPanelTiles;
    const int w = ntj - panel * kPanelTiles < kPanelTiles ? ntj - panel * kPanelTiles : kPanelTiles;
    return panel * kPanelTiles * nti + ti * w + tj % kPanelTiles;
}

// k split: first 64 of k of part z, and the parts that have k in k-block kb
__host__ __device__ inline int part_first(int kt_total, int zsplit, int z) { return int(int64_t(kt_total) * z / zsplit); }
__host__ __device__ inline void parts_of_block(int kt_total, int kt_per_block, int zsplit, int kb, int& z_lo, int& z_hi) {
    z_lo = 0;
    while (z_lo + 1 < zsplit && part_first(kt_total, zsplit, z_lo + 1) <= kb * kt_per_block) ++z_lo;
    z_hi = z_lo;
    while (z_hi + 1 < zsplit && part_first(kt_total, zsplit, z_hi + 1) < (kb + 1) * kt_per_block) ++z_hi;
}

// Whether what recomposition reads and writes (leading words, digits, C) is more than the 256 MB Infinity Cache: then C and, with few slices,
// the leading words are streamed past it (8192 x 8192 x 2048 with two slices 719 -> 653 us, 6144 x 6144 x 1024 with seven 1040 -> 1015); what fits
// there the next kernel or the next call's beta C finds (3000^3 with one slice 127 us, streamed 131).
inline bool results_stream(const Problem& p) { return double(p.m) * double(p.n) * p.batch.count * (11 + p.s_cap) > 256e6; }

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// k-range one int32 accumulator can take: |digit product| <= 2^14, an anti-diagonal sums at most
// S*kblk of them, and the aggregation adds a carry below 2^23 from the less significant
// anti-diagonals: S*kblk*2^14 + 2^23 <= 2^31 - 1.  Multiple of 256.
__host__ __device__ inline int64_t k_block_length(int S) {
    return ((int64_t(1) << 17) - (int64_t(1) << 9) - 1) / S / 256 * 256;
}

// ---- geometry of the scan's launches --------------------------------------------------
constexpr int kScanBlocksPerWg = 4;    // ESC blocks a workgroup covers (one, at 8192^3: scan and exponents 267 us against 249)
constexpr int64_t kMaxGridThreads = (int64_t(1) << 32) - 1;   // of one launch along x

// Workgroups of the scan: row blocks of op(A), then of op(B), for `groups` groups of `per` ESC blocks along k.  One launch
// takes `slab` groups: all of them, unless a launch would have too many threads (k-contiguous operands of 2^34 elements
// with ESC blocks of 16).
struct ScanGrid {
    int64_t row_blocks_a, row_blocks_b;
    int per;
    bool k64;
    int64_t groups, slab;
};
// rows_contig: stride_r == 1.  A workgroup of 256 threads covers 64 rows of such an operand, and of one with k contiguous where it reads
// 64 k of a row per load (k64), otherwise 16.  k64: ESC blocks that are one 64 of k, and longer ones, through which a wave then walks, where there are
// workgroups of 64 rows and a block for one and a half to a CU, or for half the CUs where the other operand has workgroups of its
// kind anyway.  With fewer the walk is what a call waits for (scan and exponents with 64 and 16 rows: 1955 x 36 x 2987 in blocks of 1024 28.8 us and
// 20.2, 160 x 1518 x 1783 of 256 15.0 and 12.5; beyond, 2000 x 2000 x 4096 of 512 31.3 and 36.8).  Over 3725 calls with blocks of 128 to 1024 the choice
// is 0.9 % off the better one, 64 rows always 10 %, 16 always 2 %, and 21 calls are more than 5 % slower than with 64.
inline ScanGrid scan_grid(const Problem& p, bool a_rows_contig, bool b_rows_contig) {
    ScanGrid s;
    const bool one = a_rows_contig != b_rows_contig;
    s.k64 = !(a_rows_contig && b_rows_contig) && p.esc_block % 64 == 0 &&
            (p.esc_block == 64 || (p.m + p.n) * p.k * p.batch.count >= int64_t(one ? 1 : 3) * p.num_cu * 32 * p.esc_block);
    s.row_blocks_a = p.mp / (a_rows_contig || s.k64 ? 64 : 16);
    s.row_blocks_b = p.np / (b_rows_contig || s.k64 ? 64 : 16);
    const int64_t row_blocks = s.row_blocks_a + s.row_blocks_b;
    // ESC blocks per workgroup: four, or one where four would leave fewer than four workgroups per CU: such a call waits
    // for the loads of one block after the other, a larger one is bound by the bytes read, and four blocks leave a quarter of
    // the group maxima to write and to read again (scan and exponents with four and with one: 200x300x260 11.6 us and 9.9,
    // 1000^3 14.3 and 12.1, 2048^3 21.4 and 22.5, 8192^3 249 and 267)
    s.per = p.batch.count * row_blocks * ((p.G + kScanBlocksPerWg - 1) / kScanBlocksPerWg) < int64_t(4) * p.num_cu ? 1 : kScanBlocksPerWg;
    s.groups = (p.G + s.per - 1) / s.per;
    const int64_t fit = kMaxGridThreads / 256 / row_blocks;
    s.slab = s.groups < fit ? s.groups : fit;
    return s;
}

// ---- small calls, whose stages share launches ---------------------------------------------
// Scan and exponents in one launch, where a workgroup can hold all of k of its rows.  Up to 1024 of k it takes 2 to 4 us less (64 x 64 x 500
// with seven slices 36.7 -> 30.5 us a call, 200 x 300 x 260 31.8 -> 30.2, 512^3 41.4 -> 39.9, 1024^3 58.9 -> 56.6); beyond, the few workgroups
// are the slower way (512 x 512 x 2048 63.1 -> 64.4, 700 x 700 x 2000 79.7 -> 81.7).
inline bool scan_once(const Problem& p) {
    return p.k <= 1024 && p.G <= kScanOnceBlocks && (p.mp + p.np) / kOnceRows <= kScanOnceParts;
}

constexpr int kDecidePairs = 64;             // edge of a wave's block of pairs
// LDS of a workgroup that decides: 64 KB, of which the tables of both operands take what the kernel's own variables leave (432 bytes)
constexpr int kDecideLds = 64 * 1024, kDecideOwnLds = 1024;
// Most blocks, and most blocks times table rows and four for their end: what every workgroup computes, and computes again on packed int16 if
// all spans are wide.  Level then with the ESC kernel (300^3 34.1 -> 35.3 us falling back, 200 x 300 x 260 33.7 -> 30.3); with 64 blocks of two
// rows (512 x 512 x 64) 32.3 -> 36.8.
constexpr int kDecideBlocks = 32, kDecideWork = 400;
// bytes of the tables: encoded rows of eight, two operands, and an exponent per row
inline int64_t decide_table_bytes(const Problem& p) {
    const int64_t chunks = (2 * p.G + kEncChunk - 1) / kEncChunk * 2;
    return (round_up(p.m, 64) + round_up(p.n, 64)) * (chunks * 16 + 4);
}
// ESC, verdict and slicing in one launch, as far as the sizes go (decide_in_slice): while all of it is one round of workgroups.  200 x 300 x
// 260 (nine slices) 30.2 us in four launches, 26.2 in three, 256^3 26.9 and 23.3, 96 x 80 x 112 23.7 and 18.4.  With more (four problems of
// 200 x 300 x 260) what every workgroup computes is computed several times on a CU: 38.7 and 39.0, and 70 instead of 39 where all spans are
// beyond the encoding.
inline bool decide_fits(const Problem& p) {
    const int64_t blocks = ((p.m + kDecidePairs - 1) / kDecidePairs) * ((p.n + kDecidePairs - 1) / kDecidePairs);
    return scan_once(p) && blocks <= kDecideBlocks && blocks * (2 * p.G + 4) <= kDecideWork &&
           decide_table_bytes(p) <= kDecideLds - kDecideOwnLds && (p.mp + p.np) / 64 * (p.kp / 32) * p.batch.count <= p.num_cu;
}

// ---- walk of the ESC kernel ------------------------------------------------------------
// Position -> block of 128 x 128 pairs (nbi x nbj of them), for `workgroups` that take every workgroups-th position; as many
// workgroups as blocks take them as they come, fewer share them out.  A row of A or a column of B that is wide or zero
// leaves a whole row or column of blocks open, to be computed again the long way, and neither may meet the same few
// workgroups.  So block columns come one after the other, each turned against the last, and once more per walk over all
// workgroups; by eight blocks at a time where that leaves enough places, so that an XCD (every eighth workgroup) keeps to
// an eighth of the rows' tables for eight such walks.  (Straight, with `workgroups` a multiple of nbi, one zero row at
// 8192^3 was 64 open blocks for 8 workgroups: 666 us for the ESC, now 149.  Turned by one block, with all rows' tables in
// every XCD's L2, a call without open blocks took 84 us; straight 75, now 78, and at 4096^3 38 -> 35.)
__host__ __device__ inline void esc_block_at(int64_t position, int64_t nbi, int64_t nbj, int64_t workgroups, int64_t& bi,
                                             int64_t& bj) {
    bj = position / nbi;
    if (nbi * nbj <= workgroups) {
        bi = position - bj * nbi;
        return;
    }
    const int64_t walk = bj * nbi / workgroups, turn = bj + walk;
    const int64_t by_xcd = nbi / 8 % 2 == 0 ? 8 : 16;      // with nbi itself, an odd number of eights from column to column
    bi = (position + (nbi % 8 == 0 && nbi >= 64 ? by_xcd * turn + walk / 8 : turn)) % nbi;
}

// ---- stage launchers (each only enqueues) --------------------------------------------
// element (r, l) of an operand (r: row of op(A) / column of op(B), l: along k) is at X[r*stride_r + l*stride_l]
struct Operand {
    const double* X;
    int64_t stride_r, stride_l;
    int64_t rows, rows_p;
};
void launch_scan(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p);
// both in one launch (scan_once)
void launch_scan_exponents(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, bool encode,
                           const KnownRecord& known);
// row and column exponents, the cleared control record, and (encode) the BF16 tables of the ESC
void launch_exponents(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, bool encode,
                      const KnownRecord& known);
// coarsened ESC and the verdict (per-block mode: slice counts and dealing order of the blocks as well)
void launch_esc_verdict(hipStream_t st, const Workspace& w, const Problem& p, const oz_opts_t& o, const oz_heuristic_t& hm,
                        oz_result_t* user_result);
// records that need no kernel's result.  kind: 0 unguarded or OZ_NATIVE, 2 nothing to multiply (record says "emulated,
// 0 slices"), 3 native by the cost model alone (nothing scanned)
oz_result_t known_verdict(const Problem& p, const oz_opts_t& o, int kind);
void launch_known_record(hipStream_t st, const KnownRecord& known);
// whether the problems of p.batch can share the launches of an emulated call: few enough units of C for all of them, or small
// calls (LaunchPlan)
bool can_batch(const Problem& p);
// ESC, verdict and slicing of a call so small that every workgroup of the slicing can decide for itself
bool decide_in_slice(const Problem& p);
void launch_esc_slice(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, const oz_opts_t& o,
                      const oz_heuristic_t& hm, oz_result_t* user_result);
void launch_slice(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p);
// per-block mode: blocks of the slice GEMM's first launch, and whether they are sorted by slice count
void tile_order_shape(const Problem& p, int& first, int& deal);
// allows the slice GEMM its LDS on the current device (a property of the device: set when a handle is made for it)
bool prepare_gemm_i8();
// Returns what the recomposition still has to put together; small calls are recomposed in the same launch (kDone).  fallback: what
// such a launch needs to be the native product as well, if the verdict says so (A == nullptr: it has a launch of its own);
// fell_back: it is.
struct Fallback;
SplitPlan launch_gemm_i8(hipStream_t st, const Workspace& w, const Problem& p, double alpha, double beta, double* C, int64_t ldc,
                         const Fallback& fallback, bool& fell_back);
void launch_recompose(hipStream_t st, const Workspace& w, const Problem& p, const SplitPlan& split, double alpha,
                      double beta, double* C, int64_t ldc);
// rec == nullptr: run unconditionally; otherwise run only when rec->res.fallback != 0.
// scratch (may be nullptr): device memory the kernel may use for partial products when it splits the
// k range of a product with few tiles; nothing else may use it while the GEMM runs
// known: a record to write on the way
void launch_dgemm_f64(hipStream_t st, const Record* rec, const KnownRecord& known, bool ta, bool tb, int64_t m, int64_t n,
                      int64_t k, double alpha, const double* A, int64_t lda, const double* B,
                      int64_t ldb, double beta, double* C, int64_t ldc, int num_cu, const Batch& batch = Batch{},
                      void* scratch = nullptr, size_t scratch_bytes = 0);
void launch_scale_c(hipStream_t st, int64_t m, int64_t n, double beta, double* C, int64_t ldc);
// complex product by the 4M method: split an interleaved complex matrix into planar parts (conj negates
// the imaginary part), and combine the planar product with alpha, beta and the interleaved C
void launch_zsplit(hipStream_t st, const void* Z, int64_t ld, int64_t rows, int64_t cols, double* re, double* im,
                   bool conj);
// p_step: 0, or elements to the products that are still to be subtracted from Pr and added to Pi
void launch_zcombine(hipStream_t st, const double* Pr, const double* Pi, int64_t p_step, int64_t m, int64_t n, double ar, double ai,
                     double br, double bi, void* C, int64_t ldc);

}  // namespace oz
