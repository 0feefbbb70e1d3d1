// The FP64 tiles straight from memory, run on the host with the library's own walk over k: every lane of every wave loads its
// fragments from operands that end where a page without access begins, and the MFMA steps are added up.  Reads lines
// "m n k kb kt waves a_rows b_rows pad" (the tile multiplies k [kb, kb + k) of kt; pad: leading dimensions beyond the least); prints
// per line "outside wrong": loads that met the page (the walk is left at the first), and elements of the tile that differ from the product.
#include <setjmp.h>
#include <signal.h>
#include <sys/mman.h>
#include <unistd.h>

#include <cstdio>
#include <cstring>
#include <vector>

#include "oz_f64_walk.h"

using namespace oz;

struct KeepNothing {
    void order() const {}
    void scalar(int64_t&) const {}
};

static sigjmp_buf outside;
static void on_fault(int) { siglongjmp(outside, 1); }

// `count` doubles between two pages without access, ending at the second one
struct Guarded {
    void* base;
    size_t bytes;
    double* x;
    explicit Guarded(size_t count) {
        const size_t page = size_t(sysconf(_SC_PAGESIZE)), body = (count * 8 + page - 1) / page * page;
        bytes = body + 2 * page;
        base = mmap(nullptr, bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        mprotect(static_cast<char*>(base) + page, body, PROT_READ | PROT_WRITE);
        x = reinterpret_cast<double*>(static_cast<char*>(base) + page + body) - count;
    }
    ~Guarded() { munmap(base, bytes); }
};

// element (r, l) of an operand at x[r * sr + l * sl]; whole numbers, so that sums are exact
static void fill(double* x, int64_t rows, int64_t k, int64_t sr, int64_t sl, int salt) {
    for (int64_t r = 0; r < rows; ++r)
        for (int64_t l = 0; l < k; ++l) x[r * sr + l * sl] = double((r * 7 + l * 13 + salt) % 19 - 9);
}

template <bool AC, bool BC, int NI, int NJ>
static long long tile(const double* A, int64_t a_sr, int64_t a_sl, int64_t m, const double* B, int64_t b_sr, int64_t b_sl, int64_t n, int64_t i0,
                      int64_t j0, int64_t kb, int64_t k, int waves) {
    std::vector<double> sum(16 * NI * 16 * NJ, 0.0);
    for (int wave = 0; wave < waves; ++wave) {
        const WaveShare share = wave_share(k, wave, waves);
        if (share.first == 0) continue;
        // An MFMA step adds, for each of the four lane groups, the outer product of what its lanes hold.  All lanes load the same
        // steps in the same order: each lane's walk is recorded, then the steps are multiplied.
        std::vector<std::vector<double>> va(64), vb(64);
        for (int lane = 0; lane < 64; ++lane) {
            DirectSide<AC, NI> a;
            DirectSide<BC, NJ> b;
            a.init(A, a_sr, a_sl, i0, m, kb + share.lo, lane);
            b.init(B, b_sr, b_sl, j0, n, kb + share.lo, lane);
            walk_share(share, a, b, lane, [&](int s) {
                for (int f = 0; f < NI; ++f) va[lane].push_back(a.v[s][f]);
                for (int f = 0; f < NJ; ++f) vb[lane].push_back(b.v[s][f]);
            }, KeepNothing{});
        }
        const size_t steps = va[0].size() / NI;
        for (size_t s = 0; s < steps; ++s)
            for (int g = 0; g < 4; ++g)
                for (int j = 0; j < 16 * NJ; ++j)
                    for (int i = 0; i < 16 * NI; ++i)
                        sum[j * 16 * NI + i] += va[g * 16 + i % 16][s * NI + i / 16] * vb[g * 16 + j % 16][s * NJ + j / 16];
    }
    long long wrong = 0;
    for (int64_t j = j0; j < n && j < j0 + 16 * NJ; ++j)
        for (int64_t i = i0; i < m && i < i0 + 16 * NI; ++i) {
            double want = 0.0;
            for (int64_t l = kb; l < kb + k; ++l) want += A[i * a_sr + l * a_sl] * B[j * b_sr + l * b_sl];
            wrong += sum[(j - j0) * 16 * NI + i - i0] != want;
        }
    return wrong;
}

template <int NI, int NJ>
static long long last_tile(const double* A, int64_t a_sr, int64_t a_sl, int64_t m, const double* B, int64_t b_sr, int64_t b_sl, int64_t n,
                           int64_t kb, int64_t k, int waves, bool ar, bool br) {
    const int64_t i0 = (m - 1) / (16 * NI) * (16 * NI), j0 = (n - 1) / (16 * NJ) * (16 * NJ);
#define OZ_TILE(AC, BC) tile<AC, BC, NI, NJ>(A, a_sr, a_sl, m, B, b_sr, b_sl, n, i0, j0, kb, k, waves)
    return ar ? (br ? OZ_TILE(true, true) : OZ_TILE(true, false)) : (br ? OZ_TILE(false, true) : OZ_TILE(false, false));
#undef OZ_TILE
}

int main() {
    signal(SIGSEGV, on_fault);
    long long m, n, k, kb, kt, pad;
    int waves, ar, br;
    while (std::scanf("%lld %lld %lld %lld %lld %d %d %d %lld", &m, &n, &k, &kb, &kt, &waves, &ar, &br, &pad) == 9) {
        const int64_t lda = (ar ? m : kt) + pad, ldb = (br ? n : kt) + pad;
        const int64_t a_sr = ar ? 1 : lda, a_sl = ar ? lda : 1, b_sr = br ? 1 : ldb, b_sl = br ? ldb : 1;
        Guarded A((m - 1) * a_sr + (kt - 1) * a_sl + 1), B((n - 1) * b_sr + (kt - 1) * b_sl + 1);
        fill(A.x, m, kt, a_sr, a_sl, 3);
        fill(B.x, n, kt, b_sr, b_sl, 11);
        volatile long long wrong = 0, met = 0;
        if (sigsetjmp(outside, 1) == 0) {
            wrong = wrong + last_tile<1, 1>(A.x, a_sr, a_sl, m, B.x, b_sr, b_sl, n, kb, k, waves, ar, br);
            wrong = wrong + last_tile<2, 2>(A.x, a_sr, a_sl, m, B.x, b_sr, b_sl, n, kb, k, waves, ar, br);
            wrong = wrong + last_tile<3, 4>(A.x, a_sr, a_sl, m, B.x, b_sr, b_sl, n, kb, k, waves, ar, br);
        } else {
            met = met + 1;
        }
        std::printf("%lld %lld\n", static_cast<long long>(met), static_cast<long long>(wrong));
    }
    return 0;
}
