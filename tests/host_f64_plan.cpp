// The choices of the native FP64 GEMM on the host, without scratch memory.  Reads lines "m n k a_rows b_rows beta ld" (ld 0: the least
// leading dimensions); prints per line "direct ti tj mode": the tile (ti 0: none fits the grid) and the form of the K loop on LDS tiles.
#include <cstdio>

#include "oz_f64_plan.h"

using namespace oz;

int main() {
    long long m, n, k, ld;
    int ar, br, beta;
    while (std::scanf("%lld %lld %lld %d %d %d %lld", &m, &n, &k, &ar, &br, &beta, &ld) == 7) {
        const int64_t lda = ld ? ld : (ar ? m : k), ldb = ld ? ld : (br ? n : k);
        const F64Plan p = choose_f64(f64_size(m, n, k, 1, false, beta != 0, ar, lda, br, ldb), 256, 0);
        std::printf("%d %d %d %d\n", int(p.direct), p.ti, p.tj,
                    f64_mode(wide_offsets(m, n, k, std::max(lda, ldb)), m, n, k, p.ti ? p.ti : 64, p.tj ? p.tj : 64));
    }
    return 0;
}
