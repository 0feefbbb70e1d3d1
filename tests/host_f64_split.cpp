// Tile and parts of k of the native FP64 GEMM on the host, with 64 MB of scratch memory.  Reads lines "m n k a_rows b_rows beta guarded"; prints
// per line "ti tj parts".
#include <cstdio>

#include "oz_f64_plan.h"

using namespace oz;

int main() {
    long long m, n, k;
    int ar, br, beta, guarded;
    while (std::scanf("%lld %lld %lld %d %d %d %d", &m, &n, &k, &ar, &br, &beta, &guarded) == 7) {
        const F64Plan p = choose_f64(f64_size(m, n, k, 1, guarded != 0, beta != 0, ar, ar ? m : k, br, br ? n : k), 256, size_t(64) << 20);
        std::printf("%d %d %d\n", p.ti, p.tj, p.zsplit);
    }
    return 0;
}
