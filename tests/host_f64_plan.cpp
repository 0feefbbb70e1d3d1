// The choices of the native FP64 GEMM on the host.  Reads lines "m n k"; prints per line "mode direct ti": the form of the K loop
// on tiles of 64 through LDS, whether the tiles straight from memory are chosen, and their edge (0: none fits the grid).
#include <cstdio>

#include "oz_f64_plan.h"

using namespace oz;

int main() {
    long long m, n, k;
    while (std::scanf("%lld %lld %lld", &m, &n, &k) == 3) {
        const F64Plan p = choose_f64(F64Size{m, n, k, 1, false}, 256, nullptr, 0);
        std::printf("%d %d %d\n", f64_mode(wide_offsets(m, n, k, std::max(m, k)), m, n, k, 64, 64), int(p.direct), p.ti);
    }
    return 0;
}
