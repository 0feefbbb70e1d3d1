// Whether a guarded call that falls back holds the FP64 product in its last launch, on the host.  Reads lines
// "m n k a_rows b_rows beta most_slices edge scratch_bytes"; prints per line "folds".
#include <cstdio>

#include "oz_f64_plan.h"
#include "oz_gemm_plan.h"

using namespace oz;

int main() {
    long long m, n, k, scratch;
    int ar, br, beta, s_cap, edge;
    while (std::scanf("%lld %lld %lld %d %d %d %d %d %lld", &m, &n, &k, &ar, &br, &beta, &s_cap, &edge, &scratch) == 9) {
        const F64Size size = f64_size(m, n, k, 1, true, beta != 0, ar, ar ? m : k, br, br ? n : k);
        const int64_t tiles = ((m + 31) / 32) * ((n + 31) / 32);
        std::printf("%d\n", int(f64_folds(size, 256, size_t(scratch), edge, edge == 32 && !(tiles > 256 && s_cap <= kSmallPairSlices))));
    }
    return 0;
}
