// Reads "T features K qkv swiglu" lines and prints how a projection of that size is tiled (gemm_plan; host arithmetic alone):
// tile rows, tile features, tiles that split their k range, ways they split it.
#include <cstdio>

#include "relserve_internal.h"

int main() {
    int T, K, qkv, swiglu;
    long long features;
    while (std::scanf("%d %lld %d %d %d", &T, &features, &K, &qkv, &swiglu) == 5) {
        const relserve::GemmPlan p = relserve::gemm_plan(T, features, K, qkv != 0, swiglu != 0, true);
        std::printf("%d %d %d %d\n", p.rows, p.cols, p.tail_tiles, p.splits);
    }
    return 0;
}
