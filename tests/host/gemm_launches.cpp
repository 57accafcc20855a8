// Reads "T features K qkv swiglu scratch" lines and prints the launches of a projection of that size (gemm_plan; host arithmetic
// alone): tile rows, tile features, tiles that split their k range, ways they split it, columns of the first launch of two, the tile
// rows of either, whether split tiles run as halves.
#include <cstdio>

#include "relserve_internal.h"

int main() {
    int T, K, qkv, swiglu, scratch;
    long long features;
    while (std::scanf("%d %lld %d %d %d %d", &T, &features, &K, &qkv, &swiglu, &scratch) == 6) {
        const relserve::GemmPlan p = relserve::gemm_plan(T, features, K, qkv != 0, swiglu != 0, scratch != 0);
        std::printf("%d %d %d %d %d %d %d %d\n", p.rows, p.cols, p.tail_tiles, p.splits, p.cols1, p.rows1, p.rows2, p.halves ? 1 : 0);
    }
    return 0;
}
