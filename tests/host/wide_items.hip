// How the wide products' work items are dealt to the workgroups of a grid: for
// each "grid items" on stdin, a line with the item of every workgroup (-1:
// none).  Host code only.
#include <cstdio>

#include "gemm_wide_dev.h"

int main() {
    long grid, items;
    while (std::scanf("%ld %ld", &grid, &items) == 2) {
        for (long b = 0; b < grid; ++b) std::printf("%lld ", static_cast<long long>(gnn::wide::xcd_item(b, items)));
        std::printf("\n");
    }
    return 0;
}
