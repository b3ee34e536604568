// Split plans of the folded two-layer backward, printed for each shape on
// stdin (kind f0 f1 n_out cap_m1 cap_m2): whether the folded launch takes it,
// each layer's split count of the partials' job and of the reduction, and the
// bytes of partials that the reduction reads beside the workspace's size.
// Host code only: no device pointer is dereferenced and nothing is launched.
#include <cstdio>

#include "bwd_pull_dev.h"
#include "gnn.h"

using namespace gnn;

int main() {
    long kind, f0, f1, n_out, cap1, cap2;
    char *fake = reinterpret_cast<char *>(uintptr_t(1) << 24);
    while (std::scanf("%ld %ld %ld %ld %ld %ld", &kind, &f0, &f1, &n_out, &cap1, &cap2) == 6) {
        auto *f = reinterpret_cast<float *>(fake);
        auto *i32 = reinterpret_cast<int32_t *>(fake);
        auto *i64 = reinterpret_cast<int64_t *>(fake);
        const gnn_block b{cap2, cap1, cap2 * 25, i64, i64, i64, i32, i64, i32, f};
        const TwoBwdPlan t =
            plan_two_bwd(static_cast<int>(kind), b, fake, fake, f0, i64, cap1, reinterpret_cast<uint16_t *>(fake), f1,
                         fake, i32, f, f, n_out, nullptr, f, f, f, nullptr, nullptr, nullptr, nullptr, f, f, f, nullptr,
                         nullptr, nullptr, 0.f);
        size_t ws = 0;
        if (gnn_two_layer_bwd_workspace_size(static_cast<gnn_agg>(kind), f0, f1, n_out, cap1, cap2, &ws) != GNN_OK)
            return 1;
        const size_t part1 = gbwd::dw_part_bytes(t.p1.pw, t.a1.K(), f1), part2 = gbwd::dw_part_bytes(t.p2.pw, t.a2.K(), n_out);
        std::printf("%d %d %d %d %d %zu %zu\n", t.pull ? 1 : 0, t.p1.pw.map.nsplit, t.p1.pw.nsplit, t.p2.pw.map.nsplit,
                    t.p2.pw.nsplit, round_up(part1, size_t(256)) + part2, ws);
    }
    return 0;
}
