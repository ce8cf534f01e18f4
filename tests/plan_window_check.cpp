// Prints which layers of a plan the library runs together: one line per window, "first n: layers whose GEMMs share a launch"; layers in no window run
// alone.  With an argument: only those layers of a window whose shared launch has one round of large tiles.  Host arithmetic only; the addresses are never followed.  Input: "M R p_ppm a_bits room" (p_ppm 0: the maximum; room: workspace as a multiple
// of the recommended one), then "K N bits group x y" per layer.
#include "../paper_2511_11446_amd/csrc/plan_window.h"

#include <cstdio>
#include <vector>

int main(int argc, char **)
{
    long long M, R, p_ppm, a_bits, room, K, N, bits, group, x, y;
    if (std::scanf("%lld %lld %lld %lld %lld", &M, &R, &p_ppm, &a_bits, &room) != 5) return 1;
    std::vector<ql_layer_desc> layers;
    std::vector<const void *> xs;
    std::vector<void *> ys;
    while (std::scanf("%lld %lld %lld %lld %lld %lld", &K, &N, &bits, &group, &x, &y) == 6) {
        // weights, scales and biases beyond all inputs and outputs
        const uintptr_t w = ((uintptr_t)1 << 50) + ((uintptr_t)layers.size() << 36);
        ql_layer_desc d{};
        d.K = K;
        d.N = N;
        d.w_bits = (int32_t)bits;
        d.group = (int32_t)group;
        d.w = reinterpret_cast<const void *>(w);
        d.w_scale = bits == 16 ? nullptr : reinterpret_cast<const void *>(w + ((uintptr_t)1 << 34));
        d.bias = reinterpret_cast<const void *>(w + ((uintptr_t)1 << 35));
        layers.push_back(d);
        xs.push_back(reinterpret_cast<const void *>((uintptr_t)x));
        ys.push_back(reinterpret_cast<void *>((uintptr_t)y));
    }
    ql_plan *plan = nullptr;
    if (ql_plan_create(layers.data(), (int32_t)layers.size(), M, &plan) != QL_OK) return 2;
    const size_t bytes = ql_plan_workspace_bytes(plan, M, R) * (size_t)room;
    ql_plan_destroy(plan);
    ql_daq_params dp{};
    dp.p_ppm = (int32_t)p_ppm;
    dp.a_bits = (int32_t)a_bits;
    for (size_t l = 0; l < layers.size();) {
        ql::PlanWindow w;
        ql::plan_window(layers.data(), layers.size(), l, xs.data(), ys.data(), M, R, p_ppm ? &dp : nullptr, reinterpret_cast<void *>((uintptr_t)1 << 52),
                        bytes, w);
        if (w.n == 0) {
            ++l;
            continue;
        }
        std::printf("%d %d:", (int)l, w.n);
        if (argc > 1 && !ql::qgemm_many_one_round(w.together, w.count)) w.count = 0;
        for (int i = 0; i < w.count; ++i) std::printf(" %d", (int)l + (int)(w.together[i] - w.g));
        std::printf("\n");
        l += (size_t)w.n;
    }
    return 0;
}
