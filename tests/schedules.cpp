// Host checks of plans' schedules, over plans that need no GPU: what a plan
// runs before and after its own reported schedule is set again, on it and on a
// new plan of the shape; one line per difference, then the number of plans.
#include <algorithm>
#include <cstdio>
#include <string>
#include <vector>

#include "feh_internal.hpp"

using namespace feh;

// what the launchers choose by
static std::vector<long long> route(const feh_plan &p) {
    std::vector<long long> r = {first_num_parts(p),     first_num_parts(p, 1), first_by_table(p, 0), first_per_load_case(p),
                                first_ct_pencils(p),    stencil_rows(p),       stencil_num_parts(p), cg_residual_spectral(p),
                                small_solve_ok(p, false),  small_solve_ok(p, true)};
    for (const AxisFFT &a : p.fft)
        for (int s = 0; s < a.npass; ++s) r.push_back(a.pass[s].R);
    return r;
}

int main() {
    const std::vector<std::vector<int64_t>> shapes = {
        {32, 32}, {17, 17}, {48, 48}, {30, 34}, {64, 4}, {2, 2}, {9, 2001}, {151, 151}, {1024, 64}, {300, 300},
        {9, 40, 40}, {10, 12, 12}, {90, 77, 105}, {64, 64, 64}, {15, 12, 10}, {16, 12, 10}, {128, 128, 128}};
    int looked = 0;
    for (const auto &n : shapes)
        for (int prec : {FEH_FP64, FEH_FP32})
            for (int n_load : {1, 6})
                for (int change = 0; change < 6; ++change) {
                    feh_plan *a = nullptr, *b = nullptr;
                    if (feh_plan_create(&a, (int)n.size(), n.data(), nullptr, n_load, prec, nullptr) != FEH_OK ||
                        feh_plan_create(&b, (int)n.size(), n.data(), nullptr, n_load, prec, nullptr) != FEH_OK)
                        return 1;
                    int v[64];
                    int k = feh_plan_tuning(a, v, 64);
                    if (change == 1) v[0] = 2;
                    if (change == 2) v[3] = 1 - v[3];
                    if (change == 3) v[2] = first_pencils_default(*a);
                    if (change == 4 && n.size() == 3) v[4] = 16;
                    if (change == 5) v[k - 1] = 1;
                    const std::string name = std::to_string(n[0]) + " x " + std::to_string(n[1]) +
                                             (n.size() == 3 ? " x " + std::to_string(n[2]) : "") + " prec " +
                                             std::to_string(prec) + " n_load " + std::to_string(n_load) + " change " +
                                             std::to_string(change);
                    if (change && feh_plan_set_tuning(a, v, k) != FEH_OK) std::printf("%s: refused\n", name.c_str());
                    const auto before = route(*a);
                    k = feh_plan_tuning(a, v, 64);
                    if (feh_plan_set_tuning(a, v, k) != FEH_OK || feh_plan_set_tuning(b, v, k) != FEH_OK)
                        std::printf("%s: own schedule refused\n", name.c_str());
                    if (route(*a) != before) std::printf("%s: runs otherwise once set again\n", name.c_str());
                    if (route(*b) != before) std::printf("%s: a new plan runs it otherwise\n", name.c_str());
                    feh_plan_destroy(a);
                    feh_plan_destroy(b);
                    ++looked;
                }
    std::printf("looked at %d\n", looked);
    return 0;
}
