// Host checks of the buffers of the finite-strain solver on nodal vectors, over
// plans that need no GPU: one line per plan and derivative kind whose layout
// does not hold what the solve puts there, then the number of layouts looked at.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

#include "feh_internal.hpp"

using namespace feh;

static int looked = 0;

static void look(const std::vector<int64_t> &n, int prec, int n_load, int layout, int kind) {
    feh_plan *plan = nullptr;
    if (feh_plan_create(&plan, (int)n.size(), n.data(), nullptr, n_load, prec, nullptr) != FEH_OK) return;
    if (layout >= 0) {
        int v[64];
        const int k = feh_plan_tuning(plan, v, 64);
        v[3] = layout;
        if (feh_plan_set_tuning(plan, v, k) != FEH_OK) std::printf("schedule refused\n");
    }
    feh_plan &p = *plan;
    const FiniteWork w = finite_layout(p, kind);
    size_t bytes = 0;
    feh_finite_strain_workspace_bytes(plan, kind, &bytes);
    char name[128];
    std::snprintf(name, sizeof name, "%d x %d x %d prec %d n_load %d layout %d kind %d", (int)n[0], (int)n[1],
                  n.size() == 3 ? (int)n[2] : 1, prec, n_load, layout, kind);
    if (w.total > bytes) std::printf("%s: %zu bytes in a buffer of %zu\n", name, w.total, bytes);
    {
        // the one-workgroup solve's outcome is written while other workgroups
        // still read Fbar (in the sums) and has to leave alone what it returns besides
        const size_t D = p.dim, from = w.outcome, to = from + 5 * p.L * sizeof(double);
        const struct {
            const char *what;
            size_t at, bytes;
        } others[] = {{"Fbar", w.cg.sums, p.L * D * D * 8}, {"the last Fbar", w.cg.ebar, p.L * D * D * 8},
                      {"u", w.u, p.L * D * (size_t)p.N * 8}};
        for (const auto &x : others)
            if (from < x.at + x.bytes && x.at < to) std::printf("%s: outcome runs into %s\n", name, x.what);
        if (to > w.total) std::printf("%s: outcome past the buffer\n", name);
    }
    {
        // as the solve runs: no kernel may leave more sums a row than the rows are apart
        NodalScope scope(p, reinterpret_cast<char *>(size_t(1) << 40), w.cg);
        p.part_stride = w.part_stride;
        p.metric = 1 + kind;
        const size_t most = (size_t)std::max(first_num_parts(p), nodal_num_parts(p));
        if (most > w.part_stride) std::printf("%s: %zu sums in rows of %zu\n", name, most, w.part_stride);
        if (nodal_marches(p, kind) && (size_t)stencil_num_parts(p) > w.part_stride)
            std::printf("%s: %d sums of the march in rows of %zu\n", name, stencil_num_parts(p), w.part_stride);
    }
    ++looked;
    feh_plan_destroy(plan);
}

int main() {
    const std::vector<std::vector<int64_t>> shapes = {
        {9, 40, 40}, {10, 12, 12}, {9, 2001}, {8, 40, 40}, {16, 12, 12}, {4, 2001}, {64, 48, 48}, {128, 9, 10},
        {2, 2}, {2, 3}, {2, 4}, {2, 7}, {2, 8}, {2, 9}, {2, 14}, {2, 15}, {2, 16}, {3, 2}, {17, 17}, {64, 64}, {512, 3}, {1024, 64}, {31, 33}, {2, 2, 2}, {2, 2, 31},
        {45, 50, 39}, {3, 300, 5}, {128, 128, 128}};
    for (const auto &n : shapes)
        for (int prec : {FEH_FP64, FEH_FP32})
            for (int n_load : {1, 2, 6, 7, 13, 16, 64})
                for (int layout : {-1, 0, 1})
                    for (int kind : {FEH_DERIV_FE, FEH_DERIV_FD, FEH_DERIV_CD, FEH_DERIV_LS})
                        if (nodal_kind(kind, (int)n.size())) look(n, prec, n_load, layout, kind);
    std::printf("looked at %d\n", looked);
    return 0;
}
