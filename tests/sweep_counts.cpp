// The autotuner's n_sweeps is the number of passes over the state that each form
// makes: counted here as the kernels that the library's host code launches.
#include "fake_hip.h"

#include <cstdint>
#include <cstdio>

#include "../include/sv.h"

static int sweeps_launched()
{
    int count = 0;
    for (const std::string& n : launched)
        for (const char* k : {"k_tile", "k_gate", "k_diag", "k_fused"}) count += n.find(k) != std::string::npos;
    return count;
}

int main()
{
    int failures = 0;
    // layers of U3 and CZ, and a lone X with three controls; 3 qubits: a sweep per gate
    for (int n : {3, 9, 14, 20, 26}) {
        std::vector<sv_op> ops;
        std::vector<double> params;
        for (int layer = 0; layer < 6; ++layer) {
            for (int q = 0; q < n; ++q) {
                sv_op op{};
                op.kind = SV_U3;
                op.n_targets = 1;
                op.targets[0] = q;
                for (int j = 0; j < 3; ++j) {
                    op.param[j] = (int)params.size();
                    params.push_back(0.1 + 0.01 * (double)params.size());
                }
                ops.push_back(op);
            }
            for (int q = layer % 2; q + 1 < n; q += 2) {
                sv_op op{};
                op.kind = SV_Z;
                op.n_targets = op.n_controls = 1;
                op.targets[0] = q + 1;
                op.controls[0] = q;
                op.param[0] = op.param[1] = op.param[2] = -1;
                ops.push_back(op);
            }
        }
        sv_state s = nullptr;
        if (sv_alloc(n, 1, nullptr, nullptr, &s) != SV_OK) return 2;
        auto list = [&] { return sv_run(s, ops.data(), (int)ops.size(), params.data(), 0, (int)params.size()); };
        launched.clear();
        if (list() != SV_OK) return 2;
        const int in_lists = sweeps_launched();
        sv_fusion_choice best{}, trials[16];
        int count = 0;
        if (sv_fused_autotune(s, ops.data(), (int)ops.size(), params.data(), (int)params.size(), 7u, 1, &best, trials, 16,
                              &count) != SV_OK)
            return 2;
        for (int i = 0; i < count; ++i) {
            int want = in_lists;
            if (trials[i].mode >= 0) {
                std::vector<sv_block> blocks(ops.size());
                std::vector<double> mats(ops.size() * (size_t(2) << (2 * trials[i].max_k)));
                int nb = 0;
                if (sv_fuse_plan(n, ops.data(), (int)ops.size(), params.data(), (int)params.size(), trials[i].max_k,
                                 blocks.data(), (int)blocks.size(), mats.data(), &nb) != SV_OK)
                    return 2;
                launched.clear();
                if (sv_apply_fused(s, blocks.data(), nb, trials[i].mode) != SV_OK) return 2;
                want = sweeps_launched();
            }
            if (trials[i].n_sweeps != want) {
                std::printf("%d qubits, mode %d, max_k %d: n_sweeps %d, launched %d\n", n, trials[i].mode,
                            trials[i].max_k, trials[i].n_sweeps, want);
                ++failures;
            }
        }
        if (count < 2 || (n > 3 && in_lists * 4 > (int)ops.size())) return 3;
        sv_free(s);
    }
    return failures ? 1 : 0;
}
