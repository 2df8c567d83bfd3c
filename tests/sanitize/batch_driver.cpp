// Items of ragged batches as the built library plans them, asked on the host: a
// line of the standard input holds a batch of AUTO instances (count, then dim, M
// and samples of each); for each batch the items' samples and M, 32 x 32 kind only.
#include <cstdio>
#include <vector>

#include "../../paper_2011_13695_amd/csrc/internal.h"
#include "../../paper_2011_13695_amd/csrc/batch.h"

int main() {
    int cnt;
    while (std::scanf("%d", &cnt) == 1) {
        std::vector<mdgmi_format> f(cnt);
        std::vector<mdgmi_instance> inst(cnt);
        for (int q = 0; q < cnt; q++) {
            long long n;
            if (std::scanf("%d %d %lld", &f[q].dim, &f[q].M, &n) != 3) return 1;
            while ((1 << f[q].m) < f[q].M) f[q].m++;
            f[q].max_abs = f[q].max_norm2 = 1.0;
            inst[q] = {&f[q], nullptr, nullptr, n, 0.1};
        }
        mdgmi::BatchPlan P;
        if (mdgmi::plan_batch(inst.data(), cnt, MDGMI_PATH_AUTO, mdgmi::tuned_item_pairs(), P) != MDGMI_OK) return 2;
        for (int k = 0; k < P.n_mfma_items; k++)
            std::printf("%lld:%d ", (long long)(P.items[k].s1 - P.items[k].s0), P.insts[P.items[k].inst].M);
        std::printf("\n");
    }
    return 0;
}
