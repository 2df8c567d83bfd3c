// Launch rules of the 32 x 32 matrix-core shapes, asked of the built library on
// the host: for every format, split, mode, number of points and samples given on
// a line of the standard input (dim M split mode n_snr n), the blocks per point,
// threads, sample columns per wave and whether a tile's points are split.
#include <cstdio>

#include "../../paper_2011_13695_amd/csrc/internal.h"

int main() {
    int dim, M, split, mode, n_snr;
    long long n;
    while (std::scanf("%d %d %d %d %d %lld", &dim, &M, &split, &mode, &n_snr, &n) == 6) {
        mdgmi_format f;
        f.dim = dim;
        f.M = M;
        while ((1 << f.m) < M) f.m++;
        const mdgmi::LaunchCfg c = mdgmi::mfma_cfg(&f, n, n_snr, mode, split);
        std::printf("%d %d %d %d\n", c.blocks_per_snr, c.threads, c.variant, (int)c.split_points);
    }
    return 0;
}
