// Host check of the one-sided work lists of the periodic real space (no GPU
// calls; the library's own builder, its translation unit included whole):
// every item holds at most 64 targets (kind 1) or 64 sources (kind 2) of one
// part against a part of at most 256; every ordered pair of particles is met
// exactly once; every (particle, slot) is written exactly once.
#include "api.cpp"

#include <cstdio>

int main()
{
    int bad = 0;
    for (int64_t n : {1, 64, 65, 255, 256, 257, 300, 511, 512, 513, 769, 1025, 1500}) {
        Boxes b;
        b.off = {0, n};
        b.eps = {0.01};
        b.max_n = n;
        TileCfg cfg = symmetric_cfg(b, 4, 64);
        cfg.group = kOneSided;
        WorkList wl;
        build_worklist(b, n, cfg, wl);
        const int64_t P = (n + 255) / 256;
        std::vector<int> met((size_t)(n * n), 0), slot((size_t)(n * P), 0);
        for (const WorkItem &w : wl.items) {
            const bool react = w.kind == 2;
            const int64_t a0 = react ? w.j0 : w.i0, a1 = react ? w.j1 : w.i1;
            const int64_t c0 = react ? w.i0 : w.j0, c1 = react ? w.i1 : w.j1;
            if ((w.kind != 1 && w.kind != 2) || a0 < 0 || a1 > n || c0 < 0 || c1 > n ||
                a1 <= a0 || a1 - a0 > 64 || c1 - c0 > 256) {
                std::printf("FAIL: item shape, n = %ld\n", (long)n);
                return 1;
            }
            const int32_t s = react ? w.rslice : w.slice;
            if (s < 0 || s >= P || s != c0 / 256) {
                std::printf("FAIL: slot number, n = %ld\n", (long)n);
                return 1;
            }
            for (int64_t k = a0; k < a1; ++k) {
                ++slot[(size_t)(k * P + s)];
                for (int64_t j = c0; j < c1; ++j)
                    ++met[(size_t)(k * n + j)];
            }
        }
        for (int v : met)
            bad |= v != 1;
        for (int v : slot)
            bad |= v != 1;
        for (const IntBlock &ib : wl.blocks)
            bad |= ib.n_slices != P;
        if (bad) {
            std::printf("FAIL: coverage, n = %ld\n", (long)n);
            return 1;
        }
    }
    std::printf("all ok\n");
    return 0;
}
