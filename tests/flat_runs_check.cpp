// Every tile of many layers against flat_runs(): none reaches further than all it returns, and what it returns are tiles.
#include "../paper_1811_01532_amd/csrc/flat_runs.h"

#include <cstdio>
#include <random>

int main() {
    std::mt19937 rng(1811);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    long layers = 0;
    for (int i = 0; i < 6000; ++i) {
        const bool small = i % 3 == 0;
        const int OH = pick(1, small ? 16 : 120), OW = i % 5 == 0 ? OH : pick(1, small ? 16 : 120);
        const int images = pick(1, 1 + 40000 / (OH * OW)), M = images * OH * OW;
        for (int bm : {64, 128, 160, 192, 224}) {
            const wap::FlatRuns f = wap::flat_runs(M, OH, OW, bm);
            bool met[4] = {false, false, false, false};
            const int R = 1 + 2 * pick(0, 3), S = 1 + 2 * pick(0, 3);
            const long PW = OW + S - 1, PH = OH + R - 1;
            auto padded = [&](long m) { return (m / (OH * OW) * PH + m / OW % OH) * PW + m % OW; };  // of pixel m at the filter's first tap
            long patch = 0;
            for (long m0 = 0; m0 < M; m0 += bm) {
                const long ml = (m0 + bm <= M ? m0 + bm : M) - 1;
                const int pixels = (int)(ml - m0 + 1), rows = (int)(ml / OW - m0 / OW), ends = (int)(ml / (OH * OW) - m0 / (OH * OW));
                patch = std::max(patch, padded(ml) - padded(m0) + (R - 1) * PW + S);
                bool within = false;
                for (int k = 0; k < f.n; ++k) {
                    within |= pixels <= f.run[k].pixels && rows <= f.run[k].rows && ends <= f.run[k].images;
                    // the most rows of any tile stand for the tiles without an end of an image
                    met[k] |= pixels == f.run[k].pixels && rows == f.run[k].rows && ends >= f.run[k].images;
                }
                if (!within) return std::printf("%d x %d x %d, %d pixels: tile at %ld\n", images, OH, OW, bm, m0), 1;
            }
            for (int k = 0; k < f.n; ++k)
                if (!met[k]) return std::printf("%d x %d x %d, %d pixels: no tile %d %d %d\n", images, OH, OW, bm, f.run[k].pixels, f.run[k].rows, f.run[k].images), 1;
            if (wap::flat_patch(f, OW, R, S) != patch) return std::printf("%d x %d x %d, %d pixels, %d x %d: patch %ld\n", images, OH, OW, bm, R, S, patch), 1;
            ++layers;
        }
    }
    std::printf("%ld\n", layers);
    return 0;
}
