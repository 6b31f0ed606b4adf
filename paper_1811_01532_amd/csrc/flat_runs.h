// How far the flat tiles of a layer reach: runs of bm output pixels in raster order, cut from its images from the first pixel on.
#ifndef WAP_FLAT_RUNS_H
#define WAP_FLAT_RUNS_H

#include <algorithm>
#include <numeric>

namespace wap {

// A tile's pixels, and how many ends of a row and of an image lie between its first and its last.
struct FlatRun {
    int pixels, rows, images;
};
// The furthest tiles: every tile is exceeded or equalled in all three numbers by one of these, each of which is a tile.
struct FlatRuns {
    int n = 0;
    FlatRun run[4];
};

// Without a walk over the tiles (tens of thousands on an odd map: up to 0.3 ms a call): a tile's row ends follow from where in a row it
// starts, and starts are multiples of gcd(bm, OW) apart, all of them once there are OW / gcd tiles; an end of an image lies in one tile,
// and after bm / gcd(bm, OH * OW) images these tiles repeat.
inline FlatRuns flat_runs(int M, int OH, int OW, int bm) {
    FlatRuns f;
    const int image = OH * OW, full = M / bm, rest = M % bm;
    if (rest) {  // the last tile, cut short
        const int at = M - rest;
        f.run[f.n++] = {rest, (at % OW + rest - 1) / OW, (at % image + rest - 1) / image};
    }
    if (full == 0) return f;
    const int most = (OW - 1 + bm - 1) / OW;  // row ends of a tile
    if (image >= bm) {  // at most one end of an image in a tile
        const int apart = std::gcd(bm, OW);
        int rows = 0;
        if (full >= OW / apart) rows = (OW - apart + bm - 1) / OW;
        else
            for (int k = 0, s = 0; k < full && rows < most; ++k, s = (s + bm) % OW) rows = std::max(rows, (s + bm - 1) / OW);
        f.run[f.n++] = {bm, rows, 0};
        // pixels of a tile in front of an end of an image: rows + 1 is reached where they end 1 .. over pixels behind a row's end
        const int base = (bm - 1) / OW, over = (bm - 1) % OW, step = std::gcd(bm, image), cycle = bm / step;
        const int ends = (int)std::min((long)M / image - 1, ((long)full * bm - 1) / image);  // in tiles that are not cut short
        bool any = false, more = false;
        auto end_at = [&](int before) {
            if (before == 0) return;  // a tile ends there too
            const int behind = before % OW;
            any = true;
            more = behind >= 1 && behind <= over;
        };
        if (ends >= cycle)
            for (int before = step; before < bm && !more; before += step) end_at(before);
        else
            for (int i = 0, before = 0; i < ends && !more; ++i) {
                before += image % bm;
                if (before >= bm) before -= bm;
                end_at(before);
            }
        if (any) f.run[f.n++] = {bm, base + more, 1};
    } else {
        const int few = bm / image - (bm % image == 0), tiles = std::min(full, image / std::gcd(bm, image));
        // ends of an image in a tile: `few` at least (none more where a tile is whole images), or one more
        int rows[2] = {-1, -1};
        for (int k = 0, s = 0; k < tiles; ++k, s = (s + bm) % image) {
            int& r = rows[(s + bm - 1) / image - few];
            r = std::max(r, (s % OW + bm - 1) / OW);
        }
        for (int i = 0; i < 2; ++i)
            if (rows[i] >= 0) f.run[f.n++] = {bm, rows[i], few + i};
    }
    return f;
}

// most pixels of a zero-padded patch (rows of OW + S - 1) that one of these tiles reads under an R x S filter
inline int flat_patch(const FlatRuns& f, int OW, int R, int S) {
    const int PW = OW + S - 1;
    int worst = 0;
    for (int i = 0; i < f.n; ++i) worst = std::max(worst, f.run[i].pixels - 1 + f.run[i].rows * (S - 1) + (f.run[i].images + 1) * (R - 1) * PW + S);
    return worst;
}

}  // namespace wap

#endif
