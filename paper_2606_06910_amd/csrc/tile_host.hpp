// tile_host.hpp -- box lists of the kernels that work on TILE_X x TILE_Y x TILE_Z
// boxes (host side, shared by the second- and first-order paths).
#pragma once
#include "fdtd_dev.hpp"

#include <algorithm>
#include <vector>

// Boxes of a brick (tile_boxes) on a large grid.  One XCD runs about 128 boxes at a time; measured on the
// first-order step at 544^3 (us per step): columns of boxes along z 1842, bricks of 32 1868, 128 1859, 256 1742,
// 512 1749 (counted reads 7.4 GB in columns, 5.8 GB in bricks of 256); three gradients of 100 steps 25.2 ms in
// columns, 24.3 in bricks.
constexpr size_t kTileBrick = 256;
constexpr size_t kTileAhead = 1024;  // boxes one XCD's list may be ahead of another's

// Boxes of a grid in bricks: a brick is the set of boxes that run on one XCD at about the same time, so
// it is grown (by doubling its shortest side) towards a cube of `want` boxes, whose faces share the least
// halo with its neighbours.  `brick` receives each box's brick number.  Each box is marked with the axes
// whose band (layer and 4 points) it meets.
inline void tile_boxes(const int n[3], const int lo[3], const int hi[3], int shot, size_t want,
                       std::vector<TileItem> &v, std::vector<int> &brick) {
    const int ext[3] = {TILE_X, TILE_Y, TILE_Z};
    int nb[3], b[3] = {1, 1, 1};
    for (int d = 0; d < 3; ++d) nb[d] = (n[d] + ext[d] - 1) / ext[d];
    while ((size_t)b[0] * b[1] * b[2] < want) {
        int s = -1;   // shortest side that can still grow
        for (int d = 2; d >= 0; --d)
            if (b[d] < nb[d] && (s < 0 || b[d] * ext[d] < b[s] * ext[s])) s = d;
        if (s < 0) break;
        b[s] *= 2;
    }
    auto meets = [&](int d, int c0, int len) {
        const int c1 = std::min(c0 + len, n[d]);
        return (lo[d] > 0 && c0 < lo[d] + FDTD_R) || (hi[d] > 0 && c1 > n[d] - hi[d] - FDTD_R);
    };
    int id = brick.empty() ? 0 : brick.back() + 1;
    for (int X = 0; X < nb[0]; X += b[0])
        for (int Y = 0; Y < nb[1]; Y += b[1])
            for (int Z = 0; Z < nb[2]; Z += b[2], ++id)
                for (int tx = X; tx < std::min(X + b[0], nb[0]); ++tx)
                    for (int ty = Y; ty < std::min(Y + b[1], nb[1]); ++ty)
                        for (int tz = Z; tz < std::min(Z + b[2], nb[2]); ++tz) {
                            const int x0 = tx * ext[0], y0 = ty * ext[1], z0 = tz * ext[2];
                            v.push_back(TileItem{shot | (meets(0, x0, ext[0]) ? TILE_XB : 0) |
                                                     (meets(1, y0, ext[1]) ? TILE_YB : 0) |
                                                     (meets(2, z0, ext[2]) ? TILE_ZB : 0),
                                                 x0, y0, z0});
                            brick.push_back(id);
                        }
}

// The boxes of several grids (their lo, hi layers) in launch order: each brick goes to the XCD with the
// least work so far (workgroup b runs on XCD b mod 8); a box costs 4 and 3 more for each axis whose band
// it meets, about its instruction count.
struct TileGrid {
    int n[3], lo[3], hi[3], shot;
    size_t boxes() const {
        return (size_t)((n[0] + TILE_X - 1) / TILE_X) * ((n[1] + TILE_Y - 1) / TILE_Y) * ((n[2] + TILE_Z - 1) / TILE_Z);
    }
};
inline std::vector<TileItem> tile_list(const std::vector<TileGrid> &grids) {
    size_t all = 0;
    for (const TileGrid &g : grids) all += g.boxes();
    size_t want = 8;   // a power of two, at least 24 bricks (three per XCD) where there are so many boxes
    while (want < kTileBrick && 2 * want <= all / 24) want *= 2;
    std::vector<TileItem> v;
    std::vector<int> brick;
    v.reserve(all);
    brick.reserve(all);
    for (const TileGrid &g : grids) tile_boxes(g.n, g.lo, g.hi, g.shot, want, v, brick);
    std::vector<TileItem> seq[8];
    long cost[8] = {};
    for (size_t i = 0; i < v.size();) {
        size_t j = i, least = seq[0].size();
        long c = 0;
        for (; j < v.size() && brick[j] == brick[i]; ++j)
            c += 4 + 3 * (!!(v[j].flags & TILE_XB) + !!(v[j].flags & TILE_YB) + !!(v[j].flags & TILE_ZB));
        for (const auto &q : seq) least = std::min(least, q.size());
        int to = -1;   // the XCD with the least work, among those not far ahead in boxes
        for (int x = 0; x < 8; ++x)
            if (seq[x].size() <= least + kTileAhead && (to < 0 || cost[x] < cost[to])) to = x;
        seq[to].insert(seq[to].end(), v.begin() + i, v.begin() + j);
        cost[to] += c;
        i = j;
    }
    size_t rows = 0;
    for (const auto &s : seq) rows = std::max(rows, s.size());
    std::vector<TileItem> out(rows * 8, TileItem{-1, 0, 0, 0});
    for (int x = 0; x < 8; ++x)
        for (size_t i = 0; i < seq[x].size(); ++i) out[i * 8 + x] = seq[x][i];
    while (!out.empty() && out.back().flags < 0) out.pop_back();
    return out;
}
// most items tile_list can give for grids of so many boxes in all (a brick holds less than 2 kTileBrick)
inline size_t tile_list_bound(size_t boxes) { return boxes + 8 * (kTileAhead + 2 * kTileBrick); }
