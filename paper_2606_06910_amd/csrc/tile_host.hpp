// tile_host.hpp -- box lists of the kernels that work on TILE_X x TILE_Y x TILE_Z
// boxes (host side, shared by the second- and first-order paths).
#pragma once
#include "fdtd_dev.hpp"

#include <algorithm>
#include <vector>

// Boxes of a brick (tile_boxes) on a large grid.  One XCD runs about 128 boxes at a time; measured on the
// first-order step at 544^3 with cubic bricks (us per step): columns of boxes along z 1842, bricks of 32 boxes
// 1868, 128 1859, 256 1742, 512 1749 (counted reads 7.4 GB in columns, 5.8 GB in bricks of 256).
constexpr size_t kTileBrick = 256;
constexpr size_t kTileAhead = 1024;  // boxes one XCD's list may be ahead of another's

// The boxes of one launch: those of the inner region (k_inner), the others that meet one band at most (k_face) and
// the rest (k_tile).
enum TilePart { TILE_INNER, TILE_FACES, TILE_EDGES };
// One grid's boxes: its size, its layers, the number its items carry.
struct TileGrid {
    int n[3], lo[3], hi[3], shot;
    int least = 0;   // the inner region keeps off a face as if its layer were so thick at least
    size_t boxes() const {
        return (size_t)((n[0] + TILE_X - 1) / TILE_X) * ((n[1] + TILE_Y - 1) / TILE_Y) * ((n[2] + TILE_Z - 1) / TILE_Z);
    }
    // the inner region for k_inner's boxes of ib.x x TILE_Y x ib.z points: whole boxes inside the grid that meet no
    // band, first points on multiples of ib.x (16-bit stores of half a line are slow: 768^3 FP16 2090 -> 1645 us per
    // step) and of k_tile's boxes; false if empty
    bool inner(InnerBox ib, int r0[3], int r1[3]) const {
        const int ext[3] = {ib.x, TILE_Y, TILE_Z};
        for (int d = 0; d < 3; ++d) {
            const int l = std::max(lo[d], least), h = std::max(hi[d], least);
            const int a = l > 0 ? l + FDTD_R : 0, b = h > 0 ? n[d] - h - FDTD_R : n[d];
            r0[d] = (a + ext[d] - 1) / ext[d] * ext[d];
            r1[d] = b / ext[d] * ext[d];
        }
        r1[2] = r0[2] + (r1[2] - r0[2]) / ib.z * ib.z;
        return r0[0] < r1[0] && r0[1] < r1[1] && r0[2] < r1[2];
    }
};

// Boxes in bricks: a brick is the set of boxes that run on one XCD at about the same time, grown (by doubling
// one side at a time) to `want` boxes of the least halo.  A halo of 4 to 8 points costs as many rows or planes
// along y and z but a whole 128-byte line on each side along x, so x sides grow to 8 times the others (us per
// step, cubes of boxes against this: 300^3 170 -> 161, first-order 544^3 1610 -> 1556).  The region of the grid
// is [r0, r1) in boxes of ext points, less the inner region [x0, x1) where given; `brick` receives each box's
// brick number, and each box is marked with the axes whose band (layer and 4 points) it meets.
inline void tile_boxes(const TileGrid &g, const int ext[3], const int r0[3], const int r1[3], const int *x0,
                       const int *x1, TilePart part, size_t want, std::vector<TileItem> &v,
                       std::vector<int> &brick) {
    const int wt[3] = {8, 1, 1};
    int nb[3], b[3] = {1, 1, 1};
    for (int d = 0; d < 3; ++d) nb[d] = (r1[d] - r0[d] + ext[d] - 1) / ext[d];
    while ((size_t)b[0] * b[1] * b[2] < want) {
        int s = -1;   // the side that can still grow and whose faces cost most
        for (int d = 2; d >= 0; --d)
            if (b[d] < nb[d] && (s < 0 || b[d] * ext[d] * wt[s] < b[s] * ext[s] * wt[d])) s = d;
        if (s < 0) break;
        b[s] *= 2;
    }
    auto meets = [&](int d, int c0) {
        const int c1 = std::min(c0 + ext[d], g.n[d]);
        return (g.lo[d] > 0 && c0 < g.lo[d] + FDTD_R) || (g.hi[d] > 0 && c1 > g.n[d] - g.hi[d] - FDTD_R);
    };
    int id = brick.empty() ? 0 : brick.back() + 1;
    for (int X = 0; X < nb[0]; X += b[0])
        for (int Y = 0; Y < nb[1]; Y += b[1])
            for (int Z = 0; Z < nb[2]; Z += b[2], ++id)
                for (int tx = X; tx < std::min(X + b[0], nb[0]); ++tx)
                    for (int ty = Y; ty < std::min(Y + b[1], nb[1]); ++ty)
                        for (int tz = Z; tz < std::min(Z + b[2], nb[2]); ++tz) {
                            const int c[3] = {r0[0] + tx * ext[0], r0[1] + ty * ext[1], r0[2] + tz * ext[2]};
                            bool skip = x0 != nullptr;
                            for (int d = 0; skip && d < 3; ++d) skip = c[d] >= x0[d] && c[d] < x1[d];
                            if (skip) continue;
                            const bool m[3] = {meets(0, c[0]), meets(1, c[1]), meets(2, c[2])};
                            const bool edge = m[0] + m[1] + m[2] > 1;
                            if ((part == TILE_FACES && edge) || (part == TILE_EDGES && !edge)) continue;
                            v.push_back(TileItem{g.shot | (m[0] ? TILE_XB : 0) | (m[1] ? TILE_YB : 0) |
                                                     (m[2] ? TILE_ZB : 0),
                                                 c[0], c[1], c[2]});
                            brick.push_back(id);
                        }
}

// The boxes of several grids in launch order: each brick goes to the XCD with the least work so far (workgroup
// b runs on XCD b mod 8); a box costs 4 and 3 more for each axis whose band it meets, about its instruction
// count.  A part that has no launch of its own is empty, its boxes in the next.
inline std::vector<TileItem> tile_list(const std::vector<TileGrid> &grids, InnerBox ib = {}, TilePart part = TILE_EDGES) {
    if ((part == TILE_INNER && ib.z == 0) || (part == TILE_FACES && !ib.face)) return {};
    const bool inner = part == TILE_INNER;
    const int ext[3] = {inner ? ib.x : TILE_X, TILE_Y, inner ? ib.z : TILE_Z}, zero[3] = {0, 0, 0};
    size_t all = 0;
    for (const TileGrid &g : grids) all += g.boxes() * TILE_X * TILE_Z / (ext[0] * ext[2]);
    size_t want = 8;   // a power of two, at least 24 bricks (three per XCD) where there are so many boxes
    while (want < kTileBrick && 2 * want <= all / 24) want *= 2;
    std::vector<TileItem> v;
    std::vector<int> brick;
    v.reserve(all);
    brick.reserve(all);
    for (const TileGrid &g : grids) {
        int r0[3], r1[3];
        const bool has = ib.z > 0 && g.inner(ib, r0, r1);
        // (TILE_INNER: no box is left out)
        if (inner && has) tile_boxes(g, ext, r0, r1, nullptr, nullptr, part, want, v, brick);
        if (!inner) tile_boxes(g, ext, zero, g.n, has ? r0 : nullptr, r1, ib.face ? part : TILE_INNER, want, v, brick);
    }
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
inline size_t tile_list_bound(size_t boxes) { return boxes + 8 * std::min(kTileAhead + 2 * kTileBrick, boxes); }
