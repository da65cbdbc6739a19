// Host-only brute force over random sets of grids: the box lists of the tile
// kernels (tile_list), for every plan of boxes in use.  The boxes of all parts
// cover each grid point exactly once; every list item starts inside its grid; the
// boxes of the inner region lie inside the grid, start on multiples of their
// width and meet no band, nor the rim that TileGrid::least keeps free; those of
// k_face meet one band at most; each other box carries the axes whose band it
// meets; and no list is longer than tile_list_bound says.  Prints "ok <cases>
// <inner boxes> <face boxes>".  With "inner", reads lines of nx ny nz, six layer
// widths, box width and depth, and prints the points of the inner region.
#include "tile_host.hpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

namespace {
unsigned long long g_seed = 12345;
int rnd(int lo, int hi) {   // [lo, hi]
    g_seed = g_seed * 6364136223846793005ull + 1442695040888963407ull;
    return lo + (int)((g_seed >> 33) % (unsigned)(hi - lo + 1));
}
bool band(const TileGrid &g, int d, int c) {   // c in the band of axis d
    return (g.lo[d] > 0 && c < g.lo[d] + FDTD_R) || (g.hi[d] > 0 && c >= g.n[d] - g.hi[d] - FDTD_R);
}
int fail(const char *what, int k) {
    printf("FAIL %s (case %d)\n", what, k);
    return 1;
}
int inner_points() {
    TileGrid g{};
    InnerBox ib;
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d", &g.n[0], &g.n[1], &g.n[2], &g.lo[0], &g.hi[0], &g.lo[1], &g.hi[1],
                 &g.lo[2], &g.hi[2], &ib.x, &ib.z) == 11) {
        long n = 0;
        for (const TileItem &w : tile_list({g}, ib, TILE_INNER)) n += w.flags < 0 ? 0 : (long)ib.x * TILE_Y * ib.z;
        printf("%ld\n", n);
    }
    return 0;
}
}  // namespace

int main(int argc, char **argv) {
    if (argc > 1 && !strcmp(argv[1], "inner")) return inner_points();
    const int cases = argc > 1 ? atoi(argv[1]) : 100;
    const InnerBox plans[] = {{TILE_X, 0, false}, {TILE_X, 8, false}, {TILE_X, 16, false},
                              {2 * TILE_X, 8, true}, {TILE_X, TILE_Z, false}};
    long inner_boxes = 0, face_boxes = 0;
    for (int k = 0; k < cases; ++k) {
        const InnerBox ib = plans[k % 5];
        const bool pv = k % 5 == 4;
        std::vector<TileGrid> grids;
        const int many = pv ? 1 : rnd(1, 5);
        for (int s = 0; s < many; ++s) {
            TileGrid g{};
            g.shot = 12 * s + rnd(0, 11);
            g.least = pv ? FDTD_R : 0;
            for (int d = 0; d < 3; ++d) {
                g.n[d] = rnd(0, 4) ? rnd(9, 110) : rnd(9, 30);
                const int most = rnd(0, 2) ? (g.n[d] - 1) / 2 : std::min(20, (g.n[d] - 1) / 2);
                g.lo[d] = rnd(0, 3) ? rnd(0, most) : 0;
                g.hi[d] = rnd(0, 3) ? rnd(0, most) : 0;
            }
            grids.push_back(g);
        }
        size_t boxes = 0;
        std::vector<std::vector<unsigned char>> seen;
        for (const TileGrid &g : grids) {
            boxes += g.boxes();
            seen.emplace_back((size_t)g.n[0] * g.n[1] * g.n[2]);
        }
        for (int part = 0; part < 3; ++part) {
            const std::vector<TileItem> list = tile_list(grids, ib, (TilePart)part);
            if (list.size() > tile_list_bound(boxes)) return fail("list above its bound", k);
            for (const TileItem &w : list) {
                if (w.flags < 0) continue;
                size_t s = 0;
                while (s < grids.size() && grids[s].shot != (w.flags & 0xff)) ++s;
                if (s == grids.size()) return fail("unknown shot", k);
                const TileGrid &g = grids[s];
                const int c[3] = {w.x0, w.y0, w.z0};
                const int ext[3] = {part == TILE_INNER ? ib.x : TILE_X, TILE_Y, part == TILE_INNER ? ib.z : TILE_Z};
                bool meets[3] = {false, false, false};
                for (int d = 0; d < 3; ++d) {
                    if (c[d] < 0 || c[d] >= g.n[d]) return fail("box outside the grid", k);
                    for (int p = c[d]; p < std::min(c[d] + ext[d], g.n[d]); ++p) meets[d] = meets[d] || band(g, d, p);
                }
                const int flags = (meets[0] ? TILE_XB : 0) | (meets[1] ? TILE_YB : 0) | (meets[2] ? TILE_ZB : 0);
                if ((w.flags & ~0xff) != flags) return fail("band flags", k);
                if (part == TILE_INNER) {
                    ++inner_boxes;
                    if (flags || w.x0 % ib.x) return fail("inner box in a band or off its multiple", k);
                    // (k_pv_tile: the v halo, 4 points, in the grid and out of every layer; one layer or rim)
                    for (int d = 0; d < 3; ++d) {
                        const int l = g.least ? std::max(g.lo[d], g.least) + FDTD_R : 0;
                        const int h = g.least ? std::max(g.hi[d], g.least) + FDTD_R : 0;
                        if (c[d] < l || c[d] + ext[d] > g.n[d] - h) return fail("inner box at the rim", k);
                    }
                }
                if (part == TILE_FACES) {
                    ++face_boxes;
                    if (meets[0] + meets[1] + meets[2] > 1) return fail("face box in two bands", k);
                }
                for (int z = c[2]; z < std::min(c[2] + ext[2], g.n[2]); ++z)
                    for (int y = c[1]; y < std::min(c[1] + ext[1], g.n[1]); ++y)
                        for (int x = c[0]; x < std::min(c[0] + ext[0], g.n[0]); ++x)
                            if (seen[s][((size_t)z * g.n[1] + y) * g.n[0] + x]++) return fail("point covered twice", k);
            }
        }
        for (const auto &v : seen)
            for (const unsigned char b : v)
                if (b != 1) return fail("point not covered", k);
    }
    // bounds where one XCD's list runs ahead: many boxes, bricks of very different weight
    for (int k = 0; k < 40; ++k) {
        TileGrid g{};
        for (int d = 0; d < 3; ++d) {
            g.n[d] = rnd(9, d == 0 ? 700 : 400);
            g.lo[d] = rnd(0, (g.n[d] - 1) / 2);
            g.hi[d] = rnd(0, (g.n[d] - 1) / 2);
        }
        for (int part = 0; part < 3; ++part)
            if (tile_list({g}, plans[k % 4], (TilePart)part).size() > tile_list_bound(g.boxes()))
                return fail("long list above its bound", k);
    }
    printf("ok %d %ld %ld\n", cases, inner_boxes, face_boxes);
    return 0;
}
