// adj_tile.hpp -- what the one-launch reverse step (kernels_adj_tile.hip) and the adjoint's host code share.
#pragma once
#include "fdtd_dev.hpp"

// One shot of a sweep as k_adj_tile sees it.  zeta_b and psi_b of every axis lie
// in two buffers each, which alternate: reverse step n reads buffer (n + 1) & 1
// and writes buffer n & 1.
struct AdjTile {
    const char *mu;          // ring slot 0 of the mu levels (first byte of the field)
    long mstride;            // bytes between ring slots
    const char *m;           // first byte of the field
    const char *lay;         // the layer arrays at the offsets below (32 bits reach them all)
    uint32_t t_zetab[2][3], t_psib[2][3];
    const float *prof;
    int nx, ny, nz, P, PY, S, WX, SY, nmax;
    int Llo[3], Lhi[3];
    float w2[3][5], w1[3][5];
    // receivers grouped by location: element of a field, receivers ridx[gstart[g]] .. of the group
    const int *gpos, *gstart, *ridx;
    const float *resid;      // dJ/dtraces [nt][nrec]
    int nrec;
};

// groups of the receivers that lie in a box of the list
struct AdjGroups {
    int lo, hi;
};

void fdtd_launch_adj_tile(const AdjTile *descs, const TileItem *work, const AdjGroups *grp, int nwork, int n, int m0,
                          int m1, int m2, hipStream_t st);
