// pv_tile.hpp -- what the one-launch first-order step (kernels_pv_tile.hip) and pv_api.hip share.
#pragma once
#include "fdtd_dev.hpp"

// One step of k_pv_tile.  p, v_d and psi_v,d lie in two buffers each, which
// alternate (the neighbouring boxes read the old ones); psi_p,d is updated in
// place.  Pointers are the first bytes of the fields.
struct PvTile {
    const float *in[7];      // p, v_x, v_y, v_z, psi_v x3
    float *out[7];
    float *psp[3];
    const float *prof;       // [axis][b, a, kinv][nmax]
    const float *wav;
    const int32_t *rec;      // receivers of the step before (nrec = 0: none), recorded by extra blocks
    float *row;
    int nrec, nwork;
    int n[3], lo[3], hi[3], src[3];
    int nmax, wav_n, step, P, S;
    float lam;
    float w[5];
};

// work: the boxes of k_pv_tile (g.nwork of them); inner: nin boxes without any layer in reach
void pv_launch_tile(const PvTile &g, const TileItem *work, const TileItem *inner, int nin, hipStream_t st);
