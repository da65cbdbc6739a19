// kernels_pv_tile.hip -- one step of the first-order pressure-velocity system in
// one launch (gfx950): both stages of pv_api.hip on boxes of TILE_X x TILE_Y x
// TILE_Z points.
//
// The pressure stage of a box needs v_d at 4 points on each side along d, which
// the box computes itself from p on 8 points on each side and the old v_d and
// psi_v,d on 4: v^{n+1/2} is never read back (32 instead of 48 bytes per point
// and step from memory) and a step is one launch instead of two.  Operation for
// operation the two stages' arithmetic, so the bits are theirs.
//
// On large grids the boxes out of every layer's reach and inside the grid by their
// halo take a launch of their own, built without layers and edges (IN: 67 VGPRs
// instead of 108, five blocks per CU instead of four).
//
// What bounds it: on small grids the chain of one block, as in k_tile; on large
// ones the halos' traffic (544^3: 4.3 GB read and 2.9 GB written per step, counted,
// 4.7 TB/s; the step cannot do without 5.8 GB; the interior's 118 M points take 950
// us, the other 43 M 565) and 142 VALU instructions per plane of 64 points.
// 31 KB of LDS.  Before (two stages, one thread per point below 256^3, z-marching
// above) and after, us per step: 64^3 13.1 -> 9.3, 96^3 26 -> 16, 131 x 118 x 97 41
// -> 25, 256^3 297 -> 207, 384^3 729 -> 569, 544^3 1921 -> 1508, 640^3 2948 -> 2463.
#include "pv_tile.hpp"
#include "tile_dev.hpp"

namespace {
constexpr int F = FDTD_R;
constexpr int UW = TX + 4 * F, UH = TY + 4 * F;      // p: 8 columns and rows on each side
constexpr int VXW = TX + 2 * F, VYH = TY + 2 * F;    // new v_x, v_y: 4 on each side
template <bool NT> __device__ __forceinline__ void put(Rsrc r, uint32_t vo, uint32_t so, float v) {
    if constexpr (NT) Buf<float>::st(r, vo, so, v);
    else Buf<float>::stc(r, vo, so, v);
}
template <bool NT> __device__ __forceinline__ float once(Rsrc r, uint32_t vo, uint32_t so) {
    return NT ? Buf<float>::ldnt(r, vo, so) : Buf<float>::ld(r, vo, so);
}
}  // namespace

// NT: the non-temporal hint on every store and on the loads of psi_p, on grids that no cache holds from one
// step to the next; IN: boxes whose p halo lies in the frame and v halo in the grid, away from every layer
template <bool NT, bool IN>
__global__ __launch_bounds__(256, IN ? 5 : 4) void k_pv_tile(const PvTile g, const TileItem *__restrict__ work) {
    const int t = (int)threadIdx.x;
    if (!IN && (int)blockIdx.x >= g.nwork) {
        // receivers of the step before this one
        const float *p = g.in[0] + kFieldLead + 4 * (long)g.S + 4 * (long)g.P;
        for (int r = ((int)blockIdx.x - g.nwork) * 256 + t; r < g.nrec; r += 256 * ((int)gridDim.x - g.nwork))
            g.row[r] = p[(long)g.rec[3 * r + 2] * g.S + (long)g.rec[3 * r + 1] * g.P + g.rec[3 * r]];
        return;
    }
    const TileItem wi = work[blockIdx.x];
    if (wi.flags < 0) return;   // the idle items that pad the list
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int x0 = wi.x0, y0 = wi.y0, z0 = wi.z0;
    const int lx = t % TX, ly = t / TX;
    const int x = x0 + lx, y = y0 + ly;
    const bool act = IN || (x < nx && y < ny);
    const int xlo = g.lo[0], xhi = g.hi[0], ylo = g.lo[1], yhi = g.hi[1], zlo = g.lo[2], zhi = g.hi[2];
    // axes along which the box or its v halo meets a layer (psi_v, psi_p)
    const int axes = IN ? 0 : wi.flags;
    const int xb = axes & TILE_XB, yb = axes & TILE_YB, zb = axes & TILE_ZB;
    auto on = [](int b) { return IN ? b : again(b); };

    __shared__ float U[TZ][UH][UW];     // p at (x0 - 8 + c, y0 - 8 + r, z0 + p); corners unused
    __shared__ float VX[TZ][TY][VXW];   // new v_x at (x0 - 4 + c, y0 + r, z0 + p), 0 outside the grid
    __shared__ float VY[TZ][VYH][TX];   // new v_y at (x0 + c, y0 - 4 + r, z0 + p)

    const int P = g.P;
    const uint32_t Sb = (uint32_t)g.S * 4u;
    const uint32_t f0 = ((uint32_t)((F + z0) * g.S) + (uint32_t)(kFieldLead - F)) * 4u;   // plane z0 of a field
    auto elem = [&](int xp, int yp) { return (uint32_t)((yp + F) * P + xp + F) * 4u; };
    // positions outside the zero frame read zero
    auto off = [&](int xp, int yp) -> uint32_t {
        return IN || (xp >= -F && xp < nx + F && yp >= -F && yp < ny + F) ? elem(xp, yp) : kBufSkip;
    };
    auto in_grid = [&](int xp, int yp) { return IN || (xp >= 0 && xp < nx && yp >= 0 && yp < ny); };

    // ---- loads: p on the box grown by 8, v on the box grown by 4 ----
    constexpr int QN = TZ + 4 * F, VN = TZ + 2 * F;
    const Rsrc rp = make_rsrc(g.in[0]);
    float q[QN];   // p at z0 - 8 .. z0 + TZ + 7
    const uint32_t vq = off(x, y), vc = act ? vq : kBufSkip, slast = f0 + (uint32_t)(nz + F - 1 - z0) * Sb;
    {
        // (planes outside the frame are read as the nearest frame plane: no tap of any point of the grid)
        uint32_t so = f0 - F * Sb;
#pragma unroll
        for (int o = F; o < QN; ++o, so += Sb) q[o] = Buf<float>::ld(rp, vq, IN || o < 3 * F ? so : min(so, slast));
        so = IN || z0 >= F ? f0 - 2 * F * Sb : f0;
#pragma unroll
        for (int o = 0; o < F; ++o, so += Sb) q[o] = Buf<float>::ld(rp, vq, so);
    }
    const int yn = ly < F ? y0 - F + ly : y0 + F + ly, yf = ly < F ? yn - F : yn + F;
    const int c8 = t & 7, hr = (t >> 3) & (TY - 1), hp = uniform(t >> 6);
    const int xn = c8 < F ? x0 - F + c8 : x0 + TX - F + c8, xf = c8 < F ? xn - F : xn + F;
    const uint32_t sh = f0 + (uint32_t)hp * Sb;
    const float hxn = Buf<float>::ld(rp, off(xn, y0 + hr), sh), hxf = Buf<float>::ld(rp, off(xf, y0 + hr), sh);
    float hyn[TZ], hyf[TZ];
    {
        const uint32_t v1 = off(x, yn), v2 = off(x, yf);
        uint32_t so = f0;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Sb) {
            hyn[p] = Buf<float>::ld(rp, v1, so);
            hyf[p] = Buf<float>::ld(rp, v2, so);
        }
    }
    const bool gxn = in_grid(xn, y0 + hr), gyn = in_grid(x, yn);
    const uint32_t vxh = gxn ? elem(xn, y0 + hr) : kBufSkip, vyh = gyn ? elem(x, yn) : kBufSkip;
    float vx[TZ], vxn, vy[TZ], vyn[TZ], vz[VN];
    {
        const Rsrc rx = make_rsrc(g.in[1]), ry = make_rsrc(g.in[2]), rz = make_rsrc(g.in[3]);
        vxn = Buf<float>::ld(rx, vxh, sh);
        uint32_t so = f0;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Sb) {
            vx[p] = Buf<float>::ld(rx, vc, so);
            vy[p] = Buf<float>::ld(ry, vc, so);
            vyn[p] = Buf<float>::ld(ry, vyh, so);
        }
        so = f0 - F * Sb;
#pragma unroll
        for (int o = 0; o < VN; ++o, so += Sb) vz[o] = Buf<float>::ld(rz, vc, IN ? so : min(so, slast));
    }
    const Rsrc rpr = make_rsrc(g.prof);
    auto prof = [&](int d, int f, int c) -> float {
        return Buf<float>::ld(rpr, (uint32_t)c * 4u, (uint32_t)((d * 3 + f) * g.nmax) * 4u);
    };
    // psi_v of the layers the box or its v halo meets; profiles b, a, kinv
    bool sx = false, sxn = false, sy = false, syn = false;
    float px[TZ], pxn, py[TZ], pyn[TZ], pz[VN], ax[3], axn[3], ay[3], ayn[3], az[3];
    if (xb) {
        const Rsrc r = make_rsrc(g.in[4]);
        sx = act && in_slab(x, nx, xlo, xhi);
        sxn = gxn && in_slab(xn, nx, xlo, xhi);
        pxn = Buf<float>::ld(r, sxn ? vxh : kBufSkip, sh);
#pragma unroll
        for (int p = 0; p < TZ; ++p) px[p] = Buf<float>::ld(r, sx ? vc : kBufSkip, f0 + p * Sb);
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            ax[f] = prof(0, f, min(x, nx - 1));
            axn[f] = prof(0, f, min(max(xn, 0), nx - 1));
        }
    }
    if (yb) {
        const Rsrc r = make_rsrc(g.in[5]);
        sy = act && in_slab(y, ny, ylo, yhi);
        syn = gyn && in_slab(yn, ny, ylo, yhi);
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            py[p] = Buf<float>::ld(r, sy ? vc : kBufSkip, f0 + p * Sb);
            pyn[p] = Buf<float>::ld(r, syn ? vyh : kBufSkip, f0 + p * Sb);
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            ay[f] = prof(1, f, min(y, ny - 1));
            ayn[f] = prof(1, f, min(max(yn, 0), ny - 1));
        }
    }
    // z: bit o of zm: plane z0 - 4 + o lies in a layer; of zg: it lies in the grid
    const uint32_t zg = IN ? (1u << VN) - 1u : plane_bits<VN>(z0 - F, 0, nz);
    uint32_t zm = 0;
    if (zb) {
        zm = (plane_bits<VN>(z0 - F, 0, zlo) | plane_bits<VN>(z0 - F, nz - zhi, nz));
        const Rsrc r = make_rsrc(g.in[6]);
        uint32_t so = f0 - F * Sb;
#pragma unroll
        for (int o = 0; o < VN; ++o, so += Sb)
            if ((zm >> o) & 1u) pz[o] = Buf<float>::ld(r, vc, so);
        const int zl = min(max(z0 - F + (t & 15), 0), nz - 1);
#pragma unroll
        for (int f = 0; f < 3; ++f) az[f] = prof(2, f, zl);
    }

    // ---- p to LDS ----
    const int rn = ly < F ? ly : ly + TY, cn = c8 < F ? c8 : c8 + TX;   // row of yn in VY, column of xn in VX
    float *const Uc = &U[0][ly + 2 * F][lx + 2 * F];
    constexpr int UP = UH * UW;
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        Uc[p * UP] = q[p + 2 * F];
        U[p][rn + F][lx + 2 * F] = hyn[p];
        U[p][ly < F ? rn : rn + 2 * F][lx + 2 * F] = hyf[p];
    }
    U[hp][hr + 2 * F][cn + F] = hxn;
    U[hp][hr + 2 * F][c8 < F ? cn : cn + 2 * F] = hxf;
    float w[5];
#pragma unroll
    for (int l = 0; l < 5; ++l) w[l] = g.w[l];
    const float nlam = -g.lam;
    const int np = IN ? TZ : nz - z0;   // planes of the box inside the grid (TZ or fewer)
    // kinv grad + psi, psi <- b psi + a grad first; grad outside the layer
    auto stretched = [](float grad, float &psi, float b, float a, float kinv) {
        psi = fmaf(b, psi, a * grad);
        return fmaf(kinv, grad, psi);
    };
    // v_z along the column
    {
        const Rsrc ro = make_rsrc(g.out[3]), rq = make_rsrc(g.out[6]);
        const uint32_t z1 = zm;
#pragma unroll
        for (int o = 0; o < VN; ++o) {
            float gr = d1_lds(&q[o + F], 1, w);
            if ((z1 >> o) & 1u) {
                gr = stretched(gr, pz[o], lane_value(az[0], o), lane_value(az[1], o), lane_value(az[2], o));
                if (o >= F && o < F + TZ) put<NT>(rq, vc, f0 + (o - F) * Sb, pz[o]);
            }
            vz[o] = (zg >> o) & 1u ? fmaf(nlam, gr, vz[o]) : 0.0f;
            if (o >= F && o < F + TZ && o - F < on(np)) put<NT>(ro, vc, f0 + (o - F) * Sb, vz[o]);
        }
    }
    __syncthreads();
    // ---- v_x, v_y on the box grown by 4; the box's own is stored ----
    {
        const Rsrc ro = make_rsrc(g.out[1]), rq = make_rsrc(g.out[4]);
        const int n1 = on(np), b1 = on(xb);
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            float gr = d1_lds(Uc + p * UP, 1, w);
            if (b1) {
                const float s1 = stretched(gr, px[p], ax[0], ax[1], ax[2]);
                if (sx) gr = s1;
                if (p < n1) put<NT>(rq, sx ? vc : kBufSkip, f0 + p * Sb, px[p]);
            }
            const float v = act ? fmaf(nlam, gr, vx[p]) : 0.0f;
            VX[p][ly][lx + F] = v;
            if (p < n1) put<NT>(ro, vc, f0 + p * Sb, v);
        }
        float gr = d1_lds(&U[hp][hr + 2 * F][cn + F], 1, w);
        if (b1) {
            const float s1 = stretched(gr, pxn, axn[0], axn[1], axn[2]);
            if (sxn) gr = s1;
        }
        VX[hp][hr][cn] = gxn ? fmaf(nlam, gr, vxn) : 0.0f;
    }
    {
        const Rsrc ro = make_rsrc(g.out[2]), rq = make_rsrc(g.out[5]);
        const int n1 = on(np), b1 = on(yb);
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            float gr = d1_lds(Uc + p * UP, UW, w), gn = d1_lds(&U[p][rn + F][lx + 2 * F], UW, w);
            if (b1) {
                const float s1 = stretched(gr, py[p], ay[0], ay[1], ay[2]);
                const float s2 = stretched(gn, pyn[p], ayn[0], ayn[1], ayn[2]);
                if (sy) gr = s1;
                if (syn) gn = s2;
                if (p < n1) put<NT>(rq, sy ? vc : kBufSkip, f0 + p * Sb, py[p]);
            }
            const float v = act ? fmaf(nlam, gr, vy[p]) : 0.0f;
            VY[p][ly + F][lx] = v;
            VY[p][rn][lx] = gyn ? fmaf(nlam, gn, vyn[p]) : 0.0f;
            if (p < n1) put<NT>(ro, vc, f0 + p * Sb, v);
        }
    }
    // psi_p of the box
    float ox[TZ], oy[TZ], oz[TZ];
    if (on(xb)) {
        const Rsrc r = make_rsrc(g.psp[0]);
#pragma unroll
        for (int p = 0; p < TZ; ++p) ox[p] = once<NT>(r, sx ? vc : kBufSkip, f0 + p * Sb);
    }
    if (on(yb)) {
        const Rsrc r = make_rsrc(g.psp[1]);
#pragma unroll
        for (int p = 0; p < TZ; ++p) oy[p] = once<NT>(r, sy ? vc : kBufSkip, f0 + p * Sb);
    }
    if (on(zb)) {
        const Rsrc r = make_rsrc(g.psp[2]);
        const uint32_t z1 = (uint32_t)on((int)zm);
#pragma unroll
        for (int p = 0; p < TZ; ++p)
            if ((z1 >> (p + F)) & 1u) oz[p] = once<NT>(r, vc, f0 + p * Sb);
    }
    __syncthreads();

    // ---- pressure ----
    const Rsrc ro = make_rsrc(g.out[0]), qx = make_rsrc(g.psp[0]), qy = make_rsrc(g.psp[1]), qz = make_rsrc(g.psp[2]);
    const bool src = g.wav && g.step < g.wav_n && x == g.src[0] && y == g.src[1];
    float sw = 0.0f;
    if (src) sw = g.wav[g.step];
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        if (p >= on(np)) break;
        float gx = d1_lds(&VX[p][ly][lx + F], 1, w), gy = d1_lds(&VY[p][ly + F][lx], TX, w),
              gz = d1_lds(&vz[p + F], 1, w);
        if (on(xb)) {
            const float s1 = stretched(gx, ox[p], ax[0], ax[1], ax[2]);
            if (sx) gx = s1;
            put<NT>(qx, sx ? vc : kBufSkip, f0 + p * Sb, ox[p]);
        }
        if (on(yb)) {
            const float s1 = stretched(gy, oy[p], ay[0], ay[1], ay[2]);
            if (sy) gy = s1;
            put<NT>(qy, sy ? vc : kBufSkip, f0 + p * Sb, oy[p]);
        }
        if (((uint32_t)on((int)zm) >> (p + F)) & 1u) {
            gz = stretched(gz, oz[p], lane_value(az[0], p + F), lane_value(az[1], p + F), lane_value(az[2], p + F));
            put<NT>(qz, vc, f0 + p * Sb, oz[p]);
        }
        float div = 0.0f;
        div += gx;
        div += gy;
        div += gz;
        float pn = fmaf(nlam, div, q[p + 2 * F]);
        if (src && z0 + p == g.src[2]) pn = fmaf(g.lam, sw, pn);
        put<NT>(ro, vc, f0 + p * Sb, pn);
    }
}

void pv_launch_tile(const PvTile &g, const TileItem *work, const TileItem *inner, int nin, hipStream_t st) {
    const int rb = g.nrec > 0 ? (g.nrec + 255) / 256 : 0;
    // the hint pays once the 17 fields (68 bytes per point) outgrow the 256 MiB last-level cache by half: us per
    // step without / with it, 128^3 28.7 / 34.7, 192^3 90 / 87, 256^3 214 / 204, 384^3 632 / 594, 544^3 1742 / 1668
    const bool nt = (double)g.n[0] * g.n[1] * g.n[2] >= 6e6;
    if (nin > 0) hipLaunchKernelGGL((k_pv_tile<true, true>), dim3((unsigned)nin), dim3(256), 0, st, g, inner);
    const dim3 grid((unsigned)(g.nwork + rb));
    if (g.nwork + rb == 0) return;
    if (nt) hipLaunchKernelGGL((k_pv_tile<true, false>), grid, dim3(256), 0, st, g, work);
    else hipLaunchKernelGGL((k_pv_tile<false, false>), grid, dim3(256), 0, st, g, work);
}
