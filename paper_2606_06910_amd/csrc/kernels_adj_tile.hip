// kernels_adj_tile.hip -- one reverse step of the adjoint sweep in one launch
// (gfx950): the passes k_adj_p1, k_adj_p2 and k_adj_p3 of adjoint.hip in one,
// for every shot of the sweep.
//
// A block owns a box of TILE_X x TILE_Y x TILE_Z points, as k_tile does going
// forward.  Along an axis d whose band the box meets, it forms E_d on the box
// grown by 8 points (from mu^{n+1} and the old zeta_b), W_d on the box grown by
// 4 (from E_d and the old psi_b) and K_d = kinv E_d, all in LDS (x, y) or
// registers (z), and never writes them: a slab point's E, K and W cost 12 bytes
// written and some 50 read per axis and step as arrays.  The new zeta_b and
// psi_b go to the other of two buffers, because the neighbouring blocks read
// the old ones.  Operation for operation the passes' arithmetic (outside the
// slabs kinv = 1 and E = mu, so K is mu there with the same bits, and W is 0).
//
// The residuals that enter mu^n before step n - 1 are added by the block that
// wrote the point, once its box is written: the list says which receiver
// locations lie in the box.  With that, the increments written by the
// recomputed steps themselves and checkpoints saved in one launch, a reverse
// step is two launches and not four: forward and gradient of one shot of 0.89 M
// points, 100 steps, 5.45 -> 4.68 ms; of three shots of 7.7 M, 24.0 -> 22.2 ms.
//
// What bounds it: instruction issue and load latency at four waves per SIMD, as
// in k_tile (119 VGPRs, 31 KB of LDS: E is turned into K where it lies, which
// costs two barriers and saves 13 KB).  Three batched shots of 7.7 M points in
// all (15-cell layers, 64 % of the points in a band): the three passes 36 + 46 +
// 89 us, this kernel 84 us per reverse step (0.26 GB counted: 3.1 TB/s);
// one shot of 0.89 M points: 8.5 + 8.9 + 18 -> 19 us.
#include "adj_tile.hpp"
#include "tile_dev.hpp"

namespace {
constexpr int EXW = TX + 4 * FDTD_R, EYH = TY + 4 * FDTD_R;   // E (then K): 8 points on each side
constexpr int WXW = TX + 2 * FDTD_R, WYH = TY + 2 * FDTD_R;   // W: 4 on each side
typedef __attribute__((address_space(4))) const AdjTile ConstAdj;
}  // namespace

__global__ __launch_bounds__(256, 4) void k_adj_tile(const AdjTile *__restrict__ descs,
                                                     const TileItem *__restrict__ work,
                                                     const AdjGroups *__restrict__ grp, int n, int m0, int m1, int m2) {
    const TileItem wi = work[blockIdx.x];
    if (wi.flags < 0) return;   // the idle items that pad the list
    const ConstAdj &s = *(const ConstAdj *)(uintptr_t)(descs + (wi.flags & 0xff));
    const int t = (int)threadIdx.x;
    const int nx = s.nx, ny = s.ny, nz = s.nz;
    const int x0 = wi.x0, y0 = wi.y0, z0 = wi.z0;
    const int lx = t % TX, ly = t / TX;
    const int x = x0 + lx, y = y0 + ly;
    const bool act = x < nx && y < ny;
    const int xlo = s.Llo[0], xhi = s.Lhi[0], ylo = s.Llo[1], yhi = s.Lhi[1], zlo = s.Llo[2], zhi = s.Lhi[2];
    const int xb = wi.flags & TILE_XB, yb = wi.flags & TILE_YB, zb = wi.flags & TILE_ZB;
    const int old = (n + 1) & 1, cur = n & 1;   // layer buffers read and written by reverse step n

    __shared__ float EX[TZ][TY][EXW];   // E_x at (x0 - 8 + c, y0 + r, z0 + p), mu outside the slabs; then K_x
    __shared__ float EY[TZ][EYH][TX];   // E_y at (x0 + c, y0 - 8 + r, z0 + p); then K_y
    __shared__ float WX[TZ][TY][WXW], WY[TZ][WYH][TX];

    // one descriptor per mu level, for m and for the layer arrays; plane by plane a running scalar offset.
    // Lanes whose position lies outside the frame that every field carries read zero; planes outside it are
    // not read.
    constexpr int F = FDTD_R;
    const Rsrc r1 = make_rsrc(s.mu + (long)m1 * s.mstride), rl = make_rsrc(s.lay);
    const int P = s.P;
    const uint32_t Sb = (uint32_t)s.S * 4u;
    const uint32_t f0 = ((uint32_t)((F + z0) * s.S) + (uint32_t)(kFieldLead - F)) * 4u;
    auto off = [&](int xp, int yp) -> uint32_t {
        return xp >= -F && xp < nx + F && yp >= -F && yp < ny + F ? (uint32_t)((yp + F) * P + xp + F) * 4u : kBufSkip;
    };

    // ---- loads of mu^{n+1} and the old zeta_b ----
    constexpr int QN = TZ + 4 * F;
    float q[QN];   // mu^{n+1} at z0 - 8 .. z0 + TZ + 7 of the column; then E_z; then K_z
    const uint32_t vq = off(x, y), slast = f0 + (uint32_t)(nz + F - 1 - z0) * Sb;
    {
        uint32_t so = f0 - F * Sb;
#pragma unroll
        for (int o = F; o < QN - F; ++o, so += Sb) q[o] = Buf<float>::ld(r1, vq, o < 3 * F ? so : min(so, slast));
    }
    const int yn = ly < F ? y0 - F + ly : y0 + F + ly, yf = ly < F ? yn - F : yn + F;
    const int c8 = t & 7, hr = (t >> 3) & (TY - 1), hp = uniform(t >> 6);
    const int xn = c8 < F ? x0 - F + c8 : x0 + TX - F + c8, xf = c8 < F ? xn - F : xn + F;
    const uint32_t sh = f0 + (uint32_t)hp * Sb;
    float hxn = Buf<float>::ld(r1, off(xn, y0 + hr), sh), hxf;
    float hyn[TZ], hyf[TZ];
    {
        const uint32_t v = off(x, yn);
        uint32_t so = f0;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Sb) hyn[p] = Buf<float>::ld(r1, v, so);
    }
    const Rsrc rpr = make_rsrc(s.prof);
    auto prof = [&](int d, int f, int c) -> float {
        return Buf<float>::ld(rpr, (uint32_t)c * 4u, (uint32_t)((d * 4 + f) * s.nmax) * 4u);
    };
    // x: own column, near halo (W and E), far halo (E)
    const uint32_t Spx = (uint32_t)(s.PY * s.WX) * 4u, fx = (uint32_t)(z0 + F) * Spx;
    bool sx = false, sxn = false, sxf = false;
    uint32_t vx = kBufSkip, vxn = kBufSkip;
    float zx[TZ], zxn, zxf, ax[4], axn[4], axf[4];   // profiles b, a, kinv, dkinv (as far as needed)
    if (xb) {
        const uint32_t side = (uint32_t)(nz + 2 * F) * Spx - (uint32_t)(nx - xhi) * 4u;
        auto xoff = [&](int xp, int yp) -> uint32_t {
            const uint32_t e = (uint32_t)((yp + F) * s.WX + xp) * 4u;
            return xp < xlo ? e : e + side;
        };
        const uint32_t ze = s.t_zetab[old][0] + fx;
        hxf = Buf<float>::ld(r1, off(xf, y0 + hr), sh);
        sx = act && slab_point(x, nx, xlo, xhi);
        sxn = y0 + hr < ny && slab_point(xn, nx, xlo, xhi);
        sxf = y0 + hr < ny && slab_point(xf, nx, xlo, xhi);
        vx = sx ? xoff(x, y) : kBufSkip;
        vxn = sxn ? xoff(xn, y0 + hr) : kBufSkip;
        uint32_t so = ze;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Spx) zx[p] = Buf<float>::ld(rl, vx, so);
        zxn = Buf<float>::ld(rl, vxn, ze + (uint32_t)hp * Spx);
        zxf = Buf<float>::ld(rl, sxf ? xoff(xf, y0 + hr) : kBufSkip, ze + (uint32_t)hp * Spx);
        const int cn = min(max(xn, 0), nx - 1), cf = min(max(xf, 0), nx - 1);
#pragma unroll
        for (int f = 0; f < 4; ++f) ax[f] = prof(0, f, min(x, nx - 1));
#pragma unroll
        for (int f = 1; f < 4; ++f) axn[f] = prof(0, f, cn);
#pragma unroll
        for (int f = 1; f < 3; ++f) axf[f] = prof(0, f, cf);
    }
    // y: the thread's row, its near and its far halo row
    const uint32_t Spy = (uint32_t)(s.SY * nx) * 4u, fy = (uint32_t)(z0 + F) * Spy;
    bool sy = false, syn = false, syf = false;
    uint32_t vy = kBufSkip, vyn = kBufSkip;
    float zy[TZ], zyn[TZ], zyf[TZ], ay[4], ayn[4], ayf[4];
    if (yb) {
        auto yoff = [&](int yp) -> uint32_t { return (uint32_t)(slab_pos(yp, ny, ylo, yhi) * nx + x) * 4u; };
        sy = act && slab_point(y, ny, ylo, yhi);
        syn = x < nx && slab_point(yn, ny, ylo, yhi);
        syf = x < nx && slab_point(yf, ny, ylo, yhi);
        vy = sy ? yoff(y) : kBufSkip;
        vyn = syn ? yoff(yn) : kBufSkip;
        const uint32_t vyf = syf ? yoff(yf) : kBufSkip, vf = off(x, yf);
        uint32_t so = f0, sz = s.t_zetab[old][1] + fy;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Sb, sz += Spy) {
            hyf[p] = Buf<float>::ld(r1, vf, so);
            zy[p] = Buf<float>::ld(rl, vy, sz);
            zyn[p] = Buf<float>::ld(rl, vyn, sz);
            zyf[p] = Buf<float>::ld(rl, vyf, sz);
        }
        const int cn = min(max(yn, 0), ny - 1), cf = min(max(yf, 0), ny - 1);
#pragma unroll
        for (int f = 0; f < 4; ++f) ay[f] = prof(1, f, min(y, ny - 1));
#pragma unroll
        for (int f = 1; f < 4; ++f) ayn[f] = prof(1, f, cn);
#pragma unroll
        for (int f = 1; f < 3; ++f) ayf[f] = prof(1, f, cf);
    }
    // z: the column over z0 - 8 .. z0 + TZ + 7 (bit o of zm: plane z0 - 8 + o lies in a layer; the window meets
    // one layer only); the profiles of those planes, one per lane
    const uint32_t Spz = (uint32_t)(s.PY * nx) * 4u;
    const uint32_t vz = act ? (uint32_t)((y + F) * nx + x) * 4u : kBufSkip;
    uint32_t zm = 0, fz = 0;   // fz: plane z0 - 8 in a z layer array
    float zz[QN], az[4];
    if (zb) {
        const uint32_t zlm = plane_bits<QN>(z0 - 2 * F, 0, zlo);
        zm = zlm | plane_bits<QN>(z0 - 2 * F, nz - zhi, nz);
        fz = (uint32_t)(z0 - 2 * F + (zlm ? 0 : zlo - (nz - zhi))) * Spz;
        // (z0 - 8 .. z0 - 5 of a box at the low face: no tap, read as plane z0)
        uint32_t su = z0 >= F ? f0 - 2 * F * Sb : f0, sv = f0 + (TZ + F) * Sb;
#pragma unroll
        for (int o = 0; o < F; ++o, su += Sb, sv += Sb) {
            q[o] = Buf<float>::ld(r1, vq, su);
            q[TZ + 3 * F + o] = Buf<float>::ld(r1, vq, min(sv, slast));
        }
        uint32_t so = s.t_zetab[old][2] + fz;
#pragma unroll
        for (int o = 0; o < QN; ++o, so += Spz)
            if ((zm >> o) & 1u) zz[o] = Buf<float>::ld(rl, vz, so);
        const int zl = min(max(z0 - 2 * F + (t & 31), 0), nz - 1);
#pragma unroll
        for (int f = 0; f < 4; ++f) az[f] = prof(2, f, zl);
    }

    // ---- E: kinv mu + a (zeta_b + mu) in the slabs, mu elsewhere; zeta_b <- b (zeta_b + mu) ----
    float w1[3][5], w2[3][5];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int l = 0; l < 5; ++l) {
            w1[d][l] = s.w1[d][l];
            w2[d][l] = s.w2[d][l];
        }
    const int np = nz - z0;   // planes of the box inside the grid (TZ or fewer)
    const int rn = ly < F ? ly : ly + TY, rf = ly < F ? rn : rn + 2 * F;   // rows of yn in WY, of yf in EY
    const int cn = c8 < F ? c8 : c8 + TX, cf = c8 < F ? cn : cn + 2 * F;   // columns of xn in WX, of xf in EX
    float c[TZ], ex[TZ], ey[TZ], eyn[TZ], exn;
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        c[p] = ex[p] = ey[p] = q[p + 2 * F];
        eyn[p] = hyn[p];
    }
    exn = hxn;
    auto e_of = [](float lb, float zt, float kinv, float a) { return fmaf(kinv, lb, a * zt); };
    if (again(xb)) {
        const int n1 = again(np);
        const uint32_t ze = s.t_zetab[cur][0] + fx;
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            const float zt = zx[p] + c[p];
            if (sx) ex[p] = e_of(c[p], zt, ax[2], ax[1]);
            if (p < n1) Buf<float>::stc(rl, vx, ze + p * Spx, ax[0] * zt);
        }
        if (sxn) exn = e_of(hxn, zxn + hxn, axn[2], axn[1]);
        EX[hp][hr][cf] = sxf ? e_of(hxf, zxf + hxf, axf[2], axf[1]) : hxf;
    }
    if (again(yb)) {
        const int n1 = again(np);
        const uint32_t ze = s.t_zetab[cur][1] + fy;
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            const float zt = zy[p] + c[p];
            if (sy) ey[p] = e_of(c[p], zt, ay[2], ay[1]);
            if (p < n1) Buf<float>::stc(rl, vy, ze + p * Spy, ay[0] * zt);
            if (syn) eyn[p] = e_of(hyn[p], zyn[p] + hyn[p], ayn[2], ayn[1]);
            EY[p][rf][lx] = syf ? e_of(hyf[p], zyf[p] + hyf[p], ayf[2], ayf[1]) : hyf[p];
        }
    }
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        EX[p][ly][lx + 2 * F] = ex[p];
        EY[p][ly + 2 * F][lx] = ey[p];
        EY[p][rn + F][lx] = eyn[p];
    }
    EX[hp][hr][cn + F] = exn;
    if (again(zb)) {
        const uint32_t z1 = (uint32_t)again((int)zm), ze = s.t_zetab[cur][2] + fz;
#pragma unroll
        for (int o = 0; o < QN; ++o)
            if ((z1 >> o) & 1u) {
                const float zt = zz[o] + q[o];
                if (o >= 2 * F && o < 2 * F + TZ) Buf<float>::stc(rl, vz, ze + o * Spz, lane_value(az[0], o) * zt);
                q[o] = e_of(q[o], zt, lane_value(az[2], o), lane_value(az[1], o));
            }
    }
    // ---- the other loads: old psi_b, mu^{n+2}, m ----
    const Rsrc r2 = make_rsrc(s.mu + (long)m2 * s.mstride), rm = make_rsrc(s.m);
    const uint32_t vc = act ? vq : kBufSkip;
    float second[TZ], mm[TZ], px[TZ], pxn, py[TZ], pyn[TZ], pz[TZ + 2 * F];
    if (again(xb)) {
        const uint32_t po = s.t_psib[old][0] + fx;
        pxn = Buf<float>::ld(rl, vxn, po + (uint32_t)hp * Spx);
#pragma unroll
        for (int p = 0; p < TZ; ++p) px[p] = Buf<float>::ld(rl, vx, po + p * Spx);
    }
    if (again(yb)) {
        const uint32_t po = s.t_psib[old][1] + fy;
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            py[p] = Buf<float>::ld(rl, vy, po + p * Spy);
            pyn[p] = Buf<float>::ld(rl, vyn, po + p * Spy);
        }
    }
    if (again(zb)) {
        const uint32_t z1 = (uint32_t)again((int)zm);
        uint32_t so = s.t_psib[old][2] + fz + F * Spz;
#pragma unroll
        for (int o = 0; o < TZ + 2 * F; ++o, so += Spz) {
            pz[o] = 0.0f;
            if ((z1 >> (o + F)) & 1u) pz[o] = Buf<float>::ld(rl, vz, so);
        }
    }
    {
        uint32_t so = f0;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Sb) {
            second[p] = Buf<float>::ldnt(r2, vc, so);
            mm[p] = Buf<float>::ld(rm, vc, so);
        }
    }
    __syncthreads();

    // ---- W = dkinv E + a (psi_b - D1 E) in the slabs, 0 elsewhere; psi_b <- b (psi_b - D1 E) ----
    if (again(xb)) {
        const int n1 = again(np);
        const uint32_t po = s.t_psib[cur][0] + fx;
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            const float pt = px[p] - d1_lds(&EX[p][ly][lx + 2 * F], 1, w1[0]);
            WX[p][ly][lx + F] = sx ? fmaf(ax[3], ex[p], ax[1] * pt) : 0.0f;
            if (p < n1) Buf<float>::stc(rl, vx, po + p * Spx, ax[0] * pt);
        }
        const float pt = pxn - d1_lds(&EX[hp][hr][cn + F], 1, w1[0]);
        WX[hp][hr][cn] = sxn ? fmaf(axn[3], exn, axn[1] * pt) : 0.0f;
    }
    if (again(yb)) {
        const int n1 = again(np);
        const uint32_t po = s.t_psib[cur][1] + fy;
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            const float pt = py[p] - d1_lds(&EY[p][ly + 2 * F][lx], TX, w1[1]);
            WY[p][ly + F][lx] = sy ? fmaf(ay[3], ey[p], ay[1] * pt) : 0.0f;
            if (p < n1) Buf<float>::stc(rl, vy, po + p * Spy, ay[0] * pt);
            const float pn = pyn[p] - d1_lds(&EY[p][rn + F][lx], TX, w1[1]);
            WY[p][rn][lx] = syn ? fmaf(ayn[3], eyn[p], ayn[1] * pn) : 0.0f;
        }
    }
    float wz[TZ + 2 * F];
    if (again(zb)) {
        const uint32_t z1 = (uint32_t)again((int)zm), po = s.t_psib[cur][2] + fz;
#pragma unroll
        for (int o = 0; o < TZ + 2 * F; ++o) {
            wz[o] = 0.0f;
            if ((z1 >> (o + F)) & 1u) {
                const float pt = pz[o] - d1_lds(&q[o + F], 1, w1[2]);
                wz[o] = fmaf(lane_value(az[3], o + F), q[o + F], lane_value(az[1], o + F) * pt);
                if (o >= F && o < F + TZ)
                    Buf<float>::stc(rl, vz, po + (o + F) * Spz, lane_value(az[0], o + F) * pt);
            }
        }
        // K_z over the taps
#pragma unroll
        for (int o = F; o < QN - F; ++o)
            if ((z1 >> o) & 1u) q[o] = lane_value(az[2], o) * q[o];
    }
    // ---- K = kinv E over the taps (the halo's outer half is not read again) ----
    if (again(xb | yb)) {
        __syncthreads();
        if (again(xb)) {
#pragma unroll
            for (int p = 0; p < TZ; ++p) {
                if (sx) ex[p] = ax[2] * ex[p];
                EX[p][ly][lx + 2 * F] = ex[p];
            }
            EX[hp][hr][cn + F] = sxn ? axn[2] * exn : exn;
        }
        if (again(yb)) {
#pragma unroll
            for (int p = 0; p < TZ; ++p) {
                if (sy) ey[p] = ay[2] * ey[p];
                EY[p][ly + 2 * F][lx] = ey[p];
                EY[p][rn + F][lx] = syn ? ayn[2] * eyn[p] : eyn[p];
            }
        }
        __syncthreads();
    }

    // ---- mu^n = 2 mu^{n+1} - mu^{n+2} + m sum_d [D2 K_d - D1 W_d] ----
    const Rsrc rw = make_rsrc(s.mu + (long)m0 * s.mstride);
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        if (p >= again(np)) break;
        const float *gx = &EX[p][ly][lx + 2 * F], *gy = &EY[p][ly + 2 * F][lx];
        float xl[4], xh[4], yl[4], yh[4], zl[4], zh[4];
#pragma unroll
        for (int l = 1; l <= 4; ++l) {
            xl[l - 1] = gx[-l];
            xh[l - 1] = gx[l];
            yl[l - 1] = gy[-l * TX];
            yh[l - 1] = gy[l * TX];
            zl[l - 1] = q[p + 8 - l];
            zh[l - 1] = q[p + 8 + l];
        }
        float g[3] = {d2_axis(w2[0], ex[p], xl, xh), d2_axis(w2[1], ey[p], yl, yh), d2_axis(w2[2], q[p + 8], zl, zh)};
        if (again(xb)) g[0] = g[0] - d1_lds(&WX[p][ly][lx + F], 1, w1[0]);
        if (again(yb)) g[1] = g[1] - d1_lds(&WY[p][ly + F][lx], TX, w1[1]);
        if (again(zb)) g[2] = g[2] - d1_lds(&wz[p + F], 1, w1[2]);
        Buf<float>::stc(rw, vc, f0 + p * Sb, leapfrog(mm[p], (g[0] + g[1]) + g[2], c[p], second[p]));
    }

    // ---- the residuals that enter mu^n before the next step (as k_adj_resid) ----
    const AdjGroups gr = grp[blockIdx.x];
    if (n == 0 || gr.lo >= gr.hi) return;
    __syncthreads();   // (the points written above)
    const float *row = s.resid + (long)(n - 1) * s.nrec, *m = (const float *)s.m;
    float *mu = (float *)(s.mu + (long)m0 * s.mstride);
    for (int g = gr.lo + t; g < gr.hi; g += 256) {
        const int i = s.gpos[g];
        float r = 0.0f;
        for (int k = s.gstart[g]; k < s.gstart[g + 1]; ++k) r += row[s.ridx[k]];
        mu[i] = fmaf(m[i], r, mu[i]);
    }
}

void fdtd_launch_adj_tile(const AdjTile *descs, const TileItem *work, const AdjGroups *grp, int nwork, int n, int m0,
                          int m1, int m2, hipStream_t st) {
    if (nwork > 0)
        hipLaunchKernelGGL(k_adj_tile, dim3((unsigned)nwork), dim3(256), 0, st, descs, work, grp, n, m0, m1, m2);
}
