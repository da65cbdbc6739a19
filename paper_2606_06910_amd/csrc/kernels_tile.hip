// kernels_tile.hip -- one leapfrog step of a shot in one launch (k_tile), or on
// large grids two or three: k_inner for the boxes outside every band, in 16-bit
// storage k_face for the other boxes that meet one band at most, k_tile for the
// rest (gfx950).
//
// A block of k_tile owns a box of TILE_X x TILE_Y x TILE_Z points, inside or outside the
// layers, and does the whole step there: psi, zeta and u^{n+1} (paper, section
// "CPML Boundary Layers"; the arithmetic is lap_point's, operation for
// operation, so the bits are those of every other variant).  psi_d at the
// neighbours along d is recomputed from u^n and the old psi_d of the box grown
// by 4 points along d (the u^n box grown by 8), so no pass has to come before
// the update; the new psi goes to the other of two psi buffers (the old one is
// still being read by the neighbouring blocks).  Receivers of a step are
// recorded by extra blocks of the next step's launch.
//
// What bounds it: at 64^3 (one block per CU) the chain of one block: launch,
// list item, loads, two barriers, stores; from 128^3 up instruction issue (117
// VALU and 90 scalar instructions per plane of 64 points on a 160^3 grid with
// 20-cell layers, VALU busy 33 % of the time) and the load latency that four waves
// per SIMD leave open.
// Why this box: 32 points are a 128-byte line; 4 planes keep the column (20
// planes of u^n), its old psi and the second state within 114 VGPRs and the
// three LDS arrays within 31 KB, so that four blocks share a CU; asking for
// five spills 21 VGPRs (160^3: 28.7 -> 43 us per step).  Every load is issued
// before the first wait, and one buffer descriptor covers the whole shot
// (seven of them, and tests kept in scalar register pairs, cost 30 scalar
// spills and 10 %).  Per step, before (psi passes, naive or z-march and band
// kernels, record) and after: 64^3 19.5 -> 8.0 us, 101 x 87 x 119 (eager) 38 ->
// 14 us, 160^3 100 -> 29 us (142 Gpts/s, 4.0 TB/s of the algorithmic bytes), 24
// batched shots of 96 .. 288 points per axis, with k_inner, 1.45 -> 1.14 ms.
#include "fdtd_launch.hpp"
#include "tile_dev.hpp"

#include <type_traits>

namespace {
constexpr int UW = TX + 4 * FDTD_R, UH = TY + 4 * FDTD_R;   // LDS plane of u^n: 8 columns and rows on each side
constexpr int PXW = TX + 2 * FDTD_R, PYH = TY + 2 * FDTD_R; // new psi_x rows, new psi_y columns: 4 on each side
// the descriptors read as constant memory: no store of the kernel changes them, so they may be loaded at once
typedef __attribute__((address_space(4))) const TileDesc ConstDesc;
constexpr int AX_ANY = TILE_XB | TILE_YB | TILE_ZB;
// The descriptor of a box's shot.  ONE: a launch over one shot, descs its descriptor, which then loads beside the
// list item and not after it.  Always read from the device, where a new source or model goes: captured steps stay
// valid.
template <bool ONE> __device__ __forceinline__ const ConstDesc &shot_desc(const TileDesc *descs, const TileItem &wi) {
    return *(const ConstDesc *)(uintptr_t)(descs + (ONE ? 0 : wi.flags & 0xff));
}
}  // namespace

// one box.  INC: the
// increment u^{n+1} - u^n is stored too (an adjoint sweep keeps it), 4 bytes per
// point here against 12 in a pass of its own; a template flag, because as a test in
// the kernel it cost plain steps 1 % (160^3).  AX: the axes whose band the box meets
// (TILE_XB etc.), or AX_ANY, where the item says which.
template <typename T, int AX, bool NT, bool INC>
__device__ __forceinline__ void tile_box(const ConstDesc &s, const TileItem &wi, const TileStep &A,
                                         const int *__restrict__ stepc, float *lds) {
    const int t = (int)threadIdx.x;
    const int nx = s.nx, ny = s.ny, nz = s.nz;
    const int x0 = wi.x0, y0 = wi.y0, z0 = wi.z0;
    const int lx = t % TX, ly = t / TX;
    const int x = x0 + lx, y = y0 + ly;
    const bool act = x < nx && y < ny;
    const int xlo = s.Llo[0], xhi = s.Lhi[0], ylo = s.Llo[1], yhi = s.Lhi[1], zlo = s.Llo[2], zhi = s.Lhi[2];
    // axes whose band the box meets: only these need psi, zeta and the wider u^n halo
    const int axes = AX == AX_ANY ? wi.flags : AX;
    const int xb = axes & TILE_XB, yb = axes & TILE_YB, zb = axes & TILE_ZB;
    auto on = [](int b) { return AX == AX_ANY ? again(b) : b; };

    // u^n at (x0 - 8 + c, y0 - 8 + r, z0 + p), corners unused; new psi_x at (x0 - 4 + c, y0 + r, z0 + p) and new psi_y
    // at (x0 + c, y0 - 4 + r, z0 + p), 0 outside the slabs (one place for both where a box has one of them at most)
    auto U = (float (*)[UH][UW])lds;
    auto PX = (float (*)[TY][PXW])(lds + TZ * UH * UW);
    auto PY = (float (*)[PYH][TX])(lds + TZ * UH * UW + (AX == AX_ANY ? TZ * TY * PXW : 0));

    // One descriptor per field, based 8 planes before the box, and one for the layer arrays and profiles (32-bit
    // offsets reach them all, the tile rule sees to it): position at a lane offset, plane by plane a running
    // scalar offset.  Lanes whose position lies outside the frame that every field carries read zero; planes
    // outside it are not read.
    const int P = s.P, esz = (int)sizeof(T), fy = s.fy, fz = s.fz;
    const long base = (long)(fz + z0 - 2 * FDTD_R) * s.S;
    const Rsrc ru = make_rsrc(s.u[A.iu] + base * esz), rl = make_rsrc(s.lay);
    const uint32_t Sb = (uint32_t)s.S * (uint32_t)esz, Smb = (uint32_t)s.S * 4u;
    // offset of (-4, -fy, z0) from a field's first byte: with elem() below, of (x, y, z0)
    const uint32_t lead = (uint32_t)(2 * FDTD_R * s.S) + (uint32_t)(kFieldLead - FDTD_R);
    const uint32_t fu = lead * esz, fm = lead * 4u;
    auto elem = [&](int xp, int yp) { return (uint32_t)((yp + fy) * P + xp + FDTD_R); };
    auto off = [&](int xp, int yp) -> uint32_t {
        return xp >= -FDTD_R && xp < nx + FDTD_R && yp >= -fy && yp < ny + fy ? elem(xp, yp) * (uint32_t)esz : kBufSkip;
    };

    // ---- every load of the box, before anything waits ----
    // own column: u^n at z0 - 8 .. z0 + TZ + 7 (the outer 4 on each side only for psi_z); a plane past the
    // frame (no tap of any point of the grid) is read as the last frame plane
    constexpr int QN = TZ + 4 * FDTD_R;
    float q[QN];
    const uint32_t vq = off(x, y);
    const uint32_t slast = fu + (uint32_t)(nz + fz - 1 - z0) * Sb;
    {
        uint32_t so = fu - FDTD_R * Sb;
#pragma unroll
        for (int o = FDTD_R; o < QN - FDTD_R; ++o, so += Sb) q[o] = Buf<T>::ld(ru, vq, o < 3 * FDTD_R ? so : min(so, slast));
    }
    // y halo: 4 rows above and below the box, then the next 4 for psi_y: one row of each per thread
    const int yn = ly < FDTD_R ? y0 - FDTD_R + ly : y0 + FDTD_R + ly;
    const int yf = ly < FDTD_R ? yn - FDTD_R : yn + FDTD_R;
    // x halo: 4 columns left and right of the box, then the next 4 for psi_x; wave w takes plane w
    const int c8 = t & 7, hr = (t >> 3) & (TY - 1), hp = uniform(t >> 6);
    const int xn = c8 < FDTD_R ? x0 - FDTD_R + c8 : x0 + TX - FDTD_R + c8;
    const int xf = c8 < FDTD_R ? xn - FDTD_R : xn + FDTD_R;
    const uint32_t sh = fu + (uint32_t)hp * Sb;
    const float hxn = Buf<T>::ld(ru, off(xn, y0 + hr), sh);
    const uint32_t vyn = off(x, yn), vc = act ? vq : kBufSkip, vcm = act ? elem(x, y) * 4u : kBufSkip;
    float hyn[TZ], hyf[TZ], hxf, second[TZ], mm[TZ];
    {
        const Rsrc rs = make_rsrc((IsInc<T>::v ? s.dinc : s.u[A.iu ^ 1]) + base * esz), rm = make_rsrc(s.m + base * 4);
        uint32_t so = fu, sm = fm;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Sb, sm += Smb) {
            hyn[p] = Buf<T>::ld(ru, vyn, so);
            second[p] = NT ? Buf<T>::ldnt(rs, vc, so) : Buf<T>::ld(rs, vc, so);
            mm[p] = NT ? Buf<float>::ldnt(rm, vcm, sm) : Buf<float>::ld(rm, vcm, sm);
        }
    }
    auto prof = [&](int d, int f, int c) -> float {
        return Buf<float>::ld(rl, (uint32_t)c * 4u, s.t_prof + (uint32_t)((d * 4 + f) * s.nmax) * 4u);
    };
    // x layers: own psi and zeta, and psi of the 4 columns on each side (psi_index layout)
    const uint32_t Spx = (uint32_t)(s.PY * s.WX) * 4u;
    uint32_t xpn = 0, xze = 0;   // new psi and zeta at plane z0
    bool bx = false, sx = false, hsx = false;
    uint32_t vx = kBufSkip;
    float pxo[TZ], zx[TZ], dx[TZ], pxh, ax[4], ahx[2];   // dx: D1 u^n at the column's points
    if (xb) {
        const uint32_t fo = (uint32_t)(z0 + fz) * Spx, xpo = s.t_psi[A.iu][0] + fo;
        xpn = s.t_psi[A.iu ^ 1][0] + fo;
        xze = s.t_zeta[0] + fo;
        const uint32_t side = (uint32_t)(nz + 2 * fz) * Spx - (uint32_t)(nx - xhi) * 4u;
        auto xoff = [&](int xp, int yp) -> uint32_t {
            const uint32_t e = (uint32_t)((yp + fy) * s.WX + xp) * 4u;
            return xp < xlo ? e : e + side;
        };
        hxf = Buf<T>::ld(ru, off(xf, y0 + hr), sh);
        bx = act && in_band(x, nx, xlo, xhi);
        sx = act && slab_point(x, nx, xlo, xhi);
        vx = sx ? xoff(x, y) : kBufSkip;
        hsx = y0 + hr < ny && slab_point(xn, nx, xlo, xhi);
        pxh = Buf<float>::ld(rl, hsx ? xoff(xn, y0 + hr) : kBufSkip, xpo + (uint32_t)hp * Spx);
        uint32_t so = xpo, sz = xze;
#pragma unroll
        for (int p = 0; p < TZ; ++p, so += Spx, sz += Spx) {
            pxo[p] = Buf<float>::ld(rl, vx, so);
            zx[p] = Buf<float>::ld(rl, vx, sz);
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) ax[f] = prof(0, f, min(x, nx - 1));
#pragma unroll
        for (int f = 0; f < 2; ++f) ahx[f] = prof(0, f, min(max(xn, 0), nx - 1));
    }
    // y layers
    const uint32_t Spy = (uint32_t)(s.SY * nx) * 4u;
    uint32_t ypn = 0, yze = 0;
    bool by = false, sy = false, hsy = false;
    uint32_t vy = kBufSkip;
    float pyo[TZ], pyh[TZ], zy[TZ], dy[TZ], ay[4], ahy[2];
    if (yb) {
        const uint32_t fo = (uint32_t)(z0 + fz) * Spy, ypo = s.t_psi[A.iu][1] + fo;
        ypn = s.t_psi[A.iu ^ 1][1] + fo;
        yze = s.t_zeta[1] + fo;
        auto yoff = [&](int yp) -> uint32_t { return (uint32_t)(slab_pos(yp, ny, ylo, yhi) * nx + x) * 4u; };
        const uint32_t vyf = off(x, yf);
        by = act && in_band(y, ny, ylo, yhi);
        sy = act && slab_point(y, ny, ylo, yhi);
        vy = sy ? yoff(y) : kBufSkip;
        hsy = x < nx && slab_point(yn, ny, ylo, yhi);
        const uint32_t vyh = hsy ? yoff(yn) : kBufSkip;
        uint32_t su = fu, so = ypo, sz = yze;
#pragma unroll
        for (int p = 0; p < TZ; ++p, su += Sb, so += Spy, sz += Spy) {
            hyf[p] = Buf<T>::ld(ru, vyf, su);
            pyo[p] = Buf<float>::ld(rl, vy, so);
            pyh[p] = Buf<float>::ld(rl, vyh, so);
            zy[p] = Buf<float>::ld(rl, vy, sz);
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) ay[f] = prof(1, f, min(y, ny - 1));
#pragma unroll
        for (int f = 0; f < 2; ++f) ahy[f] = prof(1, f, min(max(yn, 0), ny - 1));
    }
    // z layers: the column's psi at z0 - 4 .. z0 + TZ + 3 (bit o of zm: plane z0 - 4 + o lies in a layer; the
    // window meets one layer only, the tile rule sees to that too); the profiles of those planes, one per lane
    const uint32_t Spz = (uint32_t)(s.PY * nx) * 4u;
    const uint32_t vz = act ? (uint32_t)((y + fy) * nx + x) * 4u : kBufSkip;
    constexpr int PN = TZ + 2 * FDTD_R;
    float pz[PN], zz[TZ], dz[TZ], az[4];
    uint32_t zm = 0, zpn = 0, zze = 0;   // new psi and zeta at plane z0 - 4
    if (zb) {
        const uint32_t zlm = plane_bits<PN>(z0 - FDTD_R, 0, zlo);
        zm = zlm | plane_bits<PN>(z0 - FDTD_R, nz - zhi, nz);
        // slab position of plane z0 - 4 (as if it lay in the layer of the window)
        const uint32_t fo = (uint32_t)(z0 - FDTD_R + (zlm ? 0 : zlo - (nz - zhi))) * Spz;
        const uint32_t zpo = s.t_psi[A.iu][2] + fo;
        zpn = s.t_psi[A.iu ^ 1][2] + fo;
        zze = s.t_zeta[2] + fo;
        // (z0 - 8 .. z0 - 5 of a box at the low face: no tap, read as plane z0)
        uint32_t su = z0 >= FDTD_R ? fu - 2 * FDTD_R * Sb : fu, sh2 = fu + (TZ + FDTD_R) * Sb;
#pragma unroll
        for (int o = 0; o < FDTD_R; ++o, su += Sb, sh2 += Sb) {
            q[o] = Buf<T>::ld(ru, vq, su);
            q[TZ + 3 * FDTD_R + o] = Buf<T>::ld(ru, vq, min(sh2, slast));
        }
        uint32_t so = zpo;
#pragma unroll
        for (int o = 0; o < PN; ++o, so += Spz) {
            pz[o] = 0.0f;
            if ((zm >> o) & 1u) pz[o] = Buf<float>::ld(rl, vz, so);
        }
        uint32_t sz = zze + FDTD_R * Spz;
#pragma unroll
        for (int p = 0; p < TZ; ++p, sz += Spz) {
            zz[p] = 0.0f;
            if ((zm >> (p + FDTD_R)) & 1u) zz[p] = Buf<float>::ld(rl, vz, sz);
        }
        const int zl = min(max(z0 - FDTD_R + (t & 15), 0), nz - 1);
#pragma unroll
        for (int f = 0; f < 4; ++f) az[f] = prof(2, f, zl);
    }

    // ---- u^n of the box's planes and their halo to LDS ----
    const int rn = ly < FDTD_R ? ly : ly + TY;   // row of yn in PY
    float *const Uc = &U[0][ly + 8][lx + 8];     // the column's place in plane 0
    constexpr int UP = UH * UW;
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        Uc[p * UP] = q[p + 8];
        U[p][rn + 4][lx + 8] = hyn[p];
    }
    const int cn = c8 < FDTD_R ? c8 : c8 + TX;   // column of xn in PX
    U[hp][hr + 8][cn + 4] = hxn;
    if (on(xb)) U[hp][hr + 8][c8 < FDTD_R ? cn : cn + 8] = hxf;
    if (on(yb)) {
#pragma unroll
        for (int p = 0; p < TZ; ++p) U[p][ly < FDTD_R ? rn : rn + 8][lx + 8] = hyf[p];
    }
    __syncthreads();

    // ---- new psi of the box grown by 4 along each axis; the box's own is stored ----
    const int np = nz - z0;   // planes of the box inside the grid (TZ or fewer)
    float w1[3][5];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int l = 0; l < 5; ++l) w1[d][l] = s.w1[d][l];
    if (on(xb)) {
        const int n1 = again(np);
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            dx[p] = d1_lds(Uc + p * UP, 1, w1[0]);
            const float v = sx ? psi_update(ax[0], pxo[p], ax[1], dx[p]) : 0.0f;
            PX[p][ly][lx + 4] = v;
            if (p < n1) Buf<float>::stc(rl, vx, xpn + p * Spx, v);
        }
        const float v = psi_update(ahx[0], pxh, ahx[1], d1_lds(&U[hp][hr + 8][cn + 4], 1, w1[0]));
        PX[hp][hr][cn] = hsx ? v : 0.0f;
    }
    if (on(yb)) {
        const int n1 = again(np);
#pragma unroll
        for (int p = 0; p < TZ; ++p) {
            dy[p] = d1_lds(Uc + p * UP, UW, w1[1]);
            const float v = sy ? psi_update(ay[0], pyo[p], ay[1], dy[p]) : 0.0f;
            const float h = hsy ? psi_update(ahy[0], pyh[p], ahy[1], d1_lds(&U[p][rn + 4][lx + 8], UW, w1[1])) : 0.0f;
            PY[p][ly + 4][lx] = v;
            PY[p][rn][lx] = h;
            if (p < n1) Buf<float>::stc(rl, vy, ypn + p * Spy, v);
        }
    }
    if (on(zb)) {
        const uint32_t z1 = (uint32_t)again((int)zm);
#pragma unroll
        for (int o = 0; o < PN; ++o)
            if (((z1 >> o) & 1u) || (o >= FDTD_R && o < FDTD_R + TZ)) {
                float lo[4], hi[4];
#pragma unroll
                for (int l = 1; l <= 4; ++l) {
                    lo[l - 1] = q[o + 4 - l];
                    hi[l - 1] = q[o + 4 + l];
                }
                const float d1 = d1_axis(w1[2], lo, hi);
                if (o >= FDTD_R && o < FDTD_R + TZ) dz[o - FDTD_R] = d1;
                if (!((z1 >> o) & 1u)) continue;
                pz[o] = psi_update(lane_value(az[0], o), pz[o], lane_value(az[1], o), d1);
                if (o >= FDTD_R && o < FDTD_R + TZ) Buf<float>::stc(rl, vz, zpn + o * Spz, pz[o]);
            }
    }
    Coef K;
    K.cc = s.cc;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int l = 0; l < 5; ++l) K.w2[d][l] = s.w2[d][l];
    if (on(xb | yb)) __syncthreads();

    // ---- the update ----
    const Rsrc rw = make_rsrc(s.u[A.iu ^ 1] + base * esz), rs = IsInc<T>::v ? make_rsrc(s.dinc + base * esz) : rw;
    const Rsrc ri = INC ? make_rsrc(s.inc + A.inc * s.inc_slot + base * esz) : rw;
    const int src_tile = uniform(s.sx >= x0 && s.sx < x0 + TX && s.sy >= y0 && s.sy < y0 + TY && s.sz >= z0 &&
                                 s.sz < z0 + TZ);
    float srcamp = 0.0f;
    if (src_tile && s.wav != nullptr) {
        const int n = *stepc + A.k;
        if (n >= 0 && n < s.src_nt) srcamp = s.wav[n] * s.src_scale;
    }
#pragma unroll
    for (int p = 0; p < TZ; ++p) {
        if (p >= again(np)) break;
        const float *c0 = Uc + p * UP;
        float xl[4], xh[4], yl[4], yh[4], zl[4], zh[4];
#pragma unroll
        for (int l = 1; l <= 4; ++l) {
            xl[l - 1] = c0[-l];
            xh[l - 1] = c0[l];
            yl[l - 1] = c0[-l * UW];
            yh[l - 1] = c0[l * UW];
            zl[l - 1] = q[p + 8 - l];
            zh[l - 1] = q[p + 8 + l];
        }
        const float c = q[p + 8];
        float lt;
        if (!on(xb | yb | zb)) {
            lt = lap_interior(K, c, xl, xh, yl, yh, zl, zh);
        } else {
            const bool bz = zb && in_band(again(z0 + p), nz, zlo, zhi);
            float L[3] = {d2_axis(K.w2[0], c, xl, xh), d2_axis(K.w2[1], c, yl, yh), d2_axis(K.w2[2], c, zl, zh)};
            if (on(xb)) {
                float zn = 0.0f;
                const float e = cpml_axis(L[0], dx[p], d1_lds(&PX[p][ly][lx + 4], 1, w1[0]), ax[2],
                                          ax[3], ax[1], ax[0], sx, zx[p], &zn);
                if (bx) L[0] = e;
                Buf<float>::stc(rl, vx, xze + p * Spx, zn);
            }
            if (on(yb)) {
                float zn = 0.0f;
                const float e = cpml_axis(L[1], dy[p], d1_lds(&PY[p][ly + 4][lx], TX, w1[1]), ay[2],
                                          ay[3], ay[1], ay[0], sy, zy[p], &zn);
                if (by) L[1] = e;
                Buf<float>::stc(rl, vy, yze + p * Spy, zn);
            }
            if (bz) {
                float pl[4], ph[4], zn = 0.0f;
#pragma unroll
                for (int l = 1; l <= 4; ++l) {
                    pl[l - 1] = pz[p + 4 - l];
                    ph[l - 1] = pz[p + 4 + l];
                }
                const bool sz = ((uint32_t)again((int)zm) >> (p + 4)) & 1u;
                L[2] = cpml_axis(L[2], dz[p], d1_axis(w1[2], pl, ph), lane_value(az[2], p + 4),
                                 lane_value(az[3], p + 4), lane_value(az[1], p + 4), lane_value(az[0], p + 4), sz, zz[p],
                                 &zn);
                if (sz) Buf<float>::stc(rl, vz, zze + (p + 4) * Spz, zn);
            }
            lt = (L[0] + L[1]) + L[2];
            const bool none = act && !(bx || by || bz);
            if (__any(none)) {
                const float li = lap_interior(K, c, xl, xh, yl, yh, zl, zh);
                if (none) lt = li;
            }
        }
        const bool src = again(src_tile) && z0 + p == s.sz && x == s.sx && y == s.sy;
        const Upd up = time_update<T>(mm[p], lt, c, second[p], src, srcamp);
        if constexpr (NT) {
            Buf<T>::st(rw, vc, fu + p * Sb, up.u);
            if constexpr (IsInc<T>::v) Buf<T>::st(rs, vc, fu + p * Sb, up.d);
        } else {
            Buf<T>::stc(rw, vc, fu + p * Sb, up.u);
            if constexpr (IsInc<T>::v) Buf<T>::stc(rs, vc, fu + p * Sb, up.d);
        }
        if constexpr (INC) Buf<T>::st(ri, vc, fu + p * Sb, up.u - c);
    }
}

// FP32 boxes of TX x TY x IZ points outside every band and wholly inside the grid
// (TileItem flags: the shot only): u^{n+1} alone, from the box's column and an
// LDS box with a 4-point halo along x and y.  Bound by HBM: 512^3 with 20-cell
// layers, 96 M points in 333 us, 4.6 TB/s of the 16 bytes a point cannot do
// without, 5.3 TB/s counted (u^n is fetched 1.57 times: whole lines at the bricks'
// x faces); the z-march takes 586 us for them on the half of the CUs the band
// kernel leaves it, and 345 us on all.  The memory's latency is hidden by other
// blocks and not by a register queue along z: boxes of 16 planes, which 512^3
// takes, hold 84 VGPRs and 40 KB of LDS, four blocks per CU, those of 8 planes 52
// and 20 KB, eight.
template <int IZ, bool INC>
__device__ __forceinline__ void inner_box(const ConstDesc &s, const TileItem &wi, const TileStep &A,
                                          const int *__restrict__ stepc) {
    constexpr int F = FDTD_R, LW = TX + 2 * F, LH = TY + 2 * F, LP = LW * LH, XH = IZ / 4;
    __shared__ float U[IZ * LP];   // u^n at (x0 - 4 + c, y0 - 4 + r, z0 + p); corners unused
    const int t = (int)threadIdx.x, lx = t % TX, ly = t / TX;
    const int x0 = wi.x0, y0 = wi.y0, z0 = wi.z0, P = s.P;
    const long base = (long)(s.fz + z0 - F) * s.S;   // descriptors based 4 planes before the box
    const Rsrc ru = make_rsrc(s.u[A.iu] + base * 4), rw = make_rsrc(s.u[A.iu ^ 1] + base * 4);
    const Rsrc rm = make_rsrc(s.m + base * 4);
    const uint32_t Sb = (uint32_t)s.S * 4u;
    // offsets of plane z0, and of the column (row y0 + ly, the row of the y halo, the x halo's place) in a plane
    const uint32_t fu = (uint32_t)(F * s.S + (s.fy + y0) * P + kFieldLead + x0) * 4u;
    const uint32_t vc = (uint32_t)(ly * P + lx) * 4u;
    // (lane offsets are unsigned: halos are addressed from the box's first halo row or column)
    const uint32_t vy = (uint32_t)((ly < F ? ly : ly + TY) * P + lx) * 4u;
    const uint32_t fy = fu - (uint32_t)(F * P) * 4u;
    const int c8 = t & 7, hr = (t >> 3) & (TY - 1), hp = uniform(t >> 6);
    const uint32_t vx = (uint32_t)(hr * P + (c8 < F ? c8 : c8 + TX)) * 4u;
    const uint32_t fx = fu - (uint32_t)F * 4u + (uint32_t)hp * Sb;
    float q[IZ + 2 * F], hy[IZ], hx[XH], second[IZ], mm[IZ];
    {
        uint32_t so = fu - F * Sb;
#pragma unroll
        for (int o = 0; o < IZ + 2 * F; ++o, so += Sb) q[o] = Buf<float>::ld(ru, vc, so);
        so = fy;
#pragma unroll
        for (int p = 0; p < IZ; ++p, so += Sb) hy[p] = Buf<float>::ld(ru, vy, so);
        so = fx;
#pragma unroll
        for (int p = 0; p < XH; ++p, so += 4 * Sb) hx[p] = Buf<float>::ld(ru, vx, so);
        so = fu;
#pragma unroll
        for (int p = 0; p < IZ; ++p, so += Sb) {
            second[p] = Buf<float>::ldnt(rw, vc, so);
            mm[p] = Buf<float>::ldnt(rm, vc, so);
        }
    }
    float *const Uc = U + (ly + F) * LW + lx + F;
    float *const Uy = U + (ly < F ? ly : ly + TY) * LW + lx + F;
    float *const Ux = U + hp * LP + (hr + F) * LW + (c8 < F ? c8 : c8 + TX);
#pragma unroll
    for (int p = 0; p < IZ; ++p) {
        Uc[p * LP] = q[p + F];
        Uy[p * LP] = hy[p];
    }
#pragma unroll
    for (int p = 0; p < XH; ++p) Ux[4 * p * LP] = hx[p];
    __syncthreads();
    const int src_box = uniform(s.sx >= x0 && s.sx < x0 + TX && s.sy >= y0 && s.sy < y0 + TY && s.sz >= z0 &&
                                s.sz < z0 + IZ);
    float srcamp = 0.0f;
    if (src_box && s.wav != nullptr) {
        const int n = *stepc + A.k;
        if (n >= 0 && n < s.src_nt) srcamp = s.wav[n] * s.src_scale;
    }
    Coef K;
    K.cc = s.cc;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int l = 0; l < 5; ++l) K.w2[d][l] = s.w2[d][l];
    const Rsrc ri = INC ? make_rsrc(s.inc + A.inc * s.inc_slot + base * 4) : rw;
    uint32_t so = fu;
#pragma unroll
    for (int p = 0; p < IZ; ++p, so += Sb) {
        const float *c0 = Uc + p * LP;
        float xl[4], xh[4], yl[4], yh[4], zl[4], zh[4];
#pragma unroll
        for (int l = 1; l <= 4; ++l) {
            xl[l - 1] = c0[-l];
            xh[l - 1] = c0[l];
            yl[l - 1] = c0[-l * LW];
            yh[l - 1] = c0[l * LW];
            zl[l - 1] = q[p + F - l];
            zh[l - 1] = q[p + F + l];
        }
        const float lt = lap_interior(K, q[p + F], xl, xh, yl, yh, zl, zh);
        const bool src = again(src_box) && z0 + p == s.sz && x0 + lx == s.sx && y0 + ly == s.sy;
        const Upd up = time_update<float>(mm[p], lt, q[p + F], second[p], src, srcamp);
        Buf<float>::st(rw, vc, so, up.u);
        if constexpr (INC) Buf<float>::st(ri, vc, so, up.u - q[p + F]);
    }
}
// The same in 16-bit storage: boxes of 2 TX x TY x IZ points, two neighbours along x to
// a lane.  With one point to a lane the kernel was bound by the instructions of its
// 16-bit loads and stores, each half a line wide; a pair takes one access where two
// points took two, and a row of the box is one whole line, which the non-temporal
// stores need.  611 x 387 x 453 BF16, 16-cell layers: 68 M points in 280 us (boxes 32
// wide) -> 178 us for 69 M (12 bytes a point: 4.6 TB/s); 768^3 FP16 332 M points in
// 866 us (4.6 TB/s, 5.3 counted).  94 VGPRs (BF16: 103) and 37 KB of LDS (FP32, read
// eight bytes at a time): four blocks per CU.
template <typename T, int IZ>
__device__ __forceinline__ void inner_pair(const ConstDesc &s, const TileItem &wi, const TileStep &A,
                                           const int *__restrict__ stepc) {
    constexpr int F = FDTD_R, LW = 2 * TX + 2 * F, LH = TY + 2 * F, LP = LW * LH;
    static_assert(IZ * TY * F == 256, "one x-halo pair per thread");
    __shared__ float2 U[IZ * LP / 2];   // u^n at (x0 - 4 + c, y0 - 4 + r, z0 + p); corners unused
    const int t = (int)threadIdx.x, lx = t % TX, ly = t / TX;
    const int x0 = wi.x0, y0 = wi.y0, z0 = wi.z0, P = s.P, esz = (int)sizeof(T);
    const long base = (long)(s.fz + z0 - F) * s.S;   // descriptors based 4 planes before the box
    const Rsrc ru = make_rsrc(s.u[A.iu] + base * esz), rw = make_rsrc(s.u[A.iu ^ 1] + base * esz);
    const Rsrc rs = make_rsrc(s.dinc + base * esz), rm = make_rsrc(s.m + base * 4);
    const uint32_t Sb = (uint32_t)s.S * (uint32_t)esz, Smb = (uint32_t)s.S * 4u;
    const uint32_t f0 = (uint32_t)(F * s.S + (s.fy + y0) * P + kFieldLead + x0);
    const uint32_t fu = f0 * (uint32_t)esz, fm = f0 * 4u;
    const uint32_t vc = (uint32_t)(ly * P + 2 * lx) * (uint32_t)esz, vm = 2u * vc;
    const uint32_t vy = (uint32_t)((ly < F ? ly : ly + TY) * P + 2 * lx) * (uint32_t)esz;
    const uint32_t fy = fu - (uint32_t)(F * P) * (uint32_t)esz;
    // x halo: pair c4 of row hr of plane hp
    const int c4 = t & 3, hr = (t >> 2) & (TY - 1), hp = t / (4 * TY), hc = c4 < 2 ? 2 * c4 : 2 * c4 + 2 * TX;
    const uint32_t vx = (uint32_t)(hp * s.S + hr * P + hc) * (uint32_t)esz, fx = fu - (uint32_t)F * (uint32_t)esz;
    float2 q[IZ + 2 * F], hy[IZ], hx, second[IZ], mm[IZ];
    {
        uint32_t so = fu - F * Sb;
#pragma unroll
        for (int o = 0; o < IZ + 2 * F; ++o, so += Sb) q[o] = Buf2<T>::ld(ru, vc, so);
        so = fy;
#pragma unroll
        for (int p = 0; p < IZ; ++p, so += Sb) hy[p] = Buf2<T>::ld(ru, vy, so);
        hx = Buf2<T>::ld(ru, vx, fx);
        so = fu;
        uint32_t sm = fm;
#pragma unroll
        for (int p = 0; p < IZ; ++p, so += Sb, sm += Smb) {
            second[p] = Buf2<T>::ldnt(rs, vc, so);
            mm[p] = Buf2<float>::ldnt(rm, vm, sm);
        }
    }
    float2 *const Uc = U + ((ly + F) * LW + 2 * lx + F) / 2;
    float2 *const Uy = U + ((ly < F ? ly : ly + TY) * LW + 2 * lx + F) / 2;
#pragma unroll
    for (int p = 0; p < IZ; ++p) {
        Uc[p * LP / 2] = q[p + F];
        Uy[p * LP / 2] = hy[p];
    }
    U[(hp * LP + (hr + F) * LW + hc) / 2] = hx;
    __syncthreads();
    const int src_box = uniform(s.sx >= x0 && s.sx < x0 + 2 * TX && s.sy >= y0 && s.sy < y0 + TY && s.sz >= z0 &&
                                s.sz < z0 + IZ);
    float srcamp = 0.0f;
    if (src_box && s.wav != nullptr) {
        const int n = *stepc + A.k;
        if (n >= 0 && n < s.src_nt) srcamp = s.wav[n] * s.src_scale;
    }
    Coef K;
    K.cc = s.cc;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int l = 0; l < 5; ++l) K.w2[d][l] = s.w2[d][l];
    uint32_t so = fu;
#pragma unroll
    for (int p = 0; p < IZ; ++p, so += Sb) {
        const float2 *c0 = Uc + p * LP / 2;
        float xr[2 * F + 2];   // x - 4 .. x + 5
        float2 yl[4], yh[4];
#pragma unroll
        for (int l = 0; l < F + 1; ++l) {
            const float2 v = l == F / 2 ? q[p + F] : c0[l - F / 2];
            xr[2 * l] = v.x;
            xr[2 * l + 1] = v.y;
        }
#pragma unroll
        for (int l = 1; l <= 4; ++l) {
            yl[l - 1] = c0[-l * LW / 2];
            yh[l - 1] = c0[l * LW / 2];
        }
        float2 un, dn;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            auto at = [&](const float2 &v) { return k ? v.y : v.x; };
            float xl[4], xh[4], ya[4], yb[4], zl[4], zh[4];
#pragma unroll
            for (int l = 1; l <= 4; ++l) {
                xl[l - 1] = xr[F + k - l];
                xh[l - 1] = xr[F + k + l];
                ya[l - 1] = at(yl[l - 1]);
                yb[l - 1] = at(yh[l - 1]);
                zl[l - 1] = at(q[p + F - l]);
                zh[l - 1] = at(q[p + F + l]);
            }
            const float c = at(q[p + F]);
            const float lt = lap_interior(K, c, xl, xh, ya, yb, zl, zh);
            const bool src = again(src_box) && z0 + p == s.sz && x0 + 2 * lx + k == s.sx && y0 + ly == s.sy;
            const Upd up = time_update<T>(at(mm[p]), lt, c, at(second[p]), src, srcamp);
            (k ? un.y : un.x) = up.u;
            (k ? dn.y : dn.x) = up.d;
        }
        Buf2<T>::st(rw, vc, so, un);
        Buf2<T>::st(rs, vc, so, dn);
    }
}

template <typename T, int IZ, bool ONE, bool INC>
__global__ __launch_bounds__(256) void k_inner(const TileDesc *__restrict__ descs, const TileItem *__restrict__ work,
                                               TileStep A, const int *__restrict__ stepc) {
    const TileItem wi = work[blockIdx.x];
    if (wi.flags < 0) return;   // the idle items that pad the list
    const ConstDesc &s = shot_desc<ONE>(descs, wi);
    if constexpr (IsInc<T>::v) inner_pair<T, IZ>(s, wi, A, stepc);
    else inner_box<IZ, INC>(s, wi, A, stepc);
}

// Boxes that meet one band at most, in 16-bit storage: tile_box built for each case
// holds 79 VGPRs and 27 KB of LDS where the build for any box holds 116 and 31, so
// six blocks share a CU and not four.  In 16-bit storage k_tile is bound by latency
// and instruction issue, and that pays: 768^3 FP16 35.9 -> 34.9 ms for 20 steps, 611 x
// 387 x 453 BF16 20.4 -> 19.8 ms for 40.  In FP32 it does not (512^3 283 us for k_tile
// alone, 227 + 56 for both; 24 batched shots 864, 544 + 337): its boxes already move
// 4.4 to 4.8 TB/s, counted, at four blocks per CU.
template <typename T>
__device__ __forceinline__ void face_box(const ConstDesc &s, const TileItem &wi, const TileStep &A,
                                         const int *__restrict__ stepc, float *lds) {
    const int ax = uniform(wi.flags & AX_ANY);
    if (ax == 0) tile_box<T, 0, false, false>(s, wi, A, stepc, lds);
    else if (ax == TILE_XB) tile_box<T, TILE_XB, false, false>(s, wi, A, stepc, lds);
    else if (ax == TILE_YB) tile_box<T, TILE_YB, false, false>(s, wi, A, stepc, lds);
    else tile_box<T, TILE_ZB, false, false>(s, wi, A, stepc, lds);
}
template <typename T, bool ONE>
__global__ __launch_bounds__(256, 6) void k_face(const TileDesc *__restrict__ descs, const TileItem *__restrict__ work,
                                                 TileStep A, const int *__restrict__ stepc) {
    __shared__ float lds[TZ * UH * UW + TZ * PYH * TX];
    const TileItem wi = work[blockIdx.x];
    if (wi.flags < 0) return;   // the idle items that pad the list
    face_box<T>(shot_desc<ONE>(descs, wi), wi, A, stepc, lds);
}
template <typename T, bool ONE, bool NT, bool INC>
__global__ __launch_bounds__(256, 4) void k_tile(const DevShot *__restrict__ shots, const TileDesc *__restrict__ descs,
                                                 const TileItem *__restrict__ work, TileStep A,
                                                 const int *__restrict__ stepc) {
    __shared__ float lds[TZ * UH * UW + TZ * TY * PXW + TZ * PYH * TX];
    const int t = (int)threadIdx.x;
    if ((int)blockIdx.x >= A.nwork) {
        // receivers of the step before this one (the newest level is complete now)
        const int n = *stepc + A.k;
        const DevShot &s = shots[A.rec_lo + (int)blockIdx.x - A.nwork];
        if (s.traces == nullptr || n - 1 >= s.trace_cap) return;
        const T *u = (const T *)s.u[A.iu];
        for (int r = t; r < s.nrec; r += 256) {
            const int32_t *q = s.rec + 3 * r;
            const long c = (long)q[2] * s.S + (long)q[1] * s.P + q[0];
            s.traces[(long)(n - 1) * s.nrec + r] = Store<T>::ld(u + c) * s.inv_scale;
        }
        return;
    }
    const TileItem wi = work[blockIdx.x];
    if (wi.flags < 0) return;   // the idle items that pad the list
    tile_box<T, AX_ANY, NT, INC>(shot_desc<ONE>(descs, wi), wi, A, stepc, lds);
}

// launch f(ONE, NT, INC as std::bool_constant); only FP32 fields have the non-temporal build and increments
template <typename T, typename F>
static void with_flags(bool one, bool nt, bool inc, F f) {
    auto a = [&](auto ONE) {
        if constexpr (!IsInc<T>::v) {
            auto b = [&](auto NT) { inc ? f(ONE, NT, std::true_type{}) : f(ONE, NT, std::false_type{}); };
            nt ? b(std::true_type{}) : b(std::false_type{});
        } else {
            f(ONE, std::false_type{}, std::false_type{});
        }
    };
    one ? a(std::true_type{}) : a(std::false_type{});
}

template <typename T, int IZ>
static void launch_inner_t(const TileDesc *d_descs, const TileItem *work, const TileStep &A, const int *stepc,
                           bool one, hipStream_t st) {
    with_flags<T>(one, true, A.inc >= 0, [&](auto ONE, auto, auto INC) {
        hipLaunchKernelGGL((k_inner<T, IZ, ONE.value, INC.value>), dim3((unsigned)A.nwork), dim3(256), 0, st, d_descs,
                           work, A, stepc);
    });
}
template <typename T>
static void launch_tile_t(const DevShot *d_shots, const TileDesc *d_descs, const TileItem *work, const TileStep &A,
                          int nrec, const int *stepc, bool one, hipStream_t st) {
    with_flags<T>(one, A.nt, A.inc >= 0, [&](auto ONE, auto NT, auto INC) {
        hipLaunchKernelGGL((k_tile<T, ONE.value, NT.value, INC.value>), dim3((unsigned)(A.nwork + nrec)), dim3(256), 0,
                           st, d_shots, d_descs, work, A, stepc);
    });
}

template <typename T>
static void launch_face_t(const TileDesc *d_descs, const TileItem *work, const TileStep &A, const int *stepc,
                          bool one, hipStream_t st) {
    const dim3 grid((unsigned)A.nwork);
    if (one) hipLaunchKernelGGL((k_face<T, true>), grid, dim3(256), 0, st, d_descs, work, A, stepc);
    else hipLaunchKernelGGL((k_face<T, false>), grid, dim3(256), 0, st, d_descs, work, A, stepc);
}
void fdtd_launch_face(int stor, const TileDesc *d_descs, const TileItem *work, const TileStep &A, const int *stepc,
                      bool one, hipStream_t st) {
    if (A.nwork <= 0) return;
    if (stor == 1) launch_face_t<_Float16>(d_descs, work, A, stepc, one, st);
    else launch_face_t<__bf16>(d_descs, work, A, stepc, one, st);
}

void fdtd_launch_tile(int stor, const DevShot *d_shots, const TileDesc *d_descs, const TileItem *work,
                      const TileStep &A, int nrec, const int *stepc, bool one, hipStream_t st) {
    if (A.nwork + nrec <= 0) return;
    if (stor == 1) launch_tile_t<_Float16>(d_shots, d_descs, work, A, nrec, stepc, one, st);
    else if (stor == 2) launch_tile_t<__bf16>(d_shots, d_descs, work, A, nrec, stepc, one, st);
    else launch_tile_t<float>(d_shots, d_descs, work, A, nrec, stepc, one, st);
}

void fdtd_launch_inner(int stor, InnerBox ib, const TileDesc *d_descs, const TileItem *work, const TileStep &A,
                       const int *stepc, bool one, hipStream_t st) {
    if (A.nwork <= 0) return;
    if (stor == 1) launch_inner_t<_Float16, 8>(d_descs, work, A, stepc, one, st);
    else if (stor == 2) launch_inner_t<__bf16, 8>(d_descs, work, A, stepc, one, st);
    else if (ib.z == 16) launch_inner_t<float, 16>(d_descs, work, A, stepc, one, st);
    else launch_inner_t<float, 8>(d_descs, work, A, stepc, one, st);
}
