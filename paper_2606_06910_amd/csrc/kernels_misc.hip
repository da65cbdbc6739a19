// kernels_misc.hip -- setup, conversion and ghost-exchange kernels (gfx950).
//
//  k_fill_zero       zero a byte range with 16-byte stores (used instead of a
//                    runtime memset so that captured work never contains one)
//  k_vel_to_m        m = v^2 dt^2 into the padded field layout, and max(v)
//  k_field           dense float32 <-> padded storage (scale applied)
//  k_copy_jobs       strided box copies: ghost-face pack into contiguous
//                    buffers and unpack into the opposite ghost rows (the
//                    loopback stands in for the neighbour of one GPU's
//                    pencil-yz share, paper section "Multi-GPU Decomposition
//                    and Halo Exchange")
//  k_pack            the arrays of a state copied one after another (checkpoints)
//  k_finite          flag any NaN/Inf in a field
#include "fdtd_dev.hpp"

#include <algorithm>

__global__ __launch_bounds__(256) void k_fill_zero(uint4 *p, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// grid: (blocks, jobs)
__global__ __launch_bounds__(256) void k_fill_jobs(const FillJob *__restrict__ jobs) {
    const FillJob j = jobs[blockIdx.y];
    uint4 *p = (uint4 *)j.p;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < j.n16; i += stride)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// m = v^2 dt^2, the largest v and whether any v is not finite and > 0, in one
// pass over v.  Blocks stride over the rows and keep their maximum in a
// register, so that each ends in one atomic: with one per row piece on the same
// word the atomics were all of the time.  fdtd_set_velocity as a whole: 512^3
// 6.2 -> 0.31 ms, 768^3 20.9 -> 0.89 ms, 160^3 0.37 -> 0.11 ms.
__global__ __launch_bounds__(256) void k_vel_to_m(const float *__restrict__ v, float *__restrict__ m, int nx, int ny,
                                                 int rows, int P, int S, double dt2,
                                                 unsigned int *__restrict__ vmax_bits, unsigned int *__restrict__ bad) {
    float top = 0.0f;
    bool wrong = false;
    for (int r = (int)blockIdx.x; r < rows; r += (int)gridDim.x) {
        const int z = r / ny, y = r - z * ny;
        const float *vr = v + (long)r * nx;
        float *mr = m + (long)z * S + (long)y * P;
        for (int x = (int)threadIdx.x; x < nx; x += 256) {
            const float vv = vr[x];
            mr[x] = (float)((double)vv * (double)vv * dt2);
            wrong = wrong || !(vv > 0.0f) || !isfinite(vv);
            top = fmaxf(top, vv);
        }
    }
    // block maximum of the bit patterns (v > 0, so float order == unsigned order)
    __shared__ unsigned int red[4], any[4];
    unsigned int b = __float_as_uint(fmaxf(top, 0.0f));
    for (int o = 32; o > 0; o >>= 1) b = max(b, (unsigned int)__shfl_xor((int)b, o));
    const bool w = __any(wrong);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = b;
        any[threadIdx.x >> 6] = w;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicMax(vmax_bits, max(max(red[0], red[1]), max(red[2], red[3])));
        if (any[0] | any[1] | any[2] | any[3]) atomicOr(bad, 1u);
    }
}

// Dense float32 <-> padded storage, four modes: get u (times `f`), set u, and
// for 16-bit state (u^n, d^n) get and set u^{n-1} = u^n - d^n.  A thread takes 4
// consecutive points of a row (the padded rows start on 256 bytes, and a 16-byte
// access of the dense array needs 4-byte alignment only), the last piece of a row
// point by point; the threads of a block run on through the rows of a plane,
// so that narrow rows leave no lanes idle.  Bound by HBM.  Before (a thread per
// point, a block per 256 points of a row) and after, get / set of u^n: 512^3 FP32
// 310 / 340 -> 188 / 194 us (5.7 TB/s), 768^3 FP16 1065 / 1005 -> 456 / 459 us, 611
// x 387 x 453 BF16 302 / 265 -> 116 / 161 us.
// grid: (pieces of a plane / 256, nz)
enum { FIELD_GET, FIELD_SET, FIELD_GET_PREV, FIELD_SET_PREV };
typedef float dense4 __attribute__((ext_vector_type(4), aligned(4)));
template <typename T, int MODE>
__global__ __launch_bounds__(256) void k_field(T *__restrict__ u, T *__restrict__ d, float *__restrict__ dense, int nx,
                                              int ny, int npr, int P, int S, float f) {
    const int t = (int)(blockIdx.x * 256u + threadIdx.x);
    if (t >= npr * ny) return;
    const int y = t / npr, x = (t - y * npr) * 4;
    const long i = (long)blockIdx.y * S + (long)y * P + x;
    float *dn = dense + ((long)blockIdx.y * ny + y) * nx + x;
    const int k = nx - x;   // points of the piece (4 or fewer)
    dense4 a = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (MODE == FIELD_SET || MODE == FIELD_SET_PREV) {
        if (k >= 4) a = *(const dense4 *)dn;
        else
            for (int j = 0; j < k; ++j) a[j] = dn[j];
    }
    // (a padded row holds at least 4 elements past its last point, so 4 can always be read)
    float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f), e = q;
    if constexpr (MODE != FIELD_SET) q = Store<T>::ld4(u + i);
    if constexpr (MODE == FIELD_GET_PREV) e = Store<T>::ld4(d + i);
    if constexpr (MODE == FIELD_GET) {
        a = dense4{q.x * f, q.y * f, q.z * f, q.w * f};
    } else if constexpr (MODE == FIELD_GET_PREV) {
        a = dense4{(q.x - e.x) * f, (q.y - e.y) * f, (q.z - e.z) * f, (q.w - e.w) * f};
    } else if constexpr (MODE == FIELD_SET) {
        a = dense4{a.x * f, a.y * f, a.z * f, a.w * f};
    } else {
        a = dense4{q.x - a.x * f, q.y - a.y * f, q.z - a.z * f, q.w - a.w * f};
    }
    if constexpr (MODE == FIELD_GET || MODE == FIELD_GET_PREV) {
        if (k >= 4) *(dense4 *)dn = a;
        else
            for (int j = 0; j < k; ++j) dn[j] = a[j];
    } else {
        T *w = (MODE == FIELD_SET ? u : d) + i;
        if (k >= 4) Store<T>::st4(w, make_float4(a.x, a.y, a.z, a.w));
        else
            for (int j = 0; j < k; ++j) Store<T>::st(w + j, a[j]);
    }
}

// One row of a job per group of lanes: `lanes` consecutive threads copy a row
// in vb-byte pieces (16-byte pieces for FP32 rows that allow them), a block
// takes 256 / lanes rows per pass and strides over the job's rows; the only
// index arithmetic is one 32-bit division per row.  grid: (row blocks, njobs)
template <typename V>
__device__ __forceinline__ void copy_row(const char *s, char *d, int nv, int tv, int lanes) {
    for (int v = tv; v < nv; v += lanes) ((V *)d)[v] = ((const V *)s)[v];
}
__global__ __launch_bounds__(256) void k_copy_jobs(const CopyJob *__restrict__ jobs) {
    const CopyJob j = jobs[blockIdx.y];
    const int nrows = j.ey * j.ez;
    const int nv = j.ex * j.esz / j.vb;            // pieces per row
    const int lanes = nv < 256 ? nv : 256;         // threads per row
    const int rp = 256 / lanes;                    // rows per block pass
    const int tr = (int)threadIdx.x / lanes, tv = (int)threadIdx.x - tr * lanes;
    if (tr >= rp) return;
    for (int r = (int)blockIdx.x * rp + tr; r < nrows; r += (int)gridDim.x * rp) {
        const int z = r / j.ey, y = r - z * j.ey;
        const char *s = (const char *)j.src + ((long)z * j.sz + (long)y * j.sy) * j.esz;
        char *d = (char *)j.dst + ((long)z * j.dz + (long)y * j.dy) * j.esz;
        switch (j.vb) {
        case 16: copy_row<uint4>(s, d, nv, tv, lanes); break;
        case 8: copy_row<uint2>(s, d, nv, tv, lanes); break;
        case 4: copy_row<uint32_t>(s, d, nv, tv, lanes); break;
        default: copy_row<uint16_t>(s, d, nv, tv, lanes); break;
        }
    }
}

// grid: (blocks, 8 ranges); range r starts on the next multiple of 256 bytes after range r - 1
__global__ __launch_bounds__(256) void k_pack(const PackJob j) {
    size_t off = 0;
    for (int r = 0; r < (int)blockIdx.y; ++r) off += (j.n16[r] + 15) & ~(size_t)15;
    const uint4 *s = (const uint4 *)j.src[blockIdx.y];
    uint4 *d = (uint4 *)j.dst + off;
    const size_t n = j.n16[blockIdx.y], stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) d[i] = s[i];
}

template <typename T>
__global__ __launch_bounds__(256) void k_finite(const T *__restrict__ u, int nx, int ny, int P, int S,
                                               unsigned int *__restrict__ bad) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= nx) return;
    float f = Store<T>::ld(u + (long)blockIdx.z * S + (long)blockIdx.y * P + x);
    if (!isfinite(f)) atomicOr(bad, 1u);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void fdtd_launch_fill_zero(void *p, size_t bytes, hipStream_t st) {
    size_t n16 = bytes / 16;
    if (n16 == 0) return;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, st, (uint4 *)p, n16);
}
void fdtd_launch_fill_jobs(const void *jobs, int njobs, size_t max_n16, hipStream_t st) {
    if (njobs <= 0 || max_n16 == 0) return;
    const size_t blocks = std::min<size_t>((max_n16 + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_jobs, dim3((unsigned)blocks, njobs), dim3(256), 0, st, (const FillJob *)jobs);
}
void fdtd_launch_vel_to_m(const float *v, float *m, int nx, int ny, int nz, int P, int S, double dt2,
                          unsigned int *vmax_bits, unsigned int *bad, hipStream_t st) {
    const int rows = ny * nz;
    hipLaunchKernelGGL(k_vel_to_m, dim3((unsigned)std::min(rows, 4096)), dim3(256), 0, st, v, m, nx, ny, rows, P, S, dt2,
                       vmax_bits, bad);
}
template <typename T, int MODE>
static void field_t(void *u, void *d, float *dense, int nx, int ny, int nz, int P, int S, float f, hipStream_t st) {
    const int npr = (nx + 3) / 4;
    const dim3 grid((unsigned)(((long)npr * ny + 255) / 256), (unsigned)nz);
    hipLaunchKernelGGL((k_field<T, MODE>), grid, dim3(256), 0, st, (T *)u, (T *)d, dense, nx, ny, npr, P, S, f);
}
template <typename T> static void gf(const void *u, float *dst, int nx, int ny, int nz, int P, int S, float inv, hipStream_t st) {
    field_t<T, FIELD_GET>((void *)u, nullptr, dst, nx, ny, nz, P, S, inv, st);
}
template <typename T> static void sf(void *u, const float *src, int nx, int ny, int nz, int P, int S, float sc, hipStream_t st) {
    field_t<T, FIELD_SET>(u, nullptr, (float *)src, nx, ny, nz, P, S, sc, st);
}
template <typename T>
static void fin(const void *u, int nx, int ny, int nz, int P, int S, unsigned int *bad, hipStream_t st) {
    hipLaunchKernelGGL(k_finite<T>, dim3((nx + 255) / 256, ny, nz), dim3(256), 0, st, (const T *)u, nx, ny, P, S, bad);
}
#define MISC_DISPATCH(stor, F, ...)                                                                      \
    do {                                                                                                  \
        if ((stor) == 1) F<_Float16>(__VA_ARGS__);                                                        \
        else if ((stor) == 2) F<__bf16>(__VA_ARGS__);                                                     \
        else F<float>(__VA_ARGS__);                                                                       \
    } while (0)

void fdtd_launch_get_field(int stor, const void *u, float *dst, int nx, int ny, int nz, int P, int S, float inv,
                           hipStream_t st) {
    MISC_DISPATCH(stor, gf, u, dst, nx, ny, nz, P, S, inv, st);
}
void fdtd_launch_set_field(int stor, void *u, const float *src, int nx, int ny, int nz, int P, int S, float sc,
                           hipStream_t st) {
    MISC_DISPATCH(stor, sf, u, src, nx, ny, nz, P, S, sc, st);
}
void fdtd_launch_finite(int stor, const void *u, int nx, int ny, int nz, int P, int S, unsigned int *bad,
                        hipStream_t st) {
    MISC_DISPATCH(stor, fin, u, nx, ny, nz, P, S, bad, st);
}
template <typename T>
static void gp(const void *u, const void *d, float *dst, int nx, int ny, int nz, int P, int S, float inv, hipStream_t st) {
    field_t<T, FIELD_GET_PREV>((void *)u, (void *)d, dst, nx, ny, nz, P, S, inv, st);
}
template <typename T>
static void sp(const void *u, void *d, const float *src, int nx, int ny, int nz, int P, int S, float sc, hipStream_t st) {
    field_t<T, FIELD_SET_PREV>((void *)u, d, (float *)src, nx, ny, nz, P, S, sc, st);
}
void fdtd_launch_get_prev(int stor, const void *u, const void *d, float *dst, int nx, int ny, int nz, int P, int S,
                          float inv, hipStream_t st) {
    MISC_DISPATCH(stor, gp, u, d, dst, nx, ny, nz, P, S, inv, st);
}
void fdtd_launch_set_prev(int stor, const void *u, void *d, const float *src, int nx, int ny, int nz, int P, int S,
                          float sc, hipStream_t st) {
    MISC_DISPATCH(stor, sp, u, d, src, nx, ny, nz, P, S, sc, st);
}
void fdtd_launch_pack(const PackJob &j, hipStream_t st) {
    size_t n = 0;
    for (const auto v : j.n16) n = v > n ? v : n;
    const size_t gx = (n + 1023) / 1024;   // four pieces per thread of the longest range
    if (n > 0) hipLaunchKernelGGL(k_pack, dim3((unsigned)(gx < 2048 ? gx : 2048), 8), dim3(256), 0, st, j);
}
void fdtd_launch_copy_jobs(const void *jobs, int njobs, long max_rows, hipStream_t st) {
    if (njobs <= 0 || max_rows <= 0) return;
    const unsigned gx = (unsigned)(max_rows < 1024 ? max_rows : 1024);
    hipLaunchKernelGGL(k_copy_jobs, dim3(gx, njobs), dim3(256), 0, st, (const CopyJob *)jobs);
}


// Streaming ceiling of the interior update's access mix: o = a + b * c over
// float4 lanes (three streams read, one written, 16 bytes per lane), a
// grid-stride loop with `unroll` independent float4 per thread in flight.
template <int U>
__global__ __launch_bounds__(256) void k_stream_probe(const float4 *__restrict__ a, const float4 *__restrict__ b,
                                                     const float4 *__restrict__ c, float4 *__restrict__ o, size_t n4) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + (U - 1) * stride < n4; i += U * stride) {
        float4 x[U], y[U], z[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            x[k] = a[i + k * stride];
            y[k] = b[i + k * stride];
            z[k] = c[i + k * stride];
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            o[i + k * stride] = make_float4(fmaf(y[k].x, z[k].x, x[k].x), fmaf(y[k].y, z[k].y, x[k].y),
                                            fmaf(y[k].z, z[k].z, x[k].z), fmaf(y[k].w, z[k].w, x[k].w));
    }
    for (; i < n4; i += stride) {
        const float4 x = a[i], y = b[i], z = c[i];
        o[i] = make_float4(fmaf(y.x, z.x, x.x), fmaf(y.y, z.y, x.y), fmaf(y.z, z.z, x.z), fmaf(y.w, z.w, x.w));
    }
}
// The same mix in one-shot blocks: block i streams the 256 U consecutive
// float4 pieces from 256 U i on (thread t the pieces t, t + 256, ...) and
// exits; the stores carry the non-temporal hint, as the field stores do.
typedef float fdtd_v4f __attribute__((ext_vector_type(4)));
template <int U>
__global__ __launch_bounds__(256) void k_stream_chunk(const float4 *__restrict__ a, const float4 *__restrict__ b,
                                                     const float4 *__restrict__ c, float4 *__restrict__ o, size_t n4) {
    const size_t base = (size_t)blockIdx.x * 256 * U + threadIdx.x;
    float4 x[U], y[U], z[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const size_t i = base + (size_t)k * 256;
        if (i < n4) {
            x[k] = a[i];
            y[k] = b[i];
            z[k] = c[i];
        }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const size_t i = base + (size_t)k * 256;
        if (i < n4) {
            const fdtd_v4f r = {fmaf(y[k].x, z[k].x, x[k].x), fmaf(y[k].y, z[k].y, x[k].y),
                                fmaf(y[k].z, z[k].z, x[k].z), fmaf(y[k].w, z[k].w, x[k].w)};
            __builtin_nontemporal_store(r, (fdtd_v4f *)&o[i]);
        }
    }
}
void fdtd_launch_stream_probe(const float *a, const float *b, const float *c, float *o, size_t n4, int blocks,
                              int unroll, hipStream_t st) {
    const dim3 g((unsigned)blocks), t(256);
    const float4 *A = (const float4 *)a, *B = (const float4 *)b, *C = (const float4 *)c;
    if (blocks == 0) {
        const int u = unroll >= 4 ? 4 : (unroll == 2 ? 2 : 1);
        const dim3 gc((unsigned)((n4 + 256 * (size_t)u - 1) / (256 * (size_t)u)));
        if (u == 4) hipLaunchKernelGGL(k_stream_chunk<4>, gc, t, 0, st, A, B, C, (float4 *)o, n4);
        else if (u == 2) hipLaunchKernelGGL(k_stream_chunk<2>, gc, t, 0, st, A, B, C, (float4 *)o, n4);
        else hipLaunchKernelGGL(k_stream_chunk<1>, gc, t, 0, st, A, B, C, (float4 *)o, n4);
        return;
    }
    if (unroll >= 4) hipLaunchKernelGGL(k_stream_probe<4>, g, t, 0, st, A, B, C, (float4 *)o, n4);
    else if (unroll == 2) hipLaunchKernelGGL(k_stream_probe<2>, g, t, 0, st, A, B, C, (float4 *)o, n4);
    else hipLaunchKernelGGL(k_stream_probe<1>, g, t, 0, st, A, B, C, (float4 *)o, n4);
}

__global__ void k_set_int(int *p, int v) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}
void fdtd_launch_set_int(int *p, int v, hipStream_t st) {
    hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, p, v);
}
