// Conjugate-gradient vector kernels of the MoDL module (MoDL section, Eq. 6-8): the solve of
// (A^H A + mu I) x = b by a fixed number of CG steps from zero, one system per batch sample.  The operator
// itself is the fused SENSE sweep (xs = mu, gs = 1, y = 0), which also takes over the inner product and the update of the search
// direction where it can (sense_cg); the kernels here are the vector updates between two applications.  Every scalar of the recurrence stays on the device:
// a workgroup writes its partial inner product, and each consumer sums the partials of its sample in a fixed
// order, so a solve is a plain sequence of launches with no host synchronisation and a reproducible result.
#include "internal.h"

namespace gleam {

constexpr int kCgThreads = 256;

namespace {

// Sum over the workgroup, in thread 0.
__device__ inline double block_sum(double v, double* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kCgThreads / 64; ++w) v += red[w];
    return v;
}

// Sums of two sets of a sample's partials (kCgBlocksMax at most), the same values in every thread: each wave adds up both sets
// by itself, strided per lane in a fixed order and then across the lanes, so that no barrier stands between the launch and the
// first update.  All loads of a lane are in flight together: one after the other, 512 partials cost the updates 1.3 us each
// (1 x 256 x 24 x 160: 13.1 and 9.5 us).
__device__ inline double2 sum_partials(const double* __restrict__ u, int nu, const double* __restrict__ v, int nv) {
    constexpr int N = kCgBlocksMax / 64;
    const int lane = threadIdx.x & 63;
    double x[N], y[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int i = lane + 64 * k;
        x[k] = y[k] = 0.0;
        if (i < nu) x[k] = u[i];
        if (i < nv) y[k] = v[i];
    }
    double a = x[0], b = y[0];
#pragma unroll
    for (int k = 1; k < N; ++k) {
        a += x[k];
        b += y[k];
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
    }
    return make_double2(a, b);
}

}  // namespace

// grid (nb, B).  r = c1*u + c2*v (v may be null), p = r, x = 0, rr[b][blk] = partial <r, r>.
// x may alias u (each element is read before it is overwritten by the same lane).
__global__ __launch_bounds__(kCgThreads) void cg_init_kernel(const float2* u, const float2* __restrict__ v, float c1, float c2,
                                                             long long n, float2* x, float2* __restrict__ r,
                                                             float2* __restrict__ p, double* __restrict__ rr) {
    __shared__ double red[kCgThreads / 64];
    const long long base = (long long)blockIdx.y * n;
    double s = 0.0;
    for (long long i = (long long)blockIdx.x * kCgThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kCgThreads) {
        float2 t = u[base + i];
        t.x *= c1; t.y *= c1;
        if (v) {
            const float2 w = v[base + i];
            t.x += c2 * w.x; t.y += c2 * w.y;
        }
        x[base + i] = make_float2(0.f, 0.f);
        r[base + i] = t;
        p[base + i] = t;
        s += (double)t.x * t.x + (double)t.y * t.y;
    }
    s = block_sum(s, red);
    if (threadIdx.x == 0) rr[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// pq[b][blk] = partial Re <p, q>
__global__ __launch_bounds__(kCgThreads) void cg_dot_kernel(const float2* __restrict__ p, const float2* __restrict__ q, long long n,
                                                            double* __restrict__ pq) {
    __shared__ double red[kCgThreads / 64];
    const long long base = (long long)blockIdx.y * n;
    double s = 0.0;
    for (long long i = (long long)blockIdx.x * kCgThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kCgThreads) {
        const float2 a = p[base + i], b = q[base + i];
        s += (double)a.x * b.x + (double)a.y * b.y;
    }
    s = block_sum(s, red);
    if (threadIdx.x == 0) pq[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// a = <r,r> / <p,q> (0 when the denominator is not positive); x += a p; r -= a q; rr_new partials.
__global__ __launch_bounds__(kCgThreads) void cg_update_xr_kernel(float2* __restrict__ x, float2* __restrict__ r,
                                                                  const float2* __restrict__ p, const float2* __restrict__ q,
                                                                  long long n, const double* __restrict__ rr_old,
                                                                  const double* __restrict__ pq, int n_pq,
                                                                  double* __restrict__ rr_new) {
    __shared__ double red[kCgThreads / 64];
    const int nb = gridDim.x;
    const long long base = (long long)blockIdx.y * n, step = (long long)gridDim.x * kCgThreads;
    constexpr int U = 4;   // elements in flight per lane; the first ones are fetched while the scalars are summed
    float2 pv[U], qv[U], xv[U], rv[U];
    long long i = (long long)blockIdx.x * kCgThreads + threadIdx.x;
    const auto fetch = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * step < n) {
                const long long at = base + i + u * step;
                pv[u] = p[at]; qv[u] = q[at]; xv[u] = x[at]; rv[u] = r[at];
            }
    };
    fetch();
    const double2 nd = sum_partials(rr_old + (size_t)blockIdx.y * nb, nb, pq + (size_t)blockIdx.y * n_pq, n_pq);
    const float a = nd.y > 0.0 ? (float)(nd.x / nd.y) : 0.f;
    double s = 0.0;
    while (i < n) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * step < n) {
                const long long at = base + i + u * step;
                xv[u].x += a * pv[u].x; xv[u].y += a * pv[u].y;
                rv[u].x -= a * qv[u].x; rv[u].y -= a * qv[u].y;
                x[at] = xv[u];
                r[at] = rv[u];
                s += (double)rv[u].x * rv[u].x + (double)rv[u].y * rv[u].y;
            }
        i += U * step;
        fetch();
    }
    s = block_sum(s, red);
    if (threadIdx.x == 0) rr_new[(size_t)blockIdx.y * nb + blockIdx.x] = s;
}

// beta = <r,r>_new / <r,r>_old (0 when the old one is not positive); p = r + beta p.
__global__ __launch_bounds__(kCgThreads) void cg_update_p_kernel(const float2* __restrict__ r, float2* __restrict__ p, long long n,
                                                                 const double* __restrict__ rr_old,
                                                                 const double* __restrict__ rr_new) {
    const int nb = gridDim.x;
    const double2 s = sum_partials(rr_old + (size_t)blockIdx.y * nb, nb, rr_new + (size_t)blockIdx.y * nb, nb);
    const float beta = s.x > 0.0 ? (float)(s.y / s.x) : 0.f;
    const long long base = (long long)blockIdx.y * n;
    for (long long i = (long long)blockIdx.x * kCgThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kCgThreads) {
        const float2 rv = r[base + i];
        float2 pv = p[base + i];
        pv.x = rv.x + beta * pv.x;
        pv.y = rv.y + beta * pv.y;
        p[base + i] = pv;
    }
}

__global__ __launch_bounds__(kCgThreads) void fill_zero_kernel(float2* __restrict__ x, long long n) {
    for (long long i = (long long)blockIdx.x * kCgThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kCgThreads)
        x[i] = make_float2(0.f, 0.f);
}

static inline size_t align256(size_t v) { return (v + 255) / 256 * 256; }

static int cg_blocks(long long n) {
    long long nb = (n + 4 * kCgThreads - 1) / (4 * kCgThreads);   // at least four elements per lane
    return (int)(nb < 1 ? 1 : (nb > kCgBlocksMax ? kCgBlocksMax : nb));
}

size_t cg_scratch_bytes(const gleam_geom& g) {
    const size_t img = align256((size_t)g.B * g.T * g.D * g.H * g.W * sizeof(float2));
    return 3 * img + align256((size_t)3 * g.B * kCgBlocksMax * sizeof(double));
}

hipError_t fill_zero(float2* x, long long n, hipStream_t st) {
    long long nb = (n + kCgThreads - 1) / kCgThreads;
    if (nb > 2048) nb = 2048;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)nb), dim3(kCgThreads), 0, st, x, n);
    return hipGetLastError();
}

hipError_t cg_solve(const gleam_geom& g, const float2* S, const unsigned char* M, float mu, int n_cg, const float2* u,
                    const float2* v, float c1, float c2, float2* x, float2* kbuf, void* scratch, hipStream_t st) {
    const long long n = g.T * g.D * g.H * g.W;
    const size_t img = align256((size_t)g.B * n * sizeof(float2));
    unsigned char* base = (unsigned char*)scratch;
    float2* r = (float2*)base;
    float2* p = (float2*)(base + img);
    float2* q = (float2*)(base + 2 * img);
    double* sc = (double*)(base + 3 * img);
    const int nb = cg_blocks(n);
    const size_t per = (size_t)g.B * nb;
    double* rr[2] = {sc, sc + per};
    double* pq = sc + 2 * per;
    const dim3 grid((unsigned)nb, (unsigned)g.B), block(kCgThreads);
    const double vec_bytes = 8.0 * (double)g.B * (double)n;
    {
        KernelScope ks("cg_init", 0.0, (v ? 5.0 : 4.0) * vec_bytes, st);
        hipLaunchKernelGGL(cg_init_kernel, grid, block, 0, st, u, v, c1, c2, n, x, r, p, rr[0]);
    }
    // Where the tiles of the operator's row sweeps allow it, the inner product rides on the last sweep and the update of the
    // search direction on the first sweep of the next application: four launches per step instead of six, and p and q are not read
    // again.  The products are summed in double as before, in another order.
    // Every tile of the first sweep sums the partials of its samples for itself, and every workgroup of the update those of the
    // inner product, so many of them cost more than the launches they save.  A module of 10 steps, all apart / by the rule below /
    // with up to 512 partials of the inner product (samples x coils x size: sums, partials; us):
    //     2 x 8 x 320 x 256         80,  160    982 /  934 /  926     1 x 5 x 4 x 128 x 256    128,  171    851 /  775 /  775
    //     4 x 12 x 320 x 368       115,  320   2196 / 2299 / 2286     1 x 15 x 320 x 368       115,  320   1100 / 1126 / 1087
    //     1 x 8 x 640 x 320        200,  320   1145 / 1145 / 1105     2 x 15 x 640 x 368       230,  640   2385 / 2393 / 2393
    //     1 x 5 x 256 x 24 x 160   512, 2048   2162 / 2160 / 2155     1 x 8 x 20 x 192 x 160   512, 1920   1791 / 1788 / 1786
    // The update inside the sweep, over 115 calls of 96 x 96 to 640 x 192, 2 to 16 coils, 1 to 4 samples: 3.2 % of the module gained in
    // the geometric mean, up to 9 % where launches count, and up to 4 % lost by 12 coils, of which a tile of 16 lines holds one
    // row with a quarter of its lines empty.
    constexpr int kFusedPartials = 256;
    static_assert(kFusedPartials <= kCgBlocksMax, "what sum_partials takes");
    const int room = 3 * kCgBlocksMax - 2 * nb, n_dot = cg_fused_dot_partials(g, room < kFusedPartials ? room : kFusedPartials);
    const int n_pq = n_dot ? n_dot : nb;
    const bool fuse_p = nb <= kCgFusedSums && cg_fused_update(g);
    for (int k = 0; k < n_cg; ++k) {
        double* cur = rr[k & 1];
        double* nxt = rr[(k + 1) & 1];
        CgFusion f{};
        f.dot = n_dot ? pq : nullptr;
        f.dot_per = n_dot;
        if (fuse_p && k > 0) {   // p = r + beta p with the sums of the step before: nxt holds the older one
            f.x_rw = p; f.r = r; f.rr_old = nxt; f.rr_new = cur; f.nb = nb;
        }
        const hipError_t e = sense_cg(g, p, S, M, mu, 1.f, q, kbuf, f, st);   // q = (A^H A + mu I) p
        if (e != hipSuccess) return e;
        if (!n_dot) {
            KernelScope ks("cg_dot", 0.0, 2.0 * vec_bytes, st);
            hipLaunchKernelGGL(cg_dot_kernel, grid, block, 0, st, (const float2*)p, (const float2*)q, n, pq);
        }
        {
            KernelScope ks("cg_update_xr", 0.0, 6.0 * vec_bytes, st);
            hipLaunchKernelGGL(cg_update_xr_kernel, grid, block, 0, st, x, r, (const float2*)p, (const float2*)q, n,
                               (const double*)cur, (const double*)pq, n_pq, nxt);
        }
        if (!fuse_p && k + 1 < n_cg) {   // the search direction of a step that is never taken is not needed
            KernelScope ks("cg_update_p", 0.0, 3.0 * vec_bytes, st);
            hipLaunchKernelGGL(cg_update_p_kernel, grid, block, 0, st, (const float2*)r, p, n, (const double*)cur,
                               (const double*)nxt);
        }
    }
    return hipGetLastError();
}

}  // namespace gleam
