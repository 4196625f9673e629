// SENSE normal operator / data-consistency step on gfx950:
//     out = xs * x + gs * S^H F^H Omega (F S x - y)          (Eq. 1-3; A = Omega F S)
// as 2d-1 sweeps over the coil k-space buffer for a d-dimensional transform:
//   rows_expand  : coil multiply fused into the load of the transform along W (contiguous axis)
//   cols_*       : strided axes, a tile of neighbouring columns per workgroup; the middle sweep does
//                  forward transform, mask / residual (in registers) and inverse transform of its axis
//                  in one go
//   rows_reduce  : inverse transform along W with conj(S) multiply, coil sum and the DC update fused
//                  into the store (the per-coil images are never written).
// sense_staged.hip has the same sweeps with whole transforms in LDS, for the calls that take those.
#include <hip/hip_runtime.h>
#include <type_traits>

#include "fft_core.h"
#include "internal.h"

namespace gleam {

// Lines (rows or columns) per workgroup tile and threads per workgroup, by transform length: 16 lines on 256 threads, a thread
// or two per butterfly, so that a tile is short from its first load to its last store and several workgroups share a CU (reducing rows of
// 368 on 384 threads: 37 us instead of 31 for 2 x 15 x 640 of them); 8 lines of 640 points (one tile of 16 would fill half of
// LDS), 64 lines where the whole transform is one butterfly.  MANY, for calls of many tiles (kManyTiles): 64 lines of 32 points, which
// are two butterflies a line (16 lines leave 224 of 256 threads without one), and 128 lines of 8 to 12 points (64 leave most
// threads idle in the coil sum).
template <int N> constexpr bool rows_have_many() { return N == 32 || (N >= 8 && N <= 12); }
template <int N, bool MANY = false> constexpr int rows_lines() { return N > 384 ? 8 : MANY ? (N == 32 ? 64 : 128) : N == 46 || N <= 24 ? 64 : 16; }
template <int N> constexpr int reduce_threads() { return 256; }
template <int N> constexpr int expand_threads() { return N == 320 ? 320 : N == 368 ? 384 : 256; }
template <int N> constexpr int fused_lines() { return N <= 32 ? 64 : N == 64 || N == 96 ? 32 : rows_lines<N>(); }
// Waves per SIMD that the compiler is asked to leave registers for.
template <int N> constexpr int rows_min_waves() { return N <= 256 && N != 46 ? 4 : 1; }
// Columns: 64 bytes a row of 640 points, 128 bytes otherwise; 256 bytes (WIDE) for 96 .. 256 points where there are tiles enough
// (8 x 256 x 160 x 160: the sweep along 256 points 196 -> 179 us; 2 x 8 x 320 x 256, with 256 tiles of 16 columns: 11.8 -> 13.5).
// Not the sweep that reads y (MODE 3) along 256 points: 512 threads share a CU with others only if they keep to 128 registers, and y
// makes it 141.  Three workgroups of 256 threads, nothing spilled, instead of two of 512 with 25 values spilled: the operator of
// a step, 8 x 256 x 160 x 160, 1023 -> 923 us, 4 x 16 x 256 x 256 55.8 -> 48.6.
template <int N, int MODE> constexpr bool cols_have_wide() { return N >= 96 && N <= 256 && !(N == 256 && MODE == 3); }
template <int N, bool WIDE> constexpr int cols_lines() { return N > 384 ? 8 : N <= 24 || N == 46 ? 64 : WIDE ? 32 : 16; }
template <int N, bool WIDE> constexpr int cols_threads() {
    return N <= 24 ? 64 : N == 46 ? 256 : N > 384 ? 256 : N == 320 ? 320 : N == 368 ? 384 : reduce_threads<N>() * cols_lines<N, WIDE>() / 16;
}
template <int N, int MODE> constexpr int cols_min_waves() {
    return N == 256 ? (MODE == 3 ? 3 : 4) : N == 368 ? 3 : 1;
}

struct RowsArgs {
    const float2* x;      // image [B][T][DH][W]
    const float2* S;      // coils [B][C][DH][W]
    float2* k;            // k-space [B][C][T][DH][W]
    float2* out;          // image (reduce only)
    long long DH;         // D*H rows per frame
    unsigned C, T;
    unsigned tiles;       // tiles per frame; tile number = frame * tiles + tile
    unsigned n_tiles, first;   // in all, and the launch's first
    unsigned cg, cg_inv;  // coils transformed together, and 65536 / cg rounded up: line / cg = (line * cg_inv) >> 16
    unsigned groups;      // expand: workgroups that share the coils of a tile
    unsigned lr;          // image rows per tile
    float scale;          // expand: axis_scale; reduce: what the inverse transforms still lack; fused: N^-1/2
    float xs, gs;         // reduce: out = xs*x + gs*g
    // Centred transform (frequency and spatial origin in the middle of every transformed axis; all lengths are even):
    // F_c = (-1)^(n/2) D F D per axis with D = diag((-1)^index), so the operator is the uncentred one on D x and
    // (sign) D y, times D.  cen: 0 / 1; par_h, par_d: whether the row index h / d takes part in the parity (the
    // axis is transformed); Hh: H, to split a row index into (d, h); ysign_bit: 1 when the product of the
    // (-1)^(n/2) over the transformed axes is -1.
    int cen, par_h, par_d, ysign_bit;
    unsigned Hh;
};
struct RowsCgArgs : RowsArgs {   // (apart, so that the plain sweeps' argument block stays as short as it was: + 0.4 us a call with it)
    CgFusion cg_job;
};
template <bool CG> using RowsArgsOf = typename std::conditional<CG, RowsCgArgs, RowsArgs>::type;

// v with its sign flipped when bit is 1 (bit is 0 or 1)
__device__ __forceinline__ float2 flip_sign(float2 v, unsigned bit) {
    return make_float2(__uint_as_float(__float_as_uint(v.x) ^ (bit << 31)), __uint_as_float(__float_as_uint(v.y) ^ (bit << 31)));
}
// parity of the transformed row coordinates of row dh = d*H + h (0 when the transform is not centred)
__device__ __forceinline__ unsigned row_parity(const RowsArgs& a, unsigned dh) {
    if (!a.cen) return 0u;
    const unsigned d = dh / a.Hh, h = dh - d * a.Hh;
    return ((a.par_h ? h : 0u) + (a.par_d ? d : 0u)) & 1u;
}

// A row tile: a.lr image rows of one frame x a.cg coils.  Line l = r * cg + c is coil c0 + c of image row row0 + r; a line
// past the tile's rows, the frame's or the coils reads the last one there is, and nothing of it is kept.
struct RowTile {
    long long frame, row0, b;   // frame b * T + t; first image row inside the frame; sample
    unsigned t, rows;           // image rows of the tile inside the frame
    __device__ __forceinline__ RowTile(const RowsArgs& a, unsigned id) {
        const unsigned f = id / a.tiles, bb = f / a.T;
        frame = f; b = bb; t = f - bb * a.T;
        row0 = (long long)(id - f * a.tiles) * a.lr;
        rows = a.DH - row0 < a.lr ? (unsigned)(a.DH - row0) : a.lr;
    }
};
struct RowLine {
    unsigned r, c;
    bool real;
    __device__ __forceinline__ RowLine(const RowsArgs& a, const RowTile& tile, unsigned line, unsigned ncg) {
        const unsigned rr = (line * a.cg_inv) >> 16, cc = line - rr * a.cg;
        real = rr < tile.rows && cc < ncg;
        r = rr < tile.rows ? rr : tile.rows - 1;
        c = cc < ncg ? cc : ncg - 1;
    }
};

// D x of a centred transform: the sign of value q of a butterfly whose first one has parity `par`
template <int R, int T> __device__ __forceinline__ void alternate(float2 (&u)[R], unsigned par) {
#pragma unroll
    for (int q = 0; q < R; ++q) u[q] = flip_sign(u[q], (par ^ (unsigned)(q * T)) & 1u);
}

// Forward transform along W of S*x, without and with the solver's update of x.
//
// Without: a tile is L image rows, and the workgroup goes through every `groups`-th coil.  A coil at a time moves long runs of k-space and coil maps, and neighbouring
// workgroups, which are at about the same coil, keep all memory channels busy: the coils of a volume lie multiples of 1 MiB
// apart, and with all of them in one tile, 8 x 256 x 160 x 160 took 196 us, 202 us with a workgroup per coil side by side, and
// takes 175 us = 5.1 TB/s like this.
template <int N, bool MANY>
__global__ __launch_bounds__(expand_threads<N>(), (rows_min_waves<N>())) void rows_expand_kernel(RowsArgs a) {
    constexpr int L = rows_lines<N, MANY>(), NT = expand_threads<N>();
    __shared__ float2 buf[Tile<N, L, true>::kElems];
    // workgroups go to the eight XCDs in turn: those that share a tile to the same one, whose L2 holds its image rows
    const unsigned slot = blockIdx.x >> 3, id = a.first + slot / a.groups * 8 + (blockIdx.x & 7);
    if (id >= a.n_tiles) return;   // uniform for the workgroup
    const RowTile tile(a, id);
    const long long sstride = a.DH * N, kstride = a.T * sstride;
    const float2* const x = a.x + (tile.frame * a.DH + tile.row0) * N;
    const float2* const S = a.S + (tile.b * a.C * a.DH + tile.row0) * N;
    float2* const k = a.k + ((tile.b * a.C * a.T + tile.t) * a.DH + tile.row0) * N;
    for (unsigned c = slot % a.groups; c < a.C; c += a.groups) {
        fft_tile<N, L, NT, true>(
            buf,
            [&](unsigned line, unsigned i, auto step, auto& u, int) {
                constexpr int T = decltype(step)::value, R = sizeof(u) / sizeof(float2);
                const unsigned o = (line < tile.rows ? line : tile.rows - 1) * N + i;
                const float2 *const xp = x + o, *const sp = S + c * sstride + o;
                float2 xv[R], sv[R];
#pragma unroll
                for (int q = 0; q < R; ++q) { xv[q] = xp[q * T]; sv[q] = sp[q * T]; }
#pragma unroll
                for (int q = 0; q < R; ++q) u[q] = cmul(sv[q], xv[q]);
                if (a.cen) alternate<R, T>(u, row_parity(a, (unsigned)tile.row0 + line) + i);
            },
            [&](unsigned line, unsigned i, auto step, auto& u, int) {
                constexpr int P = decltype(step)::value;
                if (line < tile.rows) {
                    float2* const kp = k + c * kstride + line * N + i;
#pragma unroll
                    for (int q = 0; q < (int)(sizeof(u) / sizeof(float2)); ++q) kp[q * P] = make_float2(u[q].x * a.scale, u[q].y * a.scale);
                }
            });
        if (c + a.groups < a.C) __syncthreads();   // the next coil overwrites the exchange
    }
}

// With: x <- r + beta x first (CgFusion).  A tile is lr image rows x all coils; every coil line forms the new values for
// itself, and those of the first coil write them back behind the first exchange, when no line of the tile reads the old ones
// any more.
template <int N, bool MANY>
__global__ __launch_bounds__(expand_threads<N>(), (rows_min_waves<N>())) void rows_expand_update_kernel(RowsCgArgs a) {
    constexpr int L = rows_lines<N, MANY>(), NT = expand_threads<N>();
    __shared__ float2 buf[Tile<N, L, true>::kElems];
    const RowTile tile(a, a.first + blockIdx.x);
    const long long at = (tile.frame * a.DH + tile.row0) * N;   // first image element of the tile
    const long long sstride = a.DH * N, kstride = a.T * sstride;
    const float2* const S = a.S + (tile.b * a.C * a.DH + tile.row0) * N;
    float2* const k = a.k + ((tile.b * a.C * a.T + tile.t) * a.DH + tile.row0) * N;
    // the image, the residual, the coil maps and the partial sums are all requested before the first of them is needed
    constexpr int PER = first_butterflies(N, L, NT), R = first_points(N);
    float2 xv[PER][R], rv[PER][R], sv[PER][R];
    first_points_of<N, L, NT>([&](unsigned line, unsigned i, auto step, int m) {
        constexpr int T = decltype(step)::value;
        const RowLine ln(a, tile, line, a.C);
        const unsigned o = ln.r * N + i;
        const float2* const sp = S + ln.c * sstride + o;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            xv[m][q] = a.x[at + o + q * T];
            rv[m][q] = a.cg_job.r[at + o + q * T];
            sv[m][q] = sp[q * T];
        }
    });
    // every wave adds up the partial sums of the sample for itself
    const CgFusion& cg = a.cg_job;
    static_assert(kCgFusedSums == 128, "two partial sums per lane");
    double den = 0.0, num = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = (threadIdx.x & 63) + 64 * h;
        const bool in = i < cg.nb;
        const double o = cg.rr_old[tile.b * cg.nb + (in ? i : 0)], n = cg.rr_new[tile.b * cg.nb + (in ? i : 0)];
        den += in ? o : 0.0;
        num += in ? n : 0.0;
    }
    for (int o = 32; o > 0; o >>= 1) {
        den += __shfl_xor(den, o);
        num += __shfl_xor(num, o);
    }
    const float beta = den > 0.0 ? (float)(num / den) : 0.f;
    fft_tile<N, L, NT, true>(
        buf,
        [&](unsigned line, unsigned i, auto step, auto& u, int m) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                xv[m][q] = make_float2(fmaf(beta, xv[m][q].x, rv[m][q].x), fmaf(beta, xv[m][q].y, rv[m][q].y));
                u[q] = cmul(sv[m][q], xv[m][q]);
            }
            if (a.cen) alternate<R, decltype(step)::value>(u, row_parity(a, (unsigned)tile.row0 + RowLine(a, tile, line, a.C).r) + i);
        },
        [&](unsigned line, unsigned i, auto step, auto& u, int) {
            constexpr int P = decltype(step)::value;
            const RowLine ln(a, tile, line, a.C);
            if (ln.real) {
                float2* const kp = k + ln.c * kstride + ln.r * N + i;
#pragma unroll
                for (int q = 0; q < (int)(sizeof(u) / sizeof(float2)); ++q) kp[q * P] = make_float2(u[q].x * a.scale, u[q].y * a.scale);
            }
        });
    first_points_of<N, L, NT>([&](unsigned line, unsigned i, auto step, int m) {   // (synchronised since the points were read)
        const RowLine ln(a, tile, line, a.C);
        if (ln.real && ln.c == 0) {
            float2* const xw = cg.x_rw + at + ln.r * N + i;
#pragma unroll
            for (int q = 0; q < R; ++q) xw[q * decltype(step)::value] = xv[m][q];
        }
    });
}

// Inverse transform along W and coil reduction.  A tile is lr image rows x cg coils transformed together; then
// out = xs*x + gs * sum_c conj(S_c) * row_c is accumulated in registers, looping over coil groups when C > cg.  The per-coil
// images never leave LDS.  lr is capped so that a thread owns at most kRedAcc output values, twice as many where rows of 640 points
// would leave half of the tile's eight lines or more without work (one row a tile, up to four coils: 2 x 32 x 256 x 640, the
// sweep with one coil 179 us, 92 where it is staged through LDS; the operator 323 -> 220, with four coils 822 -> 746).
constexpr int kRedAcc = 4;
constexpr bool reduce_has_double(int N) { return N > 384; }
static inline int reduce_rows_per_tile(int N, int L, int threads, long long C) {
    const int cg = C < L ? (int)C : L, lr = L / cg;
    int most = kRedAcc * threads / N < 1 ? 1 : kRedAcc * threads / N;
    if (reduce_has_double(N) && 2 * most * cg <= L) most = 2 * kRedAcc * threads / N;
    return lr < most ? lr : most;
}

// The coil sum of one tile, PER values per thread.  The coil maps of the first kMaps coils of a group, as a rule all there
// are, are requested ahead of its transform.
template <int N, int L, int NT, int PER> struct CoilSum {
    static constexpr int kMaps = (N > 384 && PER <= 4 ? 8 : 16) / PER;
    using Lay = Tile<N, L, true>;
    float2 acc[PER], sv[PER][kMaps];
    const float2* sp[PER];   // coil map of the first coil at the thread's values
    long long sstride;
    unsigned at[PER];        // their places in the line of the first coil
    bool own[PER];
    __device__ __forceinline__ CoilSum(const RowsArgs& a, const RowTile& tile, const float2* S) {
        sstride = a.DH * N;
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const unsigned e = threadIdx.x + m * NT, r = e / N;   // index over the rows of the tile
            own[m] = r < tile.rows;
            at[m] = own[m] ? Lay::at(r * a.cg, e % N) : 0;
            sp[m] = S + (own[m] ? e : 0);
            acc[m] = make_float2(0.f, 0.f);
        }
    }
    __device__ __forceinline__ void maps(unsigned c, unsigned end) {   // of coils c .. c + kMaps - 1, as far as there are any
#pragma unroll
        for (int j = 0; j < kMaps; ++j)
            if (c + j < end) {
#pragma unroll
                for (int m = 0; m < PER; ++m) sv[m][j] = sp[m][(c + j) * sstride];
            }
    }
    __device__ __forceinline__ void add(const float2* buf, unsigned c0, unsigned ncg) {
        for (unsigned c = 0; c < ncg; c += kMaps) {
            if (c) maps(c0 + c, c0 + ncg);
#pragma unroll
            for (int j = 0; j < kMaps; ++j)
                if (c + j < ncg) {
#pragma unroll
                    for (int m = 0; m < PER; ++m) {
                        const float2 p = cmul_conj(buf[at[m] + (c + j) * Lay::kLine], sv[m][j]);
                        acc[m].x += p.x; acc[m].y += p.y;
                    }
                }
        }
    }
};

// out[at] = xs * x[at] + gs * g, with the sign of a centred transform (D g)
__device__ __forceinline__ float2 dc_value(const RowsArgs& a, float2 g, long long at, unsigned par) {
    const float gs = a.gs * a.scale, s = a.cen && par ? -gs : gs;
    float2 res = make_float2(s * g.x, s * g.y);
    if (a.xs != 0.f) {
        const float2 xv = a.x[at];
        res.x = fmaf(a.xs, xv.x, res.x);
        res.y = fmaf(a.xs, xv.y, res.y);
    }
    a.out[at] = res;
    return res;
}

// DOT: every tile also writes its part of Re <x, out> (CgFusion), summed in double.
template <int N, bool MANY, int PER, bool DOT>
__global__ __launch_bounds__(reduce_threads<N>(), (rows_min_waves<N>())) void rows_reduce_kernel(RowsArgsOf<DOT> a) {
    constexpr int L = rows_lines<N, MANY>(), NT = reduce_threads<N>();
    __shared__ float2 buf[Tile<N, L, true>::kElems];
    __shared__ double red[DOT ? NT / 64 : 1];
    const RowTile tile(a, blockIdx.x + a.first);
    const long long at = (tile.frame * a.DH + tile.row0) * N;   // first image element of the tile
    const long long kstride = a.T * a.DH * N;
    const float2* const k = a.k + ((tile.b * a.C * a.T + tile.t) * a.DH + tile.row0) * N;
    CoilSum<N, L, NT, PER> sum(a, tile, a.S + (tile.b * a.C * a.DH + tile.row0) * N);
    for (unsigned c0 = 0; c0 < a.C; c0 += a.cg) {
        const unsigned ncg = a.C - c0 < a.cg ? a.C - c0 : a.cg;
        if (c0) __syncthreads();
        sum.maps(c0, c0 + ncg);
        ifft_tile<N, L, NT, true, true>(
            buf,
            [&](unsigned line, unsigned i, auto step, auto& u, int) {
                constexpr int T = decltype(step)::value, R = sizeof(u) / sizeof(float2);
                const RowLine ln(a, tile, line, ncg);
                const float2* const kp = k + (c0 + ln.c) * kstride + ln.r * N + i;
#pragma unroll
                for (int q = 0; q < R; ++q) u[q] = kp[q * T];
            },
            [&](unsigned, unsigned, auto, auto&, int) {});
        __syncthreads();
        sum.add(buf, c0, ncg);
    }
    double dot = 0.0;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        if (sum.own[m]) {
            const unsigned e = threadIdx.x + m * NT;
            const float2 res = dc_value(a, sum.acc[m], at + e, (row_parity(a, (unsigned)tile.row0 + e / N) + e % N) & 1u);
            if constexpr (DOT) {
                const float2 xv = a.x[at + e];
                dot += (double)xv.x * res.x + (double)xv.y * res.y;
            }
        }
    }
    if constexpr (DOT) {   // a tile's rows belong to one sample
        for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dot;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < NT / 64; ++w) dot += red[w];
            a.cg_job.dot[blockIdx.x + a.first] = dot;
        }
    }
}

// One transformed axis only (ndim_fft = 1: the mask does not depend on the other image axes, e.g. line masks of
// 2D Cartesian sampling after the transform along the fully sampled axis has been taken out of the data): the
// whole operator in one sweep, nothing but S, x, y and the mask is read and only the image is written.  Tiles as in
// rows_reduce_kernel; per coil group: S*x -> forward transform -> mask ? k - y : 0 -> inverse transform -> accumulate
// conj(S)*row.
template <int N, int PER, bool Y>
__global__ __launch_bounds__(expand_threads<N>()) void rows_fused_kernel(RowsArgs a, const float2* __restrict__ y,
                                                                      const unsigned char* __restrict__ M) {
    constexpr int L = fused_lines<N>(), NT = expand_threads<N>();
    __shared__ float2 buf[Tile<N, L, true>::kElems];
    const RowTile tile(a, blockIdx.x + a.first);
    const long long at = (tile.frame * a.DH + tile.row0) * N;
    const long long sstride = a.DH * N, kstride = a.T * sstride, kat = ((tile.b * a.C * a.T + tile.t) * a.DH + tile.row0) * N;
    const float2* const S = a.S + (tile.b * a.C * a.DH + tile.row0) * N;
    CoilSum<N, L, NT, PER> sum(a, tile, S);
    for (unsigned c0 = 0; c0 < a.C; c0 += a.cg) {
        const unsigned ncg = a.C - c0 < a.cg ? a.C - c0 : a.cg;
        if (c0) __syncthreads();
        fft_ifft_tile<N, L, NT, true, true>(
            buf,
            [&](unsigned line, unsigned i, auto step, auto& u, int) {
                constexpr int T = decltype(step)::value, R = sizeof(u) / sizeof(float2);
                const RowLine ln(a, tile, line, ncg);
                const float2* const xp = a.x + at + ln.r * N + i;
                const float2* const sp = S + (c0 + ln.c) * sstride + ln.r * N + i;
                float2 xv[R], sv[R];
#pragma unroll
                for (int q = 0; q < R; ++q) { xv[q] = xp[q * T]; sv[q] = sp[q * T]; }
#pragma unroll
                for (int q = 0; q < R; ++q) u[q] = cmul(sv[q], xv[q]);
                if (a.cen) alternate<R, T>(u, i);
            },
            [&](unsigned line, unsigned i, auto step, auto& u, int) {
                constexpr int P = decltype(step)::value, R = sizeof(u) / sizeof(float2);
                const RowLine ln(a, tile, line, ncg);
                const unsigned char* const mp = M + at + ln.r * N + i;
                const float2* const yp = y + kat + (c0 + ln.c) * kstride + ln.r * N + i;
                unsigned char mv[R];
                float2 yv[R];
#pragma unroll
                for (int q = 0; q < R; ++q) mv[q] = mp[q * P];
                if constexpr (Y) {
#pragma unroll
                    for (int q = 0; q < R; ++q) yv[q] = yp[q * P];
                    if (a.cen) {   // (-1)^(N/2) D y
#pragma unroll
                        for (int q = 0; q < R; ++q) yv[q] = flip_sign(yv[q], ((unsigned)a.ysign_bit + i + q * P) & 1u);
                    }
                }
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    float2 v = make_float2(u[q].x * a.scale, u[q].y * a.scale);
                    if constexpr (Y) v = make_float2(u[q].x * a.scale - yv[q].x, u[q].y * a.scale - yv[q].y);
                    u[q] = mv[q] ? v : make_float2(0.f, 0.f);
                }
            },
            [&](unsigned, unsigned, auto, auto&, int) {}, []() {});
        sum.maps(c0, c0 + ncg);
        __syncthreads();
        sum.add(buf, c0, ncg);
    }
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const unsigned e = threadIdx.x + m * NT;
        if (sum.own[m]) dc_value(a, sum.acc[m], at + e, e & 1u);
    }
}

struct ColsArgs {
    float2* k;             // k-space viewed as [outer][N][inner], transformed in place along N
    const float2* y;       // measured k-space, same view (mid only; may be null)
    const unsigned char* M;  // mask (mid only)
    unsigned inner;        // even (it is a product of transform lengths, all even); N * inner * 8 stays below 2^32
    unsigned tiles_per, n_tiles;   // column tiles per outer index, and in all
    unsigned first;                // the launch's first tile
    unsigned C, TD;        // outer = (b*C + c)*TD + td ; mask row = b*TD + td
    float scale;           // applied at the store (axis_scale)
    float fwd;             // mid: what the forward transforms still lack, applied before y is subtracted
    // Centred transform.  cen_y (mid sweep): the measured k-space enters as (sign) D y, where the parity of an
    // element is p + (column / Wrow) + (column % Wrow) (the inner index is h*W + w when three axes are transformed,
    // w alone otherwise: then column / Wrow is 0) and ysign_bit is 1 when the product of (-1)^(n/2) over the
    // transformed axes is -1.  cen_io (MODE 1 on its own, k-space to hybrid space): the centred inverse transform
    // of this axis, (-1)^(N/2) D F^H D: input and output signs by the parity of p.
    int cen_y, ysign_bit, cen_io;
    unsigned Wrow;
    // Walk the tiles from the last to the first.  The k-space buffer of the 3D workload (419 MB) is larger than the
    // Infinity Cache (256 MB), which holds what the previous sweep wrote last: a sweep that starts where the previous
    // one ended finds that part there.
    int rev;
};

// Mask bytes of a column tile ([N rows][L columns], row p at mb + p*L) into LDS.  One thread fetches a whole row
// segment with a single 8- or 16-byte load where the addresses allow it (2-byte loads per element pair would issue as
// many memory requests as the k-space tile itself); columns past `valid` read as 0.  The loads are issued by the
// constructor, and waited for in put().
template <int N, int L, int NT> struct MaskTile {
    static constexpr int Q = L > 16 ? L / 16 : 1, PER = (N * Q + NT - 1) / NT;
    using Segment = typename std::conditional<L == 8, uint2, uint4>::type;
    const unsigned char* M;
    unsigned inner, valid;
    bool vec;
    Segment v[PER];
    __device__ __forceinline__ MaskTile(const unsigned char* M_, unsigned inner_, unsigned valid_) : M(M_), inner(inner_), valid(valid_) {
        vec = valid == L && inner % L == 0 && reinterpret_cast<unsigned long long>(M) % L == 0;
#pragma unroll
        for (int m = 0; m < PER; ++m) v[m] = Segment{};
        if (vec) {
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                const unsigned e = threadIdx.x + m * NT;
                if (e < N * Q) v[m] = *reinterpret_cast<const Segment*>(M + (e / Q * inner + 16 * (e % Q)));
            }
        }
    }
    __device__ __forceinline__ void put(unsigned char* mb) const {
        if (vec) {
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                const unsigned e = threadIdx.x + m * NT;
                if (e < N * Q) *reinterpret_cast<Segment*>(mb + e * sizeof(Segment)) = v[m];
            }
        } else {
            for (unsigned i = threadIdx.x; i < N * (L / 2); i += NT) {
                const unsigned l = 2 * (i % (L / 2)), p = i / (L / 2);
                unsigned short two = 0;
                if (l < valid) two = *reinterpret_cast<const unsigned short*>(M + (p * inner + l));
                *reinterpret_cast<unsigned short*>(mb + p * L + l) = two;
            }
        }
    }
};

// Strided axis: a tile is L neighbouring columns (128 contiguous bytes per row) of one [N][inner] plane.
// MODE 0: forward, 1: inverse, 2: forward -> (mask ? k : 0) -> inverse, 3: forward -> (mask ? k - y : 0) -> inverse
// (a kernel of its own: with the y path merely compiled in, the sweep without y ran 20-30 % slower).
template <int N, int MODE, bool WIDE>
__global__ __launch_bounds__((cols_threads<N, WIDE>()), (cols_min_waves<N, MODE>())) void cols_kernel(ColsArgs a) {
    constexpr int L = cols_lines<N, WIDE>(), NT = cols_threads<N, WIDE>();
    using Lay = Tile<N, L, false>;
    __shared__ float2 buf[Lay::kSingle ? 1 : Lay::kElems];
    __shared__ __attribute__((aligned(16))) unsigned char mb[MODE >= 2 ? N * L : 16];
    // Neighbouring column tiles share 128-byte lines: each XCD (workgroups are dealt to the eight in turn) owns a contiguous
    // eighth of the tiles, so that they go to the same L2.
    const unsigned per = gridDim.x >> 3, it = a.first + (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (it >= a.n_tiles) return;   // uniform for the workgroup
    const unsigned tile = a.rev ? a.n_tiles - 1 - it : it;
    const unsigned o = tile / a.tiles_per, i0 = (tile - o * a.tiles_per) * L;
    const unsigned valid = a.inner - i0 < L ? a.inner - i0 : L;   // even
    const long long base = (long long)o * N * a.inner + i0;
    float2* const k = a.k + base;
    const auto load = [&](unsigned line, unsigned i, auto step, auto& u, int) {
        constexpr int T = decltype(step)::value, R = sizeof(u) / sizeof(float2);
        const float2* const kp = k + (line < valid ? line : 0);
#pragma unroll
        for (int q = 0; q < R; ++q) u[q] = kp[(i + q * T) * a.inner];
        if constexpr (MODE == 1) {
            if (a.cen_io) {
#pragma unroll
                for (int q = 0; q < R; ++q) u[q] = flip_sign(u[q], (i + q * T) & 1u);
            }
        }
    };
    const auto store = [&](unsigned line, unsigned i, auto step, auto& u, int) {
        constexpr int P = decltype(step)::value, R = sizeof(u) / sizeof(float2);
        if (line < valid) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                float sc = a.scale;
                if constexpr (MODE == 1) {
                    if (a.cen_io && ((i + q * P + N / 2) & 1)) sc = -sc;
                }
                k[(i + q * P) * a.inner + line] = make_float2(u[q].x * sc, u[q].y * sc);
            }
        }
    };
    if constexpr (MODE < 2) {
        if constexpr (MODE == 1) ifft_tile<N, L, NT, false, false>(buf, load, store);
        else fft_tile<N, L, NT, false>(buf, load, store);
    } else {
        const unsigned bc = o / a.TD, td = o - bc * a.TD, b = bc / a.C;
        const MaskTile<N, L, NT> mask(a.M + ((long long)(b * a.TD + td) * N * a.inner + i0), a.inner, valid);
        // y at the points the last stage hands over: T lines of i next to each other, R of them T positions apart
        constexpr int R = last_radix(N), T = N / R, PER = (L * T + NT - 1) / NT;
        float2 yv[MODE == 3 ? PER : 1][R];
        const float fs = a.fwd;
        fft_ifft_tile<N, L, NT, false, false>(
            buf, load,
            [&](unsigned line, unsigned i, auto step, auto& u, int m) {
                if constexpr (MODE == 3) {
                    if (a.cen_y) {   // (sign) D y
                        const unsigned col = i0 + line, hrow = col / a.Wrow, par = a.ysign_bit + i + hrow + (col - hrow * a.Wrow);
#pragma unroll
                        for (int q = 0; q < R; ++q) yv[m][q] = flip_sign(yv[m][q], (par + q * T) & 1u);
                    }
                }
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    float2 v = make_float2(u[q].x * fs, u[q].y * fs);
                    if constexpr (MODE == 3) v = make_float2(u[q].x * fs - yv[m][q].x, u[q].y * fs - yv[m][q].y);
                    u[q] = mb[(i + q * T) * L + line] ? v : make_float2(0.f, 0.f);
                }
            },
            store,
            [&]() {   // behind the first loads
                mask.put(mb);
                if constexpr (Lay::kSingle) __syncthreads();   // (otherwise the exchange between the stages comes first)
                if constexpr (MODE == 3) {
#pragma unroll
                    for (int m = 0; m < PER; ++m) {
                        const unsigned idx = threadIdx.x + m * NT, line = idx % L, i = idx / L;
                        if (PER * NT == L * T || idx < L * T) {
                            const float2* const yp = a.y + base + (line < valid ? line : 0);
#pragma unroll
                            for (int q = 0; q < R; ++q) yv[m][q] = yp[(i + q * T) * a.inner];
                        }
                    }
                }
            });
    }
}

// ------------------------------------------------------------------ host dispatch
bool fft_size_supported(long long n) {
    switch (n) {
#define X(N) case N:
        GLEAM_FFT_SIZES(X)
#undef X
        return true;
        default: return false;
    }
}

// Tiles from which the row sweeps take more lines to a tile (MANY).  The operator without / with, us: 4 x 16 x 8 x 640 x 32 (20480
// tiles) 136 / 102, 2 x 20 x 8 x 256 x 32 (5120) 53.5 / 41.4, 16 x 400 x 16 x 32 (6400) 55.5 / 55.6, 16 x 20 x 64 x 32 (1280)
// 18.3 / 20.6, 4 x 20 x 160 x 32 (800) 16.0 / 16.2, 8 x 64 x 32 (32) 10.4 / 12.4; 4 x 16 x 8 x 640 x 8 (5120) 47.6 / 34.5, 16 x
// 400 x 16 x 10 (1600) 36.4 / 35.1, 16 x 20 x 64 x 8 (320) 11.8 / 12.0.
constexpr long long kManyTiles = 2048;
template <int N> static int rows_lines_for(const gleam_geom& g) {
    if constexpr (rows_have_many<N>()) {
        if (g.B * g.C * g.T * g.D * g.H >= kManyTiles * rows_lines<N>()) return rows_lines<N, true>();
    }
    return rows_lines<N>();
}
static int rows_lines_of(const gleam_geom& g) {
    switch (g.W) {
#define X(NN) case NN: return rows_lines_for<NN>(g);
        GLEAM_FFT_SIZES(X)
#undef X
        default: return 1;
    }
}
static int reduce_rows_of(const gleam_geom& g) {
    switch (g.W) {
#define X(NN) case NN: return reduce_rows_per_tile(NN, rows_lines_for<NN>(g), reduce_threads<NN>(), g.C);
        GLEAM_FFT_SIZES(X)
#undef X
        default: return 1;
    }
}

// A launch takes at most so many tiles (the threads of a grid are counted in 32 bits); more go into several launches.
constexpr long long kLaunchTiles = 1LL << 22;

// Workgroups up to which the coils of a tile are spread over several.
constexpr long long kExpandGroups = 2048;
// Where the single sweep of one transformed axis stays with the kernel staged through LDS, which needs half the registers (a CU
// holds four or five of its workgroups, of this one's one to three) and whose tiles go across frames (staged / here, us):
//   - Rows of kFusedStaged points and more.  8 coils, 20 x 160 rows: 38 and 22 us at 256 points, 45 and 51 at 320, 59 and 65 at 368,
//     91 and 106 at 640.
//   - Frames that leave more than a fifth of their tiles' rows empty, from more than kFusedTiles tiles on (what the card holds at once):
//     1600 frames of 1 x 160, 4 coils 10.0 / 17.5; of 20 x 24, 4 coils 17.8 / 26.7.  400 tiles: 400 frames of 8 x 24, 4 coils
//     9.5 / 8.9.
//   - Rows of 20 and 24 points, one butterfly, which one of four waves transforms while the others wait, from half as many tiles
//     more on (with y, which takes the registers of the third workgroup, from kFusedTiles): 64 frames of 320 x 20, 2 coils
//     0.80 of the time here; 8 frames of 320 x 24, 16 coils (640 tiles) 1.28, with y 0.84.  Shorter rows only with y or of one
//     coil: 1600 frames of 64 x 16, 2 coils, with y 0.71; 1 coil 0.80; 16 coils 1.05.
//   - The 23-point stage of 46 points with y, one workgroup to a CU: from a second round of them on (2 x 8 x 641 rows, 2 coils
//     16.5 / 22.5; 320 rows of 8 coils, 40 tiles 15.3 / 12.7).
//   - With y, tiles with few coils, which use no more than about half of their lines (the coil sum holds four values per thread):
//     400 frames of 64 x 256, 1 coil 0.85; without y 1.03, 2 coils with y 0.93 to 1.1.
// Over 1561 calls of 8 to 256 points, 1 to 16 coils, frames of 1 to 320 rows, 1 to 1600 of them, the calls are 1.23 (with y 1.16) times
// as fast as with the staged kernel alone and 1.07 (1.10) times as with this one alone.
constexpr int kFusedStaged = 320;
constexpr long long kFusedTiles = 512;
// Tiles from which the column sweeps take 32 columns instead of 16 (256 bytes a row).
constexpr long long kWideTiles = 2048;

// Fills in the tiling of a row sweep, `cg` coils per tile; the number of tiles.
static long long tile_rows(const gleam_geom& g, long long cg, long long rows, RowsArgs& a) {
    a.cg = (unsigned)cg;
    a.cg_inv = (65536u + a.cg - 1) / a.cg;
    a.lr = (unsigned)rows;
    a.groups = 1;
    a.tiles = (unsigned)((a.DH + a.lr - 1) / a.lr);
    const long long n = g.B * g.T * a.tiles;
    a.n_tiles = (unsigned)n;
    return n;
}

// Values per thread of a reducing sweep: 1, 2, 4 (kRedAcc) or 8, as many as the tile's rows need.
template <int N, bool MANY, int PER> static void launch_reduce_t(const RowsCgArgs& a, dim3 grid, hipStream_t st) {
    if (a.cg_job.dot) hipLaunchKernelGGL((rows_reduce_kernel<N, MANY, PER, true>), grid, dim3(reduce_threads<N>()), 0, st, a);
    else hipLaunchKernelGGL((rows_reduce_kernel<N, MANY, PER, false>), grid, dim3(reduce_threads<N>()), 0, st, (const RowsArgs&)a);
}
template <int N, bool MANY> static void launch_rows_t(bool reduce, const RowsCgArgs& a, dim3 grid, hipStream_t st) {
    const int per = ((int)a.lr * N + reduce_threads<N>() - 1) / reduce_threads<N>();
    if (!reduce) {
        if (a.cg_job.r) hipLaunchKernelGGL((rows_expand_update_kernel<N, MANY>), grid, dim3(expand_threads<N>()), 0, st, a);
        else hipLaunchKernelGGL((rows_expand_kernel<N, MANY>), grid, dim3(expand_threads<N>()), 0, st, (const RowsArgs&)a);
    } else if (per <= 1) launch_reduce_t<N, MANY, 1>(a, grid, st);
    else if (per <= 2) launch_reduce_t<N, MANY, 2>(a, grid, st);
    else if (per <= 4 || !reduce_has_double(N)) launch_reduce_t<N, MANY, 4>(a, grid, st);
    else if constexpr (reduce_has_double(N)) launch_reduce_t<N, MANY, 8>(a, grid, st);
}
template <int N> static void launch_rows_fused_t(const gleam_geom& g, RowsArgs a, const float2* y, const unsigned char* M, hipStream_t st) {
    if constexpr (N < kFusedStaged) {
        constexpr int L = fused_lines<N>(), NT = expand_threads<N>();
        const long long n = tile_rows(g, g.C < L ? g.C : L, reduce_rows_per_tile(N, L, NT, g.C), a);
        const int per = ((int)a.lr * N + NT - 1) / NT;
        for (long long first = 0; first < n; first += kLaunchTiles) {
            a.first = (unsigned)first;
            const dim3 grid((unsigned)(n - first < kLaunchTiles ? n - first : kLaunchTiles));
            if (y) {
                if (per <= 1) hipLaunchKernelGGL((rows_fused_kernel<N, 1, true>), grid, dim3(NT), 0, st, a, y, M);
                else if (per <= 2) hipLaunchKernelGGL((rows_fused_kernel<N, 2, true>), grid, dim3(NT), 0, st, a, y, M);
                else hipLaunchKernelGGL((rows_fused_kernel<N, 4, true>), grid, dim3(NT), 0, st, a, y, M);
            } else {
                if (per <= 1) hipLaunchKernelGGL((rows_fused_kernel<N, 1, false>), grid, dim3(NT), 0, st, a, y, M);
                else if (per <= 2) hipLaunchKernelGGL((rows_fused_kernel<N, 2, false>), grid, dim3(NT), 0, st, a, y, M);
                else hipLaunchKernelGGL((rows_fused_kernel<N, 4, false>), grid, dim3(NT), 0, st, a, y, M);
            }
        }
    }
}

static hipError_t launch_rows(const gleam_geom& g, bool reduce, RowsCgArgs a, hipStream_t st) {
    const int L = rows_lines_of(g);
    const bool plain = !reduce && !a.cg_job.r;
    const long long cg = plain ? 1 : g.C < L ? g.C : L;
    const long long n = tile_rows(g, cg, reduce ? reduce_rows_of(g) : L / cg, a);
    if (plain) {   // as many coils in turn as leave kExpandGroups workgroups
        const long long turns = n * g.C / kExpandGroups;
        a.groups = (unsigned)(turns <= 1 ? g.C : turns >= g.C ? 1 : (g.C + turns - 1) / turns);
    }
    const long long most = plain ? kLaunchTiles / a.groups / 8 * 8 + 8 : kLaunchTiles;
    for (long long first = 0; first < n; first += most) {
        a.first = (unsigned)first;
        const long long m = n - first < most ? n - first : most;
        const dim3 grid((unsigned)(plain ? (m + 7) / 8 * 8 * a.groups : m));
        switch (g.W) {
#define X(NN)                                                                         \
    case NN:                                                                          \
        if (rows_have_many<NN>() && L != rows_lines<NN>())                            \
            launch_rows_t<NN, rows_have_many<NN>()>(reduce, a, grid, st);             \
        else                                                                          \
            launch_rows_t<NN, false>(reduce, a, grid, st);                            \
        break;
            GLEAM_FFT_SIZES(X)
#undef X
            default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

template <int N> static bool fused_staged_t(const gleam_geom& g, bool y) {
    constexpr int L = fused_lines<N>();
    const long long cg = g.C < L ? g.C : L, per = reduce_rows_per_tile(N, L, expand_threads<N>(), g.C);
    const long long rows = g.D * g.H, of_frame = (rows + per - 1) / per, tiles = g.B * g.T * of_frame;
    if (N >= kFusedStaged) return true;
    if (N == 46 && y && tiles > kFusedTiles / 2) return true;
    if (tiles <= kFusedTiles) return false;
    if (5 * rows < 4 * of_frame * per) return true;
    if (N <= 24 && tiles > kFusedTiles * 3 / 2) return y || N > 16 || g.C == 1;
    return y && (N <= 24 ? N > 16 : 20 * per * cg < 11 * L);
}
static bool fused_staged(const gleam_geom& g, bool y) {
    switch (g.W) {
#define X(NN) case NN: return fused_staged_t<NN>(g, y);
        GLEAM_FFT_SIZES(X)
#undef X
        default: return false;
    }
}

static hipError_t launch_rows_fused(const gleam_geom& g, const RowsArgs& a, const float2* y, const unsigned char* M, hipStream_t st) {
    switch (g.W) {
#define X(NN) case NN: launch_rows_fused_t<NN>(g, a, y, M, st); break;
        GLEAM_FFT_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int N, int MODE, bool WIDE> static void launch_cols_t(long long outer, ColsArgs a, hipStream_t st) {
    constexpr int L = cols_lines<N, WIDE>();
    a.tiles_per = (a.inner + L - 1) / L;
    const long long n = outer * a.tiles_per;
    if constexpr (!WIDE && cols_have_wide<N, MODE>()) {
        if (n >= 2 * kWideTiles) return launch_cols_t<N, MODE, true>(outer, a, st);
    }
    a.n_tiles = (unsigned)n;
    for (long long first = 0; first < n; first += kLaunchTiles) {
        a.first = (unsigned)first;
        const long long m = n - first < kLaunchTiles ? n - first : kLaunchTiles;
        const dim3 grid((unsigned)((m + 7) / 8 * 8)), block(cols_threads<N, WIDE>());   // a multiple of 8 for the split over the XCDs
        hipLaunchKernelGGL((cols_kernel<N, MODE, WIDE>), grid, block, 0, st, a);
    }
}
template <int N> static void launch_cols_n(int mode, long long outer, const ColsArgs& a, hipStream_t st) {
    if (mode == 0) launch_cols_t<N, 0, false>(outer, a, st);
    else if (mode == 1) launch_cols_t<N, 1, false>(outer, a, st);
    else if (a.y == nullptr) launch_cols_t<N, 2, false>(outer, a, st);
    else launch_cols_t<N, 3, false>(outer, a, st);
}
static hipError_t launch_cols(int mode, int N, long long outer, const ColsArgs& a, hipStream_t st) {
    switch (N) {
#define X(NN) case NN: launch_cols_n<NN>(mode, outer, a, st); break;
        GLEAM_FFT_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// The transforms are orthonormal, N^-1/2 per axis.  A sweep that only stores its values for the next one scales them by the power of
// two nearest to that, which rounds nothing; what is missing is made up for where the values are multiplied anyway, ahead of
// the mask and in the coil sum.
static float axis_scale(long long n) { return (float)exp2(rint(-0.5 * log2((double)n))); }

static hipError_t sense_sweeps(const gleam_geom& g, const float2* x, const float2* S, const unsigned char* M, const float2* y, float xs,
                               float gs, float2* out, float2* kbuf, const CgFusion& cg, hipStream_t st) {
    const long long DH = g.D * g.H;
    RowsCgArgs ra{};
    ra.cg_job = cg;
    ra.x = x; ra.S = S; ra.k = kbuf; ra.out = out;
    ra.C = (unsigned)g.C; ra.T = (unsigned)g.T; ra.DH = DH;
    const double ortho = 1.0 / sqrt((double)(g.W * (g.ndim_fft >= 2 ? g.H : 1) * (g.ndim_fft >= 3 ? g.D : 1)));
    ra.scale = g.ndim_fft == 1 ? (float)ortho : axis_scale(g.W);
    ra.xs = xs; ra.gs = gs;
    ra.cen = g.centred ? 1 : 0; ra.par_h = g.ndim_fft >= 2; ra.par_d = g.ndim_fft >= 3; ra.Hh = (unsigned)g.H;
    {
        long long half = g.W / 2 + (g.ndim_fft >= 2 ? g.H / 2 : 0) + (g.ndim_fft >= 3 ? g.D / 2 : 0);
        ra.ysign_bit = (int)(half & 1);
    }
    const double E8 = 8.0 * (double)(g.B * g.C * g.T * g.D * g.H * g.W);   // bytes of one k-space sweep
    const double P8 = 8.0 * (double)(g.B * g.T * g.D * g.H * g.W);          // bytes of one image
    const double S8 = E8 / (double)g.T, M1 = P8 / 8.0;
    hipError_t e;
    if (g.ndim_fft == 1) {   // one transformed axis: the whole operator in one sweep, no k-space buffer
        if (fused_staged(g, y != nullptr)) return sense_dc_staged(g, x, S, M, y, xs, gs, out, kbuf, st);
        KernelScope ks("sense_rows_fused", 0.0, S8 + P8 + (y ? E8 : 0.0) + M1 + P8 + (xs != 0.f ? P8 : 0.0), st);
        return launch_rows_fused(g, ra, y, M, st);
    }
    {
        KernelScope ks("sense_rows_expand", 0.0, S8 + P8 + E8, st);
        e = launch_rows(g, false, ra, st);
    }
    if (e != hipSuccess) return e;

    ColsArgs ca{};
    ca.k = kbuf; ca.y = y; ca.M = M; ca.C = (unsigned)g.C;
    ca.cen_y = (g.centred && y) ? 1 : 0; ca.ysign_bit = ra.ysign_bit; ca.cen_io = 0; ca.Wrow = (unsigned)g.W;
    if (g.ndim_fft == 2) {
        ca.inner = (unsigned)g.W; ca.TD = (unsigned)(g.T * g.D);
        ca.scale = axis_scale(g.H);
        ca.fwd = (float)(ortho / axis_scale(g.W));
        ra.scale = (float)(ortho / axis_scale(g.H));
        {
            KernelScope ks("sense_cols_mid", 0.0, 2.0 * E8 + (y ? E8 : 0.0) + M1, st);
            e = launch_cols(2, (int)g.H, g.B * g.C * g.T * g.D, ca, st);
        }
        if (e != hipSuccess) return e;
    } else {
        ColsArgs ha = ca;  // H axis: [B*C*T*D][H][W]
        ha.cen_y = 0;
        ha.rev = 1;
        ha.inner = (unsigned)g.W; ha.TD = (unsigned)(g.T * g.D);
        ha.scale = axis_scale(g.H);
        {
            KernelScope ks("sense_cols_fwd", 0.0, 2.0 * E8, st);
            e = launch_cols(0, (int)g.H, g.B * g.C * g.T * g.D, ha, st);
        }
        if (e != hipSuccess) return e;
        ca.inner = (unsigned)(g.H * g.W); ca.TD = (unsigned)g.T;  // D axis: [B*C*T][D][H*W]
        ca.scale = axis_scale(g.D);
        ca.fwd = (float)(ortho / axis_scale(g.W) / axis_scale(g.H));
        ra.scale = (float)(ortho / axis_scale(g.D) / axis_scale(g.H));
        {
            KernelScope ks("sense_cols_mid", 0.0, 2.0 * E8 + (y ? E8 : 0.0) + M1, st);
            e = launch_cols(2, (int)g.D, g.B * g.C * g.T, ca, st);
        }
        if (e != hipSuccess) return e;
        {
            KernelScope ks("sense_cols_inv", 0.0, 2.0 * E8, st);
            e = launch_cols(1, (int)g.H, g.B * g.C * g.T * g.D, ha, st);
        }
        if (e != hipSuccess) return e;
    }
    KernelScope ks("sense_rows_reduce", 0.0, E8 + S8 + P8 + (xs != 0.f ? P8 : 0.0), st);
    return launch_rows(g, true, ra, st);
}

hipError_t sense_dc(const gleam_geom& g, const float2* x, const float2* S, const unsigned char* M,
                    const float2* y, float xs, float gs, float2* out, float2* kbuf, hipStream_t st) {
    return sense_sweeps(g, x, S, M, y, xs, gs, out, kbuf, CgFusion{}, st);
}

hipError_t sense_cg(const gleam_geom& g, const float2* x, const float2* S, const unsigned char* M, float xs, float gs, float2* out,
                    float2* kbuf, const CgFusion& f, hipStream_t st) {
    return sense_sweeps(g, x, S, M, nullptr, xs, gs, out, kbuf, f, st);
}

int cg_fused_dot_partials(const gleam_geom& g, int max_partials) {
    const long long per = reduce_rows_of(g), n = g.T * ((g.D * g.H + per - 1) / per);
    return g.ndim_fft == 1 || n > max_partials ? 0 : (int)n;
}

bool cg_fused_update(const gleam_geom& g) { return g.ndim_fft > 1 && g.C <= rows_lines_of(g); }

// Measured k-space to hybrid space: the inverse transform (centred when the geometry says so) along the outermost
// transformed axis, in place: H for two transformed axes, D for three.
hipError_t kspace_to_hybrid(const gleam_geom& g, float2* y, hipStream_t st) {
    ColsArgs ca{};
    ca.k = y; ca.C = (unsigned)g.C; ca.Wrow = (unsigned)g.W;
    ca.cen_io = g.centred ? 1 : 0;
    int n;
    long long outer;
    if (g.ndim_fft == 2) {
        outer = g.B * g.C * g.T * g.D; ca.inner = (unsigned)g.W; ca.TD = (unsigned)(g.T * g.D); n = (int)g.H;
    } else {
        outer = g.B * g.C * g.T; ca.inner = (unsigned)(g.H * g.W); ca.TD = (unsigned)g.T; n = (int)g.D;
    }
    ca.scale = 1.0f / sqrtf((float)n);
    const double E8 = 8.0 * (double)(g.B * g.C * g.T * g.D * g.H * g.W);
    KernelScope ks("kspace_to_hybrid", 0.0, 2.0 * E8, st);
    return launch_cols(1, n, outer, ca, st);
}

}  // namespace gleam
