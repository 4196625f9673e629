// Weight gradient of a float32 layer of nine taps (three along the rows) with 68 to 124 output and 68 to 100 input channels.
//
// The gradient is a matrix of Co rows and 9 * Ci columns.  Two workgroups of eight waves share it: a wave takes the F = Co / 32 whole
// blocks of 32 rows in 6 / F blocks of 32 columns, across the borders of the taps, and so reads F + 6 / F operands for six matrix
// instructions; what is left of rows and columns goes by 4 x 4 blocks, sixteen to a v_mfma_f32_4x4x1_f32 (as many multiply-adds a
// cycle), kQuads of those to a wave.  100 -> 100 channels: 84 blocks in 14 waves and 249 small ones in two.
//
// A chunk is a segment of 32 pixels of an image row, staged as float4; pixels past the end of the row get g = 0, and taps outside the
// image are stored as 0, so the matrix instructions need no masks.  Two chunks lie in LDS: while one is multiplied the next is
// fetched, slot by slot in the first half of the multiplications, and stored in the second, between one barrier and the next.  Rows
// of fixed length make every LDS address a register and a constant, and the operands of a step are read during the one before.
// 100 -> 100 channels at 4 x 320 x 256: 536 us, 110 TFLOP/s; 750 us with one chunk in LDS between two barriers, operands read
// where they were needed (the compiler had moved the reads back) and the LDS addresses of every step computed.  What bounds it: the
// matrix cores, 0.70 of the time.
//
// Both instructions add their products with fused multiply-adds in the order of the pixels: the sums are the same bits as
// those of wgrad_pipe_kernel with as many workgroups.
#include "prox_common.h"
#include "xcd.h"

namespace gleam {

namespace {
constexpr int kUnits = 6, kQuads = 8;       // matrix instructions per wave and step
constexpr int kPx = 32;                     // pixels per chunk
constexpr int kRowG = 132, kRowA = 104;     // floats per staged pixel: at most 124 and 100 channels, and four of padding
constexpr int kSlabG = kPx * kRowG, kSlab = kSlabG + 3 * (kPx + 2) * kRowA;
constexpr int kSlotsG = 2, kSlotsA = 5;     // float4 per thread and chunk
typedef float floatx4 __attribute__((ext_vector_type(4)));
struct CoverSplit {
    int F, ncol, quads;   // blocks of 32 rows, columns, blocks of 4 x 4
    __host__ __device__ CoverSplit(int Co, int ncol_)
        : F(Co / 32), ncol(ncol_), quads(Co % 32 / 4 * (ncol_ / 4) + Co / 32 * 8 * (ncol_ % 32 / 4)) {}
    __host__ __device__ int unit_waves() const { return (ncol / 32 + kUnits / F - 1) / (kUnits / F); }
    __host__ __device__ int waves() const { return unit_waves() + (quads + 16 * kQuads - 1) / (16 * kQuads); }
};
}  // namespace

template <int F>
__global__ __launch_bounds__(512) void wgrad_cover_kernel(WgradArgs a, float* bias_partial) {
    constexpr int CU = kUnits / F;
    extern __shared__ __attribute__((aligned(16))) float smem[];   // [2][kSlab]
    const PixDims d = a.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 31, h = lane >> 5;
    const int Co4 = a.Co / 4, Ci4 = a.Ci / 4, n_g4 = kPx * Co4;
    const int ncol = 9 * a.Ci;
    const CoverSplit cover(a.Co, ncol);
    const int job = wave * 2 + blockIdx.y;
    const bool units = job < cover.unit_waves(), quads = !units && job < cover.waves();

    // The float4 slots of this thread, the same for every chunk: where they lie in LDS (what there are no slots for goes to the
    // padding of row tid % 32), their pixel, their offset from the chunk's first pixel.  Bits 8.. of an input slot's pixel: row tap,
    // 3: no slot.
    const int spare = (tid & 31) * kRowG + 128;
    const int row_stride = (d.kt == 3 ? d.D * d.H : d.kd == 3 ? d.H : 1) * d.W;
    int g_lds[kSlotsG], g_px[kSlotsG], g_off[kSlotsG], a_lds[kSlotsA], a_px[kSlotsA], a_off[kSlotsA];
#pragma unroll
    for (int i = 0; i < kSlotsG; ++i) {
        const int v = tid + i * 512, p = v / Co4, c = 4 * (v % Co4);
        const bool is = v < n_g4;
        g_lds[i] = is ? p * kRowG + c : spare;
        g_px[i] = is ? p : 1 << 30;
        g_off[i] = p * a.Co + c;
    }
#pragma unroll
    for (int i = 0; i < kSlotsA; ++i) {
        const int v = tid + i * 512, rt = v / ((kPx + 2) * Ci4), r = v % ((kPx + 2) * Ci4), p = r / Ci4, c = 4 * (r % Ci4);
        const bool is = rt < 3;
        a_lds[i] = is ? kSlabG + (rt * (kPx + 2) + p) * kRowA + c : spare;
        a_px[i] = (is ? rt : 3) << 8 | p;
        a_off[i] = is ? ((rt - 1) * row_stride + p - 1) * a.Ci + c : 0;
    }
    float4 rg[kSlotsG], ra[kSlotsA], bsum[kSlotsG];
#pragma unroll
    for (int i = 0; i < kSlotsG; ++i) bsum[i] = make_float4(0.f, 0.f, 0.f, 0.f);

    const int segs = (d.W + kPx - 1) / kPx;
    const XcdRange xr = xcd_range((d.Q / d.W) * segs);
    PixDims cd = d;
    cd.W = segs;
    // (there are fewer than 2^31 chunks: 64 channels of as many pixels have no room)
    auto coord = [&](int q) {
        PixCoord c;
        c.w = q % segs;
        q /= segs;
        c.h = q % d.H;
        q /= d.H;
        c.dd = q % d.D;
        c.t = q / d.D % d.T;
        return c;
    };
    PixCoord cc = coord((int)xr.first);   // segment, row, slice, frame of the chunk to fetch
    const PixCoord cstep = coord((int)xr.stride);
    int crow = (int)xr.first / segs;      // its image row
    const int rstep = (int)xr.stride / segs;
    const float *gbase = a.g, *abase = a.a;
    int w0 = 0, w_end = 0;
    unsigned rows_ok = 0u, ok = 0u;
    // `is` false: there is no such chunk, and zeros are stored
    auto next = [&](bool is) {
        rows_ok = 0u;
        if (is) {
            const int at = d.kt == 3 ? cc.t : d.kd == 3 ? cc.dd : cc.h, n = d.kt == 3 ? d.T : d.kd == 3 ? d.D : d.H;
            rows_ok = (at > 0 ? 1u : 0u) | 2u | (at + 1 < n ? 4u : 0u);
            w0 = cc.w * kPx;
            const long long q0 = (long long)crow * d.W + w0;
            gbase = a.g + q0 * a.Co;
            abase = a.a + q0 * a.Ci;
            crow += rstep + (cc.w + cstep.w >= segs ? 1 : 0);
            pix_advance(cc, cstep, cd);
        }
        w_end = is ? d.W : 0;
        ok = 0u;
    };
    // Loads are unconditional (what is outside reads the chunk's first pixel); masks and ReLU, on the bit patterns, at the store.
    auto fetch = [&](int i) {
        if (i < kSlotsG) {
            const bool in = w0 + g_px[i] < w_end;
            rg[i] = *reinterpret_cast<const float4*>(gbase + (in ? g_off[i] : 0));
            ok |= (in ? 1u : 0u) << i;
        } else if (i < kSlotsG + kSlotsA) {
            const int j = i - kSlotsG;
            const bool in = ((rows_ok >> (a_px[j] >> 8)) & 1u) != 0u && (unsigned)(w0 + (a_px[j] & 255) - 1) < (unsigned)w_end;
            ra[j] = *reinterpret_cast<const float4*>(abase + (in ? a_off[j] : 0));
            ok |= (in ? 1u : 0u) << i;
        }
    };
    const int floor = a.relu_in ? 0 : (int)0x80000000;
    auto stash = [&](float* buf, int i) {
        if (i < 0 || i >= kSlotsG + kSlotsA) return;
        const int mk = -(int)((ok >> i) & 1u);
        auto part = [&](float x) {
            int b = __float_as_int(x);
            if (i >= kSlotsG) b = b > floor ? b : floor;
            return __int_as_float(b & mk);
        };
        const float4 r = i < kSlotsG ? rg[i] : ra[i - kSlotsG];
        const float4 v = make_float4(part(r.x), part(r.y), part(r.z), part(r.w));
        *reinterpret_cast<float4*>(buf + (i < kSlotsG ? g_lds[i] : a_lds[i - kSlotsG])) = v;
        if (i < kSlotsG) {
            bsum[i].x += v.x; bsum[i].y += v.y; bsum[i].z += v.z; bsum[i].w += v.w;
        }
    };

    // Every role of a wave walks the chunks with the same barriers: step(buf, other, s), s < 16, multiplies pixels 2s and 2s + 1.
    auto walk = [&](auto&& begin, auto&& step) {
        if (xr.first < xr.end) {
            next(true);
#pragma unroll
            for (int i = 0; i < kSlotsG + kSlotsA; ++i) fetch(i);
#pragma unroll
            for (int i = 0; i < kSlotsG + kSlotsA; ++i) stash(smem, i);
        }
        __syncthreads();
        int at = 0;
        next(xr.first + xr.stride < xr.end);
        for (long long chunk = xr.first; chunk < xr.end; chunk += xr.stride) {
            float* const buf = smem + at;
            at = kSlab - at;
            float* const other = smem + at;
            begin(buf);
#pragma unroll
            for (int s = 0; s < kPx / 2; ++s) {
                step(buf, s);
                if (s < kSlotsG + kSlotsA) fetch(s);
                stash(other, s - kPx / 4);
            }
            next(chunk + 2 * xr.stride < xr.end);   // (under the last matrix instructions)
            __syncthreads();
        }
    };
    auto column = [&](int n) {   // LDS offset of a column, at pixel 0
        const int tap = n / a.Ci;
        return kSlabG + (tap / 3 * (kPx + 2) + tap % 3) * kRowA + n % a.Ci;
    };
    auto quad_block = [&](int j, int& row, int& col) {   // first row and column; false: there is none
        const int t = ((job - cover.unit_waves()) * kQuads + j) * 16 + (lane >> 2);
        const int n_rows = a.Co % 32 / 4 * (ncol / 4), rem = ncol % 32 / 4;
        row = col = 0;
        if (!quads || t >= cover.quads) return false;
        row = t < n_rows ? a.Co / 32 * 32 + t / (ncol / 4) * 4 : (t - n_rows) / rem * 4;
        col = t < n_rows ? t % (ncol / 4) * 4 : ncol / 32 * 32 + (t - n_rows) % rem * 4;
        return true;
    };
    float* const dst = a.partial + (size_t)blockIdx.x * a.Co * ncol;
    if (units) {
        floatx16 acc[CU][F];
#pragma unroll
        for (int j = 0; j < CU; ++j)
#pragma unroll
            for (int r = 0; r < F; ++r)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[j][r][e] = 0.f;
        int at_c[CU];
#pragma unroll
        for (int j = 0; j < CU; ++j) {
            const int c = job * CU + j;
            at_c[j] = column((c < ncol / 32 ? c * 32 : 0) + m) + h * kRowA;
        }
        float av[2][F], bv[2][CU];
        auto read = [&](const float* buf, int s) {
#pragma unroll
            for (int r = 0; r < F; ++r) av[s & 1][r] = buf[h * kRowG + m + 2 * s * kRowG + 32 * r];
#pragma unroll
            for (int j = 0; j < CU; ++j) bv[s & 1][j] = buf[at_c[j] + 2 * s * kRowA];
        };
        walk([&](const float* buf) { read(buf, 0); },
             [&](const float* buf, int s) {
                 if (s + 1 < kPx / 2) read(buf, s + 1);
                 __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                 for (int j = 0; j < CU; ++j)
#pragma unroll
                     for (int r = 0; r < F; ++r) acc[j][r] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s & 1][r], bv[s & 1][j], acc[j][r], 0, 0, 0);
             });
#pragma unroll
        for (int j = 0; j < CU; ++j) {
            const int c = job * CU + j;
            if (c >= ncol / 32) continue;
#pragma unroll
            for (int b = 0; b < F; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) dst[(32 * b + 8 * (r / 4) + 4 * h + r % 4) * ncol + 32 * c + m] = acc[j][b][r];
        }
    } else if (quads) {
        floatx4 acc[kQuads];
        int at_r[kQuads], at_c[kQuads];   // lane 4 * block + row, + column
#pragma unroll
        for (int j = 0; j < kQuads; ++j) {
            acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
            int row, col;
            (void)quad_block(j, row, col);
            at_r[j] = row + (lane & 3);
            at_c[j] = column(col + (lane & 3));
        }
        float av[2][2][kQuads], bv[2][2][kQuads];
        auto read = [&](const float* buf, int s) {
#pragma unroll
            for (int j = 0; j < kQuads; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    av[s & 1][p][j] = buf[at_r[j] + (2 * s + p) * kRowG];
                    bv[s & 1][p][j] = buf[at_c[j] + (2 * s + p) * kRowA];
                }
        };
        walk([&](const float* buf) { read(buf, 0); },
             [&](const float* buf, int s) {
                 if (s + 1 < kPx / 2) read(buf, s + 1);
                 __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                 for (int p = 0; p < 2; ++p)
#pragma unroll
                     for (int j = 0; j < kQuads; ++j) acc[j] = __builtin_amdgcn_mfma_f32_4x4x1f32(av[s & 1][p][j], bv[s & 1][p][j], acc[j], 0, 0, 0);
             });
#pragma unroll
        for (int j = 0; j < kQuads; ++j) {
            int row, col;
            if (!quad_block(j, row, col)) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[(row + r) * ncol + col + (lane & 3)] = acc[j][r];
        }
    } else {
        walk([](const float*) {}, [](const float*, int) {});   // stages only
    }
    if (bias_partial != nullptr && blockIdx.y == 0) {
        // slot v summed channels 4 * (v % Co4).. over its pixels (every wave is past the last chunk's barrier)
        float4* red = reinterpret_cast<float4*>(smem);
#pragma unroll
        for (int i = 0; i < kSlotsG; ++i) red[tid + i * 512] = bsum[i];
        __syncthreads();
        if (tid < a.Co) {
            const int c4 = tid / 4, e = tid % 4;
            float t = 0.f;
            for (int v = c4; v < n_g4; v += Co4) {
                const float4 x = red[v];
                t += e == 0 ? x.x : (e == 1 ? x.y : (e == 2 ? x.z : x.w));
            }
            bias_partial[(size_t)blockIdx.x * a.Co + tid] = t;
        }
    }
}

// More than eight channel blocks, of which sixteen waves hold the matrix; the slots of a thread hold the channels.
bool wgrad_cover_applies(const PixDims& d, int Co, int Ci) {
    const int blocks = (Co + 31) / 32 * ((Ci + 31) / 32);
    return d.kw == 3 && d.kt * d.kd * d.kh == 3 && Co % 4 == 0 && Ci % 4 == 0 && (Co / 32 == 2 || Co / 32 == 3) && blocks > 8 && blocks <= 16 &&
           CoverSplit(Co, 9 * Ci).waves() <= 16 && Co <= 128 && 3 * (kPx + 2) * (Ci / 4) <= 512 * kSlotsA;
}

// (a function per kernel: each has to be allowed its LDS)
template <int F>
static hipError_t launch_wgrad_cover_t(const WgradArgs& a, float* bias_partial, int n_split, hipStream_t st) {
    constexpr size_t lds = 2 * kSlab * sizeof(float);   // 118656 bytes: a workgroup per CU
    static const hipError_t e = hipFuncSetAttribute((const void*)wgrad_cover_kernel<F>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(wgrad_cover_kernel<F>, dim3(n_split, 2), dim3(512), lds, st, a, bias_partial);
    return hipGetLastError();
}

hipError_t launch_wgrad_cover(const WgradArgs& a, float* bias_partial, int n_split, hipStream_t st) {
    return a.Co / 32 == 2 ? launch_wgrad_cover_t<2>(a, bias_partial, n_split, st) : launch_wgrad_cover_t<3>(a, bias_partial, n_split, st);
}

}  // namespace gleam
