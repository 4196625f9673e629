// Direct float32 convolution with two output channels: the last layer of a network whose other kernels do not take its channel
// count (they want multiples of 16), and the gradient with respect to its input image.
//
// The kernel of prox.hip multiplies 32 output channels for two.  Here a lane is a pixel and holds both sums, chains of fused
// multiply-adds in the order in which that kernel's matrix instructions add their products (row tap, chunk of 8 or 16 input
// channels, tap along W, group of 8 channels, then channels e and 4 + e of the group in turn): the results are the same bits,
// which is what lets the greedy iteration have it.  A wave stages the 64 + 2 pixels x 16 channels of a row tap in LDS of its own
// (80 bytes a pixel: sixteen lanes read sixteen different 16-byte slots), fetched into registers while the chunk before is
// multiplied; no barriers.  A tap outside the image reads a pixel of zeros instead.  The weights are wave-uniform scalar loads, laid
// out in the order of their use (weights.hip).
//
// 100 -> 2 channels at 4 x 320 x 256: 119 us, 191 by the kernel of prox.hip.  What bounds it is waiting, for LDS and for scalar loads:
// the 131 MB it reads take 25 us, its multiply-adds 15.
#include "prox_common.h"
#include "xcd.h"

namespace gleam {

namespace {
constexpr int kStride = 20;     // floats per staged pixel: 16 channels and 4 of padding
constexpr int kPixels = 64;     // per wave
}  // namespace

template <int CK, int KW>
__global__ __launch_bounds__(256) void conv_pair_kernel(ConvArgs a, const float* __restrict__ wts) {
    constexpr int Q4 = CK / 4, G = CK / 8, NPX = kPixels + KW - 1, LOADS = (NPX * Q4 + 63) / 64;
    __shared__ __attribute__((aligned(16))) float slab_all[4][(NPX + 1) * kStride];   // and a pixel of zeros
    const PixDims d = a.d;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float* const slab = slab_all[wave];
    const int n_kc = (a.K + CK - 1) / CK, n_ck = d.kt * d.kd * d.kh * n_kc;
    const XcdRange xr = xcd_range((d.Q + 4 * kPixels - 1) / (4 * kPixels));
    long long tile = xr.first;
    if (tile >= xr.end) return;
    if (lane < kStride / 4) *reinterpret_cast<float4*>(slab + NPX * kStride + 4 * lane) = make_float4(0.f, 0.f, 0.f, 0.f);
    const int floor = a.relu_in ? 0 : (int)0x80000000;   // ReLU on the bit patterns
    float bias[2] = {0.f, 0.f};
    if (a.bias) { bias[0] = a.bias[0]; bias[1] = a.bias[1]; }

    // quad v of a staged chunk: pixel v / Q4, channel quad v % Q4.
    long long f_tile = tile;
    ChunkIter f_ci = chunk_first(d);   // of the next chunk to fetch
    auto fetch = [&](float4* r) {
        if (f_tile >= xr.end) return;
        const long long first = f_tile * (4 * kPixels) + wave * kPixels + f_ci.off - KW / 2;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int v = lane + 64 * i, c = f_ci.kc * CK + 4 * (v % Q4);
            long long q = first + v / Q4;
            q = q < 0 ? 0 : q < d.Q ? q : d.Q - 1;   // such pixels meet taps outside the image, or no output
            r[i] = v < NPX * Q4 && c < a.K ? *reinterpret_cast<const float4*>(a.in + q * a.K + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        f_tile = f_ci.c + 1 == n_ck ? f_tile + xr.stride : f_tile;
        f_ci = chunk_next(f_ci, n_kc, n_ck, d);
    };
    auto relu = [&](float x) { return __int_as_float(__float_as_int(x) > floor ? __float_as_int(x) : floor); };

    long long q = tile * (4 * kPixels) + wave * kPixels + lane;
    PixCoord qc = pix_coord(q < d.Q ? q : 0, d);
    const PixCoord qstep = pix_coord(xr.stride * (4 * kPixels), d);
    ChunkIter ci = chunk_first(d);
    float4 r[LOADS];
    fetch(r);
    unsigned valid = 0u;
    float acc[2] = {0.f, 0.f};
    while (true) {
        if (ci.c == 0) {
            valid = q < d.Q ? tap_validity_at(qc, d) : 0u;
            acc[0] = acc[1] = 0.f;
        }
        // (LDS operations of a wave are executed in order)
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int v = lane + 64 * i;
            if (v < NPX * Q4)
                *reinterpret_cast<float4*>(slab + (v / Q4) * kStride + 4 * (v % Q4)) = make_float4(relu(r[i].x), relu(r[i].y), relu(r[i].z), relu(r[i].w));
        }
        __builtin_amdgcn_wave_barrier();
        fetch(r);
        const float* w = wts + (size_t)(ci.rt * n_kc + ci.kc) * (KW * CK * 2);
        const int groups = (a.K - ci.kc * CK + 7) / 8;   // that hold channels, of G
#pragma unroll
        for (int dw = 0; dw < KW; ++dw) {
            const float* x = slab + ((valid >> (ci.rt * KW + dw)) & 1u ? lane + dw : NPX) * kStride;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (G > 1 && g >= groups) break;   // uniform
                const float4 lo = *reinterpret_cast<const float4*>(x + 8 * g), hi = *reinterpret_cast<const float4*>(x + 8 * g + 4);
                const float xl[4] = {lo.x, lo.y, lo.z, lo.w}, xh[4] = {hi.x, hi.y, hi.z, hi.w};
                const float* wg = w + (dw * G + g) * 16;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[0] = fmaf(xl[e], wg[4 * e], acc[0]);
                    acc[1] = fmaf(xl[e], wg[4 * e + 1], acc[1]);
                    acc[0] = fmaf(xh[e], wg[4 * e + 2], acc[0]);
                    acc[1] = fmaf(xh[e], wg[4 * e + 3], acc[1]);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (ci.c + 1 == n_ck) {
            if (q < d.Q) {
                float2 o = make_float2(acc[0] + bias[0], acc[1] + bias[1]);
                if (a.relu_out) o = make_float2(fmaxf(o.x, 0.f), fmaxf(o.y, 0.f));
                if (a.add) {
                    const float2 s = reinterpret_cast<const float2*>(a.add)[q];
                    o.x += s.x;
                    o.y += s.y;
                }
                reinterpret_cast<float2*>(a.out)[q] = o;
            }
            pix_advance(qc, qstep, d);
            tile += xr.stride;
            if (tile >= xr.end) break;
            q += xr.stride * (4 * kPixels);
        }
        ci = chunk_next(ci, n_kc, n_ck, d);
    }
}

// The line, in pixels: up to 32768 the direct kernel's workgroups of 128 have a CU each, its unused output channels cost nothing and
// its waits are shorter (a training step with one hidden pair of layers, us with this kernel / without: 100 channels, 20480 pixels
// 331.9/320.1, 40960 497.5/499.1, 65536 578.2/580.2, 92160 726/742, 122880 925/960; 12 channels 111.1/109.3, 133.5/135.2,
// 142.6/144.6, 154.3/158.2, 164.3/170.8).
constexpr long long kPairPixels = 32768;
bool conv_pair_applies(const PixDims& d, int K, int Nn) { return Nn == 2 && d.Q > kPairPixels && K >= 8 && K % 4 == 0 && (d.kw == 1 || d.kw == 3); }

size_t conv_pair_weight_floats(int K, int taps) { return (size_t)taps * (K <= 8 ? 8 : (K + 15) / 16 * 16) * 2; }

hipError_t launch_conv_pair(const ConvArgs& a, hipStream_t st) {
    const long long n_tiles = (a.d.Q + 4 * kPixels - 1) / (4 * kPixels), cap = 1536;   // six workgroups per CU
    const dim3 grid((unsigned)(((n_tiles < cap ? n_tiles : cap) + 7) / 8 * 8));       // XCD-aware split needs a multiple of 8
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, a, a.wt); };
    if (a.K <= 8) {
        if (a.d.kw == 3) go(conv_pair_kernel<8, 3>);
        else go(conv_pair_kernel<8, 1>);
    } else {
        if (a.d.kw == 3) go(conv_pair_kernel<16, 3>);
        else go(conv_pair_kernel<16, 1>);
    }
    return hipGetLastError();
}

}  // namespace gleam
