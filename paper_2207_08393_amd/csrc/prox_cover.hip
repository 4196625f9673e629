// Direct float32 convolution, three taps along W, all output channels in one workgroup (gfx950).
//
// The kernel of prox.hip deals the output channels in blocks of 64 and multiplies what is left of the last one by zeros: 100
// channels cost 128.  Here a wave has floor(N / 32) tiles of 32 channels x 32 pixels for each of its two blocks of 32 pixels
// (v_mfma_f32_32x32x2_f32) and the remaining channels in fours, 64 pixels at a time (v_mfma_f32_4x4x1_f32, sixteen blocks that
// share one set of four channels; the same 64 multiply-adds a cycle).  Both instructions add their products one by one, each
// with a fused multiply-add, in the order of k (compared bit for bit with a chain of fmaf over 512 terms), and the order of the
// k is that of prox.hip: the results are the same bits.
#include <hip/hip_runtime.h>

#include <climits>
#include <utility>

#include "prox_common.h"
#include "xcd.h"

namespace gleam {

typedef float floatx4q __attribute__((ext_vector_type(4)));

// acc += w(4 channels of quad Q, k) * x(pixel = lane, k); lane 4 * Q + i of w holds channel i
template <int Q>
__device__ __forceinline__ floatx4q mfma_quad(float w, float x, floatx4q acc) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(w, x, acc, 4, Q, 0);
}

template <int... Q>
__device__ __forceinline__ void mfma_quads(float w, float x, floatx4q* acc, std::integer_sequence<int, Q...>) {
    ((acc[Q] = mfma_quad<Q>(w, x, acc[Q])), ...);
}

// What bounds it: the fp32 matrix cores and 1280 blocks on 512 workgroups.  100 -> 100 channels, 3x3, 4 x 320 x 256: 703 -> 565 us,
// 104 TFLOP/s (108 issued of 157; prox.hip issued 112 for 84); a greedy iteration of eight modules 81.4 -> 72.3 ms.
// Blocks of 256 pixels, chunks of one row tap x 16 input channels in two LDS buffers filled by direct loads, as in prox.hip
// (layouts and swizzle are described there).  With two blocks of 32 pixels per wave a weight operand read from LDS serves two
// matrix instructions and a pixel operand NJ of them.  The pixel operands of the fours are those of the tiles, exchanged between
// the halves of a wave (v_permlane32_swap): lane = pixel, both quads of k.
// HALF: the last chunk holds at most eight channels, the rest of it is zero weights and is not multiplied.  (A copy of the loop
// for it, as in prox.hip, spilled 300 registers.)
template <int NB, bool HALF>
__global__ __launch_bounds__(256, 2) void conv_cover_kernel(ConvArgs a) {
    constexpr int NW = 4, PJ = 2, CK = 16, KW = 3;
    constexpr int TM = NW * 32 * PJ, G = CK / 8, NJ = NB / 32, NQ = NB % 32 / 4, Q4 = CK / 4, RP = 16 / Q4;
    constexpr int kSlab = ((TM + KW - 1) * Q4 + 63) / 64, kW4 = KW * CK * NB / 4, kWOps = (kW4 + 63) / 64;   // loads of 64 lanes
    constexpr int MAXS = (kSlab + NW - 1) / NW, MAXW = (kWOps + NW - 1) / NW;
    // two LDS objects, so that reads of one need not wait for the direct loads into the other
    __shared__ float bufA[(kSlab + kWOps) * 256];
    __shared__ float bufB[(kSlab + kWOps) * 256];
    const PixDims d = a.d;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 31, h = lane >> 5;
    const int n_kc = (a.K + CK - 1) / CK;
    const int floor = a.relu_in ? 0 : INT_MIN;   // the smallest bit pattern an operand keeps: ReLU as an integer maximum
    const int nck = d.kt * d.kd * d.kh * n_kc;
    const long long n_tiles = (d.Q + TM - 1) / TM;
    const long long last_quad = d.Q * a.K - 4;            // highest legal quad start
    // last first pixel of a slab of which no quad of any chunk starts outside the tensor
    const long long last_start = d.Q - (n_kc * CK + a.K - 1) / a.K - kSlab * 64 / Q4 + 1;

    // quad v of a slab: pixel v / Q4, channel quad v % Q4 ^ key(pixel); 64 quads and so the key advance by whole periods
    static_assert(64 / Q4 % (RP * Q4) == 0, "the key of a lane is the same for all of its quads");
    const int s_pp = lane / Q4, s_c4 = (lane % Q4) ^ ((s_pp / RP) % Q4);
    const unsigned s_off = (unsigned)(s_pp * a.K + 4 * s_c4);

    auto issue = [&](long long tile, const ChunkIter& ci, float* dst) {
        const long long qs = tile * TM + ci.off - KW / 2;
        if (qs >= 0 && qs <= last_start) {   // uniform
            const float* base = a.in + qs * a.K + ci.kc * CK;
#pragma unroll
            for (int i = 0; i < MAXS; ++i) {
                const int o = wave + i * NW;
                if (o < kSlab)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + o * (64 / Q4) * a.K + s_off),
                                                     (__attribute__((address_space(3))) void*)(dst + o * 256), 16, 0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < MAXS; ++i) {
                const int o = wave + i * NW;
                if (o < kSlab) {
                    long long off = (qs + o * (64 / Q4) + s_pp) * a.K + ci.kc * CK + 4 * s_c4;
                    off = off < 0 ? 0 : (off > last_quad ? last_quad : off);
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a.in + off),
                                                     (__attribute__((address_space(3))) void*)(dst + o * 256), 16, 0, 0);
                }
            }
        }
        const float* src = a.wt + (size_t)(ci.rt * n_kc + ci.kc) * (size_t)(KW * CK * NB);
        float* wdst = dst + kSlab * 256;
#pragma unroll
        for (int i = 0; i < MAXW; ++i) {
            const int o = wave + i * NW;
            if (o < kWOps) {
                const int v = o * 64 + lane;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + 4 * (v < kW4 ? v : 0)),
                                                 (__attribute__((address_space(3))) void*)(wdst + o * 256), 16, 0, 0);
            }
        }
    };

    // LDS float offsets of this lane's pixel operand per (tap along W, 8-channel group); the second block of 32 pixels has the
    // same key, so it lies 32 * CK further
    int p_off[KW][G];
#pragma unroll
    for (int dw = 0; dw < KW; ++dw) {
        const int pix = wave * (32 * PJ) + m + dw;
#pragma unroll
        for (int g = 0; g < G; ++g) p_off[dw][g] = pix * CK + 4 * ((2 * g + h) ^ ((pix / RP) % Q4));
    }
    const int wa_lane = (h * NB + m) * 4;
    const int wq_lane = (32 * NJ + (lane < 4 * NQ ? lane : 0)) * 4;   // weights of the fours: lane = channel

    const XcdRange xr = xcd_range(n_tiles);
    long long tile = xr.first;
    ChunkIter ci = chunk_first(d);
    if (tile < xr.end) issue(tile, ci, bufA);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    long long q0 = (tile < xr.end ? tile : 0) * TM + wave * (32 * PJ) + m;
    PixCoord qc[PJ];
#pragma unroll
    for (int pj = 0; pj < PJ; ++pj) qc[pj] = pix_coord(q0 + 32 * pj < d.Q ? q0 + 32 * pj : 0, d);
    const PixCoord qstep = pix_coord(xr.stride * TM, d);
    unsigned vbits[PJ];
    floatx16 acc[PJ][NJ];
    floatx4q accq[NQ ? NQ : 1];

    auto finish = [&](float v0, float v1, float v2, float v3, long long q, int co0) {
        float v[4] = {v0, v1, v2, v3};
        const long long o = q * a.Nn + co0;
        if (a.bias) {
            const float4 bv = *reinterpret_cast<const float4*>(a.bias + co0);
            v[0] += bv.x; v[1] += bv.y; v[2] += bv.z; v[3] += bv.w;
        }
        if (a.relu_out) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
        }
        float4 ref = make_float4(1.f, 1.f, 1.f, 1.f);
        if (a.mask_ref) ref = *reinterpret_cast<const float4*>(a.mask_ref + o);
        const float rr[4] = {ref.x, ref.y, ref.z, ref.w};
        if (a.mask_acc) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = rr[i] > 0.f ? v[i] : 0.f;
        }
        if (a.add) {
            float4 av = *reinterpret_cast<const float4*>(a.add + o);
            // (keeps it one load of 16 bytes: the compiler may move the one of .x to where it is needed)
            asm volatile("" : "+v"(av.x), "+v"(av.y), "+v"(av.z), "+v"(av.w));
            const float aa[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += (a.mask_add && !(rr[i] > 0.f)) ? 0.f : aa[i];
        }
        *reinterpret_cast<float4*>(a.out + o) = make_float4(v[0], v[1], v[2], v[3]);
    };

    auto step = [&](const float* slab, float* nxt) {
        if (ci.c == 0) {
#pragma unroll
            for (int pj = 0; pj < PJ; ++pj) {
                vbits[pj] = q0 + 32 * pj < d.Q ? tap_validity_at(qc[pj], d) : 0u;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[pj][j][r] = 0.f;
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) accq[q] = floatx4q{0.f, 0.f, 0.f, 0.f};
        }
        const bool last = ci.c + 1 == nck;
        const long long ntile = last ? tile + xr.stride : tile;
        const ChunkIter nci = chunk_next(ci, n_kc, nck, d);
        if (ntile < xr.end) issue(ntile, nci, nxt);
        const float* wl = slab + kSlab * 256 + wa_lane;
        const float* wq = slab + kSlab * 256 + wq_lane;
        const int rt = ci.rt;
        // unit: one tap along W x 8 input channels; its operands are read before the matrix instructions of the unit before
        float4 pb[G][PJ], wa[G][NJ], qa[G][2];
        auto load_unit = [&](int dw, int g) {
#pragma unroll
            for (int pj = 0; pj < PJ; ++pj) pb[g][pj] = *reinterpret_cast<const float4*>(slab + p_off[dw][g] + 32 * CK * pj);
#pragma unroll
            for (int j = 0; j < NJ; ++j) wa[g][j] = *reinterpret_cast<const float4*>(wl + ((dw * G + g) * 2 * NB + 32 * j) * 4);
            if constexpr (NQ > 0) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    qa[g][e] = *reinterpret_cast<const float4*>(wq + ((dw * G + g) * 2 + e) * NB * 4);
            }
        };
        auto unit = [&](int dw, int g) {
            // ReLU and zero padding on the bit patterns, as in prox.hip
            float x[PJ][4];
#pragma unroll
            for (int pj = 0; pj < PJ; ++pj) {
                const int okm = -(int)((vbits[pj] >> (rt * KW + dw)) & 1u);
                const float f[4] = {pb[g][pj].x, pb[g][pj].y, pb[g][pj].z, pb[g][pj].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int b = __float_as_int(f[e]);
                    b = b > floor ? b : floor;
                    x[pj][e] = __int_as_float(b & okm);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float xq[2] = {0.f, 0.f};
                if constexpr (NQ > 0) {
                    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[0][e]), __float_as_uint(x[1][e]), false, false);
                    xq[0] = __uint_as_float(s[0]);
                    xq[1] = __uint_as_float(s[1]);
                }
#pragma unroll
                for (int pj = 0; pj < PJ; ++pj) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const float4 w = wa[g][j];
                        acc[pj][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(e == 0 ? w.x : e == 1 ? w.y : e == 2 ? w.z : w.w, x[pj][e],
                                                                          acc[pj][j], 0, 0, 0);
                    }
                    if constexpr (NQ > 0) {   // the products of quad pj of k
                        const float4 w4 = qa[g][pj];
                        const float w = e == 0 ? w4.x : e == 1 ? w4.y : e == 2 ? w4.z : w4.w;
                        mfma_quads(w, xq[pj], accq, std::make_integer_sequence<int, NQ>{});
                    }
                }
            }
        };
        const bool half = HALF && ci.kc == n_kc - 1;   // uniform
        load_unit(0, 0);
#pragma unroll
        for (int dw = 0; dw < KW; ++dw) {
            load_unit(dw, 1);
            unit(dw, 0);
            if (dw + 1 < KW) load_unit(dw + 1, 0);
            if (!half) unit(dw, 1);
        }
        if (last) {
#pragma unroll
            for (int pj = 0; pj < PJ; ++pj) {
                const long long q = q0 + 32 * pj;
                if (q >= d.Q) continue;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg)
                        finish(acc[pj][j][4 * rg], acc[pj][j][4 * rg + 1], acc[pj][j][4 * rg + 2], acc[pj][j][4 * rg + 3], q,
                               32 * j + 8 * rg + 4 * h);
            }
            const long long q = q0 + 32 * h;   // lane = pixel
#pragma unroll
            for (int i = 0; i < NQ; ++i)
                if (q < d.Q) finish(accq[i][0], accq[i][1], accq[i][2], accq[i][3], q, 32 * NJ + 4 * i);
        }
        __builtin_amdgcn_s_waitcnt(0);   // the next chunk's direct loads have landed in LDS
        __syncthreads();                 // ... and every wave is done reading the current buffer
        if (last) {
            q0 += xr.stride * TM;
#pragma unroll
            for (int pj = 0; pj < PJ; ++pj) pix_advance(qc[pj], qstep, d);
        }
        tile = ntile;
        ci = nci;
    };
    while (tile < xr.end) {
        step(bufA, bufB);
        if (tile >= xr.end) break;
        step(bufB, bufA);
    }
}

template <int NB>
static void launch_cover(const ConvArgs& a, hipStream_t st) {
    constexpr size_t lds = (size_t)2 * ((258 * 4 + 63) / 64 + (3 * 16 * NB / 4 + 63) / 64) * 1024;   // static in the kernel
    static_assert(lds <= 80 * 1024, "two workgroups on a CU");
    const long long n_tiles = (a.d.Q + 255) / 256, cap = 512;
    const dim3 grid((unsigned)(((n_tiles < cap ? n_tiles : cap) + 7) / 8 * 8));   // XCD-aware split needs a multiple of 8
    const bool half = a.K % 16 != 0 && a.K % 16 <= 8;
    if (half) hipLaunchKernelGGL((conv_cover_kernel<NB, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((conv_cover_kernel<NB, false>), grid, dim3(256), 0, st, a);
}

int conv_cover_channels(const PixDims& d, int K, int Nn) {
    if (d.kw != 3 || K % 4 != 0 || K <= 8 || Nn % 4 != 0 || Nn <= 32) return 0;
    // 64 channels fit the blocks of prox.hip; with more than two fours a unit has more of the short instructions than it gains
    // (48 channels: a greedy iteration of two modules 2 % faster to 3 % slower at 131072 to 327680 pixels)
    if (Nn == 64 || Nn % 32 > 8 || Nn > 104) return 0;
    // A block of 256 pixels for two workgroups on every CU.  The same call, us, prox.hip / here: 98304 pixels: 36 channels
    // 1109 / 1088, 96 2773 / 2735, 100 3239 / 3323; 81920: 96 2424 / 2602, 100 2830 / 3154; 131072: 36 1369 / 1226,
    // 96 3526 / 3057, 100 4159 / 3750; 327680: 2810 / 2489, 8250 / 7007, 9748 / 8604.
    if (d.Q < 256LL * 512) return 0;
    return Nn;
}

hipError_t launch_conv_cover(const ConvArgs& a, hipStream_t st) {
    switch (a.Nn) {
        case 36: launch_cover<36>(a, st); break;
        case 40: launch_cover<40>(a, st); break;
        case 68: launch_cover<68>(a, st); break;
        case 72: launch_cover<72>(a, st); break;
        case 96: launch_cover<96>(a, st); break;
        case 100: launch_cover<100>(a, st); break;
        case 104: launch_cover<104>(a, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace gleam
