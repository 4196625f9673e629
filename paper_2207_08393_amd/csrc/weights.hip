// The weights of a pass as its kernels read them: re-laid, rounded, split or transformed, every layer in one launch.
//
// What bounds it: the launch.  A dependent launch takes 4.2 - 4.8 us here whatever it does, and the largest of these jobs
// (128 x 128 channels, 3x3) moves 1 MB.  With a launch of its own per layer the eight that a training step of the 128-channel
// bfloat16 chain or of a 100-channel residual network makes were 38 us; the two that are left, one before the forward and one
// before the data-gradient launches, are 10.  Calls of several modules make those of up to sixteen modules at once.  A thread makes
// one element of an image or what one (output, input) channel pair becomes; reads of neighbouring threads are neighbouring where the
// form allows it, and all of it stays in L2.
#include "prox_common.h"

namespace gleam {

namespace {

__device__ __forceinline__ float weight_at(const WeightJob& j, int n, int tap, int k) {
    return j.w[n * j.sn + (j.flip ? j.taps - 1 - tap : tap) * j.st + k * j.sk];
}

// LDS images conv_mfma_kernel<NB, CK>, conv_dlds_kernel and conv_cover_kernel copy verbatim.  Image (rt, kc, nb) holds
// row-tap rt, input-channel chunk kc and output-channel block nb as [kw][CK/8][2][NB][4]: element (dw, k = 8g + 4h + s, n) at
// (((dw*G + g)*2 + h)*NB + n)*4 + s, zero where k or n runs past the layer.
// The bfloat16 images are [kw][CK/16][2][NB][8], with 16g + 8h + s.
template <int Q, typename T> __device__ __forceinline__ T image_element(const WeightJob& j, int i) {
    const int img_elems = j.kw * j.CK * j.NB, n_kc = (j.K + j.CK - 1) / j.CK, n_nb = (j.Nn + j.NB - 1) / j.NB;
    const int img = i / img_elems, e = i % img_elems;
    const int s = e % Q, n = (e / Q) % j.NB, hg = (e / Q) / j.NB;   // hg = (dw*G + g)*2 + h
    const int G = j.CK / (2 * Q);
    const int h = hg & 1, g = (hg >> 1) % G, dw = (hg >> 1) / G;
    const int nb = img % n_nb, kc = (img / n_nb) % n_kc, rt = img / (n_nb * n_kc);
    const int k = kc * j.CK + 2 * Q * g + Q * h + s, nn = nb * j.NB + n;
    const float v = k < j.K && nn < j.Nn ? weight_at(j, nn, rt * j.kw + dw, k) : 0.f;
    if constexpr (sizeof(T) == 2) return f32_to_bf16(v);
    else return v;
}

// conv_bf16_2d_kernel: wt[((((ny*n_kc + kc)*9 + tap)*2 + hq)*64 + nn)*8 + kk], k = 16*kc + 8*hq + kk, n = 64*ny + nn; one zero
// quad follows
__device__ __forceinline__ void bf16_tile(const WeightJob& j, int i) {
    unsigned short* const wt = static_cast<unsigned short*>(j.out);
    const int total = 9 * j.K * j.Nn;
    if (i < 8) wt[total + i] = 0;
    if (i >= total) return;
    const int kk = i & 7, nn = (i >> 3) & 63, hq = (i >> 9) & 1, rest = i >> 10;
    const int tap = rest % 9, ck = rest / 9, n_kc = j.K / 16;
    wt[i] = f32_to_bf16(weight_at(j, 64 * (ck / n_kc) + nn, tap, 16 * (ck % n_kc) + 8 * hq + kk));
}

// conv_bf16_rw_kernel, as A operands: wt[((((ny*4 + wave)*9 + tap)*NKC + kc)*64 + lane)*8 + s] = W[n = 128*ny + 32*wave +
// (lane & 31)][tap][k = 16*kc + 8*(lane >> 5) + s]; one zero quad follows
__device__ __forceinline__ void bf16_resident(const WeightJob& j, int i) {
    unsigned short* const wt = static_cast<unsigned short*>(j.out);
    const int total = 9 * j.K * j.Nn, nkc = j.K / 16;
    if (i < 8) wt[total + i] = 0;
    if (i >= total) return;
    const int s = i & 7, lane = (i >> 3) & 63;
    int rest = i >> 9;
    const int kc = rest % nkc;
    rest /= nkc;
    const int tap = rest % 9, block = rest / 9;   // block = 4*ny + wave
    wt[i] = f32_to_bf16(weight_at(j, 32 * block + (lane & 31), tap, 16 * kc + 8 * (lane >> 5) + s));
}

// conv_pair_kernel, in the order of use: [row tap][chunk of CK input channels][tap along W][group of 8][e][half][n], n < 2, of input
// channel 8 * group + 4 * half + e of the chunk
__device__ __forceinline__ void pair_form(const WeightJob& j, int i) {
    const int n = i & 1, half = (i >> 1) & 1, e = (i >> 2) & 3, G = j.CK / 8;
    int rest = i >> 4;
    const int g = rest % G;
    rest /= G;
    const int dw = rest % j.kw;
    rest /= j.kw;
    const int n_kc = (j.K + j.CK - 1) / j.CK, kc = rest % n_kc, rt = rest / n_kc;
    const int k = kc * j.CK + 8 * g + 4 * half + e;
    static_cast<float*>(j.out)[i] = k < j.K ? weight_at(j, n, rt * j.kw + dw, k) : 0.f;
}

// two-channel-output kernels: [n][tap][k], n < 2.  round_bf: the values are rounded to bfloat16 (kept as float32), for the kernels
// that multiply bfloat16 data with float32 arithmetic: weights that meet bfloat16 data are bfloat16 values in every kernel.
__device__ __forceinline__ void thin_out(const WeightJob& j, int i) {
    const float v = weight_at(j, i / (j.K * j.taps), (i / j.K) % j.taps, i % j.K);
    static_cast<float*>(j.out)[i] = j.round_bf ? bf16_to_f32(f32_to_bf16(v)) : v;
}

// conv_split_kernel, transformed along the rows and split, one thread per (output channel, input channel) padded to 32 and 16:
// u[block of 32 outputs][chunk = kd * n_kc + kc][ky][position][part][lane = 32 * (k / 8 % 2) + n % 32][k % 8]
__device__ __forceinline__ void split_form(const WeightJob& j, int i) {
    constexpr int kChunk = 16, kOperand = 64 * 8;
    const int n_kc = (j.K + kChunk - 1) / kChunk, Kp = n_kc * kChunk, n_kd = j.taps / 9;
    const int k = i % Kp, n = i / Kp;
    const bool in = k < j.K && n < j.Nn;
    for (int kd = 0; kd < n_kd; ++kd) {
        unsigned short* dst = static_cast<unsigned short*>(j.out) + ((size_t)(n / 32) * (n_kd * n_kc) + kd * n_kc + k / kChunk) * (36 * kOperand) +
                              (32 * ((k % kChunk) / 8) + n % 32) * 8 + k % 8;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            float g[3];
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) g[kx] = in ? weight_at(j, n, (kd * 3 + ky) * 3 + kx, k) : 0.f;
            const float uu[4] = {g[0], 0.5f * (g[0] + g[1] + g[2]), 0.5f * (g[0] - g[1] + g[2]), g[2]};
#pragma unroll
            for (int nu = 0; nu < 4; ++nu) {
                float r = uu[nu];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const unsigned short s = (unsigned short)pack_bf16x2(r, 0.f);   // (keeps every NaN, unlike f32_to_bf16)
                    dst[((ky * 4 + nu) * 3 + p) * kOperand] = s;
                    r -= bf16_to_f32(s);
                }
            }
        }
    }
}

// conv_time_split_kernel, split, one thread per (output channel, input channel) padded to 32 and to whole chunks:
// u[block of 32 outputs][tap][chunk][part][lane = 32 * (k / 8 % 2) + n % 32][k % 8]
__device__ __forceinline__ void time_split_form(const WeightJob& j, int i) {
    const int k = i % (16 * j.CK), n = i / (16 * j.CK);   // CK: chunks
    const bool in = k < j.K && n < j.Nn;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        unsigned short* dst = static_cast<unsigned short*>(j.out) + (((size_t)(n / 32) * 3 + t) * j.CK + k / 16) * (3 * 64 * 8) +
                              (32 * ((k % 16) / 8) + n % 32) * 8 + k % 8;
        float r = in ? weight_at(j, n, t, k) : 0.f;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned short s = (unsigned short)pack_bf16x2(r, 0.f);
            dst[p * (64 * 8)] = s;
            r -= bf16_to_f32(s);
        }
    }
}

// U = G g G^T for every (depth tap, output channel n, input channel k) as the LDS images of conv_wino_kernel (NBLK 64, one depth
// tap) and conv_wino3_kernel (NBLK 32, three):
// u[(((((ny*KD + kd)*n_kc + kc)*16 + pos)*2 + hq)*NBLK + nn)*4 + kk], n = NBLK*ny + nn, k = 8*kc + 4*hq + kk, pos = 4*xi + nu; one
// zero quad follows
template <int KD, int NBLK> __device__ __forceinline__ void wino_form(const WeightJob& j, int i) {
    float* const u = static_cast<float*>(j.out);
    if (i == 0) {
        float* z = u + (size_t)16 * KD * j.K * j.Nn;
        z[0] = z[1] = z[2] = z[3] = 0.f;
    }
    const int k = i % j.K, n = i / j.K;
    const int ny = n / NBLK, nn = n % NBLK, kc = k / 8, hq = (k % 8) / 4, kk = k % 4, n_kc = j.K / 8;
    for (int kd = 0; kd < KD; ++kd) {
        float g[3][3];
#pragma unroll
        for (int t = 0; t < 9; ++t) g[t / 3][t % 3] = weight_at(j, n, kd * 9 + t, k);
        float gg[4][3];   // G g
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            gg[0][b] = g[0][b];
            gg[1][b] = 0.5f * (g[0][b] + g[1][b] + g[2][b]);
            gg[2][b] = 0.5f * (g[0][b] - g[1][b] + g[2][b]);
            gg[3][b] = g[2][b];
        }
        float* dst = u + (((((size_t)(ny * KD + kd) * n_kc + kc) * 16) * 2 + hq) * NBLK + nn) * 4 + kk;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float uu[4] = {gg[x][0], 0.5f * (gg[x][0] + gg[x][1] + gg[x][2]), 0.5f * (gg[x][0] - gg[x][1] + gg[x][2]), gg[x][2]};
#pragma unroll
            for (int nu = 0; nu < 4; ++nu) dst[(size_t)(4 * x + nu) * 2 * NBLK * 4] = uu[nu];
        }
    }
}

}  // namespace

__global__ __launch_bounds__(256) void prepare_weights_kernel(WeightBatch b) {
    WeightJob j = b.job[blockIdx.y];
    j.w += blockIdx.z * b.w_step;
    j.out = static_cast<char*>(j.out) + blockIdx.z * b.out_step;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= j.threads) return;
    switch (j.form) {   // uniform for the workgroup
        case kWeightsImage: static_cast<float*>(j.out)[i] = image_element<4, float>(j, i); break;
        case kWeightsImageBf16: static_cast<unsigned short*>(j.out)[i] = image_element<8, unsigned short>(j, i); break;
        case kWeightsBf16Tile: bf16_tile(j, i); break;
        case kWeightsBf16Resident: bf16_resident(j, i); break;
        case kWeightsThinOut: thin_out(j, i); break;
        case kWeightsSplit: split_form(j, i); break;
        case kWeightsPair: pair_form(j, i); break;
        case kWeightsTimeSplit: time_split_form(j, i); break;
        case kWeightsWino: wino_form<1, 64>(j, i); break;
        default: wino_form<3, 32>(j, i); break;
    }
}

hipError_t prepare_weights(WeightBatch& b, hipStream_t st) {
    if (b.n < 1) return hipSuccess;
    long long most = 0;
    double bytes = 0.0;
    for (int i = 0; i < b.n; ++i) {
        WeightJob& j = b.job[i];
        const long long kn = (long long)j.K * j.Nn;
        auto up = [](long long v, long long m) { return (v + m - 1) / m * m; };
        switch (j.form) {
            case kWeightsImage:
            case kWeightsImageBf16: j.threads = j.taps * up(j.K, j.CK) * up(j.Nn, j.NB); break;
            case kWeightsBf16Tile:
            case kWeightsBf16Resident: j.threads = 9 * kn; break;
            case kWeightsThinOut: j.threads = j.taps * kn; break;
            case kWeightsPair: j.threads = j.taps * up(j.K, j.CK) * 2; break;
            case kWeightsTimeSplit: j.threads = 16 * j.CK * up(j.Nn, 32); break;
            case kWeightsSplit: j.threads = up(j.K, 16) * up(j.Nn, 32); break;
            default: j.threads = kn; break;
        }
        most = j.threads > most ? j.threads : most;
        const double per = j.form == kWeightsImage ? 4 : j.form == kWeightsSplit ? 72.0 * j.taps / 9 : j.form == kWeightsTimeSplit ? 18 : j.form == kWeightsWino ? 64 :
                           j.form == kWeightsWino3 ? 192 : j.form == kWeightsThinOut || j.form == kWeightsPair ? 4 : 2;   // written per thread
        bytes += 4.0 * j.taps * (double)kn + per * (double)j.threads;
    }
    KernelScope ks("weights_image", 0.0, bytes * (1 + b.more), st);
    hipLaunchKernelGGL(prepare_weights_kernel, dim3((unsigned)((most + 255) / 256), (unsigned)b.n, (unsigned)(1 + b.more)), dim3(256), 0, st, b);
    return hipGetLastError();
}

}  // namespace gleam
