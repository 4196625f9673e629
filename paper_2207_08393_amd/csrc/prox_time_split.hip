// Temporal 3x1x1 convolution (forward and data gradient, float32) on the bfloat16 matrix cores: the arithmetic of prox_split.hip
// (every operand the sum of three bfloat16 numbers, six partial products, the five small ones in accumulators of their own),
//     out[t][p][n] = b[n] + sum over kt and k of W[n][kt][k] * in[t + kt - 1][p][k].
//
// Work split.  An input frame serves the output frames before it, of it and behind it, so a wave walks the frames of 32 pixels and
// splits every input once for all three: the accumulators of three output frames rotate (the walk is written out over the three
// rotations), and an output leaves when the frame behind it has been added.  A wave owns 32 output channels; contraction chunks are
// 16 input channels.  A lane's operand is eight consecutive channels of its pixel, which go from memory to its registers (a frame
// ahead, through a buffer resource that spans the frame: pixels and channels past the end arrive as zeros, a frame that is not there
// is an empty resource); the split of the next chunk rides between the matrix instructions of this one.  The split weights of a
// workgroup's output channels stay in LDS (72 KB at most, so that two workgroups share a CU), laid out lane by lane, and each is
// reloaded into its registers as soon as the chunk before has used it.  No barrier behind the first.  Waves of a workgroup take 2
// blocks of output channels by 2 blocks of pixels, or 4 blocks of pixels where the weights are larger or there is one such block.
// Where the segments of a call are fewer than the chip's workgroups the frames are cut into runs, of two frames more than they yield.
//
// What bounds it: matrix cores and vector instructions, which take turns (4.6 of these to a matrix instruction: the split, and 48
// moves a frame that pass the accumulators on; writing the walk out over three sets instead spilled 60 registers).  64 -> 64 channels
// at 20 x 192 x 160: 165 / 155 us forward / data gradient with the walk on the float32 matrix cores, 107 / 117 here (0.85 PFLOP/s
// issued); 48 -> 48 at 10 x 320 x 192, which that walk does not take: 135 with one tap at a time, 76 / 98 here.  Products as
// [pixel][channel], so that a store is two pixels' 128 bytes: as [channel][pixel], 16 bytes of 32 pixels each, 120 / 142 us.
#include "split.h"

namespace gleam {

namespace {

constexpr int kChunk = 16;                    // input channels per chunk: the depth of one matrix instruction
constexpr unsigned kOutside = 0x80000000u;    // an offset outside every buffer resource

// chunks the kernel is compiled for
int time_split_chunks(int K) {
    const int n = (K + kChunk - 1) / kChunk;
    return n <= 4 ? n : n <= 6 ? 6 : 8;
}
int time_split_blocks(int K, int Nn) {        // blocks of 32 output channels per workgroup
    return (Nn + 31) / 32 % 2 == 0 && time_split_chunks(K) <= 4 ? 2 : 1;
}

}  // namespace

// EPI: the call has a ReLU mask or a tensor to add
template <int NKC, bool EPI>
__global__ __launch_bounds__(256, 2) void conv_time_split_kernel(TimeSplitArgs a) {
    extern __shared__ uint4 smem[];           // [block of outputs][tap][chunk][part][lane]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 31, h = lane >> 5;
    const int cb = a.NB == 2 ? wave & 1 : 0, pb = a.NB == 2 ? wave >> 1 : wave;
    const int n0 = 32 * (a.NB * (int)blockIdx.y + cb);
    constexpr int kBlock = 9 * NKC * 64;      // quads of a block's weights
    const int n_w = a.NB * kBlock;
    {
        const uint4* src = reinterpret_cast<const uint4*>(a.u) + (size_t)blockIdx.y * n_w;
        for (int i = tid; i < n_w; i += 256) smem[i] = src[i];
    }
    __syncthreads();
    const uint4* const wl = smem + cb * kBlock + lane;
    const float bias = a.bias && n0 + m < a.Nn ? a.bias[n0 + m] : 0.f;

    const unsigned in_bytes = (unsigned)(a.P * a.K * 4), out_bytes = (unsigned)(a.P * a.Nn * 4);
    const int in_floor = a.relu_in ? 0 : (int)0x80000000;   // ReLU on the bit patterns: negative floats are negative integers
    // as in prox_split.hip: a ReLU at the output takes what is below zero and lets NaN pass, without one NaN leaves as infinity
    const int out_class = a.relu_out ? 0x3c : 0x3;
    const float out_instead = a.relu_out ? 0.f : __builtin_huge_valf();
    const int no_acc = a.mask_acc ? 0 : -1, no_add = a.mask_add ? 0 : -1;

    struct Sum {
        floatx16 acc, low;   // sums of the leading products, and of the other five
    };
    Sum s1, s2;
    bf16x8 w[3][3];          // [tap][part] of the chunk in hand
    uint4v raw[NKC][2];

    for (long long item = blockIdx.x; item < a.n_items; item += gridDim.x) {
        const long long seg = item % a.segs, rest = item / a.segs;
        const int t0 = (int)(rest % a.runs) * a.run, t1 = t0 + a.run < a.T ? t0 + a.run : a.T;
        const long long vol = rest / a.runs;
        const unsigned p = (unsigned)(seg * a.seg_px) + 32u * pb + m;
        const unsigned in_lane = (p * (unsigned)a.K + 8u * h) * 4u;
        const int f0 = t0 > 0 ? t0 - 1 : 0, f1 = t1 < a.T ? t1 : a.T - 1;   // first and last input frame
        // accumulator register r is pixel 8 (r / 4) + 4 h + r % 4 of the block, channel n0 + m
        const unsigned out_lane = n0 + m < a.Nn ? ((p - m + 4u * h) * (unsigned)a.Nn + n0 + m) * 4u : kOutside;
        auto request = [&](int f, int c) __attribute__((always_inline)) {   // this lane's channels of chunk c
            const bool ok = f <= f1;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(a.in + (vol * a.T + (ok ? f : 0)) * a.P * a.K), 0, ok ? in_bytes : 0u, 0x00020000);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const bool in = c < NKC - 2 || kChunk * c + 8 * h + 4 * q < a.K;
                raw[c][q] = load16(r, in ? in_lane + (unsigned)(64 * c + 16 * q) : kOutside, 0);
            }
        };
        auto pair = [&](int c, int i, SplitWords& s) __attribute__((always_inline)) {   // channels 2 i, 2 i + 1 of the lane's eight
            const int x = (int)raw[c][i >> 1][2 * (i & 1)], y = (int)raw[c][i >> 1][2 * (i & 1) + 1];
            split_pair(__int_as_float(x > in_floor ? x : in_floor), __int_as_float(y > in_floor ? y : in_floor), i, s);
        };
        auto load_w = [&](int c, int part) __attribute__((always_inline)) {
#pragma unroll
            for (int kt = 0; kt < 3; ++kt) w[kt][part] = __builtin_bit_cast(bf16x8, wl[((kt * NKC + c) * 3 + part) * 64]);
        };
        auto store = [&](const Sum& s, int t) __attribute__((always_inline)) {   // output frame t
            const long long frame = (vol * a.T + t) * a.P * a.Nn;
            const __amdgpu_buffer_rsrc_t r_out = __builtin_amdgcn_make_buffer_rsrc((void*)(a.out + frame), 0, out_bytes, 0x00020000);
            float ref[16], add[16];
            auto at = [&](int r) { return out_lane + (unsigned)((8 * (r >> 2) + (r & 3)) * a.Nn) * 4u; };
            if constexpr (EPI) {
                const __amdgpu_buffer_rsrc_t r_ref = __builtin_amdgcn_make_buffer_rsrc(
                    (void*)(a.mask_ref ? a.mask_ref + frame : a.out), 0, a.mask_ref ? out_bytes : 0u, 0x00020000);
                const __amdgpu_buffer_rsrc_t r_add = __builtin_amdgcn_make_buffer_rsrc((void*)(a.add ? a.add + frame : a.out), 0,
                                                                                        a.add ? out_bytes : 0u, 0x00020000);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    ref[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_ref, at(r), 0, 0));
                    add[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_add, at(r), 0, 0));
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float v = (s.acc[r] + s.low[r]) + bias;
                v = __builtin_amdgcn_classf(v, out_class) ? out_instead : v;
                if constexpr (EPI) {
                    const int pass = ref[r] > 0.f ? -1 : 0;
                    v = __int_as_float(__float_as_int(v) & (pass | no_acc));
                    v += __int_as_float(__float_as_int(add[r]) & (pass | no_add));
                }
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r_out, at(r), 0, 0);
            }
        };
        auto clear = [&](Sum& s) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s.acc[r] = s.low[r] = 0.f;
        };

        Split cur;
        // Input frame f: taps 0, 1, 2 into the output frames f + 1, f, f - 1; the last is complete then.  s1, s2: the sums of
        // the frames f and f - 1 so far; behind the call those of f + 1 and f.
        auto frame = [&](int f) __attribute__((always_inline)) {
            Sum s0;
            clear(s0);
            auto product = [&](int pr) __attribute__((always_inline)) {
#pragma unroll
                for (int kt = 2; kt >= 0; --kt) {
                    Sum& s = kt == 0 ? s0 : kt == 1 ? s1 : s2;
                    floatx16& x = pr + 1 < kProducts ? s.low : s.acc;
                    x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.p[kPartB[pr]], w[kt][kPartA[pr]], x, 0, 0, 0);
                }
            };
#pragma unroll
            for (int c = 0; c < NKC; ++c) {
                const int nc = c + 1 < NKC ? c + 1 : 0;
                SplitWords next;                         // of the next frame behind the last chunk
                // written in the order it is to run in: the matrix instructions, between them the next chunk's split, and its
                // weights as soon as those they replace have been used
                product(0);
                __builtin_amdgcn_sched_barrier(0);
                load_w(nc, 2);
                pair(nc, 0, next);
                product(1);
                __builtin_amdgcn_sched_barrier(0);
                pair(nc, 1, next);
                product(2);
                __builtin_amdgcn_sched_barrier(0);
                pair(nc, 2, next);
                product(3);
                __builtin_amdgcn_sched_barrier(0);
                load_w(nc, 1);
                pair(nc, 3, next);
                product(4);
                __builtin_amdgcn_sched_barrier(0);
                request(c + 1 < NKC ? f + 1 : f + 2, nc);
                product(5);
                __builtin_amdgcn_sched_barrier(0);
                load_w(nc, 0);
                cur = next.done();
                pin(cur);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (f > t0) store(s2, f - 1);
            s2 = s1;
            s1 = s0;
        };
#pragma unroll
        for (int c = 0; c < NKC; ++c) request(f0, c);
        clear(s1);
        clear(s2);
        load_w(0, 2);
        load_w(0, 1);
        load_w(0, 0);
        {
            SplitWords first;
#pragma unroll
            for (int i = 0; i < 4; ++i) pair(0, i, first);
            cur = first.done();
        }
        request(f0 + 1, 0);
        for (int f = f0; f <= f1; ++f) frame(f);
        if (t1 == a.T) store(s2, t1 - 1);   // no frame behind the last
    }
}

bool conv_time_split_applies(const PixDims& d, int K, int Nn) {
    const double P = (double)d.D * d.H * d.W;
    // byte offsets inside a frame, and those of a segment past its end, stay below the out-of-frame marker
    return d.kt == 3 && d.kd == 1 && d.kh == 1 && d.kw == 1 && K % 4 == 0 && Nn % 4 == 0 && K <= 128 && Nn <= kMaxChannels &&
           4.0 * (P + 128) * (K > Nn ? K : Nn) < 2.0e9;
}

size_t conv_time_split_weight_floats(int K, int Nn) { return (size_t)((Nn + 31) / 32) * 9 * time_split_chunks(K) * 64 * 4; }
int conv_time_split_chunks(int K) { return time_split_chunks(K); }

// (a function per kernel: each has to be allowed more than 64 KB of LDS)
template <int NKC, bool EPI>
static hipError_t launch_conv_time_split_e(const TimeSplitArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    static const hipError_t e = hipFuncSetAttribute((const void*)conv_time_split_kernel<NKC, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((conv_time_split_kernel<NKC, EPI>), grid, dim3(256), lds, st, a);
    return hipGetLastError();
}

template <int NKC>
static hipError_t launch_conv_time_split_t(const TimeSplitArgs& a, dim3 grid, size_t lds, hipStream_t st) {
    return a.mask_ref || a.add ? launch_conv_time_split_e<NKC, true>(a, grid, lds, st) : launch_conv_time_split_e<NKC, false>(a, grid, lds, st);
}

hipError_t launch_conv_time_split(TimeSplitArgs a, const PixDims& d, hipStream_t st) {
    a.T = d.T;
    a.P = (long long)d.D * d.H * d.W;
    a.NB = time_split_blocks(a.K, a.Nn);
    a.seg_px = 128 / a.NB;
    a.segs = (a.P + a.seg_px - 1) / a.seg_px;
    const int ny = (a.Nn + 31) / 32 / a.NB, nkc = time_split_chunks(a.K);
    const long long volumes = d.Q / (d.T * a.P), cap = 512 / ny > 8 ? 512 / ny : 8;   // two workgroups per CU in total
    const long long fit = cap / (volumes * a.segs), most = (d.T + 3) / 4;             // runs of four frames and more
    const long long want = fit < 1 ? 1 : fit < most ? fit : most;
    a.run = (int)((d.T + want - 1) / want);
    a.runs = (d.T + a.run - 1) / a.run;
    a.n_items = volumes * a.segs * a.runs;
    const size_t lds = (size_t)a.NB * 9 * nkc * 1024;
    const dim3 grid((unsigned)(a.n_items < cap ? a.n_items : cap), (unsigned)ny);
    switch (nkc) {
        case 1: return launch_conv_time_split_t<1>(a, grid, lds, st);
        case 2: return launch_conv_time_split_t<2>(a, grid, lds, st);
        case 3: return launch_conv_time_split_t<3>(a, grid, lds, st);
        case 4: return launch_conv_time_split_t<4>(a, grid, lds, st);
        case 6: return launch_conv_time_split_t<6>(a, grid, lds, st);
        default: return launch_conv_time_split_t<8>(a, grid, lds, st);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Weight gradient of the same layers on split operands:
//     dW[co][kt][ci] = sum over samples, frames t and pixels p of g[t][p][co] * x[t + kt - 1][p][ci].
// Input frame tau meets the gradients of frames tau + 1, tau and tau - 1, so a wave walks the frames of 16 pixels (the depth of one
// matrix instruction) with the operands of three gradient frames in registers, and forms two new operands for eighteen matrix
// instructions.  A lane of an operand is one channel at eight pixels, read from memory four bytes at a time a frame ahead
// (neighbouring lanes are neighbouring channels: 128 bytes of two pixels a load), so there is no staging and no barrier; pixels,
// channels and frames that are not there arrive as zeros through a buffer resource per frame.  A workgroup of 4 waves owns 32
// output x 32 input channels; the frames of all pixel groups are dealt to the waves in equal contiguous runs, and at the end the four
// waves' sums meet in LDS and leave as one partial sum in the layout of the weights.
//
// What bounds it: as above, 88 vector instructions to 18 matrix instructions.  64 -> 64 channels at 20 x 192 x 160: 128 - 138 us with
// the walk on the float32 matrix cores, 105 - 108 here; 48 -> 48 at 20 x 96 x 256, by itself on the float32 matrix cores with three
// taps staged apart: 215 us, 78 here.
template <bool RELU>
__global__ __launch_bounds__(256, 2) void wgrad_time_split_kernel(TimeWgradArgs a) {
    __shared__ __attribute__((aligned(16))) float ex[4 * 1024];   // one tap: 4 waves
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 31, h = lane >> 5;
    const int nib = (a.Ci + 31) / 32;
    const int co0 = 32 * ((int)blockIdx.y / nib), ci0 = 32 * ((int)blockIdx.y % nib);
    // runs are contiguous per XCD (workgroups go to the 8 XCDs in turn)
    const long long part = 4 * ((blockIdx.x & 7) * (long long)(gridDim.x >> 3) + (blockIdx.x >> 3)) + wave;
    const long long first = part * a.n_items / (4LL * gridDim.x), last = (part + 1) * a.n_items / (4LL * gridDim.x);
    const unsigned x_bytes = (unsigned)(a.P * a.Ci * 4), g_bytes = (unsigned)(a.P * a.Co * 4);

    floatx16 acc[3], low[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] = low[k][r] = 0.f;
    float bsum = 0.f;

    for (long long unit = first; unit < last;) {
        const int t0 = (int)(unit % a.T);
        const long long grp = unit / a.T;
        const int n = (int)(last - unit < a.T - t0 ? last - unit : a.T - t0);   // frames of this run
        unit += n;
        const long long vol = grp / a.segs;
        const unsigned p0 = 16u * (unsigned)(grp % a.segs) + 8u * h;
        unsigned xo[8], go[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            xo[e] = ci0 + m < a.Ci ? ((p0 + e) * (unsigned)a.Ci + ci0 + m) * 4u : kOutside;
            go[e] = co0 + m < a.Co ? ((p0 + e) * (unsigned)a.Co + co0 + m) * 4u : kOutside;
        }
        float rx[8], rg[8];
        auto load_x = [&](int f) __attribute__((always_inline)) {
            const bool ok = f >= 0 && f < a.T;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(a.a + (vol * a.T + (ok ? f : 0)) * a.P * a.Ci), 0,
                                                                               ok ? x_bytes : 0u, 0x00020000);
#pragma unroll
            for (int e = 0; e < 8; ++e) rx[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, xo[e], 0, 0));
        };
        auto load_g = [&](int f) __attribute__((always_inline)) {
            const bool ok = f >= 0 && f < a.T;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(a.g + (vol * a.T + (ok ? f : 0)) * a.P * a.Co), 0,
                                                                               ok ? g_bytes : 0u, 0x00020000);
#pragma unroll
            for (int e = 0; e < 8; ++e) rg[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, go[e], 0, 0));
        };
        auto x_pair = [&](int i, SplitWords& s) __attribute__((always_inline)) {
            float x = rx[2 * i], y = rx[2 * i + 1];
            if (RELU) {   // on the bit patterns: negative floats are negative integers
                x = __int_as_float(__float_as_int(x) > 0 ? __float_as_int(x) : 0);
                y = __int_as_float(__float_as_int(y) > 0 ? __float_as_int(y) : 0);
            }
            split_pair(x, y, i, s);
        };
        float bnew = 0.f;
        auto g_pair = [&](int i, SplitWords& s) __attribute__((always_inline)) {
            bnew += rg[2 * i] + rg[2 * i + 1];
            split_pair(rg[2 * i], rg[2 * i + 1], i, s);
        };
        Split z[3], v;   // gradients of frames tau + 1, tau, tau - 1 (rotating), input of frame tau
        auto form_g = [&](Split& out, bool counts) __attribute__((always_inline)) {
            SplitWords s;
            bnew = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) g_pair(i, s);
            bsum += counts ? bnew : 0.f;
            out = s.done();
        };
        load_g(t0 - 1);
        load_x(t0);
        form_g(z[0], false);
        load_g(t0);
        {
            SplitWords s;
#pragma unroll
            for (int i = 0; i < 4; ++i) x_pair(i, s);
            v = s.done();
        }
        form_g(z[1], true);
        load_g(t0 + 1);
        form_g(z[2], n > 1);
        load_x(t0 + 1);
        load_g(t0 + 2);
        // frame t0 + i: z[k], z[k + 1], z[k + 2] (k = i % 3) are the gradients of the frames before it, of it and behind it
        auto step = [&](int i, auto k_c) __attribute__((always_inline)) {
            constexpr int k = decltype(k_c)::value;
            Split &zm = z[k], &zz = z[(k + 1) % 3], &zp = z[(k + 2) % 3];
            auto product = [&](int kt, int p) __attribute__((always_inline)) {
                const Split& g = kt == 0 ? zp : kt == 1 ? zz : zm;
                floatx16& s = p + 1 < kProducts ? low[kt] : acc[kt];
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g.p[kPartA[p]], v.p[kPartB[p]], s, 0, 0, 0);
            };
            // written in the order it is to run in: eighteen matrix instructions (the gradient that is replaced first) and between
            // them the eight pairs of the two new operands
            SplitWords zw, vw;
            bnew = 0.f;
            product(2, 0);
            product(1, 0);
            product(0, 0);
            __builtin_amdgcn_sched_barrier(0);
            x_pair(0, vw);
            product(2, 1);
            product(1, 1);
            __builtin_amdgcn_sched_barrier(0);
            x_pair(1, vw);
            product(2, 2);
            product(0, 1);
            __builtin_amdgcn_sched_barrier(0);
            x_pair(2, vw);
            product(2, 3);
            product(1, 2);
            __builtin_amdgcn_sched_barrier(0);
            x_pair(3, vw);
            product(2, 4);
            product(0, 2);
            __builtin_amdgcn_sched_barrier(0);
            load_x(t0 + i + 2);
            product(2, 5);
            product(1, 3);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(0, zw);
            product(0, 3);
            product(1, 4);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(1, zw);
            product(0, 4);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(2, zw);
            product(1, 5);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(3, zw);
            product(0, 5);
            __builtin_amdgcn_sched_barrier(0);
            load_g(t0 + i + 3);
            bsum += i + 2 < n ? bnew : 0.f;
            v = vw.done();
            zm = zw.done();
            pin(v);
            pin(zm);
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int i = 0; i < n; i += 3) {
            step(i, std::integral_constant<int, 0>{});
            if (i + 1 < n) step(i + 1, std::integral_constant<int, 1>{});
            if (i + 2 < n) step(i + 2, std::integral_constant<int, 2>{});
        }
    }

    // the four waves' sums, one tap at a time; wave w finishes a quarter of the accumulator registers
    float* const out = a.partial + (size_t)blockIdx.x * a.Co * 3 * a.Ci;
#pragma unroll
    for (int kt = 0; kt < 3; ++kt) {
        if (kt) __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) ex[(wave * 16 + r) * 64 + lane] = acc[kt][r] + low[kt][r];
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int at = (4 * wave + rr) * 64 + lane;
            const int co = co0 + 8 * wave + 4 * h + rr, ci = ci0 + m;
            if (co < a.Co && ci < a.Ci) out[((size_t)co * 3 + kt) * a.Ci + ci] = (ex[at] + ex[1024 + at]) + (ex[2048 + at] + ex[3072 + at]);
        }
    }
    if (a.bias_partial && ci0 == 0) {
        __syncthreads();
        const float tot = bsum + __shfl_xor(bsum, 32);
        if (h == 0) ex[wave * 32 + m] = tot;
        __syncthreads();
        if (tid < 32 && co0 + tid < a.Co)
            a.bias_partial[(size_t)blockIdx.x * a.Co + co0 + tid] = (ex[tid] + ex[32 + tid]) + (ex[64 + tid] + ex[96 + tid]);
    }
}

bool wgrad_time_split_applies(const PixDims& d, int Ci, int Co) {
    const double P = (double)d.D * d.H * d.W;
    return d.kt == 3 && d.kd == 1 && d.kh == 1 && d.kw == 1 && Ci % 4 == 0 && Co % 4 == 0 && 4.0 * (P + 16) * (Ci > Co ? Ci : Co) < 2.0e9;
}

// Partial sums: two workgroups per CU over all channel blocks, but no run of a wave shorter than eight frames (operands of three
// more are formed to start one).
int wgrad_time_split_splits(const PixDims& d, int Ci, int Co) {
    const long long P = (long long)d.D * d.H * d.W, blocks = (Co + 31) / 32 * ((Ci + 31) / 32), per = 512 / blocks;
    const long long units = d.Q / P * ((P + 15) / 16), by8 = (units + 31) / 32;
    const long long n = per < by8 ? per : by8;
    return (int)((n < 8 ? 8 : n) / 8 * 8);
}

size_t wgrad_time_split_partial_floats(const PixDims& d, int Ci, int Co) { return (size_t)wgrad_time_split_splits(d, Ci, Co) * 3 * Ci * Co; }

hipError_t launch_wgrad_time_split(TimeWgradArgs a, const PixDims& d, int relu_in, hipStream_t st) {
    a.T = d.T;
    a.P = (long long)d.D * d.H * d.W;
    a.segs = (a.P + 15) / 16;
    a.n_items = d.Q / a.P * a.segs;   // frames of all pixel groups
    const dim3 grid((unsigned)wgrad_time_split_splits(d, a.Ci, a.Co), (unsigned)((a.Co + 31) / 32 * ((a.Ci + 31) / 32)));
    if (relu_in) hipLaunchKernelGGL((wgrad_time_split_kernel<true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((wgrad_time_split_kernel<false>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace gleam
