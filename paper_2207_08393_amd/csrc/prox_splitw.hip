// Weight gradient of 3x3 and 3x3x3 layers (float32) on the bfloat16 matrix cores: the arithmetic of prox_split.hip (operands
// as sums of three bfloat16 numbers, six partial products) and the same F(2, 3) along the rows, read backwards:
//     dL/dg[ky] = G^T [ sum over rows y and pixel pairs of (A dY(y)) . (B^T d(y + ky - 1)) ],
// per transform position and row tap a [cout x pairs] . [pairs x cin] matrix product, 4 multiplications per pixel pair and
// channel pair instead of 6.
//
// Work split.  A workgroup of 4 waves owns 32 output x 32 input channels of one slice tap and walks down a 32-pixel column
// (16 pixel pairs: the depth of one matrix instruction).  Wave nu holds transform position nu: three accumulators of 32x32,
// one per row tap.  A lane of an operand is one channel at eight pixel pairs, read from LDS four bytes at a time
// (neighbouring lanes are neighbouring channels), transformed and split in registers; the input operands of the last three
// rows stay in registers, so a row costs two new operands for three products.  Row segments go from memory to LDS by
// direct loads through one buffer resource per image row (pixels outside the row, rows outside the image and channels past
// the last arrive as zeros), two rows ahead of the operands, in a ring of three buffers that are separate LDS objects.
// While the matrix instructions of a row run, the operands of the next one are formed between them.
// The pixel rows of the image are dealt to the workgroups in equal contiguous runs; at the end the four positions meet in
// LDS, G^T is applied and every workgroup writes one partial sum in the layout of the weights.
//
// What bounds it: 64 -> 64 channels at 2 x 640 x 368 takes 139 - 150 us inside a step, by card and by how long it has been busy
// (171 us with F(2x2, 3x3) on the float32 matrix cores), and 135 us by itself (1.0 PFLOP/s issued); 117 us without the splits and the direct loads, 110 us with a sixth of the matrix instructions: a barrier per
// 18 matrix instructions and wave, and 113 vector instructions and 18 LDS reads between two of them.  16 -> 16 at 64 x 64:
// 31 -> 13 us.  Tried and taken out: 64 input channels per workgroup, three waves per SIMD (both spill: 2 - 4 times slower),
// one wave per SIMD with 64 x 64 channels (225 us, moves between the register files) or with all three slice taps of a
// 3x3x3 layer (1.55 ms); the first two rows of a run as steps without products instead of ahead of the loop (20 registers
// more, 8 % slower).
#include "split.h"

namespace gleam {

namespace {

constexpr long long kSmallGrid = 256;   // workgroups up to which runs have four rows
// one row in LDS: 34 input pixels and 32 gradient pixels of 32 channels, in 16-byte quads
constexpr int kInLoads = (34 * 8 + 63) / 64, kGLoads = 32 * 8 / 64, kLoads = kInLoads + kGLoads;   // wave-wide direct loads
constexpr int kPerWave = (kLoads + 3) / 4;
constexpr int kRowFloats = kLoads * 256, kGOff = kInLoads * 256;

}  // namespace

template <int KD, bool RELU>
__global__ __launch_bounds__(256, 2) void wgrad_split_kernel(SplitWgradArgs a) {
    __shared__ __attribute__((aligned(16))) float row0[kRowFloats];
    __shared__ __attribute__((aligned(16))) float row1[kRowFloats];
    __shared__ __attribute__((aligned(16))) float row2[kRowFloats];
    __shared__ __attribute__((aligned(16))) float ex[4 * 1024];   // one row tap: 4 positions
    const int tid = threadIdx.x, lane = tid & 63;
    const int nu = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 31, h = lane >> 5;
    const int nib = (a.Ci + 31) / 32;
    const int kd = KD == 3 ? (int)blockIdx.y % 3 : 0;
    const int blk = KD == 3 ? (int)blockIdx.y / 3 : (int)blockIdx.y;
    const int co0 = 32 * (blk / nib), ci0 = 32 * (blk % nib);

    // Runs are contiguous per XCD (workgroups go to the 8 XCDs in turn): neighbouring runs and the channel blocks of a run
    // share rows in its L2.
    const long long part = (blockIdx.x & 7) * (long long)(gridDim.x >> 3) + (blockIdx.x >> 3);
    const long long first = part * a.n_rows / gridDim.x, last = (part + 1) * a.n_rows / gridDim.x;

    // Element (pixel, channel) sits at (pixel ^ (pixel / 16 & 1)) * 32 + channel: the two lane halves of a read are 16 pixels
    // apart and so fall on different banks.
    unsigned off[kPerWave];   // byte offset inside the image row, or outside every row
    auto offsets = [&](int x0) {
        int t = lane;
        asm volatile("" : "+v"(t));   // recomputed per run instead of held in registers
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const bool g = nu + 4 * i >= kInLoads;
            const int s = (g ? nu + 4 * i - kInLoads : nu + 4 * i) * 64 + t;
            const int px = (s >> 3) ^ ((s >> 7) & 1), quad = s & 7;
            const int C = g ? a.Co : a.Ci, c = (g ? co0 : ci0) + 4 * quad;
            const int xx = x0 + px - (g ? 0 : 1);
            const bool ok = xx >= 0 && xx < a.W && c < C && px < (g ? 32 : 34);
            off[i] = ok ? (unsigned)(xx * C + c) * 4u : 0x80000000u;
        }
    };
    // one row of the stream: input row yi, gradient row yg (nothing outside the image; has_g false: no gradient row)
    auto issue = [&](long long in_img, bool in_ok, long long g_img, int yi, int yg, bool has_g, float* dst) {
        const bool iok = in_ok && yi >= 0 && yi < a.H;
        const __amdgpu_buffer_rsrc_t ri = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.a + (iok ? in_img * a.H + yi : 0) * (long long)a.W * a.Ci), 0, iok ? (unsigned)a.W * a.Ci * 4u : 0u, 0x00020000);
        const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.g + (has_g ? g_img * a.H + yg : 0) * (long long)a.W * a.Co), 0, has_g ? (unsigned)a.W * a.Co * 4u : 0u, 0x00020000);
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const int o = nu + 4 * i;
            if (o < kLoads) load_lds(o >= kInLoads ? rg : ri, dst + o * 256, off[i], 0);
        }
    };

    // position nu of B^T d: d[ca] + sg * d[cb]; of A dY: y[0], y[0] + y[1], y[0] - y[1] and y[1] (the sign of
    // the last is made up for at the end)
    const int ca = nu == 0 ? 0 : (nu == 2 ? 2 : 1), cb = nu == 3 ? 3 : (nu == 2 ? 1 : 2);
    const float sg = nu == 1 ? 1.f : -1.f;
    const float gb = nu == 1 ? 1.f : nu == 2 ? -1.f : 0.f;
    auto at = [&](int px) { return (px ^ ((px >> 4) & 1)) * 32 + m; };
    // LDS offsets of pair 0, and of pair 7, whose columns 2 and 3 lie in the next sixteen pixels
    const int oa = at(16 * h + (ca & 1)) + (ca & 2) * 32, ob = at(16 * h + (cb & 1)) + (cb & 2) * 32;
    const int oa7 = at(16 * h + 14 + ca), ob7 = at(16 * h + 14 + cb);
    const int og1 = kGOff + at(16 * h + 1), og0 = nu == 3 ? og1 : kGOff + at(16 * h);

    floatx16 acc[3], low[3];   // sums of the leading products, and of the other five (see prox_split.hip)
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] = low[k][r] = 0.f;
    float bsum = 0.f;

    struct Raw {
        float x[8], y[8];   // the two columns of eight pixel pairs
    };
    auto in_read = [&](const float* buf) {
        Raw r;
        int pa = oa, pb = ob;
        asm volatile("" : "+v"(pa), "+v"(pb));   // addresses are formed here, not once for every buffer and held
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            r.x[t] = buf[t == 7 ? oa7 : pa + t * 64];
            r.y[t] = buf[t == 7 ? ob7 : pb + t * 64];
        }
        return r;
    };
    auto g_read = [&](const float* buf) {
        Raw r;
        int pa = og0, pb = og1;
        asm volatile("" : "+v"(pa), "+v"(pb));
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            r.x[t] = buf[pa + t * 64];
            r.y[t] = buf[pb + t * 64];
        }
        return r;
    };
    auto in_pair = [&](const Raw& r, int i, SplitWords& s) {
        float v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            float x = r.x[2 * i + e], y = r.y[2 * i + e];
            if (RELU) {   // on the bit patterns: negative floats are negative integers
                x = __int_as_float(__float_as_int(x) > 0 ? __float_as_int(x) : 0);
                y = __int_as_float(__float_as_int(y) > 0 ? __float_as_int(y) : 0);
            }
            v[e] = fmaf(sg, y, x);
        }
        split_pair(v[0], v[1], i, s);
    };
    float bnew = 0.f;   // sum of the gradient operand in the making; position 1: y[0] + y[1] of every pair
    auto g_pair = [&](const Raw& r, int i, SplitWords& s) {
        const float v0 = fmaf(gb, r.y[2 * i], r.x[2 * i]), v1 = fmaf(gb, r.y[2 * i + 1], r.x[2 * i + 1]);
        bnew += v0 + v1;
        split_pair(v0, v1, i, s);
    };

    Split z, v[3];   // gradient operand; input operands of the last three rows, one replaced per step
    auto product = [&](int ky, const Split& in, int p) {
        floatx16& sum = p + 1 < kProducts ? low[ky] : acc[ky];
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(z.p[kPartA[p]], in.p[kPartB[p]], sum, 0, 0, 0);
    };

    for (long long row = first; row < last;) {
        const int y0 = (int)(row % a.H);
        const long long col = row / a.H;
        const int n = (int)((last - row < a.H - y0) ? last - row : a.H - y0);   // rows of this run
        row += n;
        const int x0 = 32 * (int)(col % a.bx_n);
        const long long img = col / a.bx_n;
        long long in_img = img;
        if constexpr (KD == 3) {
            const int z = (int)(img % a.D) + kd - 1;
            if (z < 0 || z >= a.D) {   // the slice tap falls outside: only the bias gradient (from kd = 1) would be left
                continue;
            }
            in_img = img + kd - 1;
        }
        offsets(x0);
        // stream element i: input row y0 - 1 + i and, from i = 2 on, gradient row y0 + i - 2; products of element i use the
        // input rows of elements i - 2, i - 1 and i
        auto load = [&](int i, float* dst) { issue(in_img, true, img, y0 - 1 + i, y0 + i - 2, i >= 2, dst); };
        load(0, row0);
        load(1, row1);
        load(2, row2);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        // operands of the first three elements; then their buffers take the next two
        auto form = [&](const float* buf, Split& out) {
            const Raw r = in_read(buf);
            SplitWords w;
#pragma unroll
            for (int i = 0; i < 4; ++i) in_pair(r, i, w);
            out = w.done();
        };
        form(row0, v[0]);
        form(row1, v[1]);
        form(row2, v[2]);
        {
            const Raw r = g_read(row2);
            SplitWords w;
            bnew = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) g_pair(r, i, w);
            z = w.done();
            bsum += bnew;
        }
        __syncthreads();
        if (n > 1) load(3, row0);
        if (n > 2) load(4, row1);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        // step i: products of element i while the operands of element i + 1 are formed; element i + 3 is requested into the
        // buffer that element i has left
        auto step = [&](int i, auto k_c, float* own, float* next) {
            constexpr int k = decltype(k_c)::value;   // i % 3
            const bool more = i + 3 < n + 2;
            if (more) load(i + 3, own);
            __builtin_amdgcn_sched_barrier(0);
            const Raw rg = g_read(next);
            SplitWords zw, vw;
            bnew = 0.f;
            // written in the order it is to run in: eighteen matrix instructions (oldest row first, its registers take the new
            // row's operand) and between them the eight pairs of the two new operands
            Split &v0 = v[(k + 1) % 3], &v1 = v[(k + 2) % 3], &v2 = v[k];
            product(0, v0, 0);
            product(1, v1, 0);
            product(2, v2, 0);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(rg, 0, zw);
            product(0, v0, 1);
            product(0, v0, 2);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(rg, 1, zw);
            product(0, v0, 3);
            product(1, v1, 1);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(rg, 2, zw);
            product(0, v0, 4);
            product(2, v2, 1);
            __builtin_amdgcn_sched_barrier(0);
            g_pair(rg, 3, zw);
            product(0, v0, 5);
            product(1, v1, 2);
            __builtin_amdgcn_sched_barrier(0);
            const Raw rv = in_read(next);
            product(2, v2, 2);
            product(1, v1, 3);
            __builtin_amdgcn_sched_barrier(0);
            in_pair(rv, 0, vw);
            product(2, v2, 3);
            product(1, v1, 4);
            __builtin_amdgcn_sched_barrier(0);
            in_pair(rv, 1, vw);
            product(2, v2, 4);
            product(1, v1, 5);
            __builtin_amdgcn_sched_barrier(0);
            in_pair(rv, 2, vw);
            product(2, v2, 5);
            __builtin_amdgcn_sched_barrier(0);
            in_pair(rv, 3, vw);
            z = zw.done();
            v[(k + 1) % 3] = vw.done();
            pin(z);
            pin(v[(k + 1) % 3]);
            bsum += i + 1 < n + 2 ? bnew : 0.f;   // the last element has no successor
            __builtin_amdgcn_sched_barrier(0);
            // element i + 2 has arrived when at most the loads just issued are in flight
            if (more) {
                if (nu + 4 * (kPerWave - 1) < kLoads) __builtin_amdgcn_s_waitcnt(0x0f70 | kPerWave);
                else __builtin_amdgcn_s_waitcnt(0x0f70 | (kPerWave - 1));
            } else {
                __builtin_amdgcn_s_waitcnt(0x0f70);
            }
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
        };
        // the last element's step forms operands nobody uses, from a buffer it may read
        for (int i = 2; i < n + 2; i += 3) {
            step(i, std::integral_constant<int, 2>{}, row2, row0);
            if (i + 1 < n + 2) step(i + 1, std::integral_constant<int, 0>{}, row0, row1);
            if (i + 2 < n + 2) step(i + 2, std::integral_constant<int, 1>{}, row1, row2);
        }
    }

    // G^T over the four positions, one row tap at a time; wave nu finishes a quarter of the accumulator registers
    const int taps = 9 * KD;
    float* const out = a.partial + (size_t)blockIdx.x * a.Co * taps * a.Ci;
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
        if (ky) __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) ex[(nu * 16 + r) * 64 + lane] = acc[ky][r] + low[ky][r];
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            float p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = ex[(k * 16 + 4 * nu + rr) * 64 + lane];
            const int co = co0 + 8 * nu + 4 * h + rr, ci = ci0 + m;
            if (co < a.Co && ci < a.Ci) {
                float* w = out + ((size_t)co * taps + (kd * 3 + ky) * 3) * a.Ci + ci;
                w[0] = p[0] + 0.5f * (p[1] + p[2]);
                w[a.Ci] = 0.5f * (p[1] - p[2]);
                w[2 * a.Ci] = 0.5f * (p[1] + p[2]) - p[3];
            }
        }
    }
    if (a.bias_partial && ci0 == 0 && kd == KD / 2 && nu == 1) {
        const float tot = bsum + __shfl_xor(bsum, 32);
        if (h == 0 && co0 + m < a.Co) a.bias_partial[(size_t)blockIdx.x * a.Co + co0 + m] = tot;
    }
}

bool wgrad_split_applies(const PixDims& d, int Ci, int Co) {
    // 3x3x3 layers between multiples of 32 channels have a kernel on the float32 matrix cores that forms every operand once for
    // three slice taps.  By itself it is as fast on a large volume (32 -> 32 at 256 x 160 x 160: 1.49 ms there, 1.51 here),
    // between the other launches of a step, under the power limit, it is not: 1.56 - 1.66 ms there, 1.43 here, with the sums of
    // the partial results 66 and 40 us (64 -> 64 at 2 x 20 x 96 x 96: 370 + 104 and 290 + 15 us a layer, the step 2370 and 2031).
    // Under 160 row segments the step takes 166 - 178 us here and 179 - 195 there; such volumes stay there, so that the kernel,
    // which greedy iterations run, has plain modules to be compared with.
    const long long segments = d.Q / d.W * ((d.W + 31) / 32);
    return d.kt == 1 && (d.kd == 1 || d.kd == 3) && d.kh == 3 && d.kw == 3 && Ci % 4 == 0 && Co % 4 == 0 &&
           (d.kd == 1 || Ci % 32 != 0 || Co % 32 != 0 || segments >= 160) &&
           4.0 * d.W * (Ci > Co ? Ci : Co) < 2.0e9;   // byte offsets inside an image row stay below the out-of-row marker
}

static int wgrad_split_blocks(const PixDims& d, int Ci, int Co) { return (Co + 31) / 32 * ((Ci + 31) / 32) * d.kd; }

// Partial sums: two workgroups per CU over all channel blocks, but no run shorter than eight rows (two more are read to
// start one), four where that leaves CUs without a workgroup (64 x 64, 16 -> 16 channels: 13.2 -> 10.7 us on 32 instead of 16).
int wgrad_split_splits(const PixDims& d, int Ci, int Co) {
    const long long rows = d.Q / d.W * ((d.W + 31) / 32), blocks = wgrad_split_blocks(d, Ci, Co), per = 512 / blocks;
    const long long few = kSmallGrid / blocks, by8 = (rows + 7) / 8, by4 = (rows + 3) / 4;
    const long long by_rows = by8 >= few ? by8 : by4 < few ? by4 : few;
    const long long n = per < by_rows ? per : by_rows;
    return (int)((n < 8 ? 8 : n) / 8 * 8);
}

size_t wgrad_split_partial_floats(const PixDims& d, int Ci, int Co) { return (size_t)wgrad_split_splits(d, Ci, Co) * 9 * d.kd * Ci * Co; }

hipError_t launch_wgrad_split(SplitWgradArgs a, const PixDims& d, int relu_in, hipStream_t st) {
    a.H = d.H; a.W = d.W; a.D = d.D;
    a.bx_n = (d.W + 31) / 32;
    a.n_rows = d.Q / d.W * a.bx_n;
    const dim3 grid((unsigned)wgrad_split_splits(d, a.Ci, a.Co), (unsigned)wgrad_split_blocks(d, a.Ci, a.Co));
    if (d.kd == 3) {
        if (relu_in) hipLaunchKernelGGL((wgrad_split_kernel<3, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((wgrad_split_kernel<3, false>), grid, dim3(256), 0, st, a);
    } else {
        if (relu_in) hipLaunchKernelGGL((wgrad_split_kernel<1, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((wgrad_split_kernel<1, false>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace gleam
