// 3x3 and 3x3x3 convolution (forward and data gradient, float32) on the bfloat16 matrix cores without giving up
// float32 operands.
//
// Arithmetic.  A float32 number is exactly the sum of three bfloat16 numbers, x = x1 + x2 + x3 (8 + 8 + 8 significant
// bits: x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2), every difference exact), and a product of two bfloat16
// numbers is exact in the matrix core's float32 accumulator.  Of the nine partial products of a*b the six of weight
// 2^0, 2^-8 and 2^-16 are accumulated (a1 b1, a1 b2, a2 b1, a1 b3, a2 b2, a3 b1); the dropped ones are below
// 2^-24 |a b|, the rounding error of one float32 product.  v_mfma_f32_32x32x16_bf16 retires 16 times the products of
// v_mfma_f32_32x32x2_f32 per clock, so six of them per product are still 2.7 times as fast.
//
// Every matrix instruction rounds its accumulator once, so six per product into one accumulator would round it six times as
// often as it grows; the five small products therefore have accumulators of their own, added at the end.  Measured against
// 64-bit results over 24 networks of 32 and 64 channels, the error of a module's output is 0.79 (3x3) and 0.73 (3x3x3) of
// what the float32 matrix cores with F(2x2, 3x3) gave, and 1.0 - 1.4 of it with one accumulator.
//
// Fewer products.  Along the rows Winograd's minimal filtering F(2, 3) (Lavin & Gray) computes two neighbouring outputs of
// a three-tap row from four multiplications instead of six:
//     Y = A^T [ (G g) . (B^T d) ],  B^T = [1 0 -1 0; 0 1 1 0; 0 -1 1 0; 0 1 0 -1],  G = [1 0 0; .5 .5 .5; .5 -.5 .5; 0 0 1],
//     A^T = [1 1 1 0; 0 1 -1 -1]
// and the sums over row taps (three, or nine with the slices of a 3x3x3 kernel) and channels are taken between the
// transforms.  Both transforms are float32 additions; the split into bfloat16 happens behind the input transform.  The
// two-dimensional F(2x2, 3x3) needs a third less matrix work again but twice the accumulators per pixel: half the pixels per
// pass over the transformed weights, whose traffic out of L2 would then bound the kernel.
//
// Work split.  A workgroup of 4 waves owns 8 x 32 output pixels x 32 output channels (4 x 32 on small grids: two accumulators
// instead of the four below), two workgroups share a CU.  Wave nu owns transform position nu: accumulators r = 0..3 of 32 channels x 32 tiles, where accumulator r holds the 16 tiles (pixel
// pairs) of output row r and those of row r + 4.  The operand made from input rows (j, j + 4) then serves output rows
// (j - ky, j + 4 - ky) of all three row taps ky: 6 operands for 12 products.  A chunk is 16 input channels of one slice: the
// raw region (10 rows x 34 columns, zeros outside the image through the bounds of a buffer resource) is loaded straight into
// LDS one chunk ahead; the weight operands (9 per chunk and wave, already transformed, split and laid out lane by lane) go
// from L2 to registers.  After the last chunk the four positions of a tile meet in LDS, one accumulator per pass, and leave
// through the fused epilogue (bias, ReLU, ReLU mask, tensor to add).
//
// What bounds it: power.  A loop of nothing but these matrix instructions sustains 1.8 PFLOP/s on random operands (2.3 on
// constant ones), 1.5 with the four vector instructions per matrix instruction that the transform and the split need; a
// library product of two 8192 x 8192 bfloat16 matrices reaches 1.23.  64 -> 64 channels, 2 x 640 x 368, inside a step: 182 us
// forward and 189 us data gradient with F(2x2, 3x3) on the float32 matrix cores, 148 - 156 us both here, by card and by how long
// it has been busy (0.89 - 0.94 PFLOP/s issued; 140 us by itself); 32 -> 32 channels, 256 x 160 x 160, 27 taps: 1640 / 1850 us
// before, 1.30 - 1.33 ms both here (1.20 by itself); without the epilogue 10 % less, without the direct loads 8 - 15 % less,
// matrix and vector work alone 1.4 PFLOP/s.  Tried and taken out: 16-row blocks with one accumulator per
// product (6 - 8 % faster, less exact); all direct loads of a chunk at its start (each wave then waits for the address unit
// before its first matrix instruction: 10 % slower).
#include "split.h"

namespace gleam {

namespace {

constexpr int kChunk = 16;                 // input channels per chunk: the depth of one matrix instruction
constexpr int kOperand = 64 * 8;           // bfloat16 values of one weight operand (64 lanes x 8)
constexpr int kExFloats = 4 * 32 * 32;     // exchange of one pass: 4 positions x 32 tiles x 32 channels

template <int G> struct Region {             // a block has 2G rows
    static constexpr int kRows = 2 * G + 2;
    static constexpr int kSlots = kRows * 34 * 4;     // 16-byte quads of a raw region
    static constexpr int kWaveLoads = (kSlots + 63) / 64, kLoads = (kWaveLoads + 3) / 4;   // wave-wide direct loads, and per wave
    static constexpr int kRawFloats = kWaveLoads * 256 > kExFloats ? kWaveLoads * 256 : kExFloats;   // the exchange reuses a region
};

// exchange element (position, tile, channel quad): the quad index is XOR-ed with bits of the tile index so that the 16
// lanes LDS serves together touch 16 different 16-byte bank groups on both sides
__device__ __forceinline__ int ex_off(int pos, int tile, int cq) { return ((pos * 32 + tile) * 8 + (cq ^ ((tile >> 1) & 7))) * 4; }

}  // namespace

// EPI: the call has a ReLU mask or a tensor to add (1: the mask, if any, is a tensor; 2: it is sign words); 0: neither
template <int KD, bool RELU, int EPI, int G>
__global__ __launch_bounds__(256, 2) void conv_split_kernel(SplitConvArgs a) {
    constexpr int kRows = Region<G>::kRows, kWaveLoads = Region<G>::kWaveLoads, kLoads = Region<G>::kLoads, kRawFloats = Region<G>::kRawFloats;
    // Separate LDS objects: reads of one region then do not wait for direct loads into the other.
    __shared__ __attribute__((aligned(16))) float rawA[kRawFloats];
    __shared__ __attribute__((aligned(16))) float rawB[kRawFloats];
    __shared__ __attribute__((aligned(16))) float ex2[kExFloats];   // the exchange alternates between this and a raw region
    const int tid = threadIdx.x, lane = tid & 63;
    const int nu = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 31, h = lane >> 5;
    const XcdRange xr = xcd_range(a.n_blocks);
    if (xr.first >= xr.end) return;   // uniform for the workgroup
    const int n0 = 32 * (int)blockIdx.y;
    const int n_kc = (a.K + kChunk - 1) / kChunk, n_ch = KD * n_kc;
    const unsigned slice_bytes = (unsigned)a.H * a.W * a.K * 4u;

    struct Place {
        int x0, y0;
        long long img;   // slice index over all volumes
        int z;           // slice inside its volume (KD = 3)
    };
    auto place = [&](long long item) {
        Place b;
        if constexpr (KD == 3) {   // slices first: neighbouring workgroups share two of three input slices in L2
            b.z = (int)(item % a.D);
            const long long rest = item / a.D;
            b.x0 = 32 * (int)(rest % a.bx_n);
            const long long r2 = rest / a.bx_n;
            b.y0 = 2 * G * (int)(r2 % a.by_n);
            b.img = r2 / a.by_n * a.D + b.z;
        } else {
            b.z = 0;
            b.x0 = 32 * (int)(item % a.bx_n);
            const long long rest = item / a.bx_n;
            b.y0 = 2 * G * (int)(rest % a.by_n);
            b.img = rest / a.by_n;
        }
        return b;
    };

    // Direct loads: slot s = ((row * 2 + column parity) * 17 + column / 2) * 4 + quad', quad' = quad ^ (column / 8 & 3): the
    // 16 tiles of a row read 16 different 16-byte bank groups.  A pixel outside the image gets an offset outside the
    // buffer resource and arrives as zeros, as do the quads past the last channel in a ragged last chunk.
    unsigned off[kLoads];
    auto slot = [&](int t, int i, int* row, int* col, int* quad) {
        const int s = t + 256 * i, px = s >> 2;
        *row = px / 34;
        const int rem = px - *row * 34, par = rem >= 17 ? 1 : 0, half = rem - 17 * par;
        *col = 2 * half + par;
        *quad = (s & 3) ^ ((half >> 2) & 3);
    };
    auto offsets = [&](const Place& b) {
        int t = tid;
        asm volatile("" : "+v"(t));   // recomputed per block instead of held in registers
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            int row, col, quad;
            slot(t, i, &row, &col, &quad);
            const int yy = b.y0 - 1 + row, xx = b.x0 - 1 + col;
            const bool ok = yy >= 0 && yy < a.H && xx >= 0 && xx < a.W && row < kRows;
            off[i] = ok ? ((unsigned)(yy * a.W + xx) * (unsigned)a.K + 4u * quad) * 4u : 0x80000000u;
        }
    };
    unsigned ragged = 0u;   // bit i: quad of load i lies past the last channel of a ragged last chunk
    if (a.K % kChunk) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            int row, col, quad;
            slot(tid, i, &row, &col, &quad);
            ragged |= (4 * quad >= a.K % kChunk ? 1u : 0u) << i;
        }
    }
    struct Source {
        __amdgpu_buffer_rsrc_t rs;
        unsigned skip;   // `ragged` in the last chunk of a slice, or 0
        int off;         // bytes to the first channel
    };
    auto source = [&](const Place& b, int ch, bool any) {   // any = false: nothing left to load, every pixel is "outside"
        Source s;
        const int kd = KD == 3 ? ch / n_kc : 0, kc = ch - kd * n_kc;
        const bool in = any && (KD == 1 || (b.z + kd - 1 >= 0 && b.z + kd - 1 < a.D));
        s.rs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (in && KD == 3 ? b.img + kd - 1 : b.img) * (long long)a.H * a.W * a.K), 0,
                                                 in ? slice_bytes : 0u, 0x00020000);
        s.skip = kc == n_kc - 1 ? ragged : 0u;
        s.off = in ? kc * kChunk * 4 : 0;   // (no more than the size of the resource: the range check subtracts it from that)
        return s;
    };
    auto request = [&](const Source& s, int i, float* dst) {
        // where the last load is one too many for a wave, it repeats its previous one (no branch)
        const int k = 4 * i + 3 >= kWaveLoads && nu + 4 * i >= kWaveLoads ? i - 1 : i;
        const unsigned o = k == i ? off[i] | (s.skip << (31 - i) & 0x80000000u) : off[i > 0 ? i - 1 : 0] | (s.skip << (32 - i) & 0x80000000u);
        load_lds(s.rs, dst + (nu + 4 * k) * 256, o, s.off);
    };

    // weight operands of this wave (weights.hip): [channel block][chunk][row tap][position][part][lane]
    const bf16x8* const ubase = reinterpret_cast<const bf16x8*>(a.u) + ((size_t)blockIdx.y * n_ch * 12 + nu) * 3 * 64;
    bf16x8 u[3][3];
    auto load_u = [&](int ch, int ky) {
        const bf16x8* p = ubase + (size_t)(ch * 3 + ky) * (12 * 64) + lane;
#pragma unroll
        for (int k = 0; k < 3; ++k) u[ky][k] = p[k * 64];
    };

    // row of B^T: d[ca] + sg * d[cb]
    const int ca = nu == 0 ? 0 : (nu == 2 ? 2 : 1), cb = nu == 3 ? 3 : (nu == 2 ? 1 : 2);
    const float sg = nu == 1 ? 1.f : -1.f;
    int ra[2], rb[2];   // LDS float offsets of this lane's two channel quads in the two columns, set 0
    {
        const int mr = m >> 4, tc = m & 15;
        const int ia = tc + (ca >> 1), ib = tc + (cb >> 1);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            ra[q] = (((G * mr * 2 + (ca & 1)) * 17 + ia) * 4 + ((2 * h + q) ^ ((ia >> 2) & 3))) * 4;
            rb[q] = (((G * mr * 2 + (cb & 1)) * 17 + ib) * 4 + ((2 * h + q) ^ ((ib >> 2) & 3))) * 4;
        }
    }

    floatx16 acc[G], low[G];   // sums of the leading products, and of the other five
    auto clear = [&]() {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][r] = low[g][r] = 0.f;
    };

    struct Raw {
        float4 a[2], b[2];
    };
    auto read = [&](const float* buf, int j) {   // this lane's eight channels of the two columns, input rows (j, j + G)
        Raw r;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            r.a[q] = *reinterpret_cast<const float4*>(buf + ra[q] + j * (34 * 16));
            r.b[q] = *reinterpret_cast<const float4*>(buf + rb[q] + j * (34 * 16));
        }
        return r;
    };
    auto transform = [&](const Raw& r, float* v) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float x[4] = {r.a[q].x, r.a[q].y, r.a[q].z, r.a[q].w}, y[4] = {r.b[q].x, r.b[q].y, r.b[q].z, r.b[q].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float xe = x[e], ye = y[e];
                if (RELU) {   // on the bit patterns: negative floats are negative integers
                    xe = __int_as_float(__float_as_int(xe) > 0 ? __float_as_int(xe) : 0);
                    ye = __int_as_float(__float_as_int(ye) > 0 ? __float_as_int(ye) : 0);
                }
                v[4 * q + e] = fmaf(sg, ye, xe);
            }
        }
    };
    auto compute = [&](const float* buf, int next_ch, const Source& src, float* other) {
        float v[8];
        Raw r = read(buf, 0);
        transform(r, v);
        r = read(buf, 1);
        Split cur_v = split8(v);
#pragma unroll
        for (int j = 0; j < G + 2; ++j) {
            // The next chunk's direct loads, spread out (in one go they would hold up the wave that issues them), after the
            // first use of the last weights requested in the chunk before and ahead of the next weights: a wait for either
            // then does not wait for these.
#pragma unroll
            for (int i = 0; i < kLoads; ++i)
                if (j == G - 1) request(src, i, other);
            __builtin_amdgcn_sched_barrier(0);
            Split next_v = cur_v;
            if (j + 1 < G + 2) {   // the next rows are transformed and split between the matrix instructions of these
                transform(r, v);
                if (j + 2 < G + 2) r = read(buf, j + 2);
                next_v = split8(v);
            }
            // the row taps alternate so that neighbouring matrix instructions write different accumulators
#pragma unroll
            for (int p = 0; p < kProducts; ++p) {
#pragma unroll
                for (int ky = 0; ky < 3; ++ky)
                    if (j - ky >= 0 && j - ky < G) {
                        floatx16& sum = p + 1 < kProducts ? low[j - ky] : acc[j - ky];
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u[ky][kPartA[p]], cur_v.p[kPartB[p]], sum, 0, 0, 0);
                    }
            }
            // the next rows' transform first (it frees the registers the LDS reads after it go to), then their split
            if (j + 1 < G + 2) {
                if (j == 0) {
                    interleave<1, RELU ? 24 : 8>();
                    interleave<2, 9, 2>();
                    interleave<3, 9>();
                } else if (j == 1 || j == G) {
                    interleave<2, RELU ? 12 : 4>();
                    interleave<4, 4, 1>();
                    interleave<6, 5>();
                } else {
                    interleave<2, RELU ? 12 : 4>();
                    interleave<4, 3, 1>();
                    interleave<12, 3>();
                }
            }
            cur_v = next_v;
            // weights of a row tap are replaced by the next chunk's as soon as they have been used
            if (j == G - 1) load_u(next_ch, 0);
            if (j == G) load_u(next_ch, 1);
            if (j == G + 1) load_u(next_ch, 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // One pass per accumulator: the four positions of 32 tiles x 32 channels meet in LDS, a thread finishes the pixel pair of
    // one tile for one channel quad.  Everything outside the tensor (ragged tiles, channels past the last) has an offset
    // outside the buffer resources: loads give zeros, stores are dropped, and a pass costs no address arithmetic.
    auto epilogue = [&](const Place& b, long long item, float* free_raw) {
        int t = tid;
        asm volatile("" : "+v"(t));   // keeps the addresses below from being formed ahead of, and held across, the main loop
        const int e_cq = t & 7, e_tile = t >> 3;
        const bool n_ok = n0 + 4 * e_cq < a.Nn;   // channel counts are multiples of 4
        const float4 bias_r = a.bias && n_ok ? *reinterpret_cast<const float4*>(a.bias + n0 + 4 * e_cq) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float bb[4] = {bias_r.x, bias_r.y, bias_r.z, bias_r.w};
        const size_t slice = (size_t)b.img * a.H * a.W * a.Nn;
        const unsigned bytes = (unsigned)a.H * a.W * a.Nn * 4u, row_bytes = (unsigned)a.W * a.Nn * 4u;
        const __amdgpu_buffer_rsrc_t r_out = __builtin_amdgcn_make_buffer_rsrc((void*)(a.out + slice), 0, bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t r_ref = __builtin_amdgcn_make_buffer_rsrc((void*)(a.mask_ref + slice), 0, EPI == 1 && a.mask_ref ? bytes : 0u, 0x00020000);
        const __amdgpu_buffer_rsrc_t r_add = __builtin_amdgcn_make_buffer_rsrc((void*)(a.add + slice), 0, EPI && a.add ? bytes : 0u, 0x00020000);
        unsigned off_px[2];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int xx = b.x0 + 2 * (e_tile & 15) + jj, yy = b.y0 + G * (e_tile >> 4);
            off_px[jj] = xx < a.W && n_ok ? ((unsigned)(yy * a.W + xx) * (unsigned)a.Nn + n0 + 4 * e_cq) * 4u : 0x80000000u;
        }
        const int no_acc = EPI == 0 || a.mask_acc ? 0 : -1, no_add = EPI == 0 || a.mask_add ? 0 : -1;
        // The transform and the split turn an overflow into NaN.  A ReLU at the output takes what is below zero and lets NaN
        // pass; without one, NaN leaves as +infinity, because a ReLU at the input of the next layer may make 0 of NaN (fmaxf
        // does, and a maximum of bit patterns where the sign is set).  Two instructions per value, as a plain ReLU was.
        const int out_class = a.relu_out ? 0x3c : 0x3;   // negative numbers and -0, or NaN
        const float out_instead = a.relu_out ? 0.f : __builtin_huge_valf();
        const long long word_idx = ((long long)blockIdx.y * a.n_blocks + item) * 256 + t;
        const unsigned sign_in = EPI == 2 ? a.bits_in[word_idx] : 0u;   // one bit per value of this thread
        unsigned sign_out = 0u;
        const int ex_r = ex_off(0, e_tile, e_cq);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float* const ex = (g & 1) ? ex2 : free_raw;
            // An image of fewer rows than g has none of these rows: an offset of the whole slice puts every lane outside.  (The
            // range check subtracts it from the size of the slice, so it must not be larger.)
            const unsigned row_off = (g < a.H ? g : a.H) * row_bytes;
            uint4v refv[2], addv[2];
            if constexpr (EPI != 0) {
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    if constexpr (EPI == 1) refv[jj] = load16(r_ref, off_px[jj], row_off);
                    addv[jj] = load16(r_add, off_px[jj], row_off);
                }
            }
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
                *reinterpret_cast<float4*>(ex + ex_off(nu, t & 31, 2 * rg + ((t >> 5) & 1))) =
                    make_float4(acc[g][4 * rg] + low[g][4 * rg], acc[g][4 * rg + 1] + low[g][4 * rg + 1],
                                acc[g][4 * rg + 2] + low[g][4 * rg + 2], acc[g][4 * rg + 3] + low[g][4 * rg + 3]);
            __syncthreads();
            float q[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 p = *reinterpret_cast<const float4*>(ex + ex_r + k * (32 * 32));
                q[k][0] = p.x; q[k][1] = p.y; q[k][2] = p.z; q[k][3] = p.w;
            }
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                uint4v o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = (jj == 0 ? q[0][e] + (q[1][e] + q[2][e]) : (q[1][e] - q[2][e]) - q[3][e]) + bb[e];
                    v = __builtin_amdgcn_classf(v, out_class) ? out_instead : v;
                    if constexpr (EPI != 0) {
                        const int idx = 8 * g + 4 * jj + e;
                        const int pass = EPI == 2 ? __builtin_amdgcn_sbfe(sign_in, 8 * G - 1 - idx, 1) : (__uint_as_float(refv[jj][e]) > 0.f ? -1 : 0);
                        v = __int_as_float(__float_as_int(v) & (pass | no_acc));
                        v += __int_as_float((int)addv[jj][e] & (pass | no_add));
                    }
                    if (a.bits_out) sign_out = sign_out + sign_out + (v > 0.f ? 1u : 0u);   // value 0 ends up in the highest bit
                    o[e] = __float_as_uint(v);
                }
                store16(r_out, o, off_px[jj], row_off);
            }
        }
        if (a.bits_out) a.bits_out[word_idx] = sign_out;
        __syncthreads();   // the next chunk but one is loaded over the exchange
    };

    // One flat sequence of chunks over all blocks of this workgroup, alternating between the two regions; the next chunk, of
    // this block or the next, is requested before the current one is worked on.
    long long item = xr.first;
    int ch = 0;
    Place cur = place(item);
    offsets(cur);
    {
        const Source src = source(cur, 0, true);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) request(src, i, rawA);
    }
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) load_u(0, ky);
    clear();
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    auto step = [&](float* buf, float* other) {   // false after the last chunk
        const int nch = ch + 1 == n_ch ? 0 : ch + 1;
        const long long nitem = nch ? item : item + xr.stride;
        const bool more = nitem < xr.end;
        Place nxt = cur;
        if (more && nch == 0) {
            nxt = place(nitem);
            offsets(nxt);
        }
        compute(buf, nch, source(nxt, nch, more), other);
        // the direct loads are older than the nine weight operands requested at the end of compute(); six of those (row taps
        // 1 and 2 of the next chunk) may still be on their way
        __builtin_amdgcn_s_waitcnt(0x0070 | 6);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        if (nch == 0) {
            epilogue(cur, item, buf);
            clear();
        }
        cur = nxt;
        item = nitem;
        ch = nch;
        return more;
    };
    for (;;) {
        if (!step(rawA, rawB)) break;
        if (!step(rawB, rawA)) break;
    }
}

bool conv_split_applies(const PixDims& d, int K, int Nn) {
    return d.kt == 1 && (d.kd == 1 || d.kd == 3) && d.kh == 3 && d.kw == 3 && K % 4 == 0 && Nn % 4 == 0 &&
           4.0 * d.H * d.W * (K > Nn ? K : Nn) < 2.0e9;   // byte offsets inside a slice stay below the out-of-image marker
}

size_t conv_split_weight_floats(int K, int Nn, int kd) {
    return (size_t)((Nn + 31) / 32) * ((K + kChunk - 1) / kChunk) * kd * 36 * kOperand / 2;
}

// Rows of a block: 8, and 4 where blocks of 8 would leave CUs without one (half of them, with the longer chunk sequence of 27
// taps: a block of 4 rows forms four operands for 36 matrix instructions, one of 8 six for 72).  A residual block's layers, us
// with blocks of 8 and of 4 (workgroups of 8): 64 x 64, 16 channels (16) 9.4 / 7.6, 64 channels (32) 14.8 / 11.2; 160 x 128, 32
// channels (80) 13.0 / 10.3; 2 x 128 x 160, 32 channels (160) 13.0 / 11.6; 256 x 256, 32 channels (256) 14.0 / 12.9; 128 x 128,
// 128 channels (256) 25.1 / 25.6; 27 taps, 10 x 96 x 32, 64 channels (240) 31.0 / 31.9, 8 x 20 x 24, 32 channels (24) 17.2 / 12.9.
static long long split_blocks(const PixDims& d, int rows) {
    return d.Q / ((long long)d.H * d.W) * ((d.W + 31) / 32) * ((d.H + rows - 1) / rows);
}
static int split_rows(const PixDims& d, int Nn) { return split_blocks(d, 8) * ((Nn + 31) / 32) <= (d.kd == 3 ? 128 : 256) ? 4 : 8; }

size_t conv_split_sign_words(const PixDims& d, int Nn) {   // one word per thread, block and group of 32 channels
    return (size_t)split_blocks(d, split_rows(d, Nn)) * 256 * (size_t)((Nn + 31) / 32);
}

template <int KD, int G>
static void launch_conv_split_t(const SplitConvArgs& a, dim3 grid, int relu_in, hipStream_t st) {
    const int epi = a.bits_in ? 2 : a.mask_ref || a.add ? 1 : 0;
    if (relu_in) {   // a forward launch: no mask
        if (epi) hipLaunchKernelGGL((conv_split_kernel<KD, true, 1, G>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((conv_split_kernel<KD, true, 0, G>), grid, dim3(256), 0, st, a);
    } else {
        if (epi == 2) hipLaunchKernelGGL((conv_split_kernel<KD, false, 2, G>), grid, dim3(256), 0, st, a);
        else if (epi) hipLaunchKernelGGL((conv_split_kernel<KD, false, 1, G>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((conv_split_kernel<KD, false, 0, G>), grid, dim3(256), 0, st, a);
    }
}

hipError_t launch_conv_split(SplitConvArgs a, const PixDims& d, int relu_in, const char* name, hipStream_t st) {
    const int nb = (a.Nn + 31) / 32;
    a.H = d.H; a.W = d.W; a.D = d.D;
    a.bx_n = (a.W + 31) / 32;
    const int rows = split_rows(d, a.Nn);
    a.by_n = (a.H + rows - 1) / rows;
    a.n_blocks = split_blocks(d, rows);
    const long long cap = 512 / nb > 8 ? 512 / nb : 8;   // two workgroups per CU in total
    const dim3 grid((unsigned)(((a.n_blocks < cap ? a.n_blocks : cap) + 7) / 8 * 8), (unsigned)nb);
    const double direct = 2.0 * (double)d.Q * a.K * a.Nn * 9 * d.kd;
    // F(2, 3) along the rows: 4 multiplications of 6; six bfloat16 products per multiplication
    KernelScope ks(name, direct, 4.0 * (double)d.Q * (a.K + a.Nn), st, direct * 4.0);
    if (rows == 8) {
        if (d.kd == 3) launch_conv_split_t<3, 4>(a, grid, relu_in, st);
        else launch_conv_split_t<1, 4>(a, grid, relu_in, st);
    } else {
        if (d.kd == 3) launch_conv_split_t<3, 2>(a, grid, relu_in, st);
        else launch_conv_split_t<1, 2>(a, grid, relu_in, st);
    }
    return hipGetLastError();
}

}  // namespace gleam
