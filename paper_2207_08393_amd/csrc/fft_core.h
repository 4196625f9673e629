// In-LDS mixed-radix Stockham FFT building blocks for gfx950 (wave64).
//
// A transform of length N is a product of radices chosen at compile time (see next_radix: e.g. 368 = 16 * 23,
// 320 = 16 * 20, 640 = 32 * 20, 46 = 2 * 23).  A stage takes R points at stride N/R, applies the stage twiddles and an
// R-point DFT held in registers, and leaves them autosorted, so the result comes out in natural order with no bit-reversal
// pass.  The first stage takes its points straight from the caller (global memory), the last one hands them straight back;
// LDS is only the exchange between two stages.  Transforms are unnormalised here; callers scale at their global store.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

// The transform lengths that have kernels.
#define GLEAM_FFT_SIZES(X) \
    X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(46) X(64) X(96) X(128) X(160) X(192) X(256) X(320) X(368) X(640)

namespace gleam {

// ------------------------------------------------------------------ compile-time trigonometry
constexpr double kPi = 3.14159265358979323846264338327950288;

constexpr double ct_sin_small(double x) {  // |x| <= pi
    double term = x, sum = x, x2 = x * x;
    for (int n = 1; n < 16; ++n) {
        term *= -x2 / ((2 * n) * (2 * n + 1));
        sum += term;
    }
    return sum;
}
constexpr double ct_cos_small(double x) {
    double term = 1.0, sum = 1.0, x2 = x * x;
    for (int n = 1; n < 16; ++n) {
        term *= -x2 / ((2 * n - 1) * (2 * n));
        sum += term;
    }
    return sum;
}
// cos / sin of 2*pi*m/R for integers, reduced to [-pi, pi] first.
constexpr double ct_cos_frac(int m, int R) {
    m %= R;
    if (2 * m > R) m -= R;
    return ct_cos_small(2.0 * kPi * m / R);
}
constexpr double ct_sin_frac(int m, int R) {
    m %= R;
    if (2 * m > R) m -= R;
    return ct_sin_small(2.0 * kPi * m / R);
}

template <int I> using ic = std::integral_constant<int, I>;
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(ic<Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// ------------------------------------------------------------------ complex helpers
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmul_conj(float2 a, float2 b) {  // a * conj(b)
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
// multiply by -i (forward) or +i (inverse)
template <bool INV> __device__ __forceinline__ float2 mul_mi(float2 a) {
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// ------------------------------------------------------------------ small DFTs in registers
template <bool INV> __device__ __forceinline__ void dft2(float2& a, float2& b) {
    float2 t = csub(a, b);
    a = cadd(a, b);
    b = t;
}

template <bool INV> __device__ __forceinline__ void dft4(float2& b0, float2& b1, float2& b2, float2& b3) {
    float2 s02 = cadd(b0, b2), d02 = csub(b0, b2);
    float2 s13 = cadd(b1, b3), d13 = mul_mi<INV>(csub(b1, b3));
    b0 = cadd(s02, s13);
    b2 = csub(s02, s13);
    b1 = cadd(d02, d13);
    b3 = csub(d02, d13);
}

template <bool INV> __device__ __forceinline__ void dft8(float2 (&u)[8]) {
    constexpr float h = 0.70710678118654752440f;
    float2 a0 = cadd(u[0], u[4]), a4 = csub(u[0], u[4]);
    float2 a1 = cadd(u[1], u[5]), a5 = csub(u[1], u[5]);
    float2 a2 = cadd(u[2], u[6]), a6 = csub(u[2], u[6]);
    float2 a3 = cadd(u[3], u[7]), a7 = csub(u[3], u[7]);
    // a5 *= w8, a6 *= w8^2, a7 *= w8^3 with w8 = exp(-+ i pi/4)
    a5 = INV ? make_float2(h * (a5.x - a5.y), h * (a5.x + a5.y)) : make_float2(h * (a5.x + a5.y), h * (a5.y - a5.x));
    a6 = mul_mi<INV>(a6);
    a7 = INV ? make_float2(-h * (a7.x + a7.y), h * (a7.x - a7.y)) : make_float2(h * (a7.y - a7.x), -h * (a7.x + a7.y));
    dft4<INV>(a0, a1, a2, a3);
    dft4<INV>(a4, a5, a6, a7);
    u[0] = a0; u[2] = a1; u[4] = a2; u[6] = a3;
    u[1] = a4; u[3] = a5; u[5] = a6; u[7] = a7;
}

// Odd prime length R by conjugate-pair folding: with a_r = u_r + u_{R-r}, b_r = u_r - u_{R-r},
//   X_q     = u_0 + sum_r cos(2 pi q r / R) a_r  -+ i sum_r sin(2 pi q r / R) b_r
//   X_{R-q} = the same with the opposite sign of the second sum,
// which halves the multiplications of the direct R x R product; all constants are literals.
template <int R, bool INV> __device__ __forceinline__ void dft_odd(float2 (&u)[R]) {
    constexpr int Hn = (R - 1) / 2;
    float2 a[Hn], b[Hn];
#pragma unroll
    for (int r = 1; r <= Hn; ++r) {
        a[r - 1] = cadd(u[r], u[R - r]);
        b[r - 1] = csub(u[r], u[R - r]);
    }
    const float2 u0 = u[0];
    float2 s = u0;
#pragma unroll
    for (int r = 0; r < Hn; ++r) s = cadd(s, a[r]);
    u[0] = s;
    static_for<Hn>([&](auto qi) {
        constexpr int q = decltype(qi)::value + 1;
        float2 A = u0, Bv = make_float2(0.f, 0.f);
        static_for<Hn>([&](auto ri) {
            constexpr int r = decltype(ri)::value + 1;
            constexpr float c = (float)ct_cos_frac(q * r, R);
            constexpr float sn = (float)ct_sin_frac(q * r, R);
            A.x = fmaf(c, a[r - 1].x, A.x);
            A.y = fmaf(c, a[r - 1].y, A.y);
            Bv.x = fmaf(sn, b[r - 1].x, Bv.x);
            Bv.y = fmaf(sn, b[r - 1].y, Bv.y);
        });
        // forward: X_q = A - i Bv ; inverse: X_q = A + i Bv
        const float2 lo = make_float2(A.x + Bv.y, A.y - Bv.x), hi = make_float2(A.x - Bv.y, A.y + Bv.x);
        u[q] = INV ? hi : lo;
        u[R - q] = INV ? lo : hi;
    });
}

// First factor of an in-register DFT of length R: R itself for the base cases (2, 4, 8, odd primes).
constexpr int first_factor(int R) {
    if (R == 2 || R == 4 || R == 8) return R;
    if (R % 8 == 0) return 8;
    if (R % 4 == 0) return 4;
    if (R % 2 == 0) return 2;
    for (int p = 3; p * p <= R; p += 2)
        if (R % p == 0) return p;
    return R;
}

// DFT of any small length held in registers.  Composite R = R1*R2 is one Cooley-Tukey step with
// literal twiddles: X[q1 + R1*q2] = sum_r2 w_R2^(r2 q2) * w_R^(r2 q1) * (sum_r1 w_R1^(r1 q1) u[r1*R2 + r2]).
template <int R, bool INV> __device__ __forceinline__ void dft_r(float2 (&u)[R]) {
    constexpr int R1 = first_factor(R);
    if constexpr (R == 1) {
    } else if constexpr (R1 == R) {
        if constexpr (R == 2) dft2<INV>(u[0], u[1]);
        else if constexpr (R == 4) dft4<INV>(u[0], u[1], u[2], u[3]);
        else if constexpr (R == 8) dft8<INV>(u);
        else dft_odd<R, INV>(u);
    } else {
        constexpr int R2 = R / R1;
        float2 y[R];
        static_for<R2>([&](auto r2c) {
            constexpr int r2 = decltype(r2c)::value;
            float2 v[R1];
            static_for<R1>([&](auto r1c) { v[decltype(r1c)::value] = u[decltype(r1c)::value * R2 + r2]; });
            dft_r<R1, INV>(v);
            static_for<R1>([&](auto q1c) {
                constexpr int q1 = decltype(q1c)::value;
                if constexpr (q1 * r2 == 0) {
                    y[q1 * R2 + r2] = v[q1];
                } else {
                    constexpr float c = (float)ct_cos_frac(q1 * r2, R);
                    constexpr float sn = (float)ct_sin_frac(q1 * r2, R);   // forward twiddle = c - i sn
                    const float2 w = make_float2(c, INV ? sn : -sn);
                    y[q1 * R2 + r2] = cmul(v[q1], w);
                }
            });
        });
        static_for<R1>([&](auto q1c) {
            constexpr int q1 = decltype(q1c)::value;
            float2 v[R2];
            static_for<R2>([&](auto r2c) { v[decltype(r2c)::value] = y[q1 * R2 + decltype(r2c)::value]; });
            dft_r<R2, INV>(v);
            static_for<R2>([&](auto q2c) { u[q1 + R1 * decltype(q2c)::value] = v[decltype(q2c)::value]; });
        });
    }
}

// ------------------------------------------------------------------ radix plan
// Radix of the stage that follows a partial product P (P divides N): whatever is left once it fits in registers (<= 24
// points), 32 where that leaves so few, otherwise the largest power of two up to 16, otherwise a small prime: few stages, few
// exchanges.
constexpr int next_radix(int N, int P) {
    int m = N / P;
    if (m <= 24) return m;
    if (m % 32 == 0 && m / 32 <= 24 && m / 16 > 24) return 32;
    if (m % 16 == 0) return 16;
    if (m % 8 == 0) return 8;
    if (m % 4 == 0) return 4;
    if (m % 2 == 0) return 2;
    for (int r = 3; r <= m; r += 2)
        if (m % r == 0) return r;
    return 1;
}

// Radix of the last stage.
constexpr int last_radix(int N) {
    int P = 1;
    while (P * next_radix(N, P) < N) P *= next_radix(N, P);
    return N / P;
}

// Forward twiddles of all stages but the first, stage after stage: w[r * P + k] = exp(-2 pi i r k / (P R)) for the stage that
// follows a partial product P.  A wave reads neighbouring k of one r.  Tables in memory, evaluated by the compiler: sincospi in
// double at the start of every workgroup, as it was before, took longer than the first loads of a small tile.
constexpr int twiddle_offset(int N, int P) {   // of the stage that follows P
    int at = 0;
    for (int p = next_radix(N, 1); p < P; p *= next_radix(N, p)) at += p * next_radix(N, p);
    return at;
}
struct Twiddle {
    float x, y;
};
// exp(-2 pi i m / n), evaluated in the first octant
constexpr Twiddle ct_twiddle(int m, int n) {
    m %= n;
    // angle = 2 pi m / n = (pi / 4) * (8 m / n): octant and what is left of it, in units of 1 / n of an eighth turn
    const int oct = 8 * m / n, rem = 8 * m - oct * n;
    const double a = kPi / 4 * ((oct & 1) ? n - rem : rem) / n;
    double c = ct_cos_small(a), s = ct_sin_small(a);
    if (((oct + 1) >> 1) & 1) {
        const double t = c;
        c = s;
        s = t;
    }
    const bool c_neg = oct >= 2 && oct < 6, s_neg = oct < 4;   // (the sine of the forward exponent is negative up to half a turn)
    return Twiddle{(float)(c_neg ? -c : c), (float)(s_neg ? -s : s)};
}
template <int N> struct TwiddleTable {
    static constexpr int kSize = twiddle_offset(N, N) > 0 ? twiddle_offset(N, N) : 1;
    Twiddle w[kSize];
    constexpr TwiddleTable() : w{} {
        int at = 0;
        for (int P = next_radix(N, 1); P < N; P *= next_radix(N, P)) {
            const int R = next_radix(N, P);
            for (int r = 0; r < R; ++r)
                for (int k = 0; k < P; ++k) w[at + r * P + k] = ct_twiddle(r * k, P * R);
            at += P * R;
        }
    }
};
template <int N> __device__ constexpr TwiddleTable<N> kTwiddles{};

// ------------------------------------------------------------------ a tile of L transforms of length N
// ROWS: the lines lie one after the other in memory (neighbouring lanes take neighbouring positions); otherwise they are
// neighbouring columns (neighbouring lanes take neighbouring lines).  Every sixteen positions the exchange buffer skips one:
// a stage writes at stride 16 (its radix) and reads at stride 1, both without bank conflicts, and in the ROWS layout the
// lines start half the banks apart.
template <int N, int L, bool ROWS> struct Tile {
    static constexpr bool kSingle = next_radix(N, 1) == N;
    static constexpr int kPadded = N + (kSingle ? 0 : (N - 1) / 16);
    static constexpr int kLine = kSingle ? (N | 1) : (kPadded + 15) / 32 * 32 + 16;   // ROWS: distance of two lines
    static constexpr int kElems = ROWS ? L * kLine : L * kPadded;
    static_assert(kLine >= kPadded, "a line holds its positions");
    __device__ static __forceinline__ unsigned at(unsigned line, unsigned pos) {
        const unsigned p = kSingle ? pos : pos + pos / 16;
        return ROWS ? line * kLine + p : p * L + line;
    }
    // element r of a butterfly that starts at `pos` and goes in steps of STEP; `from` = at(line, pos): a constant distance
    // away unless padding may fall between
    template <int STEP, bool ALIGNED> __device__ static __forceinline__ unsigned at(unsigned from, unsigned line, unsigned pos, int r) {
        if constexpr (kSingle || STEP % 16 == 0) return from + r * ((kSingle ? STEP : STEP + STEP / 16) * (ROWS ? 1 : L));
        else if constexpr (ALIGNED) return from + r * (STEP * (ROWS ? 1 : L));   // starts at a multiple of 16 and ends below the next
        else return at(line, pos + r * STEP);
    }
};

// The forward transform goes through its stages in order: the stage that follows a partial product P reads points
// i + r * T (T = N / R), multiplies them by the twiddles, transforms, and leaves them at j + r * P.  The inverse is its mirror
// image, stage by stage from the last to the first: it reads j + r * P, transforms, multiplies by the conjugate twiddles and
// leaves i + r * T.  So the points that a thread holds at the end of the forward transform are those that it begins the
// inverse with: a multiplication in between (the mask) needs no exchange, the twiddles in registers serve both directions, and
// every stage writes back where it has read.
template <int N, int P> struct Stage {
    static constexpr int R = next_radix(N, P), T = N / R;
    static constexpr bool kFirst = P == 1, kLast = P * R == N;
    static constexpr int kBefore = [] {   // the P of the stage before
        int p = 1;
        while (p < P && p * next_radix(N, p) < P) p *= next_radix(N, p);
        return p;
    }();
};
constexpr int last_stage(int N) { return N / last_radix(N); }   // P of the last stage

template <int N, int L, int NT, bool ROWS, int P> struct StageOf : Stage<N, P> {
    using Stage<N, P>::R;
    using Stage<N, P>::T;
    using Lay = Tile<N, L, ROWS>;
    static constexpr int PER = (L * T + NT - 1) / NT;   // butterflies per thread
    __device__ static __forceinline__ bool mine(int m) { return PER * NT == L * T || threadIdx.x + m * NT < L * T; }
    __device__ static __forceinline__ unsigned line(int m) { const unsigned idx = threadIdx.x + m * NT; return ROWS ? idx / T : idx % L; }
    __device__ static __forceinline__ unsigned i(int m) { const unsigned idx = threadIdx.x + m * NT; return ROWS ? idx % T : idx / L; }
    __device__ static __forceinline__ unsigned j(int m) { return (i(m) - i(m) % P) * R + i(m) % P; }
    // LDS element r of the points i + r * T, and of j + r * P
    __device__ static __forceinline__ unsigned at_i(int m, int r) { return Lay::template at<T, false>(Lay::at(line(m), i(m)), line(m), i(m), r); }
    __device__ static __forceinline__ unsigned at_j(int m, int r) { return Lay::template at<P, P == 1 && R == 16>(Lay::at(line(m), j(m)), line(m), j(m), r); }
    __device__ static __forceinline__ void twiddles(int m, float2 (&w)[R]) {
        const float2* tw = reinterpret_cast<const float2*>(kTwiddles<N>.w) + twiddle_offset(N, P) + i(m) % P;
#pragma unroll
        for (int r = 1; r < R; ++r) w[r] = tw[r * P];
    }
};

// load(line, i, step, u, m): u[r] = point i + r * step of the line; out(line, i, step, u, m): the same points of the result, u
// may be changed; m: which of the thread's butterflies it is.  The exchange buffer must not be in use when a call begins.
//
// Forward transform.  BACK: continued by the inverse (ifft_stages with FROM_LDS, which synchronises first): the points as out()
// leaves them are taken through the first of its stages.  then(): once, behind the loads of the first points.
template <int N, int L, int NT, bool ROWS, bool BACK, int P, class Load, class Out, class Then>
__device__ __forceinline__ void fft_stages(float2* __restrict__ buf, Load&& load, Out&& out, Then&& then) {
    using S = StageOf<N, L, NT, ROWS, P>;
    constexpr int R = S::R, PER = S::PER;
    float2 u[PER][R], w[PER][R];
    if constexpr (!S::kFirst) {   // on their way while the workgroup synchronises
#pragma unroll
        for (int m = 0; m < PER; ++m)
            if (S::mine(m)) S::twiddles(m, w[m]);
        __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < PER; ++m)
        if (S::mine(m)) {
            if constexpr (S::kFirst) {
                load(S::line(m), S::i(m), ic<S::T>{}, u[m], m);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) u[m][r] = buf[S::at_i(m, r)];
            }
        }
    if constexpr (S::kFirst) then();
    if constexpr (!S::kFirst && !S::kLast) __syncthreads();
#pragma unroll
    for (int m = 0; m < PER; ++m)
        if (S::mine(m)) {
            if constexpr (!S::kFirst) {
#pragma unroll
                for (int r = 1; r < R; ++r) u[m][r] = cmul(u[m][r], w[m][r]);
            }
            dft_r<R, false>(u[m]);
            if constexpr (S::kLast) {
                out(S::line(m), S::j(m), ic<P>{}, u[m], m);
                if constexpr (BACK) {
                    dft_r<R, true>(u[m]);
                    if constexpr (!S::kFirst) {
#pragma unroll
                        for (int r = 1; r < R; ++r) u[m][r] = cmul_conj(u[m][r], w[m][r]);
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) buf[S::at_i(m, r)] = u[m][r];
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) buf[S::at_j(m, r)] = u[m][r];
            }
        }
    if constexpr (!S::kLast) fft_stages<N, L, NT, ROWS, BACK, P * R>(buf, load, out, then);
}

// Inverse transform from stage P down.  FIRST: stage P begins it, with points from load(); otherwise they are in `buf` (not
// yet synchronised).  TO_LDS: the result, as out() leaves it, goes to `buf` (not yet synchronised).
template <int N, int L, int NT, bool ROWS, bool FIRST, bool TO_LDS, int P, class Load, class Out>
__device__ __forceinline__ void ifft_stages(float2* __restrict__ buf, Load&& load, Out&& out) {
    using S = StageOf<N, L, NT, ROWS, P>;
    constexpr int R = S::R, PER = S::PER;
    constexpr bool kWrite = !S::kFirst || TO_LDS;
    float2 u[PER][R], w[PER][R];
    if constexpr (!S::kFirst) {
#pragma unroll
        for (int m = 0; m < PER; ++m)
            if (S::mine(m)) S::twiddles(m, w[m]);
    }
    if constexpr (!FIRST) __syncthreads();
#pragma unroll
    for (int m = 0; m < PER; ++m)
        if (S::mine(m)) {
            if constexpr (FIRST) {
                load(S::line(m), S::j(m), ic<P>{}, u[m], m);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) u[m][r] = buf[S::at_j(m, r)];
            }
        }
    if constexpr (!FIRST && kWrite) __syncthreads();
#pragma unroll
    for (int m = 0; m < PER; ++m)
        if (S::mine(m)) {
            dft_r<R, true>(u[m]);
            if constexpr (!S::kFirst) {
#pragma unroll
                for (int r = 1; r < R; ++r) u[m][r] = cmul_conj(u[m][r], w[m][r]);
            } else {
                out(S::line(m), S::i(m), ic<S::T>{}, u[m], m);
            }
            if constexpr (kWrite) {
#pragma unroll
                for (int r = 0; r < R; ++r) buf[S::at_i(m, r)] = u[m][r];
            }
        }
    if constexpr (!S::kFirst) ifft_stages<N, L, NT, ROWS, false, TO_LDS, S::kBefore>(buf, load, out);
}

// Rows short enough for one stage: a lane per line would read memory a whole line apart, so their points pass through LDS.
template <int N, int L, int NT, bool INV, class Load, class Out>
__device__ __forceinline__ void short_rows(float2* __restrict__ buf, Load&& load, Out&& out, bool again) {
    using Lay = Tile<N, L, true>;
    constexpr int PER = (L * N + NT - 1) / NT;
    if (!again) {
        float2 v[PER][1];
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const unsigned e = threadIdx.x + m * NT;
            if (e < L * N) load(e / N, e % N, ic<1>{}, v[m], m);
        }
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const unsigned e = threadIdx.x + m * NT;
            if (e < L * N) buf[Lay::at(e / N, e % N)] = v[m][0];
        }
    }
    __syncthreads();
    for (unsigned line = threadIdx.x; line < L; line += NT) {
        float2 u[N];
#pragma unroll
        for (int r = 0; r < N; ++r) u[r] = buf[Lay::at(line, r)];
        dft_r<N, INV>(u);
#pragma unroll
        for (int r = 0; r < N; ++r) buf[Lay::at(line, r)] = u[r];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const unsigned e = threadIdx.x + m * NT;
        if (e < L * N) {
            float2 v[1] = {buf[Lay::at(e / N, e % N)]};
            out(e / N, e % N, ic<1>{}, v, m);
            buf[Lay::at(e / N, e % N)] = v[0];
        }
    }
}

// The points of a row tile that fft_tile asks for, thread by thread: butterflies, points of each, and f(line, i, step, m) for
// each of them.
constexpr int first_points(int N) { return next_radix(N, 1) == N ? 1 : next_radix(N, 1); }
constexpr int first_butterflies(int N, int L, int NT) { return (L * (N / first_points(N)) + NT - 1) / NT; }
template <int N, int L, int NT, class F> __device__ __forceinline__ void first_points_of(F&& f) {
    constexpr int T = N / first_points(N), PER = first_butterflies(N, L, NT);
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const unsigned e = threadIdx.x + m * NT;
        if (PER * NT == L * T || e < L * T) f(e / T, e % T, ic<first_points(N) == 1 ? 1 : T>{}, m);
    }
}

template <int N, int L, int NT, bool ROWS, class Load, class Out, class Then>
__device__ __forceinline__ void fft_tile(float2* buf, Load&& load, Out&& out, Then&& then) {
    if constexpr (ROWS && Tile<N, L, ROWS>::kSingle) {
        short_rows<N, L, NT, false>(buf, load, out, false);
        then();
    } else {
        fft_stages<N, L, NT, ROWS, false, 1>(buf, load, out, then);
    }
}
template <int N, int L, int NT, bool ROWS, class Load, class Out>
__device__ __forceinline__ void fft_tile(float2* buf, Load&& load, Out&& out) {
    fft_tile<N, L, NT, ROWS>(buf, load, out, []() {});
}
template <int N, int L, int NT, bool ROWS, bool TO_LDS, class Load, class Out>
__device__ __forceinline__ void ifft_tile(float2* buf, Load&& load, Out&& out) {
    if constexpr (ROWS && Tile<N, L, ROWS>::kSingle) short_rows<N, L, NT, true>(buf, load, out, false);
    else ifft_stages<N, L, NT, ROWS, true, TO_LDS, last_stage(N)>(buf, load, out);
}
// Forward, mid() on the result, inverse.
template <int N, int L, int NT, bool ROWS, bool TO_LDS, class Load, class Mid, class Out, class Then>
__device__ __forceinline__ void fft_ifft_tile(float2* buf, Load&& load, Mid&& mid, Out&& out, Then&& then) {
    if constexpr (ROWS && Tile<N, L, ROWS>::kSingle) {
        then();
        short_rows<N, L, NT, false>(buf, load, mid, false);
        short_rows<N, L, NT, true>(buf, load, out, true);
    } else if constexpr (Tile<N, L, ROWS>::kSingle) {   // columns of one stage: all in registers
        using S = StageOf<N, L, NT, ROWS, 1>;
        float2 u[S::PER][N];
#pragma unroll
        for (int m = 0; m < S::PER; ++m)
            if (S::mine(m)) load(S::line(m), S::i(m), ic<1>{}, u[m], m);
        then();
#pragma unroll
        for (int m = 0; m < S::PER; ++m)
            if (S::mine(m)) {
                dft_r<N, false>(u[m]);
                mid(S::line(m), S::i(m), ic<1>{}, u[m], m);
                dft_r<N, true>(u[m]);
                out(S::line(m), S::i(m), ic<1>{}, u[m], m);
            }
    } else {
        fft_stages<N, L, NT, ROWS, true, 1>(buf, load, mid, then);
        ifft_stages<N, L, NT, ROWS, false, TO_LDS, Stage<N, last_stage(N)>::kBefore>(buf, load, out);
    }
}

}  // namespace gleam
