// Line transforms in LDS: X(k) = sum_j x(j) exp(-+ 2 pi i j k / n) of NL lines
// at once for any n <= 1024 (sign - forward, + inverse), by mixed-radix
// self-sorting stages (Stockham): a stage of radix r reads the r elements
// j + u n / r of a group, multiplies by the twiddles and stores their r-point
// transform at (j / Ns) Ns r + j mod Ns + u Ns, Ns the product of the earlier
// radices, so input and output are both in natural order.  n is split into
// radices 8, 4, 2, 3 and 5 (in registers); a prime factor p >= 7 takes a stage
// of direct sums (p / 2 term pairs for two outputs), before the others.
// A line of n costs about n sum(r) complex multiply-adds instead of n^2.
//
// Two LDS buffers per line are alternated, one barrier per stage.  Element i
// of a line lies at i + i / 8: the stride-8 and stride-64 stores of radix-8
// stages then fall into different banks.  The twiddles of a stage lie in the
// order its lanes read them, (u, j mod Ns), behind those of the earlier stages
// ((r - 1) Ns each, n - 1 in all): reading every n / (Ns r)-th entry of one
// table of n put a stage's reads into one to four banks.  Direct-sum stages
// read the table of n roots kept behind them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace flb {

constexpr int FFT_MAX_STAGES = 12;   // 1024 = 8 8 4 4; worst case below 2^10: 7 or fewer

struct FftPlan {
    int n, stages;
    int any;                     // 1: some stage is a direct sum
    int radix[FFT_MAX_STAGES];
};

inline FftPlan fft_plan(int n) {
    FftPlan p{};
    p.n = n;
    int e = 0, m = n;
    // direct sums first: the first stage needs no twiddles
    for (int f = 7; f <= n; f += 2)
        while (m % f == 0 && f % 3 != 0 && f % 5 != 0) {
            p.radix[p.stages++] = f;
            p.any = 1;
            m /= f;
        }
    while (m % 2 == 0) {
        m /= 2;
        ++e;
    }
    // radices 8 with fours for the rest of the power of two (a two only for
    // e = 1)
    while (e > 0) {
        const int r = (e == 1) ? 1 : (e % 3 == 0 ? 3 : 2);
        p.radix[p.stages++] = 1 << r;
        e -= r;
    }
    for (int f = 3; m > 1; f += 2)
        while (m % f == 0) {
            p.radix[p.stages++] = f;
            m /= f;
        }
    return p;
}

// Complex values of precision R in LDS and in work buffers.
template <typename R> struct Cx;
template <> struct Cx<double> {
    using T = double2;
    static __device__ __forceinline__ T make(double re, double im) { return make_double2(re, im); }
};
template <> struct Cx<float> {
    using T = float2;
    static __device__ __forceinline__ T make(float re, float im) { return make_float2(re, im); }
};
template <typename R> using cx_t = typename Cx<R>::T;

// Position of element i of a line, and the elements a line of n takes.
__host__ __device__ __forceinline__ int fft_pos(int i) { return i + (i >> 3); }
__host__ __device__ __forceinline__ int fft_ld(int n) { return n + (n >> 3) + 1; }
// Twiddle entries of a plan.
__host__ __device__ __forceinline__ int fft_twiddles(const FftPlan& p) {
    return p.any ? 2 * p.n : p.n;
}

// a / b for 0 <= a < 2^22 - 1, 1 <= b <= 2^22, with rb = 1.0f / b: a + 1/2 is
// exact, the reciprocal and the product each round by at most 2^-24 of their
// value, so the quotient errs by less than (a + 1/2) / b 2^-23, below the 1 / (2 b)
// that (a + 1/2) / b is at least from an integer.
__host__ __device__ __forceinline__ int fft_div(int a, float rb) {
    return (int)(((float)a + 0.5f) * rb);
}

// The twiddles of a plan, evaluated in FP64 and rounded to R: entry
// Ns - 1 + (u - 1) Ns + k = exp(-2 pi i u k / (Ns r)) of the stage after Ns,
// then, for direct sums, entry n + j = exp(-2 pi i j / n).  No barrier.
template <typename R>
__device__ __forceinline__ void twiddles(cx_t<R>* tw, const FftPlan& p) {
    for (int e = threadIdx.x; e < fft_twiddles(p); e += blockDim.x) {
        int num = e - p.n, den = p.n;   // exp(-2 pi i num / den)
        if (num < 0) {
            int Ns = 1, r = max(p.radix[0], 1);   // e's stage: the last that starts at or before it
            for (int s = 1, at = r; s < p.stages; ++s) {
                const int rs = p.radix[s];
                if (e >= at - 1) {
                    Ns = at;
                    r = rs;
                }
                at *= rs;
            }
            const int o = e - (Ns - 1), u = fft_div(o, 1.0f / (float)Ns);
            num = (u + 1) * (o - u * Ns);
            den = Ns * r;
        }
        double s, c;
        sincospi(2.0 * (double)num / (double)den, &s, &c);
        tw[e] = Cx<R>::make((R)c, (R)-s);
    }
}

template <typename R>
__device__ __forceinline__ cx_t<R> cx_mul(cx_t<R> a, cx_t<R> w) {
    return Cx<R>::make(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}
template <typename R>
__device__ __forceinline__ cx_t<R> cx_add(cx_t<R> a, cx_t<R> b) {
    return Cx<R>::make(a.x + b.x, a.y + b.y);
}
template <typename R>
__device__ __forceinline__ cx_t<R> cx_sub(cx_t<R> a, cx_t<R> b) {
    return Cx<R>::make(a.x - b.x, a.y - b.y);
}
// -i a (forward) or +i a (inverse)
template <typename R, bool INV>
__device__ __forceinline__ cx_t<R> cx_rot(cx_t<R> a) {
    return INV ? Cx<R>::make(-a.y, a.x) : Cx<R>::make(a.y, -a.x);
}

template <typename R, bool INV, int RAD>
__device__ __forceinline__ void fft_small(cx_t<R> (&x)[RAD]) {
    using C = cx_t<R>;
    if constexpr (RAD == 2) {
        const C a = x[0];
        x[0] = cx_add<R>(a, x[1]);
        x[1] = cx_sub<R>(a, x[1]);
    } else if constexpr (RAD == 3) {
        const R s3 = R(0.86602540378443864676);
        const C t = cx_add<R>(x[1], x[2]), d = cx_sub<R>(x[1], x[2]);
        const C m = Cx<R>::make(x[0].x - R(0.5) * t.x, x[0].y - R(0.5) * t.y);
        const C r = cx_rot<R, INV>(Cx<R>::make(s3 * d.x, s3 * d.y));
        x[0] = cx_add<R>(x[0], t);
        x[1] = cx_add<R>(m, r);
        x[2] = cx_sub<R>(m, r);
    } else if constexpr (RAD == 4) {
        const C a = cx_add<R>(x[0], x[2]), b = cx_sub<R>(x[0], x[2]);
        const C c = cx_add<R>(x[1], x[3]), d = cx_rot<R, INV>(cx_sub<R>(x[1], x[3]));
        x[0] = cx_add<R>(a, c);
        x[1] = cx_add<R>(b, d);
        x[2] = cx_sub<R>(a, c);
        x[3] = cx_sub<R>(b, d);
    } else if constexpr (RAD == 5) {
        const R c1 = R(0.30901699437494742410), c2 = R(-0.80901699437494742410);
        const R s1 = R(0.95105651629515357212), s2 = R(0.58778525229247312917);
        const C t1 = cx_add<R>(x[1], x[4]), t2 = cx_add<R>(x[2], x[3]);
        const C d1 = cx_sub<R>(x[1], x[4]), d2 = cx_sub<R>(x[2], x[3]);
        const C m1 = Cx<R>::make(x[0].x + c1 * t1.x + c2 * t2.x, x[0].y + c1 * t1.y + c2 * t2.y);
        const C m2 = Cx<R>::make(x[0].x + c2 * t1.x + c1 * t2.x, x[0].y + c2 * t1.y + c1 * t2.y);
        const C r1 = cx_rot<R, INV>(Cx<R>::make(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y));
        const C r2 = cx_rot<R, INV>(Cx<R>::make(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y));
        x[0] = cx_add<R>(x[0], cx_add<R>(t1, t2));
        x[1] = cx_add<R>(m1, r1);
        x[4] = cx_sub<R>(m1, r1);
        x[2] = cx_add<R>(m2, r2);
        x[3] = cx_sub<R>(m2, r2);
    } else {
        static_assert(RAD == 8, "radices in registers: 2, 3, 4, 5, 8");
        const R h = R(0.70710678118654752440);
        C e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
        fft_small<R, INV, 4>(e);
        fft_small<R, INV, 4>(o);
        const C q = cx_rot<R, INV>(o[1]), q3 = cx_rot<R, INV>(o[3]);
        o[1] = Cx<R>::make(h * (o[1].x + q.x), h * (o[1].y + q.y));
        o[2] = cx_rot<R, INV>(o[2]);
        o[3] = Cx<R>::make(h * (q3.x - o[3].x), h * (q3.y - o[3].y));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = cx_add<R>(e[u], o[u]);
            x[u + 4] = cx_sub<R>(e[u], o[u]);
        }
    }
}

template <typename R, bool INV, int RAD>
__device__ __forceinline__ void fft_stage(const cx_t<R>* __restrict__ a, cx_t<R>* __restrict__ b,
                                          const cx_t<R>* __restrict__ tw, int NL, int n, int Ns) {
    using C = cx_t<R>;
    const int m = n / RAD, ld = fft_ld(n);
    const float rm = 1.0f / (float)m, rN = 1.0f / (float)Ns;
    tw += Ns - 1;
    for (int t = threadIdx.x; t < NL * m; t += blockDim.x) {
        const int L = fft_div(t, rm), j = t - L * m;
        const int q = fft_div(j, rN), k = j - q * Ns;
        const C* src = a + L * ld;
        C x[RAD];
#pragma unroll
        for (int u = 0; u < RAD; ++u) x[u] = src[fft_pos(j + u * m)];
        if (Ns > 1) {
#pragma unroll
            for (int u = 1; u < RAD; ++u) {
                C w = tw[(u - 1) * Ns + k];
                if (INV) w.y = -w.y;
                x[u] = cx_mul<R>(x[u], w);
            }
        }
        fft_small<R, INV, RAD>(x);
        C* dst = b + L * ld;
        const int o = q * Ns * RAD + k;
#pragma unroll
        for (int u = 0; u < RAD; ++u) dst[fft_pos(o + u * Ns)] = x[u];
    }
}

// Any odd radix, of inputs that carry their twiddles already: outputs u and
// rad - u as direct sums.  Inputs v and rad - v enter as their sum (cosines)
// and difference (sines), which both outputs share: 4 multiply-adds and 3 LDS
// reads for two inputs and two outputs, against 16 and 8 of plain sums.  The
// reads are a serial chain when a line has few outputs per lane, so a line
// of a large prime is bound by their latency.  Modified-equilibrium runs with
// plain sums and one thread per four elements -> these and one per two: 32 x 71
// FP32 5.4 -> 3.7 us a step, 101 x 53 6.0 -> 4.1, 127 x 131 11.3 -> 5.8 (FP64
// 14.2 -> 7.9), 211 x 307 33 -> 19; the spectra of 19 fields of 101^3 take 825 us.
// Not unrolled: four terms at a time took the column kernel from 67 to 98
// registers, 449 against 398 us for the spectra of 128 x 96 x 80.
// tw: the n roots.
template <typename R, bool INV>
__device__ __forceinline__ void fft_stage_any(const cx_t<R>* __restrict__ a,
                                              cx_t<R>* __restrict__ b,
                                              const cx_t<R>* __restrict__ tw, int NL, int n, int Ns,
                                              int rad) {
    using C = cx_t<R>;
    const int m = n / rad, ld = fft_ld(n), h = rad / 2, w = m * (h + 1);
    const float rw = 1.0f / (float)w, rm = 1.0f / (float)m, rN = 1.0f / (float)Ns;
    for (int t = threadIdx.x; t < NL * w; t += blockDim.x) {
        const int L = fft_div(t, rw), i = t - L * w;
        const int u = fft_div(i, rm), j = i - u * m;     // outputs u and rad - u of group j
        const int q = fft_div(j, rN), k = j - q * Ns;
        const C* src = a + L * ld;
        const int inc = u * m;                           // < n
        const C x0 = src[fft_pos(j)];
        R cr = x0.x, ci = x0.y, sr = R(0), si = R(0);
        int idx = 0;
#pragma unroll 1
        for (int v = 1; v <= h; ++v) {
            idx += inc;
            if (idx >= n) idx -= n;
            const C x = src[fft_pos(j + v * m)], y = src[fft_pos(j + (rad - v) * m)];
            const C e = tw[idx];                         // (cos, -sin)
            cr = fma(x.x + y.x, e.x, cr);
            ci = fma(x.y + y.y, e.x, ci);
            sr = fma(x.y - y.y, e.y, sr);
            si = fma(x.x - y.x, e.y, si);
        }
        if (!INV) {
            sr = -sr;
            si = -si;
        }
        C* dst = b + L * ld;
        const int o = q * Ns * rad + k;
        dst[fft_pos(o + u * Ns)] = Cx<R>::make(cr + sr, ci - si);
        if (u > 0) dst[fft_pos(o + (rad - u) * Ns)] = Cx<R>::make(cr - sr, ci + si);
    }
}

// The twiddles of a stage of radix rad after Ns > 1, in place.  tw: the n roots.
template <typename R, bool INV>
__device__ __forceinline__ void fft_twist(cx_t<R>* a, const cx_t<R>* __restrict__ tw, int NL, int n,
                                          int Ns, int rad) {
    const int m = n / rad, ld = fft_ld(n), ts = m / Ns;
    const float rn = 1.0f / (float)n, rm = 1.0f / (float)m, rN = 1.0f / (float)Ns;
    for (int t = threadIdx.x; t < NL * n; t += blockDim.x) {
        const int L = fft_div(t, rn), i = t - L * n;
        const int v = fft_div(i, rm), j = i - v * m;
        const int k = j - fft_div(j, rN) * Ns;
        cx_t<R> w = tw[k * ts * v];                      // k ts v < n
        if (INV) w.y = -w.y;
        cx_t<R>* x = a + L * ld + fft_pos(i);
        *x = cx_mul<R>(*x, w);
    }
    __syncthreads();
}

// The NL lines of `a` (line L at a + L fft_ld(n)), already visible to the
// block, are transformed through `b` and back; returns the buffer that holds
// the result.  Ends with a barrier.  tw: the plan's twiddles.
template <typename R, bool INV>
__device__ __forceinline__ cx_t<R>* fft_lines(cx_t<R>* a, cx_t<R>* b, const cx_t<R>* tw, int NL,
                                              const FftPlan& p) {
    int Ns = 1;
    for (int s = 0; s < p.stages; ++s) {
        const int r = p.radix[s];
        switch (r) {
            case 2: fft_stage<R, INV, 2>(a, b, tw, NL, p.n, Ns); break;
            case 3: fft_stage<R, INV, 3>(a, b, tw, NL, p.n, Ns); break;
            case 4: fft_stage<R, INV, 4>(a, b, tw, NL, p.n, Ns); break;
            case 5: fft_stage<R, INV, 5>(a, b, tw, NL, p.n, Ns); break;
            case 8: fft_stage<R, INV, 8>(a, b, tw, NL, p.n, Ns); break;
            default:
                if (Ns > 1) fft_twist<R, INV>(a, tw + p.n, NL, p.n, Ns, r);
                fft_stage_any<R, INV>(a, b, tw + p.n, NL, p.n, Ns, r);
                break;
        }
        __syncthreads();
        Ns *= r;
        cx_t<R>* c = a;
        a = b;
        b = c;
    }
    return a;
}

}  // namespace flb
