// Modified-equilibrium (Swift) fluctuating LB, linearized about rest, D2Q9
// (Sec. IV.B, subsection on the modified-equilibrium model).
//
// State: the deviations delta f_i from the uniform rest state, stored
// f[i * V + x + nx y].  One step with index n:
//   pull       f_i(x) = S_i(x - c_i)
//   moments    m_a = sum_i T_ai f_i                        (App. B basis)
//   equilibrium (eq. meq-yeo, linearized)  m^eq = {rho, j_x, j_y, D, 0, 0, 0, 0, -D},
//              D = d(k) rho = 6 (cs2_0 - cs2) rho - 6 kappa rho0 lap_h rho,
//              i.e. d(k) = 6 (c_s^2(k) - cs2) with c_s^2(k) = cs2_0 + kappa rho0 Lambda(k),
//              Lambda(k) = (4/3)(2 - cos kx - cos ky) + (2/3)(1 - cos kx cos ky)
//              the symbol of -lap_h (9-point isotropic Laplacian)
//   relax      m*_a = m_a - lam_a (m_a - m^eq_a) + xi_a
//   back       S_{n+1,i} = w_i sum_a T_ai m*_a / N_a.
// Noise: the covariance Xi(k) = G - C G C^T that keeps the equal-time
// correlations of eq. f-correl-yeo stationary under the step.  p_xx, p_xy,
// q_x, q_y get white noise rho0 kT N_a lam (2 - lam) / cs2; the (e, eps) pair
// has the k-dependent block
//   Xi_ee = 12 rho0 kT lam_e (2 - lam_e)(2 - 3 c2),
//   Xi_eE = 12 rho0 kT (3 c2 - 1)(lam_e + lam_g - lam_e lam_g),
//   Xi_EE = 12 rho0 kT lam_g (2 - lam_g)(5 - 3 c2),      c2 = c_s^2(k),
// whose small-rate limit is eq. noise-yeo (the (e, eps) entry at half its
// printed value: the value for which Xi is a covariance wherever the
// equilibrium populations are non-negative).  That pair is drawn as white
// normals z_e, z_eps (the site's Philox normals 0 and 5), transformed, mixed
// by the lower Cholesky factor of the block at every k, and transformed back:
//   k_meq_noise_x   normals of a row, DFT along x
//   k_meq_filter    DFT along y, Cholesky mix, inverse DFT (adjacent columns)
//   k_meq_noise_ix  inverse DFT along x
// The two white fields are real, and so are the two filtered ones (the factor
// is real and even in k): a row carries both as the real and imaginary part
// of one complex line, and only the half spectra 0 <= kx <= nx / 2 of e and
// eps are kept and transformed along y.  The filtered pair is scaled to unit
// amplitude until the last pass, so that neither field is rounded at the
// other's size.
// The noise does not depend on the state, so a launch of these three
// kernels draws and filters the noise of a batch of consecutive steps: at
// small lattices a single step's lines are far fewer blocks than the chip has
// CUs.
// Lines sit in LDS and are transformed in place where the extent is a power of
// two, else by the staged passes of fft.h (any extent up to 1024).  In place
// because a row of few steps is a chain of latencies: the staged passes look up
// their plan and twiddles by stage (512^2 FP32, one step: rows 6.9 us in place,
// 9.5 staged), and because one padded buffer leaves room for twice the lines
// (1024^2, 16 steps: 98 against 121 us).  The transforms are in the
// state's precision (R = float or double; twiddles and Cholesky factors formed
// in FP64 and rounded once) or, some of them in FP32 runs, in FP64 (MQ_THIN); the
// spectra and the filtered fields in the state's.  Then k_meq_step applies the step.
//
// 1024^2 FP32, noise per step of a 16-step launch: rows 9.0 us (6.1 if they were
// FP32), columns 11.1 us, rows back 4.5 us; 11.6, 20.3 and 11.6 us with two
// full spectra.  200 x 150 FP64, one step per call and launch: 31 us
// when extents that are not powers of two took n^2 direct sums; 6.6 us a step
// with several steps per launch (modeq_steps).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.h"
#include "fft.h"
#include "internal.h"
#include "philox.h"

namespace flb {

namespace {

constexpr int MQ_THREADS = 1024;     // of the staged line transforms, at most
constexpr int MQ_P2_THREADS = 256;   // of the in-place power-of-two passes
// FP32 noise: two real fields in one complex line round at sqrt 2 times the error
// of a line each (their independent errors at k and -k averaged out), so some
// passes run in FP64, as few as keep the rms error below that of two full
// spectra: the rows of a power of two, and rows and columns where nx is small
// and one direction carries the whole error.  Relative rms error of e, two
// spectra / all FP32 / these: 1024^2 2.44e-7 / 2.69e-7 / 2.35e-7, 128^2 2.17 /
// 2.26 / 1.99, 32 x 1024 2.12 / 2.33 / 1.19, 3 x 1024 1.68 / 1.94 / 0.95; long
// rows that are no power of two were direct sums and stay FP32 (200 x 150 5.55 /
// 2.18).  1024^2, 16 steps: the rows take 144 us, 98 in FP32.
constexpr int MQ_THIN = 64;

// tw[j] = exp(-2 pi i j / n), evaluated in FP64 and rounded to R.
template <typename R>
__device__ __forceinline__ void roots(cx_t<R>* tw, int n) {
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        double s, c;
        sincospi(2.0 * (double)j / (double)n, &s, &c);
        tw[j] = Cx<R>::make((R)c, (R)-s);
    }
}

__device__ __forceinline__ int log2i(int n) { return 31 - __clz(n); }

// Position of element j in the bit-reversed order of a 2^logn line.
__device__ __forceinline__ int brev(int j, int logn) {
    return logn == 0 ? 0 : (int)(__brev((unsigned)j) >> (32 - logn));
}

// Element i of an in-place line, and the elements a line takes: PAD as in fft.h,
// so that the elements of a pass fall into different banks.
template <bool PAD>
__host__ __device__ __forceinline__ int p2_pos(int i) { return PAD ? fft_pos(i) : i; }
template <bool PAD>
__host__ __device__ __forceinline__ int p2_ld(int n) { return PAD ? fft_ld(n) : n; }

// One in-place pass over lines of n = 2^logn elements: LR = log2 RAD radix-2
// stages at once, of the groups of RAD elements h = 2^lh apart.  The RAD-point transform is one of fft_small with one twiddle
// exp(-+ 2 pi i u pos / (RAD h)) per element u, before it in a decimation in
// time (elements in bit-reversed order on the way in), behind it in a
// decimation in frequency (on the way out).  Against a twiddle in each of the
// stages a third of the multiplications, each of which rounds.  tw: the n roots.
template <typename R, bool INV, bool DIF, bool PAD, int LR>
__device__ __forceinline__ void p2_pass(cx_t<R>* b, const cx_t<R>* __restrict__ tw, int NL, int n,
                                        int logn, int lh) {
    constexpr int RAD = 1 << LR;
    constexpr int br[8] = {0, RAD / 2, RAD >= 8 ? 2 : 1, RAD >= 8 ? 6 : 3, 1, 5, 3, 7};
    const int lg = logn - LR, h = 1 << lh, sh = lg - lh;
    for (int t = threadIdx.x; t < NL << lg; t += blockDim.x) {
        const int L = t >> lg, q = t - (L << lg), pos = q & (h - 1);
        const int i0 = ((q >> lh) << (lh + LR)) + pos;
        cx_t<R>* line = b + L * p2_ld<PAD>(n);
        cx_t<R> x[RAD];
#pragma unroll
        for (int u = 0; u < RAD; ++u) x[u] = line[p2_pos<PAD>(i0 + ((DIF ? u : br[u]) << lh))];
        auto turn = [&] {
            if (lh == 0) return;   // uniform
#pragma unroll
            for (int u = 1; u < RAD; ++u) {
                cx_t<R> w = tw[(u * pos) << sh];
                if (INV) w.y = -w.y;
                x[u] = cx_mul<R>(x[u], w);
            }
        };
        if constexpr (!DIF) turn();
        fft_small<R, INV, RAD>(x);
        if constexpr (DIF) turn();
#pragma unroll
        for (int u = 0; u < RAD; ++u) line[p2_pos<PAD>(i0 + ((DIF ? br[u] : u) << lh))] = x[u];
    }
    __syncthreads();
}

// In place, the NL lines of b (n = 2^logn), each in bit-reversed order, become
// their transforms in natural order.
template <typename R, bool INV, bool PAD>
__device__ __forceinline__ void fft_lines_dit(cx_t<R>* b, const cx_t<R>* __restrict__ tw, int NL,
                                              int n, int logn) {
    int lh = 0;
    for (; lh + 3 <= logn; lh += 3) p2_pass<R, INV, false, PAD, 3>(b, tw, NL, n, logn, lh);
    if (logn - lh == 2) p2_pass<R, INV, false, PAD, 2>(b, tw, NL, n, logn, lh);
    if (logn - lh == 1) p2_pass<R, INV, false, PAD, 1>(b, tw, NL, n, logn, lh);
}
// From natural to bit-reversed order: the same passes the other way round.
template <typename R, bool INV, bool PAD>
__device__ __forceinline__ void fft_lines_dif(cx_t<R>* b, const cx_t<R>* __restrict__ tw, int NL,
                                              int n, int logn) {
    int lh = logn / 3 * 3;
    if (logn - lh == 1) p2_pass<R, INV, true, PAD, 1>(b, tw, NL, n, logn, lh);
    if (logn - lh == 2) p2_pass<R, INV, true, PAD, 2>(b, tw, NL, n, logn, lh);
    for (lh -= 3; lh >= 0; lh -= 3) p2_pass<R, INV, true, PAD, 3>(b, tw, NL, n, logn, lh);
}

// Lower Cholesky factor of the (e, eps) noise block at wavenumber (kx, ky),
// given cos kx and cos ky, in FP64.
__device__ __forceinline__ void meq_chol(const ModEqArgs& a, double cx, double cy, double& l11,
                                         double& l21, double& l22) {
    const double pre = 12.0 * a.rho0 * a.kT;
    const double le = a.rate_bulk, lg = a.rate_ghost;
    const double lap = (4.0 / 3.0) * (2.0 - cx - cy) + (2.0 / 3.0) * (1.0 - cx * cy);
    const double c2 = a.cs2_0 + a.kappa * a.rho0 * lap;
    const double see = pre * le * (2.0 - le) * (2.0 - 3.0 * c2);
    const double sep = pre * (3.0 * c2 - 1.0) * (le + lg - le * lg);
    const double spp = pre * lg * (2.0 - lg) * (5.0 - 3.0 * c2);
    l11 = sqrt(fmax(see, 0.0));
    l21 = l11 > 0.0 ? sep / l11 : 0.0;
    l22 = sqrt(fmax(spp - l21 * l21, 0.0));
}

// Amplitudes of the filtered e and eps noise: the square roots of the largest
// diagonal entries of the block (at k = 0, where c2 is smallest).
__device__ __forceinline__ void meq_scales(const ModEqArgs& a, double& se, double& sp) {
    const double pre = 12.0 * a.rho0 * a.kT;
    const double le = a.rate_bulk, lg = a.rate_ghost;
    se = sqrt(fmax(pre * le * (2.0 - le) * (2.0 - 3.0 * a.cs2_0), 0.0));
    sp = sqrt(fmax(pre * lg * (2.0 - lg) * (5.0 - 3.0 * a.cs2_0), 0.0));
    if (!(se > 0.0)) se = 1.0;
    if (!(sp > 0.0)) sp = 1.0;
}

// Dynamic LDS of the noise kernels: two buffers of NL lines, then the
// twiddles (either precision).
extern __shared__ __align__(16) unsigned char lds_mq[];

// Half spectra of step b: e at W + 2 V b, eps hx ny values behind it, each
// (y, kx), kx = 0 .. nx / 2.  A turn is NL rows of one step.
template <typename Real, typename A, bool P2>
__global__ __launch_bounds__(MQ_THREADS) void k_meq_noise_x(ModEqArgs a, FftPlan p, int NL,
                                                            uint32_t step0, int nb,
                                                            cx_t<Real>* __restrict__ W) {
    using C = cx_t<A>;
    using S = cx_t<Real>;   // as stored
    const int n = a.nx, hx = n / 2 + 1, ld = fft_ld(n), logn = log2i(n);
    const size_t V = (size_t)a.nx * a.ny, H = (size_t)hx * a.ny;
    C* buf = (C*)lds_mq;
    C* alt = buf + NL * ld;
    C* tw = P2 ? alt : alt + NL * ld;
    if constexpr (P2) roots<A>(tw, n);
    else twiddles<A>(tw, p);
    const float rn = 1.0f / (float)n, rh = 1.0f / (float)hx;
    const uint32_t groups = (uint32_t)((a.ny + NL - 1) / NL);
    for (uint32_t g = blockIdx.x; g < groups * (uint32_t)nb; g += gridDim.x) {
        const uint32_t b = g / groups;
        const int y0 = (int)(g - b * groups) * NL, nl = min(NL, a.ny - y0);
        for (int t = threadIdx.x; t < NL * n; t += blockDim.x) {
            const int L = fft_div(t, rn), x = t - L * n;
            C v = Cx<A>::make(A(0), A(0));
            if (L < nl) {
                Real z[6];
                site_normals<3, Real>((uint32_t)(x + n * (y0 + L)), step0 + b, 0u, 0u, a.k0, a.k1, z);
                v = Cx<A>::make((A)z[0], (A)z[5]);
            }
            buf[L * ld + fft_pos(P2 ? brev(x, logn) : x)] = v;
        }
        __syncthreads();
        const C* z = buf;
        if constexpr (P2) fft_lines_dit<A, false, true>(buf, tw, NL, n, logn);
        else z = fft_lines<A, false>(buf, alt, tw, NL, p);
        S* out = W + (size_t)b * 2 * V + (size_t)y0 * hx;
        for (int t = threadIdx.x; t < nl * hx; t += blockDim.x) {
            const int L = fft_div(t, rh), k = t - L * hx;
            const C u = z[L * ld + fft_pos(k)], v = z[L * ld + fft_pos(k == 0 ? 0 : n - k)];
            out[t] = Cx<Real>::make((Real)(A(0.5) * (u.x + v.x)), (Real)(A(0.5) * (u.y - v.y)));
            out[H + t] = Cx<Real>::make((Real)(A(0.5) * (u.y + v.y)), (Real)(A(0.5) * (v.x - u.x)));
        }
        __syncthreads();   // the result is read before the next turn's loads
    }
}

// NC adjacent columns kx of one step per block.  LDS lines: e of the columns,
// then eps.  P2 (ny a power of two): in-place passes, decimation in
// frequency forward and in time back, so that position j holds wavenumber
// brev(j) in between and no line is permuted; at 1024 they take 177 us per
// 16 steps where the staged passes, with two buffers and more index
// arithmetic, take 311.  The lines are not padded: in FP64 two padded columns
// of 1024 leave one block per CU (411 against 305 us).
template <typename Real, typename A, bool P2>
__global__ __launch_bounds__(P2 ? MQ_P2_THREADS : MQ_THREADS) void k_meq_filter(
    ModEqArgs a, FftPlan p, int NC, cx_t<Real>* __restrict__ W) {
    using C = cx_t<A>;
    using S = cx_t<Real>;   // as stored
    // neighbouring column groups share cache lines: same XCD, one L2
    const uint32_t lin = xcd_remap(blockIdx.x + blockIdx.y * gridDim.x, gridDim.x * gridDim.y);
    const int n = a.ny, hx = a.nx / 2 + 1, ld = P2 ? n : fft_ld(n), logn = log2i(n);
    const uint32_t step = lin / gridDim.x;
    const int c0 = (int)(lin - step * gridDim.x) * NC, nc = min(NC, hx - c0);
    const size_t V = (size_t)a.nx * a.ny, H = (size_t)hx * n;
    S* base = W + (size_t)step * 2 * V + c0;
    C* buf = (C*)lds_mq;
    C* alt = buf + 2 * NC * ld;
    C* tw = P2 ? alt : alt + 2 * NC * ld;
    if constexpr (P2) roots<A>(tw, n);
    else twiddles<A>(tw, p);
    const float rc = 1.0f / (float)NC, rn = 1.0f / (float)nc;
    auto pos = [](int i) { return P2 ? i : fft_pos(i); };
    for (int t = threadIdx.x; t < NC * n; t += blockDim.x) {
        const int j = fft_div(t, rc), c = t - j * NC;
        C e = Cx<A>::make(A(0), A(0)), q = e;
        if (c < nc) {
            const S es = base[(size_t)j * hx + c], qs = base[H + (size_t)j * hx + c];
            e = Cx<A>::make((A)es.x, (A)es.y);
            q = Cx<A>::make((A)qs.x, (A)qs.y);
        }
        buf[c * ld + pos(j)] = e;
        buf[(NC + c) * ld + pos(j)] = q;
    }
    __syncthreads();
    C* z = buf;
    if constexpr (P2) fft_lines_dif<A, false, false>(z, tw, 2 * NC, n, logn);
    else z = fft_lines<A, false>(buf, alt, tw, 2 * NC, p);
    double se, sp;
    meq_scales(a, se, sp);
    for (int t = threadIdx.x; t < nc * n; t += blockDim.x) {
        const int j = fft_div(t, rn), c = t - j * nc;
        double sn, cx, cy, d11, d21, d22;
        sincospi(2.0 * (double)(c0 + c) / (double)a.nx, &sn, &cx);
        if constexpr (P2) cy = (double)tw[brev(j, logn)].x;
        else sincospi(2.0 * (double)j / (double)n, &sn, &cy);
        meq_chol(a, cx, cy, d11, d21, d22);
        const A l11 = (A)(d11 / se), l21 = (A)(d21 / sp), l22 = (A)(d22 / sp);
        C* pe = z + c * ld + pos(j);
        C* pq = pe + NC * ld;
        const C e = *pe, q = *pq;
        *pe = Cx<A>::make(l11 * e.x, l11 * e.y);
        *pq = Cx<A>::make(l21 * e.x + l22 * q.x, l21 * e.y + l22 * q.y);
    }
    __syncthreads();
    if constexpr (P2) fft_lines_dit<A, true, false>(z, tw, 2 * NC, n, logn);
    else z = fft_lines<A, true>(z, z == buf ? alt : buf, tw, 2 * NC, p);
    for (int t = threadIdx.x; t < nc * n; t += blockDim.x) {
        const int j = fft_div(t, rn), c = t - j * nc;
        const C e = z[c * ld + pos(j)], q = z[(NC + c) * ld + pos(j)];
        base[(size_t)j * hx + c] = Cx<Real>::make((Real)e.x, (Real)e.y);
        base[H + (size_t)j * hx + c] = Cx<Real>::make((Real)q.x, (Real)q.y);
    }
}

// X(k) = E(k) + i P(k), k = 0 .. nx - 1, from the half spectra (E(n - k) =
// conj E(k)); its inverse transform is xi_e + i xi_eps.
template <typename Real, bool P2>
__global__ __launch_bounds__(MQ_THREADS) void k_meq_noise_ix(ModEqArgs a, FftPlan p, int NL, int nb,
                                                             const cx_t<Real>* __restrict__ W,
                                                             Real* __restrict__ xi) {
    using C = cx_t<Real>;
    const int n = a.nx, hx = n / 2 + 1, ld = fft_ld(n), logn = log2i(n);
    const size_t V = (size_t)a.nx * a.ny, H = (size_t)hx * a.ny;
    C* buf = (C*)lds_mq;
    C* alt = buf + NL * ld;
    C* tw = P2 ? alt : alt + NL * ld;
    if constexpr (P2) roots<Real>(tw, n);
    else twiddles<Real>(tw, p);
    double se, sp;
    meq_scales(a, se, sp);
    const Real fe = (Real)(se / (double)V), fp = (Real)(sp / (double)V);
    const float rn = 1.0f / (float)n;
    const uint32_t groups = (uint32_t)((a.ny + NL - 1) / NL);
    for (uint32_t g = blockIdx.x; g < groups * (uint32_t)nb; g += gridDim.x) {
        const uint32_t b = g / groups;
        const int y0 = (int)(g - b * groups) * NL, nl = min(NL, a.ny - y0);
        const C* in = W + (size_t)b * 2 * V + (size_t)y0 * hx;
        for (int t = threadIdx.x; t < NL * n; t += blockDim.x) {
            const int L = fft_div(t, rn), k = t - L * n;
            C v = Cx<Real>::make(Real(0), Real(0));
            if (L < nl) {
                const int h = k < hx ? k : n - k;
                const C e = in[L * hx + h], q = in[H + L * hx + h];
                v = k < hx ? Cx<Real>::make(e.x - q.y, e.y + q.x)
                           : Cx<Real>::make(e.x + q.y, q.x - e.y);
            }
            buf[L * ld + fft_pos(P2 ? brev(k, logn) : k)] = v;
        }
        __syncthreads();
        const C* z = buf;
        if constexpr (P2) fft_lines_dit<Real, true, true>(buf, tw, NL, n, logn);
        else z = fft_lines<Real, true>(buf, alt, tw, NL, p);
        Real* out = xi + (size_t)b * 2 * V + (size_t)y0 * n;
        for (int t = threadIdx.x; t < nl * n; t += blockDim.x) {
            const int L = fft_div(t, rn), x = t - L * n;
            const C v = z[L * ld + fft_pos(x)];
            out[t] = v.x * fe;
            out[V + t] = v.y * fp;
        }
        __syncthreads();
    }
}

// v modulo n for the extents here (|v| < 2^12): a tile is many periods of a thin
// lattice, so one period at a time (1 x 900: 64 turns) took 3 us of a step.  v + 1/2
// is at least 1 / (2 n) from a multiple of n, beyond the rounding of the quotient.
__device__ __forceinline__ int wrap_mod(int v, int n) {
    const float q = floorf(((float)v + 0.5f) * __builtin_amdgcn_rcpf((float)n));
    return v - (int)q * n;
}

// T steps in one launch on tiles of TX x TY sites (as multistep.h does for the
// force-based fluid): step s is computed on the tile plus a halo of 2 (T - 1 -
// s) sites, two being the reach of a step (a pull and the density's
// neighbours), and its populations stay in LDS for step s + 1.
template <int T, int TX, int TY>
struct MeqTile {
    static constexpr int w(int s) { return TX + 4 * (T - 1 - s); }
    static constexpr int h(int s) { return TY + 4 * (T - 1 - s); }
    static constexpr int NT = (w(0) * h(0) + 63) / 64 * 64;
    static constexpr int NR = (w(0) + 2) * (h(0) + 2);
    static constexpr int NS0 = T > 1 ? 9 * w(0) * h(0) : 1;
    static constexpr int NS1 = T > 2 ? 9 * w(1) * h(1) : 1;
};

template <typename Real, int T, int TX, int TY, int S>
struct MeqStep {
    using L = Lattice<0>;
    using MT = MeqTile<T, TX, TY>;
    using M = Moments<0, Real>;
    static constexpr int W = MT::w(S), HH = MT::h(S), N = W * HH, Q = L::Q, NT = MT::NT;
    static constexpr int B = 2 * (T - 1 - S), SX = W + 2;

    static __device__ __forceinline__ bool place(const Geom& g, int x0, int y0, int& lx, int& ly,
                                                 int& x, int& y) {
        const int l = (int)threadIdx.x;
        ly = l / W;
        lx = l - ly * W;
        x = wrap_mod(x0 - B + lx, g.nx);
        y = wrap_mod(y0 - B + ly, g.ny);
        return l < N;
    }
    // the site's normals z_1 .. z_4 and its filtered noise
    static __device__ __forceinline__ void draw(const ModEqArgs& a, const Geom& g, int x0, int y0,
                                                uint32_t step, const Real* __restrict__ xi,
                                                const double2* tab, Real (&z)[6]) {
        int lx, ly, x, y;
        if (!xi || !place(g, x0, y0, lx, ly, x, y)) return;
        const uint32_t site = (uint32_t)(x + g.nx * y);
        const Real* f = xi + (size_t)S * 2 * g.V;
        const Real e = f[site], p = f[g.V + site];
        site_normals<3, Real>(site, step + S, 0u, 0u, a.k0, a.k1, z, tab);
        z[0] = e;
        z[5] = p;
    }
    // f: the site's streamed populations; rs: with S = 0, the density on the
    // region and a one-site ring; src (S > 0): the populations of step S - 1,
    // whose region is two sites wider
    static __device__ __forceinline__ void run(const ModEqArgs& a, const Geom& g, int x0, int y0,
                                               const Real* src, Real* dst, Real* rs, Real (&f)[Q],
                                               const Real* z, bool noise,
                                               Real* __restrict__ fout) {
        constexpr int PW = W + 4, PN = PW * (HH + 4);
        int lx, ly, x, y;
        const bool in = place(g, x0, y0, lx, ly, x, y);
        if constexpr (S > 0) {
            auto pulled = [&](int px, int py, Real (&h)[Q]) {
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    h[i] = src[i * PN + (py - L::cy[i]) * PW + px - L::cx[i]];
            };
            if (in) pulled(lx + 2, ly + 2, f);
            for (int l = threadIdx.x; l < SX * (HH + 2); l += NT) {
                const int ry = l / SX, rx = l - ry * SX;
                Real h[Q], acc = Real(0);
                pulled(rx + 1, ry + 1, h);
#pragma unroll
                for (int i = 0; i < Q; ++i) acc += h[i];
                rs[l] = acc;
            }
            __syncthreads();
        }
        if (!in) return;
        Real m[Q];
        M::forward(f, m);
        const int c = (ly + 1) * SX + lx + 1;
        Real lap = Real(0);
#pragma unroll
        for (int i = 1; i < Q; ++i)
            lap += Real(L::w[i]) * (rs[c + L::cy[i] * SX + L::cx[i]] - rs[c]);
        lap *= Real(6);
        const Real D = Real(6.0 * (a.cs2_0 - 1.0 / 3.0)) * m[0] - Real(6.0 * a.kappa * a.rho0) * lap;
        const Real le = Real(a.rate_bulk), ls = Real(a.rate_shear), lg = Real(a.rate_ghost);
        m[3] -= le * (m[3] - D);
        m[4] -= ls * m[4];
        m[5] -= ls * m[5];
        m[6] -= lg * m[6];
        m[7] -= lg * m[7];
        m[8] -= lg * (m[8] + D);
        if (noise) {
            m[3] += z[0];
            m[4] += Real(a.amp[0]) * z[1];
            m[5] += Real(a.amp[1]) * z[2];
            m[6] += Real(a.amp[2]) * z[3];
            m[7] += Real(a.amp[3]) * z[4];
            m[8] += z[5];
        }
        M::inverse(m, f);
        if constexpr (S + 1 < T) {
#pragma unroll
            for (int i = 0; i < Q; ++i) dst[i * N + (int)threadIdx.x] = f[i];
        } else if (x0 + lx < g.nx && y0 + ly < g.ny) {
            const uint32_t site = (uint32_t)(x + g.nx * y);
#pragma unroll
            for (int i = 0; i < Q; ++i) plane_st(fout + (size_t)i * g.V, site, f[i]);
        }
    }
};

template <typename Real, int T, int TX, int TY>
__global__ __launch_bounds__((MeqTile<T, TX, TY>::NT)) void k_meq_step(
    ModEqArgs a, Geom g, const Real* __restrict__ fin, Real* __restrict__ fout, uint32_t step,
    const Real* __restrict__ xi) {
    using L = Lattice<0>;
    using MT = MeqTile<T, TX, TY>;
    using S0 = MeqStep<Real, T, TX, TY, 0>;
    constexpr int Q = L::Q, SX = S0::SX, SY = S0::HH + 2;
    constexpr int NRING = MT::NR - S0::N;   // two rows of SX, two columns of HH
    static_assert(NRING <= MT::NT, "one ring site per thread at most");
    __shared__ Real rs[MT::NR];
    __shared__ Real s0[MT::NS0];
    __shared__ Real s1[MT::NS1];
    const uint32_t lin = xcd_remap(blockIdx.x, g.nblocks);
    const int by = (int)(lin / (uint32_t)g.nbx);
    const int x0 = (int)(lin - (uint32_t)by * (uint32_t)g.nbx) * TX, y0 = by * TY;
    // density of the pulled populations on the region and a one-site ring:
    // each thread pulls its own site (a periodic image past a ragged edge) and
    // keeps the populations, the first NRING threads pull the ring
    int lx, ly, x, y;
    const bool in = S0::place(g, x0, y0, lx, ly, x, y);
    Real f[Q], h[Q];
    if (in) pull<0, Real>(fin, x, y, 0, g, f);
    int rx = 0, ry = 0;
    if ((int)threadIdx.x < NRING) {
        const int r = (int)threadIdx.x;
        if (r < 2 * SX) {
            rx = r < SX ? r : r - SX;
            ry = r < SX ? 0 : SY - 1;
        } else {
            const int c = r - 2 * SX;   // 0 .. 2 HH - 1
            rx = c < S0::HH ? 0 : SX - 1;
            ry = 1 + (c < S0::HH ? c : c - S0::HH);
        }
        pull<0, Real>(fin, wrap_mod(x0 - S0::B - 1 + rx, g.nx), wrap_mod(y0 - S0::B - 1 + ry, g.ny), 0,
                      g, h);
    }
    const double2* tab = noise_table<Real, MT::NT>();
    Real z[T][6];   // drawn while the populations are in flight
    S0::draw(a, g, x0, y0, step, xi, tab, z[0]);
    if constexpr (T > 1) MeqStep<Real, T, TX, TY, 1>::draw(a, g, x0, y0, step, xi, tab, z[1]);
    if constexpr (T > 2) MeqStep<Real, T, TX, TY, 2>::draw(a, g, x0, y0, step, xi, tab, z[2]);
    if (in) {
        Real s = Real(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) s += f[i];
        rs[(ly + 1) * SX + lx + 1] = s;
    }
    if ((int)threadIdx.x < NRING) {
        Real s = Real(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) s += h[i];
        rs[ry * SX + rx] = s;
    }
    __syncthreads();
    const bool noise = xi != nullptr;
    S0::run(a, g, x0, y0, nullptr, s0, rs, f, z[0], noise, fout);
    if constexpr (T > 1) {
        __syncthreads();
        MeqStep<Real, T, TX, TY, 1>::run(a, g, x0, y0, s0, s1, rs, f, z[1], noise, fout);
    }
    if constexpr (T > 2) {
        __syncthreads();
        MeqStep<Real, T, TX, TY, 2>::run(a, g, x0, y0, s1, s0, rs, f, z[2], noise, fout);
    }
}

// Analysis: the nine moment fields m_a(x) = sum_i T_ai f_i(x) of the pulled
// populations, in FP64, m[a * V + site].
template <typename Real>
__global__ __launch_bounds__(256) void k_meq_moments(Geom g, const Real* __restrict__ fin,
                                                     double* __restrict__ m) {
    using L = Lattice<0>;
    const uint32_t site = blockIdx.x * 256u + threadIdx.x;
    if (site >= g.V) return;
    const int x = (int)(site % (uint32_t)g.nx), y = (int)(site / (uint32_t)g.nx);
    Real f[L::Q];
    pull<0, Real>(fin, x, y, 0, g, f);
#pragma unroll
    for (int q = 0; q < L::Q; ++q) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
            if (L::T[q][i] != 0) s += (double)L::T[q][i] * (double)f[i];
        m[(size_t)q * g.V + site] = s;
    }
}

}  // namespace

hipError_t launch_modeq_moments(const ModEqArgs& a, int prec, const void* fin, double* m,
                                hipStream_t st) {
    Geom g{};
    g.nx = a.nx;
    g.ny = a.ny;
    g.nz = 1;
    g.V = (uint32_t)((size_t)a.nx * a.ny);
    const dim3 grid((g.V + 255) / 256);
    if (prec == 0)
        hipLaunchKernelGGL(k_meq_moments<float>, grid, dim3(256), 0, st, g, (const float*)fin, m);
    else
        hipLaunchKernelGGL(k_meq_moments<double>, grid, dim3(256), 0, st, g, (const double*)fin, m);
    return hipGetLastError();
}

size_t modeq_work_bytes(int nx, int ny, int prec) {
    const size_t V = (size_t)nx * ny;
    const size_t r = prec == 0 ? sizeof(float) : sizeof(double);
    return 2 * V * (2 * r) + 2 * V * r;
}

namespace {

// Threads for `lines` lines: one per four elements, per two where a stage of
// direct sums has an output pair for each; up to one per element while the
// blocks leave the chip two wavefronts per SIMD, which then wait for each
// thread's twiddles and normals.
int mq_block(int lines, const FftPlan& p, size_t blocks) {
    int per = p.any ? 2 : 4;
    while (per > 1 && blocks * ((size_t)lines * p.n / per) < 2048 * 64) per /= 2;
    return std::min(MQ_THREADS, std::max(64, (lines * p.n / per + 63) / 64 * 64));
}

bool is_pow2(int n) { return (n & (n - 1)) == 0; }

size_t mq_lds(int lines, const FftPlan& p, size_t csize) {
    return (2 * (size_t)lines * fft_ld(p.n) + fft_twiddles(p)) * csize;
}
// One buffer of padded lines, transformed in place, and the roots.
size_t mq_lds_p2(int lines, int n, size_t csize) {
    return ((size_t)lines * fft_ld(n) + n) * csize;
}

}  // namespace

ModEqNoiseShape modeq_noise_shape(const ModEqArgs& a, int prec, int nb) {
    const size_t csize = prec == 0 ? sizeof(float2) : sizeof(double2);
    const FftPlan px = fft_plan(a.nx), py = fft_plan(a.ny);
    ModEqNoiseShape s;
    // rows per block: up to 2048 elements (512 threads) and 48 KB, fewer
    // where that leaves less than 1024 turns
    auto row_bytes = [&](int NL, size_t size) {
        return is_pow2(a.nx) ? mq_lds_p2(NL, a.nx, size) : mq_lds(NL, px, size);
    };
    auto rows = [&](size_t size, size_t* lds) {
        int NL = 16;
        while (NL > 1 && (NL * a.nx > 2048 || row_bytes(NL, size) > 49152 ||
                          (size_t)a.ny * nb < 1024 * (size_t)NL))
            NL /= 2;
        *lds = row_bytes(NL, size);
        return NL;
    };
    s.x64 = prec != 0 || is_pow2(a.nx) || a.nx <= MQ_THIN;
    s.NX = rows(s.x64 ? sizeof(double2) : csize, &s.lds_x);
    s.NI = rows(csize, &s.lds_i);
    // columns per block: two for the in-place passes (four columns halve the
    // resident blocks, 212 us at 1024^2), up to four of at most 4096 elements
    // for the staged ones as far as their lines and twiddles fit the LDS (931
    // elements with a direct sum, FP64, two columns: 164 KB); fewer where that
    // leaves less than 512 blocks
    const int hx = a.nx / 2 + 1;
    const bool p2 = is_pow2(a.ny);
    s.y64 = prec != 0 || a.nx <= MQ_THIN;
    const size_t ysize = s.y64 ? sizeof(double2) : csize;
    auto cols = [&](int NC) {
        return p2 ? (2 * (size_t)NC + 1) * a.ny * ysize : mq_lds(2 * NC, py, ysize);
    };
    s.NC = p2 ? 2 : 4;
    while (s.NC > 1 && ((!p2 && 2 * s.NC * a.ny > 4096) || cols(s.NC) > LDS_BYTES ||
                        hx * nb < 512 * s.NC))
        s.NC /= 2;
    s.lds_cols = cols(s.NC);
    return s;
}

namespace {

template <typename K>
hipError_t mq_lds_limit(K kernel, size_t lds) {
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds);
}

template <typename Real>
hipError_t launch_noise_t(const ModEqArgs& a, uint32_t step0, int nb, void* Wv, Real* xi,
                          hipStream_t st) {
    using C = cx_t<Real>;
    C* W = (C*)Wv;
    const FftPlan px = fft_plan(a.nx), py = fft_plan(a.ny);
    const ModEqNoiseShape sh = modeq_noise_shape(a, sizeof(Real) == 4 ? 0 : 1, nb);
    const bool xp2 = is_pow2(a.nx), yp2 = is_pow2(a.ny);
    // a single row of 964 or more FP64 elements with a direct sum takes up to 70 KB
    auto rows = [&](auto kern, int NL, size_t lds, auto... args) {
        const size_t turns = (size_t)((a.ny + NL - 1) / NL) * nb;
        hipError_t e = mq_lds_limit(kern, lds);
        if (e == hipSuccess)
            hipLaunchKernelGGL(kern, dim3((unsigned)std::min<size_t>(turns, 2048)),
                               dim3(mq_block(NL, px, turns)), lds, st, a, px, NL, args...);
        return e;
    };
    auto cols = [&](auto kern) {
        const dim3 grid((unsigned)((a.nx / 2 + sh.NC) / sh.NC), (unsigned)nb);
        const int nt = yp2 ? MQ_P2_THREADS : mq_block(2 * sh.NC, py, (size_t)grid.x * grid.y);
        hipError_t e = mq_lds_limit(kern, sh.lds_cols);
        if (e == hipSuccess) hipLaunchKernelGGL(kern, grid, dim3(nt), sh.lds_cols, st, a, py, sh.NC, W);
        return e;
    };
    auto rows_x = [&](auto kern) { return rows(kern, sh.NX, sh.lds_x, step0, nb, W); };
    hipError_t e = xp2      ? rows_x(k_meq_noise_x<Real, double, true>)
                   : sh.x64 ? rows_x(k_meq_noise_x<Real, double, false>)
                            : rows_x(k_meq_noise_x<Real, Real, false>);
    if (e != hipSuccess) return e;
    if (sh.y64)
        e = yp2 ? cols(k_meq_filter<Real, double, true>) : cols(k_meq_filter<Real, double, false>);
    else
        e = yp2 ? cols(k_meq_filter<Real, Real, true>) : cols(k_meq_filter<Real, Real, false>);
    if (e != hipSuccess) return e;
    e = xp2 ? rows(k_meq_noise_ix<Real, true>, sh.NI, sh.lds_i, nb, (const C*)W, xi)
            : rows(k_meq_noise_ix<Real, false>, sh.NI, sh.lds_i, nb, (const C*)W, xi);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

hipError_t launch_modeq_noise(const ModEqArgs& a, int prec, uint32_t step0, int nb, void* W,
                              void* xi, hipStream_t st) {
    if (prec == 0) return launch_noise_t<float>(a, step0, nb, W, (float*)xi, st);
    return launch_noise_t<double>(a, step0, nb, W, (double*)xi, st);
}

namespace {

template <typename Real, int T, int TX, int TY>
hipError_t step_tile(const ModEqArgs& a, const void* fin, void* fout, uint32_t step,
                     const void* xi, hipStream_t st) {
    Geom g{};
    g.nx = a.nx;
    g.ny = a.ny;
    g.nz = 1;
    g.nbx = (a.nx + TX - 1) / TX;
    g.nby = (a.ny + TY - 1) / TY;
    g.nbz = 1;
    g.nblocks = (uint32_t)(g.nbx * g.nby);
    g.V = (uint32_t)((size_t)a.nx * a.ny);
    hipLaunchKernelGGL((k_meq_step<Real, T, TX, TY>), dim3(g.nblocks),
                       dim3(MeqTile<T, TX, TY>::NT), 0, st, a, g, (const Real*)fin, (Real*)fout, step,
                       (const Real*)xi);
    return hipGetLastError();
}

template <typename Real>
hipError_t launch_step_t(const ModEqArgs& a, int T, const void* fin, void* fout, uint32_t step,
                         const void* xi, hipStream_t st) {
    if (T == 1) return step_tile<Real, 1, 64, 4>(a, fin, fout, step, xi, st);
    if (T == 2) return step_tile<Real, 2, 16, 16>(a, fin, fout, step, xi, st);
    if (T == 3) return step_tile<Real, 3, 8, 8>(a, fin, fout, step, xi, st);
    return hipErrorInvalidValue;
}

}  // namespace

// us per step with its noise, one step per launch -> T = 2 on 16 x 16 tiles ->
// T = 3 on 8 x 8 tiles: 128^2 FP32 4.53 -> 3.69 -> 3.18, 200 x 150 FP64 8.50 ->
// 6.73 -> 6.58, 256^2 FP32 6.04 -> 5.00 -> 5.23, 1024^2 FP32 45.0 -> 41.9 -> 44.5.
// So three steps while the chip is far from full, two otherwise, unless the
// tiles of a strip cover far more than its sites.
int modeq_steps(const ModEqArgs& a) {
    auto tiled = [&](size_t t) { return (a.nx + t - 1) / t * ((a.ny + t - 1) / t) * t * t; };
    const size_t V = (size_t)a.nx * a.ny;
    if (tiled(8) <= 32768) return 3;
    return tiled(16) <= 65536 || 4 * tiled(16) <= 5 * V ? 2 : 1;
}

hipError_t launch_modeq_step(const ModEqArgs& a, int prec, int T, const void* fin, void* fout,
                             uint32_t step, const void* xi, hipStream_t st) {
    return prec == 0 ? launch_step_t<float>(a, T, fin, fout, step, xi, st)
                     : launch_step_t<double>(a, T, fin, fout, step, xi, st);
}

}  // namespace flb
