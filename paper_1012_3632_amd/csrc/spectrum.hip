// Equal-time mode spectra of one state: the measurement behind the
// equilibration ratio of Sec. VI (the equal-time correlation |m_a(k)|^2 of
// every LB mode, averaged over snapshots and divided by its theoretical
// variance).
//
// Input: the q real mode fields of a periodic nx x ny x nz lattice (site
// s = x + nx (y + ny z)).  The three-dimensional DFT
//   m_a(k) = sum_x m_a(x) exp(-i k.x),  k = 2 pi (kx / nx, ky / ny, kz / nz)
// is taken one axis at a time on lines held in LDS (fft.h).  The fields are
// real, so only the half 0 <= kx <= nx / 2 is formed, kept and transformed
// along y and z (m_a(-k) is its conjugate): k_fft_rows transforms two rows of
// a field as the real and imaginary part of one complex line and separates
// them; k_fft_cols works in place on groups of adjacent lines, whose loads
// and stores touch consecutive values.  k_spec_accumulate then adds
// |m_a(k)|^2 for every mode and Re(j_alpha(k) conj j_beta(k)) for the momentum
// pairs (x, y) [2-D] or (x, y), (y, z), (z, x) [3-D], the cross spectra that
// split the momentum into longitudinal and transverse parts, at k and -k.
// The same passes give the spectra of any real fields (flb_field_spectrum),
// e.g. of interface heights.
//
// Bound: memory and LDS latency.  D3Q19 128 x 96 x 80 (19 fields, 0.98 M
// sites): 0.39 ms for the mode fields, three axes and the sums, 1.5 GB moved;
// 3.28 ms when every line was an n^2 direct sum over the full spectrum.
//
// Interface heights (the capillary test of Sec. VI): for every column across
// a planar interface, the shift h of the mean-field profile (eq. denprof)
// that best fits the column's density (eq. height-def), by Gauss-Newton.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fft.h"
#include "internal.h"

namespace flb {

namespace {

constexpr int FFT_THREADS = 512;   // at most, per block

// Dynamic LDS of the line transforms: two buffers of NL lines, then the twiddles.
extern __shared__ __align__(16) unsigned char lds_fft[];

// a / b for a < 2^51, with rb = 1.0 / b from the host (fft_div in FP64: a 64-bit
// division is hundreds of cycles at the start of every turn).
__device__ __forceinline__ size_t div_big(size_t a, double rb) {
    return (size_t)(((double)a + 0.5) * rb);
}

// Rows along x: line l of a field holds its rows 2 l (real part) and 2 l + 1
// (imaginary part; zero past the last row).  Z = A + i B separates by
// A(k) = (Z(k) + conj Z(n - k)) / 2, B(k) = (Z(k) - conj Z(n - k)) / 2i.
// NL lines per block and turn; W[field][row][kx], kx = 0 .. n / 2.
__global__ __launch_bounds__(FFT_THREADS) void k_fft_rows(const double* __restrict__ fields,
                                                          double2* __restrict__ W, FftPlan p,
                                                          int NL, uint32_t rows, size_t nlines,
                                                          double rper) {
    const int n = p.n, hx = n / 2 + 1, ld = fft_ld(n);
    double2* a = (double2*)lds_fft;
    double2* b = a + NL * ld;
    double2* tw = b + NL * ld;
    twiddles<double>(tw, p);
    const uint32_t per = (rows + 1) / 2;   // lines per field, 1 / rper
    const float rn = 1.0f / (float)n, rh = 1.0f / (float)hx, rp = 1.0f / (float)per;
    for (size_t l0 = (size_t)blockIdx.x * NL; l0 < nlines; l0 += (size_t)gridDim.x * NL) {
        const size_t f0 = div_big(l0, rper);
        const uint32_t m0 = (uint32_t)(l0 - f0 * per);   // line l0 + L: line m0 + L of field f0
        const int nl = (int)(nlines - l0 < (size_t)NL ? nlines - l0 : (size_t)NL);
        // row of the real part of line L, over all fields
        auto row_of = [&](int L, bool& pair) {
            const uint32_t m = m0 + (uint32_t)L, df = (uint32_t)fft_div((int)m, rp);
            const uint32_t r = 2 * (m - df * per);
            pair = r + 1 < rows;
            return (f0 + df) * rows + r;
        };
        auto get = [&](int t) {
            const int L = fft_div(t, rn), x = t - L * n;
            double2 v = make_double2(0.0, 0.0);
            if (L < nl) {
                bool pair;
                const double* src = fields + row_of(L, pair) * n + x;
                v.x = src[0];
                if (pair) v.y = src[n];
            }
            return v;
        };
        auto put = [&](int t, double2 v) {
            const int L = fft_div(t, rn);
            a[L * ld + fft_pos(t - L * n)] = v;
        };
        for (int t = threadIdx.x; t < NL * n; t += blockDim.x) put(t, get(t));
        __syncthreads();
        const double2* z = fft_lines<double, false>(a, b, tw, NL, p);
        for (int t = threadIdx.x; t < nl * hx; t += blockDim.x) {
            const int L = fft_div(t, rh), k = t - L * hx;
            bool pair;
            double2* dst = W + row_of(L, pair) * hx + k;
            const double2 u = z[L * ld + fft_pos(k)], v = z[L * ld + fft_pos(k == 0 ? 0 : n - k)];
            dst[0] = make_double2(0.5 * (u.x + v.x), 0.5 * (u.y - v.y));
            if (pair) dst[hx] = make_double2(0.5 * (u.y + v.y), 0.5 * (v.x - u.x));
        }
        __syncthreads();   // the result is read before the next turn's loads
    }
}

// In place along y or z: line l (l % inner adjacent, inner apart by outer)
// starts at (l % inner) + (l / inner) outer and has stride `inner`.  A block
// takes NL adjacent lines at a time; groups do not cross an `inner` run.
__global__ __launch_bounds__(FFT_THREADS) void k_fft_cols(double2* __restrict__ W, FftPlan p,
                                                          int NL, uint32_t inner, size_t outer,
                                                          uint32_t groups, size_t ngroups,
                                                          double rgroups) {
    const int n = p.n, ld = fft_ld(n);
    double2* a = (double2*)lds_fft;
    double2* b = a + NL * ld;
    double2* tw = b + NL * ld;
    twiddles<double>(tw, p);
    const float rl = 1.0f / (float)NL;
    for (size_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
        const size_t o = div_big(g, rgroups);
        const uint32_t c0 = (uint32_t)(g - o * groups) * (uint32_t)NL;
        const int nl = min(NL, (int)(inner - c0));
        double2* base = W + o * outer + c0;
        auto get = [&](int t) {
            const int j = fft_div(t, rl), c = t - j * NL;
            return c < nl ? base[(size_t)j * inner + c] : make_double2(0.0, 0.0);
        };
        auto put = [&](int t, double2 v) {
            const int j = fft_div(t, rl);
            a[(t - j * NL) * ld + fft_pos(j)] = v;
        };
        for (int t = threadIdx.x; t < NL * n; t += blockDim.x) put(t, get(t));
        __syncthreads();
        const double2* z = fft_lines<double, false>(a, b, tw, NL, p);
        for (int t = threadIdx.x; t < NL * n; t += blockDim.x) {
            const int j = fft_div(t, rl), c = t - j * NL;
            if (c < nl) base[(size_t)j * inner + c] = z[c * ld + fft_pos(j)];
        }
        __syncthreads();
    }
}

// spec[a V + s] += |W_a(s)|^2 (a < q); spec[(q + p) V + s] += Re(W_{1+al} conj W_{1+be})
// for the momentum pair p = (al, be) = (p, (p + 1) mod 3), p < npairs, at every
// wavevector s = (kx, ky, kz): from the stored half at s, or at -s where
// kx > nx / 2 (both terms are even in k).  blockIdx.y: a field, or (npairs >
// 0, blockIdx.y = 1) the D momentum rows together.
__global__ __launch_bounds__(256) void k_spec_accumulate(const double2* __restrict__ W,
                                                         double* __restrict__ spec, int q,
                                                         int npairs, int nx, int ny, int nz,
                                                         size_t V, size_t Vh) {
    const int D = npairs == 0 ? 0 : (npairs == 1 ? 2 : 3);
    const int y = (int)blockIdx.y;
    const bool mom = D > 0 && y == 1;
    const int a0 = (D > 0 && y > 1) ? y + D - 1 : y;
    const int hx = nx / 2 + 1;
    for (size_t s = (size_t)blockIdx.x * blockDim.x + threadIdx.x; s < V;
         s += (size_t)gridDim.x * blockDim.x) {
        const uint32_t r = (uint32_t)s / (uint32_t)nx;
        int kx = (int)((uint32_t)s - r * (uint32_t)nx);
        int kz = (int)(r / (uint32_t)ny);
        int ky = (int)(r - (uint32_t)kz * (uint32_t)ny);
        if (kx >= hx) {
            kx = nx - kx;
            ky = ky == 0 ? 0 : ny - ky;
            kz = kz == 0 ? 0 : nz - kz;
        }
        const double2* w = W + ((size_t)((uint32_t)kz * (uint32_t)ny + (uint32_t)ky) * hx + kx);
        if (!mom) {
            const double2 u = w[a0 * Vh];
            spec[a0 * V + s] += u.x * u.x + u.y * u.y;
            continue;
        }
        const double2 jx = w[Vh], jy = w[2 * Vh];
        spec[V + s] += jx.x * jx.x + jx.y * jx.y;
        spec[2 * V + s] += jy.x * jy.x + jy.y * jy.y;
        spec[q * V + s] += jx.x * jy.x + jx.y * jy.y;
        if (D == 3) {
            const double2 jz = w[3 * Vh];
            spec[3 * V + s] += jz.x * jz.x + jz.y * jz.y;
            spec[(q + 1) * V + s] += jy.x * jz.x + jy.y * jz.y;
            spec[(q + 2) * V + s] += jz.x * jx.x + jz.y * jx.y;
        }
    }
}

// Interface heights (capillary test): one wavefront per column c and
// interface j (blockIdx.y), its lanes over the window.  The density of column
// c at profile coordinate y is rho0 + drho[c + y ncol].  The height h minimizes
//   E(h) = sum_{k=-W..W} (rho(y0 + k) - m(y0 + k - h))^2,
//   m(u) = rho_c + sign (rho_L - rho_V)/2 tanh(2 u / w),
// the mean-field profile; Gauss-Newton from h = y0, clamped to the window,
// until the update is below 1e-13 (at most 64 iterations).  The two sums of
// every iteration are reduced over the wavefront by a fixed butterfly, so
// all lanes hold the same h and leave the loop together.
constexpr int HEIGHT_WAVES = 4;
template <typename Real>
__global__ __launch_bounds__(64 * HEIGHT_WAVES) void k_interface_heights(
    const Real* __restrict__ drho, double rho0, int n, long ncol, InterfaceSet set, double rho_c,
    double half_jump, double two_over_w, double* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const long c = (long)blockIdx.x * HEIGHT_WAVES + (threadIdx.x >> 6);
    const int j = blockIdx.y;
    if (c >= ncol) return;   // whole wavefronts leave together
    const int y0 = set.y0[j], W = set.half_window[j];
    const double s = set.sign[j] * half_jump;
    double h = (double)y0;
    for (int it = 0; it < 64; ++it) {
        double num = 0.0, den = 0.0;
        for (int k = -W + lane; k <= W; k += 64) {
            int yy = y0 + k;
            if (yy < 0) yy += n;
            if (yy >= n) yy -= n;
            const double r = rho0 + (double)drho[c + (long)yy * ncol];
            const double t = tanh(two_over_w * ((double)(y0 + k) - h));
            const double mp = s * (1.0 - t * t) * two_over_w;
            num += (r - (rho_c + s * t)) * mp;
            den += mp * mp;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            num += __shfl_xor(num, off, 64);
            den += __shfl_xor(den, off, 64);
        }
        if (!(den > 0.0)) break;
        const double hn = fmin(fmax(h - num / den, (double)(y0 - W)), (double)(y0 + W));
        const double dh = hn - h;
        h = hn;
        if (fabs(dh) < 1e-13) break;
    }
    if (lane == 0) out[(long)j * ncol + c] = h;
}

}  // namespace

hipError_t launch_interface_heights(int prec, const void* drho, double rho0, int n, long ncol,
                                    const InterfaceSet& set, double rho_L, double rho_V,
                                    double width, double* out, hipStream_t st) {
    const dim3 grid((unsigned)((ncol + HEIGHT_WAVES - 1) / HEIGHT_WAVES), set.n);
    const dim3 block(64 * HEIGHT_WAVES);
    const double rc = 0.5 * (rho_L + rho_V), half = 0.5 * (rho_L - rho_V), tw = 2.0 / width;
    if (prec == 0)
        hipLaunchKernelGGL(k_interface_heights<float>, grid, block, 0, st, (const float*)drho,
                           rho0, n, ncol, set, rc, half, tw, out);
    else
        hipLaunchKernelGGL(k_interface_heights<double>, grid, block, 0, st, (const double*)drho,
                           rho0, n, ncol, set, rc, half, tw, out);
    return hipGetLastError();
}

namespace {

// Lines per block of n elements, of `lines` adjacent ones: at most 16 (256
// consecutive bytes of a row) and as many as keep two buffers and the
// twiddles within 80 KB, two blocks per CU, but four, so that adjacent lines
// fill 64 bytes, up to 128 KB (n above 800: two); then the same number of groups with equal shares (65 lines: five groups of 13).
// At 128 x 96 x 80 the z pass took 83 us with this limit, 95-102 with 40 KB.
// Where that would give fewer than 512 blocks (total lines), fewer lines, so
// that a small lattice still spreads over the chip.
int fft_lines_per_block(const FftPlan& p, size_t lines, size_t total, size_t* lds) {
    const size_t per = 2 * (size_t)fft_ld(p.n) * sizeof(double2);
    const size_t tw = fft_twiddles(p) * sizeof(double2);
    size_t NL = 16;
    while (NL > 2 && NL * per + tw > (NL > 4 ? 81920 : 131072)) NL /= 2;
    NL = std::min(NL, std::max<size_t>(2, total / 512));
    const size_t groups = (lines + NL - 1) / NL;
    NL = (lines + groups - 1) / groups;
    *lds = NL * per + tw;
    return (int)NL;
}

// Four elements per thread: with eight (one radix-8 group each) too few
// wavefronts hide the LDS latency (x pass 119 us against 96).  Two where a
// stage of direct sums has an output pair for each.
int fft_block(int NL, const FftPlan& p) {
    const int t = (NL * p.n / (p.any ? 2 : 4) + 63) / 64 * 64;
    return t < 64 ? 64 : (t > FFT_THREADS ? FFT_THREADS : t);
}

constexpr size_t FFT_GRID = 2048;   // a block's twiddles serve all its turns

hipError_t fft_lds(const void* kernel, size_t lds) {
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

}  // namespace

hipError_t launch_spectrum(int q, int npairs, int nx, int ny, int nz, const double* fields,
                           void* work, double* spec, hipStream_t st) {
    const size_t V = (size_t)nx * ny * nz;
    const size_t hx = (size_t)nx / 2 + 1, Vh = hx * ny * nz;
    double2* W = (double2*)work;
    size_t lds = 0;
    {
        const FftPlan p = fft_plan(nx);
        const uint32_t rows = (uint32_t)((size_t)ny * nz);
        const size_t nlines = (size_t)q * ((rows + 1) / 2);
        const int NL = fft_lines_per_block(p, nlines, nlines, &lds);
        const size_t blocks = (nlines + NL - 1) / NL;
        hipError_t e = fft_lds((const void*)k_fft_rows, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_fft_rows, dim3((unsigned)std::min<size_t>(blocks, FFT_GRID)),
                           dim3(fft_block(NL, p)), lds, st, fields, W, p, NL, rows, nlines,
                           1.0 / (double)((rows + 1) / 2));
    }
    // y: hx adjacent lines per (field, z); z: hx ny adjacent lines per field
    for (int axis = 1; axis < 3; ++axis) {
        const int n = axis == 1 ? ny : nz;
        if (n == 1) continue;
        const FftPlan p = fft_plan(n);
        const size_t inner = axis == 1 ? hx : hx * ny, outer = inner * n;
        const size_t sets = axis == 1 ? (size_t)q * nz : (size_t)q;
        const int NL = fft_lines_per_block(p, inner, inner * sets, &lds);
        const uint32_t groups = (uint32_t)((inner + NL - 1) / NL);
        const size_t ngroups = groups * sets;
        hipError_t e = fft_lds((const void*)k_fft_cols, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_fft_cols, dim3((unsigned)std::min<size_t>(ngroups, FFT_GRID)),
                           dim3(fft_block(NL, p)), lds, st, W, p, NL, (uint32_t)inner, outer,
                           groups, ngroups, 1.0 / (double)groups);
    }
    const size_t blocks = (V + 255) / 256 < 4096 ? (V + 255) / 256 : 4096;
    const int ygrid = npairs == 0 ? q : q - (npairs == 1 ? 1 : 2);
    hipLaunchKernelGGL(k_spec_accumulate, dim3((unsigned)blocks, ygrid), dim3(256), 0, st, W, spec,
                       q, npairs, nx, ny, nz, V, Vh);
    return hipGetLastError();
}

}  // namespace flb
