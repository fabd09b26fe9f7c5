// Flat addressing of one periodic box: sites s = x + nx (y + ny z) taken in
// order, 256 to a block, whatever the extents, so that no lane is idle on a
// ragged row.  Shared by the batched kernels (many boxes) and the flat step of
// one box.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.h"

namespace flb {

// s / n = umulhi(s, ceil(2^32 / n)), exact while s (ceil(2^32 / n) n - 2^32) <
// 2^32, so for every s with s n < 2^32.  n = 1: the inverse 2^32 is passed as 0.
__device__ __forceinline__ uint32_t div_small(uint32_t s, uint32_t inv) {
    return inv == 0u ? s : __umulhi(s, inv);
}

// Periodic neighbourhood of site s = x + nx (y + ny z) of one box, in
// bytes: s4 = s sizeof(Real) and the wrapped byte steps to x -+ 1, y -+ 1 and
// z -+ 1 (modulo 2^32), each a selection between two uniform values, so that
// the byte offset of x + c is s4 plus up to three of them (no multiplies;
// the partial sums are shared between directions).
template <typename Real>
struct Nbr {
    uint32_t s4, dx[2], dy[2], dz[2];
    __device__ __forceinline__ Nbr(uint32_t s, int x, int y, int z, int nx, int ny, int nz, uint32_t V);
    __device__ __forceinline__ uint32_t at(int cx, int cy, int cz) const {
        uint32_t o = s4;
        if (cz) o += dz[cz > 0];
        if (cy) o += dy[cy > 0];
        if (cx) o += dx[cx > 0];
        return o;
    }
};
template <typename Real>
__device__ __forceinline__ Nbr<Real>::Nbr(uint32_t s, int x, int y, int z, int nx, int ny, int nz,
                                          uint32_t V) {
    constexpr uint32_t E = sizeof(Real);
    const uint32_t ex = E, ey = E * (uint32_t)nx, ez = ey * (uint32_t)ny;
    const uint32_t wx = ey - ex, wy = ez - ey, wz = E * V - ez;   // a wrap: period minus a step
    s4 = s * E;
    dx[0] = x == 0 ? wx : 0u - ex;
    dx[1] = x == nx - 1 ? 0u - wx : ex;
    dy[0] = y == 0 ? wy : 0u - ey;
    dy[1] = y == ny - 1 ? 0u - wy : ey;
    dz[0] = z == 0 ? wz : 0u - ez;
    dz[1] = z == nz - 1 ? 0u - wz : ez;
}

// The populations of one box (Q planes of V sites from rep) as a buffer
// resource: an access is the resource plus a uniform byte offset (plane i:
// i V sizeof(Real), an SGPR) plus the lane's 32-bit byte offset, so no lane
// forms a 64-bit address.  The record count is the box's population bytes,
// below 2^32.  V is made opaque to the compiler by
// the caller once per tile (an empty asm on an SGPR), so that the plane
// offsets are formed next to their accesses instead of being hoisted out of
// the tile loop and held.  Word 3 of the resource is the CDNA raw-buffer
// format (32-bit data format, no swizzle, no stride).
// The record count and the scalar offsets are unsigned 32-bit fields of the
// hardware; the builtins take
// them as int, so values above 2^31 pass through the cast bit for bit.
template <int LAT, typename Real>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rep_rsrc(const Real* rep, uint32_t V) {
    const uint32_t bytes = (uint32_t)Lattice<LAT>::Q * V * (uint32_t)sizeof(Real);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<Real*>(rep), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint32_t plane_soff(uint32_t Vr, int i, uint32_t esize) {
    return (uint32_t)i * Vr * esize;
}
__device__ __forceinline__ float rep_ld(__amdgpu_buffer_rsrc_t r, uint32_t Vr, int i, uint32_t boff,
                                        float) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)boff, (int)plane_soff(Vr, i, 4), 0));
}
__device__ __forceinline__ double rep_ld(__amdgpu_buffer_rsrc_t r, uint32_t Vr, int i,
                                         uint32_t boff, double) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, (int)boff, (int)plane_soff(Vr, i, 8), 0);
    return __longlong_as_double((long long)(((unsigned long long)w.y << 32) | w.x));
}
__device__ __forceinline__ void rep_st(__amdgpu_buffer_rsrc_t r, uint32_t Vr, int i, uint32_t boff,
                                       float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)boff, (int)plane_soff(Vr, i, 4), 0);
}
__device__ __forceinline__ void rep_st(__amdgpu_buffer_rsrc_t r, uint32_t Vr, int i, uint32_t boff,
                                       double v) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    u2 w;
    w.x = (unsigned int)b;
    w.y = (unsigned int)(b >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, (int)boff, (int)plane_soff(Vr, i, 8), 0);
}

template <int LAT, typename Real>
__device__ __forceinline__ void rep_pull(__amdgpu_buffer_rsrc_t rep, uint32_t Vr,
                                         const Nbr<Real>& nb, Real (&f)[Lattice<LAT>::Q]) {
    using L = Lattice<LAT>;
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        f[i] = rep_ld(rep, Vr, i, nb.at(-L::cx[i], -L::cy[i], -L::cz[i]), Real(0));
}

constexpr int FLAT_NT = 256;   // sites per block

struct FlatBox {
    int32_t nx, ny, nz;
    uint32_t V, inv_nx, inv_ny;   // the inverses of div_small
};

// One plane of V reals as a buffer resource.
template <typename Real>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const Real* p, uint32_t V) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<Real*>(p), 0,
                                             (int)(V * (uint32_t)sizeof(Real)), 0x00020000);
}

// The density and chemical potential fields of a force step.
template <typename Real>
struct FlatForce {
    const Real* drho;
    const Real* mu;
    ForceParams<Real> fp;
};

// One step of site s: KIND 0 from fin to fout, 1 and 2 the phases of an
// in-place pair (fin == fout).  With STATS the site's moments and their
// squares are added to v.  FORCE (KIND 0): F = -rho grad_h mu + eta cs2 grad_h
// rho from the fields of ff (the sums of ForceTile::force).
template <int LAT, typename Real, bool STATS, int KIND, bool FORCE = false>
__device__ __forceinline__ void flat_site(const Real* fin, Real* fout, uint32_t s, const FlatBox& B,
                                          const CollideParams<Real>& P, uint32_t replica,
                                          uint32_t key0, uint32_t key1, uint32_t step,
                                          const double2* tab, Real* v,
                                          const FlatForce<Real>& ff = FlatForce<Real>()) {
    using L = Lattice<LAT>;
    using M = Moments<LAT, Real>;
    constexpr int Q = L::Q, D = L::D;
    const uint32_t yz = div_small(s, B.inv_nx);
    const int x = (int)(s - yz * (uint32_t)B.nx);
    const uint32_t z = div_small(yz, B.inv_ny);
    const int y = (int)(yz - z * (uint32_t)B.ny);
    const __amdgpu_buffer_rsrc_t in = rep_rsrc<LAT, Real>(fin, B.V);
    const __amdgpu_buffer_rsrc_t out = rep_rsrc<LAT, Real>(fout, B.V);
    const uint32_t se = s * (uint32_t)sizeof(Real);
    uint32_t Vr = B.V;
    asm volatile("" : "+s"(Vr));
    Real f[Q], m[Q];
    if constexpr (KIND < 2) {
        rep_pull<LAT, Real>(in, Vr, Nbr<Real>(s, x, y, (int)z, B.nx, B.ny, B.nz, B.V), f);
    } else {
        // local accesses: one lane offset for every plane
#pragma unroll
        for (int i = 0; i < Q; ++i) f[i] = rep_ld(in, Vr, L::opp[i], se, Real(0));
    }
    Real F[D] = {};
    if constexpr (FORCE) {
        const Nbr<Real> nb(s, x, y, (int)z, B.nx, B.ny, B.nz, B.V);
        const __amdgpu_buffer_rsrc_t mu = plane_rsrc(ff.mu, B.V), dr = plane_rsrc(ff.drho, B.V);
        Real gm[D] = {}, gr[D] = {};
        auto grad = [&](__amdgpu_buffer_rsrc_t field, Real (&o)[D]) {
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const Real w = rep_ld(field, 0u, 0, nb.at(L::cx[i], L::cy[i], L::cz[i]), Real(0));
                const int c3[3] = {L::cx[i], L::cy[i], L::cz[i]};
#pragma unroll
                for (int a = 0; a < D; ++a)
                    if (c3[a] != 0) o[a] += Real(L::w[i] * c3[a]) * w;
            }
        };
        grad(mu, gm);
        if (ff.fp.eta != Real(0)) grad(dr, gr);   // uniform
        const Real rho = P.rho0 + rep_ld(dr, 0u, 0, se, Real(0));
#pragma unroll
        for (int a = 0; a < D; ++a) F[a] = -rho * Real(3) * gm[a] + ff.fp.eta * gr[a];
    }
    M::forward(f, m);
    if constexpr (STATS) {
#pragma unroll
        for (int a = 0; a < Q; ++a) {
            v[a] += m[a];
            v[Q + a] += m[a] * m[a];
        }
    }
    Real zn[2 * L::NPAIR];
    if (P.noise_on) site_normals<L::NPAIR, Real>(s, step, 0u, replica, key0, key1, zn, tab);
    collide_moments<LAT, Real, FORCE>(m, F, zn, P);
    M::inverse(m, f);
    uint32_t Vs = Vr;   // the store offsets are not those of the loads
    asm volatile("" : "+s"(Vs));
    if constexpr (KIND == 1) {
        int xs = x;     // nor is the neighbourhood held through the collision
        asm volatile("" : "+v"(xs));
        const Nbr<Real> nb(s, xs, y, (int)z, B.nx, B.ny, B.nz, B.V);
#pragma unroll
        for (int i = 0; i < Q; ++i)
            rep_st(out, Vs, L::opp[i], nb.at(L::cx[i], L::cy[i], L::cz[i]), f[i]);
    } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) rep_st(out, Vs, i, se, f[i]);
    }
}

}  // namespace flb
