// Device-side pieces shared by the dslash kernels: plane loads and stores
// (plain and non-temporal), link and spinor loads, and the order in which an
// XCD walks the sites of its slab.
#pragma once

#include "ov_device.h"
#include "spin.h"

namespace ov {

// Loads address a plane through a wave-uniform base pointer plus a 32-bit
// per-lane site offset, so that the compiler can use scalar-base addressing
// instead of per-lane 64-bit address arithmetic.
template <class S, class R>
__device__ __forceinline__ cx<R> ldp(const S *__restrict__ plane, unsigned site)
{
    const unsigned boff = site * (unsigned)sizeof(S);   // < 4 GiB: a plane holds at most 2^31/64 sites
    return ldc<R>((const S *)((const char *)plane + boff), 0u);
}

template <class S, class R>
__device__ __forceinline__ void stp(S *__restrict__ plane, unsigned site, cx<R> v)
{
    const unsigned boff = site * (unsigned)sizeof(S);
    stc<R>((S *)((char *)plane + boff), 0u, v);
}

// Components k = 2p and 2p+1 of one site: a single 16-byte load for the
// paired FP32 layout, two plane loads otherwise.
template <class S, class R>
__device__ __forceinline__ void ldpair(const S *__restrict__ f, int Vp, int p, unsigned site, cx<R> &a, cx<R> &b)
{
    if constexpr (Pair<S>::E == 2) {
        const float4 v = *(const float4 *)((const char *)(f + (size_t)(2 * p) * (unsigned)Vp) + site * 16u);
        a = cmk((R)v.x, (R)v.y);
        b = cmk((R)v.z, (R)v.w);
    } else {
        a = ldp<S, R>(f + (size_t)(2 * p) * (unsigned)Vp, site);
        b = ldp<S, R>(f + (size_t)(2 * p + 1) * (unsigned)Vp, site);
    }
}

template <class S, class R>
__device__ __forceinline__ void stpair(S *__restrict__ f, int Vp, int p, unsigned site, cx<R> a, cx<R> b)
{
    if constexpr (Pair<S>::E == 2) {
        *(float4 *)((char *)(f + (size_t)(2 * p) * (unsigned)Vp) + site * 16u) =
            make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
    } else {
        stp<S, R>(f + (size_t)(2 * p) * (unsigned)Vp, site, a);
        stp<S, R>(f + (size_t)(2 * p + 1) * (unsigned)Vp, site, b);
    }
}

// Non-temporal variants for operands that are touched once per launch (the
// epilogue inputs and the output): the loads and stores carry the
// non-temporal hint so that they do not displace the stencil's neighbour
// spinors and links from L2.
typedef float ov_f4 __attribute__((ext_vector_type(4)));
typedef double ov_d2 __attribute__((ext_vector_type(2)));

template <class S, class R>
__device__ __forceinline__ cx<R> ldp_nt(const S *__restrict__ plane, unsigned site)
{
    const char *p = (const char *)plane + site * (unsigned)sizeof(S);
    if constexpr (sizeof(S) == 16) {
        const ov_d2 v = __builtin_nontemporal_load((const ov_d2 *)p);
        return cmk((R)v.x, (R)v.y);
    } else if constexpr (sizeof(S) == 4) {
        const uint32_t v = __builtin_nontemporal_load((const uint32_t *)p);
        return cmk((R)bf16_lo(v), (R)bf16_hi(v));
    } else {
        return ldp<S, R>(plane, site);
    }
}

template <class S, class R>
__device__ __forceinline__ void stp_nt(S *__restrict__ plane, unsigned site, cx<R> v)
{
    char *p = (char *)plane + site * (unsigned)sizeof(S);
    if constexpr (sizeof(S) == 16) {
        ov_d2 w = {(double)v.x, (double)v.y};
        __builtin_nontemporal_store(w, (ov_d2 *)p);
    } else if constexpr (sizeof(S) == 4) {
        const uint32_t w = pack_bf16((float)v.x, (float)v.y);
        __builtin_nontemporal_store(w, (uint32_t *)p);
    } else {
        stp<S, R>(plane, site, v);
    }
}

template <class S, class R>
__device__ __forceinline__ void ldpair_nt(const S *__restrict__ f, int Vp, int p, unsigned site, cx<R> &a, cx<R> &b)
{
    if constexpr (Pair<S>::E == 2) {
        const ov_f4 v = __builtin_nontemporal_load(
            (const ov_f4 *)((const char *)(f + (size_t)(2 * p) * (unsigned)Vp) + site * 16u));
        a = cmk((R)v.x, (R)v.y);
        b = cmk((R)v.z, (R)v.w);
    } else {
        a = ldp_nt<S, R>(f + (size_t)(2 * p) * (unsigned)Vp, site);
        b = ldp_nt<S, R>(f + (size_t)(2 * p + 1) * (unsigned)Vp, site);
    }
}

template <class S, class R>
__device__ __forceinline__ void stpair_nt(S *__restrict__ f, int Vp, int p, unsigned site, cx<R> a, cx<R> b)
{
    if constexpr (Pair<S>::E == 2) {
        const ov_f4 w = {(float)a.x, (float)a.y, (float)b.x, (float)b.y};
        __builtin_nontemporal_store(w, (ov_f4 *)((char *)(f + (size_t)(2 * p) * (unsigned)Vp) + site * 16u));
    } else {
        stp_nt<S, R>(f + (size_t)(2 * p) * (unsigned)Vp, site, a);
        stp_nt<S, R>(f + (size_t)(2 * p + 1) * (unsigned)Vp, site, b);
    }
}

// Link U_mu(s): components 0..7 as pairs, component 8 on its own plane.
// REC: only the first two rows are read (components 0..5, three pairs) and
// the third is rebuilt as u_2a = conj(u_0b u_1c - u_0c u_1b), (a, b, c)
// cyclic, the identity that an SU(3) matrix (unitary, det 1) satisfies.  The
// gauge upload measures how far the stored links are from it and selects
// these kernels only where it holds to FP64 rounding; they read two thirds of
// the link bytes.
template <class R>
__device__ __forceinline__ void rebuild_row2(cx<R> (&u)[3][3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int b1 = (a + 1) % 3, c1 = (a + 2) % 3;
        const cx<R> t = csub(cmul(u[0][b1], u[1][c1]), cmul(u[0][c1], u[1][b1]));
        u[2][a] = cmk(t.x, -t.y);
    }
}

template <class S, class R, bool REC>
__device__ __forceinline__ void load_link(const S *__restrict__ U, int mu, int Vp, unsigned s, cx<R> (&u)[3][3])
{
    const S *b = U + (size_t)(mu * 9) * (unsigned)Vp;
    if constexpr (REC) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
            ldpair<S, R>(b, Vp, p, s, u[(2 * p) / 3][(2 * p) % 3], u[(2 * p + 1) / 3][(2 * p + 1) % 3]);
        rebuild_row2(u);
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p)
            ldpair<S, R>(b, Vp, p, s, u[(2 * p) / 3][(2 * p) % 3], u[(2 * p + 1) / 3][(2 * p + 1) % 3]);
        u[2][2] = ldp<S, R>(b + (size_t)8 * (unsigned)Vp, s);
    }
}

template <class S, class R>
__device__ __forceinline__ void load_spinor(const S *__restrict__ x, int Vp, unsigned s, cx<R> (&p)[4][3])
{
#pragma unroll
    for (int q = 0; q < 6; ++q)
        ldpair<S, R>(x, Vp, q, s, p[(2 * q) / 3][(2 * q) % 3], p[(2 * q + 1) / 3][(2 * q + 1) % 3]);
}

// Background phase (or its conjugate) times component (k, c) of a half
// spinor.  Which product of the imaginary part is rounded first is fixed per
// storage type and component, so that all dslash kernels agree to the last
// bit: the phase is the one FP32 factor of a BF16 hop whose products are not
// exact.  The choice itself has no numerical reason: it keeps the results that
// BF16 batches, and single BF16 vectors (`single`), had before the products
// were written out, when the compiler chose for each kernel.  A BF16 vector
// alone and in a batch therefore agree to BF16 rounding only; in FP64 and FP32
// they are the same bits.
template <class S, class R>
__device__ __forceinline__ cx<R> phase_mul(cx<R> f, cx<R> h, int k, int c, bool single)
{
    if constexpr (sizeof(S) == 4) {
        if (single || (k == 0 && c == 2)) return cmul(f, h);
    }
    return cmul_i(f, h);
}

// diag x - acc / 2, and v + c e, in the roundings that every dslash kernel uses.
template <class R>
__device__ __forceinline__ cx<R> site_term(R diag, cx<R> x, cx<R> acc)
{
    return {fma(diag, x.x, -((R)0.5 * acc.x)), fma(diag, x.y, -((R)0.5 * acc.y))};
}
template <class R>
__device__ __forceinline__ cx<R> add_scaled(cx<R> v, R c, cx<R> e)
{
    return {fma(c, e.x, v.x), fma(c, e.y, v.y)};
}

// Coordinates of a site (products instead of divisions, about twenty
// instructions each).
__device__ __forceinline__ void site_coords(const Geo &g, int s, int &xc, int &yc, int &zc, int &tc)
{
    const unsigned a = __umulhi((unsigned)s, g.mul[0]) >> g.shr[0];
    const unsigned b = __umulhi(a, g.mul[1]) >> g.shr[1];
    const unsigned c = __umulhi(b, g.mul[2]) >> g.shr[2];
    xc = s - (int)a * g.Lx;
    yc = (int)a - (int)b * g.Ly;
    zc = (int)b - (int)c * g.Lz;
    tc = (int)c;
}

// Site of position u in the slab of XCD xcd (orders 1 and 3).
__device__ __forceinline__ int slab_site(const Geo &g, int order, int cols, int xcd, int u)
{
    if (order == 3) {
        const int nt = g.Lt >> 3;
        const int q = u / g.Lxy, o = u - q * g.Lxy;
        if (q >= nt * g.Lz) return g.Vp;   // beyond the slab: no work
        const int tl = q % nt, z = q / nt;
        return o + g.Lxy * (z + g.Lz * (xcd * nt + tl));
    }
    // with cols > 1 the slab is walked one y-column (Ly/cols rows) at a time,
    // which shortens the distance between a site and its t neighbours
    const int nz = g.Lz >> 3;
    const int P = g.Lxy / cols;                 // sites of one column in one (z, t) plane
    const int per_col = P * nz * g.Lt;
    const int col = u / per_col;
    if (col >= cols) return g.Vp;               // beyond the slab: no work
    const int rem = u - col * per_col;
    const int q = rem / P, o = rem - q * P + col * P;
    const int zl = q % nz, t = q / nz;
    return o + g.Lxy * (xcd * nz + zl + g.Lz * t);
}

// One spinor as loaded, by buffer instructions: the plane is a scalar
// resource and the site a 32-bit lane offset, so a load costs no vector
// address arithmetic (with 64-bit lane addresses every load takes a 64-bit
// add).  A resource covers exactly one plane.
template <class S>
struct RawSpinor {
    using R = typename StoreT<S>::real;
    static constexpr int C = Pair<S>::E, N = 12 / C, B = C * (int)sizeof(S);   // bytes of an element
    uint32_t w[N][B / 4];

    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane(const S *f, int Vp, int q)
    {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(f + (size_t)(q * C) * (unsigned)Vp), 0, (unsigned)Vp * B,
                                                 0x00020000);
    }
    template <int AUX>
    static __device__ __forceinline__ void ld(const S *f, int Vp, int q, unsigned boff, uint32_t (&o)[B / 4])
    {
        if constexpr (B == 16) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(plane(f, Vp, q), boff, 0, AUX);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = v[i];
        } else {
            o[0] = __builtin_amdgcn_raw_buffer_load_b32(plane(f, Vp, q), boff, 0, AUX);
        }
    }
    // component h of an element
    static __device__ __forceinline__ cx<R> get(const uint32_t (&o)[B / 4], int h)
    {
        if constexpr (sizeof(S) == 16) {
            return cmk(__builtin_bit_cast(double, (uint64_t)o[0] | ((uint64_t)o[1] << 32)),
                       __builtin_bit_cast(double, (uint64_t)o[2] | ((uint64_t)o[3] << 32)));
        } else if constexpr (sizeof(S) == 8) {
            return cmk(__uint_as_float(o[2 * h]), __uint_as_float(o[2 * h + 1]));
        } else {
            return cmk(bf16_lo(o[0]), bf16_hi(o[0]));
        }
    }
    __device__ __forceinline__ void load(const S *f, int Vp, unsigned boff)
    {
#pragma unroll
        for (int q = 0; q < N; ++q) ld<0>(f, Vp, q, boff, w[q]);
    }
    __device__ __forceinline__ void spinor(cx<R> (&p)[4][3]) const
    {
#pragma unroll
        for (int k = 0; k < 12; ++k) p[k / 3][k % 3] = get(w[k / C], k % C);
    }
};

// Byte offset inside a plane of the neighbour of site s0 (wrap: the hop
// leaves the lattice; step +-stride, L the extent); across a Dirichlet
// boundary one beyond every plane, which a buffer load answers with zeros.
// Zeros times the link are nothing only where the link is finite in the
// storage type; links across such a boundary are packed as zeros.
template <class S>
__device__ __forceinline__ unsigned neighbour_offset(int s0, bool wrap, int L, int step, float bc)
{
    const unsigned o = (unsigned)(wrap ? s0 - (L - 1) * step : s0 + step) * (unsigned)RawSpinor<S>::B;
    return wrap && bc == 0.0f ? 0x80000000u : o;
}

// Link of direction mu through plane resources; `e` is the site's byte offset
// in a plane of elements of RawSpinor<S>::B bytes.
template <class S, bool REC>
__device__ __forceinline__ void load_link_buf(const S *U, int mu, int Vp, unsigned e,
                                              cx<typename StoreT<S>::real> (&u)[3][3])
{
    using Raw = RawSpinor<S>;
    const S *b = U + (size_t)(mu * 9) * (unsigned)Vp;
    constexpr int NE = (REC ? 6 : Raw::C == 2 ? 8 : 9) / Raw::C;
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        uint32_t o[Raw::B / 4];
        Raw::template ld<0>(b, Vp, q, e, o);
#pragma unroll
        for (int h = 0; h < Raw::C; ++h) u[(q * Raw::C + h) / 3][(q * Raw::C + h) % 3] = Raw::get(o, h);
    }
    if constexpr (REC) rebuild_row2(u);
    else if constexpr (Raw::C == 2) u[2][2] = ldp<S, typename StoreT<S>::real>(b + (size_t)8 * (unsigned)Vp, e / Raw::B);
}

__device__ __forceinline__ float flip_sign(float v, uint32_t bit) { return __uint_as_float(__float_as_uint(v) ^ bit); }
__device__ __forceinline__ double flip_sign(double v, uint32_t bit)
{
    return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, v) ^ ((uint64_t)bit << 32));
}

// An output component as the storage type holds it, in the canonical layout's
// complex128.
template <class S, class R>
__device__ __forceinline__ double2 stored_value(cx<R> v)
{
    if constexpr (sizeof(S) == 4) {
        const uint32_t w = pack_bf16((float)v.x, (float)v.y);
        return make_double2((double)bf16_lo(w), (double)bf16_hi(w));
    } else {
        return make_double2((double)v.x, (double)v.y);
    }
}

}  // namespace ov
