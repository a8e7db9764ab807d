// H_w / D_w for small batches: one wave per hop or per direction of the stencil.
//
// Same operator and epilogue as the site-parallel kernels:
//   y_r = a * G (D_w x_r)  +  c1 e1_r + c2 e2_r + c3 e3_r          (own site)
//
// The eight (or four) waves of a workgroup cover the same 64 sites of one
// right-hand side; each gathers one hop (or both hops of a direction) and
// leaves the link times half spinor in LDS ([hop][2 x 3 components][lane]),
// after which each sums a share of the components, hop by hop in the order of
// the site-parallel kernels, so the result has the same bits as theirs.
//
// What bounds a small batch is memory latency.  The loads of a thread (two
// links, two neighbours, its share of the own-site operands) depend on nothing
// but the site index and stand before the arithmetic, without branches between
// them, so they are all in flight together: the kernel waits for memory about
// once, where a thread that walks the eight hops one after the other, each
// behind its boundary branch, waits for the links and the spinor of every hop
// in turn.  It also has eight times the wavefronts for the same sites.
// Mean of a plain and a fused launch in a captured graph (an empty node takes
// 1.6 us), site-parallel kernel and this one:
//   FP64 12 RHS of 4^4 16.7 -> 4.5 us, FP32 4 RHS of 8^3x16 16.3 -> 5.9 us,
//   FP64 1 RHS of 16^3x32 37.7 -> 27 us, of 24^3x48 222 -> 151 us.
// Loading every argument at once at the top instead of where it is needed, and slots and field
// groups as arguments instead of lists, gained nothing (1.00x; the latter 0.94x on 4^4).
#include <type_traits>

#include "dslash_device.h"
#include "ov_internal.h"

namespace ov {

// A unit is the 16-byte element of the storage layout: one FP64 or two FP32
// components (one of BF16).
template <class S>
struct UnitOf {
    using R = typename StoreT<S>::real;
    static constexpr int C = Pair<S>::E;      // components per unit
    static constexpr int N = 12 / C;          // units per spinor
    struct T {
        cx<R> c[C];
    };
};

// Unit q of a field at byte offset e of its plane.
template <class S, bool NT>
__device__ __forceinline__ typename UnitOf<S>::T ld_unit(const S *__restrict__ f, int Vp, int q, unsigned e)
{
    using Raw = RawSpinor<S>;
    uint32_t o[Raw::B / 4];
    Raw::template ld<NT ? 2 : 0>(f, Vp, q, e, o);
    typename UnitOf<S>::T t;
#pragma unroll
    for (int h = 0; h < Raw::C; ++h) t.c[h] = Raw::get(o, h);
    return t;
}

template <class S, bool NT>
__device__ __forceinline__ void st_unit(S *__restrict__ f, int Vp, int q, unsigned site, const typename UnitOf<S>::T &t)
{
    using R = typename StoreT<S>::real;
    if constexpr (UnitOf<S>::C == 2) {
        if constexpr (NT) stpair_nt<S, R>(f, Vp, q, site, t.c[0], t.c[1]);
        else stpair<S, R>(f, Vp, q, site, t.c[0], t.c[1]);
    } else {
        if constexpr (NT) stp_nt<S, R>(f + (size_t)q * (unsigned)Vp, site, t.c[0]);
        else stp<S, R>(f + (size_t)q * (unsigned)Vp, site, t.c[0]);
    }
}

// Hops of direction MU at `site` (a real site), HOPS = 1 forward, 2 backward, 3
// both: link times half spinor to out[6 components at stride 64], the forward
// hop first, the backward hop 6 x 64 behind.
template <int MU, int HOPS, class S, bool REC>
__device__ __forceinline__ void dir_hops(const DsArgs<S> &a, const S *__restrict__ x, int site, int cmu, int Lmu,
                                         int stride, cx<typename StoreT<S>::real> ph,
                                         cx<typename StoreT<S>::real> *__restrict__ out)
{
    using R = typename StoreT<S>::real;
    using Raw = RawSpinor<S>;
    const int Vp = a.g.Vp;
    const float bc = a.g.bcf[MU];
    const bool wf = cmu == Lmu - 1, wb = cmu == 0;
    const unsigned es = (unsigned)site * (unsigned)Raw::B;
    const unsigned eu = (unsigned)(wb ? site + (Lmu - 1) * stride : site - stride) * (unsigned)Raw::B;
    cx<R> uf[3][3], ub[3][3], pf[4][3], pb[4][3];
    Raw rf, rb;
    if constexpr (HOPS & 1) rf.load(x, Vp, neighbour_offset<S>(site, wf, Lmu, stride, bc));
    if constexpr (HOPS & 2) rb.load(x, Vp, neighbour_offset<S>(site, wb, Lmu, -stride, bc));
    if constexpr (HOPS & 1) load_link_buf<S, REC>(a.U, MU, Vp, es, uf);
    if constexpr (HOPS & 2) load_link_buf<S, REC>(a.U, MU, Vp, eu, ub);
    cx<R> hf[2][3], hb[2][3];
    if constexpr (HOPS & 1) {
        rf.spinor(pf);
        project<MU, -1>(pf, hf);
    }
    if constexpr (HOPS & 2) {
        rb.spinor(pb);
        project<MU, +1>(pb, hb);
    }
    if (MU == 0) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (HOPS & 1) hf[k][c] = phase_mul<S>(ph, hf[k][c], k, c, a.n == 1);
                if constexpr (HOPS & 2) hb[k][c] = phase_mul<S>(cmk(ph.x, -ph.y), hb[k][c], k, c, a.n == 1);
            }
    }
    if (bc < 0.0f) {   // antiperiodic
        const uint32_t ff = wf ? 0x80000000u : 0u, fb = wb ? 0x80000000u : 0u;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (HOPS & 1) hf[k][c] = cmk(flip_sign(hf[k][c].x, ff), flip_sign(hf[k][c].y, ff));
                if constexpr (HOPS & 2) hb[k][c] = cmk(flip_sign(hb[k][c].x, fb), flip_sign(hb[k][c].y, fb));
            }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int aa = 0; aa < 3; ++aa) {
            if constexpr (HOPS & 1) {
                cx<R> t = REC && aa == 2 ? cmul_i(uf[aa][0], hf[k][0]) : cmul(uf[aa][0], hf[k][0]);
                cfma(t, uf[aa][1], hf[k][1]);
                cfma(t, uf[aa][2], hf[k][2]);
                out[(k * 3 + aa) * 64] = t;
            }
            if constexpr (HOPS & 2) {
                cx<R> w = MU == 0 ? cmulc(ub[0][aa], hb[k][0]) : cmulc_r(ub[0][aa], hb[k][0]);
                cfmac(w, ub[1][aa], hb[k][1]);
                cfmac(w, ub[2][aa], hb[k][2]);
                out[(6 + k * 3 + aa) * 64] = w;
            }
        }
}

// acc + component (SP, c) of (1 + SGN gamma_MU) expansion of g (stride 64).
template <int MU, int SGN, int SP, class R>
__device__ __forceinline__ cx<R> add_hop(cx<R> acc, const cx<R> *__restrict__ g, int c)
{
    constexpr int k = SP < 2 ? SP : (MU == 0 || MU == 1) ? 3 - SP : SP - 2;   // half-spinor row it takes
    const cx<R> v = g[(k * 3 + c) * 64];
    if constexpr (SP < 2) return cadd(acc, v);
    else if constexpr (MU == 0) return cadd(acc, SGN < 0 ? cnimul(v) : cimul(v));
    else if constexpr (MU == 1) return ((SGN < 0) == (SP == 2)) ? csub(acc, v) : cadd(acc, v);
    else if constexpr (MU == 2) return cadd(acc, ((SGN < 0) == (SP == 2)) ? cnimul(v) : cimul(v));
    else return SGN < 0 ? csub(acc, v) : cadd(acc, v);
}

// Sum of the eight hops for component K = 3 spin + colour, in hop order.
template <int K, class R>
__device__ __forceinline__ cx<R> sum_hops(const cx<R> *__restrict__ g)
{
    constexpr int SP = K / 3, H = 6 * 64;
    const int c = K % 3;
    cx<R> acc = cmk((R)0, (R)0);
    acc = add_hop<0, -1, SP>(acc, g, c);
    acc = add_hop<0, +1, SP>(acc, g + H, c);
    acc = add_hop<1, -1, SP>(acc, g + 2 * H, c);
    acc = add_hop<1, +1, SP>(acc, g + 3 * H, c);
    acc = add_hop<2, -1, SP>(acc, g + 4 * H, c);
    acc = add_hop<2, +1, SP>(acc, g + 5 * H, c);
    acc = add_hop<3, -1, SP>(acc, g + 6 * H, c);
    return add_hop<3, +1, SP>(acc, g + 7 * H, c);
}

// CAN: the output goes to the canonical layout (12 numbers per site, rows of 13
// in the LDS of the hops, which have been summed by then) instead of a field.
//
// dir_waves: eight waves, one hop each, have half the loads and arithmetic of a
// hop pair in a row; four waves are fewer to start and to meet at the barrier.
// Mean of a plain and a fused launch, four / eight waves:
//   FP64 12 RHS of 4^4 5.0 / 4.7 us, FP32 5 RHS of 6x5x7x10 4.8 / 4.4, FP32 4 RHS of 8^3x16 6.5 / 6.1,
//   FP64 4 RHS of 8^3x16 8.7 / 8.2, of 12^3x24 32.1 / 29.4, FP64 1 RHS of 16^3x32 28.9 / 27.3,
// but in batches that stream past the caches four read less again:
//   FP64 1 RHS of 24^3x48 159 / 163, 2 RHS 294 / 307, FP32 2 RHS 139 / 141,
// and a single call with canonical output is 10.2 / 10.4 us on 8^3x16.
template <class S, bool HW, bool EPI, bool REC, bool NT, bool CAN>
__global__ __launch_bounds__(dir_waves(NT, CAN) * 64, dir_waves(NT, CAN) == 8 && !(sizeof(S) == 16 && !REC) ? 4 : 2)
void k_dslash_dir(DsArgs<S> a)
{
    constexpr bool W8 = dir_waves(NT, CAN) == 8;
    using R = typename StoreT<S>::real;
    using U = UnitOf<S>;
    using T = typename U::T;
    __shared__ __align__(16) cx<R> hop[8 * 6 * 64];   // at least 24 KiB
    __shared__ int row_site[64];
    const Geo &g = a.g;
    const int Vp = g.Vp;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    // grid: x = XCDs x right-hand sides, y = site blocks of an XCD (one "XCD" for small lattices)
    const int xcd = a.xcd_remap ? (int)(blockIdx.x & 7) : 0;
    const int j = a.xcd_remap ? (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    int site;
    if (a.order == 1 || a.order == 3) site = slab_site(g, a.order, a.cols, xcd, (int)blockIdx.y * 64 + lane);
    else site = (xcd * (int)gridDim.y + (int)blockIdx.y) * 64 + lane;
    const int s = __builtin_amdgcn_readfirstlane(a.slots ? a.slots[j] : j);
    const size_t off = (size_t)s * (size_t)a.fstride;
    const S *x = a.x + off;

    const bool real = site < g.V;
    const int s0 = real ? site : 0;   // other lanes load site 0 and drop the result
    int xc, yc, zc, tc;
    site_coords(g, s0, xc, yc, zc, tc);
    // units this wave writes, from q0 on: of four waves three of twelve, or of six one for waves 0 and 1
    // (wave 0 has the background phase to apply) and two for waves 2 and 3
    // Of eight waves, 2 to 7 write one of six, or 0 to 3 one and 4 to 7 two of twelve.
    constexpr int NMINE = W8 ? (U::C == 2 ? 1 : 2) : U::C == 2 ? 2 : 3;
    const int q0 = W8 ? (U::C == 2 ? (wave < 2 ? 0 : wave - 2) : wave < 4 ? wave : 2 * wave - 4)
                      : U::C == 2 ? (wave < 2 ? wave : 2 * wave - 2) : 3 * wave;
    const int nmine = W8 ? (U::C == 2 ? (wave < 2 ? 0 : 1) : wave < 4 ? 1 : 2) : U::C == 2 ? (wave < 2 ? 1 : 2) : 3;
    T own[NMINE], ep[3][NMINE];
    const S *e[3] = {a.e1, a.e2, a.e3};
#pragma unroll
    for (int i = 0; i < NMINE; ++i) {
        const int q = i < nmine ? q0 + i : q0;
        own[i] = ld_unit<S, false>(x, Vp, q, (unsigned)s0 * (unsigned)RawSpinor<S>::B);
        if constexpr (EPI) {
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (e[t]) ep[t][i] = ld_unit<S, NT>(e[t] + off, Vp, q, (unsigned)s0 * (unsigned)RawSpinor<S>::B);
        }
    }
    // of eight waves the even ones take the forward hops (0 and 1 have the background phase)
    const int mu = W8 ? wave >> 1 : wave;
    cx<R> *out = hop + mu * 12 * 64 + lane;
    cx<R> ph = cmk((R)1, (R)0);
    if (mu == 0) {
        const int grp = a.fgroup ? a.fgroup[s] : 0;
        const cx<double> pd = a.phase[grp * g.Lt + tc];
        ph = cmk((R)pd.x, (R)pd.y);
    }
    auto hops = [&](auto h) {
        constexpr int H = decltype(h)::value;
        if (mu == 0) dir_hops<0, H, S, REC>(a, x, s0, xc, g.Lx, 1, ph, out);
        else if (mu == 1) dir_hops<1, H, S, REC>(a, x, s0, yc, g.Ly, g.Lx, ph, out);
        else if (mu == 2) dir_hops<2, H, S, REC>(a, x, s0, zc, g.Lz, g.Lxy, ph, out);
        else dir_hops<3, H, S, REC>(a, x, s0, tc, g.Lt, g.Lxyz, ph, out);
    };
    if constexpr (!W8) hops(std::integral_constant<int, 3>{});
    else if (wave & 1) hops(std::integral_constant<int, 2>{});
    else hops(std::integral_constant<int, 1>{});
    if (CAN && wave == 0) row_site[lane] = site;
    __syncthreads();
    if (!CAN && site >= Vp) return;   // beyond the slab or the lattice

    const R diag = (R)a.diag, sc = (R)a.a;
    const R cc[3] = {(R)a.c1, (R)a.c2, (R)a.c3};
    const cx<R> *hp = hop + lane;
    R sg[NMINE];   // gamma5: the second half of the units (taken before the waves part; hipcc 7.2 lost it there)
#pragma unroll
    for (int i = 0; i < NMINE; ++i) sg[i] = (HW && q0 + i >= U::N / 2) ? -sc : sc;
    auto finish = [&](auto qc, int i) {
        constexpr int Q = decltype(qc)::value;
        cx<R> acc[U::C];
        acc[0] = sum_hops<Q * U::C>(hp);
        if constexpr (U::C == 2) acc[1] = sum_hops<Q * U::C + 1>(hp);
        T v;
#pragma unroll
        for (int h = 0; h < U::C; ++h) {
            v.c[h] = cscale(site_term(diag, own[i].c[h], acc[h]), sg[i]);
            if constexpr (EPI) {
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    if (e[t]) v.c[h] = add_scaled(v.c[h], cc[t], ep[t][i].c[h]);
            }
            if (!real) v.c[h] = cmk((R)0, (R)0);   // padding sites hold zeros in every field
        }
        if constexpr (CAN) own[i] = v;
        else st_unit<S, NT>(a.y + off, Vp, Q, (unsigned)site, v);
    };
#define OV_UNIT(Q, I) finish(std::integral_constant<int, Q>{}, I)
    if constexpr (W8 && U::C == 2) {
        if (wave == 2) { OV_UNIT(0, 0); }
        else if (wave == 3) { OV_UNIT(1, 0); }
        else if (wave == 4) { OV_UNIT(2, 0); }
        else if (wave == 5) { OV_UNIT(3, 0); }
        else if (wave == 6) { OV_UNIT(4, 0); }
        else if (wave == 7) { OV_UNIT(5, 0); }
    } else if constexpr (W8) {
        if (wave == 0) { OV_UNIT(0, 0); }
        else if (wave == 1) { OV_UNIT(1, 0); }
        else if (wave == 2) { OV_UNIT(2, 0); }
        else if (wave == 3) { OV_UNIT(3, 0); }
        else if (wave == 4) { OV_UNIT(4, 0); OV_UNIT(5, 1); }
        else if (wave == 5) { OV_UNIT(6, 0); OV_UNIT(7, 1); }
        else if (wave == 6) { OV_UNIT(8, 0); OV_UNIT(9, 1); }
        else { OV_UNIT(10, 0); OV_UNIT(11, 1); }
    } else if constexpr (U::C == 2) {
        if (wave == 0) { OV_UNIT(0, 0); }
        else if (wave == 1) { OV_UNIT(1, 0); }
        else if (wave == 2) { OV_UNIT(2, 0); OV_UNIT(3, 1); }
        else { OV_UNIT(4, 0); OV_UNIT(5, 1); }
    } else {
        if (wave == 0) { OV_UNIT(0, 0); OV_UNIT(1, 1); OV_UNIT(2, 2); }
        else if (wave == 1) { OV_UNIT(3, 0); OV_UNIT(4, 1); OV_UNIT(5, 2); }
        else if (wave == 2) { OV_UNIT(6, 0); OV_UNIT(7, 1); OV_UNIT(8, 2); }
        else { OV_UNIT(9, 0); OV_UNIT(10, 1); OV_UNIT(11, 2); }
    }
#undef OV_UNIT
    if constexpr (CAN) {
        constexpr int ROW = 13;
        double2 *tr = reinterpret_cast<double2 *>(hop);
        __syncthreads();   // the hops have been summed
#pragma unroll
        for (int i = 0; i < NMINE; ++i)
            if (i < nmine)
#pragma unroll
                for (int h = 0; h < U::C; ++h)
                    tr[lane * ROW + (q0 + i) * U::C + h] = stored_value<S>(own[i].c[h]);
        __syncthreads();
        double2 *yc = a.yc + (long)j * g.V * 12;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int e = (int)threadIdx.x + 256 * r, row = e / 12, k = e - 12 * row;
            if (row_site[row] < g.V) yc[(long)row_site[row] * 12 + k] = tr[row * ROW + k];
        }
    }
}

template <class S, bool REC, bool NT>
static void launch_dir_kernel(const DsArgs<S> &b, bool hw, bool epi, dim3 grid, hipStream_t st)
{
    const dim3 blk(64 * dir_waves(NT, b.yc != nullptr));
    if (epi) hipLaunchKernelGGL((k_dslash_dir<S, true, true, REC, NT, false>), grid, blk, 0, st, b);
    else if (b.yc && hw) hipLaunchKernelGGL((k_dslash_dir<S, true, false, REC, NT, true>), grid, blk, 0, st, b);
    else if (b.yc) hipLaunchKernelGGL((k_dslash_dir<S, false, false, REC, NT, true>), grid, blk, 0, st, b);
    else if (hw) hipLaunchKernelGGL((k_dslash_dir<S, true, false, REC, NT, false>), grid, blk, 0, st, b);
    else hipLaunchKernelGGL((k_dslash_dir<S, false, false, REC, NT, false>), grid, blk, 0, st, b);
}

template <class S>
hipError_t launch_dslash_dir(const DsArgs<S> &a, bool hw, bool epi, hipStream_t st)
{
    if (a.n <= 0) return hipSuccess;
    DsArgs<S> b = a;
    b.cols = 1;
    if (b.order == 1 && (a.g.Lz % 8 != 0 || a.g.V % 64 != 0)) b.order = 0;
    if (b.order == 3 && (a.g.Lt % 8 != 0 || a.g.V % 64 != 0)) b.order = 0;
    const int nsb = a.g.Vp / 64;
    // from 64 site blocks on, each XCD takes a contiguous run of them, and the right-hand sides of a
    // site block follow each other on its XCD (they share the links in its L2)
    b.xcd_remap = (b.order != 0 || nsb >= 64) ? 1 : 0;
    const int ny = b.order != 0 ? (a.g.V / 8 + 63) / 64 : b.xcd_remap ? (nsb + 7) / 8 : nsb;
    if (!dslash_dir_fits(a.g) || a.n > (1 << 24) || (epi && a.yc)) return hipErrorInvalidValue;
    const dim3 grid(b.xcd_remap ? 8 * a.n : a.n, ny);
    // BF16 batches of this kernel are far smaller than the caches: they take no stream hint
    auto launch = [&](auto rec) {
        constexpr bool REC = decltype(rec)::value;
        if constexpr (sizeof(S) != 4)
            if (a.stream_hint) return launch_dir_kernel<S, REC, true>(b, hw, epi, grid, st);
        launch_dir_kernel<S, REC, false>(b, hw, epi, grid, st);
    };
    if (a.recon) launch(std::true_type{});
    else launch(std::false_type{});
    return hipGetLastError();
}

template hipError_t launch_dslash_dir<double2>(const DsArgs<double2> &, bool, bool, hipStream_t);
template hipError_t launch_dslash_dir<float2>(const DsArgs<float2> &, bool, bool, hipStream_t);
template hipError_t launch_dslash_dir<uint32_t>(const DsArgs<uint32_t> &, bool, bool, hipStream_t);

}  // namespace ov
