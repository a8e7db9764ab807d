// H_w / D_w of large batches: waves that share the links of their sites.
//
// Same operator and epilogue as the site-parallel kernels, and the same bits:
//   y_r = a * G (D_w x_r)  +  c1 e1_r + c2 e2_r + c3 e3_r          (own site)
//
// The W waves of a workgroup (2 to 8) cover the same 64 sites, each for one
// right-hand side.  The eight links of a site are staged in LDS once per
// workgroup, so that they cross HBM once per W vectors.
//
// What bounds it: FP64 and FP32 the traffic beyond L2 (plain H_w of 12 FP32
// vectors on 24^3x48: 3.4 GB at 5.9 TB/s, 1.8 GB of it neighbours read again),
// BF16 the vector arithmetic.  So loads take their addresses from scalar
// resources, boundaries cost no branch (the staged link holds the sign of an
// antiperiodic hop; a Dirichlet neighbour is fetched from beyond the plane, which
// reads as zero, and its link is packed as zeros), and with straight code the
// next neighbours are requested while one is worked on.  Mean of a plain and a
// fused launch of 12 vectors against the kernel with a branch per hop and 64-bit
// lane addresses, same shape (FP64 W 4, else W 8; z-slabs with the stream hint):
//   16^3x32  FP64 303 -> 264 us, FP32 146 -> 132, BF16 98 -> 101
//   24^3x48  FP64 1502 -> 1461,  FP32 727 -> 702, BF16 507 -> 456
// BF16 takes canonical order on 16^3x32, where that is 96 -> 91 (5 vectors 45 -> 39).
// Fewer workgroups per CU cut the traffic (two of six waves: 2.6 GB) but leave
// too few loads in flight to gain from it.
#include <type_traits>
#include <utility>

#include "dslash_site.h"

namespace ov {

// The sums are final here: keeps the compiler from putting off the arithmetic
// of a hop, with its links and neighbour held in registers, behind the loads
// of the next.
template <class R>
__device__ __forceinline__ void settle(cx<R> (&acc)[4][3])
{
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
        asm volatile("" : "+v"(acc[sp][0].x), "+v"(acc[sp][0].y), "+v"(acc[sp][1].x), "+v"(acc[sp][1].y),
                          "+v"(acc[sp][2].x), "+v"(acc[sp][2].y));
}

// acc += hop H (2 mu: forward, 2 mu + 1: backward) of the neighbour `raw`.
// `flip`: sign bit of the boundary multiplier where the stage does not hold
// it (FP64 with two rows: the sign of a rebuilt row would square away).
template <int H, class S, class LF>
__device__ __forceinline__ void add_shared_hop(const RawSpinor<S> &raw, const LF &links, uint32_t flip,
                                               cx<typename StoreT<S>::real> ph, bool single,
                                               cx<typename StoreT<S>::real> (&acc)[4][3])
{
    using R = typename StoreT<S>::real;
    constexpr int MU = H / 2, SGN = H % 2 ? 1 : -1;
    cx<R> p[4][3], h[2][3], g[2][3], u[3][3];
    raw.spinor(p);
    project<MU, SGN>(p, h);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if constexpr (MU == 0) h[k][c] = phase_mul<S>(SGN < 0 ? ph : cmk(ph.x, -ph.y), h[k][c], k, c, single);
            if constexpr (LF::RB) h[k][c] = cmk(flip_sign(h[k][c].x, flip), flip_sign(h[k][c].y, flip));
        }
    links(MU, SGN < 0 ? MU : 4 + MU, 0u, u);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int aa = 0; aa < 3; ++aa) {
            cx<R> t;
            if constexpr (SGN < 0) {
                t = LF::rebuilt && aa == 2 ? cmul_i(u[aa][0], h[k][0]) : cmul(u[aa][0], h[k][0]);
                cfma(t, u[aa][1], h[k][1]);
                cfma(t, u[aa][2], h[k][2]);
            } else {
                t = MU == 0 ? cmulc(u[0][aa], h[k][0]) : cmulc_r(u[0][aa], h[k][0]);
                cfmac(t, u[1][aa], h[k][1]);
                cfmac(t, u[2][aa], h[k][2]);
            }
            g[k][aa] = t;
        }
    expand_add<MU, SGN>(acc, g);
}

// Neighbours requested ahead.  Two fill the registers of four waves per SIMD
// (FP64: two); BF16 spends its time on arithmetic and does better with more
// waves (24^3x48, 12 RHS, one / two ahead: FP32 770 / 719 us, FP64 1530 / 1511,
// both before the epilogue below, BF16 470 / 494).
template <class S>
constexpr int share_depth() { return sizeof(S) == 4 ? 1 : 2; }

// Units of the own-site operands requested ahead in a fused launch.  FP64 has
// two waves per SIMD and twice the units of FP32; loaded one unit after the
// other, behind the stores, each cost a memory latency, and the kernel was
// behind the one that it replaced, which runs three waves per SIMD.  Microseconds
// per vector of a fused launch, 12 RHS on z-slabs with the stream hint, that
// kernel / none ahead / six ahead: 24^3x48 147.8 / 149.5 / 143.4, 24^3x24 72.6 /
// 75.9 / 71.5, 16^3x32 30.2 / 29.1 / 26.5, 32^3x32 247 / 244 / 239.  Small lattices
// lose nothing with six, 1 % with two or three in places (mean of a step, 24 RHS of
// 8^3x16, none / two / three / six: 33.6 / 34.4 / 33.9 / 32.7).  FP32 and BF16 hide
// it behind four waves and more.
template <class S>
constexpr int share_epilogue_depth() { return sizeof(S) == 16 ? 6 : 0; }

// LDS of a wave for the canonical output: four components of 64 sites, rows of
// five numbers (20 dwords: 16 lanes of a 16-byte access meet in no bank).
constexpr int kCanonRow = 5, kCanonWave = 64 * kCanonRow;

// Orders the LDS accesses of a wave's lanes before and after it.  The hardware
// keeps them in order; the fences hold the compiler to it, which the barrier
// alone does not (no instruction comes of either).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// CAN: the output goes to the canonical layout (12 numbers per site), four
// components at a time through LDS, so that a store covers 16 sites with 64
// bytes each and the pass that would convert it is not needed.
template <class S, bool HW, bool EPI, bool REC, bool NT, bool CAN>
__global__ __launch_bounds__(512, sizeof(S) == 16 ? 2 : 4) void k_dslash_share(DsArgs<S> a)
{
    using R = typename StoreT<S>::real;
    using Raw = RawSpinor<S>;
    constexpr int SL = 64, E = lds_link_components<R, REC>();
    extern __shared__ __align__(16) unsigned char lds_raw[];
    cx<R> *lk = reinterpret_cast<cx<R> *>(lds_raw);   // [8][E][64]
    const Geo &g = a.g;
    const int W = (int)(blockDim.x >> 6), lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int site = site_in_block(g, a.order, a.xcd_remap, a.cols, lane, 64);
    const bool real = site < g.V;
    const int s0 = real ? site : 0;   // other lanes load site 0 and drop the result
    int xc, yc, zc, tc;
    site_coords(g, s0, xc, yc, zc, tc);
    for (int slot = wave; slot < 8; slot += W) {
        cx<R> *dst = lk + slot * E * SL + lane;
        stage_link<S, R, REC, E, SL>(a, slot, s0, xc, yc, zc, tc, dst);
        if constexpr (E == 9) {   // antiperiodic hops: the link carries the sign
            const int mu = slot & 3;
            const int c = mu == 0 ? xc : mu == 1 ? yc : mu == 2 ? zc : tc;
            const int L = mu == 0 ? g.Lx : mu == 1 ? g.Ly : mu == 2 ? g.Lz : g.Lt;
            if (g.bcf[mu] < 0 && c == (slot < 4 ? L - 1 : 0))
#pragma unroll
                for (int k = 0; k < 9; ++k) dst[k * SL] = cmk(-dst[k * SL].x, -dst[k * SL].y);
        }
    }

    const int j = (int)blockIdx.y * W + wave;
    const bool act = j < a.n;
    const int s = __builtin_amdgcn_readfirstlane(a.slots && act ? a.slots[j] : act ? j : 0);
    const size_t off = (size_t)s * (size_t)a.fstride;
    const S *x = a.x + off;
    const bool wr[8] = {xc == g.Lx - 1, xc == 0, yc == g.Ly - 1, yc == 0, zc == g.Lz - 1, zc == 0, tc == g.Lt - 1, tc == 0};
    auto nb = [&](int h) {
        const int mu = h / 2;
        const int st = mu == 0 ? 1 : mu == 1 ? g.Lx : mu == 2 ? g.Lxy : g.Lxyz;
        const int L = mu == 0 ? g.Lx : mu == 1 ? g.Ly : mu == 2 ? g.Lz : g.Lt;
        return neighbour_offset<S>(s0, wr[h], L, h % 2 ? -st : st, g.bcf[mu]);
    };
    auto flip = [&](int h) { return wr[h] && g.bcf[h / 2] < 0.0f ? 0x80000000u : 0u; };
    const int grp = __builtin_amdgcn_readfirstlane(a.fgroup ? a.fgroup[s] : 0);
    const cx<double> pd = a.phase[grp * g.Lt + tc];
    const cx<R> ph = cmk((R)pd.x, (R)pd.y);
    const bool single = a.n == 1;

    // the neighbours of the next D hops are on their way while one is worked on
    constexpr int D = share_depth<S>();
    Raw buf[D + 1];
    auto fetch = [&](auto hc) {
        constexpr int H = decltype(hc)::value;
        if constexpr (H < 8) buf[H % (D + 1)].load(x, g.Vp, nb(H));
        else if constexpr (H == 8) buf[8 % (D + 1)].load(x, g.Vp, (unsigned)s0 * (unsigned)Raw::B);   // the site itself
    };
    if (act) {
        fetch(std::integral_constant<int, 0>{});
        if constexpr (D > 1) fetch(std::integral_constant<int, 1>{});
    }
    __syncthreads();
    if (!act || (!CAN && site >= g.Vp)) return;
    const LdsLinks<R, E, REC, SL> lf{lk, lane};
    cx<R> acc[4][3];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[sp][c] = cmk((R)0, (R)0);
    auto hop = [&](auto hc) {
        constexpr int H = decltype(hc)::value;
        fetch(std::integral_constant<int, H + D>{});
        add_shared_hop<H>(buf[H % (D + 1)], lf, flip(H), ph, single, acc);
        settle(acc);
    };
    hop(std::integral_constant<int, 0>{});
    hop(std::integral_constant<int, 1>{});
    hop(std::integral_constant<int, 2>{});
    hop(std::integral_constant<int, 3>{});
    hop(std::integral_constant<int, 4>{});
    hop(std::integral_constant<int, 5>{});
    hop(std::integral_constant<int, 6>{});
    hop(std::integral_constant<int, 7>{});

    const R diag = (R)a.diag, sc = (R)a.a;
    const R cc[3] = {(R)a.c1, (R)a.c2, (R)a.c3};
    const S *ep[3] = {a.e1, a.e2, a.e3};
    const unsigned ob = (unsigned)s0 * (unsigned)Raw::B;
    // own-site operands, A units ahead of their use
    constexpr int A = share_epilogue_depth<S>();
    uint32_t eb[A + 1][3][Raw::B / 4];
    auto operands = [&](int q) {
        if constexpr (EPI) {
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (ep[t]) Raw::template ld<NT ? 2 : 0>(ep[t] + off, g.Vp, q, ob, eb[q % (A + 1)][t]);
        }
    };
#pragma unroll
    for (int q = 0; q < A; ++q) operands(q);
#pragma unroll
    for (int q = 0; q < Raw::N; ++q) {
        if (q + A < Raw::N) operands(q + A);
        const auto &er = eb[q % (A + 1)];
        cx<R> v[Raw::C];
#pragma unroll
        for (int h = 0; h < Raw::C; ++h) {
            const int k = q * Raw::C + h;
            v[h] = cscale(site_term(diag, Raw::get(buf[8 % (D + 1)].w[q], h), acc[k / 3][k % 3]), (HW && k >= 6) ? -sc : sc);
            if constexpr (EPI) {
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    if (ep[t]) v[h] = add_scaled(v[h], cc[t], Raw::get(er[t], h));
            }
            if (!real) v[h] = cmk((R)0, (R)0);   // padding sites hold zeros in every field
        }
        S *y = a.y + off;
        if constexpr (CAN) {
            double2 *tr = reinterpret_cast<double2 *>(lds_raw + 8 * E * SL * sizeof(cx<R>)) + wave * kCanonWave;
#pragma unroll
            for (int h = 0; h < Raw::C; ++h) tr[lane * kCanonRow + (q * Raw::C + h) % 4] = stored_value<S>(v[h]);
            if ((q * Raw::C + Raw::C) % 4 == 0) {   // four components are there: the wave writes them
                const int k0 = q * Raw::C + Raw::C - 4;
                wave_lds_sync();
                double2 *yc = a.yc + (long)j * g.V * 12;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * r + (lane >> 2), srow = __shfl(site, row, 64);
                    const double2 o = tr[row * kCanonRow + (lane & 3)];
                    if (srow < g.V) {
                        ov_d2 w = {o.x, o.y};
                        __builtin_nontemporal_store(w, (ov_d2 *)(yc + (long)srow * 12 + k0 + (lane & 3)));
                    }
                }
                wave_lds_sync();   // read before the next four take their place
            }
        } else if constexpr (Raw::C == 2) {
            if constexpr (NT) stpair_nt<S, R>(y, g.Vp, q, (unsigned)site, v[0], v[1]);
            else stpair<S, R>(y, g.Vp, q, (unsigned)site, v[0], v[1]);
        } else {
            if constexpr (NT) stp_nt<S, R>(y + (size_t)q * (unsigned)g.Vp, (unsigned)site, v[0]);
            else stp<S, R>(y + (size_t)q * (unsigned)g.Vp, (unsigned)site, v[0]);
        }
    }
}

template <class S, bool HW, bool EPI, bool REC, bool NT, bool CAN>
static hipError_t launch_share_kernel(const DsArgs<S> &b, dim3 grid, size_t lds, hipStream_t st)
{
    if (lds > 64 * 1024) {   // more than the default limit of dynamic LDS
        const hipError_t e = hipFuncSetAttribute((const void *)k_dslash_share<S, HW, EPI, REC, NT, CAN>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_dslash_share<S, HW, EPI, REC, NT, CAN>), grid, dim3(64 * b.wshare), lds, st, b);
    return hipGetLastError();
}

template <class S, bool REC, bool NT>
static hipError_t launch_share_mode(const DsArgs<S> &b, bool hw, bool epi, dim3 grid, size_t lds, hipStream_t st)
{
    if (epi) return launch_share_kernel<S, true, true, REC, NT, false>(b, grid, lds, st);
    if (b.yc) return hw ? launch_share_kernel<S, true, false, REC, NT, true>(b, grid, lds, st)
                        : launch_share_kernel<S, false, false, REC, NT, true>(b, grid, lds, st);
    return hw ? launch_share_kernel<S, true, false, REC, NT, false>(b, grid, lds, st)
              : launch_share_kernel<S, false, false, REC, NT, false>(b, grid, lds, st);
}

template <class S>
hipError_t launch_dslash_share(const DsArgs<S> &a, bool hw, bool epi, hipStream_t st)
{
    using R = typename StoreT<S>::real;
    if (a.n <= 0) return hipSuccess;
    if (a.wshare < 2 || a.wshare > 8 || (epi && a.yc)) return hipErrorInvalidValue;
    DsArgs<S> b = a;
    int nbx = site_blocks(b, 64);
    const int E = a.recon ? lds_link_components<R, true>() : lds_link_components<R, false>();
    const size_t need = (size_t)8 * E * 64 * sizeof(cx<R>) + (a.yc ? (size_t)a.wshare * kCanonWave * sizeof(double2) : 0);
    const size_t cap = a.blocks_per_cu > 0 ? (size_t)(160 * 1024) / (size_t)a.blocks_per_cu - 256 : 0;
    const size_t lds = need > cap ? need : cap;
    const dim3 grid(nbx, (a.n + a.wshare - 1) / a.wshare);
    if (a.recon)
        return a.stream_hint ? launch_share_mode<S, true, true>(b, hw, epi, grid, lds, st)
                             : launch_share_mode<S, true, false>(b, hw, epi, grid, lds, st);
    return a.stream_hint ? launch_share_mode<S, false, true>(b, hw, epi, grid, lds, st)
                         : launch_share_mode<S, false, false>(b, hw, epi, grid, lds, st);
}

template hipError_t launch_dslash_share<double2>(const DsArgs<double2> &, bool, bool, hipStream_t);
template hipError_t launch_dslash_share<float2>(const DsArgs<float2> &, bool, bool, hipStream_t);
template hipError_t launch_dslash_share<uint32_t>(const DsArgs<uint32_t> &, bool, bool, hipStream_t);

}  // namespace ov
