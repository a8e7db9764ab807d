// Wilson force of the sign-function adjoint (background field, Sec. 4,
// eq. (3); the links U~ = exp(i q eta t) U are the differentiated variables).
//
// A term Re<u, dQ v> with dQ = gamma5 dD_w / norm contributes, per link,
//   G_mu(x) += -(w b / 2) [ sum_s ((1-gamma_mu) gamma5 u(x))_s v(x+mu)_s^dag
//                         + sum_s v(x)_s ((1+gamma_mu) gamma5 u(x+mu))_s^dag ]
// (w = coef, which carries 1/norm; b the boundary multiplier of the hop), so
// that dL = sum Re tr(G^dag dU~).  The accumulator G lives in FP64 planes
// [mu][3a+b][Vp]; one thread owns one forward link.
//
// (1 -/+ gamma_mu) is Hermitian, so both spin sums run over half spinors: the
// first is sum_k P-(gamma5 u(x))_k P-(v(x+mu))_k^dag with the rank-two
// projections P-, the second sum_k P+(v(x))_k P+(gamma5 u(x+mu))_k^dag.
//
// What bounds it is the accumulator, 576 bytes read and written per site
// against 384 of a pair of vectors.  A launch therefore takes the two terms of
// a recursion step with one pass over G, and the four waves of a workgroup take one
// direction each of the same 64 sites, which keeps the vectors of a site in
// one CU's cache and the loads of a thread few.  16^3x32, among the launches of
// the sweep: two terms 70 us (5.0 TB/s past L2), against 2 x 60.5 us for a thread
// that walked the four directions of one.
#include "dslash_device.h"
#include "ov_internal.h"

namespace ov {

template <int MU>
__device__ __forceinline__ void force_dir(const ForceArgs &a, int site, int cmu, int Lmu, int stride)
{
    using Raw = RawSpinor<double2>;
    const Geo &g = a.g;
    const bool wrap = (cmu == Lmu - 1);
    const unsigned es = (unsigned)site * (unsigned)Raw::B;
    const unsigned ej = neighbour_offset<double2>(site, wrap, Lmu, stride, g.bcf[MU]);
    cx<double> sum[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) sum[r][c] = cmk(0.0, 0.0);
    for (int i = 0; i < a.n; ++i) {
        Raw ru, rv, ruj, rvj;
        ru.load(a.u[i], g.Vp, es);
        rvj.load(a.v[i], g.Vp, ej);
        rv.load(a.v[i], g.Vp, es);
        ruj.load(a.u[i], g.Vp, ej);
        const double fac = -0.5 * a.coef[i] * (wrap ? (double)g.bcf[MU] : 1.0);
        cx<double> p[4][3], hl[2][3], hr[2][3];
        auto add = [&]() {   // sum += fac sum_k hl_k hr_k^dag
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    cx<double> t = cmulc(hr[0][c], hl[0][r]);
                    cfmac(t, hr[1][c], hl[1][r]);
                    sum[r][c] = cmk(fma(fac, t.x, sum[r][c].x), fma(fac, t.y, sum[r][c].y));
                }
        };
        auto gamma5 = [&]() {
#pragma unroll
            for (int s = 2; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < 3; ++c) p[s][c] = cmk(-p[s][c].x, -p[s][c].y);
        };
        ru.spinor(p);
        gamma5();
        project<MU, -1>(p, hl);
        rvj.spinor(p);
        project<MU, -1>(p, hr);
        add();
        rv.spinor(p);
        project<MU, +1>(p, hl);
        ruj.spinor(p);
        gamma5();
        project<MU, +1>(p, hr);
        add();
    }
    if (wrap && g.bcf[MU] == 0.0f) return;   // no hop, no term
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const long k = (long)(MU * 9 + r * 3 + c) * g.Vp + site;
            const double2 o = a.G[k];
            a.G[k] = make_double2(o.x + sum[r][c].x, o.y + sum[r][c].y);
        }
}

__global__ __launch_bounds__(256, 2) void k_force(ForceArgs a)
{
    const Geo &g = a.g;
    // each XCD takes a contiguous run of site blocks
    const int per = (int)(gridDim.x >> 3);
    const int site = (((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3)) * 64 + (int)(threadIdx.x & 63);
    if (site >= g.V) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int xc, yc, zc, tc;
    site_coords(g, site, xc, yc, zc, tc);
    if (wave == 0) force_dir<0>(a, site, xc, g.Lx, 1);
    else if (wave == 1) force_dir<1>(a, site, yc, g.Ly, g.Lx);
    else if (wave == 2) force_dir<2>(a, site, zc, g.Lz, g.Lxy);
    else force_dir<3>(a, site, tc, g.Lt, g.Lxyz);
}

// Canonical gradient of the base links and per-block partial dL/deta:
//   gU_mu = G_mu, except gU_0 = exp(-i q eta t) G_0;
//   dL/deta = sum_x Re tr(G_0^dag i q t U~_0),  U~_0 = exp(i q eta t) U_0.
__global__ __launch_bounds__(256) void k_force_finish(const double2 *__restrict__ G, const double2 *__restrict__ U,
                                                      const cx<double> *phase_row, double q, Geo g,
                                                      double2 *gU, double *eta_part)
{
    const int site = blockIdx.x * blockDim.x + threadIdx.x;
    double et = 0.0;
    if (site < g.V) {
        const int tc = site / g.Lxyz;
        const cx<double> ph = phase_row[tc];
        for (int mu = 0; mu < 4; ++mu)
            for (int k = 0; k < 9; ++k) {
                const double2 gk = G[(long)(mu * 9 + k) * g.Vp + site];
                cx<double> gv = {gk.x, gk.y};
                if (mu == 0) {
                    const double2 uk = U[(long)k * g.Vp + site];   // packed FP64 link planes, mu = 0
                    // Re(conj(G~) * i q t ph U)
                    cx<double> ut = cmul(ph, cmk(uk.x, uk.y));
                    cx<double> iu = cmk(-q * tc * ut.y, q * tc * ut.x);
                    et += gv.x * iu.x + gv.y * iu.y;
                    gv = cmulc(ph, gv);   // conj(ph) * G~
                }
                if (gU) gU[((long)mu * g.V + site) * 9 + k] = make_double2(gv.x, gv.y);
            }
    }
    __shared__ double sh[256];
    sh[threadIdx.x] = et;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) eta_part[blockIdx.x] = sh[0];
}

hipError_t launch_force(const ForceArgs &a, hipStream_t st)
{
    if (a.n < 1 || a.n > kForcePairs) return hipErrorInvalidValue;
    const int nb = ((a.g.V + 63) / 64 + 7) & ~7;
    hipLaunchKernelGGL(k_force, dim3(nb), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_force_finish(const double2 *G, const double2 *U, const cx<double> *phase_row, double q, Geo g,
                               double2 *gU, double *eta_part, int nb, hipStream_t st)
{
    hipLaunchKernelGGL(k_force_finish, dim3(nb), dim3(256), 0, st, G, U, phase_row, q, g, gU, eta_part);
    return hipGetLastError();
}

}  // namespace ov
