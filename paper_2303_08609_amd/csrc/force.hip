// Link derivative of the bilinear form coeff * Re <Lambda, H R> (the hopping
// term of paper Eq. (1)) for full-lattice fields given as packed even and odd
// parts.  The link U_mu(x) enters H in the forward term at x (projector
// 1 - gamma_mu, boundary phase b) and in the backward term at x + mu
// (projector 1 + gamma_mu, phase conj(b)); collecting the coefficients of dU
// gives, with dL = Re tr(g^dag dU),
//
//   g = coeff conj(b) [ sum_s w_s v_s^dag + sum_s v'_s w'_s^dag ],
//   w = (1 - gamma_mu) Lambda(x),  v = R(x + mu),
//   v' = R(x),  w' = (1 + gamma_mu) Lambda(x + mu).
//
// With project, F = TH(i U g^dag) is written (TH: traceless Hermitian part),
// the su(3) force for U -> exp(i eps X) U.
//
// The projectors have rank 2 and are, up to the factor 2, their own squares,
// so the spin sums run over the two independent rows of half spinors:
//   sum_s w_s v_s^dag = sum_{s < 2} h_s k_s^dag,
//   h = half[(1 - gamma_mu) Lambda(x)],  k = half[(1 - gamma_mu) R(x + mu)]
// (twice that for t, whose half spinors carry no factor 2), and the same with
// (1 + gamma_mu) for the second sum.
//
// One workgroup per 64 consecutive half indices and two directions, one
// wavefront per parity and direction: both are uniform in a wavefront, whose
// records lie side by side in one field (in canonical order neighbouring
// lanes alternate between the two parities' fields, which doubles the cache
// lines of every load), and the two parities are 128 consecutive sites.  The
// 3x3 results are turned through LDS and written to the canonical gauge
// layout [4][Lt][Lz][Ly][Lx][3][3] as consecutive words, where a lane writing
// its own matrix leaves 144 bytes between the lanes of a store.  FP64
// throughout.
// 16^3x32: FP64 gradient 80.7 -> 44.2 us (125 MB at least, 20 us); the
// rest is the latency of the two rounds of record loads at 3 wavefronts per
// SIMD.
#include "half_spinor.h"
#include "weo_internal.h"

namespace weo {

struct ForceParams {
    Geom g;
    double ph[4][2];
    const uint8_t* u;
    size_t link_block;
    const uint8_t* lam[2];      // Lambda, R by parity
    const uint8_t* r[2];
    double coeff;
    int project, accumulate;
};

constexpr int kForceRow = 129;  // elements of an LDS row of 128 sites

template <int SP> __device__ __forceinline__ void load_wide(const uint8_t* base, uint32_t n, uint32_t i, double2* v) {
    cx<typename St<SP>::real> w[12];
    load_rec<SP, 12>(base, n, i, w);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = make_double2(w[k].x, w[k].y);
}

// G += sum_{s < 2} a_s b_s^dag
__device__ __forceinline__ void outer_add(const double2* a, const double2* b, double2* G) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) G[3 * i + j] = fma_(a[3 * s + i], conj_(b[3 * s + j]), G[3 * i + j]);
}

// The gradient (force) of link MU at a site of parity par, half index ih.
template <int SP, int LP, bool L12, int MU>
__device__ __forceinline__ void link_gradient(const ForceParams& P, uint32_t ih, int par, const Nbr& nb, double2* G) {
    const uint32_t n = P.g.vh, jh = nb.i[2 * MU];
    double2 a[12], b[12], h[6], k[6];
#pragma unroll
    for (int e = 0; e < 9; ++e) G[e] = make_double2(0.0, 0.0);
    load_wide<SP>(P.lam[par], n, ih, a);
    load_wide<SP>(P.r[1 - par], n, jh, b);
    half_project<MU, 1>(a, h);
    half_project<MU, 1>(b, k);
    outer_add(h, k, G);
    load_wide<SP>(P.r[par], n, ih, a);
    load_wide<SP>(P.lam[1 - par], n, jh, b);
    half_project<MU, -1>(a, h);
    half_project<MU, -1>(b, k);
    outer_add(h, k, G);
    // coeff * conj(b), and the 2 of the t projectors
    double2 f = nb.edge[2 * MU] ? make_double2(P.ph[MU][0], -P.ph[MU][1]) : make_double2(1.0, 0.0);
    f = scal((MU == 3 ? 2.0 : 1.0) * P.coeff, f);
#pragma unroll
    for (int e = 0; e < 9; ++e) G[e] = mul(f, G[e]);
    if (!P.project) return;
    // F = TH(i U G^dag)
    double2 U[9], Y[9];
    cx<typename St<LP>::real> w[9];
    load_rec<LP, L12 ? 6 : 9>(P.u + (size_t)(2 * MU + par) * P.link_block, n, ih, w);
#pragma unroll
    for (int e = 0; e < (L12 ? 6 : 9); ++e) U[e] = make_double2(w[e].x, w[e].y);
    if constexpr (L12) {        // the third row in FP64
        U[6] = conj_(sub(mul(U[1], U[5]), mul(U[2], U[4])));
        U[7] = conj_(sub(mul(U[2], U[3]), mul(U[0], U[5])));
        U[8] = conj_(sub(mul(U[0], U[4]), mul(U[1], U[3])));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double2 acc = make_double2(0.0, 0.0);
#pragma unroll
            for (int q = 0; q < 3; ++q) acc = fma_(U[3 * i + q], conj_(G[3 * j + q]), acc);
            Y[3 * i + j] = imul(acc);
        }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) G[3 * i + j] = scal(0.5, add(Y[3 * i + j], conj_(Y[3 * j + i])));
    const double tr = (G[0].x + G[4].x + G[8].x) / 3.0;
    G[0].x -= tr; G[4].x -= tr; G[8].x -= tr;
    G[0].y = 0.0; G[4].y = 0.0; G[8].y = 0.0;
}

template <int SP, int LP, bool L12, class CR>
__global__ void __launch_bounds__(256, 2) k_force(const ForceParams P, typename cx_t<CR>::type* out) {
    __shared__ double2 lds[2][9 * kForceRow];
    const uint32_t lane = threadIdx.x & 63u;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int par = wv & 1, mu = 2 * (int)blockIdx.y + (wv >> 1);
    const uint32_t first = xcd_block(blockIdx.x, gridDim.x, 1) * 64, ih = first + lane;
    double2* row = lds[wv >> 1];
    if (ih < P.g.vh) {
        const Site s = decode(P.g, ih, par);
        const Nbr nb = neighbours(P.g, s);
        double2 G[9];
        switch (mu) {
            case 0: link_gradient<SP, LP, L12, 0>(P, ih, par, nb, G); break;
            case 1: link_gradient<SP, LP, L12, 1>(P, ih, par, nb, G); break;
            case 2: link_gradient<SP, LP, L12, 2>(P, ih, par, nb, G); break;
            default: link_gradient<SP, LP, L12, 3>(P, ih, par, nb, G); break;
        }
        const uint32_t pos = 2 * lane + (uint32_t)(s.x & 1);
#pragma unroll
        for (int e = 0; e < 9; ++e) row[e * kForceRow + pos] = G[e];
    }
    __syncthreads();
    // the two parities' wavefronts write half of the 128 sites each
    const uint32_t left = P.g.vh - first, m = (left < 64 ? left : 64) * 18;
    typename cx_t<CR>::type* o = out + ((size_t)mu * P.g.vh + first) * 18;
#pragma unroll
    for (uint32_t j = 0; j < 9; ++j) {
        const uint32_t e = ((uint32_t)par * 9 + j) * 64 + lane;
        if (e >= m) continue;
        double2 w = row[(e % 9) * kForceRow + e / 9];
        if (P.accumulate) { w.x += (double)o[e].x; w.y += (double)o[e].y; }
        o[e].x = (CR)w.x;
        o[e].y = (CR)w.y;
    }
}

template <class CR>
static hipError_t force_t(const Geom& g, int fmt, const double ph[4][2], const void* u, const void* le,
                          const void* lo, const void* re, const void* ro, double coeff, int flags, void* out,
                          hipStream_t s) {
    ForceParams P;
    P.g = g;
    for (int m = 0; m < 4; ++m) { P.ph[m][0] = ph[m][0]; P.ph[m][1] = ph[m][1]; }
    P.u = static_cast<const uint8_t*>(u);
    P.link_block = gauge_block_bytes(g, fmt);
    P.lam[0] = static_cast<const uint8_t*>(le);
    P.lam[1] = static_cast<const uint8_t*>(lo);
    P.r[0] = static_cast<const uint8_t*>(re);
    P.r[1] = static_cast<const uint8_t*>(ro);
    P.coeff = coeff;
    P.project = flags & 1;
    P.accumulate = (flags & 2) != 0;
    auto* O = static_cast<typename cx_t<CR>::type*>(out);
    const dim3 grid((g.vh + 63) / 64, 2), block(256);
#define WEO_F(SP, LP, L12) \
    hipLaunchKernelGGL((k_force<SP, LP, L12, CR>), grid, block, 0, s, P, O)
    switch (fmt) {
        case FMT_D_D_18: WEO_F(P_F64, P_F64, false); break;
        case FMT_D_D_12: WEO_F(P_F64, P_F64, true); break;
        case FMT_S_S_18: WEO_F(P_F32, P_F32, false); break;
        case FMT_S_S_12: WEO_F(P_F32, P_F32, true); break;
        case FMT_H_H_18: WEO_F(P_F16, P_F16, false); break;
        case FMT_H_H_12: WEO_F(P_F16, P_F16, true); break;
        case FMT_B_H_18: WEO_F(P_BF16, P_F16, false); break;
        case FMT_B_H_12: WEO_F(P_BF16, P_F16, true); break;
        default: return hipErrorInvalidValue;
    }
#undef WEO_F
    return hipGetLastError();
}

hipError_t launch_force(const Geom& g, int fmt, const double phase[4][2], const void* u, const void* lam_e,
                        const void* lam_o, const void* r_e, const void* r_o, double coeff, int flags,
                        void* g_canon, int canon_f64, hipStream_t s) {
    return canon_f64 ? force_t<double>(g, fmt, phase, u, lam_e, lam_o, r_e, r_o, coeff, flags, g_canon, s)
                     : force_t<float>(g, fmt, phase, u, lam_e, lam_o, r_e, r_o, coeff, flags, g_canon, s);
}

}  // namespace weo
