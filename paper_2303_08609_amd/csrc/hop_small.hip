// Hopping kernel for lattices too small to fill the chip (paper Sec. 2,
// Eq. (1)): the 8 terms of a site are spread over 8 wavefronts.
//
// On few sites the hop is one lane's chain of latencies: the single-rhs
// kernel fetches 8 neighbours one after the other.  Here a workgroup owns 64
// output sites and wavefront k computes term k of all of them (k = 2 mu:
// x + mu, 2 mu + 1: x - mu): one round of loads, the projected product to LDS,
// and the first wavefront sums the terms in the single-rhs kernel's order and
// runs its epilogue, whose addend it fetched meanwhile.  The direction is
// uniform in a wavefront.  With clover blocks (CLV) the second and third
// wavefront also bring the site's two blocks to LDS.
// Taken up to 2^15 sites times right-hand sides, where it stops winning
// (plain hop, single-rhs kernel -> this one, us):
//                FP64/18        FP32/18       FP16/12
//   4^4          7.2 ->  5.5   4.3 ->  3.6   4.8 -> 3.6
//   8^4         13.2 ->  6.2   5.9 ->  4.1   6.0 -> 4.3
//   12^4        13.4 ->  6.8   7.5 ->  4.2   6.5 -> 4.5
//   16^4        13.6 -> 13.6   8.3 ->  5.8   6.7 -> 5.2
//   16^3x32     20.2 -> 25.5  10.0 -> 11.4   7.2 -> 7.3
#include "clover_core.h"
#include "half_spinor.h"
#include "hop_core.h"

namespace weo {

struct SmallParams {
    HopParams h;
    const uint8_t* clv;     // the output parity's two clover blocks, or null
    size_t block_bytes;
};

template <class C, bool CLV> struct SmallLds {
    C g[8][6][64];
    C cb[CLV ? 2 : 1][CLV ? kCloverSlots : 1][CLV ? 64 : 1];
};

// Term K of the site: projection, boundary phase, SU(3) product (the
// arithmetic of hop_dir) to row K of LDS.
template <int SP, int LP, bool L12, bool DAG, bool CPH, int K, class C>
__device__ __forceinline__ void small_term(const HopParams& P, const uint8_t* in, const Nbr& nb, uint32_t ih,
                                           uint32_t lane, C (&lds)[8][6][64]) {
    constexpr int MU = K / 2;
    constexpr bool FWD = (K & 1) == 0;
    constexpr int S = FWD == DAG ? -1 : 1;      // (1 - S gamma_mu)
    using R = decltype(C().x);
    C u[9], p[12], h[6], g[6];
    load_link_as<LP, L12, false>(P.u + (size_t)(2 * MU + (FWD ? P.out_par : 1 - P.out_par)) * P.link_block, P.g.vh,
                                 FWD ? ih : nb.i[K], u);
    load_rec<SP, 12>(in, P.g.vh, nb.i[K], p);
    half_project<MU, S>(p, h);
    if constexpr (CPH) {
        const C ph = nb.edge[K] ? mk<C>((R)P.ph[MU][0], (R)(FWD ? P.ph[MU][1] : -P.ph[MU][1])) : mk<C>(R(1), R(0));
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = mul(ph, h[e]);
    } else {
        const R sg = nb.edge[K] ? (R)P.ph[MU][0] : R(1);
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = scal(sg, h[e]);
    }
    half_su3<FWD>(u, h, g);
#pragma unroll
    for (int e = 0; e < 6; ++e) lds[K][e][lane] = g[e];
}

template <bool DAG, int K, class C>
__device__ __forceinline__ void small_sum(const C (&lds)[8][6][64], uint32_t lane, C* acc) {
    constexpr int S = ((K & 1) == 0) == DAG ? -1 : 1;
    C g[6];
#pragma unroll
    for (int e = 0; e < 6; ++e) g[e] = lds[K][e][lane];
    half_rebuild<K / 2, S>(g, decltype(C().x)(1), acc);
    if constexpr (K + 1 < 8) small_sum<DAG, K + 1>(lds, lane, acc);
}

template <int SP, int LP, bool L12, bool DAG, bool CPH, bool CLV>
__global__ void __launch_bounds__(512) k_hop_small(const SmallParams Q) {
    using R = typename Arith<SP>::R;
    using C = cx<R>;
    const HopParams& P = Q.h;
    __shared__ SmallLds<C, CLV> L;
    const uint32_t lane = threadIdx.x & 63u;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t base = xcd_block(blockIdx.x, gridDim.x, P.remap) * 64, ih = base + lane;
    const bool valid = ih < P.g.vh;
    const size_t rhs = blockIdx.y;
    const uint8_t* in = P.in + rhs * P.spinor_bytes;
    RawRec<SP, 12> y;
    if (valid) {
        if (wv == 0 && P.y) y.load(P.y + rhs * P.spinor_bytes, P.g.vh, ih);
        RawRec<LP, kCloverSlots> cb;
        const bool has_block = CLV && (wv == 1 || wv == 2);
        // fetched next to the term's records, except FP64 ones, which would spill
        if (has_block && SP != P_F64) cb.load(Q.clv + (size_t)(wv - 1) * Q.block_bytes, P.g.vh, ih);
        const Nbr nb = neighbours(P.g, decode(P.g, ih, P.out_par));
        switch (wv) {
#define WEO_TERM(K) case K: small_term<SP, LP, L12, DAG, CPH, K>(P, in, nb, ih, lane, L.g); break;
            WEO_TERM(0) WEO_TERM(1) WEO_TERM(2) WEO_TERM(3) WEO_TERM(4) WEO_TERM(5) WEO_TERM(6)
            default: small_term<SP, LP, L12, DAG, CPH, 7>(P, in, nb, ih, lane, L.g);
#undef WEO_TERM
        }
        if (has_block) {
            if (SP == P_F64) cb.load(Q.clv + (size_t)(wv - 1) * Q.block_bytes, P.g.vh, ih);
            cx<typename St<LP>::real> w[kCloverSlots];
            cb.unpack(w);
#pragma unroll
            for (int k = 0; k < kCloverSlots; ++k) L.cb[wv - 1][k][lane] = mk<C>((R)w[k].x, (R)w[k].y);
        }
    }
    __syncthreads();
    if (wv != 0) return;
    double nrm = 0.0, dre = 0.0, dim = 0.0;
    if (valid) {
        C acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = czero<C>();
        small_sum<DAG, 0>(L.g, lane, acc);
        if constexpr (CLV) {
            const BlockInLds<C> b0{L.cb[0], lane}, b1{L.cb[1], lane};
            clover_apply_blocks(b0, b1, acc);
        }
        if (P.y) {              // as hop_addends
            C v[12];
            y.unpack(v);
            const R a = (R)P.alpha, c = (R)P.cy;
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                acc[k].x = fma(a, acc[k].x, c * v[k].x);
                acc[k].y = fma(a, acc[k].y, c * v[k].y);
            }
            if (P.z) {
                load_rec<SP, 12>(P.z + rhs * P.spinor_bytes, P.g.vh, ih, v);
#pragma unroll
                for (int k = 0; k < 12; ++k) acc[k] = add(acc[k], v[k]);
            }
        }
        store_rec<SP, 12>(P.out + rhs * P.spinor_bytes, P.g.vh, ih, acc);
        if (P.partial) {
            if (P.dmode) hop_reduce<SP, true>(P, rhs, ih, acc, nrm, dre, dim);
            else hop_reduce<SP, false>(P, rhs, ih, acc, nrm, dre, dim);
        }
    }
    if (P.partial) {
        const uint32_t nchunk = (P.g.vh + 63) >> 6;
        if (P.dmode) hop_partials_out<true>(P, rhs, base >> 6, nchunk, lane == 0, nrm, dre, dim);
        else hop_partials_out<false>(P, rhs, base >> 6, nchunk, lane == 0, nrm, dre, dim);
    }
}

// ------------------------------------------------------------------ host ----
bool hop_is_small(const HopLaunch& h) { return (uint64_t)h.g.vh * (uint64_t)h.nrhs <= kHopSmallSites; }

template <int SP, int LP, bool L12>
static hipError_t small_fmt(const HopLaunch& h, const SmallParams& Q, dim3 grid, hipStream_t s) {
    bool cph = false;
    for (int m = 0; m < 4; ++m) cph = cph || h.phase[m][1] != 0.0;
#define WEO_SMALL(D, CP, CL) hipLaunchKernelGGL((k_hop_small<SP, LP, L12, D, CP, CL>), grid, dim3(512), 0, s, Q)
#define WEO_SMALL_D(D)                                                                   \
    if (Q.clv) { if (cph) WEO_SMALL(D, true, true); else WEO_SMALL(D, false, true); }    \
    else { if (cph) WEO_SMALL(D, true, false); else WEO_SMALL(D, false, false); }
    if (h.dagger) { WEO_SMALL_D(true) } else { WEO_SMALL_D(false) }
#undef WEO_SMALL_D
#undef WEO_SMALL
    return hipGetLastError();
}

hipError_t launch_hop_small(const HopLaunch& h, const HopParams& P, hipStream_t s) {
    if (h.dmode && (!h.y || !h.partial || h.clv)) return hipErrorInvalidValue;
    SmallParams Q;
    Q.h = P;
    Q.block_bytes = clover_block_bytes(h.g, h.fmt);
    Q.clv = h.clv ? static_cast<const uint8_t*>(h.clv) + (size_t)(2 * h.out_par) * Q.block_bytes : nullptr;
    const dim3 grid((h.g.vh + 63) / 64, (unsigned)h.nrhs);
    switch (h.fmt) {
        case FMT_D_D_18: return small_fmt<P_F64, P_F64, false>(h, Q, grid, s);
        case FMT_D_D_12: return small_fmt<P_F64, P_F64, true>(h, Q, grid, s);
        case FMT_S_S_18: return small_fmt<P_F32, P_F32, false>(h, Q, grid, s);
        case FMT_S_S_12: return small_fmt<P_F32, P_F32, true>(h, Q, grid, s);
        case FMT_H_H_18: return small_fmt<P_F16, P_F16, false>(h, Q, grid, s);
        case FMT_H_H_12: return small_fmt<P_F16, P_F16, true>(h, Q, grid, s);
        case FMT_B_H_18: return small_fmt<P_BF16, P_F16, false>(h, Q, grid, s);
        case FMT_B_H_12: return small_fmt<P_BF16, P_F16, true>(h, Q, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace weo
