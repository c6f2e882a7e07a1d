// Multi right-hand-side hop with the links (and clover blocks) of 64 sites
// staged in LDS; picked and tuned by launch_hop (hop_mrhs.hip).
#include "clover_core.h"
#include "half_spinor.h"
#include "hop_mrhs.h"

namespace weo {

// ---- links staged in LDS, right-hand sides across wavefronts --------------------
// A workgroup of W wavefronts owns 64 output sites.  The wavefronts first
// bring the 64 sites' 8 links into LDS in the arithmetic precision, complete
// (a 12-real link's third row rebuilt) and with the boundary phase folded in
// (each wavefront some of the directions), then each walks its own
// right-hand sides (w, w + W, ...) with the single-rhs pipeline, taking the
// links from LDS.  Every link is read from memory, rebuilt and multiplied by
// its phase once per launch, and the register footprint is smaller than the
// single-rhs kernel's, whose ring holds links as well: the form for FP64,
// whose 8 links do not fit a lane's registers next to its pipeline, and a
// candidate for the other formats.  LDS holds the links as
// [direction][element][site], so the 64 lanes of a read touch consecutive
// words.  With CLV the output sites' two clover blocks are staged as well
// and multiply the sum before the epilogue (clover_core.h).
// What bounds it: memory traffic beyond L2 for FP32, vector issue for the
// clover form in FP16, latency for FP64 (12-real links, 5 rhs of 20x12x28x36:
// vector issue on 25 % of the cycles, wavefronts waiting 48 % of theirs).  At
// 218 registers FP64 has 2 wavefronts per SIMD where links staged raw left
// one: twice the neighbour records in flight read more again (12 rhs, 32^3x64,
// 6.0 -> 8.0 GB past L2) in less time (1847 -> 1762 us).  Apply, 12 rhs: clover
// FP16/12 16^3x32 105 -> 71 us, FP32/18 16^3x32 253 -> 111 us and 32^3x64
// 5.45 -> 1.92 ms (against one lane per site and rhs, which reads links and
// blocks once per rhs); BF16/12 32^3x64 1.12 -> 0.96 ms, FP64/12 5 rhs
// 20x12x28x36 240 -> 219 us (against links staged raw).
// FP32 12-real links stay 6 elements in LDS, rebuilt and given their phase at
// use: complete ones (36.9 KB) leave too few workgroups on a CU (12 rhs of
// 22x14x18x20, an apply: 99.8 us complete, 97.6 us so; the clover form,
// bound by instructions, 363 complete, 470 so for 2 rhs of 24x18x38x74).
template <int SP, bool L12, bool CLV> constexpr int lw_elems() { return SP == P_F32 && L12 && !CLV ? 6 : 9; }
template <class C, bool CLV, int NE> struct LwLds {
    C lk[8][NE][64];
    C cb[CLV ? 2 : 1][CLV ? kCloverSlots : 1][CLV ? 64 : 1];
};

// Where link t of a site is read (t = 2 mu forward, 2 mu + 1 backward; wave-uniform).
struct LinkAt {
    const uint8_t* base;
    uint32_t i;
    bool edge;
};
__device__ __forceinline__ LinkAt link_at(const HopParams& P, const Nbr& nb, uint32_t ih, int t) {
    LinkAt a;
    const int side = (t & 1) ? 1 - P.out_par : P.out_par;
    a.base = P.u + (size_t)((t & ~1) + side) * P.link_block;
    a.i = ih;
    a.edge = false;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (t == k) {
            if (k & 1) a.i = nb.i[k];
            a.edge = nb.edge[k];
        }
    return a;
}

// Links t = wv, wv + W, ... of the site to LDS (W >= 2, so at most 4): the
// loads of NB of them are issued before the first is used (FP64: 2; 4 of its
// links would not fit next to the first record).
template <int SP, int LP, bool L12, int NE, class C>
__device__ __forceinline__ void lw_stage_links(const HopParams& P, const Nbr& nb, uint32_t ih, uint32_t lane, int wv,
                                               int W, C (&lk)[8][NE][64]) {
    using R = decltype(C().x);
    constexpr int NB = SP == P_F64 ? 2 : 4;
    RawRec<LP, L12 ? 6 : 9, true> raw[NB];
    bool edge[NB];
#pragma unroll
    for (int q = 0; q < 4; q += NB) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int t = wv + (q + j) * W;
            if (t < 8) {
                const LinkAt a = link_at(P, nb, ih, t);
                raw[j].load(a.base, P.g.vh, a.i);
                edge[j] = a.edge;
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int t = wv + (q + j) * W;
            if (t < 8) {
                cx<typename St<LP>::real> w[9];
                raw[j].unpack(w);
                C u[9];
#pragma unroll
                for (int e = 0; e < (L12 ? 6 : 9); ++e) { u[e].x = (R)w[e].x; u[e].y = (R)w[e].y; }
                if constexpr (NE == 6) {
#pragma unroll
                    for (int e = 0; e < 6; ++e) lk[t][e][lane] = u[e];
                } else {
                    if constexpr (L12) complete_link(u);
                    // ph U for both hops: the backward one multiplies by (ph U)^dag
                    const int mu = t >> 1;
                    const C ph = edge[j] ? mk<C>((R)P.ph[mu][0], (R)P.ph[mu][1]) : mk<C>(R(1), R(0));
#pragma unroll
                    for (int e = 0; e < 9; ++e) lk[t][e][lane] = mul(ph, u[e]);
                }
            }
        }
    }
}

template <int LP, class C>
__device__ __forceinline__ void lw_stage_block(const MrhsParams& M, int q, uint32_t ih, uint32_t lane,
                                               C (*cb)[kCloverSlots][64]) {
    C w[kCloverSlots];
    load_block<LP>(M.clv + (size_t)q * M.block_bytes, M.h.g.vh, ih, w);
#pragma unroll
    for (int e = 0; e < kCloverSlots; ++e) cb[q][e][lane] = w[e];
}

// Most wavefronts per workgroup.
template <int SP> constexpr int lw_maxw() { return SP == P_F64 ? 8 : 12; }
// Wavefronts per SIMD asked for.
template <int SP, bool DOT> constexpr int lw_waves() { return SP == P_F64 ? 2 : (DOT ? 3 : 4); }
// Two record slots: the neighbour record of direction K + 1 is fetched while
// direction K is computed; the last direction of one right-hand side fetches
// the first record of the next.
template <int SP, bool DAG, int K, int NE, class C>
__device__ __forceinline__ void lw_step(const HopParams& P, const C (&lk)[8][NE][64], uint32_t lane,
                                        const uint8_t* in, const uint8_t* in_next, const NbrOff& no,
                                        RawRec<SP, 12> (&ring)[2], uint32_t edges, C* acc) {
    constexpr int MU = K / 2;
    constexpr int SF = DAG ? -1 : 1;
    load_spinor<SP>(K + 1 < 8 ? in : in_next, P.g.vh, no.o[(K + 1) & 7], ring[(K + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
    constexpr bool FWD = (K & 1) == 0;
    constexpr int S = FWD ? SF : -SF;
    C h[6], u[9];
    project_raw<SP, MU, S>(ring[K & 1], h);
#pragma unroll
    for (int e = 0; e < NE; ++e) u[e] = lk[K][e][lane];
    if constexpr (NE == 6) {
        using R = decltype(C().x);
        complete_link(u);
        const C ph = edges >> K & 1u ? mk<C>((R)P.ph[MU][0], (R)(FWD ? P.ph[MU][1] : -P.ph[MU][1])) : mk<C>(R(1), R(0));
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = mul(ph, h[e]);
    }
    hop_half<MU, S, FWD, PH_REAL, false>(h, u, false, C{}, acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (K + 1 < 8) lw_step<SP, DAG, K + 1>(P, lk, lane, in, in_next, no, ring, edges, acc);
}

template <int SP, int LP, bool L12, bool DAG, bool DOT, bool CLV>
__global__ void __launch_bounds__(64 * lw_maxw<SP>(), (lw_waves<SP, DOT>())) k_hop_lw(const MrhsParams M) {
    using R = typename Arith<SP>::R;
    using C = cx<R>;
    constexpr int NE = lw_elems<SP, L12, CLV>();
    __shared__ LwLds<C, CLV, NE> lds;
    const HopParams& P = M.h;
    const uint32_t n = P.g.vh;
    const uint32_t nchunk = (n + 63) >> 6;
    const uint32_t lane = threadIdx.x;                    // blockDim.x == 64
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int W = (int)blockDim.y;
    // this grid row's right-hand sides [r0, r1): rows are separate sweeps
    const int r0 = (int)blockIdx.y * M.rhs_per_row;
    const int r1 = r0 + M.rhs_per_row < M.nrhs ? r0 + M.rhs_per_row : M.nrhs;
    const uint32_t blk = xcd_block(blockIdx.x, M.nblk, P.remap);
    const SiteSpan sp = block_span(P.sched, P.g, blk, 64);
    const uint32_t ih = sp.base + lane;
    const bool valid = ih < sp.end;
    Nbr nb;
    uint32_t edges = 0;
    if (valid) {
        nb = neighbours(P.g, decode(P.g, ih, P.out_par));
        if constexpr (NE == 6)
#pragma unroll
            for (int k = 0; k < 8; ++k) edges |= (uint32_t)nb.edge[k] << k;
    }
    // the first record is on its way while the links are staged
    RawRec<SP, 12> ring[2];
    NbrOff no;
    no.set(nb);
    if (valid && r0 + wv < r1) load_spinor<SP>(P.in + (size_t)(r0 + wv) * P.spinor_bytes, n, no.o[0], ring[0]);
    if (valid) {
        // the 8 links, then the 2 blocks, dealt out to the wavefronts
        lw_stage_links<SP, LP, L12>(P, nb, ih, lane, wv, W, lds.lk);
        if constexpr (CLV) {
            if (8 % W == wv) lw_stage_block<LP>(M, 0, ih, lane, lds.cb);
            if (9 % W == wv) lw_stage_block<LP>(M, 1, ih, lane, lds.cb);
        }
    }
    __syncthreads();
    for (int rr = r0 + wv; rr < r1; rr += W) {
        const int r = opaque_uniform(rr);
        no.pin();
        double nrm = 0.0, dre = 0.0, dim = 0.0;
        if (valid) {
            const uint8_t* in = P.in + (size_t)r * P.spinor_bytes;
            const uint8_t* in_next = r + W < r1 ? in + (size_t)W * P.spinor_bytes : in;
            // an opaque copy of the lane index per right-hand side: the LDS
            // words are invariant in this loop, and without it the compiler
            // hoists all 8 links' reads out of it into registers
            uint32_t lo = lane;
            asm volatile("" : "+v"(lo));
            C acc[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = czero<C>();
            lw_step<SP, DAG, 0>(P, lds.lk, lo, in, in_next, no, ring, edges, acc);
            if constexpr (CLV) {
                const BlockInLds<C> b0{lds.cb[0], lo}, b1{lds.cb[1], lo};
                clover_apply_blocks(b0, b1, acc);
            }
            if (P.y) hop_addends<SP>(P, (size_t)r, ih, acc);
            store_rec<SP, 12, C, mrhs_nt_store<SP>()>(P.out + (size_t)r * P.spinor_bytes, n, ih, acc);
            if (P.partial) hop_reduce<SP, DOT>(P, (size_t)r, ih, acc, nrm, dre, dim);
        }
        if (P.partial) hop_partials_out<DOT>(P, (size_t)r, sp.base >> 6, nchunk, lane == 0 && valid, nrm, dre, dim);
    }
}

// ---- the same on packed FP16 pairs (FP16 spinors and links) ----------------------
// The arithmetic of k_hop_lr16 (hop_mrhs.hip: packed FP16 projection, dot2
// products with FP32 accumulation) with the links in LDS as FP16 pairs
// instead of 72 registers per lane, so 4 and more wavefronts fit a SIMD
// (FP16/12 hop, 12 rhs, 16^3x32: 30 -> 27 us with the axpy; level with the
// register form at 32^3x64, where both wait for memory).
// The links are stored so that no operand needs a sign flip: conj(ph U) for
// the forward hop, ph U for the backward one, and with h' = -i h
//     forward:  (U h).re = dot2(conj U, h),   (U h).im = dot2(conj U, h')
//     backward: (U^dag h).re = dot2(U, h),    (U^dag h).im = dot2(U, h')
// h' comes out of the projection as one more packed add per complex number.
__device__ __forceinline__ h2v mul_mi(h2v v) { return h2v{v.y, -v.x}; }    // -i v

template <int MU, int S>
__device__ __forceinline__ void pair_project(const uint32_t* p, uint32_t (*h)[3], uint32_t (*hm)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const h2v p0 = h2v_of(p[c]), p1 = h2v_of(p[3 + c]), p2 = h2v_of(p[6 + c]), p3 = h2v_of(p[9 + c]);
        h2v h0, h1, m0, m1;
        if constexpr (MU == 0) {
            h0 = S > 0 ? p0 + h2v{-p3.y, p3.x} : p0 - h2v{-p3.y, p3.x};
            h1 = S > 0 ? p1 + h2v{-p2.y, p2.x} : p1 - h2v{-p2.y, p2.x};
            m0 = S > 0 ? mul_mi(p0) + p3 : mul_mi(p0) - p3;
            m1 = S > 0 ? mul_mi(p1) + p2 : mul_mi(p1) - p2;
        } else if constexpr (MU == 1) {
            h0 = S > 0 ? p0 + p3 : p0 - p3;
            h1 = S > 0 ? p1 - p2 : p1 + p2;
            m0 = S > 0 ? mul_mi(p0) + mul_mi(p3) : mul_mi(p0) - mul_mi(p3);
            m1 = S > 0 ? mul_mi(p1) - mul_mi(p2) : mul_mi(p1) + mul_mi(p2);
        } else if constexpr (MU == 2) {
            h0 = S > 0 ? p0 + h2v{-p2.y, p2.x} : p0 - h2v{-p2.y, p2.x};
            h1 = S > 0 ? p1 - h2v{-p3.y, p3.x} : p1 + h2v{-p3.y, p3.x};
            m0 = S > 0 ? mul_mi(p0) + p2 : mul_mi(p0) - p2;
            m1 = S > 0 ? mul_mi(p1) - p3 : mul_mi(p1) + p3;
        } else {
            h0 = S > 0 ? p2 : p0;
            h1 = S > 0 ? p3 : p1;
            m0 = mul_mi(h0);
            m1 = mul_mi(h1);
        }
        h[0][c] = u32_of(h0);
        h[1][c] = u32_of(h1);
        hm[0][c] = u32_of(m0);
        hm[1][c] = u32_of(m1);
    }
}

template <int MU, int S, bool FWD>
__device__ __forceinline__ void pair_dir(const uint32_t* p, const uint32_t* u, float2* acc) {
    uint32_t h[2][3], hm[2][3];
    pair_project<MU, S>(p, h, hm);
    float2 g[6];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float re = 0.f, im = 0.f;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const uint32_t e = FWD ? u[3 * a + b] : u[3 * b + a];
                re = dot2(e, h[s][b], re);
                im = dot2(e, hm[s][b], im);
            }
            g[3 * s + a] = make_float2(re, im);
        }
    half_rebuild<MU, S>(g, 1.0f, acc);
}

// as lw_stage_links
template <bool L12, bool CPH>
__device__ __forceinline__ void pair_stage(const HopParams& P, const Nbr& nb, uint32_t ih, uint32_t lane, int wv, int W,
                                           uint32_t (&lk)[8][9][64]) {
    RawRec<P_F16, L12 ? 6 : 9, true> raw[4];
    bool edge[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = wv + j * W;
        if (t < 8) {
            const LinkAt a = link_at(P, nb, ih, t);
            raw[j].load(a.base, P.g.vh, a.i);
            edge[j] = a.edge;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = wv + j * W;
        if (t < 8) {
            Link16 L;
            const int mu = t >> 1;
            link16_of<L12, CPH>(raw[j], edge[j], make_float2((float)P.ph[mu][0], (float)P.ph[mu][1]), L);
            const uint32_t conj = (t & 1) ? 0u : 0x80000000u;
#pragma unroll
            for (int e = 0; e < 9; ++e) lk[t][e][lane] = L.e[e] ^ conj;
        }
    }
}

template <bool DAG, int D, int K>
__device__ __forceinline__ void pair_step(const HopParams& P, const uint32_t (&lk)[8][9][64], uint32_t lane,
                                          const uint8_t* in, const uint8_t* in_next, const NbrOff& no,
                                          RawRec<P_F16, 12> (&ring)[D + 1], float2* acc) {
    constexpr int MU = K / 2;
    constexpr int SF = DAG ? -1 : 1;
    load_spinor<P_F16>(K + D < 8 ? in : in_next, P.g.vh, no.o[(K + D) & 7], ring[(K + D) % (D + 1)]);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t p[12], u[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = lk[K][e][lane];
    rec16_words(ring[K % (D + 1)], p);
    pair_dir<MU, (K & 1) == 0 ? SF : -SF, (K & 1) == 0>(p, u, acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (K + 1 < 8) pair_step<DAG, D, K + 1>(P, lk, lane, in, in_next, no, ring, acc);
}

template <bool L12, bool DAG, bool CPH, int D>
__global__ void __launch_bounds__(64 * 12, 4) k_hop_lw16(const MrhsParams M) {
    static_assert(8 % (D + 1) == 0, "ring size must divide the 8 directions");
    __shared__ uint32_t lk[8][9][64];
    const HopParams& P = M.h;
    const uint32_t n = P.g.vh;
    const uint32_t nchunk = (n + 63) >> 6;
    const uint32_t lane = threadIdx.x;                    // blockDim.x == 64
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int W = (int)blockDim.y;
    const int r0 = (int)blockIdx.y * M.rhs_per_row;
    const int r1 = r0 + M.rhs_per_row < M.nrhs ? r0 + M.rhs_per_row : M.nrhs;
    const uint32_t blk = xcd_block(blockIdx.x, M.nblk, P.remap);
    const SiteSpan sp = block_span(P.sched, P.g, blk, 64);
    const uint32_t ih = sp.base + lane;
    const bool valid = ih < sp.end;
    Nbr nb;
    NbrOff no;
    RawRec<P_F16, 12> ring[D + 1];
    if (valid) {
        nb = neighbours(P.g, decode(P.g, ih, P.out_par));
        no.set(nb);
        if (r0 + wv < r1) {
#pragma unroll
            for (int k = 0; k < D; ++k) load_spinor<P_F16>(P.in + (size_t)(r0 + wv) * P.spinor_bytes, n, no.o[k], ring[k]);
        }
        pair_stage<L12, CPH>(P, nb, ih, lane, wv, W, lk);
    }
    __syncthreads();
    for (int rr = r0 + wv; rr < r1; rr += W) {
        const int r = opaque_uniform(rr);
        no.pin();
        uint32_t lo = lane;                               // opaque as in k_hop_lw
        asm volatile("" : "+v"(lo));
        double nrm = 0.0, dre = 0.0, dim = 0.0;
        if (valid) {
            const uint8_t* in = P.in + (size_t)r * P.spinor_bytes;
            const uint8_t* in_next = r + W < r1 ? in + (size_t)W * P.spinor_bytes : in;
            float2 acc[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = make_float2(0.f, 0.f);
            pair_step<DAG, D, 0>(P, lk, lo, in, in_next, no, ring, acc);
            if (P.y) hop_addends<P_F16>(P, (size_t)r, ih, acc);
            store_rec<P_F16, 12, float2, mrhs_nt_store<P_F16>()>(P.out + (size_t)r * P.spinor_bytes, n, ih, acc);
            if (P.partial) hop_reduce<P_F16>(P, (size_t)r, ih, acc, nrm, dre, dim);
        }
        if (P.partial) hop_partials_out(P, (size_t)r, sp.base >> 6, nchunk, lane == 0 && valid, nrm, dre, dim);
    }
}

// ------------------------------------------------------------------ host ----
template <int SP, int LP, bool L12>
static hipError_t lw_fmt(const HopLaunch& h, const MrhsParams& M, dim3 grid, dim3 block, hipStream_t s) {
#define WEO_LW(DG, DT, CL) hipLaunchKernelGGL((k_hop_lw<SP, LP, L12, DG, DT, CL>), grid, block, 0, s, M)
    if (h.clv) {
        if (h.dmode) return hipErrorInvalidValue;        // the clover epilogue fuses no dot
        if (h.dagger) WEO_LW(true, false, true); else WEO_LW(false, false, true);
    } else if (h.dmode) {
        if (!h.partial) return hipErrorInvalidValue;
        if (h.dagger) WEO_LW(true, true, false); else WEO_LW(false, true, false);
    } else {
        if (h.dagger) WEO_LW(true, false, false); else WEO_LW(false, false, false);
    }
#undef WEO_LW
    return hipGetLastError();
}

int lw_max_waves(int fmt) {
    switch (fmt_info(fmt).spinor_prec) {
        case P_F64: return lw_maxw<P_F64>();
        case P_F32: return lw_maxw<P_F32>();
        default: return lw_maxw<P_F16>();
    }
}

// LDS-staged form: W wavefronts of 64 sites per workgroup
hipError_t launch_hop_lw(const HopLaunch& h, const MrhsParams& M, int W, dim3 grid, hipStream_t s) {
    if (W > lw_max_waves(h.fmt)) return hipErrorInvalidValue;
    const dim3 block(64, (unsigned)W);
    switch (h.fmt) {
        case FMT_D_D_18: return lw_fmt<P_F64, P_F64, false>(h, M, grid, block, s);
        case FMT_D_D_12: return lw_fmt<P_F64, P_F64, true>(h, M, grid, block, s);
        case FMT_S_S_18: return lw_fmt<P_F32, P_F32, false>(h, M, grid, block, s);
        case FMT_S_S_12: return lw_fmt<P_F32, P_F32, true>(h, M, grid, block, s);
        case FMT_H_H_18: return lw_fmt<P_F16, P_F16, false>(h, M, grid, block, s);
        case FMT_H_H_12: return lw_fmt<P_F16, P_F16, true>(h, M, grid, block, s);
        case FMT_B_H_18: return lw_fmt<P_BF16, P_F16, false>(h, M, grid, block, s);
        case FMT_B_H_12: return lw_fmt<P_BF16, P_F16, true>(h, M, grid, block, s);
        default: return hipErrorInvalidValue;
    }
}

template <bool L12, int D>
static hipError_t lw16_fmt(const HopLaunch& h, const MrhsParams& M, dim3 grid, dim3 block, hipStream_t s) {
    const bool cph = !phases_are_signs(h);
#define WEO_LW16(DG, CP) hipLaunchKernelGGL((k_hop_lw16<L12, DG, CP, D>), grid, block, 0, s, M)
    if (h.dagger) { if (cph) WEO_LW16(true, true); else WEO_LW16(true, false); }
    else { if (cph) WEO_LW16(false, true); else WEO_LW16(false, false); }
#undef WEO_LW16
    return hipGetLastError();
}

hipError_t launch_hop_lw16(const HopLaunch& h, const MrhsParams& M, int W, int depth, dim3 grid, hipStream_t s) {
    if (W > 12 || h.dmode || h.clv) return hipErrorInvalidValue;
    const dim3 block(64, (unsigned)W);
    switch (h.fmt) {
        case FMT_H_H_18: return depth == 3 ? lw16_fmt<false, 3>(h, M, grid, block, s) : lw16_fmt<false, 1>(h, M, grid, block, s);
        case FMT_H_H_12: return depth == 3 ? lw16_fmt<true, 3>(h, M, grid, block, s) : lw16_fmt<true, 1>(h, M, grid, block, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace weo
