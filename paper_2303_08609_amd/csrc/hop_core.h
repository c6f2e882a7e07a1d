// Device building blocks of the hopping-term kernels of the even-odd Wilson operator (paper Sec. 2, Eq. (1)
// and the serial algorithm of Fig. 2): for every output site x of one parity
//
//   out(x) = sum_mu [ (1 - gamma_mu) b+ U_mu(x) in(x+mu)
//                   + (1 + gamma_mu) b- U_mu(x-mu)^dag in(x-mu) ]
//
// computed per direction as: spin projection to a two-component half spinor,
// an SU(3) product on its two colour vectors, reconstruction of the lower
// components and accumulation.  "dagger" swaps the projectors.
//
// gamma matrices are the Dirac representation; with psi = (p0, p1, p2, p3)
// (spin components, each a colour 3-vector) and S = +1 for (1 - gamma_mu),
// S = -1 for (1 + gamma_mu), the projections used below are
//   x: h0 = p0 + S i p3, h1 = p1 + S i p2;  lower = (-S i h1, -S i h0)
//   y: h0 = p0 + S p3,   h1 = p1 - S p2;    lower = (-S h1,    S h0)
//   z: h0 = p0 + S i p2, h1 = p1 - S i p3;  lower = (-S i h0,  S i h1)
//   t: S = +1: 2 (p2, p3) in the lower pair only; S = -1: 2 (p0, p1) upper only.
//
// One lane per output site; the lanes of a wavefront are consecutive sites, so
// every plane load is one coalesced 1 KiB request.  No atomics: each output
// record has exactly one writer.
#pragma once

#include "half_spinor.h"
#include "weo_device.h"
#include "weo_internal.h"

namespace weo {

// Per-precision kernel shape, chosen by measurement on MI355X at 32^3x64:
//   pipe  d >= 1: the raw words of neighbour k + d are loaded while neighbour
//         k is computed (a register ring of d + 1 records, kept in order by
//         scheduling barriers); 0: one direction at a time as written.
//   nt    links are read with streaming (non-temporal) loads: every link is
//         used once per hop, so it should not evict the spinors that the
//         neighbouring sites re-read through L2.
//   nt_store  the output records are written with streaming stores.
// FP64 keeps regular link loads (its streaming variant measured slower) and
// a one-deep ring (a two-deep ring spills), and streams its output (hop
// 349 -> 336 us at 32^3x64; neutral to slightly slower for the narrower
// formats); FP16/BF16 records are small enough for a two-deep ring.
// WEO_HOP_PIPE / WEO_NT_LINKS / WEO_NT_STORE (-D) override all precisions at
// once for experiments.
template <int SP> struct HopShape;
template <> struct HopShape<P_F64> {
    static constexpr int pipe = 1; static constexpr bool nt = false; static constexpr bool nt_store = true;
};
template <> struct HopShape<P_F32> {
    static constexpr int pipe = 1; static constexpr bool nt = true; static constexpr bool nt_store = false;
};
template <> struct HopShape<P_F16> {
    static constexpr int pipe = 2; static constexpr bool nt = true; static constexpr bool nt_store = false;
};
template <> struct HopShape<P_BF16> {
    static constexpr int pipe = 2; static constexpr bool nt = true; static constexpr bool nt_store = false;
};
#ifdef WEO_HOP_PIPE
template <int SP> constexpr int hop_pipe() { return WEO_HOP_PIPE; }
#else
template <int SP> constexpr int hop_pipe() { return HopShape<SP>::pipe; }
#endif
#ifdef WEO_NT_LINKS
template <int SP> constexpr bool hop_nt() { return WEO_NT_LINKS != 0; }
#else
template <int SP> constexpr bool hop_nt() { return HopShape<SP>::nt; }
#endif
#ifdef WEO_NT_STORE
template <int SP> constexpr bool hop_nt_store() { return WEO_NT_STORE != 0; }
#else
template <int SP> constexpr bool hop_nt_store() { return HopShape<SP>::nt_store; }
#endif
//   WEO_WAVES_F32 / WEO_WAVES_F64: minimum waves per SIMD requested (0 = the
//   compiler's choice).
#ifndef WEO_WAVES_F32
#define WEO_WAVES_F32 0
#endif
#ifndef WEO_WAVES_F64
#define WEO_WAVES_F64 0
#endif

// FP16 links of the 12-real formats are converted to FP32 where they are
// unpacked (an empty asm pins the converted values).  Left alone, the
// compiler folds the conversions into mixed-precision FMAs and keeps the raw
// words live longer: FP16/FP16/12 then needs 150 VGPRs instead of 101
// (3 instead of 4 waves per SIMD) and its hop runs 8 % slower.  The 18-real
// formats measured no gain from it.
template <int SP, int LP, bool L12> constexpr bool hop_pin_f16() { return L12; }

template <class V> __device__ __forceinline__ void pin_values(V* v, int n) {
#pragma unroll
    for (int k = 0; k < n; ++k) asm volatile("" : "+v"(v[k].x), "+v"(v[k].y));
}

template <int SP> struct Arith { using R = float; };
template <> struct Arith<P_F64> { using R = double; };

struct HopParams {
    Geom g;
    int out_par;
    int remap;
    double ph[4][2];
    const uint8_t* u;       // packed gauge field
    const uint8_t* in;      // nrhs fields of parity 1 - out_par
    uint8_t* out;           // nrhs fields of parity out_par
    const uint8_t* y;       // axpy addend (parity out_par) or null
    const uint8_t* z;       // second addend (with y only) or null
    double cy;              // coefficient of y
    // fused dot with the output (needs partial; kernels built with DOT only):
    // dmode 1: <dw, out>, 2: <out, y>; real and imaginary partials per 64
    // sites into pdre, pdim
    int dmode;
    const uint8_t* dw;
    double* pdre;
    double* pdim;
    double alpha;
    double* partial;
    size_t spinor_bytes;    // bytes of one packed spinor field
    size_t link_block;      // bytes of one (mu, parity) link block
    Sched sched;            // workgroup -> sites order
};

// The kernel for lattices that leave the chip idle (hop_small.hip, with the
// timings that set the limit on sites times right-hand sides).
constexpr uint64_t kHopSmallSites = 1u << 15;
bool hop_is_small(const HopLaunch& h);
hipError_t launch_hop_small(const HopLaunch& h, const HopParams& P, hipStream_t s);

// Epilogue of a hop with addends: acc = alpha acc + cy y (+ z) for rhs r at
// site ih (cy = 1 rounds exactly as a plain axpy).
template <int SP, class C>
__device__ __forceinline__ void hop_addends(const HopParams& P, size_t r, uint32_t ih, C* acc) {
    using R = decltype(C().x);
    C yv[12];
    load_rec<SP, 12>(P.y + r * P.spinor_bytes, P.g.vh, ih, yv);
    const R a = (R)P.alpha, c = (R)P.cy;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        acc[k].x = fma(a, acc[k].x, c * yv[k].x);
        acc[k].y = fma(a, acc[k].y, c * yv[k].y);
    }
    if (P.z) {
        C zv[12];
        load_rec<SP, 12>(P.z + r * P.spinor_bytes, P.g.vh, ih, zv);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            acc[k].x += zv[k].x;
            acc[k].y += zv[k].y;
        }
    }
}

// Per-lane contributions of the output record acc (rhs r, site ih) to the
// fused reductions, taken on the value as stored (rounded to SP): ||out||^2
// and, with P.dmode, the complex dot <dw, out> = sum conj(dw) out (1) or
// <out, y> = sum conj(out) y (2).
// DOT is a compile-time switch: the dot code costs registers even when not
// taken, which pushed the link-resident kernels to a lower occupancy.
template <int SP, bool DOT = false, class C>
__device__ __forceinline__ void hop_reduce(const HopParams& P, size_t r, uint32_t ih, const C* acc, double& nrm,
                                           double& dre, double& dim) {
    C st[12];
    if constexpr (SP == P_F64 || SP == P_F32) {
#pragma unroll
        for (int k = 0; k < 12; ++k) st[k] = acc[k];
    } else {
        round_rec<SP, 12>(acc, st);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) nrm += (double)st[k].x * (double)st[k].x + (double)st[k].y * (double)st[k].y;
    if constexpr (DOT) {
        C w[12];
        load_rec<SP, 12>((P.dmode == 1 ? P.dw : P.y) + r * P.spinor_bytes, P.g.vh, ih, w);
        const double sg = P.dmode == 1 ? 1.0 : -1.0;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const double ox = st[k].x, oy = st[k].y, wx = w[k].x, wy = w[k].y;
            dre += ox * wx + oy * wy;
            dim += sg * (wx * oy - wy * ox);
        }
    }
}

// The wavefront's sums of hop_reduce for rhs r into the partial arrays (one
// entry per 64 sites); every lane of the wavefront calls it.
template <bool DOT = false>
__device__ __forceinline__ void hop_partials_out(const HopParams& P, size_t r, uint32_t chunk, uint32_t nchunk,
                                                 bool lead, double nrm, double dre, double dim) {
    const double t = wave_sum64(nrm);
    if (lead && chunk < nchunk) P.partial[r * nchunk + chunk] = t;
    if constexpr (DOT) {
        const double a = wave_sum64(dre), b = wave_sum64(dim);
        if (lead && chunk < nchunk) {
            P.pdre[r * nchunk + chunk] = a;
            P.pdim[r * nchunk + chunk] = b;
        }
    }
}

// conj(a b - c d), 8 fused operations.
template <class C> __device__ __forceinline__ C cross_conj(C a, C b, C c, C d) {
    C r;
    r.x = fma(c.y, d.y, fma(-c.x, d.x, fma(-a.y, b.y, a.x * b.x)));
    r.y = fma(c.y, d.x, fma(c.x, d.y, fma(-a.y, b.x, -a.x * b.y)));
    return r;
}
// Row 2 of a 12-real link, conj(row0 x row1), exact for det U = 1.
template <class C> __device__ __forceinline__ void complete_link(C* u) {
    u[6] = cross_conj(u[1], u[5], u[2], u[4]);
    u[7] = cross_conj(u[2], u[3], u[0], u[5]);
    u[8] = cross_conj(u[0], u[4], u[1], u[3]);
}

// Link U as 9 complex numbers (row-major); a 12-real record is completed.
template <int LP, bool L12, bool NT = false, class C>
__device__ __forceinline__ void load_link(const uint8_t* base, uint32_t n, uint32_t i, C* u) {
    if constexpr (L12) {
        load_rec<LP, 6, NT>(base, n, i, u);
        complete_link(u);
    } else {
        load_rec<LP, 9, NT>(base, n, i, u);
    }
}

// Link record of a precision possibly narrower than the arithmetic type.
template <int LP, bool L12, bool NT, class C>
__device__ __forceinline__ void load_link_as(const uint8_t* base, uint32_t n, uint32_t i, C* u) {
    using LR = typename St<LP>::real;
    if constexpr (sizeof(LR) == sizeof(decltype(C().x))) {
        load_link<LP, L12, NT>(base, n, i, u);
    } else {
        cx<LR> w[9];
        load_link<LP, L12, NT>(base, n, i, w);
#pragma unroll
        for (int k = 0; k < 9; ++k) { u[k].x = w[k].x; u[k].y = w[k].y; }
    }
}

// Boundary phases a kernel is built for: any real ones, any complex ones, or
// (the usual case) 1 in x, y and z and a real one in t, where the products
// with the other directions' phases are left out.  The FP16/12 hop is bound
// by its vector instructions and its traffic about equally; this, the FP16
// projection (add_halves) and the fused third row (cross_conj) took it from
// 1548 to 1386 vector instructions per site: apply at 48^3x96 706 -> 694 us,
// clover apply of 12 FP16 fields of 16^3x32 75 -> 70 us.
enum : int { PH_REAL = 0, PH_CPLX = 1, PH_REAL_T = 2 };

inline int phase_mode(const double ph[4][2]) {
    bool one = true;
    for (int m = 0; m < 4; ++m) {
        if (ph[m][1] != 0.0) return PH_CPLX;
        if (m < 3 && ph[m][0] != 1.0) one = false;
    }
    return one ? PH_REAL_T : PH_REAL;
}

// One direction from its half spinor h: boundary phase, product with U (FWD)
// or U^dag (!FWD), reconstruction and accumulation.  The phase is applied
// without a branch, so that the loads of the next neighbours can be scheduled
// ahead of this arithmetic.  (Callers that fold the phase into the link pass
// APPLY_PHASE = false.)
template <int MU, int S, bool FWD, int PH, bool APPLY_PHASE, class C>
__device__ __forceinline__ void hop_half(C* h, const C* u, bool edge, C phase, C* acc) {
    if constexpr (APPLY_PHASE && PH == PH_CPLX) {
        const C ph = edge ? phase : mk<C>(1, 0);
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = mul(ph, h[e]);
    } else if constexpr (APPLY_PHASE && (PH == PH_REAL || MU == 3)) {
        const auto sg = edge ? phase.x : decltype(phase.x)(1);
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = scal(sg, h[e]);
    }
    C g[6];
    half_su3<FWD>(u, h, g);
    half_rebuild<MU, S>(g, decltype(C().x)(1), acc);
}

// One direction: project with (1 - S gamma_mu), then hop_half.
template <int MU, int S, bool FWD, int PH, class C, bool APPLY_PHASE = true>
__device__ __forceinline__ void hop_dir(const C* p, const C* u, bool edge, C phase, C* acc) {
    C h[6];
    half_project<MU, S>(p, h);
    hop_half<MU, S, FWD, PH, APPLY_PHASE>(h, u, edge, phase, acc);
}

// a + b or a - b of two FP16 halves (selected by AH, BH) of packed words, in
// FP32: one instruction where converting both and adding takes three.
template <bool AH, bool BH, bool NEG>
__device__ __forceinline__ float add_halves(uint32_t a, uint32_t b) {
    float r;
#define WEO_MIX(ONE, SEL) asm("v_fma_mix_f32 %0, %1, " ONE ", %2 op_sel:" SEL " op_sel_hi:[1,0,1]" : "=v"(r) : "v"(b), "v"(a))
    if constexpr (NEG) {
        if constexpr (AH && BH) WEO_MIX("-1.0", "[1,0,1]");
        else if constexpr (AH) WEO_MIX("-1.0", "[0,0,1]");
        else if constexpr (BH) WEO_MIX("-1.0", "[1,0,0]");
        else WEO_MIX("-1.0", "[0,0,0]");
    } else {
        if constexpr (AH && BH) WEO_MIX("1.0", "[1,0,1]");
        else if constexpr (AH) WEO_MIX("1.0", "[0,0,1]");
        else if constexpr (BH) WEO_MIX("1.0", "[1,0,0]");
        else WEO_MIX("1.0", "[0,0,0]");
    }
#undef WEO_MIX
    return r;
}
// a + i b (NEG: a - i b), a + b (a - b) of packed complex numbers
template <bool NEG> __device__ __forceinline__ float2 add_i(uint32_t a, uint32_t b) {
    return make_float2(add_halves<false, true, !NEG>(a, b), add_halves<true, false, NEG>(a, b));
}
template <bool NEG> __device__ __forceinline__ float2 add_1(uint32_t a, uint32_t b) {
    return make_float2(add_halves<false, false, NEG>(a, b), add_halves<true, true, NEG>(a, b));
}

// half_project of a record as loaded: FP16 records without converting their
// values first (x, y, z; the values are those of half_project, FP32 sums of
// exact operands).
template <int SP, int MU, int S, class C>
__device__ __forceinline__ void project_raw(const RawRec<SP, 12>& r, C* h) {
    if constexpr (SP == P_F16 && MU < 3) {
        uint32_t p[12];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            p[4 * q] = r.w[q].x; p[4 * q + 1] = r.w[q].y; p[4 * q + 2] = r.w[q].z; p[4 * q + 3] = r.w[q].w;
        }
        constexpr bool N = S < 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if constexpr (MU == 0) {
                h[c] = add_i<N>(p[c], p[9 + c]);
                h[3 + c] = add_i<N>(p[3 + c], p[6 + c]);
            } else if constexpr (MU == 1) {
                h[c] = add_1<N>(p[c], p[9 + c]);
                h[3 + c] = add_1<!N>(p[3 + c], p[6 + c]);
            } else {
                h[c] = add_i<N>(p[c], p[6 + c]);
                h[3 + c] = add_i<!N>(p[3 + c], p[9 + c]);
            }
        }
    } else {
        C p[12];
        r.unpack(p);
        half_project<MU, S>(p, h);
    }
}

// Both neighbours of direction MU for one rhs.
template <int SP, int LP, bool L12, bool DAG, int CPH, int MU, class C>
__device__ __forceinline__ void hop_mu(const HopParams& P, const uint8_t* in, const Nbr& nb,
                                       uint32_t ih, C* acc) {
    constexpr int SF = DAG ? -1 : 1;      // forward term: (1 - SF gamma)
    const uint32_t n = P.g.vh;
    C phase;
    phase.x = (decltype(C().x))P.ph[MU][0];
    phase.y = (decltype(C().x))P.ph[MU][1];
    {
        C u[9], p[12];
        load_link_as<LP, L12, hop_nt<SP>()>(P.u + (size_t)(2 * MU + P.out_par) * P.link_block, n, ih, u);
        load_rec<SP, 12>(in, n, nb.i[2 * MU], p);
        hop_dir<MU, SF, true, CPH>(p, u, nb.edge[2 * MU], phase, acc);
    }
    {
        C u[9], p[12];
        const uint32_t j = nb.i[2 * MU + 1];
        load_link_as<LP, L12, hop_nt<SP>()>(P.u + (size_t)(2 * MU + 1 - P.out_par) * P.link_block, n, j, u);
        load_rec<SP, 12>(in, n, j, p);
        hop_dir<MU, -SF, false, CPH>(p, u, nb.edge[2 * MU + 1], conj_(phase), acc);
    }
}

// ---- pipelined form ---------------------------------------------------------
// Neighbour k = 2 mu + (0: forward x + mu, 1: backward x - mu).
template <int SP, int LP, bool L12>
struct NbrRaw {
    RawRec<SP, 12> sp;
    RawRec<LP, L12 ? 6 : 9, hop_nt<SP>()> ln;
};

template <int SP, int LP, bool L12, int K>
__device__ __forceinline__ void issue(const HopParams& P, const uint8_t* in, const Nbr& nb, uint32_t ih,
                                      NbrRaw<SP, LP, L12>& r) {
    constexpr int MU = K / 2;
    const uint32_t n = P.g.vh;
    if constexpr ((K & 1) == 0) {
        r.ln.load(P.u + (size_t)(2 * MU + P.out_par) * P.link_block, n, ih);
    } else {
        r.ln.load(P.u + (size_t)(2 * MU + 1 - P.out_par) * P.link_block, n, nb.i[K]);
    }
    r.sp.load(in, n, nb.i[K]);
}

template <int SP, int LP, bool L12, bool DAG, int CPH, int K, class C>
__device__ __forceinline__ void consume(const HopParams& P, const Nbr& nb, const NbrRaw<SP, LP, L12>& r,
                                        C* acc) {
    constexpr int MU = K / 2;
    constexpr int SF = DAG ? -1 : 1;
    using R = decltype(C().x);
    constexpr bool FWD = (K & 1) == 0;
    constexpr int S = FWD ? SF : -SF;
    C h[6], u[9];
    project_raw<SP, MU, S>(r.sp, h);
    {
        using LR = typename St<LP>::real;
        cx<LR> w[9];
        r.ln.unpack(w);
        if constexpr (hop_pin_f16<SP, LP, L12>() && LP == P_F16) pin_values(w, L12 ? 6 : 9);
#pragma unroll
        for (int k = 0; k < (L12 ? 6 : 9); ++k) { u[k].x = (R)w[k].x; u[k].y = (R)w[k].y; }
        if constexpr (L12) complete_link(u);
    }
    C phase;
    phase.x = (R)P.ph[MU][0];
    phase.y = (R)P.ph[MU][1];
    if constexpr (!FWD) phase = conj_(phase);
    hop_half<MU, S, FWD, CPH, true>(h, u, nb.edge[K], phase, acc);
}

template <int SP, int LP, bool L12, bool DAG, int CPH, int D, int K, class C>
__device__ __forceinline__ void pipe_step(const HopParams& P, const uint8_t* in, const Nbr& nb, uint32_t ih,
                                          NbrRaw<SP, LP, L12> (&ring)[D + 1], C* acc) {
    if constexpr (K + D < 8) issue<SP, LP, L12, K + D>(P, in, nb, ih, ring[(K + D) % (D + 1)]);
    __builtin_amdgcn_sched_barrier(0);
    consume<SP, LP, L12, DAG, CPH, K>(P, nb, ring[K % (D + 1)], acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (K + 1 < 8) pipe_step<SP, LP, L12, DAG, CPH, D, K + 1>(P, in, nb, ih, ring, acc);
}

template <int SP, int LP, bool L12, bool DAG, int CPH, int D, int K = 0>
__device__ __forceinline__ void pipe_prologue(const HopParams& P, const uint8_t* in, const Nbr& nb, uint32_t ih,
                                              NbrRaw<SP, LP, L12> (&ring)[D + 1]) {
    if constexpr (K < D) {
        issue<SP, LP, L12, K>(P, in, nb, ih, ring[K]);
        pipe_prologue<SP, LP, L12, DAG, CPH, D, K + 1>(P, in, nb, ih, ring);
    }
}

}  // namespace weo
