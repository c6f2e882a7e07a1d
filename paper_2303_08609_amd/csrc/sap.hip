// Schwarz alternating procedure (SAP) on two-coloured Dirichlet blocks of
// the Wilson matrix D_W = 1 - kappa H (Eq. (1)), and the vector kernels of
// the flexible GCR solver it preconditions.
//
// The lattice is cut into blocks of extent b = (bx, by, bz, bt) (n_mu =
// L_mu / b_mu blocks along mu, each 1 or even), coloured by the parity of the
// block coordinates.  One sweep over the blocks of one colour runs nmr steps
// of the minimal residual iteration on each block's own system D_L e = rho_L
// (every hop leaving the block dropped; where n_mu = 1 the hop across the
// lattice edge stays inside) and adds e to the solution.  The residual is
// carried, not recomputed: inside a swept block it is the MR residual; on the
// blocks of the other colour it changes only by the hops out of the swept
// blocks, +kappa H e, which the next sweep of that colour adds when it loads
// its blocks (from the increment e of the previous sweep, kept in dprev).
//
// The block solves run in FP32 (FP32 spinors and links, FP64 block sums):
// SAP is a preconditioner of a flexible Krylov method, so its accuracy only
// affects the iteration count, and FP32 keeps a block's residual, solution
// and links in one CU's LDS and registers (FP64 would spill).
//
// One workgroup per block (lane = site, at most 256 sites), so a block's
// whole solve runs out of LDS and registers: the block residual is shared
// through LDS for the in-block hops, the block sums of MR reduce within the
// wavefronts and through LDS, and the fields are read and written once per
// sweep.  Two kernels: k_sap_block, and k_sap_sweep for the block shapes
// whose faces do not fit the scratch fields (in it the workgroups of the
// other colour exit at once).
#include "half_spinor.h"
#include "hop_core.h"
#include "weo_internal.h"

namespace weo {

struct SapParams {
    Geom g;
    int b[4], nb[4];        // block extents; blocks per direction
    int bvol;               // sites per block
    int colour;
    int nmr;
    double kappa;
    double ph[4][2];
    const uint8_t* u;
    size_t link_block;
    size_t half_bytes;      // one parity of one field
    uint8_t* rho;           // nrhs full fields [rhs][even | odd]: residual (read, written)
    uint8_t* phi;           // solution, += the block solutions
    const uint8_t* dprev;   // block solutions of the previous sweep (other colour) or null
    uint8_t* dout;          // block solutions of this sweep
};

template <int SP> struct SapLds {
    using R = typename Arith<SP>::R;
    cx<R> res[12][kSapMaxSites];      // the block residual, shared for the in-block hops
    cx<R> e[12][kSapMaxSites];        // the block solution (each lane its own slot)
    double red[4][3];
};

// One hop term K = 2 mu (+mu) or 2 mu + 1 (-mu) of site x (parity p, half
// index ih) on the neighbour record psi, weighted by w (0 drops the term).
template <int SP, int LP, bool L12, int K, class C>
__device__ __forceinline__ void sap_term(const SapParams& P, const uint8_t* ubase, const Nbr& nb, uint32_t ih,
                                         int p, const C* psi, bool on, C* acc) {
    constexpr int MU = K / 2;
    constexpr bool FWD = (K & 1) == 0;
    using R = decltype(C().x);
    C u[9];
    load_link_as<LP, L12, false>(ubase + (size_t)(2 * MU + (FWD ? p : 1 - p)) * P.link_block, P.g.vh,
                                 FWD ? ih : nb.i[K], u);
    const R pr = (R)P.ph[MU][0], pi = (R)(FWD ? P.ph[MU][1] : -P.ph[MU][1]);
    C w = nb.edge[K] ? mk<C>(pr, pi) : mk<C>(R(1), R(0));
    w = on ? w : mk<C>(R(0), R(0));
    hop_dir<MU, FWD ? 1 : -1, FWD, PH_CPLX>(psi, u, true, w, acc);
}

template <int SP, int LP, bool L12>
__global__ void __launch_bounds__(kSapMaxSites) k_sap_sweep(const SapParams P) {
    using R = typename Arith<SP>::R;
    using C = cx<R>;
    __shared__ SapLds<SP> L;
    uint32_t bi = blockIdx.x;
    int bc[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) { bc[m] = (int)(bi % (uint32_t)P.nb[m]); bi /= (uint32_t)P.nb[m]; }
    if (((bc[0] + bc[1] + bc[2] + bc[3]) & 1) != P.colour) return;      // the whole workgroup
    const int l = threadIdx.x;
    const bool act = l < P.bvol;
    const int ls = act ? l : 0;
    int lc[4], stride[4];
    {
        int r = ls, s = 1;
#pragma unroll
        for (int m = 0; m < 4; ++m) { lc[m] = r % P.b[m]; r /= P.b[m]; stride[m] = s; s *= P.b[m]; }
    }
    Site st;
    st.x = bc[0] * P.b[0] + lc[0];
    st.y = bc[1] * P.b[1] + lc[1];
    st.z = bc[2] * P.b[2] + lc[2];
    st.t = bc[3] * P.b[3] + lc[3];
    st.xh = st.x >> 1;
    st.ih = (uint32_t)st.xh + (uint32_t)P.g.lxh * ((uint32_t)st.y + (uint32_t)P.g.ly *
                                                   ((uint32_t)st.z + (uint32_t)P.g.lz * (uint32_t)st.t));
    const int p = (st.x + st.y + st.z + st.t) & 1;
    const Nbr nb = neighbours(P.g, st);
    // in-block neighbours (local index, and whether the hop stays inside)
    int nl[8];
    bool in[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const bool whole = P.nb[m] == 1;
        const bool f = lc[m] + 1 < P.b[m], b = lc[m] > 0;
        in[2 * m] = act && (f || whole);
        in[2 * m + 1] = act && (b || whole);
        nl[2 * m] = f ? ls + stride[m] : ls - (P.b[m] - 1) * stride[m];
        nl[2 * m + 1] = b ? ls - stride[m] : ls + (P.b[m] - 1) * stride[m];
    }
    const size_t fb = 2 * P.half_bytes;
    const size_t off = (size_t)blockIdx.y * fb;
    const uint32_t n = P.g.vh;
    C res[12];
    if (act) load_rec<SP, 12>(P.rho + off + (size_t)p * P.half_bytes, n, st.ih, res);
    else
#pragma unroll
        for (int k = 0; k < 12; ++k) res[k] = czero<C>();
    // hops into the block from the previous sweep's solutions on the
    // neighbouring blocks: rho += kappa H dprev on the block's faces
    if (P.dprev) {
        C acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = czero<C>();
        const uint8_t* dp = P.dprev + off + (size_t)(1 - p) * P.half_bytes;
        bool any = false;
#pragma unroll
        for (int k = 0; k < 8; ++k) any = any || (act && !in[k]);
        if (any) {
#define WEO_SAP_EXT(K)                                                        \
            if (act && !in[K]) {                                              \
                C q[12];                                                      \
                load_rec<SP, 12>(dp, n, nb.i[K], q);                          \
                sap_term<SP, LP, L12, K>(P, P.u, nb, st.ih, p, q, true, acc);      \
            }
            WEO_SAP_EXT(0) WEO_SAP_EXT(1) WEO_SAP_EXT(2) WEO_SAP_EXT(3)
            WEO_SAP_EXT(4) WEO_SAP_EXT(5) WEO_SAP_EXT(6) WEO_SAP_EXT(7)
#undef WEO_SAP_EXT
            const R kap = (R)P.kappa;
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                res[k].x = fma(kap, acc[k].x, res[k].x);
                res[k].y = fma(kap, acc[k].y, res[k].y);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) L.e[k][l] = czero<C>();
    const int nw = (blockDim.x + 63) >> 6;
#pragma unroll 1
    for (int it = 0; it < P.nmr; ++it) {
        __syncthreads();                       // readers of the previous residual are done
#pragma unroll
        for (int k = 0; k < 12; ++k) L.res[k][l] = res[k];
        __syncthreads();
        C q[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) q[k] = czero<C>();
        // the links stay in registers across the MR steps (the compiler
        // hoists their loads out of the loop)
#define WEO_SAP_IN(K)                                                         \
        {                                                                     \
            const uint8_t* ub = P.u;                                          \
            C v[12];                                                          \
            const int j = in[K] ? nl[K] : l;                                  \
            _Pragma("unroll") for (int k = 0; k < 12; ++k) v[k] = L.res[k][j]; \
            sap_term<SP, LP, L12, K>(P, ub, nb, st.ih, p, v, in[K], q);           \
            __builtin_amdgcn_sched_barrier(0);                                \
        }
        WEO_SAP_IN(0) WEO_SAP_IN(1) WEO_SAP_IN(2) WEO_SAP_IN(3)
        WEO_SAP_IN(4) WEO_SAP_IN(5) WEO_SAP_IN(6) WEO_SAP_IN(7)
#undef WEO_SAP_IN
        // q = D_L res = res - kappa H_L res
        const R kap = (R)P.kappa;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            q[k].x = act ? fma(-kap, q[k].x, res[k].x) : R(0);
            q[k].y = act ? fma(-kap, q[k].y, res[k].y) : R(0);
            const double qx = q[k].x, qy = q[k].y, rx = res[k].x, ry = res[k].y;
            s0 += qx * rx + qy * ry;           // <q, res>
            s1 += qx * ry - qy * rx;
            s2 += qx * qx + qy * qy;           // <q, q>
        }
        s0 = wave_sum64(s0);
        s1 = wave_sum64(s1);
        s2 = wave_sum64(s2);
        if ((l & 63) == 0) { L.red[l >> 6][0] = s0; L.red[l >> 6][1] = s1; L.red[l >> 6][2] = s2; }
        __syncthreads();
        double t0 = 0.0, t1 = 0.0, t2 = 0.0;
        for (int w = 0; w < nw; ++w) { t0 += L.red[w][0]; t1 += L.red[w][1]; t2 += L.red[w][2]; }
        const double a0 = t2 > 0.0 ? t0 / t2 : 0.0, a1 = t2 > 0.0 ? t1 / t2 : 0.0;
        const C al = mk<C>((R)a0, (R)a1);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            L.e[k][l] = fma_(al, res[k], L.e[k][l]);
            res[k] = sub(res[k], mul(al, q[k]));
        }
    }
    if (!act) return;
    C e[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) e[k] = L.e[k][l];
    const size_t po = off + (size_t)p * P.half_bytes;
    store_rec<SP, 12>(P.rho + po, n, st.ih, res);
    store_rec<SP, 12>(P.dout + po, n, st.ih, e);
    C ph[12];
    load_rec<SP, 12>(P.phi + po, n, st.ih, ph);
#pragma unroll
    for (int k = 0; k < 12; ++k) ph[k] = add(ph[k], e[k]);
    store_rec<SP, 12>(P.phi + po, n, st.ih, ph);
}

// ---- the block sweep with projected faces ----------------------------------------
// k_sap_block: the same sweep with everything between sweeps kept in block
// order.  A block's own 4 links per site stay in registers for the whole
// sweep: the forward hop of direction mu multiplies the neighbour's projected
// residual by U_mu(x), and the backward hop is multiplied at its source, which
// owns that link, and handed over through LDS as a half spinor.  The coupling
// between blocks is exchanged the same way: a block writes only the projected
// half spinors of its faces (the upper ones already times U^dag), so the
// receiver reads no full increments and no foreign links.  Residual, solution
// and faces are [block][plane][site of the block] in the workspace: a
// wavefront reads consecutive 16-byte words, where the lattice order gives a
// 4^4 block pieces of 32 bytes.  The source is read and the solution written
// in lattice order in the first and last cycle only.  Only one colour's
// blocks are launched, x neighbours on one XCD (they share cache lines of the
// links).
// What bounds it: vector issue and latency, at 2 wavefronts per SIMD (256
// registers and 74 KB of LDS for 256 sites).  Counters at 32^3x64, 4^4 blocks:
// about 1300 vector instructions per lane and step (200 of them the FP64 block
// sums) issue on 58 % of the cycles, the wavefronts wait 21 % of theirs, and
// 0.95 GB read and 0.16 written in 295 us are 3.8 TB/s.  One sweep at 32^3x64 with 4^4 blocks and
// 4 steps: 290 us, against 1390 us for k_sap_sweep, whose 8 links per site
// and solution cost half the occupancy and whose neighbour reads fetch whole
// cache lines for 32 bytes.
struct SapBlockParams {
    Geom g;
    int b[4], nb[4];        // block extents; blocks per direction
    int cb[4];              // blocks of one colour per direction (nb, halved along the first split direction)
    FastDiv d_b[4];         // division by b
    int split;              // that direction; -1 when one block spans the lattice
    int bvol;
    int colour;
    int nmr;
    float kappa;
    float ph[4][2];
    int wrap[4];            // a block spans mu and the phase there is not 1
    int foff[4];            // 16-byte words of a block's faces before direction mu
    int fwords;             // 16-byte words of one block's faces
    const uint8_t* u;
    size_t link_block;
    size_t half_bytes;      // one parity of one field
    size_t field_words;     // 16-byte words of one field in block order
    size_t face_words;      // 16-byte words of the faces of one colour's blocks, one rhs
    const uint8_t* eta;     // residual in lattice order (first cycle) or null
    uint4* rho;             // residual in block order: read when eta is null
    int rho_out;            // write it back
    const uint4* fin;       // faces of the other colour's last sweep or null
    uint4* fout;            // faces of this sweep or null
    const uint4* pin;       // solution so far in block order, or null
    const uint8_t* pin_lat; // ... or in lattice order, or null (both null: zero)
    uint4* pout;            // solution in block order, or null:
    uint8_t* pout_lat;      // ... in lattice order
};

__device__ __forceinline__ void sap_load12(const uint4* p, uint32_t stride, float2* v) {
#pragma unroll
    for (int k = 0; k < 6; ++k) St<P_F32>::unpack16(p[k * stride], v + 2 * k);
}
__device__ __forceinline__ void sap_store12(uint4* p, uint32_t stride, const float2* v) {
#pragma unroll
    for (int k = 0; k < 6; ++k) p[k * stride] = St<P_F32>::pack16(v + 2 * k);
}

// Sum over the wavefront, valid in lane 63: DPP moves within the rows of 16
// lanes and broadcasts between them, where __shfl_xor takes six round trips
// through the LDS hardware.
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_last(double v) {
    v = dpp_add<0xb1, 0xf>(v);      // quad_perm 1,0,3,2
    v = dpp_add<0x4e, 0xf>(v);      // quad_perm 2,3,0,1
    v = dpp_add<0x141, 0xf>(v);     // row_half_mirror: the other quad of 8
    v = dpp_add<0x140, 0xf>(v);     // row_mirror: the other half of 16
    v = dpp_add<0x142, 0xa>(v);     // row_bcast15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);  // row_bcast31 into rows 2 and 3
}

// NT lanes per workgroup (bvol <= NT); slot NT of every LDS row is zero and
// stands for the neighbour of a hop that leaves the block.
template <int NT> struct SapBlockLds {
    float2 res[12][NT + 1];
    float2 bw[4][6][NT + 1];
    double red[NT / 64][3];
};

// A lane's place in its block and in the lattice.
struct SapLane {
    int lc[4];              // coordinates in the block
    uint32_t f[4];          // local index without coordinate mu (its place in a mu face)
    int p;                  // parity
    uint32_t ih;            // half index
};
__device__ __forceinline__ SapLane sap_lane(const SapBlockParams& P, const int* bc, int l) {
    SapLane a;
    int r = l, s = 1;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int k = (int)fdiv((uint32_t)r, P.d_b[m]);
        a.lc[m] = r - k * P.b[m];
        a.f[m] = (uint32_t)(l - r * s + s * k);
        r = k;
        s *= P.b[m];
    }
    const int x = bc[0] * P.b[0] + a.lc[0], y = bc[1] * P.b[1] + a.lc[1], z = bc[2] * P.b[2] + a.lc[2],
              t = bc[3] * P.b[3] + a.lc[3];
    a.ih = (uint32_t)(x >> 1) + (uint32_t)P.g.lxh * ((uint32_t)y + (uint32_t)P.g.ly *
                                                     ((uint32_t)z + (uint32_t)P.g.lz * (uint32_t)t));
    a.p = (x + y + z + t) & 1;
    return a;
}

// The block's neighbour d = +-1 along MU, numbered among its colour's blocks:
// the same compressed coordinates except along MU (the halved direction's
// coordinate is the same before halving).
template <int MU>
__device__ __forceinline__ uint32_t sap_nbr_block(const SapBlockParams& P, const int* bc, int d) {
    int c[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) c[m] = bc[m];
    c[MU] += d;
    if (c[MU] == P.nb[MU]) c[MU] = 0;
    if (c[MU] < 0) c[MU] = P.nb[MU] - 1;
    uint32_t a = 0;
#pragma unroll
    for (int m = 3; m >= 0; --m) a = a * (uint32_t)P.cb[m] + (uint32_t)(m == P.split ? c[m] >> 1 : c[m]);
    return a;
}

// Hops into the block across its two mu faces from the neighbouring blocks'
// last increments.  The loads of all eight faces are issued first
// (sap_faces_load), then added (sap_faces_add): a lane waits for memory once
// instead of once per face.
struct SapFaceRaw {
    uint4 up[3], dn[3];     // upper face of the block: from above; lower face: from below
};
template <int MU>
__device__ __forceinline__ void sap_faces_load(const SapBlockParams& P, const uint4* fin, const int* bc,
                                               const SapLane& a, bool act, SapFaceRaw& w) {
    if (P.nb[MU] == 1) return;
    const uint32_t nf = (uint32_t)(P.bvol / P.b[MU]);
    if (act && a.lc[MU] == P.b[MU] - 1) {
        const uint4* p = fin + (size_t)sap_nbr_block<MU>(P, bc, 1) * P.fwords + P.foff[MU] + a.f[MU];
#pragma unroll
        for (int k = 0; k < 3; ++k) w.up[k] = p[k * nf];
    }
    if (act && a.lc[MU] == 0) {
        const uint4* p = fin + (size_t)sap_nbr_block<MU>(P, bc, -1) * P.fwords + P.foff[MU] + 3 * nf + a.f[MU];
#pragma unroll
        for (int k = 0; k < 3; ++k) w.dn[k] = p[k * nf];
    }
}
template <int MU, class C>
__device__ __forceinline__ void sap_faces_add(const SapBlockParams& P, const int* bc, const SapLane& a, const C* u,
                                              bool act, const SapFaceRaw& w, C* acc) {
    if (P.nb[MU] == 1) return;
    C h[6], g[6];
    if (act && a.lc[MU] == P.b[MU] - 1) {       // (1 - gamma_mu) of the block above's lower face
#pragma unroll
        for (int k = 0; k < 3; ++k) St<P_F32>::unpack16(w.up[k], h + 2 * k);
        if (bc[MU] == P.nb[MU] - 1) {
            const C ph = mk<C>(P.ph[MU][0], P.ph[MU][1]);
#pragma unroll
            for (int k = 0; k < 6; ++k) h[k] = mul(ph, h[k]);
        }
        half_su3<true>(u, h, g);
        half_rebuild<MU, 1>(g, 1.0f, acc);
    }
    if (act && a.lc[MU] == 0) {                 // U^dag (1 + gamma_mu) of the block below's upper face
#pragma unroll
        for (int k = 0; k < 3; ++k) St<P_F32>::unpack16(w.dn[k], g + 2 * k);
        if (bc[MU] == 0) {
            const C ph = mk<C>(P.ph[MU][0], -P.ph[MU][1]);
#pragma unroll
            for (int k = 0; k < 6; ++k) g[k] = mul(ph, g[k]);
        }
        half_rebuild<MU, -1>(g, 1.0f, acc);
    }
}

template <int MU, class C>
__device__ __forceinline__ void sap_faces_out(const SapBlockParams& P, uint4* fout, int lc, uint32_t f, const C* u,
                                              bool act, const C* e) {
    if (P.nb[MU] == 1) return;
    const uint32_t nf = (uint32_t)(P.bvol / P.b[MU]);
    C h[6], g[6];
    if (act && lc == 0) {
        half_project<MU, 1>(e, h);
        uint4* p = fout + P.foff[MU] + f;
#pragma unroll
        for (int k = 0; k < 3; ++k) p[k * nf] = St<P_F32>::pack16(h + 2 * k);
    }
    if (act && lc == P.b[MU] - 1) {
        half_project<MU, -1>(e, h);
        half_su3<false>(u, h, g);
        uint4* p = fout + P.foff[MU] + 3 * nf + f;
#pragma unroll
        for (int k = 0; k < 3; ++k) p[k * nf] = St<P_F32>::pack16(g + 2 * k);
    }
}

// the backward hop of direction MU at its source: U^dag (1 + gamma_mu) res
template <int MU, int NT, class C>
__device__ __forceinline__ void sap_bw_out(SapBlockLds<NT>& L, int l, const C* u, const C* res) {
    C h[6], g[6];
    half_project<MU, -1>(res, h);
    half_su3<false>(u, h, g);
#pragma unroll
    for (int k = 0; k < 6; ++k) L.bw[MU][k][l] = g[k];
}

// both hops of direction MU inside the block: jf / jb are the local indices
// of x +- mu (slot NT where the hop leaves the block)
template <int MU, int NT, bool WRAP, class C>
__device__ __forceinline__ void sap_hops(const SapBlockParams& P, const SapBlockLds<NT>& L, int jf, int jb, int lc,
                                         const C* u, C* q) {
    C h[6], g[6];
    {
        C v[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = L.res[k][jf];
        half_project<MU, 1>(v, h);
    }
    if (WRAP && P.wrap[MU]) {
        const C w = lc == P.b[MU] - 1 ? mk<C>(P.ph[MU][0], P.ph[MU][1]) : mk<C>(1.0f, 0.0f);
#pragma unroll
        for (int k = 0; k < 6; ++k) h[k] = mul(w, h[k]);
    }
    half_su3<true>(u, h, g);
    half_rebuild<MU, 1>(g, 1.0f, q);
#pragma unroll
    for (int k = 0; k < 6; ++k) g[k] = L.bw[MU][k][jb];
    if (WRAP && P.wrap[MU]) {
        const C w = lc == 0 ? mk<C>(P.ph[MU][0], -P.ph[MU][1]) : mk<C>(1.0f, 0.0f);
#pragma unroll
        for (int k = 0; k < 6; ++k) g[k] = mul(w, g[k]);
    }
    half_rebuild<MU, -1>(g, 1.0f, q);
}

// WRAP: some direction is spanned by one block and has a phase other than 1.
template <bool L12, int NT, bool WRAP>
__global__ void __launch_bounds__(NT, 2) k_sap_block(const SapBlockParams P) {
    using C = float2;
    __shared__ SapBlockLds<NT> L;
    const uint32_t blk = xcd_block(blockIdx.x, gridDim.x, 1);
    int bc[4];
    {
        uint32_t r = blk;
        int sum = 0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            bc[m] = (int)(r % (uint32_t)P.cb[m]);
            r /= (uint32_t)P.cb[m];
            if (m != P.split) sum += bc[m];
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (m == P.split) bc[m] = 2 * bc[m] + ((sum + P.colour) & 1);
    }
    const int l = threadIdx.x;
    const bool act = l < P.bvol;
    const uint32_t n = P.g.vh;
    const uint32_t cblk = blk + (P.colour ? gridDim.x : 0);             // among all blocks, colour 0 first
    const size_t field = (size_t)blockIdx.y * P.field_words + (size_t)cblk * 6 * P.bvol;
    int jf[4], jb[4], lw[4];
    C u[4][9], res[12], e[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) { res[k] = czero<C>(); e[k] = czero<C>(); }
    {
        const SapLane a = sap_lane(P, bc, act ? l : 0);
        SapFaceRaw fr[4];
        if (P.fin) {
            const uint4* fin = P.fin + (size_t)blockIdx.y * P.face_words;
            sap_faces_load<0>(P, fin, bc, a, act, fr[0]);
            sap_faces_load<1>(P, fin, bc, a, act, fr[1]);
            sap_faces_load<2>(P, fin, bc, a, act, fr[2]);
            sap_faces_load<3>(P, fin, bc, a, act, fr[3]);
        }
        if (act) {
            if (P.eta) {
                const size_t lat = (size_t)(2 * blockIdx.y + a.p) * P.half_bytes;
                load_rec<P_F32, 12>(P.eta + lat, n, a.ih, res);
            } else {
                sap_load12(P.rho + field + l, (uint32_t)P.bvol, res);
            }
        }
        int s = 1;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int bm = P.b[m], ls = act ? l : 0;
            const bool cut = P.nb[m] > 1;               // a hop across the block's face leaves it
            load_link_as<P_F32, L12, false>(P.u + (size_t)(2 * m + a.p) * P.link_block, n, a.ih, u[m]);
            jf[m] = a.lc[m] + 1 < bm ? ls + s : (cut ? NT : ls - (bm - 1) * s);
            jb[m] = a.lc[m] > 0 ? ls - s : (cut ? NT : ls + (bm - 1) * s);
            lw[m] = a.lc[m];
            s *= bm;
        }
        if (P.fin) {
            C acc[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = czero<C>();
            sap_faces_add<0>(P, bc, a, u[0], act, fr[0], acc);
            sap_faces_add<1>(P, bc, a, u[1], act, fr[1], acc);
            sap_faces_add<2>(P, bc, a, u[2], act, fr[2], acc);
            sap_faces_add<3>(P, bc, a, u[3], act, fr[3], acc);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                res[k].x = fma(P.kappa, acc[k].x, res[k].x);
                res[k].y = fma(P.kappa, acc[k].y, res[k].y);
            }
        }
    }
    if (l < 12) L.res[l][NT] = czero<C>();
    if (l < 24) L.bw[l / 6][l % 6][NT] = czero<C>();
#pragma unroll 1
    for (int it = 0; it < P.nmr; ++it) {
        // no lane is still reading the previous step's residual: every lane
        // passed the barrier of its block sums after its last LDS read
#pragma unroll
        for (int k = 0; k < 12; ++k) L.res[k][l] = res[k];
        sap_bw_out<0>(L, l, u[0], res);
        __builtin_amdgcn_sched_barrier(0);
        sap_bw_out<1>(L, l, u[1], res);
        __builtin_amdgcn_sched_barrier(0);
        sap_bw_out<2>(L, l, u[2], res);
        __builtin_amdgcn_sched_barrier(0);
        sap_bw_out<3>(L, l, u[3], res);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        C q[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) q[k] = czero<C>();
        sap_hops<0, NT, WRAP>(P, L, jf[0], jb[0], lw[0], u[0], q);
        __builtin_amdgcn_sched_barrier(0);
        sap_hops<1, NT, WRAP>(P, L, jf[1], jb[1], lw[1], u[1], q);
        __builtin_amdgcn_sched_barrier(0);
        sap_hops<2, NT, WRAP>(P, L, jf[2], jb[2], lw[2], u[2], q);
        __builtin_amdgcn_sched_barrier(0);
        sap_hops<3, NT, WRAP>(P, L, jf[3], jb[3], lw[3], u[3], q);
        __builtin_amdgcn_sched_barrier(0);
        // q = D_L res = res - kappa H_L res; block sums <q, res>, <q, q>
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            q[k].x = act ? fma(-P.kappa, q[k].x, res[k].x) : 0.0f;
            q[k].y = act ? fma(-P.kappa, q[k].y, res[k].y) : 0.0f;
            const double qx = q[k].x, qy = q[k].y, rx = res[k].x, ry = res[k].y;
            s0 += qx * rx + qy * ry;
            s1 += qx * ry - qy * rx;
            s2 += qx * qx + qy * qy;
            __builtin_amdgcn_sched_barrier(0);
        }
        s0 = wave_sum_last(s0);
        s1 = wave_sum_last(s1);
        s2 = wave_sum_last(s2);
        if ((l & 63) == 63) { L.red[l >> 6][0] = s0; L.red[l >> 6][1] = s1; L.red[l >> 6][2] = s2; }
        __syncthreads();
        double t0 = 0.0, t1 = 0.0, t2 = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) { t0 += L.red[w][0]; t1 += L.red[w][1]; t2 += L.red[w][2]; }
        const double inv = t2 > 0.0 ? 1.0 / t2 : 0.0, a0 = t0 * inv, a1 = t1 * inv;
        const C al = mk<C>((float)a0, (float)a1);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            e[k] = fma_(al, res[k], e[k]);
            res[k] = sub(res[k], mul(al, q[k]));
        }
    }
    // the lane's place again, from an index the compiler does not know, so that
    // it holds no register during the steps
    int l2 = l;
    asm volatile("" : "+v"(l2));
    const SapLane a = sap_lane(P, bc, act ? l2 : 0);
    const size_t lat = (size_t)(2 * blockIdx.y + a.p) * P.half_bytes, bo = field + l2;
    C v[12];
    const bool add_to = P.pin != nullptr || P.pin_lat != nullptr;
    if (add_to && act) {
        if (P.pin) sap_load12(P.pin + bo, (uint32_t)P.bvol, v);
        else load_rec<P_F32, 12>(P.pin_lat + lat, n, a.ih, v);
    }
    if (P.fout) {
        uint4* fo = P.fout + (size_t)blockIdx.y * P.face_words + (size_t)blk * P.fwords;
        sap_faces_out<0>(P, fo, a.lc[0], a.f[0], u[0], act, e);
        sap_faces_out<1>(P, fo, a.lc[1], a.f[1], u[1], act, e);
        sap_faces_out<2>(P, fo, a.lc[2], a.f[2], u[2], act, e);
        sap_faces_out<3>(P, fo, a.lc[3], a.f[3], u[3], act, e);
    }
    if (!act) return;
    if (P.rho_out) sap_store12(P.rho + bo, (uint32_t)P.bvol, res);
    if (add_to) {
#pragma unroll
        for (int k = 0; k < 12; ++k) e[k] = add(v[k], e[k]);
    }
    if (P.pout) sap_store12(P.pout + bo, (uint32_t)P.bvol, e);
    else store_rec<P_F32, 12>(P.pout_lat + lat, n, a.ih, e);
}

}  // namespace weo

// ---- flexible GCR vectors ------------------------------------------------------
// Fields as flat arrays of 16-byte chunks (two FP32 or one FP64 complex).
namespace weo {

template <int SP> struct GChunk;
template <> struct GChunk<P_F32> {
    static constexpr int N = 2;
    __device__ static void unpack(const uint4& w, double2* v) {
        v[0] = make_double2(__uint_as_float(w.x), __uint_as_float(w.y));
        v[1] = make_double2(__uint_as_float(w.z), __uint_as_float(w.w));
    }
    __device__ static uint4 pack(const double2* v) {
        return make_uint4(__float_as_uint((float)v[0].x), __float_as_uint((float)v[0].y),
                          __float_as_uint((float)v[1].x), __float_as_uint((float)v[1].y));
    }
};
template <> struct GChunk<P_F64> {
    static constexpr int N = 1;
    __device__ static void unpack(const uint4& w, double2* v) {
        v[0].x = __hiloint2double((int)w.y, (int)w.x);
        v[0].y = __hiloint2double((int)w.w, (int)w.z);
    }
    __device__ static uint4 pack(const double2* v) {
        const unsigned long long a = (unsigned long long)__double_as_longlong(v[0].x);
        const unsigned long long b = (unsigned long long)__double_as_longlong(v[0].y);
        return make_uint4((unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32));
    }
};

constexpr int kGcrWG = 1024;
struct GcrVecs {
    const uint4* v[kGcrMax];
    int n;
};
struct GcrCoef {
    double re[kGcrMax], im[kGcrMax];
};

// part[(l 2 + {re, im}) nwg + wg] = sum over the workgroup's chunks of conj(a_l) b
template <int SP>
__global__ void __launch_bounds__(256) k_gcr_dots(uint64_t nch, GcrVecs A, const uint4* b, double* part) {
    using K = GChunk<SP>;
    double sr[kGcrMax], si[kGcrMax];
#pragma unroll
    for (int l = 0; l < kGcrMax; ++l) sr[l] = si[l] = 0.0;
    for (uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nch; c += (uint64_t)gridDim.x * blockDim.x) {
        double2 bv[K::N];
        K::unpack(b[c], bv);
#pragma unroll
        for (int l = 0; l < kGcrMax; ++l) {
            if (l < A.n) {
                double2 av[K::N];
                K::unpack(A.v[l][c], av);
#pragma unroll
                for (int e = 0; e < K::N; ++e) {
                    sr[l] = fma(av[e].x, bv[e].x, fma(av[e].y, bv[e].y, sr[l]));
                    si[l] = fma(av[e].x, bv[e].y, fma(-av[e].y, bv[e].x, si[l]));
                }
            }
        }
    }
    __shared__ double red[4][2 * kGcrMax];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int l = 0; l < kGcrMax; ++l) {
        if (l < A.n) {
            const double a = wave_sum64(sr[l]), c = wave_sum64(si[l]);
            if (lane == 0) { red[w][2 * l] = a; red[w][2 * l + 1] = c; }
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * A.n) {
        double t = 0.0;
        for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += red[q][threadIdx.x];
        part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// b += sum_l c_l a_l; partials ||b||^2 at part[0 .. nwg) and, with r, <b, r>
// at part[nwg .. 3 nwg) (re then im)
template <int SP>
__global__ void __launch_bounds__(256) k_gcr_update(uint64_t nch, GcrVecs A, GcrCoef cf, uint4* b, const uint4* r,
                                                    double* part) {
    using K = GChunk<SP>;
    double nn = 0.0, dr = 0.0, di = 0.0;
    for (uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nch; c += (uint64_t)gridDim.x * blockDim.x) {
        double2 bv[K::N];
        K::unpack(b[c], bv);
#pragma unroll
        for (int l = 0; l < kGcrMax; ++l) {
            if (l < A.n) {              // constant indices keep the arguments in registers
                double2 av[K::N];
                K::unpack(A.v[l][c], av);
#pragma unroll
                for (int e = 0; e < K::N; ++e) {
                    bv[e].x = fma(cf.re[l], av[e].x, fma(-cf.im[l], av[e].y, bv[e].x));
                    bv[e].y = fma(cf.re[l], av[e].y, fma(cf.im[l], av[e].x, bv[e].y));
                }
            }
        }
        const uint4 wv = K::pack(bv);
        b[c] = wv;
        if (part) {
            double2 st[K::N];
            K::unpack(wv, st);                 // the stored values
            double2 rv[K::N];
            if (r) K::unpack(r[c], rv);
#pragma unroll
            for (int e = 0; e < K::N; ++e) {
                nn = fma(st[e].x, st[e].x, fma(st[e].y, st[e].y, nn));
                if (r) {
                    dr = fma(st[e].x, rv[e].x, fma(st[e].y, rv[e].y, dr));
                    di = fma(st[e].x, rv[e].y, fma(-st[e].y, rv[e].x, di));
                }
            }
        }
    }
    if (!part) return;
    __shared__ double red[4][3];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    nn = wave_sum64(nn);
    dr = wave_sum64(dr);
    di = wave_sum64(di);
    if (lane == 0) { red[w][0] = nn; red[w][1] = dr; red[w][2] = di; }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
        for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += red[q][threadIdx.x];
        part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

}  // namespace weo

// ------------------------------------------------------------------ host ----
namespace weo {

template <int SP, int LP, bool L12>
static hipError_t sap_launch(const SapParams& P, dim3 grid, dim3 block, hipStream_t s) {
    hipLaunchKernelGGL((k_sap_sweep<SP, LP, L12>), grid, block, 0, s, P);
    return hipGetLastError();
}

hipError_t launch_sap_sweep(const Geom& g, int fmt, const SapGeom& sg, int colour, int nmr, double kappa,
                            const double ph[4][2], const void* u, void* rho, void* phi, const void* dprev,
                            void* dout, int nrhs, hipStream_t s) {
    SapParams P;
    P.g = g;
    for (int m = 0; m < 4; ++m) { P.b[m] = sg.b[m]; P.nb[m] = sg.nb[m]; P.ph[m][0] = ph[m][0]; P.ph[m][1] = ph[m][1]; }
    P.bvol = sg.bvol;
    P.colour = colour;
    P.nmr = nmr;
    P.kappa = kappa;
    P.u = static_cast<const uint8_t*>(u);
    P.link_block = gauge_block_bytes(g, fmt);
    P.half_bytes = spinor_field_bytes(g, fmt);
    P.rho = static_cast<uint8_t*>(rho);
    P.phi = static_cast<uint8_t*>(phi);
    P.dprev = static_cast<const uint8_t*>(dprev);
    P.dout = static_cast<uint8_t*>(dout);
    const dim3 grid((unsigned)sg.nblocks, (unsigned)nrhs);
    const dim3 block((unsigned)((sg.bvol + 63) / 64 * 64));
    switch (fmt) {
        case FMT_S_S_18: return sap_launch<P_F32, P_F32, false>(P, grid, block, s);
        case FMT_S_S_12: return sap_launch<P_F32, P_F32, true>(P, grid, block, s);
        default: return hipErrorInvalidValue;
    }
}

int make_sap_geom(const Geom& g, const int block[4], SapGeom* sg) {
    const int L[4] = {g.lx, g.ly, g.lz, g.lt};
    int vol = 1, nbt = 1;
    for (int m = 0; m < 4; ++m) {
        const int b = block[m];
        if (b < 1 || b > L[m] || L[m] % b) return -1;
        const int n = L[m] / b;
        if (n != 1 && (n & 1)) return -1;
        sg->b[m] = b;
        sg->nb[m] = n;
        vol *= b;
        nbt *= n;
        if (vol > kSapMaxSites) return -1;
    }
    sg->bvol = vol;
    sg->nblocks = nbt;
    return 0;
}

// 16-byte words of one block's projected faces (2 faces of 3 words per site
// for every direction the lattice is cut in); off[mu]: those before mu.
static int sap_face_words(const SapGeom& sg, int* off) {
    int w = 0;
    for (int m = 0; m < 4; ++m) {
        if (off) off[m] = w;
        if (sg.nb[m] > 1) w += 6 * (sg.bvol / sg.b[m]);
    }
    return w;
}

// Whether the faces of all blocks fit two of the three scratch fields (one
// field is 6 words per site, one colour's faces lie in each): every layout
// with sum 1 / b_mu <= 2 over the cut directions: 2^4 (2) and (1, 4, 4, 4)
// (1.75) do, (1, 2, 2, 4) (2.25) and (1, 2, 2, 2) (2.5) do not.  The others
// take k_sap_sweep.
static bool sap_blocks_fit(const SapGeom& sg) { return sap_face_words(sg, nullptr) <= 12 * sg.bvol; }

template <bool L12, bool WRAP>
static hipError_t sap_block_launch(const SapBlockParams& P, dim3 grid, hipStream_t s) {
    if (P.bvol <= 64) hipLaunchKernelGGL((k_sap_block<L12, 64, WRAP>), grid, dim3(64), 0, s, P);
    else if (P.bvol <= 128) hipLaunchKernelGGL((k_sap_block<L12, 128, WRAP>), grid, dim3(128), 0, s, P);
    else hipLaunchKernelGGL((k_sap_block<L12, 256, WRAP>), grid, dim3(256), 0, s, P);
    return hipGetLastError();
}

static hipError_t sap_apply_blocks(const Geom& g, int fmt, const SapGeom& sg, int ncy, int nmr, double kappa,
                                   const double ph[4][2], const void* u, const void* eta, void* psi, void* rho,
                                   void* d0, void* d1, int nrhs, hipStream_t s) {
    const bool two = sg.nblocks > 1;
    SapBlockParams P;
    P.g = g;
    P.split = -1;
    bool wrap = false;
    for (int m = 0; m < 4; ++m) {
        P.b[m] = sg.b[m];
        P.d_b[m] = make_fastdiv((uint32_t)sg.b[m]);
        P.nb[m] = P.cb[m] = sg.nb[m];
        if (P.split < 0 && sg.nb[m] > 1) { P.split = m; P.cb[m] = sg.nb[m] / 2; }
        P.ph[m][0] = (float)ph[m][0];
        P.ph[m][1] = (float)ph[m][1];
        P.wrap[m] = sg.nb[m] == 1 && (ph[m][0] != 1.0 || ph[m][1] != 0.0);
        wrap = wrap || P.wrap[m];
    }
    P.bvol = sg.bvol;
    P.nmr = nmr;
    P.kappa = (float)kappa;
    P.fwords = sap_face_words(sg, P.foff);
    P.u = static_cast<const uint8_t*>(u);
    P.link_block = gauge_block_bytes(g, fmt);
    P.half_bytes = spinor_field_bytes(g, fmt);
    P.field_words = (size_t)sg.nblocks * sg.bvol * 6;
    P.face_words = (size_t)(sg.nblocks / 2) * P.fwords;
    P.rho = static_cast<uint4*>(rho);
    // Faces within one field (sum 1 / b_mu <= 1, e.g. 4^4): both colours in
    // d1, the solution in block order in d0 until the last cycle.  Else one
    // colour in each and the solution in lattice order throughout.
    const bool small = P.fwords <= 6 * sg.bvol;
    uint4* face[2] = {small ? static_cast<uint4*>(d1) : static_cast<uint4*>(d0),
                      small ? static_cast<uint4*>(d1) + (size_t)nrhs * P.face_words : static_cast<uint4*>(d1)};
    uint4* pblk = small ? static_cast<uint4*>(d0) : nullptr;
    const dim3 grid((unsigned)(two ? sg.nblocks / 2 : 1), (unsigned)nrhs);
    for (int cy = 0; cy < ncy; ++cy)
        for (int c = 0; c < (two ? 2 : 1); ++c) {
            const bool first = cy == 0, last = cy == ncy - 1;
            P.colour = c;
            P.eta = first ? static_cast<const uint8_t*>(eta) : nullptr;
            P.rho_out = !last;
            P.fin = two && !(first && c == 0) ? face[1 - c] : nullptr;
            P.fout = two && !(last && c == 1) ? face[c] : nullptr;
            P.pin = first ? nullptr : pblk;
            P.pin_lat = first || pblk ? nullptr : static_cast<const uint8_t*>(psi);
            P.pout = last ? nullptr : pblk;
            P.pout_lat = static_cast<uint8_t*>(psi);
            hipError_t e = hipErrorInvalidValue;
            if (fmt == FMT_S_S_18) e = wrap ? sap_block_launch<false, true>(P, grid, s) : sap_block_launch<false, false>(P, grid, s);
            if (fmt == FMT_S_S_12) e = wrap ? sap_block_launch<true, true>(P, grid, s) : sap_block_launch<true, false>(P, grid, s);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t sap_apply(const Geom& g, int fmt, const SapGeom& sg, int ncy, int nmr, double kappa,
                     const double ph[4][2], const void* u, const void* eta, void* psi, void* rho, void* d0,
                     void* d1, int nrhs, hipStream_t s) {
    if (sap_blocks_fit(sg)) return sap_apply_blocks(g, fmt, sg, ncy, nmr, kappa, ph, u, eta, psi, rho, d0, d1, nrhs, s);
    const size_t bytes = (size_t)nrhs * 2 * spinor_field_bytes(g, fmt);
    hipError_t e = hipMemcpyAsync(rho, eta, bytes, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    if ((e = launch_zero(psi, bytes, s)) != hipSuccess) return e;
    // with one block along every direction there is one colour and no hop
    // between blocks
    const bool two = sg.nblocks > 1;
    const void* prev = nullptr;
    for (int cy = 0; cy < ncy; ++cy)
        for (int c = 0; c < (two ? 2 : 1); ++c) {
            void* out = c ? d1 : d0;
            e = launch_sap_sweep(g, fmt, sg, c, nmr, kappa, ph, u, rho, psi, prev, out, nrhs, s);
            if (e != hipSuccess) return e;
            prev = two ? out : nullptr;
        }
    return hipSuccess;
}

uint32_t gcr_wg(const Geom& gb, int fmt) {
    const uint64_t nch = spinor_field_bytes(gb, fmt) / 16;
    const uint64_t w = (nch + 255) / 256;
    return (uint32_t)(w < (uint64_t)kGcrWG ? w : (uint64_t)kGcrWG);
}

static GcrVecs gcr_vecs(int n, const void* const* v) {
    GcrVecs a;
    a.n = n;
    for (int l = 0; l < kGcrMax; ++l) a.v[l] = static_cast<const uint4*>(l < n ? v[l] : v[0]);
    return a;
}

hipError_t launch_gcr_dots(const Geom& gb, int fmt, int n, const void* const* a, const void* b, double* part,
                           hipStream_t s) {
    if (n < 1 || n > kGcrMax) return hipErrorInvalidValue;
    const uint64_t nch = spinor_field_bytes(gb, fmt) / 16;
    const GcrVecs A = gcr_vecs(n, a);
    const dim3 grid(gcr_wg(gb, fmt)), block(256);
    const uint4* bp = static_cast<const uint4*>(b);
    if (fmt_info(fmt).spinor_prec == P_F64)
        hipLaunchKernelGGL((k_gcr_dots<P_F64>), grid, block, 0, s, nch, A, bp, part);
    else if (fmt_info(fmt).spinor_prec == P_F32)
        hipLaunchKernelGGL((k_gcr_dots<P_F32>), grid, block, 0, s, nch, A, bp, part);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_gcr_update(const Geom& gb, int fmt, int n, const void* const* a, const double* cre,
                             const double* cim, void* b, const void* r, double* part, hipStream_t s) {
    if (n < 0 || n > kGcrMax) return hipErrorInvalidValue;
    const uint64_t nch = spinor_field_bytes(gb, fmt) / 16;
    const void* dummy[1] = {b};
    const GcrVecs A = gcr_vecs(n, n ? a : dummy);
    GcrCoef cf;
    for (int l = 0; l < kGcrMax; ++l) { cf.re[l] = l < n ? cre[l] : 0.0; cf.im[l] = l < n ? cim[l] : 0.0; }
    const dim3 grid(gcr_wg(gb, fmt)), block(256);
    uint4* bp = static_cast<uint4*>(b);
    const uint4* rp = static_cast<const uint4*>(r);
    if (fmt_info(fmt).spinor_prec == P_F64)
        hipLaunchKernelGGL((k_gcr_update<P_F64>), grid, block, 0, s, nch, A, cf, bp, rp, part);
    else if (fmt_info(fmt).spinor_prec == P_F32)
        hipLaunchKernelGGL((k_gcr_update<P_F32>), grid, block, 0, s, nch, A, cf, bp, rp, part);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace weo
