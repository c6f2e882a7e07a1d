// Shared by the multi right-hand-side hop kernels (hop_mrhs.hip, hop_lw.hip).
#pragma once

#include "hop_core.h"

namespace weo {

// Output records of the multi-RHS kernels are written with streaming stores
// in every precision: with many fields per site the output lines would
// otherwise take L2 from the input records that the +-z and +-t neighbours
// read again (FP32/18 and FP16/12 at 12 rhs: 4 % faster).  -D
// WEO_MRHS_NT_STORE=0 restores regular stores for comparison.
#ifdef WEO_MRHS_NT_STORE
template <int SP> constexpr bool mrhs_nt_store() { return WEO_MRHS_NT_STORE != 0; }
#else
template <int SP> constexpr bool mrhs_nt_store() { return true; }
#endif

// Byte offsets of the 8 neighbours in a spinor plane (16 bytes a site).  Loops
// over right-hand sides take them and the field index through opaque copies
// in every iteration: the compiler otherwise keeps a 64-bit address per
// plane and neighbour in registers across the loop (FP16/12 link-resident
// form: 248 registers, 2 wavefronts per SIMD) instead of addressing with
// scalar bases and one 32-bit offset per neighbour.
struct NbrOff {
    uint32_t o[8];
    __device__ __forceinline__ void set(const Nbr& nb) {
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = nb.i[k] * 16u;
    }
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(o[k]));
    }
};
__device__ __forceinline__ int opaque_uniform(int r) {
    asm volatile("" : "+v"(r));
    return __builtin_amdgcn_readfirstlane(r);
}
template <int SP>
__device__ __forceinline__ void load_spinor(const uint8_t* __restrict__ base, uint32_t n, uint32_t off,
                                            RawRec<SP, 12>& r) {
    const size_t pb = (size_t)n * 16;
#pragma unroll
    for (int p = 0; p < Rec<SP, 12>::NFULL; ++p) r.w[p] = ld16<false>(base + p * pb + off);
}

struct MrhsParams {
    HopParams h;
    int nrhs;
    uint32_t nblk;      // site blocks of blockDim.x sites
    int rhs_per_row;    // LDS-staged form: right-hand sides per grid row
    const uint8_t* clv; // LDS-staged form: the output parity's two clover blocks, or null
    size_t block_bytes;
};

// ---- FP16 pairs (FP16 spinors and links) ----------------------------------------
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h2v h2v_of(uint32_t w) { return __builtin_bit_cast(h2v, w); }
__device__ __forceinline__ uint32_t u32_of(h2v v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2(h2v_of(a), h2v_of(b), c, false);
}
__device__ __forceinline__ uint32_t swap_pair(uint32_t w) { return __builtin_amdgcn_alignbit(w, w, 16); }

struct Link16 {
    uint32_t e[9];       // U_ab as FP16 pairs, row-major
};

// Link of direction k of the site (raw FP16 words), third row rebuilt for
// 12 reals, boundary phase ph folded in on edge hops (ph U forward,
// (ph U)^dag = conj(ph) U^dag backward, so the stored link is ph U either way).
template <bool L12, bool CPH>
__device__ __forceinline__ void link16_of(const RawRec<P_F16, L12 ? 6 : 9, true>& r, bool edge, float2 ph, Link16& L) {
    constexpr int NW = L12 ? 6 : 9;
    uint32_t w[9];
#pragma unroll
    for (int p = 0; p < Rec<P_F16, NW>::NFULL; ++p) {
        w[4 * p] = r.w[p].x; w[4 * p + 1] = r.w[p].y; w[4 * p + 2] = r.w[p].z; w[4 * p + 3] = r.w[p].w;
    }
    if constexpr (Rec<P_F16, NW>::TAILB == 8) { w[4 * Rec<P_F16, NW>::NFULL] = r.t8.x; w[4 * Rec<P_F16, NW>::NFULL + 1] = r.t8.y; }
    if constexpr (Rec<P_F16, NW>::TAILB == 4) w[4 * Rec<P_F16, NW>::NFULL] = r.t4;
    if constexpr (L12) {
        float2 u[9];
#pragma unroll
        for (int k = 0; k < 6; ++k) u[k] = h2_to_f2(w[k]);
        complete_link(u);
#pragma unroll
        for (int k = 6; k < 9; ++k) w[k] = f2_to_h2(u[k]);
    }
    if constexpr (CPH) {
        const float2 f = edge ? ph : make_float2(1.f, 0.f);
#pragma unroll
        for (int k = 0; k < 9; ++k) L.e[k] = f2_to_h2(mul(f, h2_to_f2(w[k])));
    } else {
        // a real phase +-1: a sign flip of both halves where it is -1
        const uint32_t flip = (edge && ph.x < 0.f) ? 0x80008000u : 0u;
#pragma unroll
        for (int k = 0; k < 9; ++k) L.e[k] = w[k] ^ flip;
    }
}

template <bool L12, bool CPH>
__device__ __forceinline__ void link16_load(const uint8_t* base, uint32_t n, uint32_t i, bool edge, float2 ph,
                                            Link16& L) {
    RawRec<P_F16, L12 ? 6 : 9, true> r;
    r.load(base, n, i);
    link16_of<L12, CPH>(r, edge, ph, L);
}

__device__ __forceinline__ void rec16_words(const RawRec<P_F16, 12>& r, uint32_t* p) {
#pragma unroll
    for (int q = 0; q < 3; ++q) { p[4 * q] = r.w[q].x; p[4 * q + 1] = r.w[q].y; p[4 * q + 2] = r.w[q].z; p[4 * q + 3] = r.w[q].w; }
}

// Every phase 1 or -1, as the sign-flip form of the packed FP16 links needs
// (an open direction has phase 0).
inline bool phases_are_signs(const HopLaunch& h) {
    for (int m = 0; m < 4; ++m)
        if (h.phase[m][1] != 0.0 || (h.phase[m][0] != 1.0 && h.phase[m][0] != -1.0)) return false;
    return true;
}

// The packed FP16 form with LDS-staged links in MrhsCfg::nr: record ring
// depth 1 / 3, MrhsCfg::s wavefronts.  Not selectable from outside.
constexpr int kNrLw16 = -7, kNrLw16Deep = -8;
hipError_t launch_hop_lw16(const HopLaunch& h, const MrhsParams& M, int W, int depth, dim3 grid, hipStream_t s);

int lw_max_waves(int fmt);      // most wavefronts per workgroup of the LDS-staged form
hipError_t launch_hop_lw(const HopLaunch& h, const MrhsParams& M, int W, dim3 grid, hipStream_t s);

}  // namespace weo
