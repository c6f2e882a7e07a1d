// Half spinors: the projection of a spinor with (1 - S gamma_mu), the SU(3)
// product on its two colour vectors, and the rebuilt full spinor (the rules
// stated in hop_core.h).  Shared by the kernels that store or exchange
// projected spinors instead of full ones.
#pragma once

#include "weo_device.h"

namespace weo {

// h = the two independent spin rows of (1 - S gamma_mu) p (for t the two
// surviving rows without their factor 2).
template <int MU, int S, class C>
__device__ __forceinline__ void half_project(const C* p, C* h) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const C p0 = p[c], p1 = p[3 + c], p2 = p[6 + c], p3 = p[9 + c];
        C h0, h1;
        if constexpr (MU == 0) {
            h0 = S > 0 ? add(p0, imul(p3)) : sub(p0, imul(p3));
            h1 = S > 0 ? add(p1, imul(p2)) : sub(p1, imul(p2));
        } else if constexpr (MU == 1) {
            h0 = S > 0 ? add(p0, p3) : sub(p0, p3);
            h1 = S > 0 ? sub(p1, p2) : add(p1, p2);
        } else if constexpr (MU == 2) {
            h0 = S > 0 ? add(p0, imul(p2)) : sub(p0, imul(p2));
            h1 = S > 0 ? sub(p1, imul(p3)) : add(p1, imul(p3));
        } else {
            h0 = S > 0 ? p2 : p0;
            h1 = S > 0 ? p3 : p1;
        }
        h[c] = h0;
        h[3 + c] = h1;
    }
}

// acc += a * (the full spinor of (1 - S gamma_mu) rebuilt from half spinor g)
template <int MU, int S, class C, class R>
__device__ __forceinline__ void half_rebuild(const C* g, R a, C* acc) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const C g0 = g[c], g1 = g[3 + c];
        C u0 = g0, u1 = g1, l0, l1;         // upper rows; lower rows
        if constexpr (MU == 0) {
            l0 = S > 0 ? scal(R(-1), imul(g1)) : imul(g1);
            l1 = S > 0 ? scal(R(-1), imul(g0)) : imul(g0);
        } else if constexpr (MU == 1) {
            l0 = S > 0 ? scal(R(-1), g1) : g1;
            l1 = S > 0 ? g0 : scal(R(-1), g0);
        } else if constexpr (MU == 2) {
            l0 = S > 0 ? scal(R(-1), imul(g0)) : imul(g0);
            l1 = S > 0 ? imul(g1) : scal(R(-1), imul(g1));
        }
        if constexpr (MU == 3) {
            // (1 - S gamma_t) = 2 x the projector on rows 2, 3 (S > 0) or 0, 1
            const int o = S > 0 ? 6 : 0;
            acc[o + c].x = fma(R(2) * a, g0.x, acc[o + c].x);
            acc[o + c].y = fma(R(2) * a, g0.y, acc[o + c].y);
            acc[o + 3 + c].x = fma(R(2) * a, g1.x, acc[o + 3 + c].x);
            acc[o + 3 + c].y = fma(R(2) * a, g1.y, acc[o + 3 + c].y);
        } else {
            acc[c].x = fma(a, u0.x, acc[c].x);         acc[c].y = fma(a, u0.y, acc[c].y);
            acc[3 + c].x = fma(a, u1.x, acc[3 + c].x); acc[3 + c].y = fma(a, u1.y, acc[3 + c].y);
            acc[6 + c].x = fma(a, l0.x, acc[6 + c].x); acc[6 + c].y = fma(a, l0.y, acc[6 + c].y);
            acc[9 + c].x = fma(a, l1.x, acc[9 + c].x); acc[9 + c].y = fma(a, l1.y, acc[9 + c].y);
        }
    }
}

// g = U h (FWD) or U^dag h on both colour vectors of a half spinor.
template <bool FWD, class C>
__device__ __forceinline__ void half_su3(const C* u, const C* h, C* g) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if constexpr (FWD) {
                C t = mul(u[3 * a], h[3 * s]);
                t = fma_(u[3 * a + 1], h[3 * s + 1], t);
                g[3 * s + a] = fma_(u[3 * a + 2], h[3 * s + 2], t);
            } else {
                C t = mulc(u[a], h[3 * s]);
                t = fmac_(u[3 + a], h[3 * s + 1], t);
                g[3 * s + a] = fmac_(u[6 + a], h[3 * s + 2], t);
            }
        }
}

}  // namespace weo
