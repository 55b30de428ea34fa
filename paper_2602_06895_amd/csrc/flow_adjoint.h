// Reverse mode of the inverse rational-quadratic spline within its bin.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace msx {

// gp = derivatives of ge ld + ax x with respect to (y, x0, w, y0, h, d0, d1),
// with x = S^-1(y) and ld = log (S^-1)'(y) = -log S'(x) in the bin at (x0, y0)
// of width w, height h and knot slopes d0, d1.
//
// Forward derivatives through the closed-form root, of y, w, h, d0 and d1 only
// (x = x0 + ..., and y enters as y - y0); a derivative that is zero has no
// term.  Which product of a sum is fused is written out, so every kernel gets
// the same bits: the results are rounded to BF16, and a last bit that moves
// with the compiler's choice would move such a rounding.
__device__ __forceinline__ void spline_inverse_adjoint(float y, float w, float y0, float h, float d0, float d1,
                                                       float ge, float ax, float (&gp)[7]) {
#pragma clang fp contract(off)
    auto fma = [](float a, float b, float c) { return __builtin_fmaf(a, b, c); };
    const float iw = 1.0f / w, s = h * iw, dy = y - y0;
    const float kap = d1 + d0 - 2.0f * s, sd = fma(h, iw, -d0), dk = dy * kap;
    // the root of qa xi^2 + qb xi + qc
    const float qa = fma(h, sd, dk), qb = fma(h, d0, -dk), qc = -(s * dy);
    const float sq = sqrtf(fmaxf(fma(qb, qb, -(4.0f * (qa * qc))), 1e-30f)), hs = 0.5f / sq;
    const float ib = 1.0f / (-qb - sq), n2 = 2.0f * qc, xi = n2 * ib;
    const float xc = fma(-n2, ib, 1.0f), om = xi * xc;  // 1 - xi, xi (1 - xi)
    // S' = s^2 (d1 xi^2 + 2 s om + d0 xc^2) / den^2
    const float den = fma(kap, om, s), t = d1 * xi, u = d0 * xc, ss = s * s;
    const float sum = fma(u, xc, fma(t, xi, 2.0f * (s * om)));
    const float iden = 1.0f / den, inum = 1.0f / (ss * sum);

    // derivative of xi from those of the coefficients (gc: of qc, 0 where NC)
    auto root = [&](auto nc, float ga, float gb, float gc, bool y_or_slope) {
        const float p = decltype(nc)::value ? ga * qc : (y_or_slope ? fma(ga, qc, qa * gc) : fma(qa, gc, ga * qc));
        const float g = fma(gb, qb, qb * gb) - 4.0f * p;
        const float gd = fma(-g, hs, -gb);
        return (decltype(nc)::value ? -(xi * gd) : 2.0f * gc - xi * gd) * ib;
    };
    // ax x' + ge ld' from xi' (gx), that of den (gden), of d1 xi (gt), of d0 xc
    // (gu), of s om (gm), of s (gs, 0 where NS) and of x
    auto total = [&](auto ns, float gx, float gden, float gt, float gu, float gm, float gs, float gX) {
        const float ga = fma(t, gx, gt * xi), gb = fma(u, -gx, gu * xc);
        const float gsum = (ga + 2.0f * gm) + gb;
        const float gnum = decltype(ns)::value ? ss * gsum : fma(fma(gs, s, s * gs), sum, ss * gsum);
        const float gld = 2.0f * (gden * iden) - gnum * inum;
        return fma(ax, gX, ge * gld);
    };
    auto om_of = [&](float gx) { return fma(gx, xc, xi * -gx); };
    {  // y
        const float gx = root(std::false_type{}, kap, -kap, -s, true), go = om_of(gx);
        gp[0] = total(std::true_type{}, gx, kap * go, d1 * gx, -(d0 * gx), s * go, 0.0f, gx * w);
        gp[1] = ax;
        gp[3] = -gp[0];
    }
    {  // w
        const float gs = -s * iw, gk = -2.0f * gs;
        const float gx = root(std::false_type{}, h * gs + dy * gk, -(dy * gk), -(gs * dy), false), go = om_of(gx);
        gp[2] = total(std::false_type{}, gx, fma(-s, iw, fma(gk, om, kap * go)), d1 * gx, -(d0 * gx), fma(gs, om, s * go), gs,
                      fma(gx, w, xi));
    }
    {  // h
        const float gk = -2.0f * iw;
        const float gx = root(std::false_type{}, fma(h, iw, sd) + dy * gk, d0 - dy * gk, -(iw * dy), false), go = om_of(gx);
        gp[4] = total(std::false_type{}, gx, iw + fma(gk, om, kap * go), d1 * gx, -(d0 * gx), fma(iw, om, s * go), iw, gx * w);
    }
    {  // d0
        const float gx = root(std::true_type{}, dy - h, h - dy, 0.0f, true), go = om_of(gx);
        gp[5] = total(std::true_type{}, gx, fma(kap, go, om), d1 * gx, fma(d0, -gx, xc), s * go, 0.0f, gx * w);
    }
    {  // d1
        const float gx = root(std::true_type{}, dy, -dy, 0.0f, true), go = om_of(gx);
        gp[6] = total(std::true_type{}, gx, fma(kap, go, om), fma(d1, gx, xi), -(d0 * gx), s * go, 0.0f, gx * w);
    }
}

}  // namespace msx
