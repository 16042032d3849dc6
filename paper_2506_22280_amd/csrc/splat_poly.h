// splat_poly.h -- the exact model's exponent over one 8x8 pixel block as a quartic polynomial.
//
// A pixel's value is |e| 2^X sign(amp) with X = E/q - log2(q)/2 + log2|amp|, E and q the record's
// quadratics (common.h). q differs from its value at a block's centre by under a per cent (the
// perspective over 8 pixels), so E/q and log2 q are expanded there: with s, t the pixel's column
// and row less the centre's, q = q00 (1 + p10 s + p01 t + p20 s^2 + p11 st + p02 t^2) and
// E = q00 (e00 + e10 s + ...), the series y = E/q follows from y q = E coefficient by coefficient,
// and log2 q to second order. A pixel then costs 2.5 multiply-adds and one exp2 (two columns at
// +-s share the even and odd parts) instead of a reciprocal square root, an exp2 and seven others.
//
// The series is cut after total degree 4. With l and c the largest linear and quadratic part of
// q / q00 - 1 over the block, and rho the largest distance of its pixels from its centre in standard
// deviations of the Gaussian, what is left out changes a pixel's value by at most about
// (rho^2 + 1/2) (l^3 + 2 l c + c^2) / 2 of the Gaussian's peak (poly_error, derived there): the
// quadratic part is small like l, but takes up two degrees. The set-up evaluates the bound per
// (view, Gaussian) and marks the record: the plain series up to POLY_PLAIN, direct evaluation above
// POLY_FOLD, and between them the degree-5 terms folded into the lower ones (each power replaced by
// its closest lower polynomial over the block's pixel positions, the log to third order), which
// leaves an eighth of the value's error. The moments keep the order of the plain series, and with
// that half the bound, relative to the amplitude's gradient, in the gradients of orientation and
// scale; hence the limit on folded records, at the error of the FP32 evaluation by forward
// differences (Gaussians of one to four pixels: 1e-6 to 4e-6). Evaluated directly as well are
// Gaussians with rho^2 above POLY_RHO2 (0.6 of a pixel if round): the series is a small difference of
// terms of the order of rho^2 there, and its FP32 rounding exceeds that of the forward differences
// (largest error of an image, pitch 0.5 mm, aspects up to 3: 0.3 pixels 1.3e-5 against 5.8e-6 of its
// maximum, 0.5 pixels 6.7e-6 against 3.2e-6, 0.6 and 0.8 pixels the same).
#pragma once

#include "common.h"

#define POLY_PLAIN 2.0e-6f
#define POLY_FOLD 4.0e-6f
#define POLY_RHO2 64.0f
#define POLY_HL 0.72134752044448170f   // log2(e) / 2

// Index of s^i t^j (i + j <= 4) among the 15 coefficients and moments.
__host__ __device__ constexpr int pidx(int i, int j)
{
    const int d = i + j;
    return d * (d + 1) / 2 + j;
}

struct BlockPoly {
    float c[15];                        // X (without log2|amp|)
    float p10, p01, p20, p11, p02;      // q / q00 - 1
    float iq, lrs;                      // 1 / q00, -log2(q00) / 2
    float du, dv;                       // the block's centre less the footprint's
};

// Largest squared distance of a block's pixels from its centre in deviations of the Gaussian
__host__ __device__ inline float poly_rho2(float Huu, float Huv, float Hvv)
{
    return 12.25f * (Huu + 2.0f * fabsf(Huv) + Hvv);
}

// Bound, in units of the Gaussian's peak, on the error of a pixel's value by the plain series over any
// block whose centre lies within (ru, rv) pixels of the projected mean: H, g and G the record's
// quadratic forms (q = 1 + 2 g.d + d^T G d). With L and C the linear and quadratic part of q / q00 - 1
// (|L| <= l, |C| <= c), y_n the part of degree n of E/q and A the distance of the block's centre from
// the mean in deviations, dividing out the series leaves, over 1 + L + C and to second order in c,
//   (-L^3 + 2 L C + C^2) y2 + C^2 y1  and, of the logarithm, (-L C + L^3/3 - C^2/2) / 2,
// in natural units, where |y1| <= A rho and |y2| <= rho^2 / 2 to first order; the pixel's own value, at
// most exp(-(A - rho)^2 / 2) of the peak, keeps its product with A below rho + 0.61. 1/q00 <= iq, as
// G is positive. NaN or infinite where q may come near 0. Measured against FP64 over Gaussians of
// 0.15 to 6 pixels, aspects up to 9 and pitches of 0.4 to 11 mm, the worst error is 0.93 of it.
__host__ __device__ inline float poly_error(float Huu, float Huv, float Hvv, float gu, float gv,
                                            float Guu, float Guv, float Gvv, float ru, float rv)
{
    const float q = 1.0f - 2.0f * (fabsf(gu) * ru + fabsf(gv) * rv);
    const float iq = q > 0.5f ? 1.0f / q : INFINITY;
    const float l = 7.0f * iq *
                    (fabsf(gu) + fabsf(gv) + Guu * ru + fabsf(Guv) * (ru + rv) + Gvv * rv);
    const float c = 12.25f * iq * (Guu + 2.0f * fabsf(Guv) + Gvv);
    const float rho2 = iq * poly_rho2(Huu, Huv, Hvv);
    return 0.5f * (rho2 + 0.5f) * (l * (l * l + 2.0f * c) + c * c) +
           (rho2 + 0.61f * sqrtf(rho2)) * c * c;
}

// The record's marks: Guu >= +0 is stored negative if the plain series is not enough, Huu' <= -0 is
// stored positive if the folded one is not either.
__device__ __forceinline__ bool mark_fold(const float4 r1) { return signbit(r1.w); }
__device__ __forceinline__ bool mark_direct(const float4 r0) { return !signbit(r0.z); }

// The series of one record about the block centre (cx, cy) in pixel-index coordinates; fold
// (uniform over the wave): with the degree-5 terms. Not live: the series of log2 0, minus infinity
// everywhere, whatever the record's own would be (a record marked direct need not have a finite one).
__device__ __forceinline__ void block_poly(const float4 r0, const float4 r1, const float4 r2,
                                           float cx, float cy, bool fold, bool live, BlockPoly &b)
{
    const float Huu = -fabsf(r0.z), Huv = r0.w, Hvv = r1.x, gu = r1.y, gv = r1.z, Guu = fabsf(r1.w);
    const float Guv = r2.x, Gvv = fabsf(r2.y);
    const float du = cx - r0.x, dv = cy - r0.y;
    b.du = du;
    b.dv = dv;
    const float mE = Huu * du, tE = fmaf(Huv, dv, mE), nE = Hvv * dv;
    const float E00 = fmaf(dv, nE, du * tE), E10 = tE + mE, E01 = fmaf(Huv, du, nE + nE);
    const float tq = fmaf(Guv, dv, fmaf(Guu, du, gu)), nq = fmaf(Gvv, dv, gv);
    const float q00 = fmaf(dv, nq, fmaf(du, tq, 1.0f)), q10 = fmaf(Guu, du, tq);
    const float q01 = fmaf(Guv, du, fmaf(Gvv, dv, nq));
    const float rs = live ? __builtin_amdgcn_rsqf(q00) : 0.0f, iq = rs * rs;
    b.iq = iq;
    b.lrs = __builtin_amdgcn_logf(rs);
    const float p10 = q10 * iq, p01 = q01 * iq, p20 = Guu * iq, p11 = Guv * iq, p02 = Gvv * iq;
    b.p10 = p10; b.p01 = p01; b.p20 = p20; b.p11 = p11; b.p02 = p02;
    const float y00 = E00 * iq;
    const float y10 = fmaf(-p10, y00, E10 * iq), y01 = fmaf(-p01, y00, E01 * iq);
    const float y20 = fmaf(-p10, y10, fmaf(-p20, y00, Huu * iq));
    const float y11 = fmaf(-p10, y01, fmaf(-p01, y10, fmaf(-p11, y00, Huv * iq)));
    const float y02 = fmaf(-p01, y01, fmaf(-p02, y00, Hvv * iq));
    const float y30 = -fmaf(p10, y20, p20 * y10);
    const float y21 = -fmaf(p10, y11, fmaf(p01, y20, fmaf(p20, y01, p11 * y10)));
    const float y12 = -fmaf(p10, y02, fmaf(p01, y11, fmaf(p02, y10, p11 * y01)));
    const float y03 = -fmaf(p01, y02, p02 * y01);
    b.c[pidx(4, 0)] = -fmaf(p10, y30, p20 * y20);
    b.c[pidx(3, 1)] = -fmaf(p10, y21, fmaf(p01, y30, fmaf(p20, y11, p11 * y20)));
    b.c[pidx(2, 2)] = -fmaf(p10, y12, fmaf(p01, y21, fmaf(p20, y02, fmaf(p02, y20, p11 * y11))));
    b.c[pidx(1, 3)] = -fmaf(p10, y03, fmaf(p01, y12, fmaf(p02, y11, p11 * y02)));
    b.c[pidx(0, 4)] = -fmaf(p01, y03, p02 * y02);
    b.c[pidx(3, 0)] = y30; b.c[pidx(2, 1)] = y21; b.c[pidx(1, 2)] = y12; b.c[pidx(0, 3)] = y03;
    // - log2(q) / 2 to second order
    b.c[pidx(0, 0)] = y00 + b.lrs;
    b.c[pidx(1, 0)] = fmaf(-POLY_HL, p10, y10);
    b.c[pidx(0, 1)] = fmaf(-POLY_HL, p01, y01);
    b.c[pidx(2, 0)] = fmaf(-POLY_HL, fmaf(-0.5f * p10, p10, p20), y20);
    b.c[pidx(1, 1)] = fmaf(-POLY_HL, fmaf(-p10, p01, p11), y11);
    b.c[pidx(0, 2)] = fmaf(-POLY_HL, fmaf(-0.5f * p01, p01, p02), y02);
    if (fold) {
        const float y40 = b.c[pidx(4, 0)], y31 = b.c[pidx(3, 1)], y22 = b.c[pidx(2, 2)];
        const float y13 = b.c[pidx(1, 3)], y04 = b.c[pidx(0, 4)];
        const float y50 = -fmaf(p10, y40, p20 * y30);
        const float y41 = -fmaf(p10, y31, fmaf(p01, y40, fmaf(p20, y21, p11 * y30)));
        const float y32 = -fmaf(p10, y22, fmaf(p01, y31, fmaf(p20, y12, fmaf(p02, y30, p11 * y21))));
        const float y23 = -fmaf(p10, y13, fmaf(p01, y22, fmaf(p20, y03, fmaf(p02, y21, p11 * y12))));
        const float y14 = -fmaf(p10, y04, fmaf(p01, y13, fmaf(p02, y12, p11 * y03)));
        const float y05 = -fmaf(p01, y04, p02 * y03);
        // over s = +-1/2, ..., +-7/2: s^5 ~ 15.5 s^3 - 47.3125 s, s^4 ~ 12.5 s^2 - 21.0625 and
        // s^3 t^2 ~ 9.25 s t^2 + 6.375 s^3 - 9.25 6.375 s (minimax fits)
        b.c[pidx(3, 0)] = fmaf(15.5f, y50, fmaf(6.375f, y32, y30));
        b.c[pidx(0, 3)] = fmaf(15.5f, y05, fmaf(6.375f, y23, y03));
        b.c[pidx(2, 1)] = fmaf(12.5f, y41, fmaf(9.25f, y23, y21));
        b.c[pidx(1, 2)] = fmaf(12.5f, y14, fmaf(9.25f, y32, y12));
        b.c[pidx(1, 0)] = fmaf(-47.3125f, y50,
                               fmaf(-21.0625f, y14, fmaf(-58.96875f, y32, b.c[pidx(1, 0)])));
        b.c[pidx(0, 1)] = fmaf(-47.3125f, y05,
                               fmaf(-21.0625f, y41, fmaf(-58.96875f, y23, b.c[pidx(0, 1)])));
        // - log2(q) / 2, third order
        const float a = POLY_HL * p10, d = POLY_HL * p01;
        b.c[pidx(3, 0)] = fmaf(a, fmaf(-p10 * (1.0f / 3.0f), p10, p20), b.c[pidx(3, 0)]);
        b.c[pidx(2, 1)] = fmaf(a, fmaf(-p10, p01, p11), fmaf(d, p20, b.c[pidx(2, 1)]));
        b.c[pidx(1, 2)] = fmaf(d, fmaf(-p10, p01, p11), fmaf(a, p02, b.c[pidx(1, 2)]));
        b.c[pidx(0, 3)] = fmaf(d, fmaf(-p01 * (1.0f / 3.0f), p01, p02), b.c[pidx(0, 3)]);
    }
}

// X on the rows at +t (k[0]) and -t (k[1]) as polynomials in s: k[.][i] the coefficient of s^i
// (s^4 is c[pidx(4, 0)] on every row).
__device__ __forceinline__ void poly_rows(const float (&c)[15], float t, float (&k)[2][4])
{
    const float t2 = t * t;
    const float e0 = fmaf(t2, fmaf(t2, c[pidx(0, 4)], c[pidx(0, 2)]), c[pidx(0, 0)]);
    const float o0 = fmaf(t2, c[pidx(0, 3)], c[pidx(0, 1)]);
    const float e1 = fmaf(t2, c[pidx(1, 2)], c[pidx(1, 0)]);
    const float o1 = fmaf(t2, c[pidx(1, 3)], c[pidx(1, 1)]);
    const float e2 = fmaf(t2, c[pidx(2, 2)], c[pidx(2, 0)]);
    k[0][0] = fmaf(t, o0, e0);
    k[1][0] = fmaf(-t, o0, e0);
    k[0][1] = fmaf(t, o1, e1);
    k[1][1] = fmaf(-t, o1, e1);
    k[0][2] = fmaf(t, c[pidx(2, 1)], e2);
    k[1][2] = fmaf(-t, c[pidx(2, 1)], e2);
    k[0][3] = fmaf(t, c[pidx(3, 1)], c[pidx(3, 0)]);
    k[1][3] = fmaf(-t, c[pidx(3, 1)], c[pidx(3, 0)]);
}

// X at the columns +s (xp) and -s (xm) of a row with coefficients k.
__device__ __forceinline__ void poly_cols(const float (&k)[4], float c40, float s, float &xp,
                                          float &xm)
{
    const float s2 = s * s;
    const float e = fmaf(s2, fmaf(s2, c40, k[2]), k[0]), o = fmaf(s2, k[3], k[1]);
    xp = fmaf(s, o, e);
    xm = fmaf(-s, o, e);
}

// The backward's twelve partial sums from the block-centred moments M_ij = sum w s^i t^j of
// w = g r 2^x (r = q^-1/2, x = E/q): S0 = sum w, and with a = w / q the sums of a and of a x
// against 1, du, dv and their products (see k_splat_bwd). 1/q = iq (1 + r10 s + ...) to second
// order (third and fourth moments of a to the order they have left), x by its series. (Taking the
// fourth moments from the second ones by minimax fits would save 7% of the instructions, but the
// rotations' gradients then lose a digit.)
__device__ __forceinline__ void poly_sums(const BlockPoly &b, const float (&M)[15], float (&S)[12])
{
    const float r10 = -b.p10, r01 = -b.p01, r20 = fmaf(b.p10, b.p10, -b.p20);
    const float r11 = fmaf(2.0f * b.p10, b.p01, -b.p11), r02 = fmaf(b.p01, b.p01, -b.p02);
    // moments of a / iq
    float A[10];
#pragma unroll
    for (int d = 0; d <= 2; ++d)
#pragma unroll
        for (int j = 0; j <= d; ++j) {
            const int i = d - j;
            float v = fmaf(r20, M[pidx(i + 2, j)],
                           fmaf(r11, M[pidx(i + 1, j + 1)], r02 * M[pidx(i, j + 2)]));
            v = fmaf(r10, M[pidx(i + 1, j)], fmaf(r01, M[pidx(i, j + 1)], v));
            A[pidx(i, j)] = M[pidx(i, j)] + v;
        }
#pragma unroll
    for (int j = 0; j <= 3; ++j)
        A[pidx(3 - j, j)] = fmaf(r10, M[pidx(4 - j, j)],
                                 fmaf(r01, M[pidx(3 - j, j + 1)], M[pidx(3 - j, j)]));
    // x = E/q: the exponent without its log2 part
    const float y00 = b.c[0] - b.lrs;
    const float y10 = fmaf(POLY_HL, b.p10, b.c[pidx(1, 0)]);
    const float y01 = fmaf(POLY_HL, b.p01, b.c[pidx(0, 1)]);
    const float y20 = fmaf(POLY_HL, fmaf(-0.5f * b.p10, b.p10, b.p20), b.c[pidx(2, 0)]);
    const float y11 = fmaf(POLY_HL, fmaf(-b.p10, b.p01, b.p11), b.c[pidx(1, 1)]);
    const float y02 = fmaf(POLY_HL, fmaf(-0.5f * b.p01, b.p01, b.p02), b.c[pidx(0, 2)]);
    const float y30 = b.c[pidx(3, 0)], y21 = b.c[pidx(2, 1)], y12 = b.c[pidx(1, 2)];
    const float y03 = b.c[pidx(0, 3)];
    // moments of a x / iq. quad(i, j): the part of x up to second order against s^i t^j
    auto mom = [&](int i, int j) { return i + j <= 3 ? A[pidx(i, j)] : M[pidx(i, j)]; };
    auto quad = [&](int i, int j, float v) {
        v = fmaf(y02, mom(i, j + 2), v);
        v = fmaf(y11, mom(i + 1, j + 1), v);
        v = fmaf(y20, mom(i + 2, j), v);
        v = fmaf(y01, mom(i, j + 1), v);
        v = fmaf(y10, mom(i + 1, j), v);
        return fmaf(y00, mom(i, j), v);
    };
    auto cubic = [&](int i, int j) {
        return fmaf(y30, mom(i + 3, j),
                    fmaf(y21, mom(i + 2, j + 1), fmaf(y12, mom(i + 1, j + 2), y03 * mom(i, j + 3))));
    };
    const float X00 = quad(0, 0, cubic(0, 0));
    const float X10 = quad(1, 0, cubic(1, 0)), X01 = quad(0, 1, cubic(0, 1));
    const float X20 = quad(2, 0, 0.0f), X11 = quad(1, 1, 0.0f), X02 = quad(0, 2, 0.0f);
    // about the footprint's centre (du = s + b.du, dv = t + b.dv)
    const float du = b.du, dv = b.dv, iq = b.iq;
    const float A00 = A[0], A10 = A[pidx(1, 0)], A01 = A[pidx(0, 1)];
    S[0] = M[0];
    S[1] = iq * fmaf(du, fmaf(du, A00, 2.0f * A10), A[pidx(2, 0)]);
    S[2] = iq * fmaf(du, fmaf(dv, A00, A01), fmaf(dv, A10, A[pidx(1, 1)]));
    S[3] = iq * fmaf(dv, fmaf(dv, A00, 2.0f * A01), A[pidx(0, 2)]);
    S[4] = iq * fmaf(du, fmaf(du, X00, 2.0f * X10), X20);
    S[5] = iq * fmaf(du, fmaf(dv, X00, X01), fmaf(dv, X10, X11));
    S[6] = iq * fmaf(dv, fmaf(dv, X00, 2.0f * X01), X02);
    S[7] = iq * fmaf(du, X00, X10);
    S[8] = iq * fmaf(dv, X00, X01);
    S[9] = iq * fmaf(2.0f * 0.69314718055994531f, X00, A00);
    S[10] = iq * fmaf(du, A00, A10);
    S[11] = iq * fmaf(dv, A00, A01);
}
