// Adjoint of the per-hit thin-film solve (reverse sweep with segment
// recomputation).  See gwg_device.h for the formulation.  Always double
// precision: the covector and the recomputed vectors carry the full
// conditioning of the stack.
#pragma once
#include "gwg_device.h"

namespace gwg {

struct V2d { double br, bi, cr, ci; };

__device__ inline void step_real_d(V2d& v, double C, double X, double Y)
{
    double br = fma(C, v.br, X * v.ci);
    double bi = fma(C, v.bi, -(X * v.cr));
    double cr = fma(C, v.cr, Y * v.bi);
    double ci = fma(C, v.ci, -(Y * v.br));
    v.br = br; v.bi = bi; v.cr = cr; v.ci = ci;
}

__device__ inline void step_cplx_d(V2d& v, cd C, cd X, cd Y)
{
    cd B = mk(v.br, v.bi), Cv = mk(v.cr, v.ci);
    cd mX = mk(X.im, -X.re), mY = mk(Y.im, -Y.re);
    cd b = cadd(cmul(C, B), cmul(mX, Cv));
    cd c = cadd(cmul(mY, B), cmul(C, Cv));
    v.br = b.re; v.bi = b.im; v.cr = c.re; v.ci = c.im;
}

// Entries of one layer for both polarizations.  Lossless: C real, X/Y real
// (imaginary parts zero).  Absorbing: complex.
struct LayerEnt { cd C, Xs, Ys, Xp, Yp; bool real; };

__device__ inline LayerEnt layer_entries(const LaneSlots3& sl, int s, bool cplx, double k0, double t)
{
    LayerEnt e;
    e.real = !cplx;
    if (!cplx) {
        double kq, xs, ys, xp, yp, C, S;
        sl.lossless(s, kq, xs, ys, xp, yp);
        layer_cs(kq, t, &C, &S);
        e.C = mk(C, 0.0);
        e.Xs = mk(S * xs, 0.0); e.Ys = mk(S * ys, 0.0);
        e.Xp = mk(S * xp, 0.0); e.Yp = mk(S * yp, 0.0);
    } else {
        double Pl[4];
        sl.absorbing(s, Pl);
        CTv<double> C, Xs, Ys, Xp, Yp;
        layer_cplx(Pl, k0, t, &C, &Xs, &Ys, &Xp, &Yp);
        e.C = mk(C.re, C.im); e.Xs = mk(Xs.re, Xs.im); e.Ys = mk(Ys.re, Ys.im);
        e.Xp = mk(Xp.re, Xp.im); e.Yp = mk(Yp.re, Yp.im);
    }
    return e;
}

__device__ inline void apply_layer(V2d& vs, V2d& vp, const LayerEnt& e)
{
    if (e.real) {
        step_real_d(vs, e.C.re, e.Xs.re, e.Ys.re);
        step_real_d(vp, e.C.re, e.Xp.re, e.Yp.re);
    } else {
        step_cplx_d(vs, e.C, e.Xs, e.Ys);
        step_cplx_d(vp, e.C, e.Xp, e.Yp);
    }
}

// u^T <- u^T M for M = [[C, -iX], [-iY, C]]:  u1' = u1 C - i u2 Y,  u2' = -i u1 X + u2 C
__device__ inline void cov_step(cd& u1, cd& u2, cd C, cd X, cd Y)
{
    cd mY = mk(Y.im, -Y.re), mX = mk(X.im, -X.re);
    cd n1 = cadd(cmul(u1, C), cmul(u2, mY));
    cd n2 = cadd(cmul(u1, mX), cmul(u2, C));
    u1 = n1; u2 = n2;
}

// u^T <- u^T M for a lossless layer, M = [[C, -iX], [-iY, C]] with real C, X, Y.
__device__ inline void cov_step_real(cd& u1, cd& u2, double C, double X, double Y)
{
    const double a = fma(u1.re, C, Y * u2.im), b = fma(u1.im, C, -(Y * u2.re));
    const double c = fma(u2.re, C, X * u1.im), d = fma(u2.im, C, -(X * u1.re));
    u1 = mk(a, b);
    u2 = mk(c, d);
}

// Adjoint of one mirror hit.  Adds d(2 Re(Gs c_s + Gp c_p))/dt_j for every
// layer into grad_row (this mirror's row of the calling wave's LDS
// accumulator, stack order), where c = r (reflect) or t (transmit).
// sl: this lane's slot table (N^2 of slot s: sl.nsq[2 s], sl.nsq[2 s + 1]).
// chk: this lane's checkpoint storage, component k of checkpoint c at
// chk[(c * 8 + k) * cstride].
__device__ inline void tmm_adjoint(const double* __restrict__ thk, const uint8_t* __restrict__ slot,
                                   int L, bool front, const LaneSlots3& sl, uint32_t cplx_mask, double k0,
                                   double kappa2, double eta0s, double eta0p, bool reflect, cd Gs, cd Gp,
                                   double* grad_row, double* __restrict__ chk, int64_t cstride)
{
    const double* nsq_c = sl.nsq;
    // 1) exit -> incident sweep, checkpoints w_{kSeg}, w_{2 kSeg}, ...
    V2d vs = { 1.0, 0.0, eta0s, 0.0 };
    V2d vp = { 1.0, 0.0, eta0p, 0.0 };
    for (int jj = L - 1; jj >= 0; --jj) {
        int idx = front ? jj : (L - 1 - jj);
        double t = thk[idx];
        if (t != 0.0) {
            int s = slot[idx];
            LayerEnt e = layer_entries(sl, s, (cplx_mask >> s) & 1u, k0, t);
            apply_layer(vs, vp, e);
        }
        if (jj > 0 && (jj % kSeg) == 0) {
            double* c = chk + (int64_t)(jj / kSeg) * 8 * cstride;
            c[0] = vs.br; c[cstride] = vs.bi; c[2 * cstride] = vs.cr; c[3 * cstride] = vs.ci;
            c[4 * cstride] = vp.br; c[5 * cstride] = vp.bi; c[6 * cstride] = vp.cr; c[7 * cstride] = vp.ci;
        }
    }
    // 2) cotangent row of the taken coefficient w.r.t. [B; C]
    cd u1s, u2s, u1p, u2p;
    {
        cd B = mk(vs.br, vs.bi), C = mk(vs.cr, vs.ci);
        cd den = cadd(cscale(B, eta0s), C);
        cd inv2 = cdiv(mk(1.0, 0.0), cmul(den, den));
        cd dB, dC;
        if (reflect) { dB = cscale(cmul(C, inv2), 2.0 * eta0s); dC = cscale(cmul(B, inv2), -2.0 * eta0s); }
        else { dB = cscale(inv2, -2.0 * eta0s * eta0s); dC = cscale(inv2, -2.0 * eta0s); }
        u1s = cmul(Gs, dB); u2s = cmul(Gs, dC);
    }
    {
        cd B = mk(vp.br, vp.bi), C = mk(vp.cr, vp.ci);
        cd den = cadd(cscale(B, eta0p), C);
        cd inv2 = cdiv(mk(1.0, 0.0), cmul(den, den));
        cd dB, dC;
        if (reflect) {   // r_p = -r_Mac
            dB = cscale(cmul(C, inv2), -2.0 * eta0p); dC = cscale(cmul(B, inv2), 2.0 * eta0p);
        } else { dB = cscale(inv2, -2.0 * eta0p * eta0p); dC = cscale(inv2, -2.0 * eta0p); }
        u1p = cmul(Gp, dB); u2p = cmul(Gp, dC);
    }
    // 3) incident -> exit covector sweep, segment by segment
    const int nseg = (L + kSeg - 1) / kSeg;
    for (int k = 0; k < nseg; ++k) {
        const int lo = k * kSeg;
        const int hi = min(lo + kSeg, L);
        V2d ws, wp;
        if (hi == L) {
            ws = V2d{ 1.0, 0.0, eta0s, 0.0 };
            wp = V2d{ 1.0, 0.0, eta0p, 0.0 };
        } else {
            const double* c = chk + (int64_t)(hi / kSeg) * 8 * cstride;
            ws = V2d{ c[0], c[cstride], c[2 * cstride], c[3 * cstride] };
            wp = V2d{ c[4 * cstride], c[5 * cstride], c[6 * cstride], c[7 * cstride] };
        }
        V2d segs[kSeg], segp[kSeg];
        double segC[kSeg], segS[kSeg];
#pragma unroll
        for (int i = kSeg - 1; i >= 0; --i) {
            const int jj = lo + i;
            segC[i] = 1.0; segS[i] = 0.0;
            if (jj < hi) {
                int idx = front ? jj : (L - 1 - jj);
                double t = thk[idx];
                int s = slot[idx];
                if (t != 0.0) {
                    if (!((cplx_mask >> s) & 1u)) {
                        double kq, xs, ys, xp, yp, C, S;
                        sl.lossless(s, kq, xs, ys, xp, yp);
                        layer_cs(kq, t, &C, &S);
                        segC[i] = C; segS[i] = S;
                        step_real_d(ws, C, S * xs, S * ys);
                        step_real_d(wp, C, S * xp, S * yp);
                    } else {
                        LayerEnt e = layer_entries(sl, s, true, k0, t);
                        apply_layer(ws, wp, e);
                    }
                }
                segs[i] = ws; segp[i] = wp;
            }
        }
#pragma unroll
        for (int i = 0; i < kSeg; ++i) {
            const int jj = lo + i;
            if (jj < hi) {
                int idx = front ? jj : (L - 1 - jj);
                double t = thk[idx];
                int s = slot[idx];
                bool cplx = (cplx_mask >> s) & 1u;
                // contraction u^T D w (D = -i k0 [[0, a], [b, 0]])
                cd Bs = mk(segs[i].br, segs[i].bi), Cs = mk(segs[i].cr, segs[i].ci);
                cd Bp = mk(segp[i].br, segp[i].bi), Cp = mk(segp[i].cr, segp[i].ci);
                cd As, Ap;
                if (!cplx) {
                    double n2 = nsq_c[2 * s];
                    double z = n2 - kappa2;
                    As = cadd(cmul(u1s, Cs), cscale(cmul(u2s, Bs), z));
                    Ap = cadd(cscale(cmul(u1p, Cp), z / n2), cscale(cmul(u2p, Bp), n2));
                } else {
                    cd N2 = mk(nsq_c[2 * s], nsq_c[2 * s + 1]);
                    cd z = csub(N2, mk(kappa2, 0.0));
                    As = cadd(cmul(u1s, Cs), cmul(z, cmul(u2s, Bs)));
                    Ap = cadd(cmul(cdiv(z, N2), cmul(u1p, Cp)), cmul(N2, cmul(u2p, Bp)));
                }
                // Re(-i k0 A) = k0 Im(A); dw/dt = 2 Re(...)
                double g = 2.0 * k0 * (As.im + Ap.im);
                atomicAdd(&grad_row[idx], g);
                // covector through layer jj
                if (t != 0.0) {
                    if (!cplx) {
                        double kq, xs, ys, xp, yp;
                        sl.lossless(s, kq, xs, ys, xp, yp);
                        const double C = segC[i], S = segS[i];
                        cov_step_real(u1s, u2s, C, S * xs, S * ys);
                        cov_step_real(u1p, u2p, C, S * xp, S * yp);
                    } else {
                        LayerEnt e = layer_entries(sl, s, true, k0, t);
                        cov_step(u1s, u2s, e.C, e.Xs, e.Ys);
                        cov_step(u1p, u2p, e.C, e.Xp, e.Yp);
                    }
                }
            }
        }
    }
}

// Adjoint of one mirror hit whose stack has no absorbing layer (every layer
// matrix has real C, X, Y).  Same contract as tmm_adjoint.  HC = false: no
// lane of the calling wave has an evanescent slot.  The slot parameters
// (x_s, y_s, x_p, y_p) are (1/q, q, q/N^2, N^2/q) for a propagating layer or
// (1/Q, -Q, -Q/N^2, N^2/Q) for an evanescent one (q = iQ), with sg = +1 or -1
// respectively:
//     z = sg y_s^2,  z / N^2 = sg y_s x_p,  N^2 = sg y_s y_p.
//
// With C = i c a layer is the real matrix R = [[C, X], [-Y, C]] on (B, c), and
// with u2' = i u2 the covector takes the same real matrix.  A layer's gradient
// needs the state w and the covector u only as two entries of Q = Re(w u^T),
//     Im(u1 C) = Q21,  Im(u2 B) = -Q12,
// and from the layer's exit side to its incident side Q goes to R Q R^-1,
// which leaves the trace alone.  So three reals a polarization pass the
// layers: with A = Q11 - Q22, b = Q12, c = Q21 and m = C A + Y b + X c,
//     b -= X m,  c -= Y m,  A = 2 C m - A
// (from C^2 + X Y = 1, circular or hyperbolic): 8 operations where walking w
// and u took 32, and no sign of C, X, Y to keep.
//     1) segment matrices S_g of K layers, from a sweep;
//     2) w_g = S_g w_{g+1} from the exit medium up, kept in scratch; the
//        cotangent rows u_0 of the taken coefficients from w_0;
//     3) down the segments: u_{g+1}, Q at the segment's exit side from it and
//        w_{g+1}, then the segment's layers upwards.
// Going up a segment a reflected hit's Q grows as the rounding it carries, and
// a transmitted one's, of constant size, gathers at most the square of the
// segment's transfer growth (as a walk of w against u would).  A reflected
// hit's covector is c (C, -B) of the state at every depth (a ratio of B and C
// is differentiated, and the layers are unimodular), which is exact where a
// covector walked down a reflection band loses itself in rounding; a
// transmitted one's grows downwards and is walked by S_g.
// Scratch of the lane: field f of block k at scr + (8 k + f) ss; blocks 0 ..
// nblk - 1: w_g, nblk .. 2 nblk - 1: S_g.
struct SegPair { SegMat s, p; };

// One polarization's covector on its way down: u of a transmitted hit, the
// factor c (in u1) of a reflected one.
struct CovRow { cd u1, u2; };

__device__ inline CovRow cov_top(const V2d& v, double eta0, bool reflect, bool p_pol, cd G)
{
    const cd den = mk(fma(v.br, eta0, v.cr), fma(v.bi, eta0, v.ci));
    const cd h = cmul(G, cdiv(mk(1.0, 0.0), cmul(den, den)));
    const double e2 = 2.0 * eta0;
    return { cscale(h, reflect ? (p_pol ? -e2 : e2) : -(e2 * eta0)), cscale(h, -e2) };
}

// Q of a covector and a state.
__device__ inline void cov_q(cd u1, cd u2, const V2d& w, double& A, double& b, double& c)
{
    A = fma(w.br, u1.re, -(w.bi * u1.im)) - fma(w.cr, u2.re, -(w.ci * u2.im));
    b = -fma(w.br, u2.im, w.bi * u2.re);
    c = fma(w.cr, u1.im, w.ci * u1.re);
}
// Square root of z (either one), also where |z|^2 leaves the range of a double.
__device__ inline cd csqrt_any(cd z)
{
    int e;
    (void)frexp(fmax(fabs(z.re), fabs(z.im)), &e);
    e &= ~1;
    const cd r = csqrt_up(mk(ldexp(z.re, -e), ldexp(z.im, -e)));
    return mk(ldexp(r.re, e / 2), ldexp(r.im, e / 2));
}
// f times a state.
__device__ inline V2d state_scale(cd f, const V2d& w)
{
    return { fma(f.re, w.br, -(f.im * w.bi)), fma(f.re, w.bi, f.im * w.br), fma(f.re, w.cr, -(f.im * w.ci)),
             fma(f.re, w.ci, f.im * w.cr) };
}
// Q of a reflected hit (covector factor c in u1) at state w.
__device__ inline void cov_refl(const CovRow& r, const V2d& w, double& A, double& b, double& c)
{
    cov_q(mk(fma(r.u1.re, w.cr, -(r.u1.im * w.ci)), fma(r.u1.re, w.ci, r.u1.im * w.cr)),
          mk(fma(r.u1.im, w.bi, -(r.u1.re * w.br)), -fma(r.u1.re, w.bi, r.u1.im * w.br)), w, A, b, c);
}
// A transmitted hit's covector past a segment: u^T S on (u1, i u2).
__device__ inline void cov_step(CovRow& r, const SegMat& m)
{
    const cd u1 = mk(fma(m.m11, r.u1.re, -(m.m21 * r.u2.im)), fma(m.m11, r.u1.im, m.m21 * r.u2.re));
    r.u2 = mk(fma(m.m12, r.u1.im, m.m22 * r.u2.re), fma(m.m22, r.u2.im, -(m.m12 * r.u1.re)));
    r.u1 = u1;
}

template <bool HC = true>
__device__ inline void tmm_adjoint_lossless(const double* __restrict__ thk, const uint8_t* __restrict__ slot,
                                            int L, bool front, const LaneSlots3& sl, double k0,
                                            double eta0s, double eta0p, bool reflect, cd Gs, cd Gp,
                                            double* grad_row, double* __restrict__ scr, int64_t ss, int nblk)
{
    if (L <= 0) return;
    constexpr int K = kSegUp;
    const int G = (L - 1) / K + 1;
    auto put = [&](int k, double a, double b, double c, double d, double e, double f, double g, double h) {
        double* o = scr + (int64_t)k * 8 * ss;
        o[0] = a; o[ss] = b; o[2 * ss] = c; o[3 * ss] = d;
        o[4 * ss] = e; o[5 * ss] = f; o[6 * ss] = g; o[7 * ss] = h;
    };
    auto get_seg = [&](int g) {
        SegPair m;
        const double* p = scr + (int64_t)(nblk + g) * 8 * ss;
        m.s = { p[0], p[ss], p[2 * ss], p[3 * ss] };
        m.p = { p[4 * ss], p[5 * ss], p[6 * ss], p[7 * ss] };
        return m;
    };
    // 1), 2)
    V2d ws = { 1.0, 0.0, eta0s, 0.0 }, wp = { 1.0, 0.0, eta0p, 0.0 };
    auto up = [&](int g, const SegPair& m) {
        seg_apply(m.s, ws.br, ws.bi, ws.cr, ws.ci);
        seg_apply(m.p, wp.br, wp.bi, wp.cr, wp.ci);
        if (g > 0) put(g, ws.br, ws.bi, ws.cr, ws.ci, wp.br, wp.bi, wp.cr, wp.ci);
    };
    for (int g = G - 1; g >= 0; --g) {
        V2d vs = { 1.0, 0.0, -1.0, 0.0 }, vp = { 1.0, 0.0, -1.0, 0.0 };
        double nsum = 0.0;
        auto layer = [&](int jj) {
            const int idx = front ? jj : (L - 1 - jj);
            double kq, xs, ys, xp, yp, C, S;
            sl.lossless(slot[idx], kq, xs, ys, xp, yp);
            layer_cs_half<double, HC>(kq, thk[idx], &C, &S, &nsum);   // t = 0 gives the identity exactly
            step_real_d(vs, C, S * xs, S * ys);
            step_real_d(vp, C, S * xp, S * yp);
        };
        const int lo = g * K, hi = min(lo + K, L);
#pragma unroll 2
        for (int j = hi - 1; j >= lo; --j) layer(j);
        // the half-period sines and cosines leave out (-1)^n of each layer
        const uint32_t sb = (uint32_t)((int)nsum & 1) << 31;
        const SegPair m = { { flip_sign(vs.br, sb), flip_sign(vs.bi, sb), flip_sign(vs.ci, sb), flip_sign(-vs.cr, sb) },
                            { flip_sign(vp.br, sb), flip_sign(vp.bi, sb), flip_sign(vp.ci, sb), flip_sign(-vp.cr, sb) } };
        put(nblk + g, m.s.m11, m.s.m12, m.s.m21, m.s.m22, m.p.m11, m.p.m12, m.p.m21, m.p.m22);
        up(g, m);
    }
    // covectors of the taken coefficients, with the gradient's factor 2 k0
    const double k2 = 2.0 * k0;
    CovRow us = cov_top(ws, eta0s, reflect, false, cscale(Gs, k2));
    CovRow up_ = cov_top(wp, eta0p, reflect, true, cscale(Gp, k2));
    // 3) the next segment's state and matrix are in flight while a segment runs
    V2d nws, nwp;
    SegPair nm;
    auto fetch = [&](int g) {
        nm = get_seg(g);
        if (g + 1 < G) {
            const double* c = scr + (int64_t)(g + 1) * 8 * ss;
            nws = V2d{ c[0], c[ss], c[2 * ss], c[3 * ss] };
            nwp = V2d{ c[4 * ss], c[5 * ss], c[6 * ss], c[7 * ss] };
        } else {
            nws = V2d{ 1.0, 0.0, eta0s, 0.0 };
            nwp = V2d{ 1.0, 0.0, eta0p, 0.0 };
        }
    };
    fetch(0);
    using LT = LayerTrig<double, HC>;
    const int step = front ? -1 : 1;
    for (int g = 0; g < G; ++g) {
        const int lo = g * K, hi = lo + K < L ? lo + K : L;
        // Software pipeline over the segment's layers, as in the forward
        // sweep: the next layer's argument is reduced from slot parameters
        // read one iteration earlier, the parameters and thickness of the one
        // after are read, and the slot index of the third.  Indices past the
        // segment's last layer stay there.
        const int last = front ? lo : L - 1 - lo;
        auto nxt = [&](int i) { return i == last ? i : i + step; };
        int idx = front ? hi - 1 : L - hi;
        double kq, xs, ys, xp, yp;
        sl.lossless(slot[idx], kq, xs, ys, xp, yp);
        const double t0 = thk[idx];
        int idn = nxt(idx);
        double kq1, xs1, ys1, xp1, yp1;
        sl.lossless(slot[idn], kq1, xs1, ys1, xp1, yp1);
        double t1 = thk[idn];
        int idn2 = nxt(idn);
        int s2 = slot[idn2];
        double As, bs, cs, Ap, bp, cp;
        if (reflect) {
            cov_refl(us, nws, As, bs, cs);
            cov_refl(up_, nwp, Ap, bp, cp);
        } else {
            cov_step(us, nm.s);
            cov_step(up_, nm.p);
            cov_q(us.u1, us.u2, nws, As, bs, cs);
            cov_q(up_.u1, up_.u2, nwp, Ap, bp, cp);
        }
        if (g + 1 < G) fetch(g + 1);
        TrigArg ta = LT::reduce(kq, t0);                    // t = 0 gives the identity exactly
        double n_unused = 0.0;
#pragma unroll 4
        for (int j = hi - 1; j >= lo; --j) {
            const int idn3 = nxt(idn2);
            double kq2, xs2, ys2, xp2, yp2;
            sl.lossless(s2, kq2, xs2, ys2, xp2, yp2);
            const double t2 = thk[idn2];
            s2 = slot[idn3];
            const TrigArg ta1 = LT::reduce(kq1, t1);        // the next layer's (the last layer's again at the end)
            double C, S;
            LT::eval(ta, &C, &S, &n_unused);
            const double sXs = S * xs, sYs = S * ys, sXp = S * xp, sYp = S * yp;
            const double gys = (HC && kq < 0.0) ? -ys : ys;       // sg y_s (an evanescent layer: sg = -1)
            // Im(u^T D w) summed over s and p, D = -i k0 [[0, a], [b, 0]]
            // (fused multiply-adds written out: the library builds without
            // contraction)
            atomicAdd(&grad_row[idx], fma(gys, fma(-yp, bp, fma(xp, cp, -(ys * bs))), cs));
            const double ms = fma(C, As, fma(sXs, cs, sYs * bs)), mp = fma(C, Ap, fma(sXp, cp, sYp * bp));
            const double C2 = C + C;
            bs = fma(-sXs, ms, bs); cs = fma(-sYs, ms, cs); As = fma(C2, ms, -As);
            bp = fma(-sXp, mp, bp); cp = fma(-sYp, mp, cp); Ap = fma(C2, mp, -Ap);
            idx = idn; ta = ta1; kq = kq1; xs = xs1; ys = ys1; xp = xp1; yp = yp1;
            idn = idn2; kq1 = kq2; xs1 = xs2; ys1 = ys2; xp1 = xp2; yp1 = yp2; t1 = t2;
            idn2 = idn3;
        }
    }
}

}  // namespace gwg
