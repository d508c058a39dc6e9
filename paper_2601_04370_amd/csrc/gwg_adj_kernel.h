// Thin-film adjoint of stored entries, sorted by mirror.
// Included by gwg_kernels.hip inside namespace gwg.
//
// A wave whose 64 entries meet one mirror from one side walks one stack in
// one direction: the layer record is one broadcast read, every lane is at the
// same layer, and the lanes' gradients of a layer can be summed before they
// reach LDS memory.  Entries in item order mix all mirrors and sides: each
// layer's thickness and slot were reads from up to 2 M rows, its gradients 64
// conflicting LDS additions, and LDS the limit (active 70 % of the time with
// a third of it bank conflicts), with room for one wave per SIMD.
//
// 1323 points x 8192 rays, 6 mirrors x 200 layers, 3.3e7 entries: entries in
// item order with w and u walked 22.4 ms; Q walked (gwg_adjoint.h) 20.3 ms,
// LDS-bound; sorted 16.4 ms (15.6 with every hit's Q walked) and 0.9 ms for the
// sort.  Bound now by vector issue (83 %; 47 instructions per layer, 44 of them
// double precision, 54 of a reflected hit, and 10
// for segment ends, sums and partly filled batches) at the clock that the
// power limit leaves it (2.0 GHz).
//
// k_entry_sort orders the entries of a group (items of one design and
// wavelength) by class = mirror, side, evanescent, reflected; k_adj_sorted
// takes units of a (group, mirror): equal shares of its batches of 64 entries
// of one class.  Both keep item order within a class, so the sums run in a
// fixed order.

constexpr int kMirClasses = 8;                          // front, evanescent, reflected
constexpr int kClasses = kMirClasses * kMaxMirrors;
constexpr int kSortWaves = 4;
constexpr int kUnitParts = 8;                           // units per (group, mirror)

struct SortDev {
    int32_t ng;                  // items per group
    int32_t groups_dl;           // groups per (design, wavelength)
    int64_t groups;
    uint32_t* order;             // entries of a group by class, relative to its first region
    int32_t* start;              // [groups][kClasses + 1] first entry of each class in order
};

// Items [a, b) of a group.
__device__ inline void group_items(const SceneDev& sc, const SortDev& so, int64_t group, int64_t* a, int64_t* b)
{
    const int64_t items_dl = (int64_t)sc.F * sc.tiles_per_point;
    const int64_t dl = group / so.groups_dl, k = group - dl * so.groups_dl;
    *a = dl * items_dl + k * so.ng;
    *b = min(*a + so.ng, (dl + 1) * items_dl);
}

__global__ void __launch_bounds__(64 * kSortWaves) k_entry_sort(SceneDev sc, const double* __restrict__ dLdI, AdjStore st,
                                                               SortDev so)
{
    __shared__ int s_at[kSortWaves][kClasses];           // counts, then the wave's next place of each class
    const int tid = threadIdx.x, lane = wave_lane(), wave = tid / 64;
    const int B = sc.bins_x * sc.bins_y;
    int64_t ia, ib;
    group_items(sc, so, blockIdx.x, &ia, &ib);
    const int64_t dl = blockIdx.x / so.groups_dl;
    const double* lt = sc.lam_tab + dl % sc.n_lsel * LT_STRIDE;
    double k2e = 1e300;                                  // smallest N^2 of a lossless slot
    for (int s = 0; s < sc.n_slots; ++s)
        if (!((sc.slot_complex >> s) & 1u)) k2e = fmin(k2e, lt[LT_SLOT + 2 * s] * lt[LT_SLOT + 2 * s]);
    for (int k = tid; k < kSortWaves * kClasses; k += 64 * kSortWaves) ((int*)s_at)[k] = 0;
    __syncthreads();
    // each wave: a contiguous share of the group's regions, 64 entries at a time
    const int64_t r_all = (ib - ia) * st.waves, r0 = ia * st.waves;
    const int64_t ra = r_all * wave / kSortWaves, rb = r_all * (wave + 1) / kSortWaves;
    auto scan = [&](auto use) {
        for (int64_t r = ra; r < rb; ++r) {
            const int64_t item = (r0 + r) / st.waves;
            if (st.ovf[item] != 0) continue;
            const int n = st.cnt[r0 + r];
            const double* g_bins = dLdI + item / sc.tiles_per_point * B;
            const double* ent = st.ent + (r0 + r) * st.cap_w * kEntFields;
            // kDeep chunks' entries, then their bins' gradients, in flight at once
            constexpr int kDeep = 4;
            for (int c = 0; c < n; c += 64 * kDeep) {
                double kap[kDeep], g[kDeep];
                int64_t meta[kDeep];
#pragma unroll
                for (int u = 0; u < kDeep; ++u) {
                    const double* e = ent + (int64_t)min(c + 64 * u + lane, n - 1) * kEntFields;
                    kap[u] = e[0];
                    meta[u] = (int64_t)e[5];
                }
#pragma unroll
                for (int u = 0; u < kDeep; ++u) g[u] = g_bins[ent_bin(meta[u])];
#pragma unroll
                for (int u = 0; u < kDeep; ++u) {
                    const int k = c + 64 * u + lane;
                    int cls = -1;
                    if (k < n && g[u] / (double)sc.N != 0.0) {
                        // slot_params takes z = N^2 - kappa^2 of at least kTinyZ in size
                        const bool evan = k2e - kap[u] * kap[u] <= -kTinyZ;
                        cls = (int)(meta[u] & 255) * kMirClasses + (int)((meta[u] >> 8) & 1) * 4 + (evan ? 2 : 0) +
                              (int)((meta[u] >> 9) & 1);
                    }
                    if (c + 64 * u < n) use(cls, (uint32_t)(r * st.cap_w + k));
                }
            }
        }
    };
    scan([&](int cls, uint32_t) { if (cls >= 0) atomicAdd(&s_at[wave][cls], 1); });
    __syncthreads();
    if (wave == 0) {
        // two classes a lane: totals, their exclusive sum, each wave's first place
        int tot[2], sum = 0;
        for (int q = 0; q < 2; ++q) {
            tot[q] = 0;
            for (int w = 0; w < kSortWaves; ++w) tot[q] += s_at[w][2 * lane + q];
            sum += tot[q];
        }
        int all;
        int at = wave_excl_scan(sum, &all);
        int32_t* start = so.start + (int64_t)blockIdx.x * (kClasses + 1);
        for (int q = 0; q < 2; ++q) {
            const int k = 2 * lane + q;
            start[k] = at;
            for (int w = 0; w < kSortWaves; ++w) {
                const int n = s_at[w][k];
                s_at[w][k] = at;
                at += n;
            }
        }
        if (lane == 63) start[kClasses] = all;
    }
    __syncthreads();
    uint32_t* order = so.order + r0 * st.cap_w;
    scan([&](int cls, uint32_t rel) {
        unsigned long long peers = __ballot(cls >= 0);
        for (int b = 0; b < 7; ++b) {
            const bool one = (cls >> b & 1) != 0;
            const unsigned long long ones = __ballot(one);
            peers &= one ? ones : ~ones;
        }
        if (cls >= 0) {
            const int rank = __popcll(peers & ((1ull << lane) - 1ull));
            order[s_at[wave][cls] + rank] = rel;
            wave_lds_sync();
            if (rank == 0) s_at[wave][cls] += __popcll(peers);
        }
        wave_lds_sync();
    });
}
static_assert(kClasses == 128, "two classes per lane, seven bits");

// ------------------------------------------------- adjoint of one class
// Lanes' layer gradients staged in LDS, [kStageRows][kStageLanes]: eight lanes
// sum a row of 64 values, 16 bytes at a time, adjacent lanes adjacent words;
// the row stride puts the two rows of 16 lanes in different banks.
constexpr int kStageRows = 8, kStageLanes = 80;

// x of the lane that a DPP control selects (within rows of 16 lanes).
template <int CTRL>
__device__ inline double dpp_move(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// Sum over the eight lanes 8 k .. 8 k + 7, the same in all of them.
__device__ inline double sum8(double x)
{
    x += dpp_move<0xb1>(x);                              // quad_perm 1 0 3 2
    x += dpp_move<0x4e>(x);                              // quad_perm 2 3 0 1
    x += dpp_move<0x141>(x);                             // row_half_mirror
    return x;
}

// What a walk carries through the layers.  Both give a layer's gradient from
// b = Q12 and c = Q21 at one of its sides and pass the layer: X = S x, Y = S y.
__device__ inline double layer_gradient(double gys, double ys, double xp, double yp, double bs, double cs, double bp, double cp)
{
    return fma(gys, fma(-yp, bp, fma(xp, cp, -(ys * bs))), cs);
}
// Three reals a polarization of Q (A = Q11 - Q22).
struct CarryQ {
    double As, bs, cs, Ap, bp, cp;
    __device__ double gradient(double gys, double ys, double xp, double yp) const
    {
        return layer_gradient(gys, ys, xp, yp, bs, cs, bp, cp);
    }
    __device__ void pass(double C, double Xs, double Ys, double Xp, double Yp)
    {
        const double ms = fma(C, As, fma(Xs, cs, Ys * bs)), mp = fma(C, Ap, fma(Xp, cp, Yp * bp));
        const double C2 = C + C;
        bs = fma(-Xs, ms, bs); cs = fma(-Ys, ms, cs); As = fma(C2, ms, -As);
        bp = fma(-Xp, mp, bp); cp = fma(-Yp, mp, cp); Ap = fma(C2, mp, -Ap);
    }
};
// A reflected hit's state times the root of twice its covector's factor c:
// Q12 = Im(c B^2) and Q21 = Im(c C^2) are products of its parts.  (Its own Q
// would do with fewer operations, but is of second order in the state: where
// the state shrinks on its way up, at a resonance of the stack, Q keeps the
// rounding of the square of what it was: cavities of 20 pairs a side, 1 pm off
// resonance, 4e-7 of the gradient where the state keeps 1e-10; 200 layers of
// random thickness, the worst of 2000: 2e-9 and 4e-11.)
struct CarryW {
    V2d s, p;
    __device__ double gradient(double gys, double ys, double xp, double yp) const
    {
        return layer_gradient(gys, ys, xp, yp, s.br * s.bi, s.cr * s.ci, p.br * p.bi, p.cr * p.ci);
    }
    __device__ void pass(double C, double Xs, double Ys, double Xp, double Yp)
    {
        step_real_d(s, C, Xs, Ys);
        step_real_d(p, C, Xp, Yp);
    }
};

// A carrier at one side of a layer, taken through n layers: up from the exit
// side of incidence-order layer j0, or (not up) down from its incident side (the
// inverse layers: S -> -S).  The layers' gradients are added to gw.
template <bool HC, class SL, class Carry>
__device__ __attribute__((always_inline)) inline void class_walk(const LayerRec* rec, int L, bool front, const SL& sl, Carry v,
                                                                 int j0, int n, bool up, double* stage, double* gw)
{
    using LT = LayerTrig<double, HC>;
    const int lane = wave_lane();
    double n_unused = 0.0;
    const uint32_t sflip = up ? 0u : 1u << 31;
    const int i0 = front ? j0 : L - 1 - j0;              // in the mirror's layer order
    const int dir = front != up ? 1 : -1;
    // as in the forward sweep: the next layer's argument is reduced from
    // slot parameters read one layer earlier, the parameters of the one
    // after are read, and the record of the third (past the stack: pads)
    const LayerRec* p = rec + i0;
    const LayerRec r0 = p[0], r1 = p[dir];
    LayerRec r2 = p[2 * dir];
    p += 3 * dir;
    double kq, xs, ys, xp, yp, kq1, xs1, ys1, xp1, yp1;
    sl.lossless_r(r0, kq, xs, ys, xp, yp);
    sl.lossless_r(r1, kq1, xs1, ys1, xp1, yp1);
    double t1 = r1.t;
    typename LT::Arg ta = LT::reduce(kq, r0.t);          // t = 0 gives the identity exactly
    for (int k0_ = 0; k0_ < n; k0_ += kStageRows) {
        const int rows = min(kStageRows, n - k0_);
        double* o = stage + lane;
#pragma unroll 4
        for (int q = 0; q < rows; ++q, o += kStageLanes) {
            const LayerRec r3 = *p;
            p += dir;
            double kq2, xs2, ys2, xp2, yp2;
            sl.lossless_r(r2, kq2, xs2, ys2, xp2, yp2);
            const typename LT::Arg ta1 = LT::reduce(kq1, t1);
            double C, S0;
            LT::eval(ta, &C, &S0, &n_unused);
            const double S = flip_sign(S0, sflip);
            const double sXs = S * xs, sYs = S * ys, sXp = S * xp, sYp = S * yp;
            const double gys = (HC && kq < 0.0) ? -ys : ys;       // sg y_s (an evanescent layer: sg = -1)
            *o = v.gradient(gys, ys, xp, yp);
            v.pass(C, sXs, sYs, sXp, sYp);
            ta = ta1; kq = kq1; xs = xs1; ys = ys1; xp = xp1; yp = yp1;
            kq1 = kq2; xs1 = xs2; ys1 = ys2; xp1 = xp2; yp1 = yp2; t1 = r2.t;
            r2 = r3;
        }
        wave_lds_sync();
        // lane: row lane / 8 (rows past the last: stale, not used)
        const double2* r = (const double2*)(stage + (lane >> 3) * kStageLanes) + (lane & 7);
        const double2 v0 = r[0], v1 = r[8], v2 = r[16], v3 = r[24];
        const double s = sum8(((v0.x + v0.y) + (v1.x + v1.y)) + ((v2.x + v2.y) + (v3.x + v3.y)));
        if ((lane & 7) == 0 && (lane >> 3) < rows) gw[i0 + dir * (k0_ + (lane >> 3))] += s;
        wave_lds_sync();
    }
}

// The method of tmm_adjoint_lossless for a wave whose lanes meet one mirror (L
// layers, rec: its records) from one side, all reflected (REFL) or all
// transmitted, all in segments of K layers.  Lanes without an entry have zero
// cotangents.  The gradient of a layer is summed over the lanes, kStageRows
// layers at a time.
// A reflected hit's scaled state goes up each segment from its exit side; blk:
// its states above the segments (64-byte blocks, block g at blk + g bstride).
// A transmitted hit's Q is formed at each segment end g from w_g and u_g and
// goes half a segment up and half a segment down; blk: its segment matrices,
// wst: room for its states w_g (block g at wst + g wstride).
template <bool HC, bool REFL, class SL>
__device__ __attribute__((always_inline)) inline void adjoint_class(const LayerRec* rec, int L, bool front, const SL& sl,
                                                                    double k0, double eta0s, double eta0p, cd Gs, cd Gp,
                                                                    int K, const double* blk, int64_t bstride, double* wst,
                                                                    int64_t wstride, double* stage, double* gw)
{
    const double k2 = 2.0 * k0;
    auto walk = [&](double As, double bs, double cs, double Ap, double bp, double cp, int j0, int n, bool up) {
        class_walk<HC>(rec, L, front, sl, CarryQ{ As, bs, cs, Ap, bp, cp }, j0, n, up, stage, gw);
    };
    auto read = [](const double* q, V2d& a, V2d& b) {
        const double2* p = (const double2*)q;
        const double2 x0 = p[0], x1 = p[1], x2 = p[2], x3 = p[3];
        a = V2d{ x0.x, x0.y, x1.x, x1.y };
        b = V2d{ x2.x, x2.y, x3.x, x3.y };
    };
    V2d ws = { 1.0, 0.0, eta0s, 0.0 }, wp = { 1.0, 0.0, eta0p, 0.0 };
    const int G = seg_of(L - 1, K) + 1;
    if constexpr (REFL) {
        V2d ts, tp;
        read(blk, ts, tp);
        const cd fs = csqrt_any(cscale(cov_top(ts, eta0s, true, false, cscale(Gs, k2)).u1, 2.0));
        const cd fp = csqrt_any(cscale(cov_top(tp, eta0p, true, true, cscale(Gp, k2)).u1, 2.0));
        for (int g = G - 1; g >= 0; --g) {
            const CarryW v = { state_scale(fs, ws), state_scale(fp, wp) };
            const int j = min((g + 1) * K, L);
            if (g > 0) read(blk + (int64_t)g * bstride, ws, wp);         // in flight
            class_walk<HC>(rec, L, front, sl, v, j - 1, j - g * K, true, stage, gw);
        }
        return;
    }
    auto get_seg = [&](int g) {
        const double2* p = (const double2*)(blk + (int64_t)g * bstride);
        const double2 a = p[0], b = p[1], c = p[2], d = p[3];
        return SegPair{ { a.x, a.y, b.x, b.y }, { c.x, c.y, d.x, d.y } };
    };
    {
        SegPair m = get_seg(G - 1);
        for (int g = G - 1; g >= 0; --g) {
            SegPair mn = m;
            if (g > 0) mn = get_seg(g - 1);
            seg_apply(m.s, ws.br, ws.bi, ws.cr, ws.ci);
            seg_apply(m.p, wp.br, wp.bi, wp.cr, wp.ci);
            if (g > 0) {
                double2* o = (double2*)(wst + (int64_t)g * wstride);
                o[0] = make_double2(ws.br, ws.bi); o[1] = make_double2(ws.cr, ws.ci);
                o[2] = make_double2(wp.br, wp.bi); o[3] = make_double2(wp.cr, wp.ci);
            }
            m = mn;
        }
    }
    CovRow us = cov_top(ws, eta0s, false, false, cscale(Gs, k2));
    CovRow up = cov_top(wp, eta0p, false, true, cscale(Gp, k2));
    for (int g = 0; g <= G; ++g) {
        // segment end g: above layer g K (g < G), below layer min(g K, L) - 1;
        // the segments' middles: (lo + hi) / 2
        const int j = min(g * K, L);
        double As, bs, cs, Ap, bp, cp;
        cov_q(us.u1, us.u2, ws, As, bs, cs);
        cov_q(up.u1, up.u2, wp, Ap, bp, cp);
        SegPair m{};
        if (g < G) {                                         // the next end's state and matrix, in flight
            m = get_seg(g);
            if (g + 1 < G) read(wst + (int64_t)(g + 1) * wstride, ws, wp);
            else { ws = V2d{ 1.0, 0.0, eta0s, 0.0 }; wp = V2d{ 1.0, 0.0, eta0p, 0.0 }; }
        }
        if (g > 0) walk(As, bs, cs, Ap, bp, cp, j - 1, j - ((g - 1) * K + j) / 2, true);
        if (g < G) {
            walk(As, bs, cs, Ap, bp, cp, j, (j + min(j + K, L)) / 2 - j, false);
            cov_step(us, m.s);
            cov_step(up, m.p);
        }
    }
}

// Adjoint of a class where the mirror has absorbing layers.  The stack is cut
// into pieces: absorbing layers, and runs of up to kSegL lossless ones (pc[0]:
// their number; pc[1 + p]: piece p's first layer in stack order, bit 15 set if
// it is an absorbing layer).  A run goes as in adjoint_class, half of it down
// from its top and half up from its exit side (a reflected hit's scaled state
// all up); an absorbing layer takes the state and the covector themselves.  (A reflected
// hit's covector is c (C, -B) there as well: absorbing layers are unimodular.)
// own: room for the runs' segment matrices, as wst.
// 363 points x 4096 rays, 201 layers, one of them silver: 14.3 ms with every
// four layers solved again between stored states, 5.4 ms in pieces, sorted.
template <bool HC, class SL>
__device__ __attribute__((always_inline)) inline void adjoint_pieces(const LayerRec* rec, int L, const uint16_t* pc, bool front,
                                                                     const SL& sl, double k0, double kappa2, double eta0s,
                                                                     double eta0p, bool refl, cd Gs, cd Gp, double* own,
                                                                     double* wst, int64_t wstride, double* stage, double* gw)
{
    const int lane = wave_lane();
    const double k2 = 2.0 * k0;
    const int P = __builtin_amdgcn_readfirstlane((int)pc[0]);
    int a = 0, b = 0;                                        // the piece's layers [a, b) in stack order
    bool absorbing = false;
    auto piece = [&](int i) {                                // i-th in incidence order
        const int p = front ? i : P - 1 - i;
        const int v = __builtin_amdgcn_readfirstlane((int)pc[1 + p]);
        a = v & 0x7fff;
        absorbing = (v >> 15) != 0;
        b = p + 1 < P ? __builtin_amdgcn_readfirstlane((int)pc[2 + p]) & 0x7fff : L;
    };
    auto entries = [&](CTv<double>& C, CTv<double>& Xs, CTv<double>& Ys, CTv<double>& Xp, CTv<double>& Yp, double* Pd) {
        const LayerRec r = rec[a];
        sl.absorbing((int)r.slot, Pd);
        layer_cplx(Pd, k0, r.t, &C, &Xs, &Ys, &Xp, &Yp);     // t = 0 gives the identity exactly
    };
    auto read = [](const double* q, V2d& x, V2d& y) {
        const double2* p = (const double2*)q;
        const double2 x0 = p[0], x1 = p[1], x2 = p[2], x3 = p[3];
        x = V2d{ x0.x, x0.y, x1.x, x1.y };
        y = V2d{ x2.x, x2.y, x3.x, x3.y };
    };
    V2<double> vs = { 1.0, 0.0, eta0s, 0.0 }, vp = { 1.0, 0.0, eta0p, 0.0 };
    for (int i = P - 1; i >= 0; --i) {
        piece(i);
        if (!absorbing) {
            int es = 0, ep = 0;
            const RecCursor cur = { rec + (front ? b - 1 : a), front ? -1 : 1 };
            lossless_sweep<double, HC, true>(cur, b - a, sl, vs, vp, es, ep, own + i * wstride, wstride, kSegL);
        } else {
            CTv<double> C, Xs, Ys, Xp, Yp;
            double Pd[4];
            entries(C, Xs, Ys, Xp, Yp, Pd);
            step_cplx(vs, C, Xs, Ys);
            step_cplx(vp, C, Xp, Yp);
        }
        if (i > 0) {
            double2* o = (double2*)(wst + i * wstride);
            o[0] = make_double2(vs.br, vs.bi); o[1] = make_double2(vs.cr, vs.ci);
            o[2] = make_double2(vp.br, vp.bi); o[3] = make_double2(vp.cr, vp.ci);
        }
    }
    V2d ws = { vs.br, vs.bi, vs.cr, vs.ci }, wp = { vp.br, vp.bi, vp.cr, vp.ci };
    CovRow us = cov_top(ws, eta0s, refl, false, cscale(Gs, k2));
    CovRow up = cov_top(wp, eta0p, refl, true, cscale(Gp, k2));
    const cd fs = csqrt_any(cscale(us.u1, 2.0)), fp = csqrt_any(cscale(up.u1, 2.0));     // of a reflected hit
    for (int i = 0; i < P; ++i) {
        piece(i);
        V2d ns = { 1.0, 0.0, eta0s, 0.0 }, np = { 1.0, 0.0, eta0p, 0.0 };       // the states below
        if (i + 1 < P) read(wst + (i + 1) * wstride, ns, np);
        if (!absorbing) {
            const int lo = front ? a : L - b, hi = front ? b : L - a;
            if (refl) {
                class_walk<HC>(rec, L, front, sl, CarryW{ state_scale(fs, ns), state_scale(fp, np) }, hi - 1, hi - lo, true,
                               stage, gw);
            } else {
                const int mid = (lo + hi) / 2;
                double As, bs, cs, Ap, bp, cp;
                cov_q(us.u1, us.u2, ws, As, bs, cs);
                cov_q(up.u1, up.u2, wp, Ap, bp, cp);
                class_walk<HC>(rec, L, front, sl, CarryQ{ As, bs, cs, Ap, bp, cp }, lo, mid - lo, false, stage, gw);
                const double2* q = (const double2*)(own + i * wstride);
                const double2 x0 = q[0], x1 = q[1], x2 = q[2], x3 = q[3];
                cov_step(us, SegMat{ x0.x, x0.y, x1.x, x1.y });
                cov_step(up, SegMat{ x2.x, x2.y, x3.x, x3.y });
                cov_q(us.u1, us.u2, ns, As, bs, cs);
                cov_q(up.u1, up.u2, np, Ap, bp, cp);
                class_walk<HC>(rec, L, front, sl, CarryQ{ As, bs, cs, Ap, bp, cp }, hi - 1, hi - mid, true, stage, gw);
            }
        } else {
            CTv<double> C, Xs, Ys, Xp, Yp;
            double Pd[4];
            entries(C, Xs, Ys, Xp, Yp, Pd);
            const cd N2 = mk(Pd[2], Pd[3]), z = csub(N2, mk(kappa2, 0.0));
            const cd Bs = mk(ws.br, ws.bi), Cs = mk(ws.cr, ws.ci), Bp = mk(wp.br, wp.bi), Cp = mk(wp.cr, wp.ci);
            cd u1s = us.u1, u2s = us.u2, u1p = up.u1, u2p = up.u2;
            if (refl) {
                u1s = cmul(us.u1, Cs); u2s = cscale(cmul(us.u1, Bs), -1.0);
                u1p = cmul(up.u1, Cp); u2p = cscale(cmul(up.u1, Bp), -1.0);
            }
            // contraction u^T D w, D = -i k0 [[0, a], [b, 0]]
            const cd As = cadd(cmul(u1s, Cs), cmul(z, cmul(u2s, Bs)));
            const cd Ap = cadd(cmul(cdiv(z, N2), cmul(u1p, Cp)), cmul(N2, cmul(u2p, Bp)));
            stage[lane] = As.im + Ap.im;
            wave_lds_sync();
            const double2* v = (const double2*)stage + (lane & 7);
            const double2 v0 = v[0], v1 = v[8], v2 = v[16], v3 = v[24];
            const double sum = sum8(((v0.x + v0.y) + (v1.x + v1.y)) + ((v2.x + v2.y) + (v3.x + v3.y)));
            if (lane == 0) gw[a] += sum;
            wave_lds_sync();
            if (!refl) {
                const cd c = mk(C.re, C.im);
                cov_step(us.u1, us.u2, c, mk(Xs.re, Xs.im), mk(Ys.re, Ys.im));
                cov_step(up.u1, up.u2, c, mk(Xp.re, Xp.im), mk(Yp.re, Yp.im));
            }
        }
        ws = ns;
        wp = np;
    }
}

struct SortedLayout { int off_pl, off_rec, off_sp, off_stage, off_grad, total; };
__host__ __device__ inline SortedLayout sorted_layout(int Lmax, int n_slots)
{
    SortedLayout s;
    int o = 0;
    s.off_pl = o; o = align16(o + (int)sizeof(PointLds));
    s.off_rec = o; o = align16(o + (int)sizeof(LayerRec) * rec_stride(Lmax));
    s.off_sp = o; o = align16(o + 8 * n_slots * LaneSlots3x::kPer * 64);
    s.off_stage = o; o = align16(o + 8 * kStageRows * kStageLanes);
    s.off_grad = o; o = align16(o + 8 * Lmax);
    s.total = o;
    return s;
}

// One wave per workgroup; scratch: per lane twice ck_blocks(Lmax) (absorbing
// slots: max_pieces) blocks of 64 bytes, block k of lane t of the grid at scratch + 8 (k nthreads + t).
template <bool LOSSLESS>
__global__ void __launch_bounds__(64, 2) k_adj_sorted(SceneDev sc, const double* __restrict__ dLdI,
                                                      double* __restrict__ partial, AdjStore st, SortDev so,
                                                      double* __restrict__ scratch,
                                                      unsigned long long* __restrict__ stats)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const SortedLayout lay = sorted_layout(sc.Lmax, sc.n_slots);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    LayerRec* s_rec = (LayerRec*)(smem + lay.off_rec);
    double* stage = (double*)(smem + lay.off_stage);
    double* gw = (double*)(smem + lay.off_grad);
    const int lane = wave_lane();
    const int B = sc.bins_x * sc.bins_y, ML = sc.M * sc.Lmax;
    const LaneSlots3x sl = { slot_lane_base((double*)(smem + lay.off_sp), sc.n_slots, LaneSlots3x::kPer, lane), pl->nsq,
                            pl->pxy };
    const int64_t wstride = (int64_t)gridDim.x * 64 * 8;
    double* wst = scratch + ((int64_t)blockIdx.x * 64 + lane) * 8;
    // segment matrices of a sweep run here
    double* own = wst + (LOSSLESS ? ck_blocks(sc.Lmax) : (int64_t)sc.max_pieces) * wstride;
    __shared__ uint16_t s_pc[kMaxPieces + 1];
    unsigned long long c_hits = 0, c_lay = 0, c_stored = 0;
    int64_t staged = -1;
    for (int k = lane; k < kStageRows * kStageLanes; k += 64) stage[k] = 0.0;

    // Units of a large launch are drawn, after a first one each, so that the
    // waves end together; draws follow one another at some 12 ns, which a
    // small launch does without.
    const int64_t n_units = so.groups * kUnitParts * sc.M;
    const bool draw = n_units > 4 * (int64_t)gridDim.x;
    for (int64_t unit = blockIdx.x; unit < n_units;
         unit = draw ? gridDim.x + draw_item(stats + ST_NEXT0) : unit + gridDim.x) {
        const int64_t row = unit / sc.M, group = row / kUnitParts;
        const int m = (int)(unit - row * sc.M), part = (int)(row - group * kUnitParts);
        const int64_t dl = group / so.groups_dl;
        const int d = (int)(dl / sc.n_lsel), l = (int)(dl - (int64_t)d * sc.n_lsel);
        int64_t ia, ib;
        group_items(sc, so, group, &ia, &ib);
        if (dl != staged) {
            // what the adjoint reads of the wavelength and the design
            const double* lt = sc.lam_tab + (int64_t)l * LT_STRIDE;
            if (lane < kMaxSlots) {
                const double nr = lt[LT_SLOT + 2 * lane], ni = lt[LT_SLOT + 2 * lane + 1];
                pl->slotN[2 * lane] = nr; pl->slotN[2 * lane + 1] = ni;
                pl->nsq[2 * lane] = nr * nr - ni * ni; pl->nsq[2 * lane + 1] = 2.0 * nr * ni;
                pl->pxy[2 * lane] = (ni == 0.0 && nr != 0.0) ? 1.0 / (nr * nr) : 0.0;
                pl->pxy[2 * lane + 1] = nr * nr - ni * ni;
            }
            if (lane < sc.M) pl->nlay[lane] = sc.nlay[(int64_t)d * sc.M + lane];
            if (lane == 0) { pl->k0 = lt[LT_K0]; pl->ng = lt[LT_NG]; }
        }
        staged = dl;
        stage_recs(s_rec, sc.thk + ((int64_t)d * sc.M + m) * sc.Lmax, sc.slot + ((int64_t)d * sc.M + m) * sc.Lmax, 1,
                   sc.Lmax, LaneSlots3x::kPer);
        for (int k = lane; k < sc.Lmax; k += 64) gw[k] = 0.0;
        if (!LOSSLESS && lane <= kMaxPieces) s_pc[lane] = sc.pieces[((int64_t)d * sc.M + m) * (kMaxPieces + 1) + lane];
        __syncthreads();
        const int L = pl->nlay[m];
        const double k0 = pl->k0, ng = pl->ng;
        const int64_t e0 = ia * st.waves * st.cap_w;     // the group's first entry
        const int32_t* start = so.start + group * (kClasses + 1) + kMirClasses * m;
        const RecStack stk = { s_rec + kRecPad };
        int batches = 0;                                     // of the mirror; this unit: [q, q_end)
        for (int cls = 0; cls < kMirClasses; ++cls) batches += (start[cls + 1] - start[cls] + 63) / 64;
        int q = (int)((int64_t)batches * part / kUnitParts);
        const int q_end = (int)((int64_t)batches * (part + 1) / kUnitParts);
        int q_cls = 0;                                       // the class's first batch
        for (int cls = 0; cls < kMirClasses && q < q_end && L > 0; ++cls) {
            const int b1 = start[cls + 1], n_b = (b1 - start[cls] + 63) / 64;
            const bool front = (cls & 4) != 0, evan = (cls & 2) != 0, refl = (cls & 1) != 0;
            const int K = ck_interval(evan);
            const int q_stop = min(q_cls + n_b, q_end);
            for (; q < q_stop; ++q) {
                const int b = start[cls] + 64 * (q - q_cls);
                const bool mine = b + lane < b1;         // other lanes: the class's last entry, zero cotangents
                const int64_t rel = so.order[e0 + min(b + lane, b1 - 1)];
                const AdjEntry en = load_entry(st, e0 + rel);
                const int64_t region = rel / st.cap_w;
                const int64_t item = ia + region / st.waves;
                const double gscale = mine ? dLdI[item / sc.tiles_per_point * B + ent_bin(en.meta)] / (double)sc.N : 0.0;
                const cd Gs = cscale(mk(en.gs_re, en.gs_im), gscale), Gp = cscale(mk(en.gp_re, en.gp_im), gscale);
                const double kappa = en.kappa;
                for (int s = 0; s < sc.n_slots; ++s) {
                    double P[NPF];
                    slot_params(pl->slotN[2 * s], pl->slotN[2 * s + 1], !LOSSLESS && ((sc.slot_complex >> s) & 1u), kappa, k0, P);
                    sl.put(s, P);
                }
                const double z0 = ng * ng - kappa * kappa;
                const double q0 = sqrt(z0 > kTinyZ ? z0 : kTinyZ), q0p = ng * ng / q0;
                // the forward stored this entry's blocks; else they are swept
                // here (the same arithmetic: whether an entry is stored
                // decides neither its batch nor its gradient)
                const int64_t k = rel - region * st.cap_w, greg = ia * st.waves + region;
                const bool stored = LOSSLESS && st.ck && greg < st.ck_regions && k < st.ck_cap && (!evan || st.ck_evan);
                const double* blk = stored ? st.ck + (greg * st.ck_cap + k) * st.ck_nb * 8 : own;
                const int64_t bstride = stored ? 8 : wstride;
                auto run = [&](auto hc) {
                    constexpr bool HC = decltype(hc)::value;
                    if constexpr (!LOSSLESS) {
                        adjoint_pieces<HC>(stk.rec, L, s_pc, front, sl, k0, kappa * kappa, q0, q0p, refl, Gs, Gp, own, wst,
                                           wstride, stage, gw);
                        return;
                    }
                    if (!stored) {
                        V2<double> vs = { 1.0, 0.0, q0, 0.0 }, vp = { 1.0, 0.0, q0p, 0.0 };
                        int es = 0, ep = 0;
                        lossless_sweep<double, HC, true>(stk.cursor(L, front), L, sl, vs, vp, es, ep, own, wstride, K, refl);
                    }
                    if (refl)
                        adjoint_class<HC, true>(stk.rec, L, front, sl, k0, q0, q0p, Gs, Gp, K, blk, bstride, wst, wstride,
                                                stage, gw);
                    else
                        adjoint_class<HC, false>(stk.rec, L, front, sl, k0, q0, q0p, Gs, Gp, K, blk, bstride, wst, wstride,
                                                 stage, gw);
                };
                if (evan) run(std::true_type{});
                else run(std::false_type{});
                if (mine) {
                    c_hits += 1;
                    c_lay += (unsigned long long)L;
                    if (stored) c_stored += (unsigned long long)L;
                }
            }
            q_cls += n_b;
        }
        __syncthreads();
        double* out = partial + row * ML + (int64_t)m * sc.Lmax;
        for (int k = lane; k < sc.Lmax; k += 64) out[k] = gw[k];
    }
    if (c_hits) atomicAdd(&stats[ST_ADJ_HITS], c_hits);
    if (c_lay) atomicAdd(&stats[ST_ADJ_LAYERS], c_lay);
    if (c_stored) atomicAdd(&stats[ST_ADJ_STORED], c_stored);
}

// The division into groups: entries of kGroupRays rays (some 4000 per mirror,
// so that few of the batches are partly filled), fewer where that leaves fewer
// than kUnitsWanted units; a group stays within one design and wavelength.
// Mirrors differ several times in their hits, so a (group, mirror) is cut into
// kUnitParts units of equal numbers of batches, else the largest ones that are
// drawn last run on alone (one unit each, in order: 21.8 ms instead of 15.9).
// At least kGroupRaysMin rays: with fewer most batches would hold one or two
// entries (27 points of 500 rays in items of 64, 40 layers: adjoint 92 us, by points 29 us).
constexpr int64_t kGroupRays = 8192, kGroupRaysMin = 512;
constexpr int64_t kUnitsWanted = 8192;
void sort_shape(const SceneDev& sc, SortDev* so)
{
    const int64_t items_dl = (int64_t)sc.F * sc.tiles_per_point;
    const int64_t rays = (int64_t)sc.D * sc.n_lsel * sc.F * sc.N;
    int64_t want = rays * sc.M * kUnitParts / kUnitsWanted;
    want = want < kGroupRaysMin ? kGroupRaysMin : want < kGroupRays ? want : kGroupRays;
    int64_t ng = want / (sc.rays_per_tile < sc.N ? sc.rays_per_tile : sc.N);
    ng = ng < 1 ? 1 : ng > items_dl ? items_dl : ng;
    so->ng = (int32_t)ng;
    so->groups_dl = (int32_t)((items_dl + ng - 1) / ng);
    so->groups = (int64_t)sc.D * sc.n_lsel * so->groups_dl;
}
int64_t sorted_rows(const SceneDev& sc)
{
    SortDev so;
    sort_shape(sc, &so);
    return so.groups / sc.D * kUnitParts;
}
int64_t sorted_ints(const SceneDev& sc)
{
    SortDev so;
    sort_shape(sc, &so);
    return so.groups * (kClasses + 1);
}
size_t sorted_smem_bytes(const SceneDev& sc) { return (size_t)sorted_layout(sc.Lmax, sc.n_slots).total; }
int64_t sorted_scratch_doubles(const SceneDev& sc, int64_t grid)
{
    return 2 * (sc.slot_complex ? (int64_t)sc.max_pieces : ck_blocks(sc.Lmax)) * 8 * 64 * grid;
}
