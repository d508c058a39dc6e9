// Direction states of collimated beams.  Included by gwg_kernels.hip inside
// namespace gwg, before the trace kernels.
//
// All rays of one (wavelength, FoV) point start in one direction, and a
// direction changes only at a face (z -> -z, exact) or in a mirror
// reflection (one normal for all mirrors).  So the rays of a point share a
// small tree of directions: the bits of a direction depend only on the
// sequence of reflections before it (7 to 36 distinct ones up to the sign of
// z, counted over 8192 rays of six-mirror points).  k_dir_states walks that
// tree once per scene, breadth first, with the walk's own operations, and
// keeps up to kDirMax directions per point with everything an event needs
// from its direction alone:
//   - the reciprocals that turn the walk's distance quotients into one
//     product and two fused multiply-adds (dir_quot: the same bits as the
//     division),
//   - kappa, the faces' coefficients and the exit's,
//   - the rotation between the face basis and the mirror basis.
// A ray is then (position, state, sign of z, cell), and its field two complex
// numbers along the face basis of its state (FaceSp): a total reflection
// multiplies them by (r_s, r_p), a mirror hit rotates them into the mirror
// basis, applies the coefficients and rotates back.  Positions, surfaces,
// branches and bins keep the general walk's operations (walk_ray) and its
// bits.  A ray that leaves the table (a reflection whose direction is not
// among the kDirMax kept, a horizontal direction, or a mirror met within 1e-4
// of normal incidence, where the mirror basis is ill defined) is traced by
// the general walk instead.
//
// The general walks are bound by instruction issue (about 500 VALU slots per
// event and wave for the geometry, 1600 with the field and the tape: three
// divisions, two square roots, two bases and four 3-vectors an event).
// Forward kernel before and after, 6 mirrors, 3 x 441 points: 8192 rays a
// point, 200 layers, gradient flag 29.3 -> 23.1 ms, memoized 14.5 -> 3.4 ms,
// angle table 12.4 -> 3.4 ms; 65536 rays a point, 40 layers, no gradient
// 93.1 -> 55.5 ms.  The walk's loop keeps its state's quantities in registers
// (read from LDS at every event instead: 17.4 ms of geometry for 8.3e8
// events; so: 13.1 ms); what is left of it is issue and LDS latency at two
// waves per SIMD.

constexpr int kDirMax = 64;           // directions kept per point
constexpr int kDirGeo = 12;           // doubles of a state's geometry part
constexpr int kDirFld = 12;           // doubles of a state's field part
constexpr int kDirWords = kDirGeo + kDirFld;
constexpr int kDirOff = 255;          // a child that is not in the table
// geometry part: |dz|, 1/|dz|, dx, 1/dx, then for dz > 0 and dz < 0 (n.d,
// 1/(n.d)), the flag word, kappa for dz > 0 and dz < 0, unused
enum { DG_ADZ = 0, DG_RDZ = 1, DG_DX = 2, DG_RDX = 3, DG_DN = 4, DG_FLAGS = 8, DG_KAP = 9 };
// field part: r_s, r_p of total reflection (complex), (c, d) of the mirror
// basis in the face basis for dz > 0 and dz < 0 (s_m = c s + d p), exit
// amplitudes flux t_s, flux t_p, and the eyebox plane offsets in x and y
enum { DF_RS = 0, DF_RP = 2, DF_ROT = 4, DF_XS = 8, DF_XP = 9, DF_EX = 10, DF_EY = 11 };
// flag word: child states (state << 1 | dz < 0) after a reflection at dz > 0
// (bits 0-7) and dz < 0 (bits 8-15), total reflection at the faces (bit 16),
// mirror basis defined at dz > 0 and dz < 0 (bits 17, 18)
constexpr uint32_t kDirTir = 1u << 16;

// n / d for finite operands from r = 1 / d correctly rounded: one fused
// correction of n r gives the correctly rounded quotient (Markstein, 1990).
__device__ inline double dir_quot(double n, double d, double r)
{
    const double q = n * r;
    return fma(fma(-q, d, n), r, q);
}

// One wave per (wavelength, FoV) point; lane i holds state i.
__global__ void __launch_bounds__(64) k_dir_states(SceneDev sc, double* __restrict__ out, int32_t* __restrict__ n_out)
{
    __shared__ int s_queue[2 * kDirMax];
    __shared__ int s_child[kDirMax][2];
    const int lane = wave_lane();
    const int64_t pt = blockIdx.x;
    const double* lt = sc.lam_tab + (pt / sc.F) * LT_STRIDE;
    const double ng = lt[LT_NG], na = lt[LT_NA];
    const double* d0 = sc.dir_tab + pt * 4;
    const double dy = d0[1];
    double ex = 0.0, ez = 0.0;                            // this lane's state: dx, |dz|
    int n = 0, qn = 0;
    unsigned long long seen0 = 0ull, seen1 = 0ull;        // queued (state, dz > 0) and (state, dz < 0)
    s_child[lane][0] = s_child[lane][1] = kDirOff;
    // state index of a direction (added if new), -1 if the table is full
    auto state = [&](double dx, double adz) {
        const unsigned long long m = __ballot(lane < n && ex == dx && ez == adz);
        if (m) return __ffsll((long long)m) - 1;
        if (n == kDirMax) return -1;
        if (lane == n) { ex = dx; ez = adz; }
        return n++;
    };
    auto push = [&](int e, int neg) {
        unsigned long long& seen = neg ? seen1 : seen0;
        if ((seen >> e) & 1ull) return;
        seen |= 1ull << e;
        if (lane == 0) s_queue[qn] = e << 1 | neg;
        ++qn;
    };
    // a direction a ray can have; total reflection at a face reaches the other sign
    auto reach = [&](int e, int neg) {
        const double dx = __shfl(ex, e, 64);
        const bool tir = (ng * ng) * (dx * dx + dy * dy) > na * na;
        push(e, neg);
        if (tir) push(e, neg ^ 1);
    };
    if (d0[2] != 0.0) reach(state(d0[0], fabs(d0[2])), d0[2] < 0.0 ? 1 : 0);
    for (int q = 0; q < qn; ++q) {
        __syncthreads();
        const int e = s_queue[q] >> 1, neg = s_queue[q] & 1;
        const double dx = __shfl(ex, e, 64), az = __shfl(ez, e, 64);
        double ox, oz;
        mirror_reflect(sc.nx, sc.nz, dx, neg ? -az : az, &ox, &oz);
        if (oz == 0.0) continue;
        const int c = state(ox, fabs(oz));
        if (c < 0) continue;
        if (lane == 0) s_child[e][neg] = c << 1 | (oz < 0.0 ? 1 : 0);
        reach(c, oz < 0.0 ? 1 : 0);
    }
    __syncthreads();
    if (lane == 0) n_out[pt] = n;
    if (lane >= n) return;
    double* g = out + (pt * kDirMax + lane) * kDirWords;
    double* f = g + kDirGeo;
    const FaceCoef fc = face_coeffs(ng, na, ex, dy, ez);
    uint32_t flags = (uint32_t)s_child[lane][0] | (uint32_t)s_child[lane][1] << 8;
    if (fc.tir) flags |= kDirTir;
    g[DG_ADZ] = ez; g[DG_RDZ] = 1.0 / ez;
    g[DG_DX] = ex; g[DG_RDX] = 1.0 / ex;
    f[DF_RS] = fc.rs.re; f[DF_RS + 1] = fc.rs.im; f[DF_RP] = fc.rp.re; f[DF_RP + 1] = fc.rp.im;
    f[DF_XS] = fc.ts.re * fc.flux; f[DF_XP] = fc.tp.re * fc.flux;
    f[DF_EX] = f[DF_EY] = 0.0;
    if (!fc.tir) {
        Ray r;
        r.dx = ex; r.dy = dy; r.dz = ez;
        double a[3];
        exit_direction(ng, na, r, fc.st2, a);
        f[DF_EX] = sc.ER * (a[0] / a[2]);
        f[DF_EY] = sc.ER * (a[1] / a[2]);
    }
    for (int neg = 0; neg < 2; ++neg) {
        const double dz = neg ? -ez : ez;
        const double dn = sc.nx * ex + sc.nz * dz;
        g[DG_DN + 2 * neg] = dn;
        g[DG_DN + 2 * neg + 1] = 1.0 / dn;
        double c[3];
        cross3(ex, dy, dz, sc.nx, 0.0, sc.nz, c);
        const double l = sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
        g[DG_KAP + neg] = ng * l;
        if (l >= 1e-4) flags |= kDirTir << (1 + neg);
        double sf[3], pf[3], sm[3];
        s_basis(ex, dy, dz, 0.0, 0.0, 1.0, sf);
        cross3_f(ex, dy, dz, sf[0], sf[1], sf[2], pf);
        s_basis(ex, dy, dz, sc.nx, 0.0, sc.nz, sm);
        f[DF_ROT + 2 * neg] = fma(sf[2], sm[2], fma(sf[1], sm[1], sf[0] * sm[0]));
        f[DF_ROT + 2 * neg + 1] = fma(pf[2], sm[2], fma(pf[1], sm[1], pf[0] * sm[0]));
    }
    g[DG_FLAGS] = __longlong_as_double((long long)flags);
    g[11] = 0.0;
}

// A workgroup's direction table in LDS: the geometry parts, then the field parts.
struct DirLds {
    const double* g;                  // [kDirMax][kDirGeo]
    const double* f;                  // [kDirMax][kDirFld]
    double dy;                        // the point's direction y (never changes)
    int root;                         // the rays' first state << 1 | dz < 0 (kDirOff: none)
};

// Load point pt's table into LDS (whole block; a barrier follows).
__device__ inline DirLds stage_dirs(const SceneDev& sc, int64_t pt, double* mem)
{
    const int n = sc.dir_n[pt];
    const double* src = sc.dirs + pt * kDirMax * kDirWords;
    double *g = mem, *f = mem + kDirMax * kDirGeo;
    for (int i = threadIdx.x; i < n * kDirWords; i += blockDim.x) {
        const int e = i / kDirWords, k = i - e * kDirWords;
        if (k < kDirGeo) g[e * kDirGeo + k] = src[i];
        else f[e * kDirFld + (k - kDirGeo)] = src[i];
    }
    const double* d0 = sc.dir_tab + pt * 4;
    DirLds t = { g, f, d0[1], n > 0 ? (d0[2] < 0.0 ? 1 : 0) : kDirOff };
    return t;
}

// A mirror hit's word on the queue: mirror | front << 8 | reflected << 9 |
// dz < 0 << 10 | state << 11 | total reflections since the last hit << 19
// (the last three of rays on the table only).
__device__ inline int hit_word(int m, int front, int refl, int neg, int e, int nt)
{
    return m | front << 8 | refl << 9 | neg << 10 | e << 11 | nt << 19;
}

// Key of a table ray's hit: (state, sign of z, mirror); the side follows from
// the direction.
__device__ inline int hit_key(int word, int M) { return ((word >> 10) & 511) * M + (word & 255); }

// Where a ray of the table ended.
struct DirFate {
    int cat, bin, nev, nh;
    int e, neg, nt;                   // final state, sign, total reflections since the last hit
    int pol;                          // first field: 0 along s, 1 along p
    bool off;                         // left the table: trace it with the general walk
};

// Geometry and branch decisions of one ray of the point: walk_ray<false>'s
// operations on positions, with the direction's quantities from the table.
// Every mirror hit h calls on_hit(h, &kappa, word) and on_hit.branch(m, refl).
// The random words of the first eight hits are drawn before the loop, where
// every lane needs them, rather than in the iteration in which some lane of
// the wave reaches its first or fifth hit.
template <class OnHit>
__device__ inline void dir_walk(const SceneDev& sc, const PointLds& pl, const DirLds& dt, int64_t id, OnHit on_hit,
                                DirFate& o)
{
    const uint32_t key1 = philox_key1(sc);
    const int64_t gid = id + sc.id_base;
    const uint32_t id0 = (uint32_t)(uint64_t)gid, id1 = (uint32_t)((uint64_t)gid >> 32);
    const u32x4 w = philox10(id0, id1, 0u, 0u, sc.key0, key1);
    u32x4 wa = philox10(id0, id1, 0u, 1u, sc.key0, key1);
    u32x4 wb = philox10(id0, id1, 1u, 1u, sc.key0, key1);
    double px = sc.px0 + u24(w.x) * sc.pw;
    double py = u24(w.y) * sc.ph - 0.5 * sc.ph;
    double pz = pl.T;
    const double nx = pl.nx, nz = pl.nz, T = pl.T, dy = dt.dy;
    const int M = pl.M, Kmax = pl.Kmax;
    int e = 0, neg = dt.root, cell = 0, last = SURF_TOP, nev = 0, nh = 0, nt = 0;
    o.pol = (int)(w.x & 1u);
    o.bin = -1;
    o.off = neg == kDirOff;
    o.cat = CAT_LOST;
    o.e = 0;
    if (o.off) return;
    // the state's quantities stay in registers between reflections
    double adz, rdz, dx, dnp, rdnp, dnn, rdnn;
    uint32_t fl;
    auto load = [&]() {
        const double* g = dt.g + e * kDirGeo;
        adz = g[DG_ADZ]; rdz = g[DG_RDZ]; dx = g[DG_DX];
        dnp = g[DG_DN]; rdnp = g[DG_DN + 1]; dnn = g[DG_DN + 2]; rdnn = g[DG_DN + 3];
        fl = (uint32_t)__double_as_longlong(g[DG_FLAGS]);
    };
    load();
    while (nev < Kmax) {
        const bool up = neg == 0;
        const double dn = up ? dnp : dnn, rdn = up ? rdnp : rdnn;
        // candidates in next_surface's order: the face ahead, end face 0, the
        // mirror ahead (the cell's left one for n.d > 0, else its right one),
        // end face 1; an earlier one keeps a tie
        const int mm = dn > 0.0 ? cell - 1 : cell;
        const bool hm = (unsigned)mm < (unsigned)M && last != mm && dn != 0.0;
        const double hp = pl.h[hm ? mm : 0];
        double best = dir_quot(up ? T - pz : pz, adz, rdz);
        const int face = up ? SURF_TOP : SURF_BOTTOM;
        int hit = last != face ? face : -1;
        const double tm = dir_quot(hp - (nx * px + nz * pz), dn, rdn);
        if (cell == 0 && dx < 0.0 && last != SURF_END0) {
            const double te = dir_quot(0.0 - px, dx, dt.g[e * kDirGeo + DG_RDX]);
            if (hit < 0 || te < best) { best = te; hit = SURF_END0; }
        }
        if (hm && (hit < 0 || tm < best)) { best = tm; hit = mm; }
        if (cell == M && dx > 0.0 && last != SURF_END1) {
            const double te = dir_quot(pl.Lx - px, dx, dt.g[e * kDirGeo + DG_RDX]);
            if (hit < 0 || te < best) { best = te; hit = SURF_END1; }
        }
        if (hit < 0 || hit >= SURF_END0) {
            if (hit >= 0) { o.cat = CAT_END; ++nev; }    // else CAT_LOST
            break;
        }
        px = px + best * dx;
        py = py + best * dy;
        pz = pz + best * (up ? adz : -adz);
        ++nev;
        last = hit;
        if (hit >= SURF_TOP) {
            pz = up ? T : 0.0;
            if (!(fl & kDirTir)) {
                o.cat = up ? CAT_EYEBOX : CAT_LEAK;      // the bin decides below
                break;
            }
            neg ^= 1;
            ++nt;
        } else {
            if (!((fl >> (17 + neg)) & 1u)) { o.off = true; break; }
            const int k = nh & 3;
            if (k == 0 && nh >= 4) {
                if (nh == 4) wa = wb;
                else wa = philox10(id0, id1, (uint32_t)(nh >> 2), 1u, sc.key0, key1);
            }
            const uint32_t word = (k & 2) ? ((k & 1) ? wa.w : wa.z) : ((k & 1) ? wa.y : wa.x);
            const int refl = word < pl.thr[hit] ? 1 : 0;
            on_hit(nh, dt.g + e * kDirGeo + DG_KAP + neg, hit_word(hit, dn < 0.0 ? 1 : 0, refl, neg, e, nt));
            on_hit.branch(hit, refl != 0);
            nt = 0;
            ++nh;
            if (refl) {
                const int c = (int)(fl >> (8 * neg)) & 255;
                if (c == kDirOff) { o.off = true; break; }
                e = c >> 1;
                neg = c & 1;
                load();
            } else {
                cell += hit == cell ? 1 : -1;
            }
        }
    }
    if (o.cat == CAT_LOST && nev >= Kmax && !o.off) o.cat = CAT_TRUNC;
    if (o.cat == CAT_EYEBOX) {
        const double* f = dt.f + e * kDirFld;
        o.bin = eyebox_cell(sc, pl, px + f[DF_EX], py + f[DF_EY]);
        if (o.bin < 0) o.cat = CAT_MISS;
    }
    o.nev = nev; o.nh = nh; o.e = e; o.neg = neg; o.nt = nt;
}

// ------------------------------------------------------------- field pass
// The field along the face basis of the ray's state.
struct FaceSp { cd s, p; };

// Rotate a field between the face basis (s, p) and the mirror basis
// (c s + d p, c p - d s), and back.
__device__ inline FaceSp to_mirror(const FaceSp& a, double c, double d)
{
    FaceSp b;
    b.s = mk(fma(c, a.s.re, d * a.p.re), fma(c, a.s.im, d * a.p.im));
    b.p = mk(fma(c, a.p.re, -(d * a.s.re)), fma(c, a.p.im, -(d * a.s.im)));
    return b;
}
__device__ inline FaceSp to_face(const FaceSp& b, double c, double d)
{
    FaceSp a;
    a.s = mk(fma(c, b.s.re, -(d * b.p.re)), fma(c, b.s.im, -(d * b.p.im)));
    a.p = mk(fma(d, b.s.re, c * b.p.re), fma(d, b.s.im, c * b.p.im));
    return a;
}
__device__ inline double sp_norm2(const FaceSp& a)
{
    return fma(a.s.re, a.s.re, a.s.im * a.s.im) + fma(a.p.re, a.p.re, a.p.im * a.p.im);
}
