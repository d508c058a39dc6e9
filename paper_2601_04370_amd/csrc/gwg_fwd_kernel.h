// Forward trace kernel.  Included by gwg_kernels.hip inside namespace gwg.
//
// Two-pass intersection (Methods, memory-saving strategies): the path of a
// ray (surfaces, branch decisions) does not depend on the coatings, so a
// wave takes its rays of a work item in pools of up to sc.pool rounds of 64:
//   1. a geometry-only walk of every ray of the pool writes each hit's kappa
//      and word (mirror, side, branch) to the ray's column of the wave's hit
//      queue and finds the ray's fate;
//   2. the pool's rays are ordered by the length of their field pass (a
//      counting sort), and the hits get their thin-film coefficients:
//      - per hit: the hits are solved densely in batches of 64, one per
//        lane, so every lane of the wave runs the same layer loop whatever
//        the path lengths;
//      - keyed (memoized solves and the angle table, collimated beams): a
//        hit's coefficients depend only on its direction state, mirror and
//        side, and the rays of an item share a few dozen such keys; the
//        workgroup solves (or interpolates) each key of the item once, into
//        LDS, with the per-hit operations, so with the per-hit bits;
//   3. the field passes, 64 rays at a time in that order, run over the
//      ray's hits: a collimated ray's field is two complex numbers along the
//      face basis of its direction state (gwg_dirs.h), its total reflections
//      between hits a power of the state's (r_s, r_p), so nothing of the
//      geometry is walked again.  The weight goes to the eyebox bins;
//   4. with ADJ (a gradient will follow), every ray that reached the eyebox
//      runs the reverse field sweep over its hits (the incoming field's
//      mirror components are on the tape) and stores one adjoint entry per
//      mirror hit (AdjStore) for the backward.
// Rays whose direction is drawn per ray, and the few that leave the
// direction table, take the general walks instead (walk_ray, with the tape
// of every event and reverse_sweep): the same paths, branches and bins.

// Thin-film coefficients of one hit for this lane (fills the lane's slot table).
template <int MODE, class SL, class Stks>
__device__ inline Coef4 hit_solve(const SceneDev& sc, const PointLds& pl, const Stks& stks,
                                  const SL& sl, int m, bool front, double kappa,
                                  bool* used_fp64, double* ck = nullptr, int64_t ckb = 8)
{
    bool hyp = false;                       // an evanescent lossless slot at this kappa
    for (int s = 0; s < sc.n_slots; ++s) {
        double P[NPF];
        slot_params(pl.slotN[2 * s], pl.slotN[2 * s + 1], kappa, pl.k0, P);
        sl.put(s, P);
        hyp |= !((sc.slot_complex >> s) & 1u) && P[0] < 0.0;
    }
    const bool circ = __ballot(hyp) == 0ull;
    const double z0 = pl.ng * pl.ng - kappa * kappa;
    const double q0 = sqrt(z0 > kTinyZ ? z0 : kTinyZ);
    const double eta0s = q0, eta0p = pl.ng * pl.ng / q0;
    const int L = pl.nlay[m];
    const auto stk = stks.mirror(m);
    const bool fp64 = (MODE == GWG_FP64) || (MODE == GWG_FP32_MIXED && near_critical(pl, sc.n_slots, kappa));
    *used_fp64 = fp64;
    if (fp64)
        return tmm_solve<double>(stk, L, front, sl, sc.slot_complex, pl.k0, eta0s, eta0p,
                                 mk(eta0s, 0.0), mk(eta0p, 0.0), mk(1.0, 0.0), circ, MODE == GWG_FP64 ? ck : nullptr,
                                 ckb, ck_interval(hyp));
    return tmm_solve<float>(stk, L, front, sl, sc.slot_complex, pl.k0, eta0s, eta0p,
                            mk(eta0s, 0.0), mk(eta0p, 0.0), mk(1.0, 0.0), circ);
}

// Dense hit p (the wave's hits in ray order) belongs to the largest lane
// whose exclusive prefix sum of hit counts (off) is <= p: lanes without hits
// share the next lane's offset and lose the search to it.  Returns its queue
// slot.  Called by all lanes of the wave (shuffles).
__device__ inline int dense_slot(int p, int off, int)
{
    int l = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const int c = l + step;
        if (__shfl(off, c, 64) <= p) l = c;
    }
    return hq_slot(l, p - __shfl(off, l, 64));
}

// Solve the wave's `total` queued hits in batches of 64 (one per lane);
// off: this lane's exclusive prefix sum of hit counts.
template <int MODE, class SL, class Stks>
__device__ inline void solve_hits(const SceneDev& sc, const PointLds& pl, const Stks& stks,
                                  const SL& sl, const HitQueue& hq, int total,
                                  int off, unsigned long long* n_fp64, unsigned long long* n_lay)
{
    const int lane = wave_lane();
    for (int b = 0; b < total; b += 64) {
        const int p = b + lane;
        const int pp = p < total ? p : total - 1;
        const int q = dense_slot(pp, off, sc.Kmax);
        if (p < total) {
            const double kappa = hq.kappa(q);
            const int meta = hq.meta(q);
            const int m = meta & 255;
            bool u64 = false;
            const Coef4 c = hit_solve<MODE>(sc, pl, stks, sl, m, (meta >> 8) & 1, kappa, &u64);
            hq.put_coef(q, c);
            *n_fp64 += u64 ? 1ull : 0ull;
            *n_lay += (unsigned long long)pl.nlay[m];
        }
    }
}

struct NoHit {
    __device__ void operator()(int, double, int) const {}
    __device__ void branch(int, bool) const {}
};
struct NoCoef {
    static constexpr bool kStoredBranch = false;
    __device__ bool refl(int) const { return false; }
    __device__ Coef4 operator()(int, double, double, double, int, bool) const
    {
        Coef4 c;
        c.rs = c.rp = c.ts = c.tp = mk(0.0, 0.0);
        return c;
    }
};
struct PutHit {
    HitQueue q;
    int off;
    __device__ void operator()(int h, double kappa, int meta) const { q.put(hq_slot(off, h), kappa, meta); }
    __device__ void branch(int, bool) const {}
};
// Coefficients of the ray's hit h from its queue entry.
struct GetCoef {
    HitQueue q;
    int off;
    static constexpr bool kStoredBranch = true;   // the geometry walk stored the branch in the meta word
    __device__ bool refl(int h) const { return (((int)q.base[q.cap + hq_slot(off, h)]) >> 9) & 1; }
    __device__ Coef4 operator()(int h, double, double, double, int, bool) const { return q.coef(hq_slot(off, h)); }
};

__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);      // this wave's LDS operations have completed (lgkmcnt = 0)
    __builtin_amdgcn_wave_barrier();
}

// ----------------------------------------------------- pooled rounds
// A wave's queue holds the hits of a pool of rounds: ncol = 64 sc.pool
// columns (one per ray) of Kmax slots, hit h of column col in slot
// h * ncol + col of each field.  The geometry walk writes fields 0 (kappa)
// and 1 (word), the per-hit solves read them in the order of field 8 and
// write each hit's taken coefficients (c_s, c_p: fields 2-5) and word (field
// 6) in the slot of the ray's place in the field-pass order (column pos), so
// that the lanes of a field pass read adjacent slots.  Field 7: the
// checkpoint slot of the hit's adjoint entry, or -1.
constexpr int kPoolFields = 9;
constexpr int kSortBins = 128;                      // field-pass length classes
constexpr int kStatCols = 16;                       // columns of the statistics' LDS counters

// doubles of global scratch per wave: the hit queue, then per column two
// 64-bit words (carried data, fate) and three 32-bit words (bin, place in
// the order, column at each place)
__host__ __device__ inline int64_t fwd_wave_doubles(const SceneDev& sc)
{
    return (int64_t)kPoolFields * 64 * sc.pool * sc.Kmax + 4 * 64 * sc.pool;
}

// Writes the ray's hits to its column.  Also counts the hits whose kappa^2
// exceeds kap2 (they may meet an evanescent layer) in *ne and marks hits
// h < 64 of them in bit h of *evm.
struct PutHitP {
    HitQueue q;
    int col, ncol;
    double kap2;
    int* ne;
    unsigned long long* evm;
    __device__ void operator()(int h, double kappa, int word) const
    {
        q.put(h * ncol + col, kappa, word);
        if (kappa * kappa > kap2) {
            ++*ne;
            if (h < 64) *evm |= 1ull << h;
        }
    }
    __device__ void branch(int, bool) const {}
};
// Keyed forwards: writes the hits and marks their keys in the item's LDS
// bit set (the read first: most hits find their key marked).
struct PutHitK {
    HitQueue q;
    int col, ncol, M;
    uint32_t* used;
    __device__ void operator()(int h, double kappa, int word) const
    {
        q.put(h * ncol + col, kappa, word);
        const int key = hit_key(word, M);
        if (!((used[key >> 5] >> (key & 31)) & 1u)) atomicOr(&used[key >> 5], 1u << (key & 31));
    }
    __device__ void branch(int, bool) const {}
};
// The general field walk's coefficients of the ray at place pos of the
// order: the taken pair (c_s, c_p) returned as both the reflected and the
// transmitted one, and the branch.
struct GetCoefP {
    HitQueue q;
    int pos, ncol;
    static constexpr bool kStoredBranch = true;
    __device__ bool refl(int h) const { return ((int)q.base[6 * (int64_t)q.cap + h * ncol + pos] >> 9) & 1; }
    __device__ Coef4 operator()(int h, double, double, double, int, bool) const
    {
        const double* b = q.base + 2 * (int64_t)q.cap + h * ncol + pos;
        const int64_t c = q.cap;
        Coef4 o;
        o.rs = o.ts = mk(b[0], b[c]);
        o.rp = o.tp = mk(b[2 * c], b[3 * c]);
        return o;
    }
};

// A hit's taken coefficients and word to the slot of its ray's place.
__device__ inline void put_taken(const HitQueue& hq, int slot, const Coef4& c, int word)
{
    const bool rf = (word >> 9) & 1;
    double* o = hq.base + 2 * (int64_t)hq.cap + slot;
    const int64_t cc = hq.cap;
    const cd cs = rf ? c.rs : c.ts, cp = rf ? c.rp : c.tp;
    o[0] = cs.re; o[cc] = cs.im; o[2 * cc] = cp.re; o[3 * cc] = cp.im;
    o[4 * cc] = (double)word;
}

// Solve a pool's ne + nc queued hits in batches of 64 (one per lane): field
// 8 lists the possibly evanescent hits' slots from its front (positions
// 0 .. ne-1) and the others' from its back (cap-1 down to cap-nc), so the
// batches of the second kind take the circular-only sweep.  colpos[col]:
// the place of column col in the field-pass order, where the hit's taken
// coefficients go.  ck (non-null): the checkpoint store; a hit whose field
// 7 holds a slot c >= 0 stores its sweep checkpoints there.
template <int MODE, class SL, class Stks>
__device__ inline void solve_pool(const SceneDev& sc, const PointLds& pl, const Stks& stks, const SL& sl,
                                  const HitQueue& hq, int ncol, const int32_t* colpos, int ne, int nc,
                                  unsigned long long* n_fp64, unsigned long long* n_lay, double* ck, int64_t ck_total)
{
    const int lane = wave_lane();
    const int total = ne + nc;
    const double* ord = hq.base + 8 * (int64_t)hq.cap;
    for (int b = 0; b < total; b += 64) {
        const int p = b + lane;
        if (p < total) {
            const int q = (int)ord[p < ne ? p : hq.cap - 1 - (p - ne)];
            const double kappa = hq.kappa(q);
            const int word = hq.meta(q);
            const int m = word & 255;
            bool u64 = false;
            double* ckp = nullptr;
            if (ck) {
                const double c = hq.base[7 * (int64_t)hq.cap + q];
                if (c >= 0.0) ckp = ck + (int64_t)c * 8;
            }
            const Coef4 c = hit_solve<MODE>(sc, pl, stks, sl, m, (word >> 8) & 1, kappa, &u64, ckp, 8 * ck_total);
            const int h = q / ncol, col = q - h * ncol;
            put_taken(hq, h * ncol + colpos[col], c, word);
            *n_fp64 += u64 ? 1ull : 0ull;
            *n_lay += (unsigned long long)pl.nlay[m];
        }
    }
}

// ------------------------------------------------------- keyed coefficients
// Key of a hit of a ray on the direction table: (state, sign of z, mirror);
// the side follows from the direction.
__host__ __device__ inline int key_words(int M) { return (2 * kDirMax * M + 31) / 32; }

// One item's keys in LDS.
struct KeyLds {
    uint32_t* used;              // [key_words] keys some hit of the item has
    uint32_t* have;              // [key_words] keys with coefficients
    uint8_t* slot;               // [2 kDirMax M] a key's slot
    uint16_t* key;               // [kFwdMemoKeys] the slots' keys
    int* n;                      // slots in use; [1]: the table overflowed
    double* coef;                // [kFwdMemoKeys][8] r_s, r_p, t_s, t_p
};

__host__ __device__ inline int key_smem_bytes(int M)
{
    return align16(8 * key_words(M)) + align16(2 * kDirMax * M) + align16(2 * kFwdMemoKeys) + 16 + 64 * kFwdMemoKeys;
}

__device__ inline KeyLds key_lds(unsigned char* mem, int M)
{
    KeyLds k;
    k.coef = (double*)mem;
    k.n = (int*)(mem + 64 * kFwdMemoKeys);
    k.key = (uint16_t*)(mem + 64 * kFwdMemoKeys + 16);
    k.slot = mem + 64 * kFwdMemoKeys + 16 + align16(2 * kFwdMemoKeys);
    k.used = (uint32_t*)(k.slot + align16(2 * kDirMax * M));
    k.have = k.used + key_words(M);
    return k;
}

// Called by the whole block: gives the keys marked since the last call slots
// and coefficients, solved by solve(kappa, mirror, front) (one per lane).
// More than cap keys in an item: sets the overflow flag (and the block goes
// on hit by hit).  Returns false on overflow.
template <class Solve>
__device__ inline bool key_resolve(const KeyLds& kl, const DirLds& dt, int M, int cap, Solve solve)
{
    const int lane = wave_lane(), wave = (int)threadIdx.x / 64, n_waves = (int)blockDim.x / 64;
    __syncthreads();
    const int n0 = kl.n[0];
    __syncthreads();
    if (wave == 0) {
        // one word of the bit set per lane (at most 64 words: 16 mirrors)
        const int nw = key_words(M);
        uint32_t fresh = lane < nw ? kl.used[lane] & ~kl.have[lane] : 0u;
        int total;
        int at = n0 + wave_excl_scan(__popc(fresh), &total);
        if (n0 + total > cap) {
            if (lane == 0) kl.n[1] = 1;
        } else {
            if (lane < nw) kl.have[lane] |= fresh;
            while (fresh) {
                const int k = lane * 32 + __ffs((int)fresh) - 1;
                fresh &= fresh - 1u;
                kl.slot[k] = (uint8_t)at;
                kl.key[at++] = (uint16_t)k;
            }
            if (lane == 0) kl.n[0] = n0 + total;
        }
    }
    __syncthreads();
    if (kl.n[1]) return false;
    const int n1 = kl.n[0];
    for (int u = n0 + wave * 64 + lane; u < n1; u += 64 * n_waves) {
        const int k = kl.key[u], es = k / M, m = k - es * M;
        const double* g = dt.g + (es >> 1) * kDirGeo;
        const Coef4 c = solve(g[DG_KAP + (es & 1)], m, g[DG_DN + 2 * (es & 1)] < 0.0);
        double* o = kl.coef + 8 * u;
        o[0] = c.rs.re; o[1] = c.rs.im; o[2] = c.rp.re; o[3] = c.rp.im;
        o[4] = c.ts.re; o[5] = c.ts.im; o[6] = c.tp.re; o[7] = c.tp.im;
    }
    __syncthreads();
    return true;
}

// ------------------------------------------------------------ field passes
// The taken coefficients of a table ray's hit h, in two steps so that the
// loads of the next hit run ahead: word(h), then coef(h, word, ...).
struct HitCoefs {                      // per-hit solves: the queue's slots at place pos
    HitQueue q;
    int pos, ncol;
    __device__ int word(int h) const { return (int)q.base[6 * (int64_t)q.cap + h * ncol + pos]; }
    __device__ void coef(int h, int, cd& cs, cd& cp) const
    {
        const double* b = q.base + 2 * (int64_t)q.cap + h * ncol + pos;
        const int64_t c = q.cap;
        cs = mk(b[0], b[c]);
        cp = mk(b[2 * c], b[3 * c]);
    }
};
struct KeyCoefs {                      // keyed: the word in the ray's column, the key's coefficients in LDS
    HitQueue q;
    int col, ncol, M;
    const uint8_t* slot;
    const double* kc;
    __device__ int word(int h) const { return q.meta(h * ncol + col); }
    __device__ void coef(int, int word, cd& cs, cd& cp) const
    {
        const double* b = kc + 8 * slot[hit_key(word, M)] + (((word >> 9) & 1) ? 0 : 4);
        cs = mk(b[0], b[1]);
        cp = mk(b[2], b[3]);
    }
};

// Field of one ray of the table from its birth to its end, over its nh hits
// (lanes without a ray: nh = 0).  Writes the incoming field's mirror
// components of hit h to the tape where tape.mr is set; returns the field at
// the ray's last state, before an exit.
template <class Coefs>
__device__ inline FaceSp dir_field(const PointLds& pl, const DirLds& dt, int pol, int nh, int e_end, int nt_end,
                                   const Coefs& src, const TapeRef& tape)
{
    FaceSp a;
    a.s = mk(pol ? 0.0 : 1.0, 0.0);
    a.p = mk(pol ? 1.0 : 0.0, 0.0);
    auto tir = [&](const double* f, int n) {
        const cd rs = mk(f[DF_RS], f[DF_RS + 1]), rp = mk(f[DF_RP], f[DF_RP + 1]);
        for (int k = 0; k < n; ++k) { a.s = cmul_f(rs, a.s); a.p = cmul_f(rp, a.p); }
    };
    int wd = 0, wn = 0;
    cd cs, cp, ns, np;
    cs = cp = ns = np = mk(0.0, 0.0);
    if (nh > 0) { wn = src.word(0); src.coef(0, wn, ns, np); }
    for (int h = 0; h < nh; ++h) {
        wd = wn; cs = ns; cp = np;
        if (h + 1 < nh) { wn = src.word(h + 1); src.coef(h + 1, wn, ns, np); }
        const int e = (wd >> 11) & 255, neg = (wd >> 10) & 1, m = wd & 255;
        const bool rf = (wd >> 9) & 1;
        const double* f = dt.f + e * kDirFld;
        tir(f, wd >> 19);
        double c = f[DF_ROT + 2 * neg], d = f[DF_ROT + 2 * neg + 1];
        FaceSp b = to_mirror(a, c, d);
        if (tape.mr) tape_put_mirror(tape, h, b.s, b.p);
        const double scale = rf ? pl.sc_r[m] : pl.sc_t[m];
        b.s = cscale(cmul_f(cs, b.s), scale);
        b.p = cscale(cmul_f(cp, b.p), scale);
        if (rf) {
            const unsigned long long fl = (unsigned long long)__double_as_longlong(dt.g[e * kDirGeo + DG_FLAGS]);
            const int ch = (int)(fl >> (8 * neg)) & 255;
            const double* fc = dt.f + (ch >> 1) * kDirFld + DF_ROT + 2 * (ch & 1);
            c = fc[0]; d = fc[1];
        }
        a = to_face(b, c, d);
    }
    tir(dt.f + e_end * kDirFld, nt_end);
    return a;
}

// Reverse field sweep of one ray of the table that left through the exit
// (the adjoint of dir_field and the exit for w = |E|^2): a is the field
// after the exit.  Calls emit(kappa, G_s, G_p, word) for every mirror hit,
// last to first, with the cotangents of reverse_sweep.
template <class Coefs, class Emit>
__device__ inline void dir_reverse(const PointLds& pl, const DirLds& dt, FaceSp a, int nh, int e_end, int nt_end,
                                   const Coefs& src, const TapeRef& tape, Emit emit)
{
    auto tir = [&](const double* f, int n) {
        const cd rs = mk(f[DF_RS], -f[DF_RS + 1]), rp = mk(f[DF_RP], -f[DF_RP + 1]);
        for (int k = 0; k < n; ++k) { a.s = cmul_f(rs, a.s); a.p = cmul_f(rp, a.p); }
    };
    const double* fx = dt.f + e_end * kDirFld;
    a.s = cscale(a.s, fx[DF_XS]);
    a.p = cscale(a.p, fx[DF_XP]);
    tir(fx, nt_end);
    struct Next { int wd; cd cs, cp; double2 t0, t1; } nx;
    nx.wd = 0;
    nx.cs = nx.cp = mk(0.0, 0.0);
    nx.t0 = nx.t1 = make_double2(0.0, 0.0);
    auto fetch = [&](int h) {
        nx.wd = src.word(h);
        src.coef(h, nx.wd, nx.cs, nx.cp);
        const double2* p = (const double2*)(tape.mr + (int64_t)h * (tape.ks / 2));
        nx.t0 = p[0];
        nx.t1 = p[64];
    };
    if (nh > 0) fetch(nh - 1);
    for (int h = nh - 1; h >= 0; --h) {
        const Next ev = nx;
        if (h > 0) fetch(h - 1);
        const int e = (ev.wd >> 11) & 255, neg = (ev.wd >> 10) & 1, m = ev.wd & 255;
        const bool rf = (ev.wd >> 9) & 1;
        const double* g = dt.g + e * kDirGeo;
        const double* f = dt.f + e * kDirFld;
        const double c = f[DF_ROT + 2 * neg], d = f[DF_ROT + 2 * neg + 1];
        double co = c, so = d;
        if (rf) {
            const int ch = (int)((unsigned long long)__double_as_longlong(g[DG_FLAGS]) >> (8 * neg)) & 255;
            const double* fc = dt.f + (ch >> 1) * kDirFld + DF_ROT + 2 * (ch & 1);
            co = fc[0]; so = fc[1];
        }
        const double scale = rf ? pl.sc_r[m] : pl.sc_t[m];
        FaceSp b = to_mirror(a, co, so);
        const cd Gs = cscale(cmul_f(cconj(b.s), mk(ev.t0.x, ev.t0.y)), scale);
        const cd Gp = cscale(cmul_f(cconj(b.p), mk(ev.t1.x, ev.t1.y)), scale);
        emit(g[DG_KAP + neg], Gs, Gp, ev.wd & 1023);
        b.s = cscale(cmul_f(cconj(ev.cs), b.s), scale);
        b.p = cscale(cmul_f(cconj(ev.cp), b.p), scale);
        a = to_face(b, c, d);
        tir(f, ev.wd >> 19);
    }
}

// Persistent workgroups draw work items; each wave handles a strided share
// of the item's rays.  Eyebox bins of the current point accumulate in LDS
// (integer atomics) and are flushed per item with integer global atomics:
// the result does not depend on scheduling.
template <int MODE, bool ADJ, bool TAB, bool MEMO>
__global__ void __launch_bounds__(256, 2) k_trace_fwd(SceneDev sc, uint64_t* __restrict__ q_out,
                                                   uint32_t* __restrict__ c_out,
                                                   unsigned long long* __restrict__ stats,
                                                   gwg_ray_record* __restrict__ rec, int64_t rec_stride,
                                                   int lds_bins, double* __restrict__ scratch, AdjStore st,
                                                   double* __restrict__ tape_scratch)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int B = sc.bins_x * sc.bins_y;
    const int WG = blockDim.x;
    const int n_waves = WG / 64;
    constexpr bool KEYED = TAB || MEMO;
    // slot table: all five values per lane, except with the keyed
    // coefficients, which solve few hits and keep their table in LDS
    using SlotTable = typename std::conditional<MEMO, LaneSlots3, LaneSlots3x>::type;
    const SmemLayout lay = smem_layout(sc.M, sc.Lmax, sc.n_slots, WG, B, lds_bins != 0, 0, SlotTable::kPer, true);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    LayerRec* s_rec = (LayerRec*)(smem + lay.off_thk);
    const RecStacks stks = { s_rec, sc.Lmax };
    double* s_sp = (double*)(smem + lay.off_sp);
    unsigned long long* s_q = (unsigned long long*)(smem + lay.off_q);
    uint32_t* s_c = (uint32_t*)(smem + lay.off_c);
    unsigned long long* s_st = (unsigned long long*)(smem + lay.off_st);
    // statistics: per-ray sums in kStatCols columns per word, so that the
    // lanes of a wave add to different addresses
    unsigned long long* s_col = (unsigned long long*)(smem + lay.total);        // power, events, mirror hits
    double* s_dir = (double*)(s_col + (NCAT + 2) * kStatCols);
    unsigned char* s_key = (unsigned char*)s_dir + dir_smem_bytes(sc);
    const bool dirs = sc.dirs != nullptr;
    const int tid = threadIdx.x, wave = tid / 64, lane = wave_lane();
    const int64_t gwave = (int64_t)blockIdx.x * n_waves + wave;
    const int cap = 64 * sc.pool * sc.Kmax;                // queue slots of a wave (a pool of rounds)
    const HitQueue hq = { scratch + gwave * fwd_wave_doubles(sc), cap };
    const SlotTable sl = { slot_lane_base(s_sp, sc.n_slots, SlotTable::kPer, tid), pl->nsq, pl->pxy };
    const double wscale = ldexp(1.0, sc.fp_shift), wcap = ldexp(1.0, 40), pscale = 16777216.0;
    for (int k = tid; k < ST_WORDS; k += WG) s_st[k] = 0ull;
    for (int k = tid; k < (NCAT + 2) * kStatCols; k += WG) s_col[k] = 0ull;
    unsigned long long n_fp64 = 0, n_lay = 0;
    const TapeRef tape = tape_lane(tape_scratch, sc.Kmax, (int64_t)gridDim.x * n_waves, gwave, lane);
    KeyLds kl{};
    if constexpr (KEYED) kl = key_lds(s_key, sc.M);
    const int key_cap = MEMO ? sc.memo : kFwdMemoKeys;
    double t_gmax = 0.0;                                 // largest cotangent component (angle table)
    unsigned long long t_ne = 0;                         // cotangent pairs emitted (angle table)

    for (int64_t it = draw_item(stats + ST_NEXT0); it < sc.n_items; it = draw_item(stats + ST_NEXT0)) {
        const int64_t item = sc.fwd_order ? (int64_t)sc.fwd_order[it] : it;
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, item, &point, &d, &l, &f, &i0, &i1);
        stage_point(sc, d, l, f, pl, nullptr, nullptr, TAB ? nullptr : s_rec, SlotTable::kPer);
        DirLds dt{};
        if (dirs) dt = stage_dirs(sc, (int64_t)l * sc.F + f, s_dir);
        int64_t n_work = 0;                               // this wave's mirror hits in this item (uniform)
        if (lds_bins)
            for (int k = tid; k < B; k += WG) { s_q[k] = 0ull; s_c[k] = 0u; }
        if constexpr (KEYED) {
            for (int k = tid; k < 2 * key_words(sc.M); k += WG) kl.used[k] = 0u;
            if (tid < 2) kl.n[tid] = 0;
        }
        __syncthreads();
        const int64_t base = point * sc.N;
        uint64_t* gq = q_out + point * B;
        uint32_t* gc = c_out + point * B;
        int64_t n_ent = 0;                                // this wave's entries in this item (uniform)
        bool keyed = KEYED && dirs;                       // the item's hits take their keys' coefficients (uniform)
        const int64_t ent0 = (item * st.waves + wave) * st.cap_w;
        const double* tab_dl = TAB ? sc.table + (int64_t)(d * sc.n_lsel + l) * sc.M * 2 * sc.table_n * 8 : nullptr;
        // coefficients of one hit (one per lane)
        auto one_hit = [&](double kappa, int m, bool front) {
            if constexpr (TAB) {
                return table_coef(tab_dl, sc.table_n, m, front, kappa, pl->ng);
            } else {
                bool u64 = false;
                const Coef4 c = hit_solve<MODE>(sc, *pl, stks, sl, m, front, kappa, &u64);
                n_fp64 += u64 ? 1ull : 0ull;
                n_lay += (unsigned long long)pl->nlay[m];
                return c;
            }
        };
        // Weight, eyebox scatter, statistics and record of a ray that ended
        auto finish = [&](bool active, int64_t id, int cat, int bin, int nev, int nh, double w, double w_in) {
            if (active) {
                const int cl = lane & (kStatCols - 1);
                atomicAdd(&s_col[NCAT * kStatCols + cl], (unsigned long long)nev);
                atomicAdd(&s_col[(NCAT + 1) * kStatCols + cl], (unsigned long long)nh);
                const double pw = w * pscale;
                atomicAdd(&s_col[cat * kStatCols + cl], (unsigned long long)rint(pw < wcap ? pw : wcap));
                if (cat == CAT_EYEBOX || cat == CAT_MISS) {
                    const double pr = (w_in - w) * pscale;
                    if (pr > 0.0)
                        atomicAdd(&s_col[CAT_FACE_R * kStatCols + cl], (unsigned long long)rint(pr < wcap ? pr : wcap));
                }
                if (cat == CAT_EYEBOX) {
                    double u = w * wscale;
                    if (!(u <= wcap)) { u = (u > wcap) ? wcap : 0.0; atomicAdd(&s_st[ST_SAT], 1ull); }
                    const unsigned long long qv = (unsigned long long)rint(u);
                    if (lds_bins) { atomicAdd(&s_q[bin], qv); atomicAdd(&s_c[bin], 1u); }
                    else { atomicAdd((unsigned long long*)&gq[bin], qv); atomicAdd(&gc[bin], 1u); }
                }
                if (rec && (id % rec_stride) == 0) {
                    gwg_ray_record* q = rec + id / rec_stride;
                    q->bin = cat == CAT_EYEBOX ? bin : -1;
                    q->category = cat;
                    q->n_events = nev;
                    q->n_prma = nh;
                    q->w = w;
                }
            }
            for (int c = 0; c < CAT_FACE_R; ++c) {
                const int n = __popcll(__ballot(active && cat == c));
                if (n && lane == c) atomicAdd(&s_st[ST_CAT + c], (unsigned long long)n);
            }
        };
        // one adjoint entry at position k of the wave's region
        auto put_entry = [&](int64_t k, double kappa, cd Gs, cd Gp, int64_t meta) {
            if constexpr (TAB) {
                const double a = fmax(fmax(fabs(Gs.re), fabs(Gs.im)), fmax(fabs(Gp.re), fabs(Gp.im)));
                t_gmax = a > t_gmax ? a : t_gmax;
                ++t_ne;
            }
            if (k < st.cap_w) {
                const int64_t e = ent0 + k;
                st.ent[e] = kappa;
                st.ent[1 * st.total + e] = Gs.re;
                st.ent[2 * st.total + e] = Gs.im;
                st.ent[3 * st.total + e] = Gp.re;
                st.ent[4 * st.total + e] = Gp.im;
                st.ent[5 * st.total + e] = (double)meta;
            }
        };
        const int ncol = 64 * sc.pool;
        const int64_t first = i0 + (int64_t)wave * 64;
        const int n_rounds = first < i1 ? (int)((i1 - first + WG - 1) / WG) : 0;      // uniform
        const int n_rounds0 = (int)((i1 - i0 + WG - 1) / WG);                          // wave 0's, the most
        // the ordering's class counts sit in this wave's slot tables, which
        // only the solves use (each hit's solve fills its lane's table first)
        uint32_t* s_hist = (uint32_t*)(s_sp + (int64_t)wave * sc.n_slots * SlotTable::kPer * kSlotLanes);
        int64_t* colinfo = (int64_t*)(hq.base + (int64_t)kPoolFields * cap);        // [ncol] carried data
        int64_t* colfate = colinfo + ncol;                                          // [ncol] fate
        int32_t* colbin = (int32_t*)(colfate + ncol);                               // [ncol] bin
        int32_t* colpos = colbin + ncol;                                            // [ncol] place of a column
        int32_t* colord = colpos + ncol;                                            // [ncol] column at a place
        const bool cks = ADJ && !KEYED && MODE == GWG_FP64 && st.ck != nullptr;
        for (int r0 = 0; r0 < (KEYED ? n_rounds0 : n_rounds); r0 += sc.pool) {
            const int nr = max(0, n_rounds - r0 < sc.pool ? n_rounds - r0 : sc.pool);
            int n_e = 0, n_c = 0;                         // the pool's possibly evanescent / other hits (uniform)
            bool any_off = false;                         // some ray of the pool walks in general (uniform)
            for (int rr = 0; rr < nr; ++rr) {
                const int col = rr * 64 + lane;
                const int64_t i = first + (int64_t)(r0 + rr) * WG + lane;
                const bool active = i < i1;
                DirFate o;
                o.cat = CAT_LOST; o.bin = -1; o.nev = o.nh = o.e = o.neg = o.nt = o.pol = 0;
                o.off = false;
                int ne = 0;
                unsigned long long evm = 0ull;             // bit h: hit h may meet an evanescent layer
                if (active) {
                    if (dirs) {
                        if constexpr (KEYED) dir_walk(sc, *pl, dt, base + i, PutHitK{ hq, col, ncol, sc.M, kl.used }, o);
                        else dir_walk(sc, *pl, dt, base + i, PutHitP{ hq, col, ncol, pl->kap2_evan, &ne, &evm }, o);
                    } else {
                        o.off = true;
                    }
                    if (o.off) {
                        Ray r;
                        Outcome oc;
                        TapeRef none = { nullptr, nullptr, 0 };
                        ne = 0;
                        evm = 0ull;
                        ray_birth(sc, *pl, base + i, r);
                        walk_ray<false, false>(sc, *pl, r, oc, PutHitP{ hq, col, ncol, pl->kap2_evan, &ne, &evm },
                                               NoCoef{}, none, nullptr);
                        o.cat = oc.cat; o.bin = oc.bin; o.nev = r.nev; o.nh = r.nprma;
                    }
                }
                any_off |= __ballot(o.off) != 0ull;
                const int nh = o.nh;
                const bool to_eyebox = active && o.cat == CAT_EYEBOX;              // fixed by geometry alone
                int total;
                (void)wave_excl_scan(nh, &total);
                n_work += total;
                // the ray's adjoint entries (rays bound for the eyebox) start
                // at kent of the wave's region; with a checkpoint store its
                // hits learn their entries' checkpoint slots
                int64_t kent = 0;
                if (ADJ) {
                    int etot;
                    const int eoff = wave_excl_scan(to_eyebox ? nh : 0, &etot);
                    kent = n_ent + eoff;
                    if (cks)
                        for (int h = 0; h < nh; ++h) {
                            const int64_t k = kent + (nh - 1 - h);
                            double c = -1.0;
                            if (to_eyebox && k < st.ck_cap) c = (double)((item * st.waves + wave) * st.ck_cap + k);
                            hq.base[7 * (int64_t)cap + h * ncol + col] = c;
                        }
                    n_ent += etot;
                }
                if constexpr (!KEYED) {
                    // solve order: the hits that may meet an evanescent layer
                    // from the front of field 8, the others from its back
                    int te, tc;
                    const int eo = wave_excl_scan(ne, &te);
                    const int co = wave_excl_scan(nh - ne, &tc);
                    int pe = n_e + eo, pc = n_c + co;
                    for (int h = 0; h < nh; ++h) {
                        const int q = h * ncol + col;
                        bool ev;
                        if (h < 64) {
                            ev = (evm >> h) & 1ull;
                        } else {
                            const double k = hq.kappa(q);
                            ev = k * k > pl->kap2_evan;
                        }
                        const int pos = ev ? pe++ : cap - 1 - pc++;
                        hq.base[8 * (int64_t)cap + pos] = (double)q;
                    }
                    n_e += te;
                    n_c += tc;
                }
                // field-pass length class (0: no ray): hits, or events of a
                // general walk, twice with a reverse sweep to follow
                const int len = o.off ? o.nev : nh;
                const int cost = len + (to_eyebox ? len : 0);
                const int key = active ? 1 + (cost < kSortBins - 2 ? cost : kSortBins - 2) : 0;
                colinfo[col] = (kent << 16) | (int64_t)(key << 1) | (to_eyebox ? 1 : 0);
                colfate[col] = (int64_t)o.cat | (int64_t)(o.off ? 1 : 0) << 3 | (int64_t)o.pol << 4 | (int64_t)nh << 5 |
                               (int64_t)o.nev << 14 | (int64_t)o.e << 23 | (int64_t)o.nt << 31;
                colbin[col] = o.bin;
            }
            __threadfence_block();
            // the field-pass order: the pool's columns by length class,
            // longest first (a counting sort)
            for (int k = lane; k < kSortBins; k += 64) s_hist[k] = 0u;
            wave_lds_sync();
            for (int rr = 0; rr < nr; ++rr) {
                const int key = (int)((colinfo[rr * 64 + lane] >> 1) & 255);
                atomicAdd(&s_hist[key], 1u);
            }
            wave_lds_sync();
            {
                // bin offsets in decreasing class order (two bins a lane)
                const int b0 = kSortBins - 1 - 2 * lane, b1 = b0 - 1;
                const int h0 = (int)s_hist[b0], h1 = (int)s_hist[b1];
                int tot;
                const int ex = wave_excl_scan(h0 + h1, &tot);
                s_hist[b0] = (uint32_t)ex;
                s_hist[b1] = (uint32_t)(ex + h0);
            }
            wave_lds_sync();
            for (int rr = 0; rr < nr; ++rr) {
                const int col = rr * 64 + lane;
                const int key = (int)((colinfo[col] >> 1) & 255);
                const int pos = (int)atomicAdd(&s_hist[key], 1u);
                colpos[col] = pos;
                colord[pos] = col;
            }
            wave_lds_sync();                              // the slot tables are the solves' again
            __threadfence_block();
            if constexpr (KEYED) {
                if (keyed) keyed = key_resolve(kl, dt, sc.M, key_cap, one_hit);
                if (!keyed || any_off) {
                    // hit by hit, each lane its own column's (rays off the
                    // direction table, or every ray without keys)
                    for (int rr = 0; rr < nr; ++rr) {
                        const int col = rr * 64 + lane;
                        const int64_t fate = colfate[col];
                        const int nh = (!keyed || ((fate >> 3) & 1)) ? (int)(fate >> 5) & 511 : 0;
                        const int pos = colpos[col];
                        for (int h = 0; h < nh; ++h) {
                            const int word = hq.meta(h * ncol + col);
                            const Coef4 c = one_hit(hq.kappa(h * ncol + col), word & 255, (word >> 8) & 1);
                            put_taken(hq, h * ncol + pos, c, word);
                        }
                    }
                    __threadfence_block();
                }
            } else {
                solve_pool<MODE>(sc, *pl, stks, sl, hq, ncol, colpos, n_e, n_c, &n_fp64, &n_lay,
                                 cks ? st.ck : nullptr, st.ck_total);
                __threadfence_block();
            }
            for (int s2 = 0; s2 < nr; ++s2) {
                const int pos = s2 * 64 + lane;
                const int col = colord[pos];
                const int64_t info = colinfo[col], fate = colfate[col];
                const int64_t i = first + (int64_t)(r0 + col / 64) * WG + (col & 63);
                const int64_t id = base + i;
                const bool active = ((info >> 1) & 255) != 0, eye = (info & 1) != 0, off = (fate >> 3) & 1;
                const int64_t kent = info >> 16;
                int cat = (int)(fate & 7), bin = colbin[col], nev = (int)(fate >> 14) & 511, nh = (int)(fate >> 5) & 511;
                const int64_t meta_bin = (int64_t)bin << 10;
                double w = 0.0, w_in = 0.0;
                const int e_end = (int)(fate >> 23) & 255, nt_end = (int)(fate >> 31) & 511;
                auto table_ray = [&](const auto& src) {
                    const TapeRef rt = { nullptr, ADJ && eye ? tape.mr : nullptr, tape.ks };
                    FaceSp a = dir_field(*pl, dt, (int)(fate >> 4) & 1, nh, e_end, nt_end, src, rt);
                    w = w_in = sp_norm2(a);
                    if (cat == CAT_EYEBOX || cat == CAT_MISS) {
                        const double* fx = dt.f + e_end * kDirFld;
                        a.s = cscale(a.s, fx[DF_XS]);
                        a.p = cscale(a.p, fx[DF_XP]);
                        w = sp_norm2(a);
                    }
                    if (ADJ && eye) {
                        int64_t k = kent;
                        dir_reverse(*pl, dt, a, nh, e_end, nt_end, src, tape, [&](double kappa, cd Gs, cd Gp, int meta) {
                            put_entry(k++, kappa, Gs, Gp, meta_bin | (int64_t)meta);
                        });
                    }
                };
                if (active && !off) {
                    if constexpr (KEYED) {
                        if (keyed) table_ray(KeyCoefs{ hq, col, ncol, sc.M, kl.slot, kl.coef });
                        else table_ray(HitCoefs{ hq, pos, ncol });
                    } else {
                        table_ray(HitCoefs{ hq, pos, ncol });
                    }
                }
                if (__ballot(active && off) != 0ull) {
                    // general field walk, tape of every event and reverse sweep
                    Ray r;
                    Outcome o;
                    o.cat = CAT_LOST;
                    int nt = 0;
                    const bool mine = active && off;
                    if (mine) {
                        ray_birth(sc, *pl, id, r);
                        const TapeRef rt = { ADJ && eye ? tape.ev : nullptr, tape.mr, tape.ks };
                        walk_ray<true, ADJ>(sc, *pl, r, o, NoHit{}, GetCoefP{ hq, pos, ncol }, rt, &nt);
                        w = o.w; w_in = o.w_in;
                    }
                    if constexpr (ADJ) {
                        const int ntw = wave_max_int(mine && eye ? nt : 0);
                        if (mine && eye) {
                            int64_t k = kent;
                            reverse_sweep(sc, *pl, r.e, tape, nt, ntw, [&](double kappa, cd Gs, cd Gp, int meta) {
                                put_entry(k++, kappa, Gs, Gp, meta_bin | (int64_t)meta);
                            });
                        }
                    }
                }
                finish(active, id, cat, bin, nev, nh, w, w_in);
            }
            __threadfence_block();                        // the next pool's solves rewrite the queue
        }
        if (ADJ && lane == 0) {
            st.cnt[item * st.waves + wave] = (int32_t)(n_ent < st.cap_w ? n_ent : st.cap_w);
            if (n_ent > st.cap_w) st.ovf[item] = 1;
        }
        if (sc.item_work && lane == 0) sc.item_work[item * n_waves + wave] = (int32_t)n_work;
        __syncthreads();
        if (lds_bins) {
            for (int k = tid; k < B; k += WG) {
                if (s_c[k]) {
                    atomicAdd((unsigned long long*)&gq[k], s_q[k]);
                    atomicAdd(&gc[k], s_c[k]);
                }
            }
        }
    }
    if (n_fp64) atomicAdd(&s_st[ST_FP64], n_fp64);
    if (n_lay) atomicAdd(&s_st[ST_LAYERS], n_lay);
    if constexpr (ADJ && TAB) {
        // nonnegative doubles order like their bit patterns
        const double gm = wave_max(t_gmax);
        if (lane == 0 && gm > 0.0) atomicMax(&sc.tab_scale[0], (unsigned long long)__double_as_longlong(gm));
        if (t_ne) atomicAdd(&sc.tab_scale[1], t_ne);
    }
    __syncthreads();
    for (int k = tid; k < NCAT + 3; k += WG) {
        unsigned long long v = 0ull;
        if (k < NCAT + 2)
            for (int c = 0; c < kStatCols; ++c) v += s_col[k * kStatCols + c];
        else
            for (int c = 0; c < CAT_FACE_R; ++c) v += s_st[ST_CAT + c];      // every ray has one category
        s_st[k < NCAT ? ST_POW + k : k == NCAT ? ST_EVENTS : k == NCAT + 1 ? ST_PRMA : ST_RAYS] = v;
    }
    __syncthreads();
    for (int k = tid; k < ST_WORDS; k += WG)
        if (s_st[k]) atomicAdd(&stats[k], s_st[k]);
}

int64_t fwd_scratch_doubles(const SceneDev& sc, int64_t grid_blocks, int wg)
{
    return grid_blocks * (wg / 64) * fwd_wave_doubles(sc);
}
