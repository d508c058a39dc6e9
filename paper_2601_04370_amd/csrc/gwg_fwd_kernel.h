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

// Thin-film coefficients of one hit for this lane (fills the lane's slot
// table).  TAKEN: only the taken pair (refl), returned as both.
template <int MODE, bool TAKEN = false, class SL, class Stks>
__device__ inline Coef4 hit_solve(int n_slots, uint32_t cplx, const PointLds& pl, const Stks& stks,
                                  const SL& sl, int m, bool front, double kappa,
                                  bool* used_fp64, double* ck = nullptr, int64_t ckb = 8, bool refl = false,
                                  bool ck_evan = true)
{
    bool hyp = false;                       // an evanescent lossless slot at this kappa
    for (int s = 0; s < n_slots; ++s) {
        double P[NPF];
        slot_params(pl.slotN[2 * s], pl.slotN[2 * s + 1], (cplx >> s) & 1u, kappa, pl.k0, P);
        sl.put(s, P);
        hyp |= !((cplx >> s) & 1u) && P[0] < 0.0;
    }
    const bool circ = __ballot(hyp) == 0ull;
    const double z0 = pl.ng * pl.ng - kappa * kappa;
    const double q0 = sqrt(z0 > kTinyZ ? z0 : kTinyZ);
    const double eta0s = q0, eta0p = pl.ng * pl.ng / q0;
    const int L = pl.nlay[m];
    const auto stk = stks.mirror(m);
    const bool fp64 = (MODE == GWG_FP64) || (MODE == GWG_FP32_MIXED && near_critical(pl, n_slots, kappa));
    *used_fp64 = fp64;
    if (fp64)
        return tmm_solve<double, TAKEN, true>(stk, L, front, sl, cplx, pl.k0, eta0s, eta0p,
                                 mk(eta0s, 0.0), mk(eta0p, 0.0), mk(1.0, 0.0), circ,
                                 MODE == GWG_FP64 && (ck_evan || !hyp) ? ck : nullptr,
                                 ckb, ck_interval(hyp), refl);
    return tmm_solve<float, TAKEN>(stk, L, front, sl, cplx, pl.k0, eta0s, eta0p,
                            mk(eta0s, 0.0), mk(eta0p, 0.0), mk(1.0, 0.0), circ, nullptr, 8, kSegL, refl);
}

// Dense hit p (the wave's hits in ray order) belongs to the largest lane
// whose exclusive prefix sum of hit counts (off) is <= p: lanes without hits
// share the next lane's offset and lose the search to it.  Returns its queue
// slot.  Called by all lanes of the wave (shuffles).
__device__ inline int dense_slot(int p, int off)
{
    int l = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const int c = l + step;
        if (__shfl(off, c, 64) <= p) l = c;
    }
    return hq_slot(l, p - __shfl(off, l, 64));
}

// This lane's solves: hits in double precision, layers.
struct HitCounts { unsigned long long fp64, lay; };

// Solve the wave's `total` queued hits in batches of 64 (one per lane);
// off: this lane's exclusive prefix sum of hit counts.
template <int MODE, class SL, class Stks>
__device__ inline HitCounts solve_hits(int n_slots, uint32_t cplx, const PointLds& pl, const Stks& stks,
                                       const SL& sl, const HitQueue& hq, int total, int off)
{
    const int lane = wave_lane();
    HitCounts n = { 0ull, 0ull };
    for (int b = 0; b < total; b += 64) {
        const int p = b + lane;
        const int pp = p < total ? p : total - 1;
        const int q = dense_slot(pp, off);
        if (p < total) {
            const double kappa = hq.kappa(q);
            const int meta = hq.meta(q);
            const int m = meta & 255;
            bool u64 = false;
            const Coef4 c = hit_solve<MODE>(n_slots, cplx, pl, stks, sl, m, (meta >> 8) & 1, kappa, &u64);
            hq.put_coef(q, c);
            n.fp64 += u64 ? 1ull : 0ull;
            n.lay += (unsigned long long)pl.nlay[m];
        }
    }
    return n;
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
// columns (one per ray) of Kmax slots.  The geometry walk writes hit h of
// column col to slot h * ncol + col of kap (kappa) and word (its word); the
// per-hit solves read them in the order of ord (h << 16 | col), the
// slot of the hit's adjoint entry (relative to the wave's region, or -1) from
// ck, and write the hit's taken coefficients and word at the
// ray's place pos in the field-pass order: word to slot h * ncol + pos of
// tword, (c_s, c_p) as two 16-byte words to tcoef, the 64 lanes of a field
// pass side by side, so that its loads are whole cache lines.
struct PoolQueue {
    double* kap;
    double2* tcoef;              // [Kmax][pool][2][64]
    int32_t *word, *tword, *ord, *ck;
    int64_t* info;               // [ncol] adjoint entry position << 16 | length class << 1 | bound for the eyebox
    int64_t* fate;               // [ncol] see fate_word
    int32_t *bin, *pos, *at;     // [ncol] bin, place of a column, column at a place
    int ncol, cap;               // cap: slots (ncol Kmax)
    __device__ double2* coef(int h, int place) const
    {
        return tcoef + ((int64_t)h * (ncol >> 6) + (place >> 6)) * 128 + (place & 63);
    }
    // a hit's taken coefficients and word to the slots of its ray's place
    __device__ void put_taken(int h, int place, const Coef4& c, int w) const
    {
        const bool rf = (w >> 9) & 1;
        const cd cs = rf ? c.rs : c.ts, cp = rf ? c.rp : c.tp;
        double2* o = coef(h, place);
        o[0] = make_double2(cs.re, cs.im);
        o[64] = make_double2(cp.re, cp.im);
        tword[h * ncol + place] = w;
    }
};
constexpr int kSortBins = 128;                      // field-pass length classes
constexpr int kStatCols = 16;                       // columns of the statistics' LDS counters

// doubles of global scratch per wave: per slot kappa, the coefficients and
// four 32-bit words, per column two 64-bit and three 32-bit words
__host__ __device__ inline int64_t fwd_wave_doubles(const SceneDev& sc)
{
    return (int64_t)7 * 64 * sc.pool * sc.Kmax + 4 * 64 * sc.pool;
}
__device__ inline PoolQueue pool_queue(double* mem, int pool, int Kmax)
{
    PoolQueue q;
    q.ncol = 64 * pool;
    q.cap = q.ncol * Kmax;
    const int64_t n = q.cap;
    q.tcoef = (double2*)mem;
    q.kap = mem + 4 * n;
    q.word = (int32_t*)(q.kap + n);
    q.tword = q.word + n;
    q.ord = q.tword + n;
    q.ck = q.ord + n;
    q.info = (int64_t*)(q.ck + n);
    q.fate = q.info + q.ncol;
    q.bin = (int32_t*)(q.fate + q.ncol);
    q.pos = q.bin + q.ncol;
    q.at = q.pos + q.ncol;
    return q;
}

// A ray's fate: category (3 bits), walked in general (1), first field along
// p (1), mirror hits (9), events (9), final state (8), total reflections
// since the last hit (9).
__device__ inline int64_t fate_word(const DirFate& o)
{
    return (int64_t)(o.cat | (o.off ? 8 : 0) | o.pol << 4 | o.nh << 5 | o.nev << 14) | (int64_t)o.e << 23 |
           (int64_t)o.nt << 31;
}

// Writes the ray's hits to its column.  Also counts the hits whose kappa^2
// exceeds kap2 (they may meet an evanescent layer) in *ne and marks hits
// h < 64 of them in bit h of *evm.
struct PutHitP {
    PoolQueue q;
    int col;
    double kap2;
    int* ne;
    unsigned long long* evm;
    __device__ void operator()(int h, double kappa, int word) const
    {
        q.kap[h * q.ncol + col] = kappa;
        q.word[h * q.ncol + col] = word;
        if (kappa * kappa > kap2) {
            ++*ne;
            if (h < 64) *evm |= 1ull << h;
        }
    }
    __device__ void operator()(int h, const double* kappa, int word) const { (*this)(h, *kappa, word); }
    __device__ void branch(int, bool) const {}
};
// Keyed forwards: writes the words (kappa follows from the state) and marks
// their keys in the item's LDS bit set (the read first: most hits find their
// key marked).
struct PutHitK {
    PoolQueue q;
    int col, M;
    uint32_t* used;
    __device__ void operator()(int h, const double*, int word) const
    {
        q.word[h * q.ncol + col] = word;
        const int key = hit_key(word, M);
        if (!((used[key >> 5] >> (key & 31)) & 1u)) atomicOr(&used[key >> 5], 1u << (key & 31));
    }
    __device__ void branch(int, bool) const {}
};
// The general field walk's coefficients of the ray at place pos of the
// order: the taken pair (c_s, c_p) returned as both the reflected and the
// transmitted one, and the branch.
struct GetCoefP {
    PoolQueue q;
    int pos;
    static constexpr bool kStoredBranch = true;
    __device__ bool refl(int h) const { return (q.tword[h * q.ncol + pos] >> 9) & 1; }
    __device__ Coef4 operator()(int h, double, double, double, int, bool) const
    {
        const double2* b = q.coef(h, pos);
        const double2 s = b[0], p = b[64];
        Coef4 o;
        o.rs = o.ts = mk(s.x, s.y);
        o.rp = o.tp = mk(p.x, p.y);
        return o;
    }
};

// LDS pointers as the out-of-line solves take them: their address space is
// part of the type, or their loads would be flat ones.
typedef __attribute__((address_space(3))) void* LdsPtr;
__device__ inline LdsPtr lds_ptr(const void* p) { return (LdsPtr)p; }

// What the solves of one item read, and where they count.
struct SolveCtx {
    LdsPtr pl, rec, sp, st;      // PointLds, the stacks' records, this lane's slot table, statistics
    int Lmax, n_slots;
    uint32_t cplx;               // absorbing slots
};

// Solve a pool's ne + nc queued hits in batches of 64 (one per lane): ord
// lists the possibly evanescent hits from its front (positions 0 .. ne-1)
// and the others from its back (cap-1 down to cap-nc), so the batches of the
// second kind take the circular-only sweep.  ck (non-null): the blocks
// of the wave's region's entries; a hit whose slot c >= 0 stores its segment
// matrices (reflected: its states) there.
// Out of line: the layer loop needs some 50 scalar registers for its
// polynomials, and inlined among the walks it had 20 of them reloaded from
// vector lanes in every four layers (211 vector instructions where 188 are
// needed; 6 mirrors of 200 layers, 1.1e10 layer steps: 19.9 -> 18.8 ms).
template <int MODE, class SL>
__device__ __attribute__((noinline)) void solve_pool(SolveCtx cx, double* mem, int pool, int Kmax, int ne, int nc,
                                                     double* ck, int ck_nb, bool ck_evan)
{
    const PointLds& pl = *(const PointLds*)cx.pl;
    const RecStacks stks = { (const LayerRec*)cx.rec, cx.Lmax };
    const SL sl = { (double*)cx.sp, pl.nsq, pl.pxy };
    unsigned long long* st = (unsigned long long*)cx.st;
    const int n_slots = __builtin_amdgcn_readfirstlane(cx.n_slots);
    const uint32_t cplx = (uint32_t)__builtin_amdgcn_readfirstlane((int)cx.cplx);
    const PoolQueue q = pool_queue(mem, pool, Kmax);
    const int lane = wave_lane();
    const int total = __builtin_amdgcn_readfirstlane(ne + nc);
    unsigned long long n_fp64 = 0, n_lay = 0;
    for (int b = 0; b < total; b += 64) {
        const int p = b + lane;
        if (p < total) {
            const int hc = q.ord[p < ne ? p : q.cap - 1 - (p - ne)], h = hc >> 16, col = hc & 0xffff;
            const int slot = h * q.ncol + col;
            const double kappa = q.kap[slot];
            const int word = q.word[slot];
            const int place = q.pos[col];
            const int m = word & 255;
            bool u64 = false;
            double* ckp = nullptr;
            if (ck) {
                const int c = q.ck[slot];
                if (c >= 0) ckp = ck + (int64_t)c * ck_nb * 8;
            }
            const Coef4 c = hit_solve<MODE, true>(n_slots, cplx, pl, stks, sl, m, (word >> 8) & 1, kappa, &u64, ckp,
                                                  8, (word >> 9) & 1, ck_evan);
            q.put_taken(h, place, c, word);
            n_fp64 += u64 ? 1ull : 0ull;
            n_lay += (unsigned long long)pl.nlay[m];
        }
    }
    if (n_fp64) atomicAdd(&st[ST_FP64], n_fp64);
    if (n_lay) atomicAdd(&st[ST_LAYERS], n_lay);
}

// One hit (one per lane), out of line for the keyed forwards.
template <int MODE, class SL>
__device__ __attribute__((noinline)) Coef4 solve_one(SolveCtx cx, double kappa, int m, bool front)
{
    const PointLds& pl = *(const PointLds*)cx.pl;
    const RecStacks stks = { (const LayerRec*)cx.rec, cx.Lmax };
    const SL sl = { (double*)cx.sp, pl.nsq, pl.pxy };
    unsigned long long* st = (unsigned long long*)cx.st;
    bool u64 = false;
    const Coef4 c = hit_solve<MODE>(__builtin_amdgcn_readfirstlane(cx.n_slots),
                                    (uint32_t)__builtin_amdgcn_readfirstlane((int)cx.cplx), pl, stks, sl, m, front, kappa,
                                    &u64);
    if (u64) atomicAdd(&st[ST_FP64], 1ull);
    atomicAdd(&st[ST_LAYERS], (unsigned long long)pl.nlay[m]);
    return c;
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
    int* n;                      // slots in use; [1]: the table overflowed; [2]: a ray left the direction table
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
// One hit of a table ray as the field passes read it.
struct HitRec { int word; double2 cs, cp; };
// Per-hit solves: the queue's slots at place pos.
struct HitCoefs {
    PoolQueue q;
    int pos;
    __device__ HitRec operator()(int h) const
    {
        const double2* b = q.coef(h, pos);
        return { q.tword[h * q.ncol + pos], b[0], b[64] };
    }
    __device__ int64_t tag(int) const { return 0; }
};
// Keyed: the word in the ray's column, the key's coefficients in LDS.
struct KeyCoefs {
    PoolQueue q;
    int col, M;
    const uint8_t* slot;
    const double* kc;
    __device__ HitRec operator()(int h) const
    {
        const int w = q.word[h * q.ncol + col];
        const double2* b = (const double2*)(kc + 8 * slot[hit_key(w, M)] + (((w >> 9) & 1) ? 0 : 4));
        return { w, b[0], b[1] };
    }
    __device__ int64_t tag(int w) const { return (int64_t)slot[hit_key(w, M)] << kEntSlotShift; }
};

// Field of one ray of the table from its birth to its end, over its nh hits.
// Hits are requested three ahead of their use: their coefficients come from
// HBM (a pool's hits are more than the L2), a latency of several hits' work
// (requested one ahead, 8-byte words: 11.7 ms for 4.3e8 hits; so: 6.1 ms).
// Writes the incoming field's mirror components of hit h to the tape where
// tape.mr is set; returns the field at the ray's last state, before an exit.
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
    HitRec n1{}, n2{}, n3{};
    if (nh > 0) n1 = src(0);
    if (nh > 1) n2 = src(1);
    if (nh > 2) n3 = src(2);
    for (int h = 0; h < nh; ++h) {
        const HitRec r = n1;
        n1 = n2; n2 = n3;
        if (h + 3 < nh) n3 = src(h + 3);
        const int e = (r.word >> 11) & 255, neg = (r.word >> 10) & 1, m = r.word & 255;
        const bool rf = (r.word >> 9) & 1;
        const double* f = dt.f + e * kDirFld;
        tir(f, r.word >> 19);
        double c = f[DF_ROT + 2 * neg], d = f[DF_ROT + 2 * neg + 1];
        FaceSp b = to_mirror(a, c, d);
        if (tape.mr) tape_put_mirror(tape, h, b.s, b.p);
        const double scale = rf ? pl.sc_r[m] : pl.sc_t[m];
        b.s = cscale(cmul_f(mk(r.cs.x, r.cs.y), b.s), scale);
        b.p = cscale(cmul_f(mk(r.cp.x, r.cp.y), b.p), scale);
        if (rf) {
            const uint32_t fl = (uint32_t)__double_as_longlong(dt.g[e * kDirGeo + DG_FLAGS]);
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
// last to first, with the cotangents of reverse_sweep.  As in that sweep the
// lanes step a common hit index down from nhw - 1, the longest of the
// calling lanes' (nh = 0: none), so that they read the same tape record
// together.
template <class Coefs, class Emit>
__device__ inline void dir_reverse(const PointLds& pl, const DirLds& dt, FaceSp a, int nh, int nhw, int e_end,
                                   int nt_end, const Coefs& src, const TapeRef& tape, Emit emit)
{
    auto tir = [&](const double* f, int n) {
        const cd rs = mk(f[DF_RS], -f[DF_RS + 1]), rp = mk(f[DF_RP], -f[DF_RP + 1]);
        for (int k = 0; k < n; ++k) { a.s = cmul_f(rs, a.s); a.p = cmul_f(rp, a.p); }
    };
    const double* fx = dt.f + e_end * kDirFld;
    a.s = cscale(a.s, fx[DF_XS]);
    a.p = cscale(a.p, fx[DF_XP]);
    tir(fx, nt_end);
    struct Rec { HitRec r; double2 t0, t1; };
    auto fetch = [&](int h) {
        Rec x{};
        if (h >= 0 && h < nh) {
            x.r = src(h);
            const double2* p = (const double2*)(tape.mr + (int64_t)h * (tape.ks / 2));
            x.t0 = p[0];
            x.t1 = p[64];
        }
        return x;
    };
    Rec n1 = fetch(nhw - 1), n2 = fetch(nhw - 2);
    for (int h = nhw - 1; h >= 0; --h) {
        const Rec ev = n1;
        n1 = n2;
        n2 = fetch(h - 2);
        if (h >= nh) continue;                          // this lane has fewer hits
        const int wd = ev.r.word;
        const int e = (wd >> 11) & 255, neg = (wd >> 10) & 1, m = wd & 255;
        const bool rf = (wd >> 9) & 1;
        const double* g = dt.g + e * kDirGeo;
        const double* f = dt.f + e * kDirFld;
        const double c = f[DF_ROT + 2 * neg], d = f[DF_ROT + 2 * neg + 1];
        double co = c, so = d;
        if (rf) {
            const int ch = (int)((uint32_t)__double_as_longlong(g[DG_FLAGS]) >> (8 * neg)) & 255;
            const double* fc = dt.f + (ch >> 1) * kDirFld + DF_ROT + 2 * (ch & 1);
            co = fc[0]; so = fc[1];
        }
        const double scale = rf ? pl.sc_r[m] : pl.sc_t[m];
        FaceSp b = to_mirror(a, co, so);
        const cd Gs = cscale(cmul_f(cconj(b.s), mk(ev.t0.x, ev.t0.y)), scale);
        const cd Gp = cscale(cmul_f(cconj(b.p), mk(ev.t1.x, ev.t1.y)), scale);
        emit(g[DG_KAP + neg], Gs, Gp, (int64_t)(wd & 1023) | src.tag(wd));
        b.s = cscale(cmul_f(mk(ev.r.cs.x, -ev.r.cs.y), b.s), scale);
        b.p = cscale(cmul_f(mk(ev.r.cp.x, -ev.r.cp.y), b.p), scale);
        a = to_face(b, c, d);
        tir(f, wd >> 19);
    }
}

// ------------------------------------------------------------ general walks
// Where a forward's adjoint entries of one wave and item go.
struct EntryOut {
    double* ent;                 // the region's first entry
    int64_t cap_w;
    double gmax;                 // largest cotangent component (angle table)
    unsigned long long n;        // entries emitted
    __device__ void put(int64_t k, double kappa, cd Gs, cd Gp, int64_t meta, bool track)
    {
        if (track) {
            const double a = fmax(fmax(fabs(Gs.re), fabs(Gs.im)), fmax(fabs(Gp.re), fabs(Gp.im)));
            gmax = a > gmax ? a : gmax;
            ++n;
        }
        if (k < cap_w) {
            double2* e = (double2*)(ent + k * kEntFields);
            e[0] = make_double2(kappa, Gs.re);
            e[1] = make_double2(Gs.im, Gp.re);
            e[2] = make_double2(Gp.im, (double)meta);
        }
    }
};

// Geometry walk of one ray (this lane's, if mine): hits to its column.
__device__ inline void general_geometry(const SceneDev& sc, const PointLds& pl, int64_t id, const PoolQueue& q,
                                        int col, DirFate& o, int& ne, unsigned long long& evm)
{
    Ray r;
    Outcome oc;
    TapeRef none = { nullptr, nullptr, 0 };
    ne = 0;
    evm = 0ull;
    ray_birth(sc, pl, id, r);
    walk_ray<false, false>(sc, pl, r, oc, PutHitP{ q, col, pl.kap2_evan, &ne, &evm }, NoCoef{}, none, nullptr);
    o.cat = oc.cat; o.bin = oc.bin; o.nev = r.nev; o.nh = r.nprma;
    o.off = true;
}

// Field walk of the rays at places pos (lanes with mine), with the tape of
// every event and, where eye, the reverse sweep and its entries.  All lanes
// of the wave call.
template <bool ADJ>
__device__ inline void general_field(const SceneDev& sc, const PointLds& pl, int64_t id, const PoolQueue& q, int pos,
                                     bool mine, bool eye, const TapeRef& tape, int64_t kent, int64_t meta_bin,
                                     bool track, EntryOut& out, double& w, double& w_in)
{
    Ray r;
    Outcome o;
    int nt = 0;
    if (mine) {
        ray_birth(sc, pl, id, r);
        const TapeRef rt = { ADJ && eye ? tape.ev : nullptr, tape.mr, tape.ks };
        walk_ray<true, ADJ>(sc, pl, r, o, NoHit{}, GetCoefP{ q, pos }, rt, &nt);
        w = o.w; w_in = o.w_in;
    }
    if constexpr (ADJ) {
        const int ntw = wave_max_int(mine && eye ? nt : 0);
        if (mine && eye) {
            int64_t k = kent;
            reverse_sweep(sc, pl, r.e, tape, nt, ntw, [&](double kappa, cd Gs, cd Gp, int meta) {
                out.put(k++, kappa, Gs, Gp, meta_bin | (int64_t)meta, track);
            });
        }
    }
}

// The same for the few rays of a collimated item that leave its direction
// table, out of line (sc in LDS): inlined, their registers cost the kernel's
// own loops spills.
template <bool TAB>
__device__ __attribute__((noinline)) void off_geometry(const SceneDev& sc, const PointLds& pl, int64_t id,
                                                       const PoolQueue& q, int col, DirFate& o, int& ne,
                                                       unsigned long long& evm)
{
    general_geometry(sc, pl, id, q, col, o, ne, evm);
}
template <bool ADJ, bool TAB>
__device__ __attribute__((noinline)) void off_field(const SceneDev& sc, const PointLds& pl, int64_t id,
                                                    const PoolQueue& q, int pos, bool mine, bool eye,
                                                    const TapeRef& tape, int64_t kent, int64_t meta_bin, bool track,
                                                    EntryOut& out, double& w, double& w_in)
{
    general_field<ADJ>(sc, pl, id, q, pos, mine, eye, tape, kent, meta_bin, track, out, w, w_in);
}

// ------------------------------------------------------------------- LDS
// The table forward solves nothing: no stacks, and only the counting sort's
// class counts in place of the slot tables.
struct FwdLayout { int off_pl, off_rec, off_sp, off_q, off_c, off_st, off_col, off_sc, off_dir, off_key, total; };

__host__ __device__ inline FwdLayout fwd_layout(const SceneDev& sc, int wg, bool lds_bins, bool dirs, bool tab, bool memo)
{
    const int B = sc.bins_x * sc.bins_y, waves = (wg + 63) / 64;
    FwdLayout s;
    int o = 0;
    s.off_pl = o; o = align16(o + (int)sizeof(PointLds));
    s.off_rec = o; o = align16(o + (tab ? 0 : (int)sizeof(LayerRec) * sc.M * rec_stride(sc.Lmax)));
    s.off_sp = o;
    o = align16(o + (tab ? 4 * kSortBins * waves
                         : 8 * sc.n_slots * (memo ? LaneSlots3::kPer : LaneSlots3x::kPer) * 64 * waves));
    s.off_q = o; o = align16(o + (lds_bins ? 8 * B : 0));
    s.off_c = o; o = align16(o + (lds_bins ? 4 * B : 0));
    s.off_st = o; o = align16(o + 8 * ST_WORDS);
    s.off_col = o; o = align16(o + (NCAT + 2) * kStatCols * 8);
    s.off_sc = o; o = align16(o + (dirs ? (int)sizeof(SceneDev) : 0));
    s.off_dir = o; o = align16(o + (dirs ? kDirMax * kDirWords * 8 : 0));
    s.off_key = o; o = align16(o + (dirs && (tab || memo) ? key_smem_bytes(sc.M) : 0));
    s.total = o;
    return s;
}

// Persistent workgroups draw work items; each wave handles a strided share
// of the item's rays.  Eyebox bins of the current point accumulate in LDS
// (integer atomics) and are flushed per item with integer global atomics:
// the result does not depend on scheduling.  DIRS: collimated beams with a
// direction table (else every ray walks in general).
template <int MODE, bool ADJ, bool TAB, bool MEMO, bool DIRS>
__global__ void __launch_bounds__(256, TAB && DIRS ? (ADJ ? 3 : 4) : 2) k_trace_fwd(SceneDev sc, uint64_t* __restrict__ q_out,
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
    constexpr bool KEYED = DIRS && (TAB || MEMO);
    // slot table: all five values per lane, except with the keyed
    // coefficients, which solve few hits and keep their table in LDS
    using SlotTable = typename std::conditional<MEMO, LaneSlots3, LaneSlots3x>::type;
    const FwdLayout lay = fwd_layout(sc, WG, lds_bins != 0, DIRS, TAB, MEMO);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    LayerRec* s_rec = (LayerRec*)(smem + lay.off_rec);
    double* s_sp = (double*)(smem + lay.off_sp);
    unsigned long long* s_q = (unsigned long long*)(smem + lay.off_q);
    uint32_t* s_c = (uint32_t*)(smem + lay.off_c);
    unsigned long long* s_st = (unsigned long long*)(smem + lay.off_st);
    // statistics: per-ray sums in kStatCols columns per word, so that the
    // lanes of a wave add to different addresses
    unsigned long long* s_col = (unsigned long long*)(smem + lay.off_col);      // power, events, mirror hits
    const int tid = threadIdx.x, wave = tid / 64, lane = wave_lane();
    // the ordering's class counts: in this wave's slot tables (at least 1.5
    // KB), which only the solves use, or in LDS of their own
    uint32_t* s_hist = (uint32_t*)(smem + lay.off_sp + wave * (TAB ? 4 * kSortBins : sc.n_slots * SlotTable::kPer * kSlotLanes * 8));
    const int64_t gwave = (int64_t)blockIdx.x * n_waves + wave;
    double* pmem = scratch + gwave * fwd_wave_doubles(sc);
    const PoolQueue pq = pool_queue(pmem, sc.pool, sc.Kmax);
    const SolveCtx cx = { lds_ptr(pl), lds_ptr(s_rec), lds_ptr(slot_lane_base(s_sp, sc.n_slots, SlotTable::kPer, tid)),
                          lds_ptr(s_st), sc.Lmax, sc.n_slots, sc.slot_complex };
    const double wscale = ldexp(1.0, sc.fp_shift), wcap = ldexp(1.0, 40), pscale = 16777216.0;
    for (int k = tid; k < ST_WORDS; k += WG) s_st[k] = 0ull;
    for (int k = tid; k < (NCAT + 2) * kStatCols; k += WG) s_col[k] = 0ull;
    SceneDev* s_sc = (SceneDev*)(smem + lay.off_sc);
    if (DIRS && tid == 0) *s_sc = sc;                     // for the rays off the table
    const TapeRef tape = tape_lane(tape_scratch, sc.Kmax, (int64_t)gridDim.x * n_waves, gwave, lane);
    KeyLds kl{};
    if constexpr (KEYED) kl = key_lds(smem + lay.off_key, sc.M);
    const int key_cap = MEMO ? sc.memo : kFwdMemoKeys;
    EntryOut out = { nullptr, st.cap_w, 0.0, 0ull };

    for (int64_t it = draw_item(stats + ST_NEXT0); it < sc.n_items; it = draw_item(stats + ST_NEXT0)) {
        const int64_t item = sc.fwd_order ? (int64_t)sc.fwd_order[it] : it;
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, item, &point, &d, &l, &f, &i0, &i1);
        stage_point(sc, d, l, f, pl, nullptr, nullptr, TAB ? nullptr : s_rec, SlotTable::kPer);
        DirLds dt{};
        if constexpr (DIRS) dt = stage_dirs(sc, (int64_t)l * sc.F + f, (double*)(smem + lay.off_dir));
        int64_t n_work = 0;                               // this wave's mirror hits in this item (uniform)
        if (lds_bins)
            for (int k = tid; k < B; k += WG) { s_q[k] = 0ull; s_c[k] = 0u; }
        if constexpr (KEYED) {
            for (int k = tid; k < 2 * key_words(sc.M); k += WG) kl.used[k] = 0u;
            if (tid < 3) kl.n[tid] = 0;
        }
        __syncthreads();
        const int64_t base = point * sc.N;
        uint64_t* gq = q_out + point * B;
        uint32_t* gc = c_out + point * B;
        int64_t n_ent = 0;                                // this wave's entries in this item (uniform)
        bool keyed = KEYED;                               // the item's hits take their keys' coefficients (uniform)
        const int64_t region = item * st.waves + wave;
        out.ent = st.ent + region * st.cap_w * kEntFields;
        const double* tab_dl = TAB ? sc.table + (int64_t)(d * sc.n_lsel + l) * sc.M * 2 * sc.table_n * 8 : nullptr;
        // coefficients of one hit (one per lane)
        auto one_hit = [&](double kappa, int m, bool front) {
            if constexpr (TAB) {
                return table_coef(tab_dl, sc.table_n, m, front, kappa, pl->ng);
            } else {
                return solve_one<MODE, SlotTable>(cx, kappa, m, front);
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
        const int64_t first = i0 + (int64_t)wave * 64;
        const int n_rounds = first < i1 ? (int)((i1 - first + WG - 1) / WG) : 0;      // uniform
        const int n_rounds0 = (int)((i1 - i0 + WG - 1) / WG);                          // wave 0's, the most
        const bool cks = ADJ && !TAB && !MEMO && MODE == GWG_FP64 && st.ck != nullptr && region < st.ck_regions;
        for (int r0 = 0; r0 < (KEYED ? n_rounds0 : n_rounds); r0 += sc.pool) {
            const int nr = max(0, n_rounds - r0 < sc.pool ? n_rounds - r0 : sc.pool);
            int n_e = 0, n_c = 0;                         // the pool's possibly evanescent / other hits (uniform)
            bool any_off = !DIRS;                         // some ray of the pool walks in general (uniform)
            for (int rr = 0; rr < nr; ++rr) {
                const int col = rr * 64 + lane;
                const int64_t i = first + (int64_t)(r0 + rr) * WG + lane;
                const bool active = i < i1;
                DirFate o;
                o.cat = CAT_LOST; o.bin = -1; o.nev = o.nh = o.e = o.neg = o.nt = o.pol = 0;
                o.off = false;
                int ne = 0;
                unsigned long long evm = 0ull;             // bit h: hit h may meet an evanescent layer
                if constexpr (DIRS) {
                    if (active) {
                        if constexpr (KEYED) dir_walk(sc, *pl, dt, base + i, PutHitK{ pq, col, sc.M, kl.used }, o);
                        else dir_walk(sc, *pl, dt, base + i, PutHitP{ pq, col, pl->kap2_evan, &ne, &evm }, o);
                    }
                    if (__ballot(o.off) != 0ull) {
                        any_off = true;
                        if (KEYED && lane == 0) kl.n[2] = 1;
                        if (o.off) {
                            // copies: only these go through memory
                            const PoolQueue pq2 = pq;
                            DirFate o2 = o;
                            int ne2;
                            unsigned long long evm2;
                            off_geometry<TAB>(*s_sc, *pl, base + i, pq2, col, o2, ne2, evm2);
                            o = o2; ne = ne2; evm = evm2;
                        }
                    }
                } else {
                    if (active) general_geometry(sc, *pl, base + i, pq, col, o, ne, evm);
                }
                const int nh = o.nh;
                const bool to_eyebox = active && o.cat == CAT_EYEBOX;              // fixed by geometry alone
                // offsets of this ray's possibly evanescent (low half) and
                // other hits in the round's
                int t2;
                const int e2 = wave_excl_scan(ne | (nh - ne) << 16, &t2);
                const int te = t2 & 0xffff, tc = t2 >> 16;
                n_work += te + tc;
                // the ray's adjoint entries (rays bound for the eyebox) start
                // at kent of the wave's region; with a store for their blocks
                // the ray's hits learn their entries' slots
                int64_t kent = 0;
                if (ADJ) {
                    int etot;
                    const int eoff = wave_excl_scan(to_eyebox ? nh : 0, &etot);
                    kent = n_ent + eoff;
                    n_ent += etot;
                }
                if constexpr (!TAB && !KEYED) {
                    // solve order: the hits that may meet an evanescent layer
                    // from the front of ord, the others from its back
                    int pe = n_e + (e2 & 0xffff), pc = n_c + (e2 >> 16);
                    for (int h = 0; h < nh; ++h) {
                        bool ev;
                        if (h < 64) {
                            ev = (evm >> h) & 1ull;
                        } else {
                            const double k = pq.kap[h * pq.ncol + col];
                            ev = k * k > pl->kap2_evan;
                        }
                        const int at = ev ? pe++ : pq.cap - 1 - pc++;
                        pq.ord[at] = h << 16 | col;
                        if (cks) {
                            const int64_t k = kent + (nh - 1 - h);
                            pq.ck[h * pq.ncol + col] = to_eyebox && k < st.ck_cap ? (int32_t)k : -1;
                        }
                    }
                    n_e += te;
                    n_c += tc;
                }
                // field-pass length class (0: no ray): hits, or events of a
                // general walk, twice with a reverse sweep to follow
                const int len = o.off ? o.nev : nh;
                const int cost = len + (to_eyebox ? len : 0);
                const int key = active ? 1 + (cost < kSortBins - 2 ? cost : kSortBins - 2) : 0;
                pq.info[col] = (kent << 16) | (int64_t)(key << 1) | (to_eyebox ? 1 : 0);
                pq.fate[col] = fate_word(o);
                pq.bin[col] = o.bin;
            }
            __threadfence_block();
            // the field-pass order: the pool's columns by length class,
            // longest first (a counting sort)
            for (int k = lane; k < kSortBins; k += 64) s_hist[k] = 0u;
            wave_lds_sync();
            for (int rr = 0; rr < nr; ++rr) {
                const int key = (int)((pq.info[rr * 64 + lane] >> 1) & 255);
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
                const int key = (int)((pq.info[col] >> 1) & 255);
                const int pos = (int)atomicAdd(&s_hist[key], 1u);
                pq.pos[col] = pos;
                pq.at[pos] = col;
            }
            wave_lds_sync();                              // s_hist is the solves' LDS again
            __threadfence_block();
            if constexpr (TAB || MEMO) {
                if constexpr (KEYED) {
                    if (keyed) keyed = key_resolve(kl, dt, sc.M, key_cap, one_hit);
                }
                if (!keyed || any_off) {
                    // hit by hit, each lane its own column's (rays off the
                    // direction table, or every ray without keys)
                    for (int rr = 0; rr < nr; ++rr) {
                        const int col = rr * 64 + lane;
                        const int64_t fate = pq.fate[col];
                        const bool off = (fate >> 3) & 1;
                        const int nh = !keyed || off ? (int)(fate >> 5) & 511 : 0;
                        const int pos = pq.pos[col];
                        for (int h = 0; h < nh; ++h) {
                            const int word = pq.word[h * pq.ncol + col];
                            const double kappa = off ? pq.kap[h * pq.ncol + col]
                                                     : dt.g[((word >> 11) & 255) * kDirGeo + DG_KAP + ((word >> 10) & 1)];
                            const Coef4 c = one_hit(kappa, word & 255, (word >> 8) & 1);
                            pq.put_taken(h, pos, c, word);
                        }
                    }
                    __threadfence_block();
                }
            } else {
                solve_pool<MODE, SlotTable>(cx, pmem, sc.pool, sc.Kmax, n_e, n_c,
                                            cks ? st.ck + region * st.ck_cap * st.ck_nb * 8 : nullptr, st.ck_nb,
                                            st.ck_evan != 0);
                __threadfence_block();
            }
            for (int s2 = 0; s2 < nr; ++s2) {
                const int pos = s2 * 64 + lane;
                const int col = pq.at[pos];
                const int64_t info = pq.info[col], fate = pq.fate[col];
                const int64_t i = first + (int64_t)(r0 + col / 64) * WG + (col & 63);
                const int64_t id = base + i;
                const bool active = ((info >> 1) & 255) != 0, eye = (info & 1) != 0, off = (fate >> 3) & 1;
                const int64_t kent = info >> 16;
                const int cat = (int)(fate & 7), bin = pq.bin[col];
                const int nev = (int)(fate >> 14) & 511, nh = (int)(fate >> 5) & 511;
                const int64_t meta_bin = (int64_t)(bin & 0xffffff) << 10;
                double w = 0.0, w_in = 0.0;
                if constexpr (DIRS) {
                    const int e_end = (int)(fate >> 23) & 255, nt_end = (int)(fate >> 31) & 511;
                    const bool mine = active && !off;
                    auto table_rays = [&](const auto& src) {
                        const TapeRef rt = { nullptr, ADJ && eye ? tape.mr : nullptr, tape.ks };
                        FaceSp a{};
                        if (mine) {
                            a = dir_field(*pl, dt, (int)(fate >> 4) & 1, nh, e_end, nt_end, src, rt);
                            w = w_in = sp_norm2(a);
                            if (cat == CAT_EYEBOX || cat == CAT_MISS) {
                                const double* fx = dt.f + e_end * kDirFld;
                                a.s = cscale(a.s, fx[DF_XS]);
                                a.p = cscale(a.p, fx[DF_XP]);
                                w = sp_norm2(a);
                            }
                        }
                        if constexpr (ADJ) {
                            const int nhw = wave_max_int(mine && eye ? nh : 0);
                            if (mine && eye) {
                                int64_t k = kent;
                                dir_reverse(*pl, dt, a, nh, nhw, e_end, nt_end, src, tape,
                                            [&](double kappa, cd Gs, cd Gp, int64_t meta) {
                                                out.put(k++, kappa, Gs, Gp, meta_bin | meta, TAB);
                                            });
                            }
                        }
                    };
                    if constexpr (KEYED) {
                        if (keyed) table_rays(KeyCoefs{ pq, col, sc.M, kl.slot, kl.coef });
                        else table_rays(HitCoefs{ pq, pos });
                    } else {
                        table_rays(HitCoefs{ pq, pos });
                    }
                    if (any_off && __ballot(active && off) != 0ull) {
                        const PoolQueue pq2 = pq;
                        const TapeRef tp2 = tape;
                        EntryOut out2 = out;
                        double w2 = 0.0, wi2 = 0.0;
                        off_field<ADJ, TAB>(*s_sc, *pl, id, pq2, pos, active && off, eye, tp2, kent,
                                            meta_bin | (int64_t)kNoSlot << kEntSlotShift, TAB, out2, w2, wi2);
                        out = out2;
                        if (active && off) { w = w2; w_in = wi2; }
                    }
                } else {
                    general_field<ADJ>(sc, *pl, id, pq, pos, active, eye, tape, kent, meta_bin, TAB, out, w, w_in);
                }
                finish(active, id, cat, bin, nev, nh, w, w_in);
            }
            __threadfence_block();                        // the next pool's solves rewrite the queue
        }
        if (ADJ && lane == 0) {
            st.cnt[region] = (int32_t)(n_ent < st.cap_w ? n_ent : st.cap_w);
            if (n_ent > st.cap_w && atomicExch(&st.ovf[item], 1) == 0) st.left[1 + atomicAdd(st.left, 1)] = (int32_t)item;
        }
        if (sc.item_work && lane == 0) sc.item_work[item * n_waves + wave] = (int32_t)n_work;
        __syncthreads();
        if constexpr (ADJ && KEYED) {
            const int n = keyed ? kl.n[0] : -1;
            if (st.n_keys) {
                if (tid == 0) {
                    st.n_keys[item] = n;
                    if (n < 0 || kl.n[2] != 0) st.unkeyed[1 + atomicAdd(st.unkeyed, 1)] = (int32_t)item;
                }
                for (int k = tid; k < n; k += WG) st.keys[item * kFwdMemoKeys + k] = kl.key[k];
            }
        }
        if (lds_bins) {
            for (int k = tid; k < B; k += WG) {
                if (s_c[k]) {
                    atomicAdd((unsigned long long*)&gq[k], s_q[k]);
                    atomicAdd(&gc[k], s_c[k]);
                }
            }
        }
    }
    if constexpr (ADJ && TAB) {
        // nonnegative doubles order like their bit patterns
        const double gm = wave_max(out.gmax);
        if (lane == 0 && gm > 0.0) atomicMax(&sc.tab_scale[0], (unsigned long long)__double_as_longlong(gm));
        if (out.n) atomicAdd(&sc.tab_scale[1], out.n);
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
