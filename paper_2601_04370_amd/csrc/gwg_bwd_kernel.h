// Adjoint trace kernels.  Included by gwg_kernels.hip inside namespace gwg.
//
// Gradient checkpointing between the tracer and the thin-film solver
// (Methods, memory-saving strategies): the path part and the thin-film part
// of the adjoint run separately.
//
// Path part.  For every ray ending in an eyebox bin, the reverse field sweep
// (reverse_sweep) gives each of its mirror hits the holomorphic cotangents
// G_s, G_p of the two coefficients the ray took.  When the forward trace was
// asked to prepare a gradient it ran this sweep itself and stored one entry
// per hit (AdjStore); otherwise, or for work items whose entry regions
// overflowed, k_trace_bwd regenerates the paths: a geometry-only walk finds
// each ray's bin and queues its hits, the hits of rays in a bin with nonzero
// dL/dI are solved, those rays are walked again with the field and a tape of
// their field-changing events, and the sweep runs on the tape.
//
// Thin-film part.  Entries are drained 64 at a time, one per lane, so every
// lane runs the same layer loop whatever the length of its ray: the adjoint
// thin-film solve of the hit adds (dL/dI[bin] / N) d(2 Re(G_s c_s + G_p c_p))/dt_j
// into the wave's private LDS row of that mirror.
//
// (Entries of lossless scenes and of scenes with few absorbing layers go to
// gwg_adj_kernel.h instead.)
//
// Each wave owns its LDS accumulator, and the partial rows are summed in a
// fixed order afterwards, so the gradient is bit-identical from run to run.

constexpr int kQFields = 6;      // kappa, Gs.re, Gs.im, Gp.re, Gp.im, meta

__device__ inline AdjEntry load_entry(const AdjStore& st, int64_t e)
{
    const double2* p = (const double2*)(st.ent + e * kEntFields);
    const double2 a = p[0], b = p[1], c = p[2];
    return { a.x, a.y, b.x, b.y, c.x, (int64_t)c.y };
}

struct Queue {
    double* base;      // this wave's queue, field f of slot p at base[f * cap + p]
    int cap;
};

__device__ inline void q_put(const Queue& q, int pos, double kappa, cd Gs, cd Gp, int meta)
{
    int p = pos % q.cap;
    q.base[0 * q.cap + p] = kappa;
    q.base[1 * q.cap + p] = Gs.re;
    q.base[2 * q.cap + p] = Gs.im;
    q.base[3 * q.cap + p] = Gp.re;
    q.base[4 * q.cap + p] = Gp.im;
    q.base[5 * q.cap + p] = (double)meta;
}

// Adjoint thin-film solve of one mirror hit (one per lane): kappa, the
// scaled cotangents and meta = mirror | front << 8 | reflected << 9.
// KIND: whether the scene has absorbing slots; the kernels are compiled for
// either, so that each keeps within the 64 KB instruction cache.
// chk: the lane's scratch (blocks of 8 doubles, stride cstride).
enum { ADJ_LOSSLESS = 1, ADJ_ABSORBING = 2 };
template <int KIND>
__device__ inline void adjoint_hit(int n_slots, uint32_t slot_complex, int Lmax, const PointLds& pl, const double* s_thk,
                                   const uint8_t* s_slot, const LaneSlots3& sl, double* gw, double kappa, cd Gs,
                                   cd Gp, int meta, double* chk, int64_t cstride)
{
    const int m = meta & 255;
    const bool front = (meta >> 8) & 1, refl = (meta >> 9) & 1;
    bool hyp = false;                       // an evanescent lossless slot at this kappa
    for (int s = 0; s < n_slots; ++s) {
        double P[NPF];
        slot_params(pl.slotN[2 * s], pl.slotN[2 * s + 1], KIND != ADJ_LOSSLESS && ((slot_complex >> s) & 1u), kappa, pl.k0, P);
        sl.put(s, P);
        hyp |= !((slot_complex >> s) & 1u) && P[0] < 0.0;
    }
    const double z0 = pl.ng * pl.ng - kappa * kappa;
    const double q0 = sqrt(z0 > kTinyZ ? z0 : kTinyZ);
    if (KIND == ADJ_LOSSLESS) {
        // waves whose lanes all see circular layers take the sweep without
        // the hyperbolic case
        const bool circ = __ballot(hyp) == 0ull;
        const int nblk = Lmax / kSegUp + 1;
        if (circ)
            tmm_adjoint_lossless<false>(s_thk + m * Lmax, s_slot + m * Lmax, pl.nlay[m], front, sl, pl.k0, q0,
                                        pl.ng * pl.ng / q0, refl, Gs, Gp, gw + m * Lmax, chk, cstride, nblk);
        else
            tmm_adjoint_lossless<true>(s_thk + m * Lmax, s_slot + m * Lmax, pl.nlay[m], front, sl, pl.k0, q0,
                                       pl.ng * pl.ng / q0, refl, Gs, Gp, gw + m * Lmax, chk, cstride, nblk);
    }
    else
        tmm_adjoint(s_thk + m * Lmax, s_slot + m * Lmax, pl.nlay[m], front, sl, slot_complex,
                    pl.k0, kappa * kappa, q0, pl.ng * pl.ng / q0, refl, Gs, Gp, gw + m * Lmax, chk,
                    cstride);
}

// What the regenerating kernel's thin-film routines read: LDS (PointLds, the
// stacks, this lane's slot table, the wave's accumulator) and the scene's sizes.
struct BwdCtx {
    LdsPtr pl, thk, slot, sp, gw;
    int Lmax, n_slots;
    uint32_t cplx;               // absorbing slots
    __device__ const PointLds& point() const { return *(const PointLds*)pl; }
    __device__ LaneSlots3 slots() const
    {
        const PointLds& p = point();
        return { (double*)sp, p.nsq, p.pxy };
    }
};

// Adjoint thin-film solve of ring-queue entry `pos` (one per lane).  It and
// bwd_solve are out of line, as the forward's solves are: inlined among the
// walks their layer loops reloaded scalar registers from vector lanes (363
// points x 8192 rays, traced again: 200 layers 17.6 -> 17.4 ms, 40 layers 7.2 ->
// 6.2 ms, 201 layers with one of silver, 75 points x 4096 rays 6.0 -> 4.8 ms).
template <int KIND>
__device__ __attribute__((noinline)) void bwd_adjoint(BwdCtx cx, Queue q, int pos, double* chk, int64_t cstride)
{
    const int p = pos % q.cap;
    adjoint_hit<KIND>(__builtin_amdgcn_readfirstlane(cx.n_slots), (uint32_t)__builtin_amdgcn_readfirstlane((int)cx.cplx),
                      __builtin_amdgcn_readfirstlane(cx.Lmax), cx.point(), (const double*)cx.thk, (const uint8_t*)cx.slot,
                      cx.slots(), (double*)cx.gw, q.base[p], mk(q.base[1 * q.cap + p], q.base[2 * q.cap + p]),
                      mk(q.base[3 * q.cap + p], q.base[4 * q.cap + p]), (int)q.base[5 * q.cap + p], chk, cstride);
}

// Solve the wave's `total` queued hits; off: as solve_hits.
template <int MODE>
__device__ __attribute__((noinline)) HitCounts bwd_solve(BwdCtx cx, HitQueue hq, int total, int off)
{
    const int Lmax = __builtin_amdgcn_readfirstlane(cx.Lmax);
    return solve_hits<MODE>(__builtin_amdgcn_readfirstlane(cx.n_slots), (uint32_t)__builtin_amdgcn_readfirstlane((int)cx.cplx),
                            cx.point(), ArrStacks{ (const double*)cx.thk, (const uint8_t*)cx.slot, Lmax,
                                                   LaneSlots3::kPer * kSlotLanes * 8 },
                            cx.slots(), hq, __builtin_amdgcn_readfirstlane(total), off);
}

// Pushes the entries of one ray onto the ring queue with the dL/dI factor applied.
struct QueueEmit {
    Queue q;
    int* pos;
    double gscale;
    __device__ void operator()(double kappa, cd Gs, cd Gp, int meta) const
    {
        q_put(q, (*pos)++, kappa, cscale(Gs, gscale), cscale(Gp, gscale), meta);
    }
};

template <int MODE, bool TAB, int KIND>
__global__ void __launch_bounds__(128, 2) k_trace_bwd(SceneDev sc, const double* __restrict__ dLdI,
                                                   double* __restrict__ partial,
                                                   double* __restrict__ scratch, int64_t sample_stride,
                                                   const int32_t* __restrict__ regen,
                                                   unsigned long long* __restrict__ stats)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int WG = blockDim.x;
    const int n_waves = (WG + 63) / 64;
    const int B = sc.bins_x * sc.bins_y;
    const SmemLayout lay = smem_layout(sc.M, sc.Lmax, sc.n_slots, WG, B, false, n_waves);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    double* s_thk = (double*)(smem + lay.off_thk);
    uint8_t* s_slot = (uint8_t*)(smem + lay.off_slot);
    double* s_sp = (double*)(smem + lay.off_sp);
    double* s_grad = (double*)(smem + lay.off_grad);
    unsigned long long* s_st = (unsigned long long*)(smem + lay.off_st);
    const int tid = threadIdx.x;
    const int wave = tid / 64;
    const int lane = wave_lane();
    const int ML = sc.M * sc.Lmax;
    double* gw = s_grad + (int64_t)wave * ML;
    const BwdCtx cx = { lds_ptr(pl), lds_ptr(s_thk), lds_ptr(s_slot),
                        lds_ptr(slot_lane_base(s_sp, sc.n_slots, LaneSlots3::kPer, tid)), lds_ptr(gw), sc.Lmax, sc.n_slots,
                        sc.slot_complex };
    const int64_t nthreads = (int64_t)gridDim.x * WG;
    const int64_t gtid = (int64_t)blockIdx.x * WG + tid;
    const int64_t gwave = (int64_t)blockIdx.x * n_waves + wave;
    // scratch: the tape (Kmax event slots of every lane), then n_chk x 8
    // checkpoint doubles per lane, then queues per wave
    const TapeRef tape = tape_lane(scratch, sc.Kmax, (int64_t)gridDim.x * n_waves, gwave, lane);
    const int64_t n_chk = adj_blocks(sc.Lmax);
    double* chk = scratch + (int64_t)sc.Kmax * kTapeStride * nthreads + gtid;
    const int qcap = 64 * (sc.Kmax + 1);
    const int64_t n_waves_total = (int64_t)gridDim.x * n_waves;
    double* qbase = scratch + ((int64_t)sc.Kmax * kTapeStride + n_chk * 8) * nthreads;
    Queue q = { qbase + gwave * (int64_t)kQFields * qcap, qcap };
    const int hcap = 64 * sc.Kmax;
    const HitQueue hq = { qbase + n_waves_total * (int64_t)kQFields * qcap + gwave * (int64_t)kHitFields * hcap, hcap };
    for (int k = tid; k < ST_WORDS; k += WG) s_st[k] = 0ull;
    unsigned long long c_rays = 0, c_ev = 0, c_hits = 0, c_lay = 0, c_fp64 = 0;
    unsigned long long c_arays = 0, c_ahits = 0, c_alay = 0;
    // angle table: coefficients are interpolated and the sweep's cotangents go
    // to the table accumulators instead of the thin-film adjoint
    constexpr bool tabm = TAB;
    const double fx = tabm ? table_fx_scale(sc) : 0.0;

    // regen (optional): only the listed items, whose stored entries overflowed
    const int64_t n_it = regen ? (int64_t)regen[0] : sc.n_items;
    for (int64_t it = draw_item(stats + ST_NEXT1); it < n_it; it = draw_item(stats + ST_NEXT1)) {
        const int64_t item = regen ? (int64_t)regen[1 + it] : it;
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, item, &point, &d, &l, &f, &i0, &i1);
        stage_point(sc, d, l, f, pl, s_thk, s_slot);
        for (int k = tid; k < n_waves * ML; k += WG) s_grad[k] = 0.0;
        __syncthreads();
        const int64_t base = point * sc.N;
        const double* g_bins = dLdI + point * B;
        const int64_t dl = (int64_t)d * sc.n_lsel + l;
        const double* tab_dl = tabm ? sc.table + dl * sc.M * 2 * sc.table_n * 8 : nullptr;
        long long* acc_dl = tabm ? sc.tab_acc + dl * sc.M * 4 * sc.table_n * 4 : nullptr;
        int qhead = 0, qcount = 0;            // wave-uniform
        for (int64_t round = 0;; ++round) {
            const int64_t wave_first = i0 + (int64_t)wave * 64 + round * WG;
            if (wave_first >= i1) break;      // uniform across the wave
            const int64_t i = wave_first + lane;
            const int64_t id = base + i;
            bool active = i < i1 && (sample_stride <= 1 || (id % sample_stride) == 0);
            Ray r;
            Outcome o;
            o.cat = CAT_LOST;
            o.bin = -1;
            int nt = 0;
            TapeRef none = { nullptr, nullptr, 0 };
            int nh = 0;
            double gscale = 0.0;
            const int own = lane;                // this lane's column of the hit queue
            if (active) {
                ray_birth(sc, *pl, id, r);
                if constexpr (TAB)
                    walk_ray<false, false>(sc, *pl, r, o, NoHit{}, NoCoef{}, none, nullptr);
                else
                    walk_ray<false, false>(sc, *pl, r, o, PutHit{ hq, own }, NoCoef{}, none, nullptr);
                // the bin is fixed by geometry alone: rays that end outside the
                // eyebox or in a bin with dL/dI = 0 carry no gradient and are
                // not regenerated further
                if (o.cat == CAT_EYEBOX) gscale = g_bins[o.bin] / (double)sc.N;
                active = gscale != 0.0;
                nh = active ? r.nprma : 0;
            }
            if (!tabm) {
                int htotal;
                const int hoff = wave_excl_scan(nh, &htotal);
                __threadfence_block();
                const HitCounts n = bwd_solve<MODE>(cx, hq, htotal, hoff);
                c_fp64 += n.fp64;
                c_lay += n.lay;
                __threadfence_block();
            }
            if (active) {
                ray_birth(sc, *pl, id, r);
                if constexpr (TAB)
                    walk_ray<true, true>(sc, *pl, r, o, NoHit{}, TabCoef{ tab_dl, sc.table_n, pl->ng, sc.nx, sc.nz }, tape, &nt);
                else
                    walk_ray<true, true>(sc, *pl, r, o, NoHit{}, GetCoef{ hq, own }, tape, &nt);
                c_rays += 1;
                c_ev += (unsigned long long)r.nev;
                c_hits += (unsigned long long)r.nprma;
            }
            const bool contrib = active;
            const int ntw = wave_max_int(contrib ? nt : 0);
            if constexpr (TAB) {
                if (contrib) {
                    c_arays += 1;
                    reverse_sweep(sc, *pl, r.e, tape, nt, ntw, TableEmit{ acc_dl, sc.table_n, pl->ng, gscale, fx });
                }
                continue;
            }
            int total;
            const int off = wave_excl_scan(contrib ? r.nprma : 0, &total);
            if (contrib) {
                c_arays += 1;
                int slotpos = qhead + qcount + off;
                reverse_sweep(sc, *pl, r.e, tape, nt, ntw, QueueEmit{ q, &slotpos, gscale });
            }
            qcount += total;
            __threadfence_block();
            // phase 2: drain full batches
            while (qcount >= 64) {
                bwd_adjoint<KIND>(cx, q, qhead + lane, chk, nthreads);
                const int m = ((int)q.base[5 * q.cap + (qhead + lane) % q.cap]) & 255;
                c_ahits += 1;
                c_alay += (unsigned long long)pl->nlay[m];
                qhead = (qhead + 64) % q.cap;
                qcount -= 64;
            }
        }
        if (qcount > 0) {
            if (lane < qcount) {
                bwd_adjoint<KIND>(cx, q, qhead + lane, chk, nthreads);
                const int m = ((int)q.base[5 * q.cap + (qhead + lane) % q.cap]) & 255;
                c_ahits += 1;
                c_alay += (unsigned long long)pl->nlay[m];
            }
            qcount = 0;
        }
        __syncthreads();
        if constexpr (TAB) continue;
        double* out = partial + item * (int64_t)ML;
        for (int k = tid; k < ML; k += WG) {
            double acc = 0.0;
            for (int w = 0; w < n_waves; ++w) acc += s_grad[(int64_t)w * ML + k];
            out[k] = acc;
        }
    }
    const unsigned long long cnt[9] = { c_rays, c_ev, c_hits, c_fp64, 0ull, c_lay, c_arays, c_ahits, c_alay };
    for (int k = 0; k < 9; ++k)
        if (cnt[k]) atomicAdd(&s_st[k], cnt[k]);
    __syncthreads();
    for (int k = tid; k < 9; k += WG)
        if (s_st[k]) atomicAdd(&stats[k], s_st[k]);
}

// One kind's queue of entry indices in a wave: n (wave-uniform) entries at
// positions 0..n-1, position p in lane p of lo (p < 64) or of hi (p >= 64).
struct KindQueue {
    int lo = -1, hi = -1, n = 0;
    // file lane's entry c if `mine` (all lanes call; entries keep lane order)
    __device__ void add(bool mine, int c, int lane)
    {
        const unsigned long long m = __ballot(mine);
        const int below = __popcll(m & ((1ull << lane) - 1ull));
        const int cnt = __popcll(m);
        // a permutation of the lanes: the entries go to lanes (n + rank) mod
        // 64, the other lanes' pushes fill the remaining lanes (unread)
        const int dst = mine ? ((n + below) & 63) : ((n + cnt + (lane - below)) & 63);
        const int got = __builtin_amdgcn_ds_permute(dst << 2, c);
        if (lane >= n && lane < n + cnt) lo = got;               // positions n .. 63
        if (lane + 64 < n + cnt) hi = got;                       // positions 64 .. n + cnt - 1
        n += cnt;
    }
    // the first min(n, 64) entries, one per lane (-1 past n)
    __device__ int take()
    {
        const int lane = (int)(threadIdx.x & 63);
        const int v = lane < n ? lo : -1;
        lo = hi;
        hi = -1;
        n = n > 64 ? n - 64 : 0;
        return v;
    }
};

// Thin-film part of the adjoint over the entries stored by the forward trace
// of scenes with a stack of more pieces than k_adj_sorted takes (an absorbing
// layer in about every second: the pieces' states would be as many as its
// four-layer segments').  Items whose
// regions overflowed are left to k_trace_bwd.
__global__ void __launch_bounds__(128, 2) k_adj_entries(SceneDev sc, const double* __restrict__ dLdI,
                                                     double* __restrict__ partial, AdjStore st,
                                                     double* __restrict__ scratch,
                                                     unsigned long long* __restrict__ stats)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int WG = blockDim.x;
    const int n_waves = (WG + 63) / 64;
    const int B = sc.bins_x * sc.bins_y;
    const SmemLayout lay = smem_layout(sc.M, sc.Lmax, sc.n_slots, WG, B, false, n_waves);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    double* s_thk = (double*)(smem + lay.off_thk);
    uint8_t* s_slot = (uint8_t*)(smem + lay.off_slot);
    double* s_sp = (double*)(smem + lay.off_sp);
    double* s_grad = (double*)(smem + lay.off_grad);
    unsigned long long* s_st = (unsigned long long*)(smem + lay.off_st);
    const int tid = threadIdx.x;
    const int wave = tid / 64;
    const int lane = wave_lane();
    const int ML = sc.M * sc.Lmax;
    double* gw = s_grad + (int64_t)wave * ML;
    const LaneSlots3 sl = { slot_lane_base(s_sp, sc.n_slots, LaneSlots3::kPer, tid), pl->nsq, pl->pxy };
    const int64_t nthreads = (int64_t)gridDim.x * WG;
    double* chk = scratch + (int64_t)blockIdx.x * WG + tid;
    for (int k = tid; k < ST_WORDS; k += WG) s_st[k] = 0ull;
    unsigned long long c_ahits = 0, c_alay = 0;

    for (int64_t it = draw_item(stats + ST_NEXT0); it < sc.n_items; it = draw_item(stats + ST_NEXT0)) {
        const int64_t item = st.order ? (int64_t)st.order[it] : it;
        if (st.ovf[item] != 0) continue;
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, item, &point, &d, &l, &f, &i0, &i1);
        stage_point(sc, d, l, f, pl, s_thk, s_slot);
        for (int k = tid; k < n_waves * ML; k += WG) s_grad[k] = 0.0;
        __syncthreads();
        const double* g_bins = dLdI + point * B;
        const int32_t* cnt = st.cnt + item * st.waves;
        int total = 0;
        for (int w = 0; w < st.waves; ++w) total += cnt[w];
        // Batches of one kind: the wave scans its chunks of 64 entries (item
        // order) and files each entry under its kind, an entry whose kappa
        // may meet an evanescent layer or one that cannot; a batch of 64 is
        // taken from a kind's queue as soon as it holds that many, the rest
        // at the end.  Most batches then take the sweeps without the
        // hyperbolic case, and a batch's entries stay close together in item
        // order (their stored sweeps share lines).  Each kind's queue is two
        // registers per lane, positions 0-63 and 64-127; entries reach their
        // positions by a lane permutation.
        KindQueue qc, qh;
        int chunk = wave;
        for (;;) {
            int v = -1;
            for (;;) {                                    // wave-uniform: the next batch
                if (qc.n >= 64) { v = qc.take(); break; }
                if (qh.n >= 64) { v = qh.take(); break; }
                if (chunk * 64 >= total) {
                    if (qc.n > 0) { v = qc.take(); break; }
                    if (qh.n > 0) { v = qh.take(); break; }
                    break;
                }
                const int c = chunk * 64 + lane;
                bool ev = false;
                if (c < total) {
                    int rr = 0, k = c;
                    while (k >= cnt[rr]) { k -= cnt[rr]; ++rr; }
                    const double kap = st.ent[((item * st.waves + rr) * st.cap_w + k) * kEntFields];
                    ev = kap * kap > pl->kap2_evan;
                }
                qc.add(c < total && !ev, c, lane);
                qh.add(c < total && ev, c, lane);
                chunk += n_waves;
            }
            if (__ballot(v >= 0) == 0ull) break;
            if (v >= 0) {
                int rr = 0, k = v;
                while (k >= cnt[rr]) { k -= cnt[rr]; ++rr; }
                const int64_t e = (item * st.waves + rr) * st.cap_w + k;
                const AdjEntry en = load_entry(st, e);
                const double kappa = en.kappa;
                const int64_t meta = en.meta;
                const int bin = ent_bin(meta);
                const double gscale = g_bins[bin] / (double)sc.N;
                if (gscale != 0.0) {
                    const cd Gs = cscale(mk(en.gs_re, en.gs_im), gscale);
                    const cd Gp = cscale(mk(en.gp_re, en.gp_im), gscale);
                    const int mm = (int)(meta & 1023);
                    adjoint_hit<ADJ_ABSORBING>(sc.n_slots, sc.slot_complex, sc.Lmax, *pl, s_thk, s_slot, sl, gw, kappa, Gs, Gp, mm, chk, nthreads);
                    c_ahits += 1;
                    c_alay += (unsigned long long)pl->nlay[mm & 255];
                }
            }
        }
        __syncthreads();
        double* out = partial + item * (int64_t)ML;
        for (int k = tid; k < ML; k += WG) {
            double acc = 0.0;
            for (int w = 0; w < n_waves; ++w) acc += s_grad[(int64_t)w * ML + k];
            out[k] = acc;
        }
    }
    if (c_ahits) atomicAdd(&s_st[ST_ADJ_HITS], c_ahits);
    if (c_alay) atomicAdd(&s_st[ST_ADJ_LAYERS], c_alay);
    __syncthreads();
    for (int k = tid; k < ST_WORDS; k += WG)
        if (s_st[k]) atomicAdd(&stats[k], s_st[k]);
}

int64_t adj_scratch_doubles(const SceneDev& sc, int64_t grid_blocks, int wg)
{
    return adj_blocks(sc.Lmax) * 8 * grid_blocks * wg;
}

int64_t bwd_scratch_doubles(const SceneDev& sc, int64_t grid_blocks, int wg)
{
    const int64_t nthreads = grid_blocks * wg;
    const int64_t n_chk = adj_blocks(sc.Lmax);
    const int64_t n_waves = grid_blocks * ((wg + 63) / 64);
    return ((int64_t)sc.Kmax * kTapeStride + n_chk * 8) * nthreads
           + n_waves * ((int64_t)kQFields * 64 * (sc.Kmax + 1) + (int64_t)kHitFields * 64 * sc.Kmax);
}
