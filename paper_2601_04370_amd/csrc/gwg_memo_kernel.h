// Memoized thin-film adjoint.  Included by gwg_kernels.hip inside namespace gwg.
//
// The FoV beams are collimated, so within one work item (one design,
// wavelength and FoV point) the mirror hits share a handful of distinct
// (kappa, mirror, side, branch) keys: kappa is computed from direction bits
// that every ray with the same event history shares exactly.  The thin-film
// part of the gradient is linear in the cotangents,
//     sum_h 2 Re(G_h dc(kappa_h)/dt) = 2 Re((sum_{h in key} G_h) dc(kappa_key)/dt),
// so the backward sums the (dL/dI-scaled) cotangents of each key in entry
// order and runs one thin-film adjoint per key; the sums run in a fixed order,
// so the gradient is deterministic.  Entries come with their key's slot
// (k_key_sums, k_key_adj) unless their item met too many keys or their ray left
// the direction table.  Those are searched: one workgroup per item, kMemoWaves
// waves each take a contiguous part of the item's entries with their own key
// table, and wave 0 merges the tables in wave and key order.  An item with
// more than kMemoKeys keys is drained hit by hit instead.

constexpr int kMemoKeys = 128;      // keys per wave table and per item
constexpr int kMemoWaves = 4;       // waves per work item

// One wave's key table and chunk staging in LDS.
struct MemoLds {
    unsigned long long* kbits;   // [kMemoKeys] bits of kappa
    int* kmeta;                  // [kMemoKeys] mirror | front << 8 | reflected << 9
    double* gsum;                // [4][kMemoKeys] sums of G_s (re, im), G_p (re, im)
    int* sidx;                   // [64] key of each lane's entry in the current chunk (-1: none)
    double* sg;                  // [4][64] the lane's scaled cotangents
};

__host__ __device__ inline int memo_wave_bytes() { return kMemoKeys * (8 + 4 + 32) + 64 * (4 + 32); }

__device__ inline MemoLds memo_table(unsigned char* base, int w)
{
    unsigned char* mb = base + w * memo_wave_bytes();
    MemoLds mt;
    mt.kbits = (unsigned long long*)mb;
    mt.gsum = (double*)(mb + 8 * kMemoKeys);
    mt.sg = (double*)(mb + 40 * kMemoKeys);
    mt.kmeta = (int*)(mb + 40 * kMemoKeys + 32 * 64);
    mt.sidx = (int*)(mb + 44 * kMemoKeys + 32 * 64);
    return mt;
}

// Entry v (in item order) -> index of its record; cnt: the item's region counts.
__device__ inline int64_t entry_index(const AdjStore& st, int64_t item, const int32_t* cnt, int v)
{
    int rr = 0, k = v;
    while (k >= cnt[rr]) { k -= cnt[rr]; ++rr; }
    return (item * st.waves + rr) * st.cap_w + k;
}

// Whether an entry's key is searched for: all of an item's, or (rest: an item
// with keys) those of rays that left the direction table.
__device__ inline bool ent_searched(int64_t meta, bool rest) { return !rest || (int)(meta >> kEntSlotShift) == kNoSlot; }

// One wave: keys by first appearance in entries [v0, v1) and the dL/dI-scaled
// cotangents summed per key, in entry order (the next chunk's records are
// loaded while the current one is processed).  Returns the number of keys,
// or -1 if they exceed kMemoKeys.
__device__ inline int memo_collect(const SceneDev& sc, const AdjStore& st, int64_t item, const int32_t* cnt,
                                   const double* g_bins, int v0, int v1, bool rest, const MemoLds& mt)
{
    const int lane = wave_lane();
    const double invN = 1.0 / (double)sc.N;
    int U = 0;
    for (int k = lane; k < 4 * kMemoKeys; k += 64) mt.gsum[k] = 0.0;
    double nk = 0.0, ng[4] = { 0.0, 0.0, 0.0, 0.0 };
    int64_t nmeta = -1;
    auto fetch = [&](int c) {
        const int v = c + lane;
        nmeta = -1;
        if (v < v1) {
            const int64_t e = entry_index(st, item, cnt, v);
            const AdjEntry en = load_entry(st, e);
            nk = en.kappa;
            nmeta = en.meta;
            ng[0] = en.gs_re; ng[1] = en.gs_im; ng[2] = en.gp_re; ng[3] = en.gp_im;
        }
    };
    fetch(v0);
    for (int c = v0; c < v1; c += 64) {
        const double ck = nk;
        const int64_t cmeta = nmeta;
        const double cg0 = ng[0], cg1 = ng[1], cg2 = ng[2], cg3 = ng[3];
        if (c + 64 < v1) fetch(c + 64);
        double gscale = 0.0;
        if (cmeta >= 0 && ent_searched(cmeta, rest)) gscale = g_bins[ent_bin(cmeta)] * invN;
        const bool valid = gscale != 0.0;
        if (__ballot(valid) == 0ull) continue;
        const unsigned long long kb = (unsigned long long)__double_as_longlong(ck);
        const int km = (int)(cmeta & 1023);
        int idx = -1;
        if (valid)
            for (int u = 0; u < U; ++u)
                if (mt.kbits[u] == kb && mt.kmeta[u] == km) { idx = u; break; }
        for (;;) {
            const unsigned long long open = __ballot(valid && idx < 0);
            if (open == 0ull) break;
            if (U == kMemoKeys) return -1;
            const int leader = __ffsll((long long)open) - 1;
            const unsigned long long lkb = __shfl(kb, leader, 64);
            const int lkm = __shfl(km, leader, 64);
            if (lane == 0) { mt.kbits[U] = lkb; mt.kmeta[U] = lkm; }
            if (valid && idx < 0 && kb == lkb && km == lkm) idx = U;
            ++U;
        }
        mt.sidx[lane] = valid ? idx : -1;
        mt.sg[lane] = cg0 * gscale; mt.sg[64 + lane] = cg1 * gscale;
        mt.sg[128 + lane] = cg2 * gscale; mt.sg[192 + lane] = cg3 * gscale;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_s_waitcnt(0xc07f);      // this wave's LDS writes are visible (lgkmcnt = 0)
        for (int k = lane; k < U; k += 64) {
            double a0 = mt.gsum[k], a1 = mt.gsum[kMemoKeys + k];
            double a2 = mt.gsum[2 * kMemoKeys + k], a3 = mt.gsum[3 * kMemoKeys + k];
            for (int j = 0; j < 64; ++j)
                if (mt.sidx[j] == k) {
                    a0 += mt.sg[j]; a1 += mt.sg[64 + j]; a2 += mt.sg[128 + j]; a3 += mt.sg[192 + j];
                }
            mt.gsum[k] = a0; mt.gsum[kMemoKeys + k] = a1;
            mt.gsum[2 * kMemoKeys + k] = a2; mt.gsum[3 * kMemoKeys + k] = a3;
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_s_waitcnt(0xc07f);
    }
    return U;
}

// Wave 0 merges the key tables of waves 1.. into its own, in wave and key
// order (nk[w]: wave w's key count, -1 if its table overflowed).  Returns the
// merged key count, or -1 if a table overflowed or the merge would.
__device__ inline int memo_merge(unsigned char* mbase, const int* nk)
{
    const int lane = wave_lane();
    const MemoLds m0 = memo_table(mbase, 0);
    for (int w = 0; w < kMemoWaves; ++w)
        if (nk[w] < 0) return -1;
    int U = nk[0];
    for (int w = 1; w < kMemoWaves; ++w) {
        const MemoLds mw = memo_table(mbase, w);
        for (int u = 0; u < nk[w]; ++u) {
            const unsigned long long kb = mw.kbits[u];
            const int km = mw.kmeta[u];
            int idx = -1;
            for (int k = lane; k < U; k += 64)
                if (m0.kbits[k] == kb && m0.kmeta[k] == km) idx = k;
            const unsigned long long hit = __ballot(idx >= 0);
            if (hit) idx = __shfl(idx, __ffsll((long long)hit) - 1, 64);
            else {
                if (U == kMemoKeys) return -1;
                idx = U++;
                if (lane == 0) {
                    m0.kbits[idx] = kb; m0.kmeta[idx] = km;
                    for (int q = 0; q < 4; ++q) m0.gsum[q * kMemoKeys + idx] = 0.0;
                }
            }
            if (lane == 0)
                for (int q = 0; q < 4; ++q) m0.gsum[q * kMemoKeys + idx] += mw.gsum[q * kMemoKeys + u];
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_s_waitcnt(0xc07f);
        }
    }
    return U;
}

// ----------------------------------------------------- entries with keys
// Items whose forward kept the entries' key slots (AdjStore::n_keys >= 0):
// an entry's index is 2 slot + reflected, so no key is searched for.  A wave
// takes 64 entries at a time, one per lane: ballots of the index's bits give
// every lane the lanes of its key, the key's entries are added pairwise (each
// lane adds the sum that starts at the next entry of its key, the distance
// doubles), and the first lane of each key adds the result to the wave's sum.
// The waves' sums are added in wave order: the order of additions is fixed.
// About 150 vector and 25 LDS instructions per 64 entries (memo_collect: some
// 100 dependent LDS reads per entry), bound by the entries' 48 bytes.
// 1.1e7 rays over 1323 points, 5292 items: sums 0.44 ms and one adjoint per key
// of a point 0.55 ms, against 5.2 ms for memo_collect and an adjoint per key
// of an item; lanes that own keys and read every entry from LDS: 1.88 ms.
constexpr int kKeyIndex = 2 * kFwdMemoKeys;             // indices of an item
static_assert(kKeyIndex == 64 * kMemoWaves, "one index per thread");

// Called by the whole block (kMemoWaves waves): the dL/dI-scaled cotangents
// of the item's entries summed per index.  Thread i gets index i's sums;
// returns whether index i has an entry with a gradient.
__device__ inline bool key_sums(const SceneDev& sc, const AdjStore& st, int64_t item, const double* g_bins, double s[4])
{
    __shared__ double2 s_stage[kMemoWaves][2][64];
    __shared__ double2 s_sum[kMemoWaves][2][kKeyIndex];
    __shared__ int s_seen[kKeyIndex];
    const int tid = threadIdx.x, lane = wave_lane(), wave = tid / 64;
    const double invN = 1.0 / (double)sc.N;
    // entries before the end of each of the item's (at most four) regions
    int end[3], total = 0;
    for (int w = 0; w < 4; ++w) {
        if (w < st.waves) total += st.cnt[item * st.waves + w];
        if (w < 3) end[w] = total;
    }
    const int per = (total + kMemoWaves - 1) / kMemoWaves;
    const int v0 = min(wave * per, total), v1 = min(v0 + per, total);
    for (int q = 0; q < 2; ++q)
        for (int k = lane; k < kKeyIndex; k += 64) s_sum[wave][q][k] = make_double2(0.0, 0.0);
    s_seen[tid] = 0;
    __syncthreads();
    const int n_bits = 32 - __builtin_clz((unsigned)max(2 * st.n_keys[item] - 1, 1));
    const unsigned long long above = lane == 63 ? 0ull : ~0ull << (lane + 1), below = (1ull << lane) - 1ull;
    double2* const sum0 = s_sum[wave][0];
    double2* const sum1 = s_sum[wave][1];
    auto fetch = [&](int c) {
        const int v = c + lane;
        AdjEntry e{};
        e.meta = -1;
        if (v < v1) {
            const int r = (v >= end[0] ? 1 : 0) + (v >= end[1] ? 1 : 0) + (v >= end[2] ? 1 : 0);
            const int k = v - (r == 0 ? 0 : r == 1 ? end[0] : r == 2 ? end[1] : end[2]);
            e = load_entry(st, (item * st.waves + r) * st.cap_w + k);
        }
        return e;
    };
    auto bin_gradient = [&](const AdjEntry& e) { return e.meta >= 0 ? g_bins[ent_bin(e.meta)] : 0.0; };
    // the entries two chunks ahead and the bin gradients one chunk ahead are in flight
    AdjEntry e0 = fetch(v0), e1 = fetch(v0 + 64);
    double g0 = bin_gradient(e0);
    for (int c = v0; c < v1; c += 64) {
        const AdjEntry en = e0;
        const double gscale = g0 * invN;
        e0 = e1;
        g0 = bin_gradient(e0);
        e1 = fetch(c + 128);
        const int slot = (int)(en.meta >> kEntSlotShift);
        const bool valid = gscale != 0.0 && en.meta >= 0 && slot != kNoSlot;
        const int idx = slot << 1 | (int)((en.meta >> 9) & 1);
        unsigned long long peers = __ballot(valid);
        if (peers == 0ull) continue;
        for (int b = 0; b < n_bits; ++b) {
            const bool one = (idx >> b & 1) != 0;
            const unsigned long long ones = __ballot(one);
            peers &= one ? ones : ~ones;
        }
        const unsigned long long later = peers & above;
        int next = valid && later != 0ull ? __ffsll((long long)later) - 1 : -1;
        double2 x = make_double2(en.gs_re * gscale, en.gs_im * gscale);
        double2 y = make_double2(en.gp_re * gscale, en.gp_im * gscale);
        while (__ballot(next >= 0) != 0ull) {
            s_stage[wave][0][lane] = x;
            s_stage[wave][1][lane] = y;
            wave_lds_sync();
            const int nn = __shfl(next, next & 63);
            if (next >= 0) {
                const double2 px = s_stage[wave][0][next], py = s_stage[wave][1][next];
                x.x += px.x; x.y += px.y;
                y.x += py.x; y.y += py.y;
                next = nn;
            }
            wave_lds_sync();
        }
        if (valid && (peers & below) == 0ull) {
            const double2 px = sum0[idx], py = sum1[idx];
            sum0[idx] = make_double2(px.x + x.x, px.y + x.y);
            sum1[idx] = make_double2(py.x + y.x, py.y + y.y);
            s_seen[idx] = 1;
        }
        wave_lds_sync();
    }
    __syncthreads();
    double2 x = s_sum[0][0][tid], y = s_sum[0][1][tid];
    for (int w = 1; w < kMemoWaves; ++w) {
        const double2 px = s_sum[w][0][tid], py = s_sum[w][1][tid];
        x.x += px.x; x.y += px.y;
        y.x += py.x; y.y += py.y;
    }
    s[0] = x.x; s[1] = x.y; s[2] = y.x; s[3] = y.y;
    return s_seen[tid] != 0;
}

// kappa and meta (mirror | front << 8 | reflected << 9) of a key.
__device__ inline void key_hit(const SceneDev& sc, int64_t dir_point, int key, int refl, double* kappa, int* meta)
{
    const int es = key / sc.M, m = key - es * sc.M;
    const double* g = sc.dirs + (dir_point * kDirMax + (es >> 1)) * kDirWords;
    *kappa = g[DG_KAP + (es & 1)];
    *meta = m | (g[DG_DN + 2 * (es & 1)] < 0.0 ? 1 << 8 : 0) | refl << 9;
}

// One workgroup per item: its sums to sum[item][kKeyIndex][4], the indices
// that have one in seen[item][kMemoWaves] (a bit each).
__global__ void __launch_bounds__(64 * kMemoWaves, 4) k_key_sums(SceneDev sc, const double* __restrict__ dLdI, AdjStore st,
                                                              double* __restrict__ sum,
                                                              unsigned long long* __restrict__ seen)
{
    for (int64_t item = blockIdx.x; item < sc.n_items; item += gridDim.x) {
        if (st.ovf[item] != 0 || st.n_keys[item] < 0) continue;
        double s[4];
        const bool nz = key_sums(sc, st, item, dLdI + item / sc.tiles_per_point * (sc.bins_x * sc.bins_y), s);
        const unsigned long long b = __ballot(nz);
        if (wave_lane() == 0) seen[item * kMemoWaves + threadIdx.x / 64] = b;
        if (nz) {
            double2* o = (double2*)(sum + (item * kKeyIndex + threadIdx.x) * 4);
            o[0] = make_double2(s[0], s[1]);
            o[1] = make_double2(s[2], s[3]);
        }
        __syncthreads();
    }
}

// The thin-film adjoints of a point's keys.  The items of a point share its
// directions, so their sums are first added per key, in item order (lane by
// lane in LDS, the next item's sums in flight), and each key then takes one
// adjoint: a wave's adjoint of 200 layers takes about 0.1 ms however few of
// its lanes have a key, and a point has tens of items.  kKeyParts workgroups
// of one wave per point, each with the same sums; they share the chunks of
// 64 keys.  The gradient of part p goes to the partial row of the point's
// p-th item with keys; the rows of its other items with keys are zeroed.
constexpr int kKeyParts = 2;
constexpr int kPointKeys = 256;                          // keys at a time; more: adjoints in between

__host__ __device__ inline int point_key_bytes(int M)
{
    return 2 * kPointKeys * 32 + align16(2 * 2 * kDirMax * M) + 2 * kPointKeys * 4 + 2 * kPointKeys * 2;
}

template <bool LOSSLESS>
__global__ void __launch_bounds__(64, 1) k_key_adj(SceneDev sc, AdjStore st, const double* __restrict__ sum,
                                                   const unsigned long long* __restrict__ seen,
                                                   double* __restrict__ partial, double* __restrict__ scratch,
                                                   unsigned long long* __restrict__ stats)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const SmemLayout lay = smem_layout(sc.M, sc.Lmax, sc.n_slots, 64, sc.bins_x * sc.bins_y, false, 1);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    double* s_thk = (double*)(smem + lay.off_thk);
    uint8_t* s_slot = (uint8_t*)(smem + lay.off_slot);
    double* s_sp = (double*)(smem + lay.off_sp);
    double* gw = (double*)(smem + lay.off_grad);
    unsigned char* mem = smem + align16(lay.total);
    double* acc = (double*)mem;                                              // [2 kPointKeys][4]
    uint16_t* slot = (uint16_t*)(mem + 2 * kPointKeys * 32);                 // [2 kDirMax M] key -> its place here
    int* has = (int*)((unsigned char*)slot + align16(2 * 2 * kDirMax * sc.M));   // [2 kPointKeys]
    uint16_t* key_of = (uint16_t*)(has + 2 * kPointKeys);                    // [kPointKeys]
    uint16_t* list = key_of + kPointKeys;                                    // [64 ..] chunk of indices
    const int lane = wave_lane();
    const int ML = sc.M * sc.Lmax;
    const LaneSlots3 sl = { slot_lane_base(s_sp, sc.n_slots, LaneSlots3::kPer, lane), pl->nsq, pl->pxy };
    const int64_t nthreads = (int64_t)gridDim.x * 64;
    double* chk = scratch + (int64_t)blockIdx.x * 64 + lane;
    const int n_key = 2 * kDirMax * sc.M;
    const int64_t n_tiles = sc.tiles_per_point;
    const int64_t n_points = sc.n_items / n_tiles;
    unsigned long long c_keys = 0, c_lay = 0;

    for (int64_t b = blockIdx.x; b < n_points * kKeyParts; b += gridDim.x) {
        const int64_t first = b / kKeyParts * n_tiles;
        const int part = (int)(b % kKeyParts);
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, first, &point, &d, &l, &f, &i0, &i1);
        const int64_t dir_point = (int64_t)l * sc.F + f;
        int keyed = 0;                                                       // the point's items with keys
        for (int64_t t = 0; t < n_tiles; t += 64) {
            const bool k = t + lane < n_tiles && st.ovf[first + t + lane] == 0 && st.n_keys[first + t + lane] >= 0;
            keyed += __popcll(__ballot(k));
        }
        const int parts = min(kKeyParts, keyed);
        if (part >= parts) continue;
        __syncthreads();                                                     // the last point's LDS is read
        stage_point(sc, d, l, f, pl, s_thk, s_slot);
        for (int k = lane; k < ML; k += 64) gw[k] = 0.0;
        int U = 0, chunk = 0;
        auto reset = [&]() {
            for (int k = lane; k < n_key; k += 64) slot[k] = 0xffff;
            for (int k = lane; k < 2 * kPointKeys; k += 64) {
                has[k] = 0;
                for (int q = 0; q < 4; ++q) acc[4 * k + q] = 0.0;
            }
            U = 0;
            __syncthreads();
        };
        // the adjoints of the keys gathered so far: this part's chunks of 64
        // indices that have a sum
        auto adjoints = [&]() {
            int n = 0;
            auto run = [&](int cnt) {
                __syncthreads();
                if (chunk % parts == part && lane < cnt) {
                    const int i = list[lane];
                    double kappa;
                    int mm;
                    key_hit(sc, dir_point, key_of[i >> 1], i & 1, &kappa, &mm);
                    const double* g = acc + 4 * i;
                    adjoint_hit<LOSSLESS ? ADJ_LOSSLESS : ADJ_ABSORBING>(sc.n_slots, sc.slot_complex, sc.Lmax, *pl, s_thk, s_slot, sl, gw, kappa, mk(g[0], g[1]),
                                                                         mk(g[2], g[3]), mm, chk, nthreads);
                    c_keys += 1;
                    c_lay += (unsigned long long)pl->nlay[mm & 255];
                }
                ++chunk;
                __syncthreads();
            };
            for (int k = 0; k < 2 * U; k += 64) {
                const bool h = k + lane < 2 * U && has[k + lane] != 0;
                const unsigned long long bal = __ballot(h);
                const int at = n + __popcll(bal & ((1ull << lane) - 1ull)), more = __popcll(bal);
                if (h && at < 64) list[at] = (uint16_t)(k + lane);
                if (n + more >= 64) {
                    run(64);
                    if (h && at >= 64) list[at - 64] = (uint16_t)(k + lane);
                    n = n + more - 64;
                } else {
                    n += more;
                }
            }
            if (n > 0) run(n);
        };
        reset();
        // the next item's keys and sums (of indices without one: not used)
        constexpr int kSets = kKeyIndex / 64;
        int nk = -1, key[kFwdMemoKeys / 64];
        unsigned long long sn[kSets];
        double2 v[kSets][2];
        auto fetch = [&](int64_t item) {
            nk = st.ovf[item] != 0 ? -1 : st.n_keys[item];
#pragma unroll
            for (int t = 0; t < kFwdMemoKeys / 64; ++t) key[t] = st.keys[item * kFwdMemoKeys + t * 64 + lane];
#pragma unroll
            for (int t = 0; t < kSets; ++t) {
                sn[t] = seen[item * kSets + t];
                const double2* p = (const double2*)(sum + (item * kKeyIndex + t * 64 + lane) * 4);
                v[t][0] = p[0];
                v[t][1] = p[1];
            }
        };
        int64_t row = -1;
        int ord = 0;
        fetch(first);
        for (int64_t t = 0; t < n_tiles; ++t) {
            const int64_t item = first + t;
            const int n = __builtin_amdgcn_readfirstlane(nk);
            int ky[kFwdMemoKeys / 64];
            unsigned long long sb[kSets];
            double2 w[kSets][2];
#pragma unroll
            for (int q = 0; q < kFwdMemoKeys / 64; ++q) ky[q] = key[q];
#pragma unroll
            for (int q = 0; q < kSets; ++q) { sb[q] = sn[q]; w[q][0] = v[q][0]; w[q][1] = v[q][1]; }
            if (t + 1 < n_tiles) fetch(item + 1);
            if (n < 0) continue;
            if (ord == part) row = item;
            else if (ord >= parts && ord % parts == part)
                for (int k = lane; k < ML; k += 64) partial[item * ML + k] = 0.0;
            ++ord;
            if (U + n > kPointKeys) {                                        // an item's keys fit an empty table
                int fresh_all = 0;
#pragma unroll
                for (int q = 0; q < kFwdMemoKeys / 64; ++q)
                    fresh_all += __popcll(__ballot(q * 64 + lane < n && slot[ky[q]] == 0xffff));
                if (U + fresh_all > kPointKeys) {
                    adjoints();
                    reset();
                }
            }
            int place[kFwdMemoKeys / 64];
#pragma unroll
            for (int q = 0; q < kFwdMemoKeys / 64; ++q) {
                const bool in = q * 64 + lane < n;
                place[q] = in ? slot[ky[q]] : 0;
                const bool fresh = in && place[q] == 0xffff;
                const unsigned long long bal = __ballot(fresh);
                if (fresh) {
                    place[q] = U + __popcll(bal & ((1ull << lane) - 1ull));
                    slot[ky[q]] = (uint16_t)place[q];
                    key_of[place[q]] = (uint16_t)ky[q];
                }
                U += __popcll(bal);
            }
#pragma unroll
            for (int q = 0; q < kSets; ++q) {
                // index 64 q + lane: branch lane & 1 of slot 32 q + lane / 2
                const int pl_ = __shfl(place[q / 2], (q & 1) * 32 + (lane >> 1));
                if (sb[q] >> lane & 1ull) {
                    const int i = 2 * pl_ + (lane & 1);
                    double2* o = (double2*)(acc + 4 * i);
                    const double2 x = o[0], y = o[1];
                    o[0] = make_double2(x.x + w[q][0].x, x.y + w[q][0].y);
                    o[1] = make_double2(y.x + w[q][1].x, y.y + w[q][1].y);
                    has[i] = 1;
                }
            }
            __syncthreads();
        }
        adjoints();
        __syncthreads();
        for (int k = lane; k < ML; k += 64) partial[row * ML + k] = gw[k];
    }
    if (c_keys) atomicAdd(&stats[ST_ADJ_HITS], c_keys);
    if (c_lay) atomicAdd(&stats[ST_ADJ_LAYERS], c_lay);
}
static_assert(kPointKeys >= kFwdMemoKeys && kKeyIndex == 2 * kFwdMemoKeys && kFwdMemoKeys % 64 == 0, "key tables");

size_t key_adj_smem_bytes(const SceneDev& sc)
{
    return (size_t)align16(smem_layout(sc.M, sc.Lmax, sc.n_slots, 64, sc.bins_x * sc.bins_y, false, 1).total) +
           (size_t)point_key_bytes(sc.M);
}
int64_t key_adj_blocks(const SceneDev& sc) { return sc.n_items / sc.tiles_per_point * kKeyParts; }
int64_t key_sum_doubles(const SceneDev& sc) { return sc.n_items * (int64_t)(kKeyIndex * 4 + kMemoWaves); }

template <bool LOSSLESS>
__global__ void __launch_bounds__(64 * kMemoWaves, 2) k_adj_memo(SceneDev sc, const double* __restrict__ dLdI,
                                                              double* __restrict__ partial, AdjStore st,
                                                              double* __restrict__ scratch,
                                                              unsigned long long* __restrict__ stats)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int B = sc.bins_x * sc.bins_y;
    const SmemLayout lay = smem_layout(sc.M, sc.Lmax, sc.n_slots, 64, B, false, 1);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    double* s_thk = (double*)(smem + lay.off_thk);
    uint8_t* s_slot = (uint8_t*)(smem + lay.off_slot);
    double* s_sp = (double*)(smem + lay.off_sp);
    double* gw = (double*)(smem + lay.off_grad);
    unsigned long long* s_st = (unsigned long long*)(smem + lay.off_st);
    unsigned char* mbase = smem + align16(lay.total);
    int* s_nkeys = (int*)(mbase + kMemoWaves * memo_wave_bytes());
    const int tid = threadIdx.x, wave = tid / 64, lane = wave_lane();
    const MemoLds mt = memo_table(mbase, wave);
    const MemoLds m0 = memo_table(mbase, 0);
    const int ML = sc.M * sc.Lmax;
    const LaneSlots3 sl = { slot_lane_base(s_sp, sc.n_slots, LaneSlots3::kPer, lane), pl->nsq, pl->pxy };     // wave 0's lanes
    const int64_t nthreads = (int64_t)gridDim.x * 64;
    double* chk = scratch + (int64_t)blockIdx.x * 64 + lane;
    for (int k = tid; k < ST_WORDS; k += 64 * kMemoWaves) s_st[k] = 0ull;
    unsigned long long c_keys = 0, c_lay = 0;

    const int64_t n_it = st.n_keys ? (int64_t)st.unkeyed[0] : sc.n_items;    // only the items with entries without keys
    for (int64_t it = draw_item(stats + ST_NEXT0); it < n_it; it = draw_item(stats + ST_NEXT0)) {
        const int64_t item = st.n_keys ? (int64_t)st.unkeyed[1 + it] : it;
        if (st.ovf[item] != 0) continue;
        const bool rest = st.n_keys && st.n_keys[item] >= 0;                 // added to k_key_adj's row
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, item, &point, &d, &l, &f, &i0, &i1);
        stage_point(sc, d, l, f, pl, s_thk, s_slot);
        for (int k = tid; k < ML; k += 64 * kMemoWaves) gw[k] = 0.0;
        const double* g_bins = dLdI + point * B;
        const int32_t* cnt = st.cnt + item * st.waves;
        int total = 0;
        for (int w = 0; w < st.waves; ++w) total += cnt[w];
        // wave w takes a contiguous part of the entries
        const int per = (total + kMemoWaves - 1) / kMemoWaves;
        const int v0 = min(wave * per, total), v1 = min(v0 + per, total);
        const int nk = memo_collect(sc, st, item, cnt, g_bins, v0, v1, rest, mt);
        if (lane == 0) s_nkeys[wave] = nk;
        __syncthreads();
        if (wave == 0) {
            const int U = memo_merge(mbase, s_nkeys);
            if (U < 0) {
                // too many keys: one thin-film adjoint per entry
                const double invN = 1.0 / (double)sc.N;
                for (int c = 0; c < total; c += 64) {
                    const int v = c + lane;
                    if (v < total) {
                        const int64_t e = entry_index(st, item, cnt, v);
                        const AdjEntry en = load_entry(st, e);
                        const int64_t meta = en.meta;
                        const double gscale = ent_searched(meta, rest) ? g_bins[ent_bin(meta)] * invN : 0.0;
                        if (gscale != 0.0) {
                            const cd Gs = cscale(mk(en.gs_re, en.gs_im), gscale);
                            const cd Gp = cscale(mk(en.gp_re, en.gp_im), gscale);
                            const int mm = (int)(meta & 1023);
                            adjoint_hit<LOSSLESS ? ADJ_LOSSLESS : ADJ_ABSORBING>(sc.n_slots, sc.slot_complex, sc.Lmax, *pl, s_thk, s_slot, sl, gw, en.kappa, Gs, Gp, mm, chk, nthreads);
                            c_keys += 1;
                            c_lay += (unsigned long long)pl->nlay[mm & 255];
                        }
                    }
                }
            } else {
                // one thin-film adjoint per key
                for (int b = 0; b < U; b += 64) {
                    const int k = b + lane;
                    if (k < U) {
                        const cd Gs = mk(m0.gsum[k], m0.gsum[kMemoKeys + k]);
                        const cd Gp = mk(m0.gsum[2 * kMemoKeys + k], m0.gsum[3 * kMemoKeys + k]);
                        const int mm = m0.kmeta[k];
                        adjoint_hit<LOSSLESS ? ADJ_LOSSLESS : ADJ_ABSORBING>(sc.n_slots, sc.slot_complex, sc.Lmax, *pl, s_thk, s_slot, sl, gw,
                                              __longlong_as_double((long long)m0.kbits[k]), Gs, Gp, mm, chk, nthreads);
                        c_keys += 1;
                        c_lay += (unsigned long long)pl->nlay[mm & 255];
                    }
                }
            }
        }
        __syncthreads();
        double* out = partial + item * (int64_t)ML;
        for (int k = tid; k < ML; k += 64 * kMemoWaves) out[k] = rest ? out[k] + gw[k] : gw[k];
    }
    if (c_keys) atomicAdd(&s_st[ST_ADJ_HITS], c_keys);
    if (c_lay) atomicAdd(&s_st[ST_ADJ_LAYERS], c_lay);
    __syncthreads();
    for (int k = tid; k < ST_WORDS; k += 64 * kMemoWaves)
        if (s_st[k]) atomicAdd(&stats[k], s_st[k]);
}

size_t memo_smem_bytes(const SceneDev& sc)
{
    return (size_t)align16(smem_layout(sc.M, sc.Lmax, sc.n_slots, 64, sc.bins_x * sc.bins_y, false, 1).total) +
           (size_t)(kMemoWaves * memo_wave_bytes() + 16);
}
