// HIP kernels for gfx950: batched thin-film solve, forward Monte Carlo trace
// with fixed-point eyebox scatter, adjoint trace, gradient reduction,
// irradiance and loss.  Launch wrappers at the end are the only entry points
// used by the host API (gwg_api.cpp).
#include <cstring>
#include <mutex>
#include <type_traits>

#include "gwg_internal.h"
#include "gwg_device.h"
#include "gwg_adjoint.h"
#include "gwg_trace.h"
#include "gwg_launch.h"

namespace gwg {

// ------------------------------------------------------------------ fills
__global__ void k_fill_u64(uint64_t* p, int64_t n, uint64_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_f64(double* p, int64_t n, double v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// --------------------------------------------------------- LDS arrangement
struct SmemLayout {
    int off_pl, off_thk, off_slot, off_sp, off_q, off_c, off_st, off_grad, total;
};

__host__ __device__ inline int align16(int x) { return (x + 15) & ~15; }

// recs: the stacks as layer records (LayerRec, off_thk; no slot array)
// rather than thickness and slot arrays.
__host__ __device__ inline SmemLayout smem_layout(int M, int Lmax, int n_slots, int wg, int B,
                                                  bool lds_bins, int n_grad_regions, int slot_per = LaneSlots3::kPer,
                                                  bool recs = false)
{
    SmemLayout s;
    int o = 0;
    s.off_pl = o; o = align16(o + (int)sizeof(PointLds));
    s.off_thk = o; o = align16(o + (recs ? (int)sizeof(LayerRec) * M * rec_stride(Lmax) : 8 * M * Lmax));
    s.off_slot = o; o = align16(o + (recs ? 0 : M * Lmax));
    s.off_sp = o; o = align16(o + 8 * n_slots * slot_per * ((wg + 63) / 64 * 64));   // whole waves
    s.off_q = o; o = align16(o + (lds_bins ? 8 * B : 0));
    s.off_c = o; o = align16(o + (lds_bins ? 4 * B : 0));
    s.off_st = o; o = align16(o + 8 * ST_WORDS);
    s.off_grad = o; o = align16(o + 8 * n_grad_regions * M * Lmax);
    s.total = o;
    return s;
}

// Stage one point's uniform data and its design's stacks into LDS: as
// thickness and slot arrays (s_thk, s_slot) or as layer records (s_rec, for
// slot tables of `per` values per slot); neither: no stacks.
__device__ inline void stage_point(const SceneDev& sc, int d, int l, int f, PointLds* pl,
                                   double* s_thk, uint8_t* s_slot, LayerRec* s_rec = nullptr, int per = 0)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    const double* lt = sc.lam_tab + (int64_t)l * LT_STRIDE;
    if (tid == 0) {
        pl->k0 = lt[LT_K0];
        pl->ng = lt[LT_NG];
        pl->na = lt[LT_NA];
        if (sc.fov_mode == 0) {
            const double* dv = sc.dir_tab + ((int64_t)l * sc.F + f) * 4;
            pl->dir[0] = dv[0]; pl->dir[1] = dv[1]; pl->dir[2] = dv[2];
        }
        double k2e = 1e300;
        for (int s = 0; s < sc.n_slots; ++s)
            if (!((sc.slot_complex >> s) & 1u)) {
                const double nr = lt[LT_SLOT + 2 * s];
                k2e = fmin(k2e, nr * nr);
            }
        pl->kap2_evan = k2e;
        for (int s = 0; s < kMaxSlots; ++s) {
            double nr = lt[LT_SLOT + 2 * s], ni = lt[LT_SLOT + 2 * s + 1];
            pl->slotN[2 * s] = nr; pl->slotN[2 * s + 1] = ni;
            pl->nsq[2 * s] = nr * nr - ni * ni; pl->nsq[2 * s + 1] = 2.0 * nr * ni;
            pl->pxy[2 * s] = (ni == 0.0 && nr != 0.0) ? 1.0 / (nr * nr) : 0.0;
            pl->pxy[2 * s + 1] = nr * nr - ni * ni;
            pl->crit[2 * s] = lt[LT_CRIT + 2 * s]; pl->crit[2 * s + 1] = lt[LT_CRIT + 2 * s + 1];
        }
        for (int m = 0; m < sc.M; ++m) {
            pl->h[m] = sc.h[m]; pl->sc_r[m] = sc.sc_r[m]; pl->sc_t[m] = sc.sc_t[m];
            pl->thr[m] = sc.thr[m];
            pl->nlay[m] = sc.nlay[(int64_t)d * sc.M + m];
        }
        pl->T = sc.T; pl->Lx = sc.Lx; pl->nx = sc.nx; pl->nz = sc.nz; pl->ER = sc.ER;
        pl->ex0 = sc.ex0; pl->ew = sc.ew; pl->ey0 = sc.ey0; pl->eh = sc.eh;
        pl->M = sc.M; pl->Kmax = sc.Kmax; pl->bins_x = sc.bins_x; pl->bins_y = sc.bins_y;
    }
    const int n = sc.M * sc.Lmax;
    const double* gthk = sc.thk + (int64_t)d * n;
    const uint8_t* gslot = sc.slot + (int64_t)d * n;
    if (s_rec)
        stage_recs(s_rec, gthk, gslot, sc.M, sc.Lmax, per);
    else if (s_thk)
        for (int i = tid; i < n; i += nt) { s_thk[i] = gthk[i]; s_slot[i] = gslot[i]; }
}

__device__ inline void decode_item(const SceneDev& sc, int64_t item, int64_t* point, int* d, int* l,
                                   int* f, int64_t* i0, int64_t* i1)
{
    int64_t pt = item / sc.tiles_per_point;
    int64_t tile = item - pt * sc.tiles_per_point;
    *point = pt;
    *f = (int)(pt % sc.F);
    int64_t rest = pt / sc.F;
    *l = (int)(rest % sc.n_lsel);
    *d = (int)(rest / sc.n_lsel);
    *i0 = tile * sc.rays_per_tile;
    int64_t e = *i0 + sc.rays_per_tile;
    *i1 = e < sc.N ? e : sc.N;
}

// Work items are drawn from a launch-wide counter (a stats word cleared
// before the launch) rather than by a fixed stride over blocks: a block that
// drew cheap items goes on to the next one, so the launch ends within about
// one item of the mean.  Every output is indexed by item, never by block,
// so results do not depend on which block ran an item.  Called by the whole
// block.
__device__ inline int64_t draw_item(unsigned long long* ctr)
{
    __shared__ long long s_item;
    __syncthreads();                                   // the previous draw has been read
    if (threadIdx.x == 0) s_item = (long long)atomicAdd(ctr, 1ull);
    __syncthreads();
    return s_item;
}

#include "gwg_table.h"
#include "gwg_dirs.h"
#include "gwg_fwd_kernel.h"
#include "gwg_bwd_kernel.h"
#include "gwg_adj_kernel.h"
#include "gwg_memo_kernel.h"
#include "gwg_table_kernel.h"
#include "gwg_omega_kernel.h"

// Gradient reduction over the per-item partials, in two launches with a
// fixed order of additions (the gradient is the same bit for bit from run to
// run): range r of kGradRanges contiguous item ranges of a design is summed
// in item order, then the range sums in range order.
constexpr int kGradRanges = 64;

// Rows of `partial`: the design's work items, or (left given) its groups of
// items, and then its regenerated items' rows (ovf) in `regen`.
__global__ void k_grad_ranges(const double* __restrict__ partial, int64_t rows_per_design, int ML,
                              const double* __restrict__ regen, int64_t items_per_design, const int32_t* __restrict__ ovf,
                              const int32_t* __restrict__ left, double* __restrict__ tmp)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y, d = blockIdx.z;
    if (k >= ML) return;
    const int64_t a = rows_per_design * r / kGradRanges, b = rows_per_design * (r + 1) / kGradRanges;
    const double* p = partial + (int64_t)d * rows_per_design * ML + k;
    double acc = 0.0;
    for (int64_t it = a; it < b; ++it) acc += p[it * ML];
    if (left && left[0] > 0) {
        const int64_t i0 = (int64_t)d * items_per_design;
        const int64_t ia = items_per_design * r / kGradRanges, ib = items_per_design * (r + 1) / kGradRanges;
        for (int64_t it = i0 + ia; it < i0 + ib; ++it)
            if (ovf[it]) acc += regen[it * ML + k];
    }
    tmp[((int64_t)d * kGradRanges + r) * ML + k] = acc;
}

__global__ void k_grad_reduce(const double* __restrict__ tmp, int ML, int D, double* __restrict__ grad)
{
    int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)D * ML) return;
    int d = (int)(gid / ML), k = (int)(gid % ML);
    const double* p = tmp + (int64_t)d * kGradRanges * ML + k;
    double acc = 0.0;
    for (int r = 0; r < kGradRanges; ++r) acc += p[(int64_t)r * ML];
    grad[gid] = acc;
}

int64_t grad_reduce_tmp_doubles(int ML, int D) { return (int64_t)D * kGradRanges * ML; }

// Work items in decreasing order of a per-(item, wave) work count summed
// over the item's waves (adjoint entries; mirror hits of the last forward),
// by a counting sort over count >> shift in one workgroup.  Items in one
// bucket are placed in no particular order; the kernels' outputs are indexed
// by item, so their results do not depend on it.
constexpr int kOrderBuckets = 2048;

__global__ void __launch_bounds__(1024) k_item_order(const int32_t* __restrict__ cnt, int waves, int64_t n_items,
                                                     int shift, int32_t* __restrict__ order)
{
    __shared__ int hist[kOrderBuckets];
    __shared__ int part[1024];
    const int t = threadIdx.x;
    auto bucket = [&](int64_t it) {
        long long n = 0;
        for (int w = 0; w < waves; ++w) n += cnt[it * waves + w];
        const long long b = n > 0 ? n >> shift : 0;     // any count maps into the histogram
        return kOrderBuckets - 1 - (int)(b < kOrderBuckets ? b : kOrderBuckets - 1);   // largest first
    };
    for (int k = t; k < kOrderBuckets; k += 1024) hist[k] = 0;
    __syncthreads();
    for (int64_t it = t; it < n_items; it += 1024) atomicAdd(&hist[bucket(it)], 1);
    __syncthreads();
    // exclusive prefix sum over the buckets: two per thread, then a scan of
    // the 1024 pair sums
    const int a0 = hist[2 * t], a1 = hist[2 * t + 1];
    part[t] = a0 + a1;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int v = t >= o ? part[t - o] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    const int base = part[t] - (a0 + a1);
    hist[2 * t] = base;
    hist[2 * t + 1] = base + a0;
    __syncthreads();
    for (int64_t it = t; it < n_items; it += 1024) order[atomicAdd(&hist[bucket(it)], 1)] = (int32_t)it;
}

hipError_t launch_item_order(const int32_t* cnt, int waves, int64_t n_items, int64_t max_count, int32_t* order,
                             hipStream_t s)
{
    int shift = 0;
    while ((max_count >> shift) >= kOrderBuckets) ++shift;
    hipLaunchKernelGGL(k_item_order, dim3(1), dim3(1024), 0, s, cnt, waves, n_items, shift, order);
    return hipGetLastError();
}

__global__ void k_mask_padding(double* grad, const int32_t* nlay, int D, int M, int Lmax)
{
    int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)D * M * Lmax) return;
    int j = (int)(gid % Lmax);
    int64_t dm = gid / Lmax;
    if (j >= nlay[dm]) grad[gid] = 0.0;
}

__global__ void k_irradiance(const uint64_t* __restrict__ q, int64_t n, double scale, double* __restrict__ irr)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        irr[i] = (double)q[i] * scale;
}

// ======================================================== thin-film queries
// SORT: a workgroup takes `chunk` queries at a time and solves them by kind:
// double precision or single, with an evanescent layer or without.  Queries of
// all kinds side by side (angles and wavelengths in any order) make nearly
// every wave run the hyperbolic case and, with mixed precision, both solves.
// The waves draw batches of 64 from the list of the chunk's queries by kind,
// the dearest first; a batch over a border of kinds runs what its queries need.
// Else: queries in order, one a lane (tmm_sorted's rule).
// Results do not depend on it.  Bound by vector issue.  2^20 queries, in order
// and by kind:
//   200 lossless layers, double precision: 469 and 422 us (40 % evanescent:
//     355 us if every wave had one kind and issued a vector instruction always)
//   201 layers, one of them silver, mixed: 1287 and 619 us
// chunk: a multiple of 64, at most kTmmChunk.
constexpr int kTmmChunk = 2048;
constexpr int kTmmKinds = 4;                 // double 0, 1; single 2, 3; without an evanescent layer: odd

// The wavelength rows and the layers' slots as they travel with the launch.
struct TmmTab { alignas(16) unsigned char b[kTmmTabBytes]; };
struct TmmNoTab {};

template <int MODE, bool VAL, bool SORT>
__global__ void __launch_bounds__(256, MODE == GWG_FP32 ? 3 : 2) k_tmm_rt(const double* __restrict__ thk, const uint8_t* __restrict__ slot_p,
                                                int L, const double* __restrict__ lam_p, int n_lambda,
                                                TmmRows rows, const int32_t* __restrict__ lidx,
                                                const double* __restrict__ theta, int64_t nq,
                                                double* __restrict__ out, int chunk,
                                                const typename std::conditional<VAL, TmmTab, TmmNoTab>::type tab)
{
    const double* lam_tab = lam_p;
    const uint8_t* slot = slot_p;
    if constexpr (VAL) {
        lam_tab = (const double*)tab.b;
        slot = tab.b + (int64_t)n_lambda * rows.stride() * 8;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    LayerRec* s_rec = (LayerRec*)smem;
    double* s_sp = (double*)(smem + sizeof(LayerRec) * rec_stride(L));
    stage_recs(s_rec, thk, slot, 1, L, LaneSlots5::kPer);
    const int tid = threadIdx.x, lane = tid & 63;
    const int n_slots = rows.n_slots;
    const LaneSlots5 sl = { slot_lane_base(s_sp, n_slots, LaneSlots5::kPer, tid) };
    const RecStack stk = { s_rec + kRecPad };
    // kappa and kind of a valid query
    auto kind_of = [&](const double* lt, double th, double* kappa, bool* fp64) {
        *kappa = lt[TR_NG] * sin(th);
        *fp64 = (MODE == GWG_FP64);
        bool evan = false;
        for (int s = 0; s < n_slots; ++s) {
            // slot_params: an evanescent lossless slot
            const double nr = lt[TR_SLOT + s];
            evan |= !((rows.cplx >> s) & 1u) && nr * nr - *kappa * *kappa <= -kTinyZ;
        }
        if (MODE == GWG_FP32_MIXED)
            for (int k = 0; k < rows.n_crit; ++k) {
                const double* c = lt + rows.crit(k);
                *fp64 |= *kappa > c[0] && *kappa < c[1];
            }
        return (*fp64 ? 0 : 2) + (evan ? 0 : 1);
    };
    auto valid = [&](int li, double th) { return li >= 0 && li < n_lambda && th >= 0.0 && th < 1.5707963267948966; };
    auto solve = [&](int64_t q) {
        const int li = lidx[q];
        const double th = theta[q];
        double* o = out + q * 8;
        if (!valid(li, th)) {
            for (int k = 0; k < 8; ++k) o[k] = __builtin_nan("");
            return;
        }
        const double* lt = lam_tab + (int64_t)li * rows.stride();
        const double k0 = lt[TR_K0], n0 = lt[TR_NG];
        const cd NE = mk(lt[TR_NA], lt[TR_NA + 1]);
        double kappa;
        bool fp64;
        const bool circ = __ballot((kind_of(lt, th, &kappa, &fp64) & 1) == 0) == 0ull;
        for (int s = 0; s < n_slots; ++s) {
            double P[NPF];
            const bool ab = (rows.cplx >> s) & 1u;
            slot_params(lt[TR_SLOT + s], ab ? lt[rows.imag(s)] : 0.0, ab, kappa, k0, P);
            sl.put(s, P);
        }
        const double z0 = n0 * n0 - kappa * kappa;
        const double q0 = sqrt(z0 > kTinyZ ? z0 : kTinyZ);
        const cd NE2 = cmul(NE, NE);
        cd zE = csub(NE2, mk(kappa * kappa, 0.0));
        if (zE.im == 0.0 && fabs(zE.re) < kTinyZ) zE.re = kTinyZ;
        const cd qE = csqrt_up(zE);
        const cd etaEp = cdiv(NE2, qE);
        // t_p factor cos(theta_0) / cos(theta_exit) = (q0 / n0) / (qE / NE)
        const cd tpf = cdiv(cscale(NE, q0 / n0), qE);
        const Coef4 c =
            fp64 ? tmm_solve<double, false, false, true>(stk, L, true, sl, rows.cplx, k0, q0, n0 * n0 / q0, qE, etaEp, tpf, circ)
                 : tmm_solve<float, false, false, true>(stk, L, true, sl, rows.cplx, k0, q0, n0 * n0 / q0, qE, etaEp, tpf, circ);
        o[0] = c.rs.re; o[1] = c.rs.im; o[2] = c.rp.re; o[3] = c.rp.im;
        o[4] = c.ts.re; o[5] = c.ts.im; o[6] = c.tp.re; o[7] = c.tp.im;
    };
    if constexpr (!SORT) {
        __syncthreads();                                         // the records
        for (int64_t q = (int64_t)blockIdx.x * 256 + tid; q < nq; q += (int64_t)gridDim.x * 256) solve(q);
        return;
    }
    __shared__ int s_n[kTmmKinds], s_next;
    uint16_t* s_list = (uint16_t*)(s_sp + (int64_t)n_slots * LaneSlots5::kPer * 256);
    for (int64_t c0 = (int64_t)blockIdx.x * chunk; c0 < nq; c0 += (int64_t)gridDim.x * chunk) {
        const int n = (int)min((int64_t)chunk, nq - c0);
        __syncthreads();                                     // the records; the last chunk's list is read
        if (tid < kTmmKinds) s_n[tid] = 0;
        if (tid == 0) s_next = 0;
        __syncthreads();
        int kind[kTmmChunk / 256], place[kTmmChunk / 256];
#pragma unroll
        for (int u = 0; u < kTmmChunk / 256; ++u) {
            const int i = u * 256 + tid;
            kind[u] = -1;
            place[u] = 0;
            if (i < n) {
                const int li = lidx[c0 + i];
                const double th = theta[c0 + i];
                double kappa;
                bool fp64;
                kind[u] = valid(li, th) ? kind_of(lam_tab + (int64_t)li * rows.stride(), th, &kappa, &fp64) : kTmmKinds - 1;
            }
            for (int k = 0; k < kTmmKinds; ++k) {
                const unsigned long long b = __ballot(kind[u] == k);
                if (b == 0ull) continue;
                int at = 0;
                if (lane == 0) at = atomicAdd(&s_n[k], __popcll(b));
                at = __builtin_amdgcn_readfirstlane(at);
                if (kind[u] == k) place[u] = at + __popcll(b & ((1ull << lane) - 1ull));
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTmmChunk / 256; ++u) {
            int first = 0;
            for (int k = 0; k < kTmmKinds; ++k) first += k < kind[u] ? s_n[k] : 0;
            if (kind[u] >= 0) s_list[first + place[u]] = (uint16_t)(u * 256 + tid);
        }
        __syncthreads();
        for (;;) {
            int b = 0;
            if (lane == 0) b = atomicAdd(&s_next, 64);
            b = __builtin_amdgcn_readfirstlane(b);
            if (b >= n) break;
            const int i = b + lane;
            if (i < n) solve(c0 + s_list[i]);
        }
    }
}

// ======================================================== loss (FP64)
// eta[d][l][f] = sum_b I  (one block per point, fixed-shape tree reduction)
__global__ void __launch_bounds__(256) k_loss_eta(const double* __restrict__ I, int B, double* __restrict__ eta)
{
    __shared__ double red[256];
    const double* row = I + (int64_t)blockIdx.x * B;
    double acc = 0.0;
    for (int b = threadIdx.x; b < B; b += blockDim.x) acc += row[b];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) eta[blockIdx.x] = red[0];
}

// E[d][b] = mean over (l, f) of I.  One block of 1024 threads per (design,
// 64 bins): wave w sums the rows k = w, w + 16, ... in order, then lane b's
// 16 wave sums are added in wave order (a fixed order).
__global__ void __launch_bounds__(1024) k_loss_eyeb(const double* __restrict__ I, int D, int nlf, int B,
                                                    double* __restrict__ E)
{
    __shared__ double part[16][64];
    const int tiles = (B + 63) / 64;
    const int d = blockIdx.x / tiles, b = (blockIdx.x % tiles) * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
    double acc = 0.0;
    if (b < B) {
        const double* p = I + (int64_t)d * nlf * B + b;
        for (int k = w; k < nlf; k += 16) acc += p[(int64_t)k * B] / (double)nlf;
    }
    part[w][threadIdx.x & 63] = acc;
    __syncthreads();
    if (w == 0 && b < B) {
        double e = 0.0;
        for (int k = 0; k < 16; ++k) e += part[k][threadIdx.x];
        E[(int64_t)d * B + b] = e;
    }
}

// Sum over the block of each thread's v: a fixed tree over the 256 threads.
__device__ inline double block_sum256(double v, double* red)
{
    __syncthreads();
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

// Per design (one block of 256 threads each): moments and the coefficients
// of dL/dI.  coef[d] = { L_d, a_e, a_f, m_e, m_f, ebar, ibar, bright };
// phi[d][f] written too.  bright weighs the throughput's mean in the
// brightness term: 1, or 1 / B for pupil images (kind 2), whose brightness is
// the mean over pupils rather than the sum over bins.  Sums are strided per thread, then a fixed tree.
__global__ void __launch_bounds__(256) k_loss_scalar(const double* __restrict__ eta, const double* __restrict__ E,
                                                     int nl, int F, int B, int kind, double w_f, double w_e,
                                                     double* __restrict__ phi, double* __restrict__ coef)
{
    __shared__ double red[256];
    const int d = blockIdx.x, t = threadIdx.x;
    const double* et = eta + (int64_t)d * nl * F;
    double* ph = phi + (int64_t)d * F;
    const double npts = (double)nl * (double)F;
    double part = 0.0;
    for (int f = t; f < F; f += 256) {
        double a = 0.0;
        for (int l = 0; l < nl; ++l) {
            const double v = et[(int64_t)l * F + f];
            a += v / (double)nl;
            part += v / npts;
        }
        ph[f] = a;
    }
    const double ibar = block_sum256(part, red);
    const double* Ed = E + (int64_t)d * B;
    part = 0.0;
    for (int b = t; b < B; b += 256) part += Ed[b] / (double)B;
    const double ebar = block_sum256(part, red);
    part = 0.0;
    for (int b = t; b < B; b += 256) part += (Ed[b] - ebar) * (Ed[b] - ebar) / (double)B;
    const double ve = block_sum256(part, red);
    part = 0.0;
    for (int f = t; f < F; f += 256) part += (ph[f] - ibar) * (ph[f] - ibar) / (double)F;   // this thread's own ph[f]
    const double vf = block_sum256(part, red);
    if (t != 0) return;
    double L, ae, af, me, mf;
    const double bright = kind == 2 ? 1.0 / (double)B : 1.0;
    if (kind == 0) {
        L = -ibar + w_e * ve + w_f * vf;
        ae = w_e; af = w_f; me = 0.0; mf = 0.0;
    } else {
        double se = sqrt(ve), sf = sqrt(vf);
        L = -ibar * bright + w_f * (sf / ibar) + w_e * (se / ebar);
        ae = se > 0.0 ? w_e / (2.0 * se * ebar) : 0.0;
        af = sf > 0.0 ? w_f / (2.0 * sf * ibar) : 0.0;
        me = -w_e * se / (ebar * ebar);
        mf = -w_f * sf / (ibar * ibar);
    }
    double* c = coef + (int64_t)d * 8;
    c[0] = L; c[1] = ae; c[2] = af; c[3] = me; c[4] = mf; c[5] = ebar; c[6] = ibar; c[7] = bright;
}

// Total loss: the designs' L_d in design order.
__global__ void k_loss_total(const double* __restrict__ coef, int D, double* __restrict__ loss)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    double total = 0.0;
    for (int d = 0; d < D; ++d) total += coef[(int64_t)d * 8];
    loss[0] = total;
}

__global__ void k_loss_grad(const double* __restrict__ E, const double* __restrict__ phi,
                            const double* __restrict__ coef, int D, int nl, int F, int B,
                            double* __restrict__ G)
{
    int64_t n = (int64_t)D * nl * F * B;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        int b = (int)(i % B);
        int64_t r = i / B;
        int f = (int)(r % F);
        r /= F;
        r /= nl;
        int d = (int)r;
        const double* c = coef + (int64_t)d * 8;
        double npts = (double)nl * (double)F;
        double ce = 2.0 * (E[(int64_t)d * B + b] - c[5]) / ((double)B * npts);
        double cf = 2.0 * (phi[(int64_t)d * F + f] - c[6]) / ((double)F * (double)nl);
        G[i] = -c[7] / npts + c[1] * ce + c[2] * cf + c[3] / ((double)B * npts) + c[4] / npts;
    }
}

// ======================================================== launch wrappers
static inline int grid_for(int64_t n, int bs, int cap = 65536)
{
    int64_t g = (n + bs - 1) / bs;
    if (g < 1) g = 1;
    return (int)(g < cap ? g : cap);
}

hipError_t launch_fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}
hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}
hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// LDS of the scene's layout by which a scene is accepted (64 KB) and a
// workgroup size picked: point data, stacks, slot tables, bins and, memoized,
// 3 KB of keys per wave.  The launch takes the direction and key tables and
// the statistics' columns on top (at most 25 KB): a workgroup may use 160 KB
// on gfx950, and two of the usual scenes' fit a CU.
size_t fwd_scene_bytes(const SceneDev& sc, int wg, bool lds_bins)
{
    return (size_t)smem_layout(sc.M, sc.Lmax, sc.n_slots, wg, sc.bins_x * sc.bins_y, lds_bins, 0,
                               sc.memo ? LaneSlots3::kPer : LaneSlots3x::kPer, true).total
           + (sc.memo ? (size_t)(wg / 64) * (24 * kFwdMemoKeys) : 0);
}
size_t fwd_smem_bytes(const SceneDev& sc, int wg, bool lds_bins)
{
    return (size_t)fwd_layout(sc, wg, lds_bins, sc.dirs != nullptr, sc.table != nullptr, sc.memo != 0).total;
}
size_t bwd_smem_bytes(const SceneDev& sc, int wg)
{
    return (size_t)smem_layout(sc.M, sc.Lmax, sc.n_slots, wg, sc.bins_x * sc.bins_y, false, (wg + 63) / 64).total;
}

template <class K>
static int blocks_per_cu(K kernel, int wg, size_t smem)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, wg, smem) != hipSuccess || n < 1) n = 1;
    return n;
}

// The forward kernel of a kind: memoized solves need the direction table, and
// the table forward solves nothing, so its precision does not matter.
using FwdKernel = void (*)(SceneDev, uint64_t*, uint32_t*, unsigned long long*, gwg_ray_record*, int64_t, int, double*,
                           AdjStore, double*);
template <int MODE, bool ADJ>
static FwdKernel fwd_kernel_mode(bool tab, bool memo, bool dirs)
{
    if (tab) return dirs ? k_trace_fwd<GWG_FP64, ADJ, true, false, true> : k_trace_fwd<GWG_FP64, ADJ, true, false, false>;
    if (memo) return k_trace_fwd<MODE, ADJ, false, true, true>;
    return dirs ? k_trace_fwd<MODE, ADJ, false, false, true> : k_trace_fwd<MODE, ADJ, false, false, false>;
}
static FwdKernel fwd_kernel(int precision, bool adj, bool tab, bool memo, bool dirs)
{
    switch (precision) {
    case GWG_FP64: return adj ? fwd_kernel_mode<GWG_FP64, true>(tab, memo, dirs) : fwd_kernel_mode<GWG_FP64, false>(tab, memo, dirs);
    case GWG_FP32_MIXED:
        return adj ? fwd_kernel_mode<GWG_FP32_MIXED, true>(tab, memo, dirs) : fwd_kernel_mode<GWG_FP32_MIXED, false>(tab, memo, dirs);
    default: return adj ? fwd_kernel_mode<GWG_FP32, true>(tab, memo, dirs) : fwd_kernel_mode<GWG_FP32, false>(tab, memo, dirs);
    }
}
int fwd_blocks_per_cu(const SceneDev& sc, bool adj, int wg, size_t smem)
{
    return blocks_per_cu(fwd_kernel(sc.precision, adj, sc.table != nullptr, sc.memo != 0, sc.dirs != nullptr), wg, smem);
}

template <bool TAB, int KIND>
static int bwd_blocks_per_cu(int precision, int wg, size_t smem)
{
    if (precision == GWG_FP64) return blocks_per_cu(k_trace_bwd<GWG_FP64, TAB, KIND>, wg, smem);
    if (precision == GWG_FP32_MIXED) return blocks_per_cu(k_trace_bwd<GWG_FP32_MIXED, TAB, KIND>, wg, smem);
    return blocks_per_cu(k_trace_bwd<GWG_FP32, TAB, KIND>, wg, smem);
}

int trace_blocks_per_cu(int kind, int precision, int wg, size_t smem)
{
    switch (kind) {
    case KIND_BWD_REGEN: return bwd_blocks_per_cu<false, ADJ_ABSORBING>(precision, wg, smem);
    case KIND_BWD_REGEN_LOSSLESS: return bwd_blocks_per_cu<false, ADJ_LOSSLESS>(precision, wg, smem);
    case KIND_BWD_REGEN_TAB: return bwd_blocks_per_cu<true, ADJ_LOSSLESS>(precision, wg, smem);
    case KIND_ADJ_SORTED:
        return blocks_per_cu(k_adj_sorted<true>, 64, smem);
    case KIND_ADJ_SORTED_ABS:
        return blocks_per_cu(k_adj_sorted<false>, 64, smem);
    case KIND_ADJ_MEMO:
        return blocks_per_cu(k_adj_memo<false>, 64 * kMemoWaves, smem);
    case KIND_ADJ_MEMO_LOSSLESS:
        return blocks_per_cu(k_adj_memo<true>, 64 * kMemoWaves, smem);
    case KIND_KEY_ADJ:
        return blocks_per_cu(k_key_adj<false>, 64, smem);
    case KIND_KEY_ADJ_LOSSLESS:
        return blocks_per_cu(k_key_adj<true>, 64, smem);
    case KIND_TABLE_ACCUM:
        return blocks_per_cu(k_table_accum, 64 * kMemoWaves, smem);
    case KIND_OMEGA:
        return std::min(blocks_per_cu(k_omega_grad<true>, wg, smem), blocks_per_cu(k_omega_grad<false>, wg, smem));
    default:
        return blocks_per_cu(k_adj_entries, wg, smem);
    }
}

hipError_t launch_trace_fwd(const SceneDev& sc, int wg, int grid_blocks, bool lds_bins, uint64_t* q, uint32_t* c,
                            unsigned long long* stats, gwg_ray_record* rec, int64_t rec_stride, double* scratch,
                            const AdjStore* adj, double* tape, hipStream_t s)
{
    const size_t sm = fwd_smem_bytes(sc, wg, lds_bins);
    FwdKernel k = fwd_kernel(sc.precision, adj != nullptr, sc.table != nullptr, sc.memo != 0, sc.dirs != nullptr);
    hipLaunchKernelGGL(k, dim3((unsigned)grid_blocks), dim3(wg), sm, s, sc, q, c, stats, rec, rec_stride, (int)lds_bins,
                       scratch, adj ? *adj : AdjStore{}, adj ? tape : nullptr);
    return hipGetLastError();
}

template <bool TAB, int KIND>
static void launch_bwd_mode(const SceneDev& sc, dim3 grid, dim3 block, size_t sm, const double* dLdI, double* partial,
                            double* scratch, int64_t sample_stride, const int32_t* regen, unsigned long long* stats,
                            hipStream_t s)
{
    switch (sc.precision) {
    case GWG_FP64:
        hipLaunchKernelGGL((k_trace_bwd<GWG_FP64, TAB, KIND>), grid, block, sm, s, sc, dLdI, partial, scratch, sample_stride,
                           regen, stats);
        break;
    case GWG_FP32_MIXED:
        hipLaunchKernelGGL((k_trace_bwd<GWG_FP32_MIXED, TAB, KIND>), grid, block, sm, s, sc, dLdI, partial, scratch,
                           sample_stride, regen, stats);
        break;
    default:
        hipLaunchKernelGGL((k_trace_bwd<GWG_FP32, TAB, KIND>), grid, block, sm, s, sc, dLdI, partial, scratch, sample_stride,
                           regen, stats);
        break;
    }
}

hipError_t launch_trace_bwd(const SceneDev& sc, int wg, int grid_blocks, const double* dLdI, unsigned long long* stats,
                            double* partial, double* scratch, int64_t sample_stride, const int32_t* regen,
                            hipStream_t s)
{
    size_t sm = bwd_smem_bytes(sc, wg);
    dim3 grid((unsigned)grid_blocks), block(wg);
    if (sc.table)                                            // no thin-film adjoints in it
        launch_bwd_mode<true, ADJ_LOSSLESS>(sc, grid, block, sm, dLdI, partial, scratch, sample_stride, regen, stats, s);
    else if (sc.slot_complex == 0u)
        launch_bwd_mode<false, ADJ_LOSSLESS>(sc, grid, block, sm, dLdI, partial, scratch, sample_stride, regen, stats, s);
    else
        launch_bwd_mode<false, ADJ_ABSORBING>(sc, grid, block, sm, dLdI, partial, scratch, sample_stride, regen, stats, s);
    return hipGetLastError();
}

hipError_t launch_adj_entries(const SceneDev& sc, int wg, int grid_blocks, const double* dLdI,
                              unsigned long long* stats, double* partial, const AdjStore& st, double* scratch,
                              hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_entries, dim3((unsigned)grid_blocks), dim3(wg), bwd_smem_bytes(sc, wg), s, sc, dLdI, partial, st,
                       scratch, stats);
    return hipGetLastError();
}

hipError_t launch_adj_sorted(const SceneDev& sc, int grid_blocks, const double* dLdI, unsigned long long* stats,
                             double* partial, const AdjStore& st, uint32_t* order, int32_t* ints, double* scratch,
                             hipStream_t s)
{
    SortDev so;
    sort_shape(sc, &so);
    so.order = order;
    so.start = ints;
    hipLaunchKernelGGL(k_entry_sort, dim3((unsigned)so.groups), dim3(64 * kSortWaves), 0, s, sc, dLdI, st, so);
    hipLaunchKernelGGL(sc.slot_complex == 0u ? k_adj_sorted<true> : k_adj_sorted<false>, dim3((unsigned)grid_blocks), dim3(64),
                       sorted_smem_bytes(sc), s, sc, dLdI, partial, st, so, scratch, stats);
    return hipGetLastError();
}

hipError_t launch_adj_memo(const SceneDev& sc, int grid_blocks, const double* dLdI, unsigned long long* stats,
                           double* partial, const AdjStore& st, double* scratch, hipStream_t s)
{
    const size_t sm = memo_smem_bytes(sc);
    if (sc.slot_complex == 0u)
        hipLaunchKernelGGL(k_adj_memo<true>, dim3((unsigned)grid_blocks), dim3(64 * kMemoWaves), sm, s, sc, dLdI, partial, st,
                           scratch, stats);
    else
        hipLaunchKernelGGL(k_adj_memo<false>, dim3((unsigned)grid_blocks), dim3(64 * kMemoWaves), sm, s, sc, dLdI, partial, st,
                           scratch, stats);
    return hipGetLastError();
}

hipError_t launch_table_build(const SceneDev& sc, double* tab, int n_cu, unsigned long long* stats, hipStream_t s)
{
    const int wg = 256;
    const int64_t dls = (int64_t)sc.D * sc.n_lsel;
    const int64_t per = (int64_t)sc.M * 2 * sc.table_n;
    // enough workgroups to fill the device twice, each with at least one wave of entries
    int64_t chunks = std::max<int64_t>(1, (2 * (int64_t)n_cu + dls - 1) / dls);
    chunks = std::min<int64_t>(chunks, (per + wg - 1) / wg);
    const size_t sm = (size_t)smem_layout(sc.M, sc.Lmax, sc.n_slots, wg, sc.bins_x * sc.bins_y, false, 0,
                                          LaneSlots3::kPer, true).total;
    const dim3 grid((unsigned)(dls * chunks)), block(wg);
    switch (sc.precision) {
    case GWG_FP64:
        hipLaunchKernelGGL(k_table_build<GWG_FP64>, grid, block, sm, s, sc, tab, (int)chunks, stats);
        break;
    case GWG_FP32_MIXED:
        hipLaunchKernelGGL(k_table_build<GWG_FP32_MIXED>, grid, block, sm, s, sc, tab, (int)chunks, stats);
        break;
    default:
        hipLaunchKernelGGL(k_table_build<GWG_FP32>, grid, block, sm, s, sc, tab, (int)chunks, stats);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_absmax(const double* x, int64_t n, unsigned long long* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_absmax, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, x, n, out);
    return hipGetLastError();
}

hipError_t launch_table_accum(const SceneDev& sc, int grid_blocks, const double* dLdI, const AdjStore& st, hipStream_t s)
{
    hipLaunchKernelGGL(k_table_accum, dim3((unsigned)grid_blocks), dim3(64 * kMemoWaves), table_accum_smem_bytes(), s, sc,
                       dLdI, st);
    return hipGetLastError();
}

hipError_t launch_key_adj(const SceneDev& sc, int grid_blocks, const double* dLdI, unsigned long long* stats,
                          double* partial, const AdjStore& st, double* sum, double* scratch, hipStream_t s)
{
    unsigned long long* seen = (unsigned long long*)(sum + sc.n_items * (int64_t)(kKeyIndex * 4));
    hipLaunchKernelGGL(k_key_sums, dim3((unsigned)std::min<int64_t>(sc.n_items, 1 << 20)), dim3(64 * kMemoWaves), 0, s, sc,
                       dLdI, st, sum, seen);
    const size_t sm = key_adj_smem_bytes(sc);
    if (sc.slot_complex == 0u)
        hipLaunchKernelGGL(k_key_adj<true>, dim3((unsigned)grid_blocks), dim3(64), sm, s, sc, st, (const double*)sum,
                           (const unsigned long long*)seen, partial, scratch, stats);
    else
        hipLaunchKernelGGL(k_key_adj<false>, dim3((unsigned)grid_blocks), dim3(64), sm, s, sc, st, (const double*)sum,
                           (const unsigned long long*)seen, partial, scratch, stats);
    return hipGetLastError();
}

hipError_t launch_table_keys(const SceneDev& sc, const double* dLdI, const AdjStore& st, hipStream_t s)
{
    hipLaunchKernelGGL(k_table_keys, dim3((unsigned)std::min<int64_t>(sc.n_items, 1 << 20)), dim3(64 * kMemoWaves), 0, s, sc,
                       dLdI, st);
    return hipGetLastError();
}
int64_t table_acc_words(const SceneDev& sc) { return (int64_t)sc.D * sc.n_lsel * sc.M * 4 * sc.table_n * 4; }

hipError_t launch_table_adj(const SceneDev& sc, int grid_blocks, double* partial, double* scratch, unsigned long long* stats,
                            hipStream_t s)
{
    const dim3 grid((unsigned)grid_blocks), block(128);
    const size_t sm = table_adj_smem_bytes(sc);
    if (sc.slot_complex == 0u)
        hipLaunchKernelGGL(k_table_adj<true>, grid, block, sm, s, sc, partial, scratch, stats);
    else
        hipLaunchKernelGGL(k_table_adj<false>, grid, block, sm, s, sc, partial, scratch, stats);
    return hipGetLastError();
}

hipError_t launch_table_reduce(const double* partial, const SceneDev& sc, double* grad, hipStream_t s)
{
    const int64_t n = (int64_t)sc.D * sc.M * sc.Lmax;
    hipLaunchKernelGGL(k_table_reduce, dim3(grid_for(n, 256, 1 << 30)), dim3(256), 0, s, partial, sc.D, sc.n_lsel, sc.M,
                       sc.Lmax, sc.nlay, grad);
    return hipGetLastError();
}

hipError_t launch_dir_states(const SceneDev& sc, double* dirs, int32_t* dir_n, hipStream_t s)
{
    hipLaunchKernelGGL(k_dir_states, dim3((unsigned)(sc.n_lsel * sc.F)), dim3(64), 0, s, sc, dirs, dir_n);
    return hipGetLastError();
}
int64_t dir_table_doubles(const SceneDev& sc) { return (int64_t)sc.n_lsel * sc.F * kDirMax * kDirWords; }

hipError_t launch_omega_grad(const SceneDev& sc, int grid_blocks, int wg, const double* W, const uint32_t* counts,
                             double* partial, double* grad, hipStream_t s)
{
    if (sc.dirs)
        hipLaunchKernelGGL(k_omega_grad<true>, dim3((unsigned)grid_blocks), dim3(wg), omega_smem_bytes(sc, wg), s, sc, W,
                           counts, partial);
    else
        hipLaunchKernelGGL(k_omega_grad<false>, dim3((unsigned)grid_blocks), dim3(wg), omega_smem_bytes(sc, wg), s, sc, W,
                           counts, partial);
    hipLaunchKernelGGL(k_omega_reduce, dim3((unsigned)sc.M), dim3(256), 0, s, (const double*)partial, sc.n_items, sc.M, grad);
    return hipGetLastError();
}

hipError_t launch_grad_reduce(const double* partial, int64_t rows_per_design, int ML, int D, const double* regen,
                              int64_t items_per_design, const int32_t* ovf, const int32_t* left, double* tmp,
                              double* grad, const int32_t* nlay, int M, int Lmax, hipStream_t s)
{
    int64_t n = (int64_t)D * ML;
    hipLaunchKernelGGL(k_grad_ranges, dim3((unsigned)((ML + 255) / 256), kGradRanges, (unsigned)D), dim3(256), 0, s,
                       partial, rows_per_design, ML, regen, items_per_design, ovf, left, tmp);
    hipLaunchKernelGGL(k_grad_reduce, dim3(grid_for(n, 256, 1 << 30)), dim3(256), 0, s, (const double*)tmp, ML, D, grad);
    hipLaunchKernelGGL(k_mask_padding, dim3(grid_for(n, 256, 1 << 30)), dim3(256), 0, s, grad, nlay, D, M, Lmax);
    return hipGetLastError();
}

hipError_t launch_irradiance(const uint64_t* q, int64_t n, double scale, double* irr, hipStream_t s)
{
    hipLaunchKernelGGL(k_irradiance, dim3(grid_for(n, 256)), dim3(256), 0, s, q, n, scale, irr);
    return hipGetLastError();
}

size_t tmm_smem_bytes(int L, int n_slots, int wg)
{
    return (size_t)(sizeof(LayerRec) * rec_stride(L) + 8 * n_slots * LaneSlots5::kPer * ((wg + 63) / 64 * 64));
}

template <int MODE>
static hipError_t launch_tmm_mode(const double* thk, const uint8_t* slot, int L, const double* lam_tab, int n_lambda,
                                  const TmmRows& rows, const int32_t* lidx, const double* theta, int64_t nq, double* out,
                                  int chunk, const TmmTab* tab, dim3 grid, size_t sm, hipStream_t s)
{
    const dim3 block(256);
    auto launch = [&](auto val, auto sort, const auto& t) {
        hipLaunchKernelGGL((k_tmm_rt<MODE, decltype(val)::value, decltype(sort)::value>), grid, block, sm, s, thk, slot, L, lam_tab,
                           n_lambda, rows, lidx, theta, nq, out, chunk, t);
    };
    if constexpr (MODE != GWG_FP32) {                            // tmm_sorted
        if (chunk) {
            if (tab) launch(std::true_type{}, std::true_type{}, *tab);
            else launch(std::false_type{}, std::true_type{}, TmmNoTab{});
            return hipGetLastError();
        }
    }
    if (tab) launch(std::true_type{}, std::false_type{}, *tab);
    else launch(std::false_type{}, std::false_type{}, TmmNoTab{});
    return hipGetLastError();
}

// Whether queries are solved by kind.  Mixed precision always: in order, one
// query near the critical angle makes its wave run both solves (uniform
// angles, in order and by kind: 2000 queries of 200 layers 143 and 96 us,
// 100000 of 400 308 and 239 us, of 2000 1500 and 1156 us; where a fifth of the
// queries are near-critical, 100000 of 200 layers 111 and 114 us, 200000 of 8,
// 40 and 200 layers 33, 64 and 219 us and 26, 42 and 118 us).  Double precision
// on lossless stacks of more than a few layers (200000 queries of 8, 40 and
// 200: 24.0, 43.8 and 134 us in order, 25.1, 41.4 and 118 by kind), unless the
// waves all run at once, two workgroups a CU: such a launch is as long as its
// longest wave, and sorting adds to it (100000 of 200 layers 73 us in order
// and 77 by kind).  Silver's complex path hides the hyperbolic case (300000
// queries of 201 layers: 225 and 234 us), and single precision hardly pays for
// it (115 and 129 us).
static bool tmm_sorted(int precision, int L, uint32_t cplx, int64_t nq, int n_cu)
{
    if (precision == GWG_FP32_MIXED) return true;
    return precision == GWG_FP64 && cplx == 0u && L >= 32 && nq > 2 * 256 * (int64_t)n_cu;
}

hipError_t launch_tmm_rt(int precision, const double* thk, const uint8_t* slot, int L,
                         const double* lam_tab, int n_lambda, const TmmRows& rows,
                         const int32_t* lidx, const double* theta, int64_t nq, double* out, int n_cu,
                         const double* host_tab, const uint8_t* host_slot, hipStream_t s)
{
    const int wg = 256;
    size_t sm = tmm_smem_bytes(L, rows.n_slots, wg);
    int chunk = 0;
    if (tmm_sorted(precision, L, rows.cplx, nq, n_cu)) {
        // as many queries a workgroup as fill the GPU once (the longer its
        // list, the fewer its mixed batches) and at least one a lane, if
        // their list fits in LDS
        const int64_t want = std::max<int64_t>(wg, (nq + 2 * n_cu - 1) / (2 * n_cu));
        chunk = (int)std::min<int64_t>(kTmmChunk, (want + 63) / 64 * 64);
        if (sm + sizeof(uint16_t) * chunk + 64 > 65536) chunk = 0;
        sm += sizeof(uint16_t) * chunk;
    }
    const dim3 grid(grid_for(nq, chunk ? chunk : wg, 8192));
    TmmTab tab;
    if (host_tab) {
        const size_t nb = sizeof(double) * rows.stride() * (size_t)n_lambda;
        std::memcpy(tab.b, host_tab, nb);
        std::memcpy(tab.b + nb, host_slot, (size_t)L);
    }
    const auto launch = precision == GWG_FP64 ? launch_tmm_mode<GWG_FP64>
                        : precision == GWG_FP32_MIXED ? launch_tmm_mode<GWG_FP32_MIXED> : launch_tmm_mode<GWG_FP32>;
    return launch(thk, slot, L, lam_tab, n_lambda, rows, lidx, theta, nq, out, chunk, host_tab ? &tab : nullptr, grid, sm, s);
}

hipError_t launch_loss(const double* I, int D, int nl, int F, int B, int kind, double w_f, double w_e,
                       double* work, double* loss, double* G, hipStream_t s)
{
    // work: eta [D nl F] | E [D B] | phi [D F] | coef [D 8]
    double* eta = work;
    double* E = eta + (int64_t)D * nl * F;
    double* phi = E + (int64_t)D * B;
    double* coef = phi + (int64_t)D * F;
    hipLaunchKernelGGL(k_loss_eta, dim3((unsigned)((int64_t)D * nl * F)), dim3(256), 0, s, I, B, eta);
    hipLaunchKernelGGL(k_loss_eyeb, dim3((unsigned)((int64_t)D * ((B + 63) / 64))), dim3(1024), 0, s, I, D, nl * F, B, E);
    hipLaunchKernelGGL(k_loss_scalar, dim3((unsigned)D), dim3(256), 0, s, eta, E, nl, F, B, kind, w_f, w_e, phi, coef);
    hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(64), 0, s, (const double*)coef, D, loss);
    if (G) hipLaunchKernelGGL(k_loss_grad, dim3(grid_for((int64_t)D * nl * F * B, 256)), dim3(256), 0, s, E, phi, coef, D, nl, F, B, G);
    return hipGetLastError();
}

// ------------------------------------------ allocation-free loss scratch
// Work buffer of gwg_loss_noalloc: a file-scope device array (each GPU the
// library runs on holds its own copy until the process ends).  On the host
// the array's name is not a device address: its address on each device is
// looked up once, with that device current, by hipGetSymbolAddress, and only
// that pointer is ever passed to kernels.
static __device__ __align__(256) double scratch[kLossScratchDoubles];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kScratchDevices] = {};
}  // namespace

hipError_t loss_scratch_setup(int device)
{
    if (device < 0 || device >= kScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = (double*)p;
    return hipSuccess;
}

double* loss_scratch(int device)
{
    if (device < 0 || device >= kScratchDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_ptr[device];
}

}  // namespace gwg
