// Learned reflection probabilities: score-function gradient.  Included by
// gwg_kernels.hip inside namespace gwg.
//
// (Methods, learned reflection probabilities) Before the thicknesses are
// optimised, the mirrors' reflection probabilities omega are optimised with
// every coating idealised as a scalar reflectance equal to omega, tracing
// geometry only.  A sampled branch then carries weight one and a ray adds 1/N
// to the bin it reaches, so the scalar irradiance is the bin count over N.
// For J = sum over points and bins of W * I (W: per-bin weights, e.g. 1 for
// the throughput or dL/dI of Eq. 1 at the scalar irradiance), the path
// probability prod(omega or 1 - omega) gives the score-function gradient
//     dJ/domega_m = sum_points 1/N sum_rays (W_bin - beta) S_m,
//     S_m = sum over the ray's hits on mirror m of
//           (reflected ? 1/omega_m : -1/(1 - omega_m)),
// unbiased for any per-point constant beta because E[S_m] = 0; beta is the
// point's own J from the forward's counts.  omega_m is the probability the
// sampling uses, thr_m / 2^32.  A ray that leaves the eyebox has W = 0.
//
// Same paths as the last forward (same items, seeds and decisions).  Each
// lane sums its rays' contributions in LDS, a wave's lanes are added in a
// fixed butterfly and the waves in order, per item; the items' sums are added
// by a fixed tree per mirror: the gradient is deterministic.
//
// Bound by the geometry walks (instruction issue and LDS latency).  On the
// direction table, with one butterfly per item
// instead of one per 64 rays, and 256 threads per mirror summing the items
// instead of one: 6 mirrors, 3 x 441 points x 8192 rays, 2.63 -> 1.28 ms; the sum over
// the items 1.16 -> 0.01 ms.

struct ScoreHit {
    double* s;            // this lane's S_m at s[m * ls]
    int ls;
    const double* inc;    // [2 M]: 1/omega_m, -1/(1 - omega_m)
    __device__ void operator()(int, double, int) const {}
    __device__ void operator()(int, const double*, int) const {}
    __device__ void branch(int m, bool refl) const { s[m * ls] += inc[2 * m + (refl ? 0 : 1)]; }
};

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The general walk of one ray: its bin (-1: none), its score in LDS.
__device__ inline int score_walk(const SceneDev& sc, const PointLds& pl, int64_t id, const ScoreHit& score)
{
    Ray r;
    Outcome o;
    TapeRef none = { nullptr, nullptr, 0 };
    ray_birth(sc, pl, id, r);
    walk_ray<false, false>(sc, pl, r, o, score, NoCoef{}, none, nullptr);
    return o.cat == CAT_EYEBOX ? o.bin : -1;
}
// ... of a ray off the direction table, out of line (sc in LDS).
__device__ __attribute__((noinline)) int score_walk_off(const SceneDev& sc, const PointLds& pl, int64_t id,
                                                        const ScoreHit& score)
{
    return score_walk(sc, pl, id, score);
}

struct OmegaLayout { int off_pl, off_s, off_acc, off_inc, off_sum, off_red, off_sc, off_dir, total; };
__host__ __device__ inline OmegaLayout omega_layout(int M, int wg, bool dirs)
{
    OmegaLayout s;
    int o = 0;
    s.off_pl = o; o = align16(o + (int)sizeof(PointLds));
    s.off_s = o; o = align16(o + 8 * M * wg);
    s.off_acc = o; o = align16(o + 8 * M * wg);
    s.off_inc = o; o = align16(o + 16 * M);
    s.off_sum = o; o = align16(o + 8 * M * (wg / 64));
    s.off_red = o; o = align16(o + 8 * wg);
    s.off_sc = o; o = align16(o + (dirs ? (int)sizeof(SceneDev) : 0));
    s.off_dir = o; o = align16(o + (dirs ? kDirMax * kDirWords * 8 : 0));
    s.total = o;
    return s;
}

template <bool DIRS>
__global__ void __launch_bounds__(256, 4) k_omega_grad(SceneDev sc, const double* __restrict__ W,
                                                  const uint32_t* __restrict__ counts, double* __restrict__ partial)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int WG = blockDim.x, n_waves = WG / 64;
    const int B = sc.bins_x * sc.bins_y, M = sc.M;
    const OmegaLayout lay = omega_layout(M, WG, DIRS);
    PointLds* pl = (PointLds*)(smem + lay.off_pl);
    double* s_S = (double*)(smem + lay.off_s);                // [M][WG] the current ray's scores
    double* s_A = (double*)(smem + lay.off_acc);              // [M][WG] the lane's sums
    double* s_inc = (double*)(smem + lay.off_inc);            // [2 M]
    double* s_sum = (double*)(smem + lay.off_sum);            // [n_waves][M]
    double* s_red = (double*)(smem + lay.off_red);            // [WG] baseline reduction
    SceneDev* s_sc = (SceneDev*)(smem + lay.off_sc);
    const int tid = threadIdx.x, wave = tid / 64, lane = wave_lane();
    const ScoreHit score = { s_S + tid, WG, s_inc };
    const double invN = 1.0 / (double)sc.N;
    if (DIRS && tid == 0) *s_sc = sc;
    for (int m = 0; m < M; ++m) s_S[m * WG + tid] = 0.0;

    for (int64_t item = blockIdx.x; item < sc.n_items; item += gridDim.x) {
        int64_t point, i0, i1;
        int d, l, f;
        decode_item(sc, item, &point, &d, &l, &f, &i0, &i1);
        __syncthreads();
        stage_point(sc, d, l, f, pl, nullptr, nullptr);
        DirLds dt{};
        if constexpr (DIRS) dt = stage_dirs(sc, (int64_t)l * sc.F + f, (double*)(smem + lay.off_dir));
        const double* Wp = W + point * B;
        const uint32_t* cp = counts + point * B;
        // the point's J (baseline): strided partial sums, then a fixed tree
        double part = 0.0;
        for (int b = tid; b < B; b += WG) part += Wp[b] * (double)cp[b];
        s_red[tid] = part;
        for (int m = 0; m < M; ++m) s_A[m * WG + tid] = 0.0;
        __syncthreads();
        if (tid < 2 * M) {
            const int m = tid >> 1;
            const double p = (double)pl->thr[m] * (1.0 / 4294967296.0);
            s_inc[tid] = (tid & 1) ? -1.0 / (1.0 - p) : (p > 0.0 ? 1.0 / p : 0.0);
        }
        for (int w = WG / 2; w > 0; w >>= 1) {
            if (tid < w) s_red[tid] += s_red[tid + w];
            __syncthreads();
        }
        const double beta = s_red[0] * invN;
        const int64_t base = point * sc.N;
        for (int64_t i = i0 + tid; i < i1; i += WG) {
            int bin;
            if constexpr (DIRS) {
                DirFate o;
                dir_walk(sc, *pl, dt, base + i, score, o);
                bin = o.bin;
                if (o.off) {
                    for (int m = 0; m < M; ++m) s_S[m * WG + tid] = 0.0;
                    const ScoreHit sc2 = score;
                    bin = score_walk_off(*s_sc, *pl, base + i, sc2);
                }
            } else {
                bin = score_walk(sc, *pl, base + i, score);
            }
            const double fw = (bin >= 0 ? Wp[bin] : 0.0) - beta;
            for (int m = 0; m < M; ++m) {
                s_A[m * WG + tid] = fma(fw, s_S[m * WG + tid], s_A[m * WG + tid]);
                s_S[m * WG + tid] = 0.0;
            }
        }
        for (int m = 0; m < M; ++m) {
            const double c = wave_sum(s_A[m * WG + tid]);
            if (lane == 0) s_sum[wave * M + m] = c;
        }
        __syncthreads();
        if (tid < M) {
            double a = 0.0;
            for (int w = 0; w < n_waves; ++w) a += s_sum[w * M + tid];
            partial[item * M + tid] = a * invN;
        }
    }
}

// LDS by which a scene is accepted (64 KB) ...
size_t omega_scene_bytes(const SceneDev& sc, int wg)
{
    const int n_waves = wg / 64;
    return (size_t)smem_layout(sc.M, sc.Lmax, sc.n_slots, wg, sc.bins_x * sc.bins_y, false, 0).total +
           sizeof(double) * ((size_t)sc.M * wg + 2 * sc.M + (size_t)n_waves * sc.M + wg);
}
// ... and the launch's.
size_t omega_smem_bytes(const SceneDev& sc, int wg) { return (size_t)omega_layout(sc.M, wg, sc.dirs != nullptr).total; }

// grad[m] = sum over items of partial[item][m]: one block of 256 threads per
// mirror, strided sums in item order, then a fixed tree.
__global__ void __launch_bounds__(256) k_omega_reduce(const double* __restrict__ partial, int64_t n_items, int M,
                                                      double* __restrict__ grad)
{
    __shared__ double red[256];
    const int m = blockIdx.x, t = threadIdx.x;
    double a = 0.0;
    for (int64_t it = t; it < n_items; it += 256) a += partial[it * M + m];
    red[t] = a;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    if (t == 0) grad[m] = red[0];
}
