// Launch wrappers of the HIP kernels (defined in gwg_kernels.hip), called by
// the host API only.
#pragma once
#include <hip/hip_runtime.h>
#include "gwg.h"
#include "gwg_internal.h"

namespace gwg {

hipError_t launch_fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s);
hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t s);

size_t fwd_scene_bytes(const SceneDev& sc, int wg, bool lds_bins);
size_t fwd_smem_bytes(const SceneDev& sc, int wg, bool lds_bins);
hipError_t launch_dir_states(const SceneDev& sc, double* dirs, int32_t* dir_n, hipStream_t s);
int64_t dir_table_doubles(const SceneDev& sc);
size_t bwd_smem_bytes(const SceneDev& sc, int wg);
size_t tmm_smem_bytes(int L, int n_slots, int wg);
int64_t bwd_scratch_doubles(const SceneDev& sc, int64_t grid_blocks, int wg);

// KIND_FWD and up: forward kernels, KIND_FWD + gradient + 2 table + 4 memoized + 8 direction table
enum { KIND_BWD_REGEN = 0, KIND_ADJ_ENTRIES = 1, KIND_ADJ_SORTED = 2, KIND_ADJ_MEMO = 3, KIND_ADJ_MEMO_LOSSLESS = 4,
       KIND_TABLE_ACCUM = 5, KIND_BWD_REGEN_TAB = 6, KIND_OMEGA = 7, KIND_FWD = 8,
       KIND_KEY_ADJ = 64, KIND_KEY_ADJ_LOSSLESS = 65, KIND_ADJ_SORTED_ABS = 66, KIND_BWD_REGEN_LOSSLESS = 67 };
int fwd_blocks_per_cu(const SceneDev& sc, bool adj, int wg, size_t smem);
int trace_blocks_per_cu(int kind, int precision, int wg, size_t smem);
int64_t fwd_scratch_doubles(const SceneDev& sc, int64_t grid_blocks, int wg);
int64_t adj_scratch_doubles(const SceneDev& sc, int64_t grid_blocks, int wg);
hipError_t launch_trace_fwd(const SceneDev& sc, int wg, int grid_blocks, bool lds_bins, uint64_t* q, uint32_t* c,
                            unsigned long long* stats, gwg_ray_record* rec, int64_t rec_stride, double* scratch,
                            const AdjStore* adj, double* tape, hipStream_t s);
hipError_t launch_trace_bwd(const SceneDev& sc, int wg, int grid_blocks, const double* dLdI, unsigned long long* stats,
                            double* partial, double* scratch, int64_t sample_stride, const int32_t* regen,
                            hipStream_t s);
hipError_t launch_adj_entries(const SceneDev& sc, int wg, int grid_blocks, const double* dLdI,
                              unsigned long long* stats, double* partial, const AdjStore& st, double* scratch,
                              hipStream_t s);
size_t memo_smem_bytes(const SceneDev& sc);
// the sorted adjoint's shape: partial rows a design, units of work, table words
int64_t sorted_rows(const SceneDev& sc);
int64_t sorted_ints(const SceneDev& sc);
size_t sorted_smem_bytes(const SceneDev& sc);
int64_t sorted_scratch_doubles(const SceneDev& sc, int64_t grid);
hipError_t launch_adj_sorted(const SceneDev& sc, int grid_blocks, const double* dLdI, unsigned long long* stats,
                             double* partial, const AdjStore& st, uint32_t* order, int32_t* ints, double* scratch,
                             hipStream_t s);
hipError_t launch_adj_memo(const SceneDev& sc, int grid_blocks, const double* dLdI, unsigned long long* stats,
                           double* partial, const AdjStore& st, double* scratch, hipStream_t s);
hipError_t launch_table_build(const SceneDev& sc, double* tab, int n_cu, unsigned long long* stats, hipStream_t s);
hipError_t launch_absmax(const double* x, int64_t n, unsigned long long* out, hipStream_t s);
size_t table_accum_smem_bytes();
hipError_t launch_table_accum(const SceneDev& sc, int grid_blocks, const double* dLdI, const AdjStore& st, hipStream_t s);
int64_t table_adj_rows(const SceneDev& sc);          // partial gradient rows (Lmax each) of the table adjoint
int64_t table_acc_words(const SceneDev& sc);         // its accumulators
size_t key_adj_smem_bytes(const SceneDev& sc);
int64_t key_adj_blocks(const SceneDev& sc);          // units of work of the keyed adjoint
int64_t key_sum_doubles(const SceneDev& sc);
size_t table_adj_smem_bytes(const SceneDev& sc);
hipError_t launch_key_adj(const SceneDev& sc, int grid_blocks, const double* dLdI, unsigned long long* stats,
                          double* partial, const AdjStore& st, double* sum, double* scratch, hipStream_t s);
hipError_t launch_table_keys(const SceneDev& sc, const double* dLdI, const AdjStore& st, hipStream_t s);
hipError_t launch_table_adj(const SceneDev& sc, int grid_blocks, double* partial, double* scratch, unsigned long long* stats,
                            hipStream_t s);
hipError_t launch_table_reduce(const double* partial, const SceneDev& sc, double* grad, hipStream_t s);
size_t omega_scene_bytes(const SceneDev& sc, int wg);
size_t omega_smem_bytes(const SceneDev& sc, int wg);
hipError_t launch_omega_grad(const SceneDev& sc, int grid_blocks, int wg, const double* W, const uint32_t* counts,
                             double* partial, double* grad, hipStream_t s);
hipError_t launch_grad_reduce(const double* partial, int64_t rows_per_design, int ML, int D, const double* regen,
                              int64_t items_per_design, const int32_t* ovf, const int32_t* left, double* tmp,
                              double* grad, const int32_t* nlay, int M, int Lmax, hipStream_t s);
int64_t grad_reduce_tmp_doubles(int ML, int D);
hipError_t launch_item_order(const int32_t* cnt, int waves, int64_t n_items, int64_t max_count, int32_t* order,
                             hipStream_t s);
hipError_t launch_irradiance(const uint64_t* q, int64_t n, double scale, double* irr, hipStream_t s);
// Wavelength rows of the thin-film queries, doubles: the free-space wavenumber,
// the incident index, the exit index (re, im), the slots' real indices, the
// imaginary ones of absorbing slots (bits of cplx), n_crit near-critical kappa
// intervals (lo, hi).
enum { TR_K0 = 0, TR_NG = 1, TR_NA = 2, TR_SLOT = 4 };
struct TmmRows {
    int32_t n_slots, n_crit;
    uint32_t cplx;
    __host__ __device__ int imag(int s) const { return TR_SLOT + n_slots + __builtin_popcount(cplx & ((1u << s) - 1u)); }
    __host__ __device__ int crit(int k) const { return TR_SLOT + n_slots + __builtin_popcount(cplx) + 2 * k; }
    __host__ __device__ int stride() const { return crit(n_crit); }
};
// Bytes of rows and slots that a thin-film launch carries (31 wavelengths of a
// 400-layer stack of four materials); with more (host_tab null) it reads them
// from device memory.
constexpr size_t kTmmTabBytes = 3584;
hipError_t launch_tmm_rt(int precision, const double* thk, const uint8_t* slot, int L,
                         const double* lam_tab, int n_lambda, const TmmRows& rows,
                         const int32_t* lidx, const double* theta, int64_t nq, double* out, int n_cu, const double* host_tab,
                         const uint8_t* host_slot, hipStream_t s);
hipError_t launch_loss(const double* I, int D, int nl, int F, int B, int kind, double w_f, double w_e,
                       double* work, double* loss, double* G, hipStream_t s);
// Doubles of work a loss of shape (D, nl, F, B) uses (launch_loss's work).
inline int64_t loss_work_doubles(int64_t D, int64_t nl, int64_t F, int64_t B)
{
    return D * nl * F + D * B + D * F + D * 8;
}
// Fixed-size device scratch of gwg_loss_noalloc (4 MiB per GPU).
constexpr int64_t kLossScratchDoubles = 1 << 19;
// Look up this device's scratch address (with `device` current); once per
// device, thread-safe.
hipError_t loss_scratch_setup(int device);
// The device address of `device`'s scratch, or null before its setup.
double* loss_scratch(int device);

}  // namespace gwg
