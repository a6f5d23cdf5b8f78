// sd_host.h -- host-side helpers shared by the C-ABI translation units
// (argument checks, workspace, launch planning).  Not part of the C ABI.
#pragma once

#include "sd.h"
#include "sd_internal.h"

namespace sd {

// Largest particle count the kernels index with 32-bit integers.
constexpr int64_t MAX_N = (int64_t(1) << 30);

// Library-owned workspace slots (one buffer each per device).
enum {
    WS_PARTIAL = 0,   // split partials of the pair kernels
    WS_STAGE,         // FP32 / FP64 staged positions of the time loop
    WS_ADJ_PARTIAL,   // split partials of the adjoint kernel
    WS_ADJ_PACK,      // packed cotangent / force staging
    WS_ADJ_TRAJ,      // recomputed trajectory of one checkpoint segment
    WS_ADJ_LAM,       // adjoint state
    WS_ADJ_CKPT,      // checkpoints when the caller passes none
    WS_TUNE,          // autotuner scratch
    WS_LUB,           // lubrication cell list
    WS_LUB_F,         // lubrication-corrected forces of a step
    WS_QPOS,          // fixed-point positions of a product in a periodic box
    WS_CLUSTER,       // run records of the precision study
    WS_MEAN,          // partial sums of sd_mean_vector
    WS_COUNT
};

sd_status fail(sd_status st, const char* fmt, ...);
sd_status check_lub(const sd_lub* lub);
sd_status check_params(const sd_params* p);
// cubic box side of validated params (0 = free space)
inline double box_side(const sd_params* p) { return p->box[0]; }
// SD_EUNSUPPORTED for a periodic box (entry points without box support)
sd_status check_free_space(const sd_params* p, const char* what);
sd_status check_n(int64_t n);
sd_status check_precision(int32_t prec);
sd_status check_ptr(const void* ptr, size_t align, const char* name);
size_t vec4_align(int32_t prec);
int device_cus();
sd_status ws_get(int which, size_t bytes, void** out);

sd_kernel_config default_config(int32_t prec, int64_t n);
// Whether the j-side workspace of the pair-symmetric kernel (variant 2) for n
// particles in blocks of `block` stays within SYM_WORKSPACE_CAP bytes.
constexpr size_t SYM_WORKSPACE_CAP = (size_t)1 << 30;
// Smallest n for which the automatic configuration takes variant 2.
constexpr int64_t SYM_MIN_N = 16384;
bool sym_fits(int64_t n, int block);
// Automatic FP64 products of at least WAVE_F64_MIN_N particles take the
// wave-symmetric kernel (variant 3) while its workspace stays within the cap,
// with two particles per lane from WAVE_ILP2_MIN_N on (one per lane gives
// twice the waves of a small product; two share each hand-over and each read
// of j).  Microseconds per mobility_apply, one-sided kernel / one / two
// particles per lane: N = 1024 16.9 / 14.3 / 16.4, 2000 18.9 / 14.2 / -,
// 3001 27.6 / 18.2 / 20.0, 4000 34.5 / 25.6 / 24.5, 6000 72.6 / 46.0 / 39.7,
// 16384 301 / 246 / 200, 40000 1730 / - / 1107.
constexpr int64_t WAVE_F64_MIN_N = 1024;
constexpr int64_t WAVE_ILP2_MIN_N = 3500;
// Automatic FP32 products: wave-symmetric from WAVE_F32_MIN_N to where the
// block-symmetric kernel (fewer j-side partials, more pairs per tile) is as
// fast, two particles per lane (with SD_FP32_KAHAN in assembly) from
// WAVE_F32_ILP2_MIN_N on.  Microseconds per mobility_apply, before / one / two
// particles per lane: N = 1024 15.5 / 13.2 / -, 2000 17.0 / 13.1 / -, 3000 21.2
// / 14.8 / -, 4096 24.5 / 19.6 / 21.0, 6007 43.9 / 30.9 / 28.5, 8192 54.4 /
// 47.2 / 42.8, 12000 107.7 / - / 77.5; block-symmetric and wave at 16384 124.2
// and 126.8 (162.5 and 132.8 with one particle in ten overlapping), 24576 243
// and 301.  Plain sums (compiled loops in both): 16384 149 and 126, 24576 277
// and 286.
constexpr int64_t WAVE_F32_MIN_N = 1024;
constexpr int64_t WAVE_F32_ILP2_MIN_N = 5000;
constexpr int64_t WAVE_PLAIN_END_N = 20000;
// The configuration for n particles; *automatic (may be null) receives whether
// it is the automatic choice (nothing forced, no tuned shape for the size).
sd_kernel_config choose_config(int32_t prec, int64_t n, bool* automatic = nullptr);
// Tuned shape of n's size class (null: none, the automatic choice applies).
void set_tuned_config(int32_t prec, int64_t n, const sd_kernel_config* c);
sd_status check_config(int32_t prec, const sd_kernel_config& c);

PairConst pair_const(const sd_params* p);
PairLaunch plan_pair(int32_t prec, int64_t n);
// a wave-symmetric launch (variant 3) with ilp particles per lane
PairLaunch plan_wave(int64_t n, int ilp);
size_t partial_bytes(const PairLaunch& L, int64_t n);
// vel (may be null): for the pair-symmetric kernel the product is finished
// here (the fold merges into vel; *merged is set), else the caller merges.
sd_status run_pair(const sd_params* p, int64_t n, const void* pos, const void* frc,
                   const double* x64, int32_t prec, double* partial, const PairLaunch& L,
                   hipStream_t st, double* vel = nullptr, bool* merged = nullptr);

// One time step's end: split rows -> v, positions and history (mode as
// launch_merge_integrate_*), and the staged copy for the next pair kernel.
// Enqueue after run_pair (without vel).
sd_status finish_step(const sd_params* p, int64_t n, const void* frc, int32_t prec,
                      const double* partial, const PairLaunch& L, double* x, double* v_prev,
                      double* v_out, double dt, int mode, void* pos_next, hipStream_t st);

void batch_release_graphs();
void run_graphs_release();

}  // namespace sd
