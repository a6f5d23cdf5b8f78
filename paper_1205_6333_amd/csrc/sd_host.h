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
    WS_STAGE,         // FP32 / FP64 staged positions of the time loop (two copies)
    WS_STEP_X,        // positions of every other step (variants 2 and 4)
    WS_ADJ_PARTIAL,   // split partials of the adjoint kernel
    WS_ADJ_PACK,      // packed cotangent
    WS_ADJ_REC,       // position records of one checkpoint segment
    WS_ADJ_TRAJ,      // recomputed trajectory of one checkpoint segment
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
// What the automatic choice runs beyond the configurations of sd.h, in FP64 and
// with compensated FP32 sums.
//
// Rows in one launch (variant 4) below ROW_*_END_N, two particles per
// work-group from ROW_ILP2_MIN_N on.  Above, each pair once: the wave-symmetric
// kernel (variant 3) for FP64 wherever its workspace fits, for FP32 up to where
// the block-symmetric kernel (variant 2: fewer j-side partials, more pairs per
// tile) is as fast.  Microseconds per Euler step, FP32, rows with two
// particles / wave-symmetric: N = 4500 19.9 / 22.2, 5324 25.3 / 26.9, 6007 30.5
// / 29.6; FP64: N = 3500 18.8 / 22.5, 4000 23.8 / 23.6, 5000 34.3 / 30.4.
// Microseconds per product, wave- / block-symmetric (compensated): N = 12000
// 77.5 / -, 16384 125.4 / 121.6 (with 0.4 near partners per particle 136.7 /
// 154.1), 24576 301 / 243.  FP64, wave-symmetric / one-sided: N = 6000 39.7 /
// 72.6, 16384 199 / 301, 40000 1107 / 1730.
constexpr int64_t ROW_F32_END_N = 5900;
constexpr int64_t ROW_F64_END_N = 4000;
constexpr int64_t ROW_ILP2_MIN_N = 1300;
// The configuration for n particles; *automatic (may be null) receives whether
// it is the automatic choice (nothing forced, no tuned shape for the size).
sd_kernel_config choose_config(int32_t prec, int64_t n, bool* automatic = nullptr);
// Tuned shape of n's size class (null: none, the automatic choice applies).
void set_tuned_config(int32_t prec, int64_t n, const sd_kernel_config* c);
sd_status check_config(int32_t prec, const sd_kernel_config& c);

PairConst pair_const(const sd_params* p);
// PLAN_CHOSEN: the forced, tuned or automatic choice; PLAN_GENERAL: the same
// without the automatic choice's own kernels; PLAN_AUTOMATIC: the automatic choice
// whatever is forced or tuned.
enum PlanMode { PLAN_CHOSEN, PLAN_GENERAL, PLAN_AUTOMATIC };
PairLaunch plan_pair(int32_t prec, int64_t n, PlanMode mode = PLAN_CHOSEN);
// The plan together with its workspace.  Where the wave-symmetric kernels'
// (up to 1 GiB, against some tens of MiB) cannot be had, the general kernel is
// planned.
sd_status plan_product(int32_t prec, int64_t n, PairLaunch* L, double** partial,
                       PlanMode mode = PLAN_CHOSEN);
// mobility_apply with checked arguments
sd_status run_product(const sd_params* p, int64_t n, const void* pos, const void* frc, double* vel,
                      int32_t prec, PlanMode mode, hipStream_t st);
// a wave-symmetric launch (variant 3) with ilp particles per lane
PairLaunch plan_wave(int64_t n, int ilp);
size_t partial_bytes(const PairLaunch& L, int64_t n);
// vel (may be null): for variants 2 to 4 the product is finished here (*merged
// is set), else the caller merges.
sd_status run_pair(const sd_params* p, int64_t n, const void* pos, const void* frc,
                   const double* x64, int32_t prec, double* partial, const PairLaunch& L,
                   hipStream_t st, double* vel = nullptr, bool* merged = nullptr);

// The last kernel of a step reads the positions of other particles than it writes.
inline bool step_apart(const PairLaunch& L) { return L.variant == 2 || L.variant == 4; }
// One time step from x_in to x_out (mode as launch_merge_integrate).  pos: the
// records of x_in; pos_next (may be null) receives those of x_out.  x_out may
// be x_in and pos_next may be pos unless step_apart(L).
sd_status run_step(const sd_params* p, int64_t n, const double* x_in, double* x_out,
                   const void* frc, double* v_prev, double* v_out, double dt, int mode,
                   int32_t prec, const void* pos, void* pos_next, double* partial,
                   const PairLaunch& L, hipStream_t st);

// A sequence of steps that starts and ends in the caller's x.  Variants 0, 1 and 3
// work in place; variants 2 and 4 (step_apart) alternate between x and a library
// copy, and between two record arrays, beginning with the copy when the number of
// steps is odd: in place their last kernel would write positions and records that
// its other work-groups still read.
struct StepBuffers {
    double* partial = nullptr;
    char* pos[2] = { nullptr, nullptr };   // records: of the current positions first
    double* copy = nullptr;                // variants 2 and 4
    double* cur = nullptr;                 // the current positions
    double* other = nullptr;               // where the next step puts them
};
sd_status step_buffers(int64_t n, int32_t prec, PairLaunch* L, StepBuffers* sb);
sd_status steps_begin(const sd_params* p, int64_t n, double* x, int64_t steps, int32_t prec,
                      const PairLaunch& L, StepBuffers* sb, hipStream_t st);
// more: another step follows (its records are staged)
sd_status steps_next(const sd_params* p, int64_t n, const void* frc, double* v_prev, double* v_out,
                     double dt, int mode, int32_t prec, const PairLaunch& L, bool more,
                     StepBuffers* sb, hipStream_t st);

void batch_release_graphs();
void run_graphs_release();

}  // namespace sd
