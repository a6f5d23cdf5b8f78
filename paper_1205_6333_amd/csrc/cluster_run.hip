// cluster_run.hip -- the numerical-stability study of Sec. 4: long Euler runs
// of one small free-space cluster (the four sedimenting spheres of Fig. 4)
// with the precision of (a) the accumulation of the hydrodynamic interactions
// and (b) the positions chosen per run.
//
// A run is latency-bound (n <= 64 spheres, tens of millions of dependent
// steps), so each run is one work-group that keeps its cluster in registers for
// every step of a call.  G lanes share sphere i: lane s of the group evaluates
// the pairs of slots s, s + G, ..., where slot k is the k-th sphere j != i in
// ascending order.  The terms of G slots are evaluated at once and then handed
// to all lanes of the group by DPP broadcasts, slot after slot, so that every
// lane forms the sums over j in the order 0..n-1 and does the same Euler update:
// the group's lanes all hold the new position.  Up to eight spheres are one wave
// (G = 16 for n <= 4, 8 for n <= 8), whose lanes fetch x_j from the other groups'
// registers; more are four waves (G = 16, 8, 4 for n <= 16, 32, 64), which
// publish the positions in LDS, two copies in turn, one barrier per step.
// Independent runs (precision variants, time steps) are independent work-groups
// of the same launch.
//
// What bounds a step is its chain of dependent operations: fetch x_j, distance,
// 1/r, coefficients, term, the additions of n - 1 terms, update.  Nanoseconds
// per step of the slowest of the twelve precision variants (and of FP64
// throughout), before, with one lane per sphere and in FP64 a square root and
// two divisions per pair / now: n = 2 714 (581) / 334 (209), 4 1163 (1053) / 442
// (242), 7 1832 (1761) / 697 (400), 12 3165 (2941) / 1187 (632), 30 7262 (7194) /
// 3308 (1937), 64 15312 (15224) / 7882 (4556).  (The slot loop leaves after the
// last slot: sixteen compares cost 200 ns of a four-sphere step.)
#include "pair_terms.h"
#include "sd.h"
#include "sd_host.h"
#include "sd_internal.h"
#include "wave_sym.h"

#include <cmath>
#include <vector>

namespace sd {

struct ClusterRunDev {
    int acc, pos;
    double dt;
    long long steps, stride;
    long long frame0;   // index of the run's first frame in traj
};

// Error-free FP32 sum: a + b = s + e exactly (Knuth's two-sum).
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e)
{
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// Double-single (hi, lo) += (bh, bl), renormalised so that |lo| <= ulp(hi)/2.
__device__ __forceinline__ void ds_add(float& hi, float& lo, float bh, float bl)
{
    float s, e;
    two_sum(hi, bh, s, e);
    e += lo + bl;
    hi = s + e;
    lo = e - (hi - s);
}

// Value v of lane K of this lane's group of G lanes (G 16, 8, 4).
template <int G, int K>
__device__ __forceinline__ int group_bcast(int v)
{
    if constexpr (G == 16) {
        return __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xf, 0xf, true);   // row_newbcast
    } else if constexpr (G == 8) {   // one half of the row of 16 after the other
        const int a = __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xf, 0xf, true);
        return __builtin_amdgcn_update_dpp(a, v, 0x150 + 8 + K, 0xf, 0xc, true);
    } else {
        return __builtin_amdgcn_update_dpp(0, v, K * 0x55, 0xf, 0xf, true);    // quad_perm
    }
}
template <int G, int K>
__device__ __forceinline__ float group_bcast(float v)
{
    return __builtin_bit_cast(float, group_bcast<G, K>(__builtin_bit_cast(int, v)));
}
template <int G, int K>
__device__ __forceinline__ double group_bcast(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = group_bcast<G, K>((int)b), hi = group_bcast<G, K>((int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// f(K), f(K + 1), ... for the slots below cnt (wave-uniform): one compare per
// slot taken and one to leave.
template <int K, int G, class F>
__device__ __forceinline__ void for_slots(int cnt, F&& f)
{
    if constexpr (K < G) {
        if (K < cnt) {
            f(std::integral_constant<int, K>());
            for_slots<K + 1, G>(cnt, f);
        }
    }
}

// Value v of lane `at` / 4 of the wave (at: byte address of the lane).
__device__ __forceinline__ float lane_fetch(int at, float v)
{
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_ds_bpermute(at, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double lane_fetch(int at, double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_ds_bpermute(at, (int)b);
    const int hi = __builtin_amdgcn_ds_bpermute(at, (int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// LDS of a run of several waves: positions of this and the last step, forces.
struct ClusterLds {
    double x[2][3][64], f[3][64];
    float hi[2][3][64], lo[2][3][64];
};

// One run, its precisions fixed at compile time (ACC: sd_acc_mode, POS:
// sd_pos_mode), so that the step loop carries no mode branches.  ONE: a single
// wave and a lane for every slot.
template <int TENSOR, int ACC, int POS, int G, bool ONE>
__device__ __forceinline__ void cluster_body(const ClusterRunDev& R, int n, const PairConst& pc,
                                             double* __restrict__ state,
                                             const double* __restrict__ force,
                                             double* __restrict__ traj, ClusterLds* lds)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int s = tid % G;
    const bool act = tid / G < n;
    const int i = act ? tid / G : 0;   // idle groups repeat sphere 0 and store nothing
    const bool owner = act && s == 0;
    double* st = state + (size_t)blockIdx.x * 6 * (size_t)n;

    // the run's position representation: FP32 (xl = 0), double-single (xh, xl)
    // or FP64 (x64; xh, xl its FP32 head and tail for the FP32 differences)
    float xh[3], xl[3];
    double x64[3], f[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double v = st[3 * i + k] + st[3 * (size_t)n + 3 * i + k];
        f[k] = force[3 * i + k];
        xh[k] = (float)v;
        xl[k] = (POS == SD_POS_FP32) ? 0.0f : (float)(v - (double)xh[k]);
        x64[k] = (POS == SD_POS_FP64) ? v : (double)xh[k] + (double)xl[k];
    }
    const float gamma = pc.gamma_f, m3g = pc.m3gamma_f, thr2 = pc.thr2_f;
    const double m3gd = -3.0 * pc.gamma;
    // FP64 pairs that the far form does not cover
    const double odd2 = (TENSOR == T_RPY && pc.overlap) ? 4.0 * pc.a * pc.a : 0.0;
    const int slots = n - 1;
    const int rounds = ONE ? 1 : (slots + G - 1) / G;
    constexpr int MAXS = !ONE ? G : (G == 16 ? 3 : 7);   // slots of a round
    // the sphere of this lane's slot of a round (a slot beyond the last repeats
    // the last: its term is not added)
    auto sphere = [&](int r) {
        const int k = min(r * G + s, slots - 1);
        return k < 0 ? 0 : k + (k >= i ? 1 : 0);
    };
    // the constant force of the sphere of this lane's slot
    int j = sphere(0);
    double fj[3];
    if constexpr (ONE) {
#pragma unroll
        for (int k = 0; k < 3; ++k) fj[k] = lane_fetch(4 * G * j, f[k]);
    } else {
        if (owner)
            for (int k = 0; k < 3; ++k) lds->f[k][i] = f[k];
        // (read after the first step's barrier)
    }
    int b = 0;   // copy of the positions in LDS
    // component k of x_j: FP64, FP32 head, FP32 tail
    auto xj64 = [&](int k) { return ONE ? lane_fetch(4 * G * j, x64[k]) : lds->x[b][k][j]; };
    auto xjh = [&](int k) { return ONE ? lane_fetch(4 * G * j, xh[k]) : lds->hi[b][k][j]; };
    auto xjl = [&](int k) { return ONE ? lane_fetch(4 * G * j, xl[k]) : lds->lo[b][k][j]; };

    long long frame = R.frame0, since = 0;  // next frame, steps since the last one
    for (long long step = 0; step < R.steps; ++step) {
        double v[3];
        double a[3] = { 0.0, 0.0, 0.0 };           // FP64 sums (physical units)
        float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;     // sums (scaled units, Eq. 7 / alpha)
        float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;     // Kahan compensation or double-single tail
        if constexpr (!ONE) {
            b ^= 1;
            if (owner) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    lds->x[b][k][i] = x64[k];
                    if (ACC != SD_ACC_FP64) lds->hi[b][k][i] = xh[k];
                    if (ACC != SD_ACC_FP64 && POS != SD_POS_FP32) lds->lo[b][k][i] = xl[k];
                }
            }
            __syncthreads();   // (the other copy's readers are past it too)
        }
#pragma unroll 1
        for (int r = 0; r < rounds; ++r) {
            if constexpr (!ONE) {
                j = sphere(r);
#pragma unroll
                for (int k = 0; k < 3; ++k) fj[k] = lds->f[k][j];
            }
            const int cnt = min(G, slots - r * G);   // slots of this round
            if constexpr (ACC == SD_ACC_FP64) {
                double d[3], t[3] = { 0.0, 0.0, 0.0 };
#pragma unroll
                for (int k = 0; k < 3; ++k) d[k] = x64[k] - xj64(k);
                const double r2 = fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2]));
                double A, Bt;
                far_coef<TENSOR>(rsqrt_f64(r2), pc.gamma, m3gd, A, Bt);
                const double sB = Bt * fma(d[0], fj[0], fma(d[1], fj[1], d[2] * fj[2]));
#pragma unroll
                for (int k = 0; k < 3; ++k) t[k] = pc.alpha * fma(A, fj[k], sB * d[k]);
                const bool odd = !(r2 > 0.0 && r2 >= odd2 && r2 < 1e300);
                if (__builtin_amdgcn_ballot_w64(odd) != 0) {   // overlap, coincident, not finite
                    if (odd) {
                        t[0] = t[1] = t[2] = 0.0;
                        near_term<TENSOR>(pc, d[0], d[1], d[2], fj[0], fj[1], fj[2], t[0], t[1],
                                          t[2]);
                    }
                }
                for_slots<0, MAXS>(cnt, [&](auto k_c) {
                    constexpr int k = decltype(k_c)::value;
                    a[0] += group_bcast<G, k>(t[0]);
                    a[1] += group_bcast<G, k>(t[1]);
                    a[2] += group_bcast<G, k>(t[2]);
                });
            } else {
                float dx = xh[0] - xjh(0), dy = xh[1] - xjh(1), dz = xh[2] - xjh(2);
                if (POS != SD_POS_FP32) {
                    dx += xl[0] - xjl(0);
                    dy += xl[1] - xjl(1);
                    dz += xl[2] - xjl(2);
                }
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                const float fx = (float)fj[0], fy = (float)fj[1], fz = (float)fj[2];
                const float rinv = __builtin_amdgcn_rsqf(r2);
                const float rinv2 = rinv * rinv, rinv3 = rinv2 * rinv;
                float A, Bt;
                if (TENSOR == T_OSEEN) {
                    A = rinv;
                    Bt = rinv3;
                } else {
                    A = fmaf(gamma, rinv3, rinv);
                    Bt = rinv3 * fmaf(m3g, rinv2, 1.0f);
                }
                const float sB = Bt * fmaf(dx, fx, fmaf(dy, fy, dz * fz));
                const float t0 = fmaf(A, fx, sB * dx);
                const float t1 = fmaf(A, fy, sB * dy);
                const float t2 = fmaf(A, fz, sB * dz);
                auto add = [&](float u0, float u1, float u2) {
                    if (ACC == SD_ACC_FP32) {
                        s0 += u0;
                        s1 += u1;
                        s2 += u2;
                    } else if (ACC == SD_ACC_KAHAN) {
                        const float y0 = u0 - c0, y1 = u1 - c1, y2 = u2 - c2;
                        const float w0 = s0 + y0, w1 = s1 + y1, w2 = s2 + y2;
                        c0 = (w0 - s0) - y0;
                        c1 = (w1 - s1) - y1;
                        c2 = (w2 - s2) - y2;
                        s0 = w0;
                        s1 = w1;
                        s2 = w2;
                    } else {
                        ds_add(s0, c0, u0, 0.0f);
                        ds_add(s1, c1, u1, 0.0f);
                        ds_add(s2, c2, u2, 0.0f);
                    }
                };
                const bool near = r2 < thr2;
                if (__builtin_amdgcn_ballot_w64(near) == 0) {
                    for_slots<0, MAXS>(cnt, [&](auto k_c) {
                        constexpr int k = decltype(k_c)::value;
                        add(group_bcast<G, k>(t0), group_bcast<G, k>(t1), group_bcast<G, k>(t2));
                    });
                } else {   // rare: near pairs in FP64, and not in the FP32 sums
                    double e[3], m[3] = { 0.0, 0.0, 0.0 };
#pragma unroll
                    for (int k = 0; k < 3; ++k) e[k] = x64[k] - xj64(k);
                    if (near)
                        near_term<TENSOR>(pc, e[0], e[1], e[2], (double)fx, (double)fy, (double)fz,
                                          m[0], m[1], m[2]);
#pragma unroll 1
                    for (int k = 0; k < cnt; ++k) {
                        const int from = 4 * (lane - s + k);
                        const float u0 = lane_fetch(from, t0), u1 = lane_fetch(from, t1),
                                    u2 = lane_fetch(from, t2);
                        const double m0 = lane_fetch(from, m[0]), m1 = lane_fetch(from, m[1]),
                                     m2 = lane_fetch(from, m[2]);
                        if (lane_fetch(from, near ? 1.0f : 0.0f) != 0.0f) {
                            a[0] += m0;
                            a[1] += m1;
                            a[2] += m2;
                        } else {
                            add(u0, u1, u2);
                        }
                    }
                }
            }
        }
        if constexpr (ACC == SD_ACC_FP64) {
#pragma unroll
            for (int k = 0; k < 3; ++k) v[k] = pc.mu0 * f[k] + a[k];
        } else {
            // Kahan: the sum is s - c; double-single: s + c
            const double sg = (ACC == SD_ACC_KAHAN) ? -1.0 : 1.0;
            v[0] = pc.mu0 * f[0] + pc.alpha * ((double)s0 + sg * (double)c0) + a[0];
            v[1] = pc.mu0 * f[1] + pc.alpha * ((double)s1 + sg * (double)c1) + a[1];
            v[2] = pc.mu0 * f[2] + pc.alpha * ((double)s2 + sg * (double)c2) + a[2];
        }
        // Euler update in the run's position precision
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double inc = R.dt * v[k];
            if (POS == SD_POS_FP32) {
                xh[k] = xh[k] + (float)inc;
                x64[k] = (double)xh[k];
            } else if (POS == SD_POS_DS) {
                const float ih = (float)inc;
                ds_add(xh[k], xl[k], ih, (float)(inc - (double)ih));
                x64[k] = (double)xh[k] + (double)xl[k];
            } else {
                x64[k] += inc;
                xh[k] = (float)x64[k];
                xl[k] = (float)(x64[k] - (double)xh[k]);
            }
        }
        if (R.stride > 0 && ++since == R.stride) {
            since = 0;
            if (owner) {
                double* fr = traj + (size_t)frame * 3 * (size_t)n;
                fr[3 * i] = x64[0];
                fr[3 * i + 1] = x64[1];
                fr[3 * i + 2] = x64[2];
            }
            ++frame;
        }
    }
    if (owner)
        for (int k = 0; k < 3; ++k) {
            if (POS == SD_POS_DS) {
                st[3 * i + k] = (double)xh[k];
                st[3 * (size_t)n + 3 * i + k] = (double)xl[k];
            } else {
                st[3 * i + k] = (POS == SD_POS_FP32) ? (double)xh[k] : x64[k];
                st[3 * (size_t)n + 3 * i + k] = 0.0;
            }
        }
}

template <int TENSOR, int G, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_cluster_run(const ClusterRunDev* __restrict__ runs, int n, PairConst pc,
              double* __restrict__ state, const double* __restrict__ force,
              double* __restrict__ traj)
{
    constexpr bool ONE = THREADS == 64;
    __shared__ std::conditional_t<ONE, char, ClusterLds> lds;
    const ClusterRunDev R = runs[blockIdx.x];
#define SD_CR(A, P)                                                                            \
    if (R.acc == A && R.pos == P) {                                                            \
        cluster_body<TENSOR, A, P, G, ONE>(R, n, pc, state, force, traj, (ClusterLds*)&lds);   \
        return;                                                                                \
    }
    SD_CR(0, 0) SD_CR(0, 1) SD_CR(0, 2) SD_CR(1, 0) SD_CR(1, 1) SD_CR(1, 2)
    SD_CR(2, 0) SD_CR(2, 1) SD_CR(2, 2) SD_CR(3, 0) SD_CR(3, 1) SD_CR(3, 2)
#undef SD_CR
}

template <int TENSOR>
static void launch_cluster_run(const ClusterRunDev* recs, int runs, int n, const PairConst& pc,
                               double* state, const double* force, double* traj, hipStream_t st)
{
#define SD_GO(G, T)                                                                             \
    hipLaunchKernelGGL((k_cluster_run<TENSOR, G, T>), dim3((unsigned)runs), dim3(T), 0, st, recs, \
                       n, pc, state, force, traj)
    if (n <= 4) SD_GO(16, 64);
    else if (n <= 8) SD_GO(8, 64);
    else if (n <= 16) SD_GO(16, 256);
    else if (n <= 32) SD_GO(8, 256);
    else SD_GO(4, 256);
#undef SD_GO
}

}  // namespace sd

using namespace sd;

extern "C" sd_status sd_cluster_run(const sd_params* p, int64_t n, int32_t runs,
                                    const sd_cluster_spec* specs, double* state,
                                    const double* force, double* traj, void* stream)
{
    sd_status st;
    if ((st = check_params(p)) || (st = check_free_space(p, "sd_cluster_run"))) return st;
    if (n < 1 || n > SD_CLUSTER_MAX_N)
        return fail(SD_EINVAL, "n must be in [1, %d] (got %lld)", SD_CLUSTER_MAX_N, (long long)n);
    if (runs < 1 || runs > SD_CLUSTER_MAX_RUNS)
        return fail(SD_EINVAL, "runs must be in [1, %d]", SD_CLUSTER_MAX_RUNS);
    if (!specs) return fail(SD_EINVAL, "specs is NULL");
    if ((st = check_ptr(state, 8, "state")) || (st = check_ptr(force, 8, "force"))) return st;
    std::vector<ClusterRunDev> rec((size_t)runs);
    long long frames = 0;
    for (int r = 0; r < runs; ++r) {
        const sd_cluster_spec& s = specs[r];
        if (s.acc < SD_ACC_FP32 || s.acc > SD_ACC_FP64)
            return fail(SD_EINVAL, "run %d: unknown accumulation mode %d", r, s.acc);
        if (s.pos < SD_POS_FP32 || s.pos > SD_POS_FP64)
            return fail(SD_EINVAL, "run %d: unknown position mode %d", r, s.pos);
        if (!(s.dt > 0.0) || !std::isfinite(s.dt))
            return fail(SD_EINVAL, "run %d: dt must be finite and > 0", r);
        if (s.steps < 0 || s.stride < 0)
            return fail(SD_EINVAL, "run %d: steps and stride must be >= 0", r);
        rec[r].acc = s.acc;
        rec[r].pos = s.pos;
        rec[r].dt = s.dt;
        rec[r].steps = s.steps;
        rec[r].stride = s.stride;
        rec[r].frame0 = frames;
        if (s.stride > 0) frames += s.steps / s.stride;
    }
    if (frames > 0 && (st = check_ptr(traj, 8, "traj"))) return st;
    hipStream_t hs = (hipStream_t)stream;
    void* buf = nullptr;
    if ((st = ws_get(WS_CLUSTER, rec.size() * sizeof(ClusterRunDev), &buf))) return st;
    // the run records go through library workspace; the upload is complete
    // (and the host vector free to go) when the call returns
    if (hipMemcpyAsync(buf, rec.data(), rec.size() * sizeof(ClusterRunDev),
                       hipMemcpyHostToDevice, hs) != hipSuccess ||
        hipStreamSynchronize(hs) != hipSuccess)
        return fail(SD_EDEVICE, "cluster-run record upload failed");
    const PairConst pc = pair_const(p);
    if (p->tensor == SD_OSEEN)
        launch_cluster_run<T_OSEEN>((const ClusterRunDev*)buf, runs, (int)n, pc, state, force, traj,
                                    hs);
    else
        launch_cluster_run<T_RPY>((const ClusterRunDev*)buf, runs, (int)n, pc, state, force, traj,
                                  hs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SD_EDEVICE, "cluster-run launch: %s", hipGetErrorString(e));
    return SD_OK;
}
