// integrate.hip -- O(N) kernels of the time loop (Sec. 3.1, step 1) and small
// helpers: FP64 -> FP32 staging of positions, split merge fused with the
// Euler / AB2 position update, packing for the adjoint loop.
#include "pair_terms.h"
#include "sd_internal.h"

#include <algorithm>

namespace sd {

template <typename P4>
__global__ void __launch_bounds__(256) k_stage(const double* __restrict__ x, P4* __restrict__ pos,
                                               int n, double qs, double* __restrict__ copy)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double v[3] = { x[3 * (size_t)i], x[3 * (size_t)i + 1], x[3 * (size_t)i + 2] };
    put_pos(pos, i, v[0], v[1], v[2], qs);
    if (copy)
        for (int k = 0; k < 3; ++k) copy[3 * (size_t)i + k] = v[k];
}

__global__ void __launch_bounds__(256) k_stage_q_from_f32(const float4* __restrict__ pos,
                                                          float4* __restrict__ q, int n, double qs)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float4 p = pos[i];
    put_pos(q, i, (double)p.x, (double)p.y, (double)p.z, qs);
}

// v_k = mu0 F + sum_s partial_s (the same order as k_merge), then
//   mode 0: x_out = x_in + dt v                       (Euler)
//   mode 1: x_out = x_in + dt v,  v_prev = v           (first AB2 step)
//   mode 2: x_out = x_in + dt (3/2 v - 1/2 v_prev), v_prev = v   (AB2)
// (x_out may be x_in)
// and the staged copy of the new positions for the next pair kernel.
template <typename F4, typename P4>
__global__ void __launch_bounds__(256)
k_merge_integrate(const double* __restrict__ partial, int S, int n, const F4* __restrict__ frc,
                  double mu0, const double* x_in, double* x_out, double* __restrict__ v_prev,
                  double* __restrict__ v_out, double dt, int mode, P4* __restrict__ pos_next,
                  double qs)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const F4 f = frc[i];
    double v[3] = { mu0 * (double)f.x, mu0 * (double)f.y, mu0 * (double)f.z };
    add_split_rows(partial, S, n, i, v[0], v[1], v[2]);
    double xn[3];
    step_particle({ x_in, x_out, v_prev, v_out, dt, mode }, i, v, xn);
    if (pos_next) put_pos(pos_next, i, xn[0], xn[1], xn[2], qs);
}

template <typename P4>
__global__ void __launch_bounds__(256) k_pack(const double* __restrict__ v, P4* __restrict__ out,
                                              int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    put_pos(out, i, v[3 * (size_t)i], v[3 * (size_t)i + 1], v[3 * (size_t)i + 2], 0.0);
}

__global__ void __launch_bounds__(256) k_fill_i32(int32_t* __restrict__ p, int32_t value, int count)
{
    for (int k = blockIdx.x * 256 + threadIdx.x; k < count; k += (int)gridDim.x * 256) p[k] = value;
}

// out = (1/n) sum_i v_i in a fixed order, in two launches: G = mean_groups(n)
// work-groups each sum a contiguous range of ceil(n / G) particles (lane t:
// particles t, t + 256, ... of the range in order, then a fixed-shape tree
// over the 256 lanes) into partial[c G + g]; one work-group then sums the G
// partials the same way.  The grouping depends on n only, so the result does
// not depend on the device or on the scheduling of the work-groups.
int64_t mean_groups(int64_t n)
{
    const int64_t g = (n + 1023) / 1024;
    return g < 1 ? 1 : (g > 1024 ? 1024 : g);
}

// the three lane sums of a 256-lane work-group -> lane 0, fixed shape
__device__ __forceinline__ void tree3(double (&red)[3][256], int t, double a0, double a1,
                                      double a2)
{
    red[0][t] = a0;
    red[1][t] = a1;
    red[2][t] = a2;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            red[0][t] += red[0][t + w];
            red[1][t] += red[1][t + w];
            red[2][t] += red[2][t + w];
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) k_mean_partial(const double* __restrict__ v, int64_t n,
                                                      int64_t chunk, int groups,
                                                      double* __restrict__ partial)
{
    __shared__ double red[3][256];
    const int t = threadIdx.x, g = blockIdx.x;
    const int64_t i0 = (int64_t)g * chunk;
    const int64_t i1 = i0 + chunk < n ? i0 + chunk : n;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int64_t i = i0 + t; i < i1; i += 256) {
        a0 += v[3 * i];
        a1 += v[3 * i + 1];
        a2 += v[3 * i + 2];
    }
    tree3(red, t, a0, a1, a2);
    if (t < 3) partial[(int64_t)t * groups + g] = red[t][0];
}

__global__ void __launch_bounds__(256) k_mean_final(const double* __restrict__ partial,
                                                    int groups, int64_t n,
                                                    double* __restrict__ out)
{
    __shared__ double red[3][256];
    const int t = threadIdx.x;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int k = t; k < groups; k += 256) {
        a0 += partial[k];
        a1 += partial[groups + k];
        a2 += partial[2 * groups + k];
    }
    tree3(red, t, a0, a1, a2);
    if (t < 3) out[t] = red[t][0] / (double)n;
}

hipError_t launch_mean_vector(const double* v, int64_t n, double* out, double* partial,
                              hipStream_t st)
{
    const int64_t g = mean_groups(n);
    const int64_t chunk = (n + g - 1) / g;
    hipLaunchKernelGGL(k_mean_partial, dim3((unsigned)g), dim3(256), 0, st, v, n, chunk, (int)g,
                       partial);
    hipLaunchKernelGGL(k_mean_final, dim3(1), dim3(256), 0, st, partial, (int)g, n, out);
    return hipGetLastError();
}

static inline dim3 grid_for(int64_t n) { return dim3((unsigned)((n + 255) / 256)); }

// 2^32 / Lb, the fixed-point scale of a periodic box (0 in free space)
static inline double q_scale(double box) { return box > 0.0 ? 4294967296.0 / box : 0.0; }

hipError_t launch_stage(bool f64, const double* x, void* pos, int n, double box, double* copy,
                        hipStream_t st)
{
    if (f64)
        hipLaunchKernelGGL((k_stage<double4>), grid_for(n), dim3(256), 0, st, x, (double4*)pos, n,
                           0.0, copy);
    else
        hipLaunchKernelGGL((k_stage<float4>), grid_for(n), dim3(256), 0, st, x, (float4*)pos, n,
                           q_scale(box), copy);
    return hipGetLastError();
}

hipError_t launch_stage_q_from_f32(const float4* pos, float4* q, int n, double box,
                                   hipStream_t st)
{
    hipLaunchKernelGGL(k_stage_q_from_f32, grid_for(n), dim3(256), 0, st, pos, q, n,
                       q_scale(box));
    return hipGetLastError();
}

hipError_t launch_merge_integrate(bool f64, const double* partial, int splits, int n,
                                  const void* frc, double mu0, const double* x_in, double* x_out,
                                  double* v_prev, double* v_out, double dt, int mode,
                                  void* pos_next, double box, hipStream_t st)
{
    if (f64)
        hipLaunchKernelGGL((k_merge_integrate<double4, double4>), grid_for(n), dim3(256), 0, st,
                           partial, splits, n, (const double4*)frc, mu0, x_in, x_out, v_prev, v_out,
                           dt, mode, (double4*)pos_next, 0.0);
    else
        hipLaunchKernelGGL((k_merge_integrate<float4, float4>), grid_for(n), dim3(256), 0, st,
                           partial, splits, n, (const float4*)frc, mu0, x_in, x_out, v_prev, v_out,
                           dt, mode, (float4*)pos_next, q_scale(box));
    return hipGetLastError();
}

hipError_t launch_pack_f32(const double* v, float4* out, int n, hipStream_t st)
{
    hipLaunchKernelGGL((k_pack<float4>), grid_for(n), dim3(256), 0, st, v, out, n);
    return hipGetLastError();
}

hipError_t launch_pack_f64(const double* v, double4* out, int n, hipStream_t st)
{
    hipLaunchKernelGGL((k_pack<double4>), grid_for(n), dim3(256), 0, st, v, out, n);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t value, int count, hipStream_t st)
{
    const int groups = std::min((count + 255) / 256, 1024);
    hipLaunchKernelGGL(k_fill_i32, dim3(groups), dim3(256), 0, st, p, value, count);
    return hipGetLastError();
}

}  // namespace sd
