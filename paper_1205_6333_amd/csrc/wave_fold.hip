// wave_fold.hip -- the fold of the wave-symmetric products: partial sums to
// velocities or to the next positions of the time loop.
#include "pair_terms.h"
#include "sd_internal.h"
#include "wave_sym.h"

namespace sd {

// Sum of the partials of a particle: its j-side partials of the blocks
// I = J - 1, J - 2, ... (and the antipode), and its split rows.  A work-group
// takes 32 particles; its eight slices of 32 lanes take every eighth term, each
// with its loads issued in groups, and the slices are added in order.  Then, by mode: velocities (mu0 F + sum), or a step of the time
// loop (as k_merge_integrate); the positions may be updated in place, since
// the pair kernel has finished with them.
template <typename V4>
__global__ void __launch_bounds__(256)
k_wave_fold(const double* __restrict__ partial, const double* __restrict__ jpart, int n, int B,
            WaveShape sh, const V4* __restrict__ frc, double mu0, double* __restrict__ vel,
            const double* x_in, double* x_out, double* __restrict__ v_prev,
            double* __restrict__ v_out, double dt, int mode, V4* __restrict__ pos_next, double qs)
{
    __shared__ double s_sum[8][3][32];
    const int t = threadIdx.x & 31, sl = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + t;
    double v[3] = { 0.0, 0.0, 0.0 };
    if (i < n) {
        const int J = i / B, o = i - J * B;
        const int half = sh.nb >> 1;
        const size_t cs = (size_t)sh.nb * (size_t)sh.lmax;
        const int Ie = J >= half ? J - half : J + half;
        const int nd = sh.h + ((sh.extra && Ie < half) ? 1 : 0);
        constexpr int G = 4;
        for (int d0 = sl; d0 < nd; d0 += 8 * G) {
            double g[G][3];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int d = d0 + 8 * u;   // block I = J - d - 1 (mod nb)
                if (d < nd) {
                    int I = J - d - 1;
                    if (I < 0) I += sh.nb;
                    const double* at = jpart + (size_t)I * sh.lmax + (size_t)d * B + o;
                    g[u][0] = at[0];
                    g[u][1] = at[cs];
                    g[u][2] = at[2 * cs];
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (d0 + 8 * u < nd)
                    for (int c = 0; c < 3; ++c) v[c] += g[u][c];
        }
        const int rows = sh.splits + 1;
        const size_t rs = 3 * (size_t)n;
        for (int r0 = sl; r0 < rows; r0 += 8 * G) {
            double g[G][3];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int r = r0 + 8 * u;
                if (r < rows) {
                    const double* at = partial + (size_t)r * rs + i;
                    g[u][0] = at[0];
                    g[u][1] = at[n];
                    g[u][2] = at[2 * (size_t)n];
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (r0 + 8 * u < rows)
                    for (int c = 0; c < 3; ++c) v[c] += g[u][c];
        }
    }
    for (int c = 0; c < 3; ++c) s_sum[sl][c][t] = v[c];
    __syncthreads();
    if (sl != 0 || i >= n) return;
    const V4 f = frc[i];
    double u[3] = { mu0 * (double)f.x, mu0 * (double)f.y, mu0 * (double)f.z };
    for (int k = 0; k < 8; ++k)
        for (int c = 0; c < 3; ++c) u[c] += s_sum[k][c][t];
    if (vel) {
        for (int c = 0; c < 3; ++c) vel[3 * (size_t)i + c] = u[c];
        return;
    }
    double xn[3];
    step_particle({ x_in, x_out, v_prev, v_out, dt, mode }, i, u, xn);
    if (pos_next) put_pos(pos_next, i, xn[0], xn[1], xn[2], qs);
}

hipError_t launch_wave_fold(const PairLaunch& L, bool f64, int n, const PairConst& pc,
                            const double* partial, const void* frc, double* vel,
                            const double* x_in, double* x_out, double* v_prev, double* v_out,
                            double dt, int mode, void* pos_next, hipStream_t st)
{
    const WaveShape sh = wave_shape_of(L, n);
    const double* jpart = (const double*)((const char*)partial + wave_jpart_offset(sh, n));
    const dim3 grid((unsigned)((n + 31) / 32)), block(256);
    const double qs = pc.box > 0.0 ? 4294967296.0 / pc.box : 0.0;
    if (f64)
        hipLaunchKernelGGL((k_wave_fold<double4>), grid, block, 0, st, partial, jpart, n, 64 * L.ilp,
                           sh, (const double4*)frc, pc.mu0, vel, x_in, x_out, v_prev, v_out, dt, mode,
                           (double4*)pos_next, qs);
    else
        hipLaunchKernelGGL((k_wave_fold<float4>), grid, block, 0, st, partial, jpart, n, 64 * L.ilp,
                           sh, (const float4*)frc, pc.mu0, vel, x_in, x_out, v_prev, v_out, dt, mode,
                           (float4*)pos_next, qs);
    return hipGetLastError();
}

}  // namespace sd
