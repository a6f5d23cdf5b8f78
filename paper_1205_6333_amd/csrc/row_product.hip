// row_product.hip -- the product of small suspensions in one launch: a
// work-group sums whole rows of M(x) F, adds the self term and writes the
// velocities or takes the time step, with no partial sums in memory.
//
// A work-group of 256 lanes owns ILP particles i; lane t takes the particles
// j = t, t + 256, ...  The 256 partial sums of each component are added in
// LDS in a fixed order.  Every ordered pair is evaluated, but nothing but the
// result leaves the work-group: below some thousands of particles that costs
// less than the split rows and the second launch of the kernels that evaluate
// a pair once.
#include "pair_terms.h"
#include "premise.h"
#include "sd_internal.h"
#include "wave_sym.h"

namespace sd {

// What becomes of the velocities.
struct RowOut {
    double* vel;           // f64[3n]: the product's result; null: a time step
    const double* x_in;    // positions before the step
    double* x_out;         // and after it (not the same array)
    double* v_prev;        // AB2 history (mode 1 and 2)
    double* v_out;         // may be null
    void* pos_next;        // records of the new positions, may be null
    double dt, mu0, qs;    // qs: fixed-point scale of a periodic box (FP32), 0 otherwise
    int mode;              // 0 Euler, 1 AB2 start, 2 AB2
};

template <typename V4>
__device__ __forceinline__ void row_finish(const RowOut& o, int i, const V4 f, const double* sum)
{
    double v[3] = { o.mu0 * (double)f.x + sum[0], o.mu0 * (double)f.y + sum[1],
                    o.mu0 * (double)f.z + sum[2] };
    if (o.vel) {
        for (int c = 0; c < 3; ++c) o.vel[3 * (size_t)i + c] = v[c];
        return;
    }
    double xn[3];
    step_particle({ o.x_in, o.x_out, o.v_prev, o.v_out, o.dt, o.mode }, i, v, xn);
    if (o.pos_next) put_pos((V4*)o.pos_next, i, xn[0], xn[1], xn[2], o.qs);
}

// Sum over the work-group of V values per lane (s: V x 256 doubles of LDS): 16
// lanes per value add 16 entries each in order, then the 16 sums by rotations.
// The totals are left in s[0 .. V).
template <int V>
__device__ __forceinline__ void group_sum(double* s, const double (&v)[V])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < V; ++k) s[k * 256 + t] = v[k];
    __syncthreads();
    double a = 0.0;
    if (t < 16 * V) {
        const double* p = s + (t >> 4) * 256 + (t & 15);
#pragma unroll
        for (int k = 0; k < 16; ++k) a += p[16 * k];
        a += row_rot<8>(a);
        a += row_rot<4>(a);
        a += row_rot<2>(a);
        a += row_rot<1>(a);
    }
    __syncthreads();
    if (t < 16 * V && (t & 15) == 0) s[t >> 4] = a;
    __syncthreads();
}

// FP32 terms in blocks of two, two blocks added in FP32, and in FP64 from
// there on; near pairs in FP64.
//
// A step of a few hundred particles is bound by latency: the launch, two or
// three dependent loads, one or two rounds of pairs and the sum in LDS.  Four
// waves share a row so that n = 256 already has 1024 of them.  Larger n are
// bound by the vector ALU and the reads of j: two particles per work-group
// share each read (four took 166 registers and were slower from n = 4500 on).
// Microseconds per Euler step, two launches of the kernels used before / one
// particle / two: n = 8 8.9 / 3.8 / 4.3, 256 13.1 / 4.0 / 4.5, 1000 14.7 / 5.6 /
// 6.0, 2000 10.9 / 9.4 / 8.2, 4000 19.1 / 21.1 / 17.5, 5324 26.9 / 32.6 / 25.3,
// 6007 29.6 / 40.8 / 30.5 (before: one-sided to 1023, then wave-symmetric).
template <int TENSOR, bool PER, int ILP>
__global__ void __launch_bounds__(256)
k_row_f32(const float4* __restrict__ pos, const float4* __restrict__ frc,
          const double* __restrict__ x64, int n, PairConst pc, RowOut out,
          unsigned long long* __restrict__ premise)
{
    __shared__ double s_sum[3 * ILP * 256];
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * ILP;
    V3<float> x[ILP];
    double acc[3 * ILP];
#pragma unroll
    for (int a = 0; a < ILP; ++a) {
        const float4 p = pos[min(i0 + a, n - 1)];
        x[a] = { p.x, p.y, p.z };
        keep(x[a]);   // in VGPRs (an SGPR operand halves the issue rate)
        acc[3 * a] = acc[3 * a + 1] = acc[3 * a + 2] = 0.0;
    }
    // the lane's own slots take its near pairs (the loop is rare, and indexed
    // registers are not to be had)
#pragma unroll
    for (int k = 0; k < 3 * ILP; ++k) s_sum[k * 256 + tid] = 0.0;
    float gamma = pc.gamma_f, m3g = pc.m3gamma_f, thr2 = pc.thr2_f, one = 1.0f;
    asm volatile("" : "+v"(gamma), "+v"(m3g), "+v"(thr2), "+v"(one));
    // particles j = j0 + 256 u + tid, u < U (full: all of them exist)
    auto body = [&](auto u_c, int j0, bool full) {
        constexpr int U = decltype(u_c)::value;
        float4 pj[U], fj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + 256 * u + tid;
            const float far = PER ? 0.0f : 1.0e15f;
            pj[u] = make_float4(far, far, far, 0.0f);
            fj[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (full || j < n) {
                pj[u] = pos[j];
                fj[u] = frc[j];
            }
        }
        uint32_t nearm = 0;   // bit a U + u: the pair of particles a and u is near
#pragma unroll
        for (int a = 0; a < ILP; ++a) {
            __builtin_amdgcn_sched_barrier(0);   // one particle's pair data live at a time
            V3<float> d[U];
            float r2[U], rmin = 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                d[u] = { pdiff<PER>(x[a].x, pj[u].x), pdiff<PER>(x[a].y, pj[u].y),
                         pdiff<PER>(x[a].z, pj[u].z) };
                r2[u] = dot(d[u], d[u]);
                rmin = u == 0 ? r2[0] : fminf(rmin, r2[u]);
            }
            if (__builtin_amdgcn_ballot_w64(rmin < thr2) != 0) {   // near or self pair
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool nr = r2[u] < thr2;
                    nearm |= nr ? 1u << (a * U + u) : 0u;
                    r2[u] = nr ? __builtin_inff() : r2[u];
                }
            }
            V3<float> y = { 0.0f, 0.0f, 0.0f }, g = y;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float rinv = __builtin_amdgcn_rsqf(r2[u]);
                const float rinv2 = rinv * rinv, rinv3 = rinv2 * rinv;
                float A = rinv, Bt = rinv3;
                if (TENSOR == T_RPY) {
                    A = fmaf(gamma, rinv3, rinv);
                    Bt = rinv3 * fmaf(m3g, rinv2, one);
                }
                const V3<float> f = { fj[u].x, fj[u].y, fj[u].z };
                const float sB = Bt * dot(d[u], f);
                g.x = fmaf(A, f.x, u % 2 == 0 ? sB * d[u].x : fmaf(sB, d[u].x, g.x));
                g.y = fmaf(A, f.y, u % 2 == 0 ? sB * d[u].y : fmaf(sB, d[u].y, g.y));
                g.z = fmaf(A, f.z, u % 2 == 0 ? sB * d[u].z : fmaf(sB, d[u].z, g.z));
                if (u == 1 || U == 1) y = g;
                else if (u % 2 == 1) y = add(y, g);
            }
            acc[3 * a] = fma(pc.alpha_sum, (double)y.x, acc[3 * a]);
            acc[3 * a + 1] = fma(pc.alpha_sum, (double)y.y, acc[3 * a + 1]);
            acc[3 * a + 2] = fma(pc.alpha_sum, (double)y.z, acc[3 * a + 2]);
        }
        if (__builtin_amdgcn_ballot_w64(nearm != 0) != 0)   // rare
#pragma unroll 1
            for (int b = 0; b < ILP * U; ++b) {
                const int a = b / U, u = b % U;
                const int i = i0 + a, jg = j0 + 256 * u + tid;
                int cls = PREMISE_OK;
                if (((nearm >> b) & 1u) && i < n && jg < n && i != jg) {
                    const float4 pi = pos[i], qj = pos[jg], f = frc[jg];
                    double dx, dy, dz;
                    near_diff_v<PER>(pi.x, pi.y, pi.z, i, qj, jg, pc, x64, dx, dy, dz);
                    double* const own = s_sum + 3 * a * 256 + tid;
                    cls = near_term<TENSOR>(pc, dx, dy, dz, (double)f.x, (double)f.y, (double)f.z,
                                            own[0], own[256], own[512]);
                }
                count_premise(premise, i < jg ? cls : (int)PREMISE_OK);
            }
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;
    typedef std::integral_constant<int, 4> Four;
    int j0 = 0;
#pragma unroll 1
    for (; j0 + 1024 <= n; j0 += 1024) body(Four(), j0, true);
    const int left = n - j0;
    if (left > 512)
        body(Four(), j0, false);
    else if (left > 256)
        body(Two(), j0, false);
    else if (left > 0)
        body(One(), j0, false);
#pragma unroll
    for (int k = 0; k < 3 * ILP; ++k) acc[k] += s_sum[k * 256 + tid];
    group_sum<3 * ILP>(s_sum, acc);
    if (tid < ILP && i0 + tid < n) row_finish(out, i0 + tid, frc[i0 + tid], s_sum + 3 * tid);
}

// The same in FP64 (microseconds per Euler step, before / one / two: n = 256 15.1
// / 4.3 / 4.3, 1200 10.0 / 7.4 / 6.7, 3000 17.6 / 22.5 / 15.4, 4000 23.6 / 36.3 /
// 23.8).
template <int TENSOR, bool PER, int ILP>
__global__ void __launch_bounds__(256)
k_row_f64(const double4* __restrict__ pos, const double4* __restrict__ frc, int n, PairConst pc,
          RowOut out, unsigned long long* __restrict__ premise)
{
    __shared__ double s_sum[3 * ILP * 256];
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * ILP;
    V3<double> x[ILP];
    double acc[3 * ILP];
#pragma unroll
    for (int a = 0; a < ILP; ++a) {
        const double4 p = pos[min(i0 + a, n - 1)];
        x[a] = { p.x, p.y, p.z };
        acc[3 * a] = acc[3 * a + 1] = acc[3 * a + 2] = 0.0;
    }
    const double gamma = pc.gamma, m3g = -3.0 * pc.gamma, thr2 = pc.thr2_d;
#pragma unroll 1
    for (int j = tid; j < n; j += 256) {
        const double4 pj = pos[j], fj = frc[j];
        const V3<double> f = { fj.x, fj.y, fj.z };
#pragma unroll
        for (int a = 0; a < ILP; ++a) {
            V3<double> d = { x[a].x - pj.x, x[a].y - pj.y, x[a].z - pj.z };
            if (PER) {   // nearest image; an exact half-box difference may take either image
                d.x = fma(-pc.box, rint(d.x * pc.ibox), d.x);
                d.y = fma(-pc.box, rint(d.y * pc.ibox), d.y);
                d.z = fma(-pc.box, rint(d.z * pc.ibox), d.z);
            }
            const double r2 = dot(d, d);
            double A, Bt;
            far_coef<TENSOR>(rsqrt_f64(r2), gamma, m3g, A, Bt);
            const bool rare = r2 < thr2 || r2 > 1e300;
            if (__builtin_amdgcn_ballot_w64(rare) != 0) {   // near or self pair
                const int i = i0 + a;
                if (r2 < thr2) {
                    int cls = PREMISE_OK;
                    A = Bt = 0.0;
                    if (i < n && i != j) cls = near_coef<TENSOR>(pc, r2, A, Bt);
                    count_premise(premise, i < j ? cls : (int)PREMISE_OK);
                } else if (r2 == __builtin_inf()) {   // r^2 overflowed: 1 / r = 0
                    A = Bt = 0.0;
                }
            }
            const double sB = Bt * dot(d, f);
            acc[3 * a] = fma(A, f.x, fma(sB, d.x, acc[3 * a]));
            acc[3 * a + 1] = fma(A, f.y, fma(sB, d.y, acc[3 * a + 1]));
            acc[3 * a + 2] = fma(A, f.z, fma(sB, d.z, acc[3 * a + 2]));
        }
    }
#pragma unroll
    for (int k = 0; k < 3 * ILP; ++k) acc[k] *= pc.alpha;
    group_sum<3 * ILP>(s_sum, acc);
    if (tid < ILP && i0 + tid < n) row_finish(out, i0 + tid, frc[i0 + tid], s_sum + 3 * tid);
}

hipError_t launch_row(const PairLaunch& L, bool f64, int tensor, const void* pos, const void* frc,
                      const double* x64, int n, const PairConst& pc, double* vel,
                      const double* x_in, double* x_out, double* v_prev, double* v_out, double dt,
                      int mode, void* pos_next, hipStream_t st)
{
    RowOut o;
    o.vel = vel;
    o.x_in = x_in;
    o.x_out = x_out;
    o.v_prev = v_prev;
    o.v_out = v_out;
    o.pos_next = pos_next;
    o.dt = dt;
    o.mu0 = pc.mu0;
    o.qs = pc.box > 0.0 && !f64 ? 4294967296.0 / pc.box : 0.0;
    o.mode = mode;
    unsigned long long* premise = nullptr;
    if (const hipError_t e = premise_counters(&premise); e != hipSuccess) return e;
    const dim3 grid((unsigned)((n + L.ilp - 1) / L.ilp)), block(256);
    const bool per = pc.box > 0.0;
#define SD_GO(T, P, I)                                                                          \
    do {                                                                                        \
        if (f64)                                                                                \
            hipLaunchKernelGGL((k_row_f64<T, P, I>), grid, block, 0, st, (const double4*)pos,   \
                               (const double4*)frc, n, pc, o, premise);                         \
        else                                                                                    \
            hipLaunchKernelGGL((k_row_f32<T, P, I>), grid, block, 0, st, (const float4*)pos,    \
                               (const float4*)frc, x64, n, pc, o, premise);                     \
    } while (0)
#define SD_ILP(T, P)                                                                            \
    do {                                                                                        \
        if (L.ilp == 2) SD_GO(T, P, 2); else SD_GO(T, P, 1);                                    \
    } while (0)
    if (tensor == T_OSEEN) {
        if (per) SD_ILP(T_OSEEN, true); else SD_ILP(T_OSEEN, false);
    } else {
        if (per) SD_ILP(T_RPY, true); else SD_ILP(T_RPY, false);
    }
#undef SD_ILP
#undef SD_GO
    return hipGetLastError();
}

}  // namespace sd
