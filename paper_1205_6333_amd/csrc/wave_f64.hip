// wave_f64.hip -- the FP64 product v = M(x) F with each pair of particles
// evaluated once (wave-symmetric schedule, wave_sym.h).
#include "pair_terms.h"
#include "premise.h"
#include "sd_internal.h"
#include "wave_sym.h"

namespace sd {

#define SD_FAR_I (-1.0e15)
#define SD_FAR_J (1.0e15)

// One particle i of a lane.
struct WaveI64 {
    double x, y, z, fx, fy, fz, s0, s1, s2;
};

__device__ __forceinline__ uint32_t high_word(double v)
{
    return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32);
}

// One pair: T F_j to the sums of i, T F_i to the term c for j (first: c is
// started).
__device__ __forceinline__ void pair_sums(WaveI64& L, double A, double Bt, double dx, double dy,
                                          double dz, double fx, double fy, double fz, bool first,
                                          double& c0, double& c1, double& c2)
{
    const double sj = Bt * fma(dx, fx, fma(dy, fy, dz * fz));
    const double si = Bt * fma(dx, L.fx, fma(dy, L.fy, dz * L.fz));
    L.s0 = fma(A, fx, fma(sj, dx, L.s0));
    L.s1 = fma(A, fy, fma(sj, dy, L.s1));
    L.s2 = fma(A, fz, fma(sj, dz, L.s2));
    c0 = fma(A, L.fx, first ? si * dx : fma(si, dx, c0));
    c1 = fma(A, L.fy, first ? si * dy : fma(si, dy, c1));
    c2 = fma(A, L.fz, first ? si * dz : fma(si, dz, c2));
}

// partial: FP64 split rows (isplits, then the diagonal row); jpart[c][I][p]:
// FP64 j-side partials.
//
// Bound by the FP64 vector ALU: N = 16384 issues 45 vector instructions per unordered
// pair (two interactions), 39 of them FP64 (one v_rsq_f64, and per two pairs the
// hand-over of three sums), one per 4.4 cycles and SIMD at clocks of 1.9 to 2.1 GHz;
// the one-sided kernel spends as much on one interaction.  N =
// 16384: 200 us per product with the fold (1.34 T interactions/s), one-sided
// kernel and merge 301 us.  Near pairs only set a bit in the hot loop and are
// evaluated after the chunk's steps: inlined in every step the branch took all
// 256 registers.
template <int TENSOR, bool PER>
__global__ void __launch_bounds__(256)
k_wave_f64(const double4* __restrict__ pos, const double4* __restrict__ frc, int n, WaveShape sh,
           PairConst pc, double* __restrict__ partial, double* __restrict__ jpart,
           unsigned long long* __restrict__ premise)
{
    constexpr int ILP = 2, B = 64 * ILP;
    __shared__ __align__(16) double s_rec[4][32 * 6];
    __shared__ double s_j[4][4 * 48];
    __shared__ double s_i[4][3 * B];
    const int tid = threadIdx.x;
    const int lane = tid & 63, q = lane & 15, row = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool diag = (int)blockIdx.x < sh.nb;
    int ib, s;
    if (diag) {
        ib = (int)blockIdx.x;
        s = sh.splits;
    } else {
        const int u = (int)blockIdx.x - sh.nb;
        s = u / sh.nb;
        ib = u - s * sh.nb;
    }
    int pbeg, pend;
    wave_range<B>(sh, diag, ib, s, w, pbeg, pend);
    WaveI64 L[ILP];
#pragma unroll
    for (int l = 0; l < ILP; ++l) {
        const int i = ib * B + l * 64 + lane;
        double4 p = make_double4(PER ? 0.0 : SD_FAR_I, PER ? 0.0 : SD_FAR_I, PER ? 0.0 : SD_FAR_I, 0.0);
        double4 f = make_double4(0.0, 0.0, 0.0, 0.0);
        if (i < n) {
            p = pos[i];
            f = frc[i];
        }
        L[l] = { p.x, p.y, p.z, f.x, f.y, f.z, 0.0, 0.0, 0.0 };
    }
    const double gamma = pc.gamma, m3g = -3.0 * pc.gamma, thr2 = pc.thr2_d;
    // r^2 outside (thr2, about 1e300), by its high word (one integer subtract
    // and a maximum for the pairs of a step): such a pair takes the rare branch
    const uint32_t hi_lo = high_word(thr2) + 1, hi_span = 0x7e37e43cu - hi_lo;
    auto diff = [&](const WaveI64& P, double x, double y, double z, double& dx, double& dy,
                    double& dz) {
        dx = P.x - x;
        dy = P.y - y;
        dz = P.z - z;
        if (PER) {   // nearest image; an exact half-box difference may take either image
            dx = fma(-pc.box, rint(dx * pc.ibox), dx);
            dy = fma(-pc.box, rint(dy * pc.ibox), dy);
            dz = fma(-pc.box, rint(dz * pc.ibox), dz);
        }
    };
    // first particle of the chunk at virtual position p
    auto chunk_start = [&](int p) {
        return diag ? ib * B + p : ((ib + 1 + p / B) % sh.nb) * B + p % B;
    };
    // row 0 loads the positions of a chunk, row 1 the forces
    const double4* const src = row == 0 ? pos : frc;
    const double fill = (row == 0 && !PER) ? SD_FAR_J : 0.0;
    auto load = [&](int p) {
        const int j = chunk_start(p) + q;
        double4 r = make_double4(fill, fill, fill, 0.0);
        if (row < 2 && j < n) r = src[j];
        return r;
    };
    double* const rec = s_rec[w];
    double4 nxt = make_double4(0.0, 0.0, 0.0, 0.0);
    if (pbeg < pend) nxt = load(pbeg);
#pragma unroll 1
    for (int p = pbeg; p < pend; p += 16) {
        wave_lds_fence();
        if (row < 2) {
            double* d = rec + q * 6 + row * 3;
            d[0] = d[16 * 6] = nxt.x;
            d[1] = d[16 * 6 + 1] = nxt.y;
            d[2] = d[16 * 6 + 2] = nxt.z;
        }
        wave_lds_fence();
        if (p + 16 < pend) nxt = load(p + 16);
        const double2* const view = (const double2*)(rec + q * 6);
        double aj0 = 0.0, aj1 = 0.0, aj2 = 0.0;
        uint32_t nearm = 0;   // bit k ILP + l: the pair of step k and particle l is near
        WaveFor<0, 16>::run([&](auto k_c) {
            constexpr int k = decltype(k_c)::value;
            // one step's pair data live at a time
            __builtin_amdgcn_sched_barrier(0);
            const double2 a = view[3 * k], b = view[3 * k + 1], c = view[3 * k + 2];
            const double fx = b.y, fy = c.x, fz = c.y;
            double dx[ILP], dy[ILP], dz[ILP], r2[ILP], A[ILP], Bt[ILP];
            uint32_t odd = 0;
#pragma unroll
            for (int l = 0; l < ILP; ++l) {
                diff(L[l], a.x, a.y, b.x, dx[l], dy[l], dz[l]);
                r2[l] = fma(dx[l], dx[l], fma(dy[l], dy[l], dz[l] * dz[l]));
                odd = max(odd, high_word(r2[l]) - hi_lo);
                far_coef<TENSOR>(rsqrt_f64(r2[l]), gamma, m3g, A[l], Bt[l]);
            }
            if (__builtin_amdgcn_ballot_w64(odd >= hi_span) != 0) {   // rare
#pragma unroll
                for (int l = 0; l < ILP; ++l) {
                    const bool nr = r2[l] < thr2;
                    // near pairs: after the steps; r^2 overflowed: 1 / r = 0
                    const bool none = nr || r2[l] == __builtin_inf();
                    A[l] = none ? 0.0 : A[l];
                    Bt[l] = none ? 0.0 : Bt[l];
                    nearm |= nr ? 1u << (k * ILP + l) : 0u;
                }
            }
            double c0 = 0.0, c1 = 0.0, c2 = 0.0;
#pragma unroll
            for (int l = 0; l < ILP; ++l)
                pair_sums(L[l], A[l], Bt[l], dx[l], dy[l], dz[l], fx, fy, fz, l == 0, c0, c1, c2);
            aj0 += row_rot<k>(c0);
            aj1 += row_rot<k>(c1);
            aj2 += row_rot<k>(c2);
            // the sums are materialised here, or their chains sink to the end
            // of the chunk with the terms of every step live
            asm volatile("" : "+v"(aj0), "+v"(aj1), "+v"(aj2));
#pragma unroll
            for (int l = 0; l < ILP; ++l)
                asm volatile("" : "+v"(L[l].s0), "+v"(L[l].s1), "+v"(L[l].s2));
        });
        if (__builtin_amdgcn_ballot_w64(nearm != 0) != 0) {   // rare: the chunk's near pairs
#pragma unroll 1
            for (int k = 0; k < 16; ++k) {
                const uint32_t bits = (nearm >> (k * ILP)) & ((1u << ILP) - 1u);
                if (__builtin_amdgcn_ballot_w64(bits != 0) == 0) continue;
                const double* r = rec + (q + k) * 6;
                const int jg = chunk_start(p) + ((q + k) & 15);
                double c0 = 0.0, c1 = 0.0, c2 = 0.0;
#pragma unroll
                for (int l = 0; l < ILP; ++l) {
                    const int i = ib * B + l * 64 + lane;
                    int cls = PREMISE_OK;
                    if (((bits >> l) & 1u) && i < n && jg < n && i != jg) {
                        double dx, dy, dz, A, Bt;
                        diff(L[l], r[0], r[1], r[2], dx, dy, dz);
                        cls = near_coef<TENSOR>(pc, fma(dx, dx, fma(dy, dy, dz * dz)), A, Bt);
                        pair_sums(L[l], A, Bt, dx, dy, dz, r[3], r[4], r[5], false, c0, c1, c2);
                    }
                    // the diagonal block meets both orderings of a pair
                    count_premise(premise, !diag || i < jg ? cls : (int)PREMISE_OK);
                }
                const int from = (lane & 48) | ((q - k) & 15);
                aj0 += __shfl(c0, from);
                aj1 += __shfl(c1, from);
                aj2 += __shfl(c2, from);
            }
        }
        if (!diag) {
            // the four rows of the wave, added in row order by one lane per
            // element and component
            double* const sj = s_j[w];
            sj[row * 48 + q] = aj0;
            sj[row * 48 + 16 + q] = aj1;
            sj[row * 48 + 32 + q] = aj2;
            wave_lds_fence();
            if (lane < 48) {
                const double sum = ((sj[lane] + sj[48 + lane]) + sj[96 + lane]) + sj[144 + lane];
                jpart[((size_t)row * sh.nb + ib) * (size_t)sh.lmax + (size_t)(p + q)] =
                    pc.alpha * sum;
            }
        }
    }
#pragma unroll
    for (int l = 0; l < ILP; ++l) {
        s_i[w][(0 * ILP + l) * 64 + lane] = L[l].s0;
        s_i[w][(1 * ILP + l) * 64 + lane] = L[l].s1;
        s_i[w][(2 * ILP + l) * 64 + lane] = L[l].s2;
    }
    __syncthreads();
    for (int t = tid; t < 3 * B; t += 256) {
        const int c = t / B, i = ib * B + t % B;
        if (i < n)
            partial[((size_t)s * 3 + c) * (size_t)n + i] =
                pc.alpha * (((s_i[0][t] + s_i[1][t]) + s_i[2][t]) + s_i[3][t]);
    }
}

hipError_t launch_wave_f64(const PairLaunch& L, int tensor, const double4* pos, const double4* frc,
                           int n, const PairConst& pc, double* partial, hipStream_t st)
{
    const WaveShape sh = wave_shape_of(L, n);
    double* jpart = (double*)((char*)partial + wave_jpart_offset(sh, n));
    unsigned long long* premise = nullptr;
    if (const hipError_t e = premise_counters(&premise); e != hipSuccess) return e;
    const dim3 grid((unsigned)(sh.nb * (sh.splits + 1))), block(256);
    const bool per = pc.box > 0.0;
#define SD_GO(T, P)                                                                          \
    hipLaunchKernelGGL((k_wave_f64<T, P>), grid, block, 0, st, pos, frc, n, sh, pc, partial, \
                       jpart, premise)
    if (tensor == T_OSEEN) {
        if (per) SD_GO(T_OSEEN, true); else SD_GO(T_OSEEN, false);
    } else {
        if (per) SD_GO(T_RPY, true); else SD_GO(T_RPY, false);
    }
#undef SD_GO
    return hipGetLastError();
}

}  // namespace sd
