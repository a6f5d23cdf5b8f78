// wave_adjoint.hip -- the adjoint of the product with each pair of particles
// evaluated once (wave-symmetric schedule, wave_sym.h).  For a pair with
// d = x_i - x_j the gradient of lam . M(x) F with respect to x_i and to x_j is
// G and -G (the definitions are in adjoint.hip), and M(x) lam takes T lam_j on
// the i side and T lam_i on the j side: both sides share the coefficients, the
// projections and G itself.
#include "pair_terms.h"
#include "sd_internal.h"
#include "wave_sym.h"

namespace sd {

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
    typedef float4 type;
};
template <>
struct Vec4<double> {
    typedef double4 type;
};

// Coefficients of a pair, scaled by 1 / alpha: T = A I + Bt d d, P = A' / r,
// Q = Bt' / r (derivatives in r).
template <typename T>
struct AdjCoef {
    T A, Bt, P, Q;
};

template <int TENSOR, typename T>
__device__ __forceinline__ AdjCoef<T> adj_far(T rinv, T gamma, T g3, T g15)
{
    AdjCoef<T> c;
    const T rinv2 = rinv * rinv, rinv3 = rinv2 * rinv, rinv5 = rinv3 * rinv2;
    if (TENSOR == T_OSEEN) {
        c.A = rinv;
        c.Bt = rinv3;
        c.P = -rinv3;
        c.Q = (T)-3 * rinv5;
    } else {
        c.A = fma(gamma, rinv3, rinv);
        c.Bt = fma(-g3, rinv5, rinv3);
        c.P = -fma(g3, rinv5, rinv3);
        c.Q = rinv5 * fma(g15, rinv2, (T)-3);
    }
    return c;
}

// The same in FP64 for a near pair (r^2 below the threshold).  Coincident
// spheres have no gradient (a measure-zero set); T there is the r -> 0 limit
// of the overlap form, or nothing.
template <int TENSOR>
__device__ __forceinline__ AdjCoef<double> adj_near_coef(const PairConst& pc, double r2)
{
    const double ialpha = 1.0 / pc.alpha;
    AdjCoef<double> c = { 0.0, 0.0, 0.0, 0.0 };
    if (r2 == 0.0) {
        if (TENSOR == T_RPY && pc.overlap) c.A = pc.mu0 * ialpha;
        return c;
    }
    const double r = sqrt(r2), ri = 1.0 / r, ri2 = ri * ri, ri3 = ri2 * ri;
    if (TENSOR == T_OSEEN) {
        c.A = ri;
        c.Bt = ri3;
        c.P = -ri3;
        c.Q = -3.0 * ri3 * ri2;
    } else if (pc.overlap && r < 2.0 * pc.a) {
        const double m = pc.mu0 * ialpha;
        c.A = m * (1.0 - 9.0 * r / (32.0 * pc.a));
        c.Bt = m * 3.0 / (32.0 * pc.a) * ri;
        c.P = -m * 9.0 / (32.0 * pc.a) * ri;
        c.Q = -m * 3.0 / (32.0 * pc.a) * ri3;
    } else {
        c.A = ri + pc.gamma * ri3;
        c.Bt = ri3 * (1.0 - 3.0 * pc.gamma * ri2);
        c.P = -ri3 * (1.0 + 3.0 * pc.gamma * ri2);
        c.Q = ri3 * ri2 * (15.0 * pc.gamma * ri2 - 3.0);
    }
    return c;
}

// One pair: G to g and cg, T lam_j to m, T lam_i to cm (the terms of j; first:
// cg and cm are started; start: g and m are started).  FINE: G is rounded into g
// without a rounding of its own.
template <typename T, bool FINE = false>
__device__ __forceinline__ void adj_pair(const AdjCoef<T>& c, const V3<T>& d, const V3<T>& fi,
                                         const V3<T>& li, const V3<T>& fj, const V3<T>& lj,
                                         V3<T>& g, V3<T>& m, V3<T>& cg, V3<T>& cm, bool first,
                                         bool start)
{
    const T uw = fma(li.x, fj.x, fma(li.y, fj.y, fma(li.z, fj.z,
                     fma(lj.x, fi.x, fma(lj.y, fi.y, lj.z * fi.z)))));
    const T li_d = dot(li, d), fj_d = dot(fj, d), lj_d = dot(lj, d), fi_d = dot(fi, d);
    const T c1 = fma(c.P, uw, c.Q * fma(li_d, fj_d, lj_d * fi_d));
    const T bli = c.Bt * li_d, bfj = c.Bt * fj_d, blj = c.Bt * lj_d, bfi = c.Bt * fi_d;
#define SD_COMP(k)                                                                              \
    do {                                                                                        \
        const T W = fma(fj_d, li.k, fma(li_d, fj.k, fma(fi_d, lj.k, lj_d * fi.k)));             \
        const T G = FINE ? fma(c1, d.k, c.Bt * W)                                               \
                         : fma(c1, d.k, fma(bfj, li.k, fma(bli, fj.k, fma(bfi, lj.k, blj * fi.k)))); \
        if (FINE) g.k = fma(c1, d.k, fma(c.Bt, W, g.k));                                        \
        else g.k = start ? G : g.k + G;                                                         \
        m.k = fma(c.A, lj.k, start ? blj * d.k : fma(blj, d.k, m.k));                           \
        cg.k = first ? G : cg.k + G;                                                            \
        cm.k = fma(c.A, li.k, first ? bli * d.k : fma(bli, d.k, cm.k));                         \
    } while (0)
    SD_COMP(x);
    SD_COMP(y);
    SD_COMP(z);
#undef SD_COMP
}

// partial: FP64 split rows of six components (position gradient, M lam), the
// diagonal row last; jpart[c][I][p]: FP64 j-side partials; both scaled by
// 1 / alpha.  T float: terms in FP32; the i side in blocks of IB terms, added
// in FP32 and compensated (Kahan) once per IK terms; the j side of a lane's
// chunk in blocks of JB steps, two of those added in FP32, and in FP64 from
// there on.  (The blocks keep the partial sums that each term is rounded into
// small: one level of 16 terms had an error of 1.1e-7 in M lam where the
// one-sided kernel's blocks of four had 0.8e-7.)  Near pairs in FP64 from x64
// (may be null: the records) in either precision.
//
// Bound by the vector ALU: N = 8192 issues 99 vector instructions per unordered pair
// in FP32, one per 3.4 cycles and SIMD, and in FP64 111, 84 of them FP64, one per 4.3,
// at a clock of 1.9 GHz.
// One particle per lane: six sums on each side and nine values of i and j fill
// the registers (two per lane spilled and gained nothing).  Three waves per
// SIMD: the bound of four spilled 40 registers and was 3 % slower in FP64, 4 %
// faster in FP32 at N = 8192 and 7 % slower there at N = 3001.  Microseconds
// per pass with the fold (one-sided kernel and merge): FP64 N = 3001 29 (134),
// FP32 N = 8192 86 (131).
// FINE (FP32, small n): the i side compensated with every term, the j side in
// blocks of two.
template <int TENSOR, typename T, bool FINE>
__global__ void __launch_bounds__(256, FINE ? 2 : 3)
k_wave_adjoint(const typename Vec4<T>::type* __restrict__ pos,
               const typename Vec4<T>::type* __restrict__ frc,
               const typename Vec4<T>::type* __restrict__ lam, const double* __restrict__ x64,
               int n, WaveShape sh, PairConst pc, double* __restrict__ partial,
               double* __restrict__ jpart)
{
    typedef typename Vec4<T>::type V4;
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int ILP = 1, B = 64 * ILP;
    // FP32 summation blocks
    constexpr int IB = 2, IK = 4, JB = FINE ? 1 : 4;
    constexpr int JH = F32 ? 8 / JB : 1;    // j-side sums per chunk, row and element
    constexpr int RS = F32 ? 12 : 10;   // values per staged record (16-byte multiples)
    __shared__ __align__(16) T s_rec[4][32 * RS];
    __shared__ T s_j[4][4 * JH * 96];
    __shared__ double s_i[4][6 * B];
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
    const T far = (T)1.0e15;
    const V3<T> zero = { (T)0, (T)0, (T)0 };
    V3<T> x[ILP], f[ILP], l[ILP], g[ILP], m[ILP];
    // FP32: sums, -compensations and the terms since the last compensated add
    V3<T> gs[ILP], ms[ILP], gc[ILP], mc[ILP], yg[ILP], ym[ILP];
#pragma unroll
    for (int a = 0; a < ILP; ++a) {
        const int i = ib * B + a * 64 + lane;
        x[a] = { -far, -far, -far };
        f[a] = l[a] = g[a] = m[a] = zero;
        gs[a] = ms[a] = gc[a] = mc[a] = yg[a] = ym[a] = zero;
        if (i < n) {
            const V4 p = pos[i], v = frc[i], u = lam[i];
            x[a] = { p.x, p.y, p.z };
            f[a] = { v.x, v.y, v.z };
            l[a] = { u.x, u.y, u.z };
        }
        // this lane's FP64 sums (near pairs first, the chunk sums at the end)
#pragma unroll
        for (int c = 0; c < 6; ++c) s_i[w][c * B + a * 64 + lane] = 0.0;
    }
    T gamma = F32 ? (T)pc.gamma_f : (T)pc.gamma, thr2 = F32 ? (T)pc.thr2_f : (T)pc.thr2_d;
    T g3 = (T)3 * gamma, g15 = (T)15 * gamma;
    // constants in VGPRs (an FP32 instruction with an SGPR operand issues at
    // half rate)
    if (F32) asm volatile("" : "+v"(gamma), "+v"(g3), "+v"(g15), "+v"(thr2));
    auto chunk_start = [&](int p) {
        return diag ? ib * B + p : ((ib + 1 + p / B) % sh.nb) * B + p % B;
    };
    const V4* src = pos;
    if (row == 1) src = frc;
    if (row == 2) src = lam;
    const T fill = row == 0 ? far : (T)0;
    // rows 0, 1, 2 of the wave load the positions, forces, cotangents of a chunk
    auto load = [&](int p) {
        const int j = chunk_start(p) + q;
        V4 r;
        r.x = r.y = r.z = fill;
        r.w = (T)0;
        if (row < 3 && j < n) r = src[j];
        return r;
    };
    T* const rec = s_rec[w];
    V4 nxt;
    nxt.x = nxt.y = nxt.z = nxt.w = (T)0;
    if (pbeg < pend) nxt = load(pbeg);
#pragma unroll 1
    for (int p = pbeg; p < pend; p += 16) {
        wave_lds_fence();
        if (row < 3) {
            T* d = rec + q * RS + row * 3;
            d[0] = d[16 * RS] = nxt.x;
            d[1] = d[16 * RS + 1] = nxt.y;
            d[2] = d[16 * RS + 2] = nxt.z;
        }
        wave_lds_fence();
        if (p + 16 < pend) nxt = load(p + 16);
        const V4* const view = (const V4*)(rec + q * RS);
        const double2* const view2 = (const double2*)(rec + q * RS);
        V3<T> ag = zero, am = zero, bg = zero, bm = zero;
        uint32_t nearm = 0;   // bit k ILP + a: the pair of step k and particle a is near
        WaveFor<0, 16>::run([&](auto k_c) {
            constexpr int k = decltype(k_c)::value;
            __builtin_amdgcn_sched_barrier(0);   // one step's pair data live at a time
            V3<T> xj, fj, lj;
            if constexpr (F32) {
                const V4 r0 = view[3 * k], r1 = view[3 * k + 1], r2v = view[3 * k + 2];
                xj = { r0.x, r0.y, r0.z };
                fj = { r0.w, r1.x, r1.y };
                lj = { r1.z, r1.w, r2v.x };
            } else {
                const double2 r0 = view2[5 * k], r1 = view2[5 * k + 1], r2v = view2[5 * k + 2],
                              r3 = view2[5 * k + 3];
                xj = { r0.x, r0.y, r1.x };
                fj = { r1.y, r2v.x, r2v.y };
                lj = { r3.x, r3.y, rec[(q + k) * RS + 8] };
            }
            V3<T> d[ILP];
            T r2[ILP];
            bool nr = false;
#pragma unroll
            for (int a = 0; a < ILP; ++a) {
                d[a] = { x[a].x - xj.x, x[a].y - xj.y, x[a].z - xj.z };
                r2[a] = dot(d[a], d[a]);
                nr = nr || r2[a] < thr2 || (!F32 && r2[a] > (T)1e300);
            }
            if (__builtin_amdgcn_ballot_w64(nr) != 0) {   // rare
#pragma unroll
                for (int a = 0; a < ILP; ++a) {
                    // near pairs: after the steps, from 1 / r = 0 here; an
                    // overflowed r^2 has 1 / r = 0 too
                    const bool none = r2[a] < thr2;
                    nearm |= none ? 1u << (k * ILP + a) : 0u;
                    if constexpr (F32)
                        r2[a] = none ? (T)__builtin_inff() : r2[a];
                    else
                        r2[a] = (none || r2[a] == __builtin_inf()) ? 1e300 : r2[a];
                }
            }
            V3<T> cg = zero, cm = zero;
#pragma unroll
            for (int a = 0; a < ILP; ++a) {
                T rinv;
                if constexpr (F32) {
                    rinv = __builtin_amdgcn_rsqf(r2[a]);
                } else {
                    rinv = rsqrt_f64(r2[a]);
                }
                const AdjCoef<T> co = adj_far<TENSOR, T>(rinv, gamma, g3, g15);
                if constexpr (FINE) {   // compensated with every term
                    g[a] = gc[a];
                    m[a] = mc[a];
                }
                adj_pair<T, FINE>(co, d[a], f[a], l[a], fj, lj, g[a], m[a], cg, cm, a == 0,
                                  F32 && !FINE && k % IB == 0);
                if constexpr (FINE) {
                    kahan(gs[a], gc[a], g[a]);
                    kahan(ms[a], mc[a], m[a]);
                }
            }
            // hand-over to the owner of the element; FP32: JB steps, then the sum
            if constexpr (F32 && k % JB == 0) {
                bg = { -row_rot<k>(cg.x), -row_rot<k>(cg.y), -row_rot<k>(cg.z) };
                bm = { row_rot<k>(cm.x), row_rot<k>(cm.y), row_rot<k>(cm.z) };
            } else {
                V3<T>& hg = F32 ? bg : ag;
                V3<T>& hm = F32 ? bm : am;
                hg = { hg.x - row_rot<k>(cg.x), hg.y - row_rot<k>(cg.y), hg.z - row_rot<k>(cg.z) };
                hm = { hm.x + row_rot<k>(cm.x), hm.y + row_rot<k>(cm.y), hm.z + row_rot<k>(cm.z) };
            }
            if constexpr (F32 && k % (2 * JB) == JB - 1) {
                ag = bg;
                am = bm;
            } else if constexpr (F32 && k % (2 * JB) == 2 * JB - 1) {
                ag = add(ag, bg);
                am = add(am, bm);
            }
            if constexpr (k % (16 / JH) == 16 / JH - 1) {   // to this row's slots
                T* const sr = s_j[w] + ((k / (16 / JH)) * 4 + row) * 96 + q;
                sr[0] = ag.x;
                sr[16] = ag.y;
                sr[32] = ag.z;
                sr[48] = am.x;
                sr[64] = am.y;
                sr[80] = am.z;
            }
            // FP32, i side: blocks of IB terms into the running sum, compensated
            // once per IK terms
            if constexpr (F32 && !FINE && k % IB == IB - 1) {
#pragma unroll
                for (int a = 0; a < ILP; ++a) {
                    yg[a] = add(k % IK == IB - 1 ? gc[a] : yg[a], g[a]);
                    ym[a] = add(k % IK == IB - 1 ? mc[a] : ym[a], m[a]);
                    if constexpr (k % IK == IK - 1) {
                        kahan(gs[a], gc[a], yg[a]);
                        kahan(ms[a], mc[a], ym[a]);
                    }
                }
            }
            // the sums are materialised here, or their chains sink to the end
            // of the chunk with the terms of every step live
            keep(F32 ? bg : ag);
            keep(F32 ? bm : am);
            if (F32) {
                keep(ag);
                keep(am);
            }
#pragma unroll
            for (int a = 0; a < ILP; ++a) {
                if (F32) {
                    keep(gs[a]);
                    keep(gc[a]);
                    keep(yg[a]);
                    keep(ms[a]);
                    keep(mc[a]);
                    keep(ym[a]);
                }
                keep(g[a]);
                keep(m[a]);
            }
        });
        V3<double> njg = { 0.0, 0.0, 0.0 }, njm = njg;   // near pairs, j side of element q
        const bool near = __builtin_amdgcn_ballot_w64(nearm != 0) != 0;
        if (near) {   // rare: the chunk's near pairs, in FP64, from memory
#pragma unroll 1
            for (int b = 0; b < 16 * ILP; ++b) {
                const bool mine = (nearm >> b) & 1u;
                if (__builtin_amdgcn_ballot_w64(mine) == 0) continue;
                const int k = b / ILP, a = b % ILP;
                const int jg = chunk_start(p) + ((q + k) & 15);
                const int i = ib * B + a * 64 + lane;
                V3<double> cg = { 0.0, 0.0, 0.0 }, cm = cg;
                if (mine && i < n && jg < n && i != jg) {
                    const T* r = rec + (q + k) * RS;
                    double* const own = &s_i[w][a * 64 + lane];
                    const V4 pi = pos[i], fv = frc[i], lv = lam[i];
                    V3<double> d = { (double)pi.x - (double)r[0], (double)pi.y - (double)r[1],
                                     (double)pi.z - (double)r[2] };
                    if (x64)
                        d = { x64[3 * (size_t)i] - x64[3 * (size_t)jg],
                              x64[3 * (size_t)i + 1] - x64[3 * (size_t)jg + 1],
                              x64[3 * (size_t)i + 2] - x64[3 * (size_t)jg + 2] };
                    const V3<double> fi = { (double)fv.x, (double)fv.y, (double)fv.z };
                    const V3<double> li = { (double)lv.x, (double)lv.y, (double)lv.z };
                    const V3<double> fj = { (double)r[3], (double)r[4], (double)r[5] };
                    const V3<double> lj = { (double)r[6], (double)r[7], (double)r[8] };
                    V3<double> gn, mn;
                    adj_pair<double>(adj_near_coef<TENSOR>(pc, dot(d, d)), d, fi, li, fj, lj, gn,
                                     mn, cg, cm, true, true);
                    own[0] += gn.x;
                    own[B] += gn.y;
                    own[2 * B] += gn.z;
                    own[3 * B] += mn.x;
                    own[4 * B] += mn.y;
                    own[5 * B] += mn.z;
                }
                const int from = (lane & 48) | ((q - k) & 15);
                njg.x -= __shfl(cg.x, from);
                njg.y -= __shfl(cg.y, from);
                njg.z -= __shfl(cg.z, from);
                njm.x += __shfl(cm.x, from);
                njm.y += __shfl(cm.y, from);
                njm.z += __shfl(cm.z, from);
            }
            // over the rows of the wave
#define SD_COMP(v)                                                                              \
    do {                                                                                        \
        v += __shfl_xor(v, 16);                                                                 \
        v += __shfl_xor(v, 32);                                                                 \
    } while (0)
            SD_COMP(njg.x);
            SD_COMP(njg.y);
            SD_COMP(njg.z);
            SD_COMP(njm.x);
            SD_COMP(njm.y);
            SD_COMP(njm.z);
#undef SD_COMP
        }
        if (!diag) {
            // the sums of the four rows, added in FP64 in a fixed order
            const T* const sj = s_j[w];
            wave_lds_fence();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int t = lane + 64 * u;   // component t / 16 of element q
                if (t < 96) {
                    double sum = (double)sj[t];
#pragma unroll
                    for (int r = 1; r < 4 * JH; ++r) sum += (double)sj[r * 96 + t];
                    if (near) {   // this lane's component: row + 4 u
                        if (u == 0)
                            sum += row == 0 ? njg.x : row == 1 ? njg.y : row == 2 ? njg.z : njm.x;
                        else
                            sum += row == 0 ? njm.y : njm.z;
                    }
                    jpart[((size_t)(t >> 4) * sh.nb + ib) * (size_t)sh.lmax + (size_t)(p + q)] = sum;
                }
            }
        }
    }
#pragma unroll
    for (int a = 0; a < ILP; ++a) {
        double* const own = &s_i[w][a * 64 + lane];
        own[0] += F32 ? (double)gs[a].x + (double)gc[a].x : (double)g[a].x;
        own[B] += F32 ? (double)gs[a].y + (double)gc[a].y : (double)g[a].y;
        own[2 * B] += F32 ? (double)gs[a].z + (double)gc[a].z : (double)g[a].z;
        own[3 * B] += F32 ? (double)ms[a].x + (double)mc[a].x : (double)m[a].x;
        own[4 * B] += F32 ? (double)ms[a].y + (double)mc[a].y : (double)m[a].y;
        own[5 * B] += F32 ? (double)ms[a].z + (double)mc[a].z : (double)m[a].z;
    }
    __syncthreads();
    for (int t = tid; t < 6 * B; t += 256) {
        const int c = t / B, i = ib * B + t % B;
        if (i < n)
            partial[((size_t)s * 6 + c) * (size_t)n + i] =
                ((s_i[0][t] + s_i[1][t]) + s_i[2][t]) + s_i[3][t];
    }
}

// Sums of a particle's partials (as k_wave_fold in wave_fold.hip, six components),
// then the end of the pass (as k_adjoint_merge):
//   single product (lam64 null): gpos = alpha P; gforce = mu0 lam + alpha F
//   Euler loop: gforce += dt (mu0 lam + alpha F); lam64 += dt alpha P, and the
//   record of the new lam for the next step.
template <typename V4>
__global__ void __launch_bounds__(256)
k_wave_adjoint_fold(const double* __restrict__ partial, const double* __restrict__ jpart, int n,
                    int B, WaveShape sh, double alpha, V4* __restrict__ lam4,
                    double* __restrict__ lam64, double mu0, double dt, double* __restrict__ gpos,
                    double* __restrict__ gforce)
{
    __shared__ double s_sum[8][6][32];
    const int t = threadIdx.x & 31, sl = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + t;
    double v[6] = { 0.0, 0.0, 0.0, 0.0, 0.0, 0.0 };
    if (i < n) {
        const int J = i / B, o = i - J * B;
        const int half = sh.nb >> 1;
        const size_t cs = (size_t)sh.nb * (size_t)sh.lmax;
        const int Ie = J >= half ? J - half : J + half;
        const int nd = sh.h + ((sh.extra && Ie < half) ? 1 : 0);
        constexpr int G = 4;
        for (int d0 = sl; d0 < nd; d0 += 8 * G) {
            double g[G][6];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int d = d0 + 8 * u;   // block I = J - d - 1 (mod nb)
                if (d < nd) {
                    int I = J - d - 1;
                    if (I < 0) I += sh.nb;
                    const double* at = jpart + (size_t)I * sh.lmax + (size_t)d * B + o;
#pragma unroll
                    for (int c = 0; c < 6; ++c) g[u][c] = at[c * cs];
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (d0 + 8 * u < nd)
                    for (int c = 0; c < 6; ++c) v[c] += g[u][c];
        }
        const int rows = sh.splits + 1;
        for (int r0 = sl; r0 < rows; r0 += 8 * G) {
            double g[G][6];
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (r0 + 8 * u < rows) {
                    const double* at = partial + (size_t)(r0 + 8 * u) * 6 * (size_t)n + i;
#pragma unroll
                    for (int c = 0; c < 6; ++c) g[u][c] = at[c * (size_t)n];
                }
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (r0 + 8 * u < rows)
                    for (int c = 0; c < 6; ++c) v[c] += g[u][c];
        }
    }
    for (int c = 0; c < 6; ++c) s_sum[sl][c][t] = v[c];
    __syncthreads();
    if (sl != 0 || i >= n) return;
    for (int c = 0; c < 6; ++c) {
        double a = 0.0;
        for (int k = 0; k < 8; ++k) a += s_sum[k][c][t];
        v[c] = alpha * a;
    }
    if (lam64) {
        double ln[3];
        for (int c = 0; c < 3; ++c) {
            const size_t e = 3 * (size_t)i + c;
            const double lo = lam64[e];
            gforce[e] += dt * (mu0 * lo + v[3 + c]);
            ln[c] = lo + dt * v[c];
            lam64[e] = ln[c];
        }
        V4 r;
        r.x = ln[0];
        r.y = ln[1];
        r.z = ln[2];
        r.w = 0;
        lam4[i] = r;
    } else {
        const V4 r = lam4[i];
        const double lv[3] = { (double)r.x, (double)r.y, (double)r.z };
        for (int c = 0; c < 3; ++c) {
            const size_t e = 3 * (size_t)i + c;
            if (gpos) gpos[e] = v[c];
            if (gforce) gforce[e] = mu0 * lv[c] + v[3 + c];
        }
    }
}

size_t wave_adjoint_bytes(const PairLaunch& L, int64_t n)
{
    const WaveShape sh = wave_shape_of(L, (int)n);
    return 2 * (wave_jpart_offset(sh, n) + wave_jpart_bytes(sh, sizeof(double)));
}

// FP32 passes below this size compensate with every term.  The one-sided kernel
// cut a short row into many FP64 parts, and in blocks the error of M lam was 1.2
// times its at N = 20 (48 1.1, 120 1.1, 700 and above 1.0); with every term 1.0, 1.0,
// 0.95.  Microseconds, blocks / every term: N = 300 11.4 / 12.1, 1000 12.0 / 12.5,
// 1500 13.3 / 15.0, 3000 23.4 / 30.0.
constexpr int FINE_END_N = 1024;

template <int TENSOR, typename T>
static hipError_t launch_t(const PairLaunch& L, const void* pos, const void* frc, void* lam,
                           const double* x64, int n, const PairConst& pc, void* ws, double* lam64,
                           double dt, double* gpos, double* gforce, hipStream_t st)
{
    typedef typename Vec4<T>::type V4;
    const WaveShape sh = wave_shape_of(L, n);
    double* partial = (double*)ws;
    double* jpart = (double*)((char*)ws + 2 * wave_jpart_offset(sh, n));
    const dim3 grid((unsigned)(sh.nb * (sh.splits + 1)));
    if (sizeof(T) == 4 && n < FINE_END_N)
        hipLaunchKernelGGL((k_wave_adjoint<TENSOR, T, sizeof(T) == 4>), grid, dim3(256), 0, st,
                           (const V4*)pos, (const V4*)frc, (const V4*)lam, x64, n, sh, pc,
                           partial, jpart);
    else
        hipLaunchKernelGGL((k_wave_adjoint<TENSOR, T, false>), grid, dim3(256), 0, st,
                           (const V4*)pos, (const V4*)frc, (const V4*)lam, x64, n, sh, pc,
                           partial, jpart);
    hipLaunchKernelGGL((k_wave_adjoint_fold<V4>), dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st,
                       partial, jpart, n, 64, sh, pc.alpha, (V4*)lam, lam64, pc.mu0, dt, gpos,
                       gforce);
    return hipGetLastError();
}

hipError_t launch_wave_adjoint(const PairLaunch& L, int tensor, bool f64, const void* pos,
                               const void* frc, void* lam, const double* x64, int n,
                               const PairConst& pc, void* ws, double* lam64, double dt,
                               double* gpos, double* gforce, hipStream_t st)
{
#define SD_GO(T)                                                                                \
    return tensor == T_OSEEN ? launch_t<T_OSEEN, T>(L, pos, frc, lam, x64, n, pc, ws, lam64, dt, \
                                                    gpos, gforce, st)                           \
                             : launch_t<T_RPY, T>(L, pos, frc, lam, x64, n, pc, ws, lam64, dt,  \
                                                  gpos, gforce, st)
    if (f64) SD_GO(double);
    SD_GO(float);
#undef SD_GO
}

}  // namespace sd
