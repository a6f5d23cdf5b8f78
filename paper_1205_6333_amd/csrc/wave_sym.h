// wave_sym.h -- block schedule and device helpers of the wave-symmetric
// kernels: every unordered pair of particles evaluated once, by waves that
// need no work-group barrier while they walk their pairs.
//
// Block schedule.  Particles are cut into nb blocks of B = 64 ILP (ILP
// particles per lane).  As in the block-symmetric kernel of mobility.hip,
// i-block I takes the blocks I + 1 .. I + h (mod nb), h = (nb - 1) / 2, and,
// when nb is even, block I + nb/2 if I < nb/2: a virtual j range in which
// every unordered pair of distinct blocks appears once.  A work-group of four
// waves owns one i-block and one split of its range;
// all four waves hold the same particles i and each walks its own chunks of
// 16 particles j.  The diagonal blocks are taken one-sided by nb extra
// work-groups, their chunks dealt to the four waves.
//
// Rows of 16 lanes.  A chunk is staged twice in a row in the wave's LDS, so
// that lane q of a 16-lane row reads element (q + k) mod 16 at the constant
// offset k; the j-side term of step k goes to the lane that owns the element
// by a DPP row rotation.  After the 16 steps the four rows of the wave are
// added in row order and stored as the j-side partial of (I, position).  The
// i-side sums of the four waves are added in wave order in FP64 and stored as
// one split row.
//
// Why four waves share an i-block: a wave alone covers 64 ILP x 16 chunks
// pairs, small enough that a few thousand particles occupy every SIMD, and
// the split rows stay as few as the work-groups' ranges.
#pragma once

#include "pair_terms.h"
#include "sd_internal.h"

#include <type_traits>

namespace sd {

// splits: work-groups (and split rows) per i-block, each 64 chunks positions;
// the diagonal row follows them.
struct WaveShape {
    int nb, h, extra, lmax, chunks, splits;
};

// chunks per wave so that a launch has about `waves` waves (at most the whole
// range; n up to 2^30, where the products exceed 32 bits)
inline WaveShape wave_shape(int n, int B, int waves)
{
    WaveShape s;
    s.nb = (n + B - 1) / B;
    s.h = (s.nb - 1) / 2;
    s.extra = (s.nb >= 2 && (s.nb & 1) == 0) ? 1 : 0;
    s.lmax = (s.h + s.extra) * B;
    const int64_t total = (int64_t)s.nb * (s.lmax / 16);
    int64_t c = (total + waves - 1) / waves;
    if (c > s.lmax / 16) c = s.lmax / 16;
    if (c < 1) c = 1;
    s.chunks = (int)c;
    s.splits = (int)((s.lmax + 64 * c - 1) / (64 * c));
    return s;
}
inline WaveShape wave_shape_of(const PairLaunch& L, int n)
{
    return wave_shape(n, 64 * L.ilp, L.jchunk);
}

// Positions [pbeg, pend) of wave w of split s: of the virtual range of i-block
// ib, or (diag) of the block itself.
template <int B>
__device__ __forceinline__ void wave_range(const WaveShape& sh, bool diag, int ib, int s, int w,
                                           int& pbeg, int& pend)
{
    if (diag) {
        pbeg = w * (B / 4);
        pend = pbeg + B / 4;
    } else {
        const int lI = (sh.h + ((sh.extra && ib < (sh.nb >> 1)) ? 1 : 0)) * B;
        pbeg = (s * 4 + w) * 16 * sh.chunks;
        pend = min(lI, pbeg + 16 * sh.chunks);
    }
}

// Workspace: the split rows and the diagonal row (f64[3n] each), then
// (256-byte aligned) the j-side partials, 3 nb lmax values of `elem` bytes.
inline size_t wave_jpart_offset(const WaveShape& s, int64_t n)
{
    return ((size_t)(s.splits + 1) * 3 * (size_t)n * sizeof(double) + 255) & ~(size_t)255;
}
inline size_t wave_jpart_bytes(const WaveShape& s, size_t elem)
{
    return 3 * (size_t)s.nb * (size_t)s.lmax * elem;
}

template <int B, int E>
struct WaveFor {
    template <class F>
    __device__ __forceinline__ static void run(F&& f)
    {
        f(std::integral_constant<int, B>());
        WaveFor<B + 1, E>::run(f);
    }
};
template <int E>
struct WaveFor<E, E> {
    template <class F>
    __device__ __forceinline__ static void run(F&&) {}
};

// value v of lane (lane - K) mod 16 of the same row of 16 lanes
template <int K>
__device__ __forceinline__ float row_rot(float v)
{
    if constexpr (K == 0) return v;
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                         0, __builtin_bit_cast(int, v), 0x120 + K, 0xf, 0xf, true));
}
template <int K>
__device__ __forceinline__ double row_rot(double v)
{
    if constexpr (K == 0) return v;
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x120 + K, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + K, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// 1 / sqrt(x), x finite and > 0: v_rsq_f64 (relative error e of about 2^-24)
// and one third-order step, y (1 + h/2 + 3 h^2/8) with h = 1 - x y^2, which
// leaves O(e^3) and the rounding of the last operations.
__device__ __forceinline__ double rsqrt_f64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double t = x * y;
    const double h = fma(-t, y, 1.0);
    return fma(y * h, fma(h, 0.375, 0.5), y);
}

// Far coefficients A', Bt' of a pair (scaled units, see PairConst).
template <int TENSOR>
__device__ __forceinline__ void far_coef(double rinv, double gamma, double m3g, double& A,
                                         double& Bt)
{
    const double rinv2 = rinv * rinv, rinv3 = rinv2 * rinv;
    if (TENSOR == T_OSEEN) {
        A = rinv;
        Bt = rinv3;
    } else {
        A = fma(gamma, rinv3, rinv);
        Bt = rinv3 * fma(m3g, rinv2, 1.0);
    }
}

// Coefficients of a near pair (r^2 below the threshold), scaled by 1 / alpha,
// from the definitions of near_term; returns its premise class.
template <int TENSOR>
__device__ __forceinline__ int near_coef(const PairConst& pc, double r2, double& A, double& Bt)
{
    const double ialpha = 1.0 / pc.alpha;
    if (r2 == 0.0) {
        A = (TENSOR == T_RPY && pc.overlap) ? pc.mu0 * ialpha : 0.0;
        Bt = 0.0;
        return PREMISE_COINCIDENT;
    }
    const double r = sqrt(r2);
    if (TENSOR == T_OSEEN) {
        A = 1.0 / r;
        Bt = A / r2;
    } else if (pc.overlap && r < 2.0 * pc.a) {
        A = pc.mu0 * ialpha * (1.0 - 9.0 * r / (32.0 * pc.a));
        Bt = pc.mu0 * ialpha * 3.0 / (32.0 * pc.a * r);
    } else {
        const double ri = 1.0 / r, ri2 = ri * ri, ri3 = ri * ri2;
        A = ri + pc.gamma * ri3;
        Bt = ri3 * (1.0 - 3.0 * pc.gamma * ri2);
    }
    return r2 < 4.0 * pc.a * pc.a ? PREMISE_SUB2A : PREMISE_OK;
}

template <typename T>
struct V3 {
    T x, y, z;
};
template <typename T>
__device__ __forceinline__ T dot(const V3<T>& a, const V3<T>& b)
{
    return fma(a.x, b.x, fma(a.y, b.y, a.z * b.z));
}

template <typename T>
__device__ __forceinline__ V3<T> add(const V3<T>& a, const V3<T>& b)
{
    return { a.x + b.x, a.y + b.y, a.z + b.z };
}
template <typename T>
__device__ __forceinline__ void keep(V3<T>& v)
{
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z));
}
// s += y with the rounding error kept: y started from the last -error c
template <typename T>
__device__ __forceinline__ void kahan(V3<T>& s, V3<T>& c, const V3<T>& y)
{
    const V3<T> t = add(s, y);
    c = { y.x - (t.x - s.x), y.y - (t.y - s.y), y.z - (t.z - s.z) };
    s = t;
}

// Orders a wave's LDS accesses across its lanes (one wave, in-order LDS: no
// barrier instruction is needed, only that the compiler keeps the order).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace sd
