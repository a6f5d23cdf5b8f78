// wave_f32.hip -- the FP32 product v = M(x) F with each pair of particles
// evaluated once (wave-symmetric schedule, wave_sym.h), for suspensions too
// small for the block-symmetric kernel of mobility.hip to fill the chip.
#include "pair_terms.h"
#include "premise.h"
#include "sd_internal.h"
#include "wave_chunk_asm.h"
#include "wave_sym.h"

namespace sd {

#define SD_FAR_I (-1.0e15f)
#define SD_FAR_J (1.0e15f)

// The near pairs of a chunk, in FP64, with i from memory (the loop is rare and
// its registers would otherwise be the kernel's): for every step k and lane
// particle a, test(k, a, i, jg) says whether the lane's pair is near; get(k, pj,
// fj) reads the staged element (q + k) mod 16.  The i side goes to the lane's
// FP64 slots own_w (component c of particle a at (2 c + a) 64 + lane), the j
// side of element q, summed over the rows of the wave, to nj.
template <int TENSOR, bool PER, class Test, class Get>
__device__ __forceinline__ void near_chunk(const float4* __restrict__ pos,
                                           const float4* __restrict__ frc,
                                           const double* __restrict__ x64, int n, int ib, bool diag,
                                           int j0, const PairConst& pc, double* own_w,
                                           unsigned long long* premise, V3<double>& nj, Test test,
                                           Get get)
{
    constexpr int ILP = 2, B = 64 * ILP;
    const int lane = threadIdx.x & 63, q = lane & 15;
#pragma unroll 1
    for (int b = 0; b < 16 * ILP; ++b) {
        const int k = b / ILP, a = b % ILP;
        const int jg = j0 + ((q + k) & 15);
        const int i = ib * B + a * 64 + lane;
        const bool mine = test(k, a, i, jg);
        if (__builtin_amdgcn_ballot_w64(mine) == 0) continue;
        V3<double> c = { 0.0, 0.0, 0.0 };
        int cls = PREMISE_OK;
        if (mine && i < n && jg < n && i != jg) {
            double* const own = own_w + a * 64 + lane;
            const float4 pi = pos[i], fi = frc[i];
            float4 pj, fj;
            get(k, pj, fj);
            V3<double> D;
            near_diff_v<PER>(pi.x, pi.y, pi.z, i, pj, jg, pc, x64, D.x, D.y, D.z);
            double A, Bt;
            cls = near_coef<TENSOR>(pc, dot(D, D), A, Bt);
            A *= pc.alpha;
            Bt *= pc.alpha;
            const double sj = Bt * (D.x * fj.x + D.y * fj.y + D.z * fj.z);
            const double si = Bt * (D.x * fi.x + D.y * fi.y + D.z * fi.z);
            own[0] += A * fj.x + sj * D.x;
            own[B] += A * fj.y + sj * D.y;
            own[2 * B] += A * fj.z + sj * D.z;
            c = { A * fi.x + si * D.x, A * fi.y + si * D.y, A * fi.z + si * D.z };
        }
        // the diagonal block meets both orderings of a pair
        count_premise(premise, !diag || i < jg ? cls : (int)PREMISE_OK);
        const int from = (lane & 48) | ((q - k) & 15);
        nj.x += __shfl(c.x, from);
        nj.y += __shfl(c.y, from);
        nj.z += __shfl(c.z, from);
    }
    nj.x += __shfl_xor(nj.x, 16);
    nj.y += __shfl_xor(nj.y, 16);
    nj.z += __shfl_xor(nj.z, 16);
    nj.x += __shfl_xor(nj.x, 32);
    nj.y += __shfl_xor(nj.y, 32);
    nj.z += __shfl_xor(nj.z, 32);
}

// j-side partials of a chunk: the two half sums of each of the wave's four rows
// (sj[8][48]), added in FP64 in a fixed order, and the near pairs.
__device__ __forceinline__ void store_rows(const float* sj, double alpha, bool near,
                                           const V3<double>& nj, double* __restrict__ jpart,
                                           const WaveShape& sh, int ib, int p)
{
    const int lane = threadIdx.x & 63, q = lane & 15, row = lane >> 4;
    wave_lds_fence();
    if (lane < 48) {   // component `row` of element q
        double t = (double)sj[lane];
#pragma unroll
        for (int r = 1; r < 8; ++r) t += (double)sj[r * 48 + lane];
        t *= alpha;
        if (near) t += row == 0 ? nj.x : row == 1 ? nj.y : nj.z;
        jpart[((size_t)row * sh.nb + ib) * (size_t)sh.lmax + (size_t)(p + q)] = t;
    }
}

// i-side sums of the four waves (si[4][3 B]), added in wave order -> split row s
template <int B>
__device__ __forceinline__ void store_sums(const double* si, int n, int ib, int s,
                                           double* __restrict__ partial)
{
    for (int t = (int)threadIdx.x; t < 3 * B; t += 256) {
        const int c = t / B, i = ib * B + t % B;
        if (i < n)
            partial[((size_t)s * 3 + c) * (size_t)n + i] =
                ((si[t] + si[3 * B + t]) + si[6 * B + t]) + si[9 * B + t];
    }
}

// partial: FP64 split rows (the diagonal row last); jpart[c][I][p]: FP64 j-side
// partials; both in physical units.
//
// Two particles per lane; the chunk loop is assembly (wave_chunk_asm.h,
// generated by gen_sym_chunk.py) with registers chosen for the VGPR read
// ports.  The chunk is staged as six doubled float arrays (x, y, z of positions
// and forces), so that every component is read into a register of the parity
// that the generated code expects.
//
// Sums.  i side: blocks of four terms, added in FP32 and compensated once per
// chunk of 16.  j side: the two terms of a step, blocks of four steps, two of
// those added in FP32, and in FP64 from there on.  (Longer blocks let each term
// be rounded into a larger partial sum: the error at N = 6007 is 0.6e-7, the
// one-sided kernel's with blocks of eight 0.65e-7, that of the block-symmetric
// kernel's 32 1.1e-7.)  Near pairs contribute nothing in FP32: the lanes that
// met one send the chunk to the rare loop, which evaluates them in FP64 on both
// sides.
//
// Bound by the vector ALU: 1321 instructions for the 32 pairs (64 interactions)
// of a lane and chunk; with the diagonal blocks and what surrounds the chunk 42 per
// unordered pair at N = 8192, one per 3.8 cycles and SIMD (6007 4.3, 12000 3.5) at a
// clock of 1.9 GHz.  The chunk pins 103 of the 128 registers that
// four waves per SIMD leave, and the compiler spills what is left beside it: 18
// values (76 bytes per lane) for the RPY tensor, 6 for Oseen, four of them reloaded
// in every chunk, the others on the near branch.  Microseconds per product with the
// fold, compiled loop / assembly: N = 6007 31.7 / 28.5, 8192 47.8 / 42.8 (one-sided
// kernel 43.9, 54.4).
template <int TENSOR, bool PER>
__global__ void __launch_bounds__(256, 4)
k_wave_f32(const float4* __restrict__ pos, const float4* __restrict__ frc,
               const double* __restrict__ x64, int n, WaveShape sh, PairConst pc,
               double* __restrict__ partial, double* __restrict__ jpart,
               unsigned long long* __restrict__ premise)
{
    constexpr int B = 128;
    typedef __attribute__((address_space(3))) float lds_float;
    constexpr int NC = 4, CS = 6 * 32;   // chunks staged at once, floats of one
    __shared__ float s_soa[4][NC * CS];
    __shared__ float s_j[4][8 * 48];
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
    // lane state in the registers that the generated chunk expects
    const float far = PER ? 0.0f : SD_FAR_I;
    float x0 = far, y0 = far, z0 = far, x1 = far, y1 = far, z1 = far;
    float f0x = 0.0f, f0y = 0.0f, f0z = 0.0f, f1x = 0.0f, f1y = 0.0f, f1z = 0.0f;
    {
        const int i0 = ib * B + lane, i1 = i0 + 64;
        if (i0 < n) {
            const float4 p = pos[i0], f = frc[i0];
            x0 = p.x; y0 = p.y; z0 = p.z;
            f0x = f.x; f0y = f.y; f0z = f.z;
        }
        if (i1 < n) {
            const float4 p = pos[i1], f = frc[i1];
            x1 = p.x; y1 = p.y; z1 = p.z;
            f1x = f.x; f1y = f.y; f1z = f.z;
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) s_i[w][c * 64 + lane] = 0.0;   // near pairs first
    }
    float s0x = 0.0f, s0y = 0.0f, s0z = 0.0f, s1x = 0.0f, s1y = 0.0f, s1z = 0.0f;   // sums
    float c0x = 0.0f, c0y = 0.0f, c0z = 0.0f, c1x = 0.0f, c1y = 0.0f, c1z = 0.0f;   // -compensation
    float k_gamma = pc.gamma_f, k_m3g = pc.m3gamma_f, k_thr2 = pc.thr2_f, k_inf = __builtin_inff();
    asm volatile("" : "+v"(k_gamma), "+v"(k_m3g), "+v"(k_thr2), "+v"(k_inf));
    auto chunk_start = [&](int p) {
        if (diag) return ib * B + p;
        const int J = ib + 1 + p / B;
        return (J >= sh.nb ? J - sh.nb : J) * B + p % B;
    };
    const uint32_t jaddr = (uint32_t)(uintptr_t)(lds_float*)(s_j[w] + row * 48 + q);
#pragma unroll 1
    for (int p = pbeg; p < pend; p += 16) {
        const int at = ((p - pbeg) / 16 & (NC - 1)) * CS;
        if (at == 0) {
            // up to four chunks, one particle per lane (no copy is fetched ahead:
            // the registers are the chunk's, and four waves per SIMD cover it)
            const int pl = p + 16 * row;
            float4 rp = make_float4(0.0f, 0.0f, 0.0f, 0.0f), rf = rp;
            if (!PER) rp = make_float4(SD_FAR_J, SD_FAR_J, SD_FAR_J, 0.0f);
            if (pl < pend) {
                const int j = chunk_start(pl) + q;
                if (j < n) {
                    rp = pos[j];
                    rf = frc[j];
                }
            }
            wave_lds_fence();
            float* const d = s_soa[w] + row * CS + q;
            d[0] = d[16] = rp.x;
            d[32] = d[48] = rp.y;
            d[64] = d[80] = rp.z;
            d[96] = d[112] = rf.x;
            d[128] = d[144] = rf.y;
            d[160] = d[176] = rf.z;
            wave_lds_fence();
        }
        const uint32_t addr = (uint32_t)(uintptr_t)(lds_float*)(s_soa[w] + at + q);
        uint64_t nearl = 0;   // lanes that met a near pair in the chunk
        // every operand is in/out or an input in the register that the
        // generated code names, so no copies are made
#define SD_WAVE_CHUNK_CALL(TEXT)                                                               \
    asm volatile(TEXT                                                                          \
                 : [s0x] "+" SD_WAVE_R_S0x(s0x), [s0y] "+" SD_WAVE_R_S0y(s0y),                 \
                   [s0z] "+" SD_WAVE_R_S0z(s0z), [s1x] "+" SD_WAVE_R_S1x(s1x),                 \
                   [s1y] "+" SD_WAVE_R_S1y(s1y), [s1z] "+" SD_WAVE_R_S1z(s1z),                 \
                   [y0x] "+" SD_WAVE_R_Y0x(c0x), [y0y] "+" SD_WAVE_R_Y0y(c0y),                 \
                   [y0z] "+" SD_WAVE_R_Y0z(c0z), [y1x] "+" SD_WAVE_R_Y1x(c1x),                 \
                   [y1y] "+" SD_WAVE_R_Y1y(c1y), [y1z] "+" SD_WAVE_R_Y1z(c1z),                 \
                   [x0] "+" SD_WAVE_R_X0x(x0), [y0] "+" SD_WAVE_R_X0y(y0),                     \
                   [z0] "+" SD_WAVE_R_X0z(z0), [x1] "+" SD_WAVE_R_X1x(x1),                     \
                   [y1] "+" SD_WAVE_R_X1y(y1), [z1] "+" SD_WAVE_R_X1z(z1),                     \
                   [f0x] "+" SD_WAVE_R_FI0x(f0x), [f0y] "+" SD_WAVE_R_FI0y(f0y),               \
                   [f0z] "+" SD_WAVE_R_FI0z(f0z), [f1x] "+" SD_WAVE_R_FI1x(f1x),               \
                   [f1y] "+" SD_WAVE_R_FI1y(f1y), [f1z] "+" SD_WAVE_R_FI1z(f1z),               \
                   [nl] "+s"(nearl)                                                            \
                 : [adr] SD_WAVE_R_ADDR(addr), [jadr] SD_WAVE_R_JADDR(jaddr),                  \
                   [gam] SD_WAVE_R_GAMMA(k_gamma), [thr] SD_WAVE_R_THR2(k_thr2),               \
                   [thro] SD_WAVE_R_THR2O(k_thr2), [inf] SD_WAVE_R_INF(k_inf),                 \
                   [m3g] SD_WAVE_R_M3G(k_m3g)                                                  \
                 : SD_WAVE_CLOBBERS, "vcc", "scc", "memory")
        if constexpr (TENSOR == T_RPY && !PER)
            SD_WAVE_CHUNK_CALL(SD_WAVE_CHUNK_RPY_FREE);
        else if constexpr (TENSOR == T_RPY)
            SD_WAVE_CHUNK_CALL(SD_WAVE_CHUNK_RPY_PER);
        else if constexpr (!PER)
            SD_WAVE_CHUNK_CALL(SD_WAVE_CHUNK_OSEEN_FREE);
        else
            SD_WAVE_CHUNK_CALL(SD_WAVE_CHUNK_OSEEN_PER);
#undef SD_WAVE_CHUNK_CALL
        V3<double> nj = { 0.0, 0.0, 0.0 };   // near pairs, j side of element q
        if (nearl != 0) {   // rare
            const float* const d = s_soa[w] + at + q;
            auto get = [&](int k, float4& pj, float4& fj) {
                pj = make_float4(d[k], d[32 + k], d[64 + k], 0.0f);
                fj = make_float4(d[96 + k], d[128 + k], d[160 + k], 0.0f);
            };
            // the threshold test of the chunk again (the same operations)
            uint32_t nearm = 0;
#pragma unroll 4
            for (int k = 0; k < 16; ++k) {
                const V3<float> P = { d[k], d[32 + k], d[64 + k] };
                const V3<float> D0 = { pdiff<PER>(x0, P.x), pdiff<PER>(y0, P.y),
                                       pdiff<PER>(z0, P.z) };
                const V3<float> D1 = { pdiff<PER>(x1, P.x), pdiff<PER>(y1, P.y),
                                       pdiff<PER>(z1, P.z) };
                nearm |= dot(D0, D0) < k_thr2 ? 1u << (2 * k) : 0u;
                nearm |= dot(D1, D1) < k_thr2 ? 2u << (2 * k) : 0u;
            }
            auto test = [&](int k, int a, int, int) { return (nearm >> (2 * k + a)) & 1u; };
            near_chunk<TENSOR, PER>(pos, frc, x64, n, ib, diag, chunk_start(p), pc,
                                         &s_i[w][0], premise, nj, test, get);
        }
        if (!diag) store_rows(s_j[w], pc.alpha_sum, nearl != 0, nj, jpart, sh, ib, p);
    }
    double* const own = &s_i[w][lane];
    own[0] += pc.alpha_sum * ((double)s0x + (double)c0x);
    own[64] += pc.alpha_sum * ((double)s1x + (double)c1x);
    own[B] += pc.alpha_sum * ((double)s0y + (double)c0y);
    own[B + 64] += pc.alpha_sum * ((double)s1y + (double)c1y);
    own[2 * B] += pc.alpha_sum * ((double)s0z + (double)c0z);
    own[2 * B + 64] += pc.alpha_sum * ((double)s1z + (double)c1z);
    __syncthreads();
    store_sums<B>(&s_i[0][0], n, ib, s, partial);
}

hipError_t launch_wave_f32(const PairLaunch& L, int tensor, const float4* pos, const float4* frc,
                           const double* x64, int n, const PairConst& pc, double* partial,
                           hipStream_t st)
{
    const WaveShape sh = wave_shape_of(L, n);
    double* jpart = (double*)((char*)partial + wave_jpart_offset(sh, n));
    unsigned long long* premise = nullptr;
    if (const hipError_t e = premise_counters(&premise); e != hipSuccess) return e;
    const dim3 grid((unsigned)(sh.nb * (sh.splits + 1))), block(256);
    const bool per = pc.box > 0.0;
#define SD_GO(T, P)                                                                             \
    hipLaunchKernelGGL((k_wave_f32<T, P>), grid, block, 0, st, pos, frc, x64, n, sh, pc, partial, \
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
