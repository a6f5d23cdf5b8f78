// lubrication.hip -- the lubrication correction of Eq. (8) folded into the
// forces with the previous step's velocities (Sec. 3.1, step 2):
//   F_i = F_ext,i - sum'_j zeta(r_i - r_j) (v_i - v_j),
//   mu0 zeta(r) = [1/(4s) - 9/40 log s] rhat rhat - 1/6 log s (I - rhat rhat),
//   s = r/a - 2 < s_cut (Sec. 2.3: s_cut = 1), clamped to s >= s_min.
// The primed sum runs over close pairs only, found with a hashed cell list
// rebuilt on the device every step: cells of side (2 + s_cut) a (free space) or
// tiling the box (at least that large), each a chain of particles in a table of
// buckets.  No bounding box, counting or sorting pass is needed: a call is three
// launches (clear the buckets, insert, forces).  The chains' order depends on
// the scheduling of the insertions, so the forces take the members of a chain
// in ascending particle index, and the 27 cells of a particle's neighbourhood
// are summed in a fixed order: the result is deterministic.  In a periodic
// cubic box cell neighbours wrap around, and each pair interacts through its
// nearest image only.  All of it is O(N x neighbours) FP64 work next to the
// O(N^2) mobility product.
#include "sd.h"
#include "sd_host.h"
#include "sd_internal.h"
#include "wave_sym.h"

#include <algorithm>
#include <cmath>

namespace sd {

// Cells and buckets.  Free space: cell floor(x / h) per axis modulo 2^32, up to
// LUB_CELL_END cells (about 2^40) from the origin, where FP64 positions resolve
// 1e-3 a: particles further out share the outermost cells, which costs time only
// (with an end of 2^30, 20000 particles at 1e10 a took 51 ms per call, at the origin
// 0.05).  Periodic: dims cells per axis tile the cube.
constexpr double LUB_CELL_END = 1097364144128.0;   // 2^40 - 2^31: not near cell 0 mod 2^32
struct CellHash {
    double ih;       // 1 / cell side
    double box;      // periodic cubic box side, 0 = free space
    int dims;        // cells per axis of the box
    unsigned mask;   // buckets - 1 (a power of two)
};

struct LubConst {
    double a, imu0, s_cut, s_min, rcut2;
    double ibox;     // 1 / box where the box is wider than two cutoffs, else 0
    PairConst pc;    // box for the nearest image
};

// Nearest image of a difference.  In a box wider than two cutoffs the product
// with 1 / box rounds to another image than the quotient only for a pair about
// half a box apart, which no image brings within the cutoff.
__device__ __forceinline__ void lub_image(const LubConst& lc, double (&d)[3])
{
    if (lc.ibox > 0.0)
        for (int k = 0; k < 3; ++k) d[k] -= lc.pc.box * rint(d[k] * lc.ibox);
    else
        nearest_image_d(lc.pc, d[0], d[1], d[2]);
}

__device__ __forceinline__ int cell_coord(const CellHash& g, double v)
{
    if (g.box > 0.0) {
        v -= g.box * floor(v / g.box);   // wrap into [0, box)
        const int c = (int)fmin(fmax(floor(v * g.ih), 0.0), 1073741824.0);
        return c >= g.dims ? g.dims - 1 : c;
    }
    return (int)(unsigned)(long long)fmin(fmax(floor(v * g.ih), -LUB_CELL_END), LUB_CELL_END);
}

// (neighbouring cells of a row along x are neighbouring buckets: nine cache
// lines per neighbourhood, not 27)
__device__ __forceinline__ unsigned bucket_of(const CellHash& g, int cx, int cy, int cz)
{
    unsigned k = (unsigned)cy * 19349663u ^ (unsigned)cz * 83492791u;
    k ^= k >> 15;
    k *= 2654435761u;
    return ((k ^ (k >> 16)) + (unsigned)cx) & g.mask;
}

// link[i]: the particle's cell, and the next particle of its bucket.
__global__ void __launch_bounds__(256) k_lub_insert(const double* __restrict__ x, int n, CellHash g,
                                                    int* __restrict__ head, int4* __restrict__ link)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int cx = cell_coord(g, x[3 * (size_t)i]), cy = cell_coord(g, x[3 * (size_t)i + 1]),
              cz = cell_coord(g, x[3 * (size_t)i + 2]);
    link[i] = make_int4(cx, cy, cz, atomicExch(&head[bucket_of(g, cx, cy, cz)], i));
}

// The m-th distinct neighbour (m = 0, 1, 2) of cell c along one axis: c - 1, c,
// c + 1, wrapped in a periodic box and without duplicates on boxes of fewer than
// three cells.  False: there is none.
__device__ __forceinline__ bool axis_neighbour(const CellHash& g, int c, int m, int& out)
{
    if (!(g.box > 0.0)) {
        out = (int)((unsigned)c - 1u + (unsigned)m);
        return true;
    }
    if (g.dims < 3) {
        out = m;
        return m < g.dims;
    }
    out = c - 1 + m;
    if (out < 0) out += g.dims;
    if (out >= g.dims) out -= g.dims;
    return true;
}

// 32 lanes per particle, one per cell of its neighbourhood (27), so that the
// chains are walked side by side: the kernel is bound by the latency of a chain
// (bucket, particle, position).  A lane takes the close particles of its cell
// LUB_TAKE at a time in ascending index; a cell with more is walked again.
// A particle's cell is kept beside its link, so that a step of the chain tests three
// integers before it loads a position (periodic fcc lattice of 202612, 12 close
// particles each: 333 us with the cells computed anew and divisions for the image
// and the unit vectors, 233 so).  Microseconds per lubrication_forces (three
// launches), where ten launches (bounding box, grid, count, three scan passes,
// scatter, sort, forces with one lane per particle) were used before: N = 100 60 ->
// 12, 5000 83 -> 13, 20000 82 -> 18, 65536 98 -> 45, 200000 156 -> 139; the lattice 253
// -> 233.
// Crowded cells (spheres that overlap: without overlap a cell holds five) are what
// sets LUB_TAKE, each further walk being a chain from its start.  Microseconds, ten
// launches / LUB_TAKE 4 / 8, random positions: 20000 with 8 per cell 401 / 133 / 116,
// with 100 3854 / 3399 / 1967; one cell of 64 185 / 348 / 237, of 2000 127e3 / 249e3 /
// 142e3; the lattice 253 / 232 / 234, 20000 at a volume fraction of 0.3 - / 31 / 31.
constexpr int LUB_TAKE = 8;

__global__ void __launch_bounds__(256)
k_lub_force(const double* __restrict__ x, const double* __restrict__ v,
            const double* __restrict__ f_ext, int n, CellHash g, const int* __restrict__ head,
            const int4* __restrict__ link, LubConst lc, double* __restrict__ f_out,
            float4* __restrict__ rec32, double4* __restrict__ rec64)
{
    const int i = blockIdx.x * 8 + (threadIdx.x >> 5);
    if (i >= n) return;   // whole groups of 32 lanes
    const int q = threadIdx.x & 31;
    const double xi[3] = { x[3 * (size_t)i], x[3 * (size_t)i + 1], x[3 * (size_t)i + 2] };
    double acc[3] = { 0.0, 0.0, 0.0 };
    int cc[3];
    bool cell = q < 27;
    const int4 ci = link[i];
    cell = axis_neighbour(g, ci.x, q % 3, cc[0]) && cell;
    cell = axis_neighbour(g, ci.y, q / 3 % 3, cc[1]) && cell;
    cell = axis_neighbour(g, ci.z, q / 9, cc[2]) && cell;
    if (cell) {
        const int first = head[bucket_of(g, cc[0], cc[1], cc[2])];
        int last = -1;
        bool more = first >= 0;
        while (more) {
            // the LUB_TAKE smallest indices above `last` of the close particles
            // of this cell (a bucket may hold other cells' particles too)
            int take[LUB_TAKE];
#pragma unroll
            for (int k = 0; k < LUB_TAKE; ++k) take[k] = 0x7fffffff;
            int4 lj;
            for (int j = first; j >= 0; j = lj.w) {
                lj = link[j];
                if (j == i || j <= last || lj.x != cc[0] || lj.y != cc[1] || lj.z != cc[2])
                    continue;
                const double xj[3] = { x[3 * (size_t)j], x[3 * (size_t)j + 1],
                                       x[3 * (size_t)j + 2] };
                double d[3] = { xi[0] - xj[0], xi[1] - xj[1], xi[2] - xj[2] };
                lub_image(lc, d);
                const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                if (!(r2 < lc.rcut2) || r2 == 0.0) continue;
                int m = j;   // into the sorted list
#pragma unroll
                for (int k = 0; k < LUB_TAKE; ++k) {
                    const int lo = min(take[k], m);
                    m = max(take[k], m);
                    take[k] = lo;
                }
            }
            more = take[LUB_TAKE - 1] != 0x7fffffff;
            last = take[LUB_TAKE - 1];
#pragma unroll
            for (int k = 0; k < LUB_TAKE; ++k) {
                const int j = take[k];
                if (j == 0x7fffffff) break;
                double d[3] = { xi[0] - x[3 * (size_t)j], xi[1] - x[3 * (size_t)j + 1],
                                xi[2] - x[3 * (size_t)j + 2] };
                lub_image(lc, d);
                const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                const double r = sqrt(r2);
                double s = r / lc.a - 2.0;
                if (s >= lc.s_cut) continue;
                if (s < lc.s_min) s = lc.s_min;
                const double ls = log(s);
                const double cP = (0.25 / s - 9.0 / 40.0 * ls) * lc.imu0;
                const double cT = (-1.0 / 6.0 * ls) * lc.imu0;
                const double ri = 1.0 / r;
                const double dv[3] = { v[3 * (size_t)i] - v[3 * (size_t)j],
                                       v[3 * (size_t)i + 1] - v[3 * (size_t)j + 1],
                                       v[3 * (size_t)i + 2] - v[3 * (size_t)j + 2] };
                const double hd = (d[0] * dv[0] + d[1] * dv[1] + d[2] * dv[2]) * ri;  // rhat . dv
                for (int k3 = 0; k3 < 3; ++k3) {
                    const double nrm = hd * d[k3] * ri;                             // (rhat rhat dv)_k
                    acc[k3] -= cP * nrm + cT * (dv[k3] - nrm);
                }
            }
        }
    }
    // over the 27 cells, fixed order: each row of 16 lanes by rotations, then the two
    for (int k = 0; k < 3; ++k) {
        acc[k] += row_rot<8>(acc[k]);
        acc[k] += row_rot<4>(acc[k]);
        acc[k] += row_rot<2>(acc[k]);
        acc[k] += row_rot<1>(acc[k]);
        acc[k] += __shfl_xor(acc[k], 16);
    }
    if (q != 0) return;
    double fo[3];
    for (int k = 0; k < 3; ++k) fo[k] = (f_ext ? f_ext[3 * (size_t)i + k] : 0.0) + acc[k];
    // the FP64 vector and/or the force record the pair kernel reads
    if (f_out)
        for (int k = 0; k < 3; ++k) f_out[3 * (size_t)i + k] = fo[k];
    if (rec32) rec32[i] = make_float4((float)fo[0], (float)fo[1], (float)fo[2], 0.0f);
    if (rec64) rec64[i] = make_double4(fo[0], fo[1], fo[2], 0.0);
}

// Buckets for n particles: a power of two, at least 2 n (at most 2^26).
static int lub_buckets(int64_t n)
{
    int b = 1024;
    while (b < 2 * n && b < (1 << 26)) b <<= 1;
    return b;
}

// f_out (f64[3n]), rec32 (f32x4[n]) and rec64 (f64x4[n]) receive the forces
// when non-null.
sd_status lub_forces_impl(const sd_params* p, const sd_lub* lub, int64_t n, const double* x,
                          const double* v, const double* f_ext, double* f_out, float4* rec32,
                          double4* rec64, hipStream_t hs)
{
    sd_status st;
    void* buf = nullptr;
    const int buckets = lub_buckets(n);
    if ((st = ws_get(WS_LUB, 4 * (size_t)buckets + sizeof(int4) * (size_t)n, &buf))) return st;
    int* head = (int*)buf;
    int4* link = (int4*)(head + buckets);
    const int nn = (int)n;
    // a pair within the cutoff lies in neighbouring cells: the side exceeds the
    // cutoff by more than the rounding of x / h (2^-12 cells at LUB_CELL_END in
    // free space)
    CellHash g;
    g.box = box_side(p);
    const double hmin = (2.0 + lub->s_cut) * p->a * (1.0 + (g.box > 0.0 ? 1e-6 : 5e-4));
    g.mask = (unsigned)buckets - 1u;
    g.dims = 0;
    double h = hmin;
    if (g.box > 0.0) {
        const double d = std::floor(g.box / hmin);
        g.dims = d < 1.0 ? 1 : (d > 1048576.0 ? 1048576 : (int)d);
        h = g.box / g.dims;
    }
    g.ih = 1.0 / h;
    hipError_t e = launch_fill_i32(head, -1, buckets, hs);
    if (e != hipSuccess) return fail(SD_EDEVICE, "fill launch: %s", hipGetErrorString(e));
    hipLaunchKernelGGL(k_lub_insert, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, hs, x, nn, g,
                       head, link);
    LubConst lc;
    lc.a = p->a;
    lc.imu0 = 6.0 * M_PI * p->eta * p->a;
    lc.s_cut = lub->s_cut;
    lc.s_min = lub->s_min;
    const double rc = (2.0 + lub->s_cut) * p->a;
    lc.rcut2 = rc * rc;
    lc.pc = pair_const(p);
    lc.ibox = g.box > 2.001 * rc ? 1.0 / g.box : 0.0;
    hipLaunchKernelGGL(k_lub_force, dim3((unsigned)((n + 7) / 8)), dim3(256), 0, hs, x, v, f_ext, nn,
                       g, head, link, lc, f_out, rec32, rec64);
    if ((e = hipGetLastError()) != hipSuccess)
        return fail(SD_EDEVICE, "lubrication launch: %s", hipGetErrorString(e));
    return SD_OK;
}

sd_status check_lub(const sd_lub* lub)
{
    if (!lub) return fail(SD_EINVAL, "lub is NULL");
    if (!(lub->s_cut > 0.0) || !std::isfinite(lub->s_cut))
        return fail(SD_EINVAL, "s_cut must be finite and > 0");
    if (!(lub->s_min > 0.0) || !(lub->s_min < lub->s_cut))
        return fail(SD_EINVAL, "s_min must be in (0, s_cut)");
    return SD_OK;
}

}  // namespace sd

using namespace sd;

extern "C" {

sd_status lubrication_forces(const sd_params* p, const sd_lub* lub, int64_t n, const double* x,
                             const double* v, const double* f_ext, double* f_out, void* stream)
{
    sd_status st;
    if ((st = check_params(p)) || (st = check_lub(lub)) || (st = check_n(n))) return st;
    if ((st = check_ptr(x, 8, "x")) || (st = check_ptr(v, 8, "v")) ||
        (st = check_ptr(f_out, 8, "f_out")))
        return st;
    if (f_ext && (uintptr_t)f_ext % 8) return fail(SD_EALIGN, "f_ext is not 8-byte aligned");
    return lub_forces_impl(p, lub, n, x, v, f_ext, f_out, nullptr, nullptr, (hipStream_t)stream);
}

sd_status sd_run_lub(const sd_params* p, const sd_lub* lub, int64_t n, double* x,
                     const double* f_ext, double* v_prev, double dt, int64_t steps, int64_t step0,
                     int32_t integrator, int32_t precision, void* stream)
{
    sd_status st;
    if ((st = check_params(p)) || (st = check_lub(lub)) || (st = check_n(n)) ||
        (st = check_precision(precision)))
        return st;
    if ((st = check_ptr(x, 8, "x")) || (st = check_ptr(f_ext, 8, "f_ext")) ||
        (st = check_ptr(v_prev, 8, "v_prev")))
        return st;
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(SD_EINVAL, "dt must be finite and > 0");
    if (integrator != SD_EULER && integrator != SD_AB2) return fail(SD_EINVAL, "unknown integrator");
    if (steps < 0 || step0 < 0) return fail(SD_EINVAL, "steps and step0 must be >= 0");
    if (steps == 0) return SD_OK;
    hipStream_t hs = (hipStream_t)stream;
    const bool f64 = precision == SD_FP64;
    const size_t rec = f64 ? 32 : 16;
    PairLaunch L;
    StepBuffers sb;
    void* F4 = nullptr;
    if ((st = step_buffers(n, precision, &L, &sb)) || (st = ws_get(WS_LUB_F, rec * (size_t)n, &F4)))
        return st;
    // per step: forces with the correction (written straight into the force
    // records of the pair kernel), then the step, which also stages the new
    // positions for the next one
    if ((st = steps_begin(p, n, x, steps, precision, L, &sb, hs))) return st;
    for (int64_t s = 0; s < steps; ++s) {
        const int64_t k = step0 + s;
        if ((st = lub_forces_impl(p, lub, n, sb.cur, v_prev, f_ext, nullptr,
                                  f64 ? nullptr : (float4*)F4, f64 ? (double4*)F4 : nullptr, hs)))
            return st;
        // Euler: x += dt v, v_prev = v;  AB2: x += dt (3/2 v - 1/2 v_prev), v_prev = v
        const int mode = (integrator == SD_EULER) ? 0 : (k == 0 ? 1 : 2);
        if ((st = steps_next(p, n, F4, mode ? v_prev : nullptr, mode ? nullptr : v_prev, dt, mode,
                             precision, L, s + 1 < steps, &sb, hs)))
            return st;
    }
    return SD_OK;
}

}  // extern "C"
