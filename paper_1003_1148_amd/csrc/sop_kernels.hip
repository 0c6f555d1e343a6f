// HIP kernels for gfx950: Verlet-list rebuild on a wrapped cell grid, the
// fused per-step kernel (SOP forces of Eq. 1 over bonds, natives and the
// list; Philox4x32-10 Box-Muller noise; first-order overdamped update of
// Eq. 2 / Algorithm 7 with compensated single-precision positions), and the
// double-precision energy reduction.
#include <algorithm>
#include <type_traits>

#include "sop_internal.hpp"
#include "sop_rng.hpp"

namespace sop {

namespace {

constexpr int WG = 256;       // threads per workgroup (4 wave64)

__device__ __forceinline__ float comp(const float4 &v, int a)
{
    return a == 0 ? v.x : (a == 1 ? v.y : v.z);
}

// Cell index along one axis: floor(x / edge) shifted by the trajectory's
// offset and wrapped into [0, n), so every position has a valid cell.
__device__ __forceinline__ int wrap_cell(float x, float inv_cell, int off, int n)
{
    float v = floorf(x * inv_cell);
    if (!(v == v))
        v = 0.0f;  // NaN positions are flagged elsewhere; keep the index in range
    v = fminf(fmaxf(v, -1.0e9f), 1.0e9f);
    int c = (static_cast<int>(v) + off) % n;
    return c < 0 ? c + n : c;
}

// The list predicate in single precision without contraction:
// fl(fl(fl(dx*dx) + fl(dy*dy)) + fl(dz*dz)) < rc2, dx = fl(xi - xj).
__device__ __forceinline__ bool within_cutoff(float4 a, float4 b, float rc2)
{
#pragma clang fp contract(off)
    const float dx = a.x - b.x;
    const float dy = a.y - b.y;
    const float dz = a.z - b.z;
    const float xx = dx * dx;
    const float yy = dy * dy;
    const float zz = dz * dz;
    const float s = xx + yy;
    const float d2 = s + zz;
    return d2 < rc2;
}

// Pair difference from compensated positions: (hi_i - hi_j) + (lo_i - lo_j).
__device__ __forceinline__ float3 pair_delta(const float4 &hi, const float4 &lo, const float4 &hj,
                                             const float4 &lj)
{
    return make_float3((hi.x - hj.x) + (lo.x - lj.x), (hi.y - hj.y) + (lo.y - lj.y),
                       (hi.z - hj.z) + (lo.z - lj.z));
}

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// ---------------------------------------------------------------------------
// Verlet-list rebuild: clear cell counts -> bin into fixed-capacity cells ->
// one workgroup per cell fills the rows of its residues
// ---------------------------------------------------------------------------
// Cell index of one residue in the wrapped grid (the trajectory's offset
// keeps independent trajectories in separate cells).
__device__ __forceinline__ int cell_index(const float4 &p, const int4 &off, const GridDev &g)
{
    const int cx = wrap_cell(p.x, g.inv_cell, off.x, g.gx);
    const int cy = wrap_cell(p.y, g.inv_cell, off.y, g.gy);
    const int cz = wrap_cell(p.z, g.inv_cell, off.z, g.gz);
    return cx + g.gx * (cy + g.gy * cz);
}

// Fixed-point copy of a position: hi + lo as a whole number of units of 2^-k
// (FixDev), modulo 2^32, and in w ten bits an axis of the periods of 2^32
// units below it.  The difference of two copies, taken in 32-bit integers, is
// exact whatever the distance of the residues from the origin, as long as
// they are less than 2^31 units apart.  x 2^k + 1.5 * 2^52, rounded once,
// holds the whole number in its low word and the periods above it; farther
// out than 2^50 units the periods are taken off first (x - P rint(x / P) is
// exact), with the same bits.
__device__ __forceinline__ int4 fix_pos(const float4 &hi, const float4 &lo, const FixDev &f)
{
    int q[3], n[3];
    if (fmaxf(fmaxf(fabsf(hi.x), fabsf(hi.y)), fabsf(hi.z)) < f.direct) {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const double v = __builtin_fma((double)comp(hi, ax) + (double)comp(lo, ax), f.scale, 0x1.8p52);
            q[ax] = __double2loint(v);
            n[ax] = __double2hiint(v);
        }
    } else {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const double x = (double)comp(hi, ax) + (double)comp(lo, ax);
            const double m = __builtin_rint(x * f.inv_period);
            const double r = __builtin_fma(-f.period, m, x);
            q[ax] = __double2loint(__builtin_fma(r, f.scale, 0x1.8p52));
            n[ax] = __double2loint(m + 0x1.8p52) - (r < 0.0 && q[ax] < 0 ? 1 : 0);
        }
    }
    return make_int4(q[0], q[1], q[2], (n[0] & 1023) | (n[1] & 1023) << 10 | (n[2] & 1023) << 20);
}

// Difference of two such positions up to 512 periods apart, exact before its
// one rounding: the bits of the plain integer difference wherever that does
// not wrap.
__device__ __forceinline__ float3 fix_full_diff(const int4 &a, const int4 &b)
{
    const unsigned qa[3] = {(unsigned)a.x, (unsigned)a.y, (unsigned)a.z};
    const unsigned qb[3] = {(unsigned)b.x, (unsigned)b.y, (unsigned)b.z};
    float d[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int dn = (int)(((unsigned)(a.w >> (10 * ax)) - (unsigned)(b.w >> (10 * ax))) << 22) >> 22;
        d[ax] = (float)__builtin_fma((double)dn, 4294967296.0, (double)qa[ax] - (double)qb[ax]);
    }
    return make_float3(d[0], d[1], d[2]);
}

// The same at any distance, from the compensated positions.
__device__ __forceinline__ float3 fix_exact_diff(const float4 &hi, const float4 &lo, const float4 &hj,
                                                 const float4 &lj, const FixDev &f)
{
    float d[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const double xi = (double)comp(hi, ax) + (double)comp(lo, ax), xj = (double)comp(hj, ax) + (double)comp(lj, ax);
        d[ax] = (float)(__builtin_rint(xi * f.scale) - __builtin_rint(xj * f.scale));
    }
    return make_float3(d[0], d[1], d[2]);
}

// Difference of two fixed-point coordinates, modulo 2^32.
__device__ __forceinline__ int fix_diff(int a, int b) { return (int)((unsigned)a - (unsigned)b); }

// A copy to 10 bits an axis, and whether one that was at `place` then may be
// further than FixDev::move from it.
__device__ __forceinline__ unsigned fix_place(const int4 &q)
{
    return (unsigned)q.x >> 22 | ((unsigned)q.y >> 22) << 10 | ((unsigned)q.z >> 22) << 20;
}

__device__ __forceinline__ bool strayed(const int4 &q, unsigned place, const FixDev &f)
{
    auto out = [&](int x, unsigned p) { return (unsigned)fix_diff(x, (int)(p << 22)) + f.move > 2u * f.move; };
    return out(q.x, place) || out(q.y, place >> 10) || out(q.z, place >> 20);
}

// Bin one residue at high part p into the grid of the next skin search:
// its cell, a slot in that cell, and a copy of p there.
__device__ __forceinline__ void bin_one(const float4 &p, int i, int traj, const GridDev &g,
                                        const int4 *__restrict__ traj_cell, int *__restrict__ count,
                                        float4 *__restrict__ cells, int *__restrict__ cell_of,
                                        unsigned *__restrict__ err)
{
    const int c = cell_index(p, traj_cell[traj], g);
    cell_of[i] = c;
    const int slot = atomicAdd(&count[c], 1);
    if (slot < CELL_CAP)
        cells[(size_t)c * CELL_CAP + slot] = make_float4(p.x, p.y, p.z, __int_as_float(i));
    else
        atomicOr(err, ERR_CELL);
}

__global__ void k_clear(int *__restrict__ a, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        a[i] = 0;
}

// Every residue binned at its current position, and its fixed-point copy.
// The last step kernel of each list period bins the positions it writes (and
// every step kernel writes the copies); this kernel serves the rebuilds that
// do not follow such a step (after new coordinates, a new step count or a
// new tile size), after k_clear.
__global__ void k_bin_all(const float4 *__restrict__ pos, int n, GridDev g, const int4 *__restrict__ traj_cell,
                          int *__restrict__ count, float4 *__restrict__ cells, int *__restrict__ cell_of,
                          unsigned *__restrict__ err, int4 *__restrict__ fix, FixDev f)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const float4 p = pos[2 * i];
    if (!isfinite(p.x) || !isfinite(p.y) || !isfinite(p.z))
        atomicOr(err, ERR_NONFINITE);
    const float4 l = pos[2 * i + 1];
    fix[i] = fix_pos(p, l, f);
    bin_one(p, i, __float_as_int(l.w), g, traj_cell, count, cells, cell_of, err);
}

// ---------------------------------------------------------------------------
// Pair terms of Eq. 1, external terms and the compensated update, shared by
// the plain and the batched schedules.
// ---------------------------------------------------------------------------

// Per-residue force and, on energy steps, double energy/virial sums.
struct Acc {
    float fx = 0.f, fy = 0.f, fz = 0.f;
    double e_b = 0.0, e_n = 0.0, e_r = 0.0, vir = 0.0;
};

struct PairConsts {
    float kf, inv_R0sq, R0sq, eh, eh12, el, el6, sg2, sg6, c6;
};

__device__ __forceinline__ PairConsts pair_consts(const StepConsts &c)
{
    PairConsts k;
    k.kf = c.k_fene;
    k.inv_R0sq = c.inv_R0sq;
    k.R0sq = c.R0sq;
    k.eh = c.eps_h;
    k.eh12 = 12.0f * c.eps_h;
    k.el = c.eps_l;
    k.el6 = 6.0f * c.eps_l;
    k.sg2 = c.sigma2;
    k.sg6 = c.sigma2 * c.sigma2 * c.sigma2;
    k.c6 = k.el6 * k.sg6;  // force coefficient 6 eps_l sigma^6 / r^8
    return k;
}

// The force arithmetic of the pair and external terms states every fused
// multiply-add and lets the compiler fuse nothing else, so a term's force has
// the same bits in every kernel that evaluates it, whether or not that
// kernel also takes the term's energy (which shares its subexpressions).
__device__ __forceinline__ float len2(const float3 &d)
{
#pragma clang fp contract(off)
    return __builtin_fmaf(d.z, d.z, __builtin_fmaf(d.y, d.y, d.x * d.x));
}

__device__ __forceinline__ void acc_force(Acc &A, float c, const float3 &d)
{
    A.fx = __builtin_fmaf(c, d.x, A.fx);
    A.fy = __builtin_fmaf(c, d.y, A.fy);
    A.fz = __builtin_fmaf(c, d.z, A.fz);
}

// FENE: -(k R0^2/2) ln(1 - (r - r0)^2/R0^2); |r - r0| >= R0 sets `broken`.
__device__ __forceinline__ void add_fene_d(Acc &A, const float3 &d, float r0, const PairConsts &k, bool rec,
                                           bool &broken)
{
#pragma clang fp contract(off)
    const float rr = __builtin_amdgcn_sqrtf(len2(d));
    const float dl = rr - r0;
    float x = __builtin_fmaf(-(dl * dl), k.inv_R0sq, 1.0f);
    if (!(x > 0.0f)) {
        broken = true;
        x = 1.0f;
    }
    acc_force(A, -k.kf * dl * fast_rcp(x * rr), d);
    if (rec) {
        const double dd = (double)dl;
        const double R0sq = (double)k.R0sq;
        A.e_b += -0.5 * (double)k.kf * R0sq * log1p(-dd * dd / R0sq);
        A.vir += -(double)rr * (double)k.kf * dd / (1.0 - dd * dd / R0sq);
    }
}

// Native contact: eps_h [(r0/r)^12 - 2 (r0/r)^6].
__device__ __forceinline__ void add_native_d(Acc &A, const float3 &d, float r02, const PairConsts &k, bool rec)
{
#pragma clang fp contract(off)
    const float ir2 = fast_rcp(len2(d));
    const float s = r02 * ir2;
    const float q = s * s * s;
    const float w = __builtin_fmaf(q, q, -q);  // q^2 - q
    acc_force(A, k.eh12 * w * ir2, d);
    if (rec) {
        A.e_n += (double)(k.eh * __builtin_fmaf(q, q, -2.0f * q));
        A.vir += (double)(k.eh12 * w);
    }
}

// The same from a difference d in fixed-point units: r02 = r0^2 in the
// caller's units, s2 = 1 / unit^2, eu = 12 eps_h unit (so the force needs no
// scaled difference).
__device__ __forceinline__ void add_native_q(Acc &A, const float3 &d, float r02, float s2, float eu,
                                             const PairConsts &k, bool rec)
{
#pragma clang fp contract(off)
    const float ir2 = fast_rcp(len2(d)) * s2;
    const float s = r02 * ir2;
    const float q = s * s * s;
    const float w = __builtin_fmaf(q, q, -q);  // q^2 - q
    acc_force(A, eu * w * ir2, d);
    if (rec) {
        A.e_n += (double)(k.eh * __builtin_fmaf(q, q, -2.0f * q));
        A.vir += (double)(k.eh12 * w);
    }
}

// Soft repulsion: eps_l (sigma/r)^6.
__device__ __forceinline__ void add_repulsive_d(Acc &A, const float3 &d, const PairConsts &k, bool rec)
{
#pragma clang fp contract(off)
    const float ir2 = fast_rcp(len2(d));
    const float ir4 = ir2 * ir2;
    acc_force(A, k.c6 * ir4 * ir4, d);
    if (rec) {
        const float q = k.sg6 * ir4 * ir2;
        A.e_r += (double)(k.el * q);
        A.vir += (double)(k.el6 * q);
    }
}

// The list-pair form of the soft repulsion: accumulates d / r^8, so the
// caller multiplies the row's sum by 6 eps_l sigma^6 once instead of every
// pair; the energy and virial terms are the full ones.
__device__ __forceinline__ void add_repulsive_u(Acc &A, const float3 &d, const PairConsts &k, bool rec)
{
#pragma clang fp contract(off)
    const float ir2 = fast_rcp(len2(d));
    const float ir4 = ir2 * ir2;
    acc_force(A, ir4 * ir4, d);
    if (rec) {
        const float q = k.sg6 * ir4 * ir2;
        A.e_r += (double)(k.el * q);
        A.vir += (double)(k.el6 * q);
    }
}

// The same from the difference d of two fixed-point copies (whole numbers of
// units, exact; rounded once by the conversion): accumulates d / r^8 with r
// in the caller's units and d in fixed-point ones.  s2 = 1 / unit^2; `live`
// false: no contribution, whatever q.
__device__ __forceinline__ void add_repulsive_q(Acc &A, const int3 &q, float s2, const PairConsts &k, bool live,
                                                bool rec)
{
#pragma clang fp contract(off)
    const float3 d = make_float3((float)q.x, (float)q.y, (float)q.z);
    const float ir2 = fast_rcp(len2(d)) * s2;
    const float ir4 = ir2 * ir2;
    acc_force(A, live ? ir4 * ir4 : 0.0f, d);
    if (rec) {
        const float q6 = live ? k.sg6 * ir4 * ir2 : 0.0f;
        A.e_r += (double)(k.el * q6);
        A.vir += (double)(k.el6 * q6);
    }
}

// Cantilever `pull` (index or -1) and tip on one residue at t_n = step*h.
__device__ __forceinline__ void add_external(Acc &A, double &e_x, double &f_rep, const float4 &hi,
                                             const float4 &lo, long long step, double h, int pull,
                                             const PullDev *pulls, const TipDev &tip, bool rec,
                                             unsigned *err)
{
#pragma clang fp contract(off)
    if (pull < 0 && !tip.on)
        return;
    const double tn = (double)step * h;
    const double px = (double)hi.x + (double)lo.x;
    const double py = (double)hi.y + (double)lo.y;
    const double pz = (double)hi.z + (double)lo.z;
    if (pull >= 0) {
        const PullDev pd = pulls[pull];
        const double dx = __builtin_fma(pd.v[0], tn, pd.anchor0[0]) - px;
        const double dy = __builtin_fma(pd.v[1], tn, pd.anchor0[1]) - py;
        const double dz = __builtin_fma(pd.v[2], tn, pd.anchor0[2]) - pz;
        A.fx += (float)(pd.kappa * dx);
        A.fy += (float)(pd.kappa * dy);
        A.fz += (float)(pd.kappa * dz);
        if (rec) {
            const double d2 = dx * dx + dy * dy + dz * dz;
            e_x += 0.5 * pd.kappa * d2;
            f_rep += pd.has_dir ? pd.kappa * (dx * pd.vhat[0] + dy * pd.vhat[1] + dz * pd.vhat[2])
                                : pd.kappa * sqrt(d2);
        }
    }
    if (tip.on) {
        const float dx = (float)(px - __builtin_fma(tip.v[0], tn, tip.c0[0]));
        const float dy = (float)(py - __builtin_fma(tip.v[1], tn, tip.c0[1]));
        const float dz = (float)(pz - __builtin_fma(tip.v[2], tn, tip.c0[2]));
        const float rr = sqrtf(len2(make_float3(dx, dy, dz)));
        const float gap = rr - (float)tip.radius;
        if (!(gap > 0.0f)) {
            atomicOr(err, ERR_TIP);
            return;
        }
        const float igap = fast_rcp(gap);
        const float sg = (float)tip.sigma * igap;
        const float s3 = sg * sg * sg;
        const float q = s3 * s3;
        const float mag_r = 6.0f * (float)tip.eps * q * igap * fast_rcp(rr);  // magnitude / r
        acc_force(A, mag_r, make_float3(dx, dy, dz));
        if (rec) {
            e_x += tip.eps * (double)q;
            if (tip.has_dir)
                f_rep += (double)(mag_r * dx) * tip.vhat[0] + (double)(mag_r * dy) * tip.vhat[1] +
                         (double)(mag_r * dz) * tip.vhat[2];
        }
    }
}

// Philox words of one residue and step: counter (index in the trajectory,
// stream id, step), key = seed.
__device__ __forceinline__ uint4 noise_words(unsigned tag, unsigned stream, long long step, const StepConsts &c)
{
    return philox10(make_uint4(tag & 0x7fffffffu, stream, (unsigned)step,
                               (unsigned)((unsigned long long)step >> 32)),
                    c.key0, c.key1);
}

// First-order update with the Gaussian components g:
// (hi, lo) <- TwoSum(hi, f h/zeta + g sqrt(2 kB T h/zeta) + lo) per axis.
// A step longer than `most` on an axis sets *moved; one that is not leaves
// finite positions finite.
__device__ __forceinline__ void update_with_noise(float4 &hi, float4 &lo, const Acc &A, const float g[3],
                                                  const StepConsts &c, float most, unsigned *moved, unsigned *err)
{
#pragma clang fp contract(off)
    if (__float_as_uint(hi.w) >> 31)
        return;  // fixed residue
    float nh[3], nl[3];
    bool within = true;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float f = ax == 0 ? A.fx : (ax == 1 ? A.fy : A.fz);
        const float h0 = comp(hi, ax), l0 = comp(lo, ax);
        const float delta = __builtin_fmaf(c.c_drift, f, c.c_noise * g[ax]);
        within &= fabsf(delta) <= most;
        const float y = delta + l0;
        const float t = h0 + y;
        const float bp = t - h0;
        const float ap = t - bp;
        nl[ax] = (h0 - ap) + (y - bp);
        nh[ax] = t;
    }
    if (__builtin_expect(!within, 0)) {
        *moved = 1u;
        if (!isfinite(nh[0]) || !isfinite(nh[1]) || !isfinite(nh[2]) || !isfinite(nl[0]) ||
            !isfinite(nl[1]) || !isfinite(nl[2]))
            atomicOr(err, ERR_NONFINITE);
    }
    hi = make_float4(nh[0], nh[1], nh[2], hi.w);
    lo = make_float4(nl[0], nl[1], nl[2], lo.w);
}

// Underdamped Langevin step (BAOAB): the velocity v stored between steps is
// the one before the last half kick of the previous step, so one kick of
// `kick` (h/m, or h/2m on the first step after velocities were set) with
// the force of this step covers that half kick and this step's first one;
// then x += (h/2) w, w = c1 w + c2 g, x += (h/2) w (compensated), v = w.
struct UdConsts {
    float kick, c1, c2, half_h;
};

__device__ __forceinline__ void underdamped_update(float4 &hi, float4 &lo, float4 &v, const Acc &A,
                                                   const float g[3], const UdConsts &u, float most, unsigned *moved,
                                                   unsigned *err)
{
#pragma clang fp contract(off)
    if (__float_as_uint(hi.w) >> 31) {
        v = make_float4(0.f, 0.f, 0.f, 0.f);  // fixed residue
        return;
    }
    float nh[3], nl[3], nv[3];
    bool within = true;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float f = ax == 0 ? A.fx : (ax == 1 ? A.fy : A.fz);
        const float w0 = __builtin_fmaf(u.kick, f, comp(v, ax));
        const float w1 = __builtin_fmaf(u.c1, w0, u.c2 * g[ax]);
        const float delta = __builtin_fmaf(u.half_h, w0, u.half_h * w1);
        within &= fabsf(delta) <= most;
        const float h0 = comp(hi, ax), l0 = comp(lo, ax);
        const float y = delta + l0;
        const float t = h0 + y;
        const float bp = t - h0;
        const float ap = t - bp;
        nl[ax] = (h0 - ap) + (y - bp);
        nh[ax] = t;
        nv[ax] = w1;
    }
    if (__builtin_expect(!within, 0))
        *moved = 1u;
    if (!isfinite(nh[0]) || !isfinite(nh[1]) || !isfinite(nh[2]) || !isfinite(nv[0]) ||
        !isfinite(nv[1]) || !isfinite(nv[2]))
        atomicOr(err, ERR_NONFINITE);
    hi = make_float4(nh[0], nh[1], nh[2], hi.w);
    lo = make_float4(nl[0], nl[1], nl[2], lo.w);
    v = make_float4(nv[0], nv[1], nv[2], 0.0f);
}

// The Gaussians (Section III.C) of one residue's step; none if it is fixed.
__device__ __forceinline__ void draw_noise(float (&g)[3], const float4 &hi, long long step, unsigned stream,
                                           const StepConsts &c)
{
    const unsigned tag = __float_as_uint(hi.w);
    if (tag >> 31)
        return;
    const uint4 w = noise_words(tag, stream, step, c);
    const float2 gxy = gaussian_pair(w);
    g[0] = gxy.x;
    g[1] = gxy.y;
    g[2] = gaussian_axis(w, 2);
}

// ---------------------------------------------------------------------------
// Plain schedule, tile staging: at each skin search, the list partners of a
// tile of consecutive residues become a sorted set of at most STAGE_MAX slots,
// and rows are rewritten as 16-bit slots into that set.
// ---------------------------------------------------------------------------
// Slots held in LDS at once by the kernels that read the staging set (12
// bytes each: 21 KiB leave room for five workgroups a CU beside the rings of
// the period's first step); a tile with more slots is taken in windows of
// this many.
template <int NL>
constexpr int stage_win() { return NL == 1 ? 3072 : (NL >= 8 ? 2559 : 1792); }
// Lane-ordered table of bonded/native entries: where there is none the
// partner is the residue itself (so that every entry can be followed); this
// bit beside the partner's id: the pair is out of the fixed-point copies'
// reach until the next rebuild.
constexpr unsigned FAR_ENTRY = 0x80000000u;

// Candidate residues (the residues of the cells around a tile) held in LDS
// at once during a rebuild; more are taken in windows of whole cells.  Small
// tiles keep less so that five workgroups fit a CU.
template <int TILE>
constexpr int cand_win() { return TILE == 64 ? 896 : 1024; }
// Distinct cells around one tile, and the bits of its open-addressing table.
template <int TILE>
constexpr int cells_max() { return TILE >= 256 ? 512 : (TILE >= 128 ? 1024 : 640); }
template <int TILE>
constexpr int chash_bits() { return TILE == 128 ? 11 : 10; }
constexpr int TREG = 8;  // bonded/native entries per residue kept in registers during a search (more: global)

struct BuildArgs {
    const int *tile_first;  // first residue of each tile, then n
    const float4 *pos;
    const int *cell_of;
    const int *count;
    const float4 *cells;
    const int4 *traj_cell;
    const int *traj_lo;
    const int *traj_hi;
    const int2 *trow;
    const float2 *tent;
    int *list_cnt;
    unsigned short *list16;
    int *stage;
    int *stage_cnt;
    unsigned *err;
    const unsigned *skin_flag;
    float4 *hi_skin;
    unsigned long long *stats;
    long long *step_base;  // graph replays: advanced once per rebuild, or NULL
    long long *step_next;
    GridDev g;
    float rc2;
    int n, cap, period;
};

// Exclusive prefix sum over the NT lanes of a workgroup (all lanes call it).
template <int NT>
__device__ __forceinline__ int block_exclusive_scan(int v, int *part, int &total)
{
    const int t = threadIdx.x;
    part[t] = v;
    __syncthreads();
    for (int off = 1; off < NT; off <<= 1) {
        const int x = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += x;
        __syncthreads();
    }
    total = part[NT - 1];
    const int r = part[t] - v;
    __syncthreads();
    return r;
}

// Along one axis of the wrapped grid (n >= 3 cells), cell c is u's own or an
// adjacent one.
__device__ __forceinline__ bool adjacent_cell(int c, int u, int n)
{
    const int d = c - u;
    return (unsigned)(d + 1) <= 2u || d == n - 1 || d == 1 - n;
}

// OR of a 32-bit value over the 64 lanes of a wave.
__device__ __forceinline__ unsigned wave_or(unsigned v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v |= (unsigned)__shfl_xor((int)v, off, 64);
    return v;
}

// One workgroup of NT lanes per tile of TILE consecutive residues; lane t
// serves residue t % TILE and part q = t / TILE of its work (NLB = NT / TILE
// parts).
//  1. The cells around the tile's residues (each residue's own and adjacent
//     cells) go into an LDS hash table and are sorted by cell index; their
//     residues, sorted by (cell, residue index), are the tile's candidates.
//  2. Per window of whole cells (at most cand_win candidates, usually one
//     window): candidates go to LDS; each residue is tested against them 32
//     at a time with the single-precision predicate r < r_list of
//     Algorithm 3, one bit per candidate, part q taking every NLB-th of the
//     32-candidate words (words outside every neighbourhood of a wave are
//     skipped).  Self, bonded and native partners are cleared; the
//     candidates some row uses get the next staging slots in sorted order;
//     each part appends its words' partners to the row at the offset the
//     lower parts leave.
// The order of a row's partners here depends on the number of parts; the
// canonical order that follows does not.
template <int TILE, bool MULTI, int NT>
__global__ __launch_bounds__(NT, NT > 256 ? 4 : (TILE == 64 ? 5 : 2)) void k_tile_build(BuildArgs a)
{
    constexpr int NLB = NT / TILE;
    constexpr int SM = STAGE_MAX;
    constexpr int CM = cand_win<TILE>();
    constexpr int NW = CM / 32;
    constexpr int CELLS_MAX = cells_max<TILE>();
    constexpr int CHASH_BITS = chash_bits<TILE>();
    constexpr int CHASH = 1 << CHASH_BITS;
    static_assert(NW * TILE >= CM, "arrival ids alias the row bits");
    // Step 1 (cell table) and step 2 (candidates, row bits) share one region.
    constexpr int P1 = (CHASH + CELLS_MAX) * 4, P2 = CM * 16 + NW * TILE * 4;
    __shared__ __align__(16) unsigned char shared_region[P1 > P2 ? P1 : P2];
    int *hkey = reinterpret_cast<int *>(shared_region);               // step 1: open addressing
    int *ccell = reinterpret_cast<int *>(shared_region + CHASH * 4);  // step 1: arrival order
    float4 *cand = reinterpret_cast<float4 *>(shared_region);         // step 2: window, sorted
    unsigned *bits = reinterpret_cast<unsigned *>(shared_region + CM * 16);  // row bits, word-major
    __shared__ unsigned sxyz[CELLS_MAX];  // sorted cells: packed coordinates
    __shared__ int cbase[CELLS_MAX + 1];
    __shared__ unsigned used[NW];
    __shared__ int wbase[NW];
    __shared__ short wlo[NW], whi[NW];    // sorted cells spanned by each word
    __shared__ short pcnt[NT];            // partners of (part, residue) in this window
    __shared__ int rowbase[TILE];         // partners of the residue in earlier windows
    __shared__ int part[NT];
    __shared__ int n_cu, bad_cells, n_used_w;

    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // every rebuild starts here (the kernels after it do not read these)
        ++a.stats[0];
        a.err[MOVED] = a.err[MOVED + 1] = 0u;
        if (a.step_base) {
            // graph replays: this rebuild starts the next list period
            const long long nb = *a.step_next;
            *a.step_base = nb;
            *a.step_next = nb + a.period;
        }
    }
    if (*a.skin_flag == 0u)
        return;  // the skin rows are still valid (uniform over the grid)
    const int tile = blockIdx.x, t = threadIdx.x;
    const int rho = t % TILE, q = t / TILE;
    const int first = a.tile_first[tile], tcnt = a.tile_first[tile + 1] - first;
    const int i = first + rho;
    const bool act = rho < tcnt;
    const bool lead = act && q == 0;  // writes the residue's count
    const GridDev g = a.g;
    if (tile == 0 && t == 0)
        ++a.stats[1];
    if (lead)
        a.hi_skin[i] = a.pos[2 * i];  // the displacement check's reference
    for (int h = t; h < CHASH; h += NT)
        hkey[h] = -1;
    if (t < TILE)
        rowbase[t] = 0;
    if (t == 0) {
        n_cu = 0;
        bad_cells = 0;
    }
    __syncthreads();

    auto hslot = [](int key) { return (int)(((unsigned)key * 2654435761u) >> (32 - CHASH_BITS)); };

    // ---- 1. cells around the tile ----
    // independent loads first; this part's bonded/native entries (u = q mod
    // NLB, the first ones kept in registers) and their partners' cells are
    // needed only in step 2
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
    int own = 0;
    int2 row = make_int2(0, 0);
    if (act) {
        p = a.pos[2 * i];
        own = a.cell_of[i];
        row = a.trow[i];
    }
    const int ntop = (row.y & 4095) + (row.y >> 12);
    // entry e = v * NLB + q, e < TPP * NLB, is this part's v-th
    constexpr int TPP = TREG > NLB ? TREG / NLB : 1;
    int tj[TPP], tm[TPP];
#pragma unroll
    for (int v = 0; v < TPP; ++v) {
        const int e = v * NLB + q;
        const float2 te = e < ntop ? a.tent[row.x + e] : make_float2(0.0f, 0.0f);
        tj[v] = __float_as_int(te.x);
    }
#pragma unroll
    for (int v = 0; v < TPP; ++v)
        tm[v] = v * NLB + q < ntop ? a.cell_of[tj[v]] : -1;
    const int tlo = (MULTI && act) ? a.traj_lo[i] : 0, thi = (MULTI && act) ? a.traj_hi[i] : 0;
    // own wrapped cell coordinates
    const int ux = own % g.gx, uy = (own / g.gx) % g.gy, uz = own / (g.gx * g.gy);
    // one lane of those in one cell enters its neighbours: the lanes of a wave
    // share a dozen cells, and LDS serves atomics on one address one by one
    bool enters = act;
    for (unsigned long long todo = __ballot(act); todo;) {
        const int l = __ffsll((long long)todo) - 1;
        const bool same = act && own == __shfl(own, l);
        enters &= !(same && (int)__lane_id() != l);
        todo &= ~__ballot(same);
    }
    if (enters) {
        for (int d = q; d < 27; d += NLB) {
            const int cx = ux + d % 3 - 1, cy = uy + (d / 3) % 3 - 1, cz = uz + d / 9 - 1;
            const int cid = (cx < 0 ? cx + g.gx : (cx >= g.gx ? cx - g.gx : cx)) +
                            g.gx * ((cy < 0 ? cy + g.gy : (cy >= g.gy ? cy - g.gy : cy)) +
                                    g.gy * (cz < 0 ? cz + g.gz : (cz >= g.gz ? cz - g.gz : cz)));
            int h = hslot(cid);
            for (int probe = 0; probe < CHASH; ++probe) {
                const int prev = atomicCAS(&hkey[h], -1, cid);
                if (prev == -1) {
                    const int m = atomicAdd(&n_cu, 1);
                    if (m < CELLS_MAX)
                        ccell[m] = cid;
                    else
                        bad_cells = 1;
                    break;
                }
                if (prev == cid)
                    break;
                h = (h + 1) & (CHASH - 1);
                if (probe == CHASH - 1)
                    bad_cells = 1;
            }
        }
    }
    __syncthreads();
    auto fail_tile = [&]() {
        // report; leave the tile with no slots and no partners
        if (t == 0) {
            atomicOr(a.err, ERR_STAGE);
            a.stage_cnt[tile] = 0;
        }
        if (lead)
            a.list_cnt[i] = 0;
    };
    if (bad_cells) {
        fail_tile();
        return;  // uniform: read after a barrier, written only before it
    }
    const int NC = n_cu;
    // coordinates packed in bx + by + bz <= 32 bits (the grid has at most 2^21 cells)
    const int bx = 32 - __clz(g.gx), by = 32 - __clz(g.gy);
    const unsigned mx = (1u << bx) - 1u, my = (1u << by) - 1u;
    auto cell_id = [&](unsigned v) { return (int)(v & mx) + g.gx * ((int)((v >> bx) & my) + g.gy * (int)(v >> (bx + by))); };
    // sort the cells by index (rank by counting; indices are distinct)
    for (int m = t; m < NC; m += NT) {
        const int c = ccell[m];
        int r = 0;
        for (int m2 = 0; m2 < NC; ++m2)
            r += ccell[m2] < c;
        sxyz[r] = (unsigned)(c % g.gx) | ((unsigned)((c / g.gx) % g.gy) << bx) |
                  ((unsigned)(c / (g.gx * g.gy)) << (bx + by));
    }
    __syncthreads();
    auto lookup = [&](int key) -> int {  // sorted number of cell `key`, or -1
        int lo = 0, hi = NC;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cell_id(sxyz[mid]) < key)
                lo = mid + 1;
            else
                hi = mid;
        }
        return (lo < NC && cell_id(sxyz[lo]) == key) ? lo : -1;
    };
    // candidate counts -> cbase (exclusive prefix in sorted cell order)
    {
        const int cper = (NC + NT - 1) / NT;
        const int m0 = min(NC, t * cper), m1 = min(NC, m0 + cper);
        int csum = 0;
        for (int m = m0; m < m1; ++m) {
            const int c = min(a.count[cell_id(sxyz[m])], CELL_CAP);
            cbase[m] = c;
            csum += c;
        }
        int M = 0;
        int cb = block_exclusive_scan<NT>(csum, part, M);
        for (int m = m0; m < m1; ++m) {
            const int c = cbase[m];
            cbase[m] = cb;
            cb += c;
        }
        if (t == 0)
            cbase[NC] = M;
    }
    __syncthreads();
    // partners' cells -> sorted cell numbers (or -1 outside the tile's cells)
#pragma unroll
    for (int v = 0; v < TPP; ++v)
        tm[v] = tm[v] >= 0 ? lookup(tm[v]) : -1;
    const int own_m = lead ? lookup(own) : -1;
    auto segment_of = [&](int ci) {  // last m with cbase[m] <= ci
        int lo = 0, hi = NC;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (cbase[mid] <= ci)
                lo = mid;
            else
                hi = mid;
        }
        return lo;
    };

    // ---- 2. windows of whole cells ----
    int *st = a.stage + (size_t)tile * SM;
    unsigned short *lrow = a.list16 + (size_t)i * a.cap;  // rows are residue-major
    auto row_store = [&](int k, unsigned short sl) {  // entry k of the residue's row
        if (k < a.cap)
            lrow[k] = sl;
    };
    int slot_base = 0;
    int *aid = reinterpret_cast<int *>(bits);
    for (int mA = 0; mA < NC;) {
        int mB = mA + 1;  // a cell holds at most CELL_CAP <= CM residues
        {
            int hi = NC;
            while (mB < hi) {
                const int mid = (mB + hi + 1) >> 1;
                if (cbase[mid] - cbase[mA] <= CM)
                    mB = mid;
                else
                    hi = mid - 1;
            }
        }
        const int base = cbase[mA], Mw = cbase[mB] - base;
        constexpr int CPT = (CM + NT - 1) / NT;  // candidates per lane
        float4 cv[CPT];
        int cm[CPT];
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const int ci = t + u * NT;
            cm[u] = ci < Mw ? segment_of(base + ci) : 0;
            cv[u] = ci < Mw ? a.cells[(size_t)cell_id(sxyz[cm[u]]) * CELL_CAP + (base + ci - cbase[cm[u]])]
                            : make_float4(0.f, 0.f, 0.f, 0.f);
            if (ci < Mw)
                aid[ci] = __float_as_int(cv[u].w);
        }
        for (int w = t; w < NW; w += NT)
            used[w] = 0u;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const int ci = t + u * NT;
            if (ci < Mw) {
                const int id = __float_as_int(cv[u].w);
                const int k0 = cbase[cm[u]] - base, k1 = cbase[cm[u] + 1] - base;
                int r = k0, k = k0;
                for (; k + 4 <= k1; k += 4) {
                    const int a0 = aid[k], a1 = aid[k + 1], a2 = aid[k + 2], a3 = aid[k + 3];
                    r += (a0 < id) + (a1 < id) + (a2 < id) + (a3 < id);
                }
                for (; k < k1; ++k)
                    r += aid[k] < id;
                cand[r] = cv[u];
            }
        }
        const int NWm = (Mw + 31) >> 5;
        for (int w = t; w < NWm; w += NT) {
            wlo[w] = (short)segment_of(base + 32 * w);
            whi[w] = (short)segment_of(base + min(32 * w + 31, Mw - 1));
        }
        __syncthreads();
        // row bits; part q (uniform over a wave) takes every NLB-th word, as
        // partners lie in few neighbouring ones
        for (int w = q; w < NWm; w += NLB) {
            bool reach = false;
            if (act)
                for (int m = wlo[w]; m <= whi[w]; ++m) {
                    const unsigned v = sxyz[m];
                    reach |= adjacent_cell((int)(v & mx), ux, g.gx) &&
                             adjacent_cell((int)((v >> bx) & my), uy, g.gy) &&
                             adjacent_cell((int)(v >> (bx + by)), uz, g.gz);
                }
            unsigned word = 0u;
            if (__any(reach)) {
                // branch-free: BB LDS reads in flight, then the tests; the
                // window's tail and inactive lanes are masked afterwards
                constexpr int BB = TILE == 64 ? 4 : 8;
#pragma unroll 1
                for (int k0 = 0; k0 < 32; k0 += BB) {
                    float4 c8[BB];
#pragma unroll
                    for (int u = 0; u < BB; ++u)
                        c8[u] = cand[32 * w + k0 + u];
#pragma unroll
                    for (int u = 0; u < BB; ++u) {
                        bool pass = within_cutoff(p, c8[u], a.rc2);
                        if (MULTI) {
                            const int j = __float_as_int(c8[u].w);
                            pass = pass & (j >= tlo) & (j < thi);
                        }
                        word |= (unsigned)pass << (k0 + u);
                    }
                }
                const int left = Mw - 32 * w;
                word &= act ? (left >= 32 ? 0xffffffffu : ((1u << left) - 1u)) : 0u;
                const unsigned u = wave_or(word);
                if ((t & 63) == 0 && u)
                    atomicOr(&used[w], u);
            }
            bits[w * TILE + rho] = word;
        }
        __syncthreads();
        // self, bonded and native partners in this window: clear their bits
        auto find = [&](int j, int m) -> int {  // window candidate of residue j in sorted cell m, or -1
            if (m < mA || m >= mB)
                return -1;
            int lo = cbase[m] - base, hi = cbase[m + 1] - base;
            const int end = hi;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (__float_as_int(cand[mid].w) < j)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            return (lo < end && __float_as_int(cand[lo].w) == j) ? lo : -1;
        };
        auto drop = [&](int r) {
            if (r >= 0)
                atomicAnd(&bits[(r >> 5) * TILE + rho], ~(1u << (r & 31)));
        };
        if (lead)
            drop(find(i, own_m));
        if (act)
            for (int e = TPP * NLB + q; e < ntop; e += NLB) {
                const int j = __float_as_int(a.tent[row.x + e].x);
                drop(find(j, lookup(a.cell_of[j])));
            }
#pragma unroll
        for (int v = 0; v < TPP; ++v)
            if (v * NLB + q < ntop)
                drop(find(tj[v], tm[v]));
        __syncthreads();
        // slots of the used candidates: prefix over the window's words (<= 32);
        // row counts of each part
        if (t < 64) {
            const int c = t < NWm ? __popc(used[t]) : 0;
            int v = c;
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(v, off, 64);
                if (t >= off)
                    v += y;
            }
            if (t < NWm)
                wbase[t] = slot_base + v - c;
            if (t == 63)
                n_used_w = v;
        }
        {
            int c = 0;
            for (int w = q; w < NWm; w += NLB)
                c += __popc(bits[w * TILE + rho]);
            pcnt[t] = (short)c;
        }
        __syncthreads();
        const int nu = n_used_w;
        if (slot_base + nu > SM) {
            fail_tile();
            return;  // uniform
        }
        // staging: each used candidate of the window takes the next slot in
        // sorted order (all lanes, one candidate each)
        for (int ci = t; ci < Mw; ci += NT) {
            const unsigned uw = used[ci >> 5];
            if ((uw >> (ci & 31)) & 1u)
                st[wbase[ci >> 5] + __popc(uw & ((1u << (ci & 31)) - 1u))] = __float_as_int(cand[ci].w);
        }
        if (act) {
            // this part's partners, after those of the lower parts
            int k = rowbase[rho];
            for (int pq = 0; pq < q; ++pq)
                k += pcnt[pq * TILE + rho];
            for (int w = q; w < NWm; w += NLB) {
                unsigned b = bits[w * TILE + rho];
                const unsigned uw = used[w];
                const int wb = wbase[w];
                while (b) {
                    const int kb = __ffs(b) - 1;
                    b &= b - 1u;
                    row_store(k++, (unsigned short)(wb + __popc(uw & ((1u << kb) - 1u))));
                }
            }
        }
        slot_base += nu;
        mA = mB;
        __syncthreads();  // the window's buffers are reused
        if (lead) {
            int c = rowbase[rho];
            for (int pq = 0; pq < NLB; ++pq)
                c += pcnt[pq * TILE + rho];
            rowbase[rho] = c;
        }
    }

    if (t == 0)
        a.stage_cnt[tile] = slot_base;
    if (!lead)
        return;
    const int cnt = rowbase[rho];
    a.list_cnt[i] = cnt;
    if (cnt > a.cap)
        atomicOr(a.err, ERR_OVERFLOW);
}

// ---------------------------------------------------------------------------
// List from the skin rows: every list_every steps each lane's skin entries
// (the partners of its residue within r_list + skin at the last skin build
// that were dealt to it, in slot order) are filtered with the
// single-precision predicate r < r_list of Algorithm 3 on the current
// positions.  The skin build runs again before the filter whenever some
// residue has moved more than skin/2 since the last one, so every pair within
// r_list is in the skin rows and the filtered rows equal a rebuild from all
// pairs, entry for entry in the same order.
// ---------------------------------------------------------------------------
struct FilterArgs {
    const int *tile_first;
    const float4 *pos;
    const int *stage;
    const int *stage_cnt;
    const uint4 *skin16;             // pieces of 8 entries, lane order
    const unsigned short *skin_len;  // entries of each lane
    const unsigned short *skin_ord;  // per tile: 1 + its residues by decreasing skin row length
    uint2 *ltop;
    const int4 *tile_top;
    uint2 *list16;                   // chunks of 4 entries, lane order
    unsigned short *llen;
    unsigned char *grho;
    WgRec *wg_rec;
    int *cell_count;
    unsigned *skin_flag;
    const int4 *fixed;               // k_filter: fixed-point copies of the positions
    unsigned *place;
    FixDev fix;
    float rc2;
    int cap, n_cells, top_rounds;
};

// Residues of a workgroup, workgroups of a tile and LDS of the kernels that
// work in lane order (NL lanes a residue).
template <int TILE, int NL>
struct Rows {
    static constexpr int RW = 256 / NL, W = TILE / RW;
    static constexpr int SW = stage_win<NL>();
    static constexpr int XS = SW + 1;   // stride of the axes; slot SW is far away
    static constexpr int BYTES = XS * 12;
    static constexpr int NPRE = 6;      // list chunks a lane keeps in registers
    static constexpr int RING = 16;     // passing entries of a lane on their way to memory
};

// Residue of group r of a tile (r < tcnt): the order of the last skin search.
__device__ __forceinline__ int ranked(const unsigned short *ord, size_t at, int r)
{
    const int o = ord[at];
    return o > 0 ? o - 1 : r;
}

// What holds for a workgroup until the next rebuild: it has a FAR_ENTRY; the
// tile's residues do not fit a cube of 2 FixDev::narrow.  Within `narrow` of
// the cube's centre (the origin) on every axis, neither the tile's residues
// nor their list partners wrap (fix_consts), and positions relative to the
// origin, all within half a period, are rounded once to single precision: list
// pairs are separated to half a unit in the last place of it (at r_list = 20 A
// 64 A: about 8e-6 A at most).  Other tiles subtract the copies themselves.
// Origin and test depend on the tile's own residues only, neither on which
// other residues are staged nor on how the tile's are dealt to workgroups.
constexpr int WG_FAR = 1, WG_WIDE = 2;
constexpr int WG_IDS32 = 4;  // the tile's slot ids do not fit stage16

// Beside a lane's skin entries: its residue's row is dealt in turn.
constexpr int SKIN_TURN = 0x8000;

// Filters the skin entries of every lane of a workgroup; returns the number
// of list entries of this lane, and the workgroup's record.  Every lane of a
// wave gets as many chunks as the wave's longest, padded with the far-away
// slot (whose term is exactly zero), so the sums run without lane masks.  Each lane tests
// its own entries and appends those that pass to its own list row, so nothing
// crosses lanes: 13 vector instructions and 3 LDS accesses an entry, where
// rows compacted across a residue's lanes took 40.  An entry goes to the
// lane's ring in LDS whether it passes or not, and stays if it does; whole
// chunks leave for memory, and padding does not pass the ring.  Bound by LDS
// accesses in the entries and by two rounds of loads before them; with those
// loads one after the other and padding through the ring the kernel of the
// filter alone took (us, with two early exits before it) 71 -> 62 at 250,000
// residues, 27 -> 24 at 75,000, 13.0 -> 11.5 at 4,801 at protein density.
template <int TILE, int NL>
__device__ __forceinline__ int filter_rows(const FilterArgs &a, int wg, int tile, int t, int first, int tcnt, int rho,
                                           unsigned char *region, unsigned short *ring, float *bb, WgRec &wr)
{
    using R = Rows<TILE, NL>;
    constexpr int SM = STAGE_MAX;
    constexpr int SW = R::SW, XS = R::XS;
    const int i = first + rho;
    float *hx = reinterpret_cast<float *>(region);
    const int S = min(a.stage_cnt[tile], SM);
    const int *st = a.stage + (size_t)tile * SM;
    const int4 top = a.tile_top[tile];
    const int chunks = lane_chunks(a.cap, NL);
    const uint4 *src = a.skin16 + (size_t)wg * (chunks / 2) * 256 + t;
    uint2 *dst = a.list16 + (size_t)wg * chunks * 256 + t;
    const int own = a.skin_len[wg * 256 + t];
    const bool turn = (own & SKIN_TURN) != 0;
    const int len = turn ? 0 : own;
    const int np = (len + 7) >> 3;
    // straight-line loads (the first STAGE_MIN slots and TOP_MIN rounds are
    // there for any tile): ids and entries first, then all their positions
    constexpr int PER = STAGE_MIN / 256;
    int ids[PER];
    unsigned te[TOP_MIN];
    uint2 *tp = a.ltop + top_index(wg, 0, t, a.top_rounds);
#pragma unroll
    for (int u = 0; u < PER; ++u)
        ids[u] = st[t + u * 256];
#pragma unroll
    for (int r = 0; r < TOP_MIN; ++r)
        te[r] = tp[r * 256].x;
    uint4 next = src[0];
    const float4 pi = a.pos[2 * i];
    const float4 pb = a.pos[2 * (first + min(t, tcnt - 1))];
    float4 hs[PER], ht[TOP_MIN];
#pragma unroll
    for (int u = 0; u < PER; ++u)
        hs[u] = a.pos[2 * ids[u]];
#pragma unroll
    for (int r = 0; r < TOP_MIN; ++r)
        ht[r] = a.pos[2 * (te[r] & ~FAR_ENTRY)];
    auto put = [&](int sl, const float4 &h) {
        hx[sl] = h.x;
        hx[XS + sl] = h.y;
        hx[2 * XS + sl] = h.z;
    };
    auto stage_window = [&](int w0, int sl0, int wn) {
        for (int sl = sl0 + t; sl < wn; sl += 256)
            put(sl, a.pos[2 * st[w0 + sl]]);
    };
#pragma unroll
    for (int u = 0; u < PER; ++u)
        put(t + u * 256, hs[u]);
    stage_window(0, STAGE_MIN, min(SW, S));
    if (t < 3)
        hx[t * XS + SW] = 1.0e18f;
    // bonded and native partners beyond the reach of the fixed-point copies
    bool far = false;
    int rounds = 0;  // that this wave has entries in
    auto reach = [&](int r, unsigned j, const float4 &h) {
        if (j != (unsigned)i) {
            const bool out = !(fmaxf(fabsf(h.x - pi.x), fmaxf(fabsf(h.y - pi.y), fabsf(h.z - pi.z))) <= a.fix.reach);
            far |= out;
            if (out != (j >= FAR_ENTRY))
                tp[r * 256].x = j ^ FAR_ENTRY;
        }
        if (__any(j != (unsigned)i))
            rounds = r + 1;
    };
#pragma unroll
    for (int r = 0; r < TOP_MIN; ++r)
        reach(r, te[r], ht[r]);
    for (int r = TOP_MIN; r < top.x + top.y; ++r) {
        const unsigned j = tp[r * 256].x;
        reach(r, j, a.pos[2 * (j & ~FAR_ENTRY)]);
    }
    // the box of the tile's residues, 64 to a wave
    if (t < TILE) {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            float mn = comp(pb, ax), mx = mn;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                mn = fminf(mn, __shfl_xor(mn, off));
                mx = fmaxf(mx, __shfl_xor(mx, off));
            }
            if ((t & 63) == 0) {
                bb[(t >> 6) * 6 + ax] = mn;
                bb[(t >> 6) * 6 + 3 + ax] = mx;
            }
        }
    }
    int flags = __syncthreads_or(far ? 1 : 0) ? WG_FAR : 0;
    {
        float o[3], half = 0.0f;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            float lo = bb[ax], hi = bb[3 + ax];
#pragma unroll
            for (int w = 1; w < TILE / 64; ++w) {
                lo = fminf(lo, bb[6 * w + ax]);
                hi = fmaxf(hi, bb[6 * w + 3 + ax]);
            }
            o[ax] = 0.5f * lo + 0.5f * hi;
            half = fmaxf(half, fmaxf(hi - o[ax], o[ax] - lo));
        }
        if (!(half < a.fix.narrow))
            flags |= WG_WIDE;
        if (!top.w)
            flags |= WG_IDS32;
        const int4 q = fix_pos(make_float4(o[0], o[1], o[2], 0.0f), make_float4(0.0f, 0.0f, 0.0f, 0.0f), a.fix);
        wr = WgRec{q.x, q.y, q.z, flags,
                   first, tcnt, S, top.z, {0, 0, 0, 0}, {0, 0, 0, 0}};
    }
    // counts of passing and of written entries, times 512: entry c of the
    // lane's row is at ring[(c mod 16) 256 + t]
    unsigned c9 = 0u, f9 = 0u;
    const unsigned t2 = 2u * (unsigned)t;
    char *rg = reinterpret_cast<char *>(ring);
    auto at = [&](unsigned k9) -> unsigned short & {
        return *reinterpret_cast<unsigned short *>(rg + ((k9 & (unsigned)(512 * (R::RING - 1))) | t2));
    };
    constexpr unsigned PAD = 4u * (unsigned)SW;
    auto flush = [&]() {
        const unsigned e0 = at(f9), e1 = at(f9 + 512u), e2 = at(f9 + 1024u), e3 = at(f9 + 1536u);
        dst[(size_t)(f9 >> 11) * 256] = make_uint2(e0 | (e1 << 16), e2 | (e3 << 16));
        f9 += 2048u;
    };
    // one piece: its entries that pass, and for which `ok` holds, are appended
    auto piece = [&](const uint4 &w, auto ok) {
        const unsigned ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int h = 0; h < 8; h += 4) {  // four reads in flight, then their tests
            unsigned e[4];
            float4 pj[4];
            bool use[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                e[u] = (ws[(h + u) >> 1] >> ((u & 1) * 16)) & 0xffffu;
                unsigned o = e[u];
                use[u] = ok(h + u, o);
                const float *p = reinterpret_cast<const float *>(region + o);
                pj[u] = make_float4(p[0], p[XS], p[2 * XS], 0.0f);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                at(c9) = (unsigned short)e[u];
                c9 += within_cutoff(pi, pj[u], a.rc2) && use[u] ? 512u : 0u;
            }
        }
        while (c9 - f9 >= 2048u)
            flush();
    };
    if (S <= SW) {
        // one window (nearly every tile): entries past the row's end are the
        // far-away slot
        for (int p = 0; p < np; ++p) {
            const uint4 w = next;
            next = src[(size_t)min(p + 1, np - 1) * 256];
            piece(w, [](int, unsigned &) { return true; });
        }
    } else {
        // window by window: the entries ascend, so a lane goes on where the
        // window before ended
        int p = 0;
        for (int w0 = 0; w0 < S; w0 += SW) {
            const int wn = min(SW, S - w0);
            if (w0 > 0) {
                __syncthreads();  // the previous window's readers are done
                stage_window(w0, 0, wn);
                __syncthreads();
            }
            while (p < np) {
                const uint4 w = src[(size_t)p * 256];
                const int valid = len - 8 * p;
                unsigned last = 0u;
                piece(w, [&](int u, unsigned &o) {
                    if (u < valid)
                        last = o;
                    o -= 4u * (unsigned)w0;
                    const bool ok = u < valid && o < 4u * (unsigned)wn;
                    o = ok ? o : 0u;
                    return ok;
                });
                if (last >= 4u * (unsigned)(w0 + wn))
                    break;  // the rest of the piece is in a later window
                ++p;
            }
        }
    }
    if (__builtin_expect(turn, 0)) {
        // a skin row dealt in turn: each lane walks the residue's whole row, in
        // ascending order, for what it has of the list: its class, or where one
        // class is more than a lane holds, in turn.  So also here the list
        // alone decides which lane sums a partner.
        const int q = t % NL, cap_lane = 8 * (chunks / 2);
        int row = own & ~SKIN_TURN;
#pragma unroll
        for (int off = 1; off < NL; off <<= 1)
            row += __shfl_xor(row, off, NL);
        const unsigned short *sk = reinterpret_cast<const unsigned short *>(src) - 8 * q;
        auto walk = [&](auto f) {  // f(entry, id) of every partner in the list
#pragma unroll 1
            for (int k = 0; k < row; ++k) {
                const int e = k / NL;
                const unsigned v = sk[((size_t)(e >> 3) * 256 + k % NL) * 8 + (e & 7)];
                const int id = st[v >> 2];
                if (within_cutoff(pi, a.pos[2 * id], a.rc2))
                    f(v, id);
            }
        };
        int most = 0;
        walk([&](unsigned, int id) { most += (id & (NL - 1)) == q ? 1 : 0; });
#pragma unroll
        for (int off = 1; off < NL; off <<= 1)
            most = max(most, __shfl_xor(most, off, NL));
        int rank = 0;
        walk([&](unsigned v, int id) {
            if ((most > cap_lane ? rank : id) % NL == q) {
                at(c9) = (unsigned short)v;
                c9 += 512u;
                if (c9 - f9 >= 2048u)
                    flush();
            }
            ++rank;
        });
    }
    const int m = (int)(c9 >> 9);
    int nk = (m + 3) >> 2;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
        nk = max(nk, __shfl_xor(nk, off));
    int kp = (int)(f9 >> 11);
    if (kp < nk) {
        // at most three entries are left in the ring; then nothing but padding
        const unsigned e0 = at(f9), e1 = at(f9 + 512u), e2 = at(f9 + 1024u);
        const int left = m & 3;
        dst[(size_t)kp * 256] = make_uint2((left > 0 ? e0 : PAD) | (left > 1 ? e1 : PAD) << 16,
                                           (left > 2 ? e2 : PAD) | PAD << 16);
        while (++kp < nk)
            dst[(size_t)kp * 256] = make_uint2(PAD | PAD << 16, PAD | PAD << 16);
    }
    a.llen[wg * 256 + t] = (unsigned short)m;
    if (t % NL == 0)
        a.grho[wg * R::RW + t / NL] = (unsigned char)rho;
    const int wave = nk | (min(top.x, rounds) << 16) | (rounds << 24);
    int *wv = reinterpret_cast<int *>(bb);
    __syncthreads();  // the box has been read, the staged positions too
    if ((t & 63) == 0)
        wv[t >> 6] = wave;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k)
        wr.waves[k] = wv[k];
    if (t == 0)
        a.wg_rec[wg] = wr;
    return m;
}

template <int TILE, int NL>
__global__ __launch_bounds__(256, NL == 1 ? 2 : 5) void k_filter(FilterArgs a)
{
    using R = Rows<TILE, NL>;
    __shared__ __align__(16) unsigned char region[R::BYTES];
    __shared__ unsigned short ring[R::RING * 256];
    __shared__ float bb[24];
    const int wg = blockIdx.x, t = threadIdx.x;
    const int tile = wg / R::W, part = wg % R::W;
    // the cell counts are read only by the skin build, which is done: clear
    // them for the next one; the flag is read only by the skin build too
    for (int k = wg * 256 + t; k < a.n_cells; k += gridDim.x * 256)
        a.cell_count[k] = 0;
    if (wg == 0 && t == 0)
        *a.skin_flag = 0u;
    const int first = a.tile_first[tile], tcnt = a.tile_first[tile + 1] - first;
    // the residue of this lane group: rows longest first
    const int r = t / NL * R::W + part;
    const bool in = r < tcnt;
    const int rho = in ? ranked(a.skin_ord, (size_t)tile * TILE + r, r) : 0;
    if (!a.fix.by_step && in && t % NL == 0)
        a.place[first + rho] = fix_place(a.fixed[first + rho]);
    WgRec wr;
    filter_rows<TILE, NL>(a, wg, tile, t, first, tcnt, rho, region, ring, bb, wr);
}

// ---------------------------------------------------------------------------
// Canonical order after a skin search: a tile's slots are renumbered in the
// order of their residues' global ids, and every skin row is dealt to its
// residue's lanes by partner id, in ascending order, whatever the cell grid.
// The list rows the filter derives keep that order (a row that has to be dealt
// in turn it deals anew), so the order in which a residue's pair terms are
// summed depends on its list alone, not on when or with which skin the last
// search ran.
// ---------------------------------------------------------------------------
struct CanonArgs {
    const int *tile_first;
    const int2 *trow;
    const int *stage_raw;
    int *stage;
    const int *stage_cnt;
    const unsigned short *rows;  // the search's rows, by residue
    const int *skin_cnt;
    const float2 *tent;
    const unsigned *skin_flag;
    uint4 *skin16;
    unsigned short *skin_len;
    unsigned short *skin_ord;
    uint2 *ltop;
    int4 *tile_top;
    unsigned short *stage16;
    int cap, top_rounds;
};

template <int TILE, int NL>
__global__ __launch_bounds__(256) void k_canon(CanonArgs a)
{
    using R = Rows<TILE, NL>;
    constexpr int RW = R::RW, W = R::W;
    constexpr int SM = STAGE_MAX;
    constexpr int MW = SM / 32;     // mask words per row, at most
    constexpr int BW = 2048;        // bitmap words: ids spanning up to 65,536 values
    // the ranks (bitmap and word prefixes, or the ids) and the masks use one
    // region in turn, so that five workgroups fit a CU (with ids, bitmap and
    // prefixes side by side three: 75,000 residues 68 against 44 us, 250,000
    // 200 against 148)
    constexpr int WORDS = SM > NL * MW + 8 * (MW + 1) ? SM : NL * MW + 8 * (MW + 1);
    static_assert(WORDS >= BW + BW / 2, "bitmap and 16-bit prefixes");
    __shared__ unsigned region[WORDS];
    int *sid = reinterpret_cast<int *>(region);
    unsigned *bmp = region;
    unsigned short *wpre = reinterpret_cast<unsigned short *>(region + BW);
    __shared__ unsigned short nslot[SM];
    __shared__ unsigned char cls[SM];
    __shared__ short slen[TILE], sord[TILE];
    __shared__ int part[256];
    __shared__ int id_lo, id_hi;
    if (*a.skin_flag == 0u)
        return;  // no search ran (uniform over the grid)
    const int wg = blockIdx.x, tile = wg / W, w = wg % W, t = threadIdx.x;
    const int first = a.tile_first[tile], tcnt = a.tile_first[tile + 1] - first;
    const int S = min(a.stage_cnt[tile], SM);
    const int *raw = a.stage_raw + (size_t)tile * SM;
    int *st = a.stage + (size_t)tile * SM;
    if (t == 0) {
        id_lo = 0x7fffffff;
        id_hi = -1;
    }
    __syncthreads();
    {
        int mn = 0x7fffffff, mx = -1;
        for (int k = t; k < S; k += 256) {
            const int id = raw[k];
            mn = min(mn, id);
            mx = max(mx, id);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {  // one atomic a wave
            mn = min(mn, __shfl_xor(mn, off));
            mx = max(mx, __shfl_xor(mx, off));
        }
        if ((t & 63) == 0) {
            atomicMin(&id_lo, mn);
            atomicMax(&id_hi, mx);
        }
    }
    __syncthreads();
    // new slot = rank of the residue id among the tile's slots (ids distinct):
    // from a bitmap of the ids when they span few enough values, else by
    // counting
    const int lo = id_lo, span = id_hi - id_lo + 1;
    if (S > 0 && span <= 32 * BW) {
        const int nw = (span + 31) >> 5;
        for (int w = t; w < nw; w += 256)
            bmp[w] = 0u;
        __syncthreads();
        for (int k = t; k < S; k += 256)
            atomicOr(&bmp[(raw[k] - lo) >> 5], 1u << ((raw[k] - lo) & 31));
        __syncthreads();
        constexpr int WPL = BW / 256;
        int c = 0;
        for (int w = t * WPL; w < min(nw, (t + 1) * WPL); ++w)
            c += __popc(bmp[w]);
        int total = 0;
        int o = block_exclusive_scan<256>(c, part, total);
        for (int w = t * WPL; w < min(nw, (t + 1) * WPL); ++w) {
            wpre[w] = (unsigned short)o;
            o += __popc(bmp[w]);
        }
        __syncthreads();
        for (int k = t; k < S; k += 256) {
            const int v = raw[k] - lo;
            nslot[k] = (unsigned short)(wpre[v >> 5] + __popc(bmp[v >> 5] & ((1u << (v & 31)) - 1u)));
        }
    } else {
        for (int k = t; k < S; k += 256)
            sid[k] = raw[k];
        __syncthreads();
        for (int k = t; k < S; k += 256) {
            const int id = sid[k];
            int r = 0;
            for (int m = 0; m < S; ++m)
                r += sid[m] < id ? 1 : 0;
            nslot[k] = (unsigned short)r;
        }
    }
    __syncthreads();
    for (int k = t; k < S; k += 256) {
        const int id = raw[k], ns = nslot[k];
        cls[ns] = (unsigned char)(id & (NL - 1));
        if (w == 0) {
            st[ns] = id;
            a.stage16[(size_t)tile * SM + ns] = (unsigned short)(id - lo);
        }
    }
    if (w == 0) {
        for (int k = S + t; k < max((S + 255) & ~255, STAGE_MIN); k += 256) {
            st[k] = S > 0 ? lo : first;
            a.stage16[(size_t)tile * SM + k] = 0;
        }
    }
    // the rows are handed to the waves longest first, so that the rows of a
    // wave have about the same length (ties in index order)
    if (t == 0)
        id_lo = id_hi = 0;  // most bonded / native entries of a residue
    for (int u = t; u < tcnt; u += 256)
        slen[u] = (short)min(a.skin_cnt[first + u], a.cap);
    __syncthreads();  // the ids are dead: the region takes the masks
    for (int u = t; u < tcnt; u += 256) {
        const int L = slen[u];
        int r = 0;
        for (int v = 0; v < tcnt; ++v)
            r += (slen[v] > L || (slen[v] == L && v < u)) ? 1 : 0;
        if (w == 0)
            a.skin_ord[(size_t)tile * TILE + r] = (unsigned short)(u + 1);
        sord[r] = (short)u;
        const int2 rw = a.trow[first + u];
        atomicMax(&id_lo, rw.y & 4095);
        atomicMax(&id_hi, rw.y >> 12);
    }
    // slots of each class (id modulo NL), as masks
    const int nw = (S + 31) >> 5, ms = nw | 1;  // mask words of a row, their stride (odd: neighbours in other banks)
    unsigned *cmask = region, *mask = region + NL * nw;
    for (int x = t; x < nw * NL; x += 256) {
        const int v = x / NL, c = x % NL;
        unsigned m = 0u;
        for (int b = 0; b < 32; ++b)
            m |= (32 * v + b < S && cls[32 * v + b] == c) ? 1u << b : 0u;
        cmask[c * nw + v] = m;
    }
    const int chunks = lane_chunks(a.cap, NL);
    const int cap_lane = 8 * (chunks / 2);  // entries of a lane that its chunks hold
    const int g = t / NL, q = t % NL;
    // rows of this workgroup held as masks at a time (all of them, unless the
    // tile stages nearly as many slots as it may)
    const int G = min(RW, (WORDS - NL * nw) / ms);
    for (int g0 = 0; g0 < RW; g0 += G) {
        // each row's partners as a mask over the slots, several lanes a row
        constexpr int NLG = 256 / RW < 4 ? 4 : 256 / RW;
        __syncthreads();  // the ranks, then the last pass's masks, are read
        for (int x = t; x < G * ms; x += 256)
            mask[x] = 0u;
        __syncthreads();
        for (int hg = t / NLG; hg < G; hg += 256 / NLG) {
            const int hr = (g0 + hg) * W + w;  // rank of the row this lane reads
            if (g0 + hg >= RW || hr >= tcnt)
                break;
            const int rho = sord[hr];
            const int len = slen[rho];
            const uint4 *rp = reinterpret_cast<const uint4 *>(a.rows + (size_t)(first + rho) * a.cap);
            unsigned *mk = mask + hg * ms;
            for (int pc = t % NLG; 8 * pc < len; pc += NLG) {
                const uint4 v = rp[pc];
                const unsigned ws[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (pc * 8 + u < len) {
                        const int ns = nslot[(ws[u >> 1] >> ((u & 1) * 16)) & 0xffffu];
                        atomicOr(&mk[ns >> 5], 1u << (ns & 31));
                    }
                }
            }
        }
        __syncthreads();
        // each lane takes its partners, in ascending order
        if (g >= g0 && g < g0 + G) {
            const unsigned *mk = mask + (g - g0) * ms, *cm = cmask + q * nw;
            const int words = g * W + w < tcnt ? nw : 0;
            uint4 *dst = a.skin16 + (size_t)wg * (chunks / 2) * 256 + t;
            unsigned a0 = 0u, a1 = 0u, a2 = 0u, a3 = 0u;  // the last eight entries, the newest on top
            int c = 0;
            auto put = [&](unsigned e) {
                a0 = __builtin_amdgcn_alignbit(a1, a0, 16);
                a1 = __builtin_amdgcn_alignbit(a2, a1, 16);
                a2 = __builtin_amdgcn_alignbit(a3, a2, 16);
                a3 = __builtin_amdgcn_alignbit(e, a3, 16);
                if ((++c & 7) == 0 && c <= cap_lane)
                    dst[(size_t)((c >> 3) - 1) * 256] = make_uint4(a0, a1, a2, a3);
            };
            // one partner, and a step to the next word when one is used up,
            // each time round: lanes wait for the longest row, not for the
            // fullest of every 64 words
            {
                unsigned b = words > 0 ? mk[0] & cm[0] : 0u, next = words > 1 ? mk[1] & cm[1] : 0u;
                for (int x = 0; x < words;) {
                    if (b) {
                        put(4u * (unsigned)(32 * x + __ffs(b) - 1));
                        b &= b - 1u;
                    }
                    if (!b) {
                        ++x;
                        b = next;
                        next = x + 1 < words ? mk[x + 1] & cm[x + 1] : 0u;
                    }
                }
            }
            int most = c;
#pragma unroll
            for (int off = 1; off < NL; off <<= 1)
                most = max(most, __shfl_xor(most, off, NL));
            const bool turn = most > cap_lane;
            if (turn) {
                // more of one class than a lane holds: the row is dealt in
                // turn, and the filter deals the list anew
                c = 0;
                int pos = 0;
                for (int x = 0; x < words; ++x)
                    for (unsigned b = mk[x]; b; b &= b - 1u, ++pos)
                        if (pos % NL == q)
                            put(4u * (unsigned)(32 * x + __ffs(b) - 1));
            }
            a.skin_len[wg * 256 + t] = (unsigned short)(turn ? c | SKIN_TURN : c);
            while (c & 7)
                put(4u * (unsigned)R::SW);  // the far-away slot
        }
    }
    // bonded and native entries: bonded rounds, then native ones
    const int kb = (id_lo + NL - 1) / NL, kn = (id_hi + NL - 1) / NL;
    const int r = g * W + w;
    const int rho = r < tcnt ? sord[r] : 0;
    const int2 rw = r < tcnt ? a.trow[first + rho] : make_int2(0, 0);
    const int nb = rw.y & 4095, ntop = nb + (rw.y >> 12);
    if (w == 0 && t == 0)
        a.tile_top[tile] = make_int4(kb, kn, S > 0 ? lo : first, S > 0 && span > 65536 ? 0 : 1);
    for (int k = 0; k < max(kb + kn, TOP_MIN); ++k) {
        const int e = k < kb ? q + k * NL : nb + q + (k - kb) * NL;
        const bool has = e < (k < kb ? nb : ntop);
        const float2 en = has ? a.tent[rw.x + e] : make_float2(__int_as_float(first + rho), 0.f);
        // bonded: r0; native: r0^2
        a.ltop[top_index(wg, k, t, a.top_rounds)] =
            make_uint2((unsigned)__float_as_int(en.x), __float_as_uint(k < kb ? en.y : en.y * en.y));
    }
}

// In the order of use: the scalar loads of a wave's first lines bring what its
// first loads need.
struct TileArgs {
    const unsigned short *stage16;
    const uint2 *ltop;
    const unsigned char *grho;
    const WgRec *wg_rec;
    const long long *step_base;
    long long step_off;
    const uint2 *noise_key;  // per residue {tag, stream id}
    const float4 *pin;
    const int4 *qin;        // fixed-point copies of the positions
    const uint2 *list16;
    const int *stage;
    int n_wg, chunks, top_rounds;
    int layer;  // of the MOVED words, read; the other is written, so that all workgroups of a launch read the same
    int has_pull, do_bin;
    FixDev fix;
    StepConsts c;
    UdConsts ud;
    float check_thr2;
    float4 *pout;
    int4 *qout;
    unsigned *err;
    float4 *vel;          // underdamped: per-residue velocity (NULL: overdamped)
    const unsigned short *llen;
    const int *pull_slot;
    const PullDev *pulls;
    double *res_energy;
    float4 *fout;
    TipDev tip;
    // the last step of a list period checks the displacements and bins its
    // new positions for the next skin search (do_bin)
    const float4 *hi_skin;
    unsigned *skin_flag;
    unsigned *place;
    const int4 *traj_cell;
    int *cell_count;
    float4 *cells;
    int *cell_of;
    GridDev g;
    FilterArgs f;           // FIRST: the filter's arguments
};

// The value of lane xor `off` (1, 2, 4 or 8, the lower ones already summed
// over, so that a mirror reaches an equal partner) by DPP: no LDS round trip.
__device__ __forceinline__ float lane_xor(float v, int off)
{
    const int x = __float_as_int(v);
    const int y = off == 1   ? __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false)   // quad_perm 1 0 3 2
                  : off == 2 ? __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xf, 0xf, false)   // quad_perm 2 3 0 1
                  : off == 4 ? __builtin_amdgcn_update_dpp(x, x, 0x141, 0xf, 0xf, false)  // row_half_mirror
                             : __builtin_amdgcn_update_dpp(x, x, 0x140, 0xf, 0xf, false); // row_mirror
    return __int_as_float(y);
}

// The plain step: one workgroup of 256 lanes per 256 / NL residues of a tile,
// NL adjacent lanes per residue, the tile's residues handed to the lanes
// longest skin row first.  What bounds it is the number of instructions its
// waves issue, so the pair loop holds one form and what can be done once a
// period or once a step is.
//  1. Every load at an address that needs no other load is issued first:
//     the tile's slot ids, the lane's list chunks (4 slots each) and its
//     bonded and native entries, all in lane order and so contiguous over a
//     wave; the positions follow.
//  2. Positions are read as fixed-point copies (16 bytes against the 32 of
//     the compensated pair); their differences are exact integers, near and
//     far from the origin.  Each lane evaluates its bonded and native
//     entries from the two copies and stages slots: the copy relative to the
//     workgroup's origin, rounded once to single precision.
//     The last RW lanes draw their residue's Gaussians (Philox and
//     Box-Muller, from the counter words that do not depend on the position)
//     and evaluate its cantilever and tip terms.
//  3. After the barrier the list chunks are summed from LDS.  Where the
//     residues do not fit around one origin (wide), or the slots one window,
//     the copies themselves are staged and subtracted.  A workgroup with a bonded or native pair out of the
//     copies' reach (far), a list whose cutoff is (list_far), and every
//     workgroup once a residue has moved too far since the rebuild (moved),
//     take the compensated positions from memory.
//     The NL partial sums of a residue are added by butterfly shuffles,
//     which give every lane the same bits.
//  4. After a second barrier the last RW lanes add the external terms and
//     the noise and take the compensated step (first-order, or BAOAB).
// FIRST (the first step after a rebuild, which then needs no filter kernel):
// the list rows are filtered from the skin rows first (filter_rows): the same
// rows, sums and bits as a filter kernel followed by a plain step.
// Against rows by residue, 32-byte positions rounded to the tile's frame by
// every reader and partners gathered through the rows (us a launch in traces of
// the calls of perf/cases.py, last steps of a period among them; the movement
// check takes up to 0.5 of the second): 250,000 residues 41.9 -> 36.2, a shell of
// 75,000 with a tip 13.9 -> 13.9, 20,000 underdamped 8.6 -> 7.4, 4,801 at protein
// density 22.3 -> 9.1, 1,000 10.8 -> 5.1, 56 4.5 -> 4.3; the first step of a
// period, with its filter, 106 -> 97, 38 -> 31, 20 -> 17, 48 -> 18, 22 -> 11, 9.3 -> 9.2.
template <int TILE, int NL, bool ENERGY, int MODE, bool FIRST>
__global__ __launch_bounds__(256, ENERGY ? 2 : (NL <= 2 ? 3 : 5)) void k_tile_step(TileArgs a)
{
    using R = Rows<TILE, NL>;
    constexpr int RW = R::RW, W = R::W;
    constexpr int SM = STAGE_MAX;
    constexpr int SW = R::SW, XS = R::XS;
    constexpr int PER = 4;           // staging slots per lane loaded together
    constexpr int EPI = 256 - RW;    // first lane of the update lanes
    constexpr int NPRE = R::NPRE;    // list chunks per lane loaded before the staging
    constexpr int TPRE = NL >= 16 ? 2 : (NL >= 8 ? 3 : TOP_MIN);  // bonded/native rounds loaded before the staging
    __shared__ __align__(16) unsigned char region[R::BYTES];  // the slots' positions by axis
    __shared__ unsigned short ring[FIRST ? R::RING * 256 : 1];
    __shared__ float bb[FIRST ? 24 : 1];
    __shared__ float f_s[3][RW];     // list + bonded/native force of each residue
    __shared__ double e_s[ENERGY ? 4 : 1][ENERGY ? RW : 1];
    if (FIRST) {
        // the cell counts were read by the skin search, which is done:
        // cleared for the binning at the end of this period; the flag too
        for (int k = blockIdx.x * 256 + threadIdx.x; k < a.f.n_cells; k += gridDim.x * 256)
            a.f.cell_count[k] = 0;
        if (blockIdx.x == 0 && threadIdx.x == 0)
            *a.f.skin_flag = 0u;
    }
    // XCD-aware order: consecutive tiles stay on one XCD's L2.
    const int per = gridDim.x >> 3;
    const int wg = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (wg >= a.n_wg)
        return;  // uniform over the workgroup
    const int t = threadIdx.x;
    const int tile = wg / W, part = wg % W;
    const int q = t % NL, g = t / NL;
    // ---- 1. loads: straight-line, in the order in which they are needed,
    // so that each wait is for its own load alone ----
    const unsigned short *st16 = a.stage16 + (size_t)tile * SM;
    const uint2 *tp = a.ltop + top_index(wg, 0, t, a.top_rounds);
    const uint2 *lp = a.list16 + (size_t)wg * a.chunks * 256 + t;
    int ids[PER];
    uint2 te[TPRE], lw[NPRE];
    int rho = 0;  // this lane group's residue in the tile
    WgRec wr{};
    if (FIRST) {
        const int r = g * W + part;  // rank of this lane group's residue
        const int first = a.f.tile_first[tile], tcnt = a.f.tile_first[tile + 1] - first;
        const bool in = r < tcnt;
        rho = in ? ranked(a.f.skin_ord, (size_t)tile * TILE + r, r) : 0;
        // what the step has as well by the step's own arguments: one set of
        // registers, none in scratch (250,000 residues 47.1 -> 46.4 us a step,
        // 75,000 16.75 -> 16.55)
        FilterArgs f = a.f;
        f.pos = a.pin;
        f.stage = a.stage;
        f.ltop = const_cast<uint2 *>(a.ltop);
        f.list16 = const_cast<uint2 *>(a.list16);
        f.llen = const_cast<unsigned short *>(a.llen);
        f.grho = const_cast<unsigned char *>(a.grho);
        f.wg_rec = const_cast<WgRec *>(a.wg_rec);
        f.fix = a.fix;
        f.top_rounds = a.top_rounds;
        filter_rows<TILE, NL>(f, wg, tile, t, first, tcnt, rho, region, ring, bb, wr);
    } else {
        rho = a.grho[wg * RW + g];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        ids[u] = st16[t + u * 256];
#pragma unroll
    for (int k = 0; k < TPRE; ++k)
        te[k] = tp[k * 256];
    // update lanes: residues in order when the workgroup holds a whole tile
    const int ue = t - EPI;
    const int ru = ue * W + part;
    int rhou = ue;
    if (W > 1 && !FIRST)
        rhou = a.grho[wg * RW + max(ue, 0)];
    int2 mv = make_int2(0, 0);
    if (!FIRST) {
        wr = a.wg_rec[wg];
        mv = reinterpret_cast<const int2 *>(a.wg_rec)[-1];
    }
    // a residue strayed since the rebuild (which this launch follows if FIRST)
    const bool moved = !FIRST && (a.layer ? mv.y : mv.x) != 0;
    const long long step = (a.step_base ? *a.step_base : 0) + a.step_off;
    const int first = wr.first, tcnt = wr.count, S = wr.slots;
    const bool upd = ue >= 0 && ru < tcnt;
    if (W > 1 && FIRST)  // this launch writes the groups' residues
        rhou = upd ? ranked(a.f.skin_ord, (size_t)tile * TILE + ru, ru) : 0;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wave = wv == 0 ? wr.waves[0] : (wv == 1 ? wr.waves[1] : (wv == 2 ? wr.waves[2] : wr.waves[3]));
    // this wave's list chunks, bonded rounds, all rounds
    const int nk = wave & 0xffff, kb = (wave >> 16) & 0xff, kall = (int)((unsigned)wave >> 24);
    const int i = first + rho;
    const int iu = first + (upd ? rhou : 0);
    const uint2 key = a.noise_key[iu];
    float4 hu = a.pin[2 * iu], lu = a.pin[2 * iu + 1];
    const int4 qi = a.qin[i];
    // ---- 2. positions, noise and external terms (update lanes), bonded/native ----
    const bool list_far = a.fix.list_far || moved, bond_far = a.fix.bond_far || moved;
    const bool fast = !list_far && !(wr.flags & WG_WIDE) && S <= SW;
    if (FIRST && !a.fix.by_step && q == 0 && g * W + part < tcnt)
        a.place[i] = fix_place(qi);
    float *sr = reinterpret_cast<float *>(region);  // x, y, z of slot s at s, XS + s, 2 XS + s
    const int *st = a.stage + (size_t)tile * SM;
    if (wr.flags & WG_IDS32) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            ids[u] = st[t + u * 256] - wr.base;
    }
    auto copy_of = [&](unsigned j) { return *reinterpret_cast<const int4 *>(reinterpret_cast<const char *>(a.qin) + (size_t)(j * 16u)); };
    int4 v[PER], pq[TPRE];
#pragma unroll
    for (int u = 0; u < PER; ++u)
        v[u] = copy_of((unsigned)(ids[u] + wr.base));
#pragma unroll
    for (int k = 0; k < TPRE; ++k)
        pq[k] = copy_of(te[k].x & ~FAR_ENTRY);
    // the list chunks last: nothing needs them before the barrier (past the
    // wave's chunks the first again, from L1: 20,000 residues 10.15 -> 9.9 us
    // a step)
#pragma unroll
    for (int k = 0; k < NPRE; ++k)
        lw[k] = lp[(k < nk ? k : 0) * 256];
    __builtin_amdgcn_sched_barrier(0);
    if (fast) {
        auto put = [&](int sl, const int4 &w) {
            sr[sl] = (float)fix_diff(w.x, wr.ox) * a.fix.unit;
            sr[XS + sl] = (float)fix_diff(w.y, wr.oy) * a.fix.unit;
            sr[2 * XS + sl] = (float)fix_diff(w.z, wr.oz) * a.fix.unit;
        };
        if (FIRST)
            __syncthreads();  // the staged positions of the filter are read
#pragma unroll
        for (int u = 0; u < PER; ++u)
            put(t + u * 256, v[u]);
        for (int sl = t + PER * 256; sl < S; sl += 256)
            put(sl, a.qin[st[sl]]);
        if (t < 3)
            sr[t * XS + SW] = 1.0e18f;  // the far-away slot
    }
    float gn[3] = {0.0f, 0.0f, 0.0f};
    Acc X;
    double e_x = 0.0, f_rep = 0.0;
    if (upd) {
        if (MODE == 0 && !(key.x >> 31)) {
            const uint4 w = noise_words(key.x, key.y, step, a.c);
            const float2 gxy = gaussian_pair(w);
            gn[0] = gxy.x;
            gn[1] = gxy.y;
            gn[2] = gaussian_axis(w, 2);
        }
        add_external(X, e_x, f_rep, hu, lu, step, a.c.h, a.has_pull ? a.pull_slot[iu] : -1, a.pulls,
                     a.tip, ENERGY, a.err);
    }
    const PairConsts k = pair_consts(a.c);
    Acc A;   // bonded and native terms
    {
        // in fixed-point units unless a pair is out of the copies' range
        const bool far = bond_far || (wr.flags & WG_FAR);
        const float eu = k.eh12 * a.fix.unit;
        bool broken = false;
        auto diff = [&](const int4 &p) {
            return make_float3((float)fix_diff(qi.x, p.x), (float)fix_diff(qi.y, p.y), (float)fix_diff(qi.z, p.z));
        };
        auto out_of_range = [&](unsigned x) { return far && (bond_far || x >= FAR_ENTRY); };
        auto delta = [&](unsigned x) {
            const unsigned j = x & ~FAR_ENTRY;
            return pair_delta(a.pin[2 * i], a.pin[2 * i + 1], a.pin[2 * j], a.pin[2 * j + 1]);
        };
        auto bond = [&](const uint2 &e, const int4 &p) {
            if (e.x != (unsigned)i) {
                const float3 d = diff(p);
                add_fene_d(A, out_of_range(e.x) ? delta(e.x)
                                                : make_float3(d.x * a.fix.unit, d.y * a.fix.unit, d.z * a.fix.unit),
                           __uint_as_float(e.y), k, ENERGY, broken);
            }
        };
        auto native = [&](const uint2 &e, const int4 &p) {
            if (e.x != (unsigned)i) {
                if (out_of_range(e.x))
                    add_native_d(A, delta(e.x), __uint_as_float(e.y), k, ENERGY);
                else
                    add_native_q(A, diff(p), __uint_as_float(e.y), a.fix.s2, eu, k, ENERGY);
            }
        };
        int rd = 0;
        if (kb == 1) {  // as in every chain of two neighbours a residue
            bond(te[0], pq[0]);
#pragma unroll
            for (int u = 1; u < TPRE; ++u)
                if (u < kall)
                    native(te[u], pq[u]);
            rd = TPRE;
        }
        for (; rd < kall; ++rd) {
            const uint2 e = tp[rd * 256];
            const int4 p = copy_of(e.x & ~FAR_ENTRY);
            if (rd < kb)
                bond(e, p);
            else
                native(e, p);
        }
        if (broken)
            atomicOr(a.err, ERR_FENE);
    }
    __syncthreads();
    // the binning's slot and the displacement check's reference, requested
    // now so that they arrive during the sums
    float4 hsk = make_float4(0.f, 0.f, 0.f, 0.f);
    if (MODE == 0 && upd && a.check_thr2 > 0.0f)
        hsk = a.hi_skin[iu];
    // the last step of a list period bins the new positions for the next
    // skin search; the cell slot is taken in the cell of the position before
    // the update (nearly always the cell of the new one), so the atomic's
    // round trip overlaps the step.  The lanes of a wave that bin into one
    // cell take consecutive slots from one atomic, issued by the group's
    // first lane (uniform branch: the whole wave takes part in the ballots).
    // The first step of a period never bins (it clears the cell counts the
    // binning at the period's end fills; a period's first step is not its last)
    const bool do_bin = MODE == 0 && !FIRST && a.do_bin;
    int bin_lead = 0, bin_rank = 0, bin_base = 0;
    int bin_c0 = -1;           // the cell of the position before the update
    int4 bin_off = {0, 0, 0, 0};  // the trajectory's cell offset, kept for after the update
    if (do_bin) {
        const bool binning = upd;
        if (binning)
            bin_off = a.traj_cell[__float_as_int(lu.w)];
        const int c0 = binning ? cell_index(hu, bin_off, a.g) : -1;
        bin_c0 = c0;
        const int lane = (int)__lane_id();
        const unsigned long long below = (1ull << lane) - 1ull;
        unsigned long long todo = __ballot(binning);
        unsigned long long mine = 0ull;
        while (todo) {
            const int lead = __ffsll((long long)todo) - 1;
            const int cl = __shfl(c0, lead);
            const unsigned long long same = __ballot(binning && c0 == cl) & todo;
            if ((same >> lane) & 1ull) {
                bin_lead = lead;
                bin_rank = __popcll(same & below);
            }
            if (lane == lead)
                mine = same;
            todo &= ~same;
        }
        if (binning && lane == bin_lead)
            bin_base = atomicAdd(&a.cell_count[c0], __popcll(mine));
    }
    // ---- 3. list partners ----
    Acc L;   // sum of d / r^8 (scaled below)
    float lscale = k.c6;
    auto entry = [](const uint2 &w, int u) { return ((u < 2 ? w.x : w.y) >> ((u & 1) * 16)) & 0xffffu; };
    if (fast) {
        const float xi = (float)fix_diff(qi.x, wr.ox) * a.fix.unit, yi = (float)fix_diff(qi.y, wr.oy) * a.fix.unit,
                    zi = (float)fix_diff(qi.z, wr.oz) * a.fix.unit;
        auto chunk = [&](const uint2 &w) {
            float3 d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float *p = reinterpret_cast<const float *>(region + entry(w, u));
                d[u] = make_float3(xi - p[0], yi - p[XS], zi - p[2 * XS]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                add_repulsive_u(L, d[u], k, ENERGY);
        };
#pragma unroll
        for (int kk = 0; kk < NPRE; ++kk)
            if (kk < nk)
                chunk(lw[kk]);
        if (nk > NPRE) {
            uint2 next = lp[NPRE * 256];
            for (int c = NPRE; c < nk; ++c) {
                const uint2 w = next;
                next = lp[min(c + 1, nk - 1) * 256];  // requested before this one is used
                chunk(w);
            }
        }
    } else if (!list_far) {
        // the copies, window by window: the entries ascend, so a lane goes
        // on where the window before ended
        lscale = k.c6 * a.fix.unit;
        const int m = a.llen[wg * 256 + t];
        int *sq = reinterpret_cast<int *>(region);
        int c = 0;
        for (int w0 = 0; w0 < S; w0 += SW) {
            __syncthreads();  // the previous window's readers are done
            for (int sl = t; sl < min(SW, S - w0); sl += 256) {
                const int4 w = a.qin[st[w0 + sl]];
                sq[sl] = w.x;
                sq[XS + sl] = w.y;
                sq[2 * XS + sl] = w.z;
            }
            __syncthreads();
            while (4 * c < m) {
                const uint2 w = lp[c * 256];
                unsigned far_end = 0u;
                int3 d[4];
                bool live[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned o = entry(w, u) - 4u * (unsigned)w0;
                    const bool has = 4 * c + u < m;
                    far_end |= has && entry(w, u) >= 4u * (unsigned)(w0 + SW) ? 1u : 0u;
                    live[u] = has && o < 4u * (unsigned)SW;
                    const int *p = reinterpret_cast<const int *>(region + (live[u] ? o : 0u));
                    d[u] = make_int3(fix_diff(qi.x, p[0]), fix_diff(qi.y, p[XS]), fix_diff(qi.z, p[2 * XS]));
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    add_repulsive_q(L, d[u], a.fix.s2, k, live[u], ENERGY);
                if (far_end)
                    break;  // the rest of the chunk is in a later window
                ++c;
            }
        }
    } else {
        const float4 hi0 = a.pin[2 * i], lo0 = a.pin[2 * i + 1];
        const int m = a.llen[wg * 256 + t];
        for (int e = 0; e < m; ++e) {
            const int j = st[entry(lp[(e >> 2) * 256], e & 3) >> 2];
            add_repulsive_u(L, pair_delta(hi0, lo0, a.pin[2 * j], a.pin[2 * j + 1]), k, ENERGY);
        }
    }
    // the residue's total over its NL lanes (butterfly: every lane gets the same bits)
    float fx = lscale * L.fx + A.fx, fy = lscale * L.fy + A.fy, fz = lscale * L.fz + A.fz;
    double eb = A.e_b, en = A.e_n, er = L.e_r, vir = A.vir + L.vir;
#pragma unroll
    for (int off = 1; off < NL; off <<= 1) {
        fx += lane_xor(fx, off);
        fy += lane_xor(fy, off);
        fz += lane_xor(fz, off);
        if (ENERGY) {
            eb += __shfl_xor(eb, off, NL);
            en += __shfl_xor(en, off, NL);
            er += __shfl_xor(er, off, NL);
            vir += __shfl_xor(vir, off, NL);
        }
    }
    if (q == 0 && g * W + part < tcnt) {
        const int fs = W > 1 ? g : rho;  // the update lane of this residue
        f_s[0][fs] = fx;
        f_s[1][fs] = fy;
        f_s[2][fs] = fz;
        if constexpr (ENERGY) {
            e_s[0][fs] = eb;
            e_s[1][fs] = en;
            e_s[2][fs] = er;
            e_s[3][fs] = vir;
        }
    }
    // this residue's slot in its cell (the group's atomic has returned)
    int bin_s0 = 0;
    if (do_bin)
        bin_s0 = __shfl(bin_base, bin_lead) + bin_rank;
    __syncthreads();
    if (!upd)
        return;
    // ---- 4. external terms, noise and the compensated update ----
    Acc F;
    F.fx = f_s[0][ue] + X.fx;
    F.fy = f_s[1][ue] + X.fy;
    F.fz = f_s[2][ue] + X.fz;
    if constexpr (ENERGY) {
        double *er_out = a.res_energy + (size_t)iu * RES_E;
        // each internal pair appears in both partners' rows
        er_out[0] = 0.5 * e_s[0][ue];
        er_out[1] = 0.5 * e_s[1][ue];
        er_out[2] = 0.5 * e_s[2][ue];
        er_out[3] = e_x;
        er_out[4] = 0.5 * e_s[3][ue];
        er_out[5] = f_rep;
    }
    if (MODE == 1) {
        a.fout[iu] = make_float4(F.fx, F.fy, F.fz, 0.0f);
        return;
    }
    float4 hi = hu, lo = lu;
    unsigned *moved_out = a.err + MOVED + (a.layer ^ 1);
    if (a.vel) {
        float4 v = a.vel[iu];
        underdamped_update(hi, lo, v, F, gn, a.ud, a.fix.jump, moved_out, a.err);
        a.vel[iu] = v;
    } else {
        update_with_noise(hi, lo, F, gn, a.c, a.fix.jump, moved_out, a.err);
    }
    a.pout[2 * iu] = hi;
    a.pout[2 * iu + 1] = lo;
    const int4 qn = fix_pos(hi, lo, a.fix);
    a.qout[iu] = qn;
    if (__builtin_expect(moved || !a.fix.by_step, 0) && (moved || strayed(qn, a.place[iu], a.fix)))
        *moved_out = 1u;
    if (a.check_thr2 > 0.0f) {
        // moved farther than skin/2 from the last skin build: the next
        // rebuild rebuilds the skin
        const float dx = hi.x - hsk.x, dy = hi.y - hsk.y, dz = hi.z - hsk.z;
        if (!(dx * dx + dy * dy + dz * dz <= a.check_thr2))
            atomicOr(a.skin_flag, 1u);
    }
    if (do_bin) {
        const int traj = __float_as_int(lo.w);
        const int c1 = cell_index(hi, bin_off, a.g);
        if (c1 == bin_c0) {
            a.cell_of[iu] = c1;
            if (bin_s0 < CELL_CAP)
                a.cells[(size_t)c1 * CELL_CAP + bin_s0] = make_float4(hi.x, hi.y, hi.z, __int_as_float(iu));
            else
                atomicOr(a.err, ERR_CELL);
        } else {
            // moved into another cell: the slot taken holds a far-away copy
            // (no predicate passes it; the id keeps the cell's ids distinct)
            // and the residue is binned again
            if (bin_s0 < CELL_CAP)
                a.cells[(size_t)bin_c0 * CELL_CAP + bin_s0] =
                    make_float4(1.0e18f, 1.0e18f, 1.0e18f, __int_as_float(iu));
            bin_one(hi, iu, traj, a.g, a.traj_cell, a.cell_count, a.cells, a.cell_of, a.err);
        }
    }
}

// ---------------------------------------------------------------------------
// Pair-based forces (Algorithm 4 with the atomic additions its text proposes
// for GPUs that have them, Algorithm 5's gathering folded into the update
// kernel): each unordered pair of the list and of the bonded and native
// entries is evaluated once, in the row of its lower residue, and +df / -df
// are added to both residues' force accumulators with hardware float
// atomics.  The order of those additions is not fixed, so forces and
// trajectories are reproducible only to rounding.
// ---------------------------------------------------------------------------
struct PairArgs {
    const unsigned short *llen;
    const unsigned char *grho;
    const int *tile_first;
    const float4 *pin;
    const int2 *trow;
    const float2 *tent;
    const uint2 *list16;
    const int *stage;
    const int *stage_cnt;
    float4 *facc;   // per residue: accumulated force
    double4 *eacc;  // per residue: {FENE, native, repulsive, virial} of the pairs in its row
    unsigned *err;
    int cap;
    StepConsts c;
};

// One workgroup per tile.  A list pair (i, j), i < j, is evaluated in
// residue i's row; +df goes to i's running sum in registers and -df to j's
// staging slot in LDS (a shared-memory float atomic); at the end each
// residue's sum and each slot's sum are added to the device-wide
// accumulators with one hardware float atomic per component.  Bonded and
// native partners, which need no slot, take device-wide atomics directly.
// Energies stay whole with the lower residue (they are summed over the
// trajectory): halves added to both with double atomics made a record step of
// 75,000 residues 305 us where one without records takes 85.
template <int TILE, int NL, bool ENERGY>
__global__ __launch_bounds__(256) void k_pair_forces(PairArgs a)
{
    using R = Rows<TILE, NL>;
    constexpr int SM = STAGE_MAX;
    constexpr int SW = R::SW;
    __shared__ float acc_s[3][SW];  // slots beyond SW take device-wide atomics
    const int wg = blockIdx.x, t = threadIdx.x;
    const int tile = wg / R::W, r = t / NL * R::W + wg % R::W, q = t % NL;
    const int first = a.tile_first[tile], tcnt = a.tile_first[tile + 1] - first;
    const int S = min(a.stage_cnt[tile], SM);
    const int *st = a.stage + (size_t)tile * SM;
    for (int sl = t; sl < min(S, SW); sl += 256) {
        acc_s[0][sl] = 0.0f;
        acc_s[1][sl] = 0.0f;
        acc_s[2][sl] = 0.0f;
    }
    __syncthreads();
    const bool act = r < tcnt;
    const int i = first + a.grho[wg * R::RW + t / NL];
    const PairConsts k = pair_consts(a.c);
    Acc own;  // residue i's share of its pairs
    if (act) {
        const float4 hi = a.pin[2 * i], lo = a.pin[2 * i + 1];
        const int m = a.llen[wg * 256 + t];
        const unsigned short *row = reinterpret_cast<const unsigned short *>(
            a.list16 + chunk_index(wg, 0, t, lane_chunks(a.cap, NL)));
        for (int e = 0; e < m; ++e) {
            const int sl = row[(e >> 2) * 1024 + (e & 3)] >> 2;
            const int j = st[sl];
            if (j <= i)
                continue;  // the pair belongs to the lower residue's row
            Acc d;
            add_repulsive_d(d, pair_delta(hi, lo, a.pin[2 * j], a.pin[2 * j + 1]), k, ENERGY);
            own.fx += d.fx;
            own.fy += d.fy;
            own.fz += d.fz;
            if (sl < SW) {
                atomicAdd(&acc_s[0][sl], -d.fx);
                atomicAdd(&acc_s[1][sl], -d.fy);
                atomicAdd(&acc_s[2][sl], -d.fz);
            } else {
                unsafeAtomicAdd(&a.facc[j].x, -d.fx);
                unsafeAtomicAdd(&a.facc[j].y, -d.fy);
                unsafeAtomicAdd(&a.facc[j].z, -d.fz);
            }
            if (ENERGY) {
                own.e_r += d.e_r;
                own.vir += d.vir;
            }
        }
        const int2 rw = a.trow[i];
        const int nb = rw.y & 4095, ntop = nb + (rw.y >> 12);
        bool broken = false;
        for (int e = q; e < ntop; e += NL) {
            const float2 te = a.tent[rw.x + e];
            const int j = __float_as_int(te.x);
            if (j <= i)
                continue;
            Acc d;
            const float3 dd = pair_delta(hi, lo, a.pin[2 * j], a.pin[2 * j + 1]);
            if (e < nb)
                add_fene_d(d, dd, te.y, k, ENERGY, broken);
            else
                add_native_d(d, dd, te.y * te.y, k, ENERGY);
            own.fx += d.fx;
            own.fy += d.fy;
            own.fz += d.fz;
            unsafeAtomicAdd(&a.facc[j].x, -d.fx);
            unsafeAtomicAdd(&a.facc[j].y, -d.fy);
            unsafeAtomicAdd(&a.facc[j].z, -d.fz);
            if (ENERGY) {
                own.e_b += d.e_b;
                own.e_n += d.e_n;
                own.vir += d.vir;
            }
        }
        if (broken)
            atomicOr(a.err, ERR_FENE);
    }
    // residue i: its NL lanes' shares, then one atomic per component
#pragma unroll
    for (int off = 1; off < NL; off <<= 1) {
        own.fx += __shfl_xor(own.fx, off, NL);
        own.fy += __shfl_xor(own.fy, off, NL);
        own.fz += __shfl_xor(own.fz, off, NL);
        if (ENERGY) {
            own.e_b += __shfl_xor(own.e_b, off, NL);
            own.e_n += __shfl_xor(own.e_n, off, NL);
            own.e_r += __shfl_xor(own.e_r, off, NL);
            own.vir += __shfl_xor(own.vir, off, NL);
        }
    }
    if (act && q == 0) {
        unsafeAtomicAdd(&a.facc[i].x, own.fx);
        unsafeAtomicAdd(&a.facc[i].y, own.fy);
        unsafeAtomicAdd(&a.facc[i].z, own.fz);
        if (ENERGY) {
            a.eacc[i] = make_double4(own.e_b, own.e_n, own.e_r, own.vir);
        }
    }
    __syncthreads();
    // the slots' shares
    for (int sl = t; sl < min(S, SW); sl += 256) {
        const float fx = acc_s[0][sl], fy = acc_s[1][sl], fz = acc_s[2][sl];
        if (fx != 0.0f || fy != 0.0f || fz != 0.0f) {
            const int j = st[sl];
            unsafeAtomicAdd(&a.facc[j].x, fx);
            unsafeAtomicAdd(&a.facc[j].y, fy);
            unsafeAtomicAdd(&a.facc[j].z, fz);
        }
    }
}

struct PairUpdArgs {
    const float4 *pin;
    float4 *pout;
    int4 *qout;
    FixDev fix;
    float4 *facc;
    double4 *eacc;
    const uint2 *noise_key;
    const int *pull_slot;
    const PullDev *pulls;
    double *res_energy;
    float4 *fout;
    unsigned *err;
    const long long *step_base;
    const float4 *hi_skin;
    unsigned *skin_flag;
    const unsigned *place;
    int layer;  // as in TileArgs, for particle-based steps, if the mode changes within a period
    float4 *vel;
    const int4 *traj_cell;
    int *cell_count;
    float4 *cells;
    int *cell_of;
    GridDev g;
    int do_bin;
    long long step_off;
    float check_thr2;
    int n, has_pull;
    StepConsts c;
    UdConsts ud;
    TipDev tip;
};

// Algorithm 5's gathering and the update: the accumulated force (cleared
// for the next step), the external terms, the noise and the compensated step.
template <bool ENERGY, int MODE>
__global__ __launch_bounds__(256) void k_pair_update(PairUpdArgs a)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= a.n)
        return;
    const long long step = (a.step_base ? *a.step_base : 0) + a.step_off;
    const float4 hi0 = a.pin[2 * i], lo0 = a.pin[2 * i + 1];
    const float4 f = a.facc[i];
    a.facc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    Acc F;
    F.fx = f.x;
    F.fy = f.y;
    F.fz = f.z;
    double e_x = 0.0, f_rep = 0.0;
    add_external(F, e_x, f_rep, hi0, lo0, step, a.c.h, a.has_pull ? a.pull_slot[i] : -1, a.pulls, a.tip,
                 ENERGY, a.err);
    if (ENERGY) {
        const double4 e = a.eacc[i];
        double *er = a.res_energy + (size_t)i * RES_E;
        er[0] = e.x;
        er[1] = e.y;
        er[2] = e.z;
        er[3] = e_x;
        er[4] = e.w;
        er[5] = f_rep;
    }
    if (MODE == 1) {
        a.fout[i] = make_float4(F.fx, F.fy, F.fz, 0.0f);
        return;
    }
    float g[3] = {0.0f, 0.0f, 0.0f};
    const uint2 key = a.noise_key[i];
    if (!(key.x >> 31)) {
        const uint4 w = noise_words(key.x, key.y, step, a.c);
        const float2 gxy = gaussian_pair(w);
        g[0] = gxy.x;
        g[1] = gxy.y;
        g[2] = gaussian_axis(w, 2);
    }
    float4 hi = hi0, lo = lo0;
    unsigned *moved_out = a.err + MOVED + (a.layer ^ 1);
    if (a.vel) {
        float4 v = a.vel[i];
        underdamped_update(hi, lo, v, F, g, a.ud, a.fix.jump, moved_out, a.err);
        a.vel[i] = v;
    } else {
        update_with_noise(hi, lo, F, g, a.c, a.fix.jump, moved_out, a.err);
    }
    a.pout[2 * i] = hi;
    a.pout[2 * i + 1] = lo;
    const int4 qn = fix_pos(hi, lo, a.fix);
    a.qout[i] = qn;
    if (a.err[MOVED + a.layer] != 0u || (!a.fix.by_step && strayed(qn, a.place[i], a.fix)))
        *moved_out = 1u;
    if (a.check_thr2 > 0.0f) {
        const float4 hs = a.hi_skin[i];
        const float dx = hi.x - hs.x, dy = hi.y - hs.y, dz = hi.z - hs.z;
        if (!(dx * dx + dy * dy + dz * dz <= a.check_thr2))
            atomicOr(a.skin_flag, 1u);
    }
    if (a.do_bin)
        bin_one(hi, i, __float_as_int(lo.w), a.g, a.traj_cell, a.cell_count, a.cells, a.cell_of, a.err);
}

// ---------------------------------------------------------------------------
// Batched ensemble: one workgroup per pack of whole trajectories, positions
// resident in LDS for n_steps steps; the list of each residue is rebuilt in
// LDS from all residues of its trajectory every list_every steps.
// ---------------------------------------------------------------------------
// The fixed-point position at byte offset `off` of the positions in LDS: one
// 16-byte read, also where only the coordinates are used (the compiler makes
// that a 12-byte one, which LDS serves no faster than two of 8 bytes: 4,096
// chains 78.4 against 74.4 us a step).
__device__ __forceinline__ int4 lds_pos(const char *base, unsigned off)
{
    typedef int vec4 __attribute__((ext_vector_type(4)));
    const vec4 v = *reinterpret_cast<const vec4 *>(base + off);
    asm volatile("" ::"v"(v));
    return make_int4(v.x, v.y, v.z, v.w);
}

// Four of them, the reads all in flight before the first is used (100 steps of
// 200 chains 1,148 -> 1,053 us, of 4,096 chains 5.96 -> 5.70 ms against a wait
// for each).
template <class M>
__device__ __forceinline__ void lds_pos4(const char *base, const unsigned (&off)[4], M m, int4 (&p)[4])
{
    typedef int vec4 __attribute__((ext_vector_type(4)));
    vec4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        v[u] = *reinterpret_cast<const vec4 *>(base + (u < m ? off[u] : 0u));
    asm volatile("" ::"v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
#pragma unroll
    for (int u = 0; u < 4; ++u)
        p[u] = make_int4(v[u].x, v[u].y, v[u].z, v[u].w);
}

struct BatchArgs {
    const float4 *pin;
    float4 *pout;
    const int2 *trow;
    const float2 *tent;
    const int *pack_off;      // first slot of each pack (n_packs + 1)
    const int *slot_res;      // residue of each slot; a pack's trajectories are consecutive
    const int *traj_lo;
    const int *traj_hi;
    const unsigned *stream_ids;
    const int *pull_slot;
    const PullDev *pulls;
    unsigned short *list;     // entry k of residue i at i*cap + k
    int *list_cnt;
    unsigned *place;          // per residue, as fix_place (unless by_step)
    unsigned *moved;          // per pack
    int *done;                // per pack: steps of this launch that k_batch took
    double *energy;
    double *f_ext;
    float4 *fout;
    unsigned *err;
    const long long *step_base;
    const float *tscale;      // per trajectory: noise amplitude factor (replica exchange), or NULL
    long long step_off;
    long long energy_every;
    int n_steps, list_every, stale, cap, has_pull;
    StepConsts c;
    FixDev fix;
    TipDev tip;
    float rc2;
};

// Deterministic per-trajectory sums of three values per residue: a tree over
// the residue's index in its trajectory, so the sums do not depend on where
// the pack holds it.  `red` is three doubles a slot; the first residue of the
// trajectory returns the sums.  (One lane that added a trajectory's values in
// order, one value after the other, made a force evaluation of the 384 chains
// of the exchange ladder 87 us; with the tree 57, and 46 with the list energies
// taken in the force sweep.)
template <int WGS>
__device__ __forceinline__ void traj_sums(double *red, int t, double (&v)[3], int tlo, int thi)
{
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k)
        red[k * WGS + t] = v[k];
    __syncthreads();
#pragma unroll 1
    for (int o = WGS / 2; o > 0; o >>= 1) {
        if (t - tlo < o && t + o < thi) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                red[k * WGS + t] += red[k * WGS + t + o];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
        v[k] = red[k * WGS + t];
}

// Batched schedule: the list partners of a residue are summed in two partial
// sums (the first and the second fours of its row's eights, each in row order)
// by one lane or two, so the sum does not depend on the lanes or on the
// packing.  Which lane sums which row is chosen at each list rebuild by a
// counting sort on the row length (longest first), so the lanes of a wave
// run loops of about the same length; which lane sums which bonded and native
// entries, once a launch by their number.
// Bound by vector instructions when the chip is full (their issue filled
// 99.8% of the cycles before the following), by the list rebuild (a third of
// a step's time, every tenth step) and the wave with the longest rows when it
// is not: integer differences of fixed-point positions in place of float ones
// with packed low parts, rows without padding, sorted native entries, list
// entries shifted through one word as they are found: 4,096 chains of 50-500
// residues 75.6 -> 62.4 us a step, 200 chains (111 packs) 14.9 -> 11.5, 384
// chains of the exchange ladder 15.4 -> 12.3.  Two partial sums, slots of
// equal row length in slot order, and the fewest entries in the wave with the
// longest rows: 54.5, 10.3 and 10.5; two lanes a residue (batch_split): 9.7.
// With the movement check, the far list in a kernel of its own and four reads
// in flight: 57.7, 10.5 and 9.7.
constexpr int NBUCKET = 64;

// FAR: the list's differences are taken over the periods (FixDev::list_far), in
// a kernel of its own, as what they take in registers the others spill.
// EXACT: a residue has moved too far since the rebuild for differences of the
// copies (or lay too far off then); all are taken from the compensated
// positions instead, shared through the layer that is written, with the same
// bits wherever the copies hold.  The other form leaves such a pack where it
// is (`done`) to a launch of this one behind it.
template <int WGS, int MODE, int SPLIT, bool FAR, bool EXACT>
__device__ __forceinline__ void batch_pack(const BatchArgs &a, int p)
{
    static_assert(SPLIT == 1 || (SPLIT == 2 && MODE == 0), "records are taken by one lane a residue");
    constexpr int TH = WGS * SPLIT;
    constexpr int TCAP = 8 * WGS;  // bonded/native entries of a pack kept in LDS
    // per residue: its fixed-point position and periods; its high part while
    // the list is rebuilt
    __shared__ int4 sq[WGS];
    float4 *shh = reinterpret_cast<float4 *>(sq);
    __shared__ unsigned short tpart[TCAP];  // bonded/native entries of the pack: byte offset in sq
    __shared__ float tr0[TCAP];             // ... and r0 (CSR in slot order)
    __shared__ unsigned short tex[TCAP];    // the same partners in ascending order (list exclusions)
    __shared__ int perm[WGS];           // row summed by each lane: residue | chunks << 16
    // list force, then bonded and native force of each residue; the
    // trajectory sums of a record step
    __shared__ __align__(8) float fsum[3 * (SPLIT + 1)][WGS];
    float (*tsum)[WGS] = fsum, (*lsum)[WGS] = fsum + 3;  // lsum: SPLIT triples
    __shared__ unsigned words[SPLIT == 1 ? 1 : WGS / 32][SPLIT == 1 ? 1 : WGS];  // rebuild: the rows as masks
    __shared__ double esum[2][MODE == 0 ? 1 : WGS];  // record steps: list energy and virial of each residue
    __shared__ int hist[WGS / 64][NBUCKET];
    __shared__ int sres[WGS];           // residue of each local slot
    __shared__ unsigned moved_s;        // a residue has moved too far since the rebuild
    __shared__ float3 bblo[WGS / 32], bbhi[WGS / 32];  // list rebuild: boxes of 32-slot blocks
    const int off = a.pack_off[p];
    const int n = a.pack_off[p + 1] - off;
    // slot of this lane; SPLIT 2: lanes in the upper half of the workgroup
    // serve the same slots as those in the lower
    const int t = SPLIT == 1 ? (int)threadIdx.x : (int)(threadIdx.x % WGS);
    const int half = SPLIT == 1 ? 0 : (int)(threadIdx.x / WGS);  // uniform over a wave
    const bool own = half == 0;          // writes the slot's state
    const bool topo = half == SPLIT - 1; // sums bonded and native entries
    const bool act = t < n;
    const int i = act ? a.slot_res[off + t] : 0;  // this lane's residue
    // local slot of a residue of the same trajectory: residue + shift
    const int shift = t - i;

    float4 hi = make_float4(0.f, 0.f, 0.f, 0.f), lo = hi;
    int tlo = 0, thi = 0;
    int2 row = make_int2(0, 0);
    int cnt = 0;
    // positions as they are in memory while this pack is stepped
    const float4 *live = MODE == 1 ? a.pin : a.pout;
    if (act) {
        hi = EXACT ? live[2 * i] : a.pin[2 * i];
        lo = EXACT ? live[2 * i + 1] : a.pin[2 * i + 1];
        tlo = a.traj_lo[i] + shift;
        thi = a.traj_hi[i] + shift;
        row = a.trow[i];
        cnt = a.list_cnt[i];
    }
    int4 qi = fix_pos(hi, lo, a.fix);
    const long long s0 = (a.step_base ? *a.step_base : 0) + a.step_off;
    const int q0 = EXACT ? a.done[p] : 0;
    const bool fresh = (q0 == 0 && a.stale) || (s0 + q0) % a.list_every == 0;  // starts with a rebuild
    if (own) {
        sq[t] = qi;
        sres[t] = i;
        if (!isfinite(hi.x) || !isfinite(hi.y) || !isfinite(hi.z))
            atomicOr(a.err, ERR_NONFINITE);
        if (t == 0)
            moved_s = fresh ? 0u : a.moved[p];
    }
    // what is compared with a residue's place: its copy, or the periods below it
    auto coarse = [&](const int4 &q) {
        return a.fix.list_far ? make_int4(q.w << 22, (q.w >> 10) << 22, (q.w >> 20) << 22, 0) : q;
    };
    const int nb = row.y & 4095, ntop = nb + (row.y >> 12);
    // the pack's bonded/native entries in LDS (entries past TCAP stay in
    // global memory)
    int tot_top = 0;
    int *scan = reinterpret_cast<int *>(fsum[0]);
    block_exclusive_scan<TH>(own ? ntop : 0, scan, tot_top);
    const int toff = scan[t] - ntop;
    const bool top_lds = toff + ntop <= TCAP;  // all of this residue's entries are in LDS
    for (int e = 0; own && e < ntop && toff + e < TCAP; ++e) {
        const float2 te = a.tent[row.x + e];
        const unsigned short j = (unsigned short)(__float_as_int(te.x) + shift);
        tpart[toff + e] = (unsigned short)(j << 4);
        tr0[toff + e] = e < nb ? te.y : te.y * te.y;  // natives: r0^2
        if (top_lds) {  // insertion into the ascending copy
            int k = e;
            while (k > 0 && tex[toff + k - 1] > j) {
                tex[toff + k] = tex[toff + k - 1];
                --k;
            }
            tex[toff + k] = j;
        }
    }
    auto partner = [&](int e) {
        return toff + e < TCAP ? (int)tpart[toff + e] >> 4 : __float_as_int(a.tent[row.x + e].x) + shift;
    };
    // rows are residue-major: entry k (a local slot) of residue i at i cap + k
    uint2 *rowp = reinterpret_cast<uint2 *>(a.list + (size_t)i * a.cap);
    const PairConsts kc = pair_consts(a.c);
    const int traj = __float_as_int(lo.w);
    // this trajectory's temperature (fixed within a launch)
    StepConsts cn = a.c;
    if (a.tscale && act)
        cn.c_noise *= a.tscale[traj];
    const unsigned stream = act ? a.stream_ids[traj] : 0u;

    // Counting sort of the pack's slots by `key` (0 <= key < NBUCKET), largest
    // first, equal ones in slot order: neighbours have much the same partners,
    // so their lanes read LDS with fewer bank conflicts (11.3 for 13.0 cycles a
    // 16-byte read, counted over the rows of the 200 chains).  The packed value of
    // the `k`-th slot goes to perm[k].
    auto sort_slots = [&](int key, int value) {
        const int wv = t >> 6, lane = t & 63;
        unsigned long long same = __ballot(act);
#pragma unroll
        for (int b = 1; b < NBUCKET; b <<= 1) {
            const unsigned long long set = __ballot((key & b) != 0);
            same &= (key & b) ? set : ~set;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        if (own)
            hist[wv][lane] = 0;
        __syncthreads();
        if (own && act && rank == 0)
            hist[wv][NBUCKET - 1 - key] = __popcll(same);
        __syncthreads();
        if (own && t < 64) {  // one wave: a bucket a lane
            int v = 0;
#pragma unroll
            for (int w = 0; w < WGS / 64; ++w)
                v += hist[w][t];
            int x = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(x, o, 64);
                if (t >= o)
                    x += y;
            }
            x -= v;
#pragma unroll
            for (int w = 0; w < WGS / 64; ++w) {
                const int c = hist[w][t];
                hist[w][t] = x;
                x += c;
            }
        }
        __syncthreads();
        if (own && act)
            perm[hist[wv][NBUCKET - 1 - key] + rank] = value;
        __syncthreads();
    };
    static_assert(NBUCKET == 64, "a bucket a lane");

    // lane -> row assignment: by length in chunks, anew at each list rebuild
    int my = 0;   // local slot | partners << 16 of the row this lane sums
    int myg = 0;  // its residue
    auto assign = [&]() {
        const int c = act ? min(cnt, a.cap) : 0;
        sort_slots(min((c + 3) >> 2, NBUCKET - 1), t | (c << 16));
        my = t < n ? perm[t] : 0;
        myg = sres[my & 0xffff];
    };

    // lane -> bonded and native entries: by number, once a launch (the longest
    // of 64 residues in slot order has about 8 natives where the mean is 3),
    // fewest first: the wave with the longest rows has the fewest entries
    __syncthreads();
    sort_slots(min(ntop, NBUCKET - 1), t);
    const int tr = t < n ? perm[n - 1 - t] : 0;  // the slot whose entries this lane sums
    int *tq = reinterpret_cast<int *>(tsum[0]);
    if (own) {
        tq[t] = toff;
        tq[WGS + t] = nb | (ntop << 12);
        tq[2 * WGS + t] = row.x;
    }
    __syncthreads();
    const int tr_off = tq[tr], tr_x = tq[2 * WGS + tr];
    const int tr_nb = t < n ? tq[WGS + tr] & 4095 : 0, tr_ntop = t < n ? tq[WGS + tr] >> 12 : 0;
    const int tr_shift = tr - sres[tr];
    const bool tr_lds = tr_off + tr_ntop <= TCAP;
    // entry e of residue `slot` (its entries at `x` and, in LDS, at `off0`)
    auto entry = [&](int off0, int x, int sh, int nbond, int e, int &j, float &r0) {
        if (off0 + e < TCAP) {
            j = tpart[off0 + e];
            r0 = tr0[off0 + e];
        } else {
            const float2 te = a.tent[x + e];
            j = (__float_as_int(te.x) + sh) << 4;
            r0 = e < nbond ? te.y : te.y * te.y;
        }
    };
    const char *sqb = reinterpret_cast<const char *>(sq);

    // one of tr's partners is out of reach of plain integer differences until
    // the next rebuild (the full ones give the same bits within it)
    bool far = false;
    auto check_reach = [&]() {
        far = FAR;
        if (!topo || FAR || EXACT)
            return;
        const float lim = a.fix.reach * (float)a.fix.scale;
        const int4 p = sq[tr];
        for (int e = 0; e < tr_ntop; ++e) {
            int j;
            float r0;
            entry(tr_off, tr_x, tr_shift, tr_nb, e, j, r0);
            const float3 d = fix_full_diff(p, lds_pos(sqb, j));
            far |= !(fmaxf(fabsf(d.x), fmaxf(fabsf(d.y), fabsf(d.z))) <= lim);
        }
    };
    __syncthreads();
    if (!fresh) {
        check_reach();
        assign();
    }

    int q = q0;
    for (; q < a.n_steps; ++q) {
        const long long step = s0 + q;
        if ((q == 0 && a.stale) || step % a.list_every == 0) {
            check_reach();
            __syncthreads();
            if (own) {
                shh[t] = hi;  // the high parts, until the rows are written
                if (__builtin_expect(!a.fix.by_step, 0) && act)
                    a.place[i] = fix_place(coarse(qi));
                if (t == 0)
                    moved_s = 0u;
            }
            {
                // boxes of the 32-slot blocks (empty slots add nothing)
                float3 bl = act ? make_float3(hi.x, hi.y, hi.z) : make_float3(3.0e38f, 3.0e38f, 3.0e38f);
                float3 bh = act ? make_float3(hi.x, hi.y, hi.z) : make_float3(-3.0e38f, -3.0e38f, -3.0e38f);
#pragma unroll
                for (int o = 1; o < 32; o <<= 1) {
                    bl.x = fminf(bl.x, __shfl_xor(bl.x, o, 64));
                    bl.y = fminf(bl.y, __shfl_xor(bl.y, o, 64));
                    bl.z = fminf(bl.z, __shfl_xor(bl.z, o, 64));
                    bh.x = fmaxf(bh.x, __shfl_xor(bh.x, o, 64));
                    bh.y = fmaxf(bh.y, __shfl_xor(bh.y, o, 64));
                    bh.z = fmaxf(bh.z, __shfl_xor(bh.z, o, 64));
                }
                if (own && (t & 31) == 0) {
                    bblo[t >> 5] = bl;
                    bbhi[t >> 5] = bh;
                }
                __syncthreads();
            }
            if (SPLIT == 2 && !own)
                hi = shh[t];  // where its slot's own lane has moved it
            if (act && own) {
                const float4 o = shh[tlo];
                if (!(fmaxf(fmaxf(fabsf(hi.x - o.x), fabsf(hi.y - o.y)), fabsf(hi.z - o.z)) <= a.fix.spread))
                    moved_s = 1u;
            }
            // Algorithm 3 over the trajectory: r < r_list, not bonded or
            // native. Candidates are tested a 32-slot block at a time into a
            // bit word (blocks whose box is out of reach of every lane of the
            // wave are skipped); the row is written four entries (one 8-byte
            // chunk) at a time.  SPLIT 2: the blocks are halved between a
            // slot's lanes, and so are the entries to write.
            int ep = 0;  // next entry of the ascending exclusion list
            const int b0 = tlo >> 5, b1 = act ? ((thi - 1) >> 5) + 1 : b0;
            const int bm = SPLIT == 1 ? b1 : (b0 + b1 + 1) >> 1;
            const int jb0 = half ? bm : b0, jb1 = half ? b1 : bm;  // this lane's blocks
            // partners of this slot among those of block jb, at bit 31 - u
            auto block_mask = [&](int jb) -> unsigned {
                const int j0 = jb << 5;
                {
                    // the box test errs on the side of testing: a skipped
                    // block is farther than r_list by a margin far above
                    // the rounding of either distance
                    const float3 bl = bblo[jb], bh = bbhi[jb];
                    const float gx = fmaxf(fmaxf(bl.x - hi.x, hi.x - bh.x), 0.0f);
                    const float gy = fmaxf(fmaxf(bl.y - hi.y, hi.y - bh.y), 0.0f);
                    const float gz = fmaxf(fmaxf(bl.z - hi.z, hi.z - bh.z), 0.0f);
                    if (!__any(gx * gx + gy * gy + gz * gz <= a.rc2 * 1.001f))
                        return 0u;
                }
                // candidate j0 + u at bit 31 - u; slots of other
                // trajectories are masked
                unsigned m = 0u;
#pragma unroll 1
                for (int u0 = 0; u0 < 32; u0 += 8) {
                    float4 c8[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        c8[u] = shh[j0 + u0 + u];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        m = m + m + (within_cutoff(hi, c8[u], a.rc2) ? 1u : 0u);
                }
                m &= 0xffffffffu >> max(tlo - j0, 0);
                if (thi - j0 < 32)
                    m &= ~(0xffffffffu >> (thi - j0));
                unsigned x = 0u;  // the residue itself and its bonded/native partners
                auto drop = [&](int j) {
                    const unsigned d = (unsigned)(j - j0);
                    x |= d < 32u ? (0x80000000u >> d) : 0u;
                };
                drop(t);
                if (top_lds) {
                    for (; ep < ntop; ++ep) {  // entries below this block were passed by skipped blocks
                        const int j = tex[toff + ep];
                        if (j >= j0 + 32)
                            break;
                        drop(j);
                    }
                } else {
                    for (int e = 0; e < ntop; ++e)
                        drop(partner(e));
                }
                return m & ~x;
            };
            // entries [start, ...) of the row; those of the first and the last
            // chunk, if not whole, one by one
            unsigned w_lo = 0u, w_hi = 0u;  // the last four, the newest on top
            int pos = 0, start = 0;
            auto some = [&](int k) {  // the newest k < 4
                const unsigned long long w = (unsigned long long)w_hi << 32 | w_lo;
                unsigned short *row16 = reinterpret_cast<unsigned short *>(rowp);
                for (int e = 0; e < k; ++e)
                    if (pos - k + e < a.cap)
                        row16[pos - k + e] = (unsigned short)(w >> (16 * (4 - k + e)));
            };
            auto put = [&](int jb, unsigned &m) {  // the first partner of m
                const int u = __builtin_clz(m);
                const unsigned v = (unsigned)((jb << 5) + u) << 4;  // byte offset in sq (one workgroup holds 1,024)
                m &= 0x7fffffffu >> u;
                w_lo = __builtin_amdgcn_alignbit(w_hi, w_lo, 16);
                w_hi = __builtin_amdgcn_alignbit(v, w_hi, 16);
                ++pos;
                if ((pos & 3) == 0) {
                    if (SPLIT == 2 && pos - start < 4)
                        some(pos - start);
                    else if (pos <= a.cap)
                        rowp[(pos >> 2) - 1] = make_uint2(w_lo, w_hi);
                }
            };
            if (SPLIT == 1) {
                for (int jb = jb0; jb < jb1; ++jb) {
                    unsigned m = block_mask(jb);
                    while (m)
                        put(jb, m);
                }
                cnt = pos;
            } else {
                for (int jb = jb0; jb < jb1; ++jb)
                    words[jb][t] = block_mask(jb);
                __syncthreads();
                int c0 = 0, c1 = 0;
                for (int jb = b0; jb < b1; ++jb)
                    (jb < bm ? c0 : c1) += __popc(words[jb][t]);
                pos = start = half ? c0 : 0;
                // a partner, and a step to the next word when one is used up,
                // each time round: lanes wait for the longest row alone
                unsigned m = jb0 < jb1 ? words[jb0][t] : 0u, next = jb0 + 1 < jb1 ? words[jb0 + 1][t] : 0u;
                for (int jb = jb0; jb < jb1;) {
                    if (m)
                        put(jb, m);
                    if (!m) {
                        ++jb;
                        m = next;
                        next = jb + 1 < jb1 ? words[jb + 1][t] : 0u;
                    }
                }
                cnt = c0 + c1;
            }
            if ((pos & 3) != 0)
                some(min(pos & 3, pos - start));
            if (act && own) {
                if (cnt > a.cap)
                    atomicOr(a.err, ERR_OVERFLOW);
                a.list_cnt[i] = cnt;
            }
            assign();  // its barriers also publish the rows written above
            if (own)
                sq[t] = qi;
            __syncthreads();
        }
        // mode 0 never records (no FP64 sums in its registers); mode 2
        // records at multiples of the energy interval, in a copy of the
        // forces and update compiled for record steps alone
        if (!EXACT && __builtin_expect(__builtin_amdgcn_readfirstlane((int)moved_s) != 0, 0))
            break;
        auto exact_diff = [&](int slot, int partner_slot) {
            const int ri = sres[slot], rj = sres[partner_slot];
            return fix_exact_diff(live[2 * ri], live[2 * ri + 1], live[2 * rj], live[2 * rj + 1], a.fix);
        };
        const bool rec_step = MODE == 1 || (MODE == 2 && a.energy_every > 0 && step % a.energy_every == 0);
        auto forces_and_update = [&](auto rec_tag) {
            constexpr bool rec = decltype(rec_tag)::value;
            {
                // ---- list partners (forces) of the row this lane was given ----
                const int r = my & 0xffff;
                const int n8 = my >> 19;
                const int4 pr = sq[r];
                // rows are read in eights, the next one requested before the
                // current one is used; the first fours of the eights and the
                // second fours are summed apart, each pair by pair in row
                // order: by one lane (SPLIT 1), or by one each
                const uint4 *rp = reinterpret_cast<const uint4 *>(a.list + (size_t)myg * a.cap);
                const uint2 *rh = reinterpret_cast<const uint2 *>(rp) + half;
                const int last = max((my >> 16) - 1, 0) >> 3, left = (my >> 16) & 7;
                Acc L, M;
                auto sweep = [&](auto general) {
                    // four partners, `m` of them the row's (all of them: a constant)
                    auto chunk = [&](Acc &L, unsigned wx, unsigned wy, auto m) {
                        const unsigned off[4] = {wx & 0xffffu, wx >> 16, wy & 0xffffu, wy >> 16};
                        int4 pj[4];
                        lds_pos4(sqb, off, m, pj);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (general()) {
                                const float3 d = fix_full_diff(pr, pj[u]);
                                if (u < m)
                                    add_repulsive_u(L,
                                                    make_float3(d.x * a.fix.unit, d.y * a.fix.unit, d.z * a.fix.unit),
                                                    kc, rec);
                            } else {
                                add_repulsive_q(L, make_int3(fix_diff(pr.x, pj[u].x), fix_diff(pr.y, pj[u].y),
                                                             fix_diff(pr.z, pj[u].z)),
                                                a.fix.s2, kc, u < m, rec);
                            }
                        }
                    };
                    constexpr std::integral_constant<int, 4> all{};
                    if (SPLIT == 1) {
                        uint4 w = rp[0];
                        for (int c = 0; c < n8; ++c) {
                            const uint4 wn = rp[min(c + 1, last)];
                            chunk(L, w.x, w.y, all);
                            chunk(M, w.z, w.w, all);
                            w = wn;
                        }
                        if (left > 0)
                            chunk(L, w.x, w.y, left);
                        if (left > 4)
                            chunk(M, w.z, w.w, left - 4);
                    } else {
                        uint2 w = rh[0];
                        for (int c = 0; c < n8; ++c) {
                            const uint2 wn = rh[2 * min(c + 1, last)];
                            chunk(L, w.x, w.y, all);
                            w = wn;
                        }
                        if (left > 4 * half)
                            chunk(L, w.x, w.y, left - 4 * half);
                    }
                };
                if constexpr (EXACT) {
                    const unsigned short *row16 = reinterpret_cast<const unsigned short *>(rp);
#pragma unroll 1
                    for (int e = 0; e < my >> 16; ++e) {
                        Acc P = (e & 4) ? M : L;
                        const float3 d = exact_diff(r, row16[e] >> 4);
                        add_repulsive_u(P, make_float3(d.x * a.fix.unit, d.y * a.fix.unit, d.z * a.fix.unit), kc, rec);
                        ((e & 4) ? M : L) = P;
                    }
                } else {
                    sweep(std::integral_constant<bool, FAR>{});
                }
                if (t < n) {
                    if (SPLIT == 2) {
                        lsum[3 * half][r] = L.fx;
                        lsum[3 * half + 1][r] = L.fy;
                        lsum[3 * half + 2][r] = L.fz;
                    } else {
                        lsum[0][r] = L.fx + M.fx;
                        lsum[1][r] = L.fy + M.fy;
                        lsum[2][r] = L.fz + M.fz;
                    }
                    if (rec) {
                        esum[0][r] = L.e_r + M.e_r;
                        esum[1][r] = L.vir + M.vir;
                    }
                }
            }
            Acc A;  // energy sums are only accumulated on record steps
            bool broken = false;
            double e_x = 0.0, f_rep = 0.0;
            // ---- bonded, then native partners: two loops, so a wave whose
            // residues have different bond counts (chain ends) runs each
            // term's code alone.  Record steps take every lane's own residue
            // (its energies belong there), others the slot sorted to the lane.
            {
                auto terms = [&](const int4 &p, int slot, int off0, int x, int sh, int nbond, int nall, auto general) {
                    auto next = [&](int e, int &j, float &r0) -> float3 {
                        if (general()) {
                            entry(off0, x, sh, nbond, e, j, r0);
                            return EXACT ? exact_diff(slot, j >> 4) : fix_full_diff(p, lds_pos(sqb, j));
                        }
                        j = tpart[off0 + e];
                        r0 = tr0[off0 + e];
                        const int4 o = lds_pos(sqb, j);
                        return make_float3((float)fix_diff(p.x, o.x), (float)fix_diff(p.y, o.y),
                                           (float)fix_diff(p.z, o.z));
                    };
                    for (int e = 0; e < nbond; ++e) {
                        int j;
                        float r0;
                        const float3 d = next(e, j, r0);
                        add_fene_d(A, make_float3(d.x * a.fix.unit, d.y * a.fix.unit, d.z * a.fix.unit), r0, kc, rec,
                                   broken);
                    }
                    for (int e = nbond; e < nall; ++e) {
                        int j;
                        float r0;
                        const float3 d = next(e, j, r0);
                        add_native_q(A, d, r0, a.fix.s2, kc.eh12 * a.fix.unit, kc, rec);
                    }
                };
                if (rec) {
                    terms(qi, t, toff, row.x, shift, nb, ntop, std::true_type{});
                } else if (topo) {
                    const int4 p = sq[tr];
                    if (FAR || EXACT || __any(far || !tr_lds))
                        terms(p, tr, tr_off, tr_x, tr_shift, tr_nb, tr_ntop, std::true_type{});
                    else
                        terms(p, tr, tr_off, tr_x, tr_shift, tr_nb, tr_ntop, std::false_type{});
                    if (t < n) {
                        tsum[0][tr] = A.fx;
                        tsum[1][tr] = A.fy;
                        tsum[2][tr] = A.fz;
                    }
                }
            }
            if (broken)
                atomicOr(a.err, ERR_FENE);
            // SPLIT 2: the slot's own lane draws its noise meanwhile
            float gn[3] = {0.0f, 0.0f, 0.0f};
            if (SPLIT == 2 && own && act)
                draw_noise(gn, hi, step, stream, cn);
            __syncthreads();
            if (!rec) {
                A.fx = tsum[0][t];
                A.fy = tsum[1][t];
                A.fz = tsum[2][t];
            }
            if (act && own) {
                add_external(A, e_x, f_rep, hi, lo, step, a.c.h, a.has_pull ? a.pull_slot[i] : -1, a.pulls,
                             a.tip, rec, a.err);
                const float ls = FAR || EXACT ? kc.c6 : kc.c6 * a.fix.unit;
                float l[3] = {lsum[0][t], lsum[1][t], lsum[2][t]};
                if (SPLIT == 2) {
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax)
                        l[ax] += lsum[3 + ax][t];
                }
                A.fx = __builtin_fmaf(ls, l[0], A.fx);
                A.fy = __builtin_fmaf(ls, l[1], A.fy);
                A.fz = __builtin_fmaf(ls, l[2], A.fz);
                if (rec) {
                    A.e_r = esum[0][t];
                    A.vir += esum[1][t];
                }
            }
            if (rec) {
                // each internal pair appears in both partners' rows
                double *red = reinterpret_cast<double *>(fsum[0]);
                double v0[3] = {0.5 * A.e_b, 0.5 * A.e_n, 0.5 * A.e_r}, v1[3] = {e_x, 0.5 * A.vir, f_rep};
                traj_sums<WGS>(red, t, v0, tlo, thi);
                traj_sums<WGS>(red, t, v1, tlo, thi);
                if (act && t == tlo) {
                    const double vals[RES_E] = {v0[0], v0[1], v0[2], v1[0], v1[1], v1[2]};
#pragma unroll
                    for (int kk = 0; kk < RES_E; ++kk) {
                        if (kk < SOP_NTERMS)
                            a.energy[(size_t)traj * SOP_NTERMS + kk] = vals[kk];
                        else
                            a.f_ext[traj] = vals[kk];
                    }
                }
                __syncthreads();
            }
            if (MODE == 1) {
                if (act && own)
                    a.fout[i] = make_float4(A.fx, A.fy, A.fz, 0.0f);
                return;
            }
            if (act && own) {
                if (SPLIT == 1)
                    draw_noise(gn, hi, step, stream, cn);
                update_with_noise(hi, lo, A, gn, cn, a.fix.jump, &moved_s, a.err);
                qi = fix_pos(hi, lo, a.fix);
                sq[t] = qi;
                if (EXACT) {
                    a.pout[2 * i] = hi;
                    a.pout[2 * i + 1] = lo;
                }
                if (__builtin_expect(!a.fix.by_step, 0) && strayed(coarse(qi), a.place[i], a.fix))
                    moved_s = 1u;
            }
            __syncthreads();
        };
        if constexpr (MODE == 1) {
            forces_and_update(std::true_type{});
            ++q;
            break;
        } else if constexpr (MODE == 0) {
            forces_and_update(std::false_type{});
        } else {
            if (rec_step)
                forces_and_update(std::true_type{});
            else
                forces_and_update(std::false_type{});
        }
    }
    if (MODE != 1 && !EXACT && act && own) {
        a.pout[2 * i] = hi;
        a.pout[2 * i + 1] = lo;
    }
    if (threadIdx.x == 0) {
        a.moved[p] = moved_s;
        if (!EXACT)
            a.done[p] = q;
    }
}

template <int WGS, int MODE, int SPLIT, bool FAR>
__global__ __launch_bounds__(WGS * SPLIT, 4) void k_batch(BatchArgs a)
{
    batch_pack<WGS, MODE, SPLIT, FAR, false>(a, blockIdx.x);
}

// The packs that k_batch left (none, as a rule: 2 us a launch), of any size.
constexpr int EXACT_GRID = 256;

template <int MODE>
__global__ __launch_bounds__(1024, 4) void k_batch_exact(BatchArgs a, int n_packs)
{
    bool left = false;
    for (int p = blockIdx.x + EXACT_GRID * threadIdx.x; p < n_packs; p += EXACT_GRID * 1024)
        left |= a.done[p] < a.n_steps;
    if (!__syncthreads_or(left))
        return;
    for (int p = blockIdx.x; p < n_packs; p += EXACT_GRID) {
        if (a.done[p] < a.n_steps)  // uniform
            batch_pack<1024, MODE, 1, false, true>(a, p);
        __syncthreads();
    }
}

// Replica exchange: one lane per attempted swap of round `round` (the
// temperatures k, k+1 with k = round mod 2, round mod 2 + 2, ... of every
// group of n_rep consecutive trajectories), Metropolis on the potential
// energies recorded at this step, with a Philox draw under a key of its
// own.  Swaps of one round touch disjoint trajectories.
__global__ void k_exchange(const double *__restrict__ energy, const double *__restrict__ kbt, int n_rep,
                           int n_groups, int *__restrict__ tidx, float *__restrict__ tscale, double kbt_ref,
                           long long round, unsigned key0, unsigned key1, unsigned long long *__restrict__ stats)
{
    const int par = (int)(round & 1);
    const int pairs = (n_rep - par) / 2;  // k = par, par + 2, ... with k + 1 < n_rep
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (pairs <= 0 || id >= n_groups * pairs)
        return;
    const int g = id / pairs, k = par + 2 * (id % pairs);
    const int base = g * n_rep;
    int ta = -1, tb = -1;
    for (int m = 0; m < n_rep; ++m) {
        const int v = tidx[base + m];
        ta = v == k ? base + m : ta;
        tb = v == k + 1 ? base + m : tb;
    }
    if (ta < 0 || tb < 0)
        return;  // not a permutation (rejected on the host)
    double Ea = 0.0, Eb = 0.0;
    for (int term = 0; term < 4; ++term) {
        Ea += energy[(size_t)ta * SOP_NTERMS + term];
        Eb += energy[(size_t)tb * SOP_NTERMS + term];
    }
    const double d = (1.0 / kbt[k] - 1.0 / kbt[k + 1]) * (Ea - Eb);
    const uint4 w = philox10(make_uint4((unsigned)g, (unsigned)k, (unsigned)round,
                                        (unsigned)((unsigned long long)round >> 32)),
                             key0 ^ 0x52455843u, key1);
    const double u = ((double)(w.x >> 9) + 0.5) * 0x1p-23;
    atomicAdd(&stats[2 * k + 1], 1ull);
    if (d >= 0.0 || u < exp(d)) {
        atomicAdd(&stats[2 * k], 1ull);
        tidx[ta] = k + 1;
        tidx[tb] = k;
        tscale[ta] = (float)sqrt(kbt[k + 1] / kbt_ref);
        tscale[tb] = (float)sqrt(kbt[k] / kbt_ref);
    }
}

__global__ void k_add_step(long long *base, long long k)
{
    if (threadIdx.x == 0 && blockIdx.x == 0)
        *base += k;
}

// One workgroup per trajectory: double sums of the per-residue records.
// Per-trajectory FP64 energy and virial sums in two fixed-order levels:
// one workgroup per chunk of at most ECHUNK residues of one trajectory, then
// one lane per trajectory over its chunks in order.
__global__ __launch_bounds__(WG) void k_reduce_chunks(const double *__restrict__ res_energy,
                                                      const int *__restrict__ chunk_lo,
                                                      double *__restrict__ chunk_sum)
{
    __shared__ double part[WG / 64][RES_E];
    const int ch = blockIdx.x;
    const int a = chunk_lo[ch], b = chunk_lo[ch + 1];
    double s[RES_E] = {0, 0, 0, 0, 0, 0};
    for (int i = a + threadIdx.x; i < b; i += WG)
#pragma unroll
        for (int k = 0; k < RES_E; ++k)
            s[k] += res_energy[(size_t)i * RES_E + k];
#pragma unroll
    for (int k = 0; k < RES_E; ++k)
        for (int m = 32; m >= 1; m >>= 1)
            s[k] += __shfl_xor(s[k], m, 64);
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < RES_E; ++k)
            part[threadIdx.x >> 6][k] = s[k];
    __syncthreads();
    if (threadIdx.x < RES_E) {
        double v = 0.0;
        for (int w = 0; w < WG / 64; ++w)
            v += part[w][threadIdx.x];
        chunk_sum[(size_t)ch * RES_E + threadIdx.x] = v;
    }
}

// One wave per trajectory: lane l takes chunks l, l + 64, ... in order, then
// a fixed butterfly over the lanes.
__global__ __launch_bounds__(WG) void k_reduce_energy(const double *__restrict__ chunk_sum,
                                                      const int *__restrict__ chunk_first, int n_traj,
                                                      double *__restrict__ energy, double *__restrict__ f_ext)
{
    const int t = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (t >= n_traj)
        return;  // uniform over the wave
    double v[RES_E] = {0, 0, 0, 0, 0, 0};
    for (int ch = chunk_first[t] + lane; ch < chunk_first[t + 1]; ch += 64)
#pragma unroll
        for (int k = 0; k < RES_E; ++k)
            v[k] += chunk_sum[(size_t)ch * RES_E + k];
#pragma unroll
    for (int k = 0; k < RES_E; ++k)
        for (int m = 32; m >= 1; m >>= 1)
            v[k] += __shfl_xor(v[k], m, 64);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < SOP_NTERMS; ++k)
            energy[(size_t)t * SOP_NTERMS + k] = v[k];
        f_ext[t] = v[SOP_NTERMS];
    }
}

// Philox words and Gaussians of every residue at one step, computed with the
// same device functions as the step kernel.
__global__ void k_noise(const float4 *__restrict__ pos, int n, const unsigned *__restrict__ stream_ids,
                        unsigned k0, unsigned k1, long long step, uint4 *__restrict__ words,
                        float4 *__restrict__ g)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const unsigned local = __float_as_uint(pos[2 * i].w) & 0x7fffffffu;
    const unsigned stream = stream_ids[__float_as_int(pos[2 * i + 1].w)];
    const uint4 w = philox10(make_uint4(local, stream, (unsigned)step,
                                        (unsigned)((unsigned long long)step >> 32)), k0, k1);
    words[i] = w;
    g[i] = make_float4(gaussian_axis(w, 0), gaussian_axis(w, 1), gaussian_axis(w, 2), 0.0f);
}

__global__ void k_set_flag(unsigned *dst, unsigned v)
{
    if (threadIdx.x == 0)
        *dst = v;
}

__global__ void k_set_step(long long *dst, long long v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0)
        *dst = v;
}

inline int blocks_for(long long n, int per) { return (int)((n + per - 1) / per); }

template <int TILE, int NL>
void canon_tile(const DevBufs &b, int cap, hipStream_t s)
{
    CanonArgs a{};
    a.tile_first = b.tile_first[tile_index(TILE)];
    a.trow = b.trow;
    a.stage_raw = b.stage_raw;
    a.stage = b.stage;
    a.stage_cnt = b.stage_cnt;
    a.rows = b.flist16;
    a.skin_cnt = b.list_cnt;
    a.tent = b.tent;
    a.skin_flag = b.skin_flag;
    a.skin16 = reinterpret_cast<uint4 *>(b.list16);
    a.skin_len = b.skin_len;
    a.skin_ord = b.skin_ord;
    a.ltop = b.ltop;
    a.tile_top = b.tile_top;
    a.stage16 = b.stage16;
    a.cap = cap;
    a.top_rounds = top_rounds(b.max_bonds, b.max_natives, NL);
    hipLaunchKernelGGL((k_canon<TILE, NL>), dim3(b.n_tiles[tile_index(TILE)] * Rows<TILE, NL>::W), dim3(256), 0, s, a);
}

FilterArgs filter_args(const DevBufs &b, int cur, int cap, int tile, int n_cells, const FixDev &fix, float rc2)
{
    FilterArgs a{};
    a.tile_first = b.tile_first[tile_index(tile)];
    a.pos = b.pos[cur];
    a.stage = b.stage;
    a.stage_cnt = b.stage_cnt;
    a.skin16 = reinterpret_cast<const uint4 *>(b.list16);
    a.skin_len = b.skin_len;
    a.skin_ord = b.skin_ord;
    a.ltop = b.ltop;
    a.tile_top = b.tile_top;
    a.list16 = reinterpret_cast<uint2 *>(b.flist16);
    a.llen = b.llen;
    a.grho = b.grho;
    a.wg_rec = b.wg_rec;
    a.cell_count = b.cell_count;
    a.skin_flag = b.skin_flag;
    a.fixed = b.fix[cur];
    a.place = b.place;
    a.rc2 = rc2;
    a.fix = fix;
    a.cap = cap;
    a.n_cells = n_cells;
    a.top_rounds = top_rounds(b.max_bonds, b.max_natives, lanes_for(tile, b.n_tiles[tile_index(tile)]));
    return a;
}

// Calls f with the tile size and the lanes per residue as compile-time constants.
template <class F>
void with_rows(int tile, int n_tiles, F &&f)
{
    using std::integral_constant;
    switch (tile) {
    case 64:
        switch (lanes_for(64, n_tiles)) {
        case 16: f(integral_constant<int, 64>{}, integral_constant<int, 16>{}); break;
        case 8: f(integral_constant<int, 64>{}, integral_constant<int, 8>{}); break;
        default: f(integral_constant<int, 64>{}, integral_constant<int, 4>{}); break;
        }
        break;
    case 128: f(integral_constant<int, 128>{}, integral_constant<int, 2>{}); break;
    default: f(integral_constant<int, 256>{}, integral_constant<int, 1>{}); break;
    }
}

int workgroups(const DevBufs &b, int tile)
{
    const int n = b.n_tiles[tile_index(tile)];
    return n * (tile * lanes_for(tile, n) / 256);
}

// Lanes of a search workgroup by the number of 64-residue tiles.  A tile's
// search is a chain of short phases that four waves alone on a CU take 44 us
// for, so while every tile has a CU to itself 16 waves share it, and up to a
// few tiles a CU eight.  Whole search (with the order of its rows), us with
// 256, 512 and 1,024 lanes: 16 tiles 109, 86, 77; 76 tiles at protein density
// 247, 179, 147; 320 tiles 105, 91, 104; 1,200 tiles 206, 208, 251.
constexpr int SEARCH_1024 = 256, SEARCH_512 = 640;

template <int TILE>
void rebuild_tile(const DevBufs &b, int cur, int n, int cap, const GridDev &g, float rc2, int multi,
                  hipStream_t s, bool advance, int period)
{
    BuildArgs a{};
    a.step_base = advance ? b.step_base : nullptr;
    a.step_next = b.step_next;
    a.period = period;
    a.tile_first = b.tile_first[tile_index(TILE)];
    a.pos = b.pos[cur];
    a.cell_of = b.cell_of;
    a.count = b.cell_count;
    a.cells = b.cells;
    a.traj_cell = b.traj_cell;
    a.traj_lo = b.traj_lo;
    a.traj_hi = b.traj_hi;
    a.trow = b.trow;
    a.tent = b.tent;
    a.list_cnt = b.list_cnt;
    a.list16 = b.flist16;
    a.stage = b.stage_raw;
    a.stage_cnt = b.stage_cnt;
    a.err = b.err;
    a.skin_flag = b.skin_flag;
    a.hi_skin = b.hi_skin;
    a.stats = b.list_stats;
    a.g = g;
    a.rc2 = rc2;
    a.n = n;
    a.cap = cap;
    const int nt = b.n_tiles[tile_index(TILE)];
    auto run = [&](auto NT) {
        constexpr int N = decltype(NT)::value;
        if (multi)
            hipLaunchKernelGGL((k_tile_build<TILE, true, N>), dim3(nt), dim3(N), 0, s, a);
        else
            hipLaunchKernelGGL((k_tile_build<TILE, false, N>), dim3(nt), dim3(N), 0, s, a);
    };
    if constexpr (TILE == 64) {
        if (nt <= SEARCH_1024)
            return run(std::integral_constant<int, 1024>{});
        if (nt <= SEARCH_512)
            return run(std::integral_constant<int, 512>{});
    }
    run(std::integral_constant<int, 256>{});
}

template <bool ENERGY, int MODE, bool FIRST = false>
void tile_dispatch(const DevBufs &b, int tile, const TileArgs &a, hipStream_t s)
{
    const int blocks = ((a.n_wg + 7) / 8) * 8;
    with_rows(tile, b.n_tiles[tile_index(tile)], [&](auto T, auto NL) {
        hipLaunchKernelGGL((k_tile_step<decltype(T)::value, decltype(NL)::value, ENERGY, MODE, FIRST>), dim3(blocks),
                           dim3(256), 0, s, a);
    });
}

}  // namespace

void launch_rebuild(const DevBufs &b, int cur, int n, int cap, int tile, const GridDev &g, const FixDev &fix,
                    float rc2, float rs2, int multi, hipStream_t s, bool advance_step_base, int list_every,
                    bool binned, bool filter)
{
    if (!binned)
        launch_bin_all(b, cur, n, g, fix, s);  // not binned by a period's last step kernel
    with_rows(tile, b.n_tiles[tile_index(tile)], [&](auto T, auto NL) {
        constexpr int TILE = decltype(T)::value;
        rebuild_tile<TILE>(b, cur, n, cap, g, rs2, multi, s, advance_step_base, list_every);
        canon_tile<TILE, decltype(NL)::value>(b, cap, s);
        if (filter)
            hipLaunchKernelGGL((k_filter<TILE, decltype(NL)::value>), dim3(workgroups(b, tile)), dim3(256), 0, s,
                               filter_args(b, cur, cap, tile, g.n_cells, fix, rc2));
    });
}

void launch_bin_all(const DevBufs &b, int cur, int n, const GridDev &g, const FixDev &fix, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear, dim3(blocks_for(g.n_cells, WG)), dim3(WG), 0, s, b.cell_count, g.n_cells);
    hipLaunchKernelGGL(k_bin_all, dim3(blocks_for(n, WG)), dim3(WG), 0, s, b.pos[cur], n, g, b.traj_cell,
                       b.cell_count, b.cells, b.cell_of, b.err, b.fix[cur], fix);
}

void launch_force_skin(const DevBufs &b, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_flag, dim3(1), dim3(64), 0, s, b.skin_flag, 1u);
}

void launch_distrust_copies(const DevBufs &b, int cur, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_flag, dim3(1), dim3(64), 0, s, b.err + MOVED + cur, 1u);
}

void launch_pair_step(const DevBufs &b, int cur, int n, int cap, int tile, const StepConsts &c,
                      const FixDev &fix, const TipDev &tip, int has_pull, bool energy, int mode, const long long *step_base,
                      long long step_off, float check_thr2, hipStream_t s, const float4 *vel,
                      const UdConsts &ud, const GridDev *bin_grid)
{
    PairArgs a{};
    a.tile_first = b.tile_first[tile_index(tile)];
    a.pin = b.pos[cur];
    a.trow = b.trow;
    a.tent = b.tent;
    a.llen = b.llen;
    a.grho = b.grho;
    a.list16 = reinterpret_cast<const uint2 *>(b.flist16);
    a.stage = b.stage;
    a.stage_cnt = b.stage_cnt;
    a.facc = b.facc;
    a.eacc = b.eacc;
    a.err = b.err;
    a.cap = cap;
    a.c = c;
    with_rows(tile, b.n_tiles[tile_index(tile)], [&](auto T, auto NL) {
        const dim3 grid(workgroups(b, tile));
        if (energy)
            hipLaunchKernelGGL((k_pair_forces<decltype(T)::value, decltype(NL)::value, true>), grid, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((k_pair_forces<decltype(T)::value, decltype(NL)::value, false>), grid, dim3(256), 0, s, a);
    });
    PairUpdArgs u{};
    u.pin = b.pos[cur];
    u.pout = b.pos[cur ^ 1];
    u.qout = b.fix[cur ^ 1];
    u.fix = fix;
    u.facc = b.facc;
    u.eacc = b.eacc;
    u.noise_key = b.noise_key;
    u.pull_slot = b.pull_slot;
    u.pulls = b.pulls;
    u.res_energy = b.res_energy;
    u.fout = b.fout;
    u.err = b.err;
    u.step_base = step_base;
    u.hi_skin = b.hi_skin;
    u.skin_flag = b.skin_flag;
    u.place = b.place;
    u.layer = cur;
    u.step_off = step_off;
    u.check_thr2 = mode == 0 ? check_thr2 : 0.0f;
    u.vel = const_cast<float4 *>(vel);
    u.ud = ud;
    u.do_bin = (mode == 0 && bin_grid) ? 1 : 0;
    if (bin_grid)
        u.g = *bin_grid;
    u.traj_cell = b.traj_cell;
    u.cell_count = b.cell_count;
    u.cells = b.cells;
    u.cell_of = b.cell_of;
    u.n = n;
    u.has_pull = has_pull;
    u.c = c;
    u.tip = tip;
    const dim3 g(blocks_for(n, WG));
    if (mode == 1) {
        if (energy)
            hipLaunchKernelGGL((k_pair_update<true, 1>), g, dim3(WG), 0, s, u);
        else
            hipLaunchKernelGGL((k_pair_update<false, 1>), g, dim3(WG), 0, s, u);
    } else {
        if (energy)
            hipLaunchKernelGGL((k_pair_update<true, 0>), g, dim3(WG), 0, s, u);
        else
            hipLaunchKernelGGL((k_pair_update<false, 0>), g, dim3(WG), 0, s, u);
    }
}

void launch_step(const DevBufs &b, int cur, int n, int cap, int tile, const StepConsts &c,
                 const FixDev &fix, const TipDev &tip, int has_pull, bool energy, int mode, const long long *step_base,
                 long long step_off, float check_thr2, hipStream_t s, int force_mode, float ud_kick,
                 const GridDev *bin_grid, float filter_rc2, int n_cells)
{
    // underdamped when ud_kick > 0 (velocities in b.vel)
    const float4 *vel = ud_kick > 0.0f ? b.vel : nullptr;
    UdConsts ud{ud_kick, c.ud_c1, c.ud_c2, (float)(0.5 * c.h)};
    if (force_mode == 1) {
        launch_pair_step(b, cur, n, cap, tile, c, fix, tip, has_pull, energy, mode, step_base, step_off,
                         check_thr2, s, vel, ud, bin_grid);
        return;
    }
    TileArgs a{};
    a.vel = const_cast<float4 *>(vel);
    a.ud = ud;
    a.do_bin = (mode == 0 && bin_grid) ? 1 : 0;
    if (bin_grid)
        a.g = *bin_grid;
    a.traj_cell = b.traj_cell;
    a.cell_count = b.cell_count;
    a.cells = b.cells;
    a.cell_of = b.cell_of;
    a.hi_skin = b.hi_skin;
    a.skin_flag = b.skin_flag;
    a.place = b.place;
    a.layer = cur;
    a.check_thr2 = mode == 0 ? check_thr2 : 0.0f;
    a.n_wg = workgroups(b, tile);
    a.pin = b.pos[cur];
    a.pout = b.pos[cur ^ 1];
    a.qin = b.fix[cur];
    a.qout = b.fix[cur ^ 1];
    a.fix = fix;
    a.list16 = reinterpret_cast<const uint2 *>(b.flist16);
    a.llen = b.llen;
    a.grho = b.grho;
    a.wg_rec = b.wg_rec;
    a.ltop = b.ltop;
    a.stage = b.stage;
    a.stage16 = b.stage16;
    a.noise_key = b.noise_key;
    a.pull_slot = b.pull_slot;
    a.pulls = b.pulls;
    a.res_energy = b.res_energy;
    a.fout = b.fout;
    a.err = b.err;
    a.step_base = step_base;
    a.step_off = step_off;
    const int nl = lanes_for(tile, b.n_tiles[tile_index(tile)]);
    a.chunks = lane_chunks(cap, nl);
    a.top_rounds = top_rounds(b.max_bonds, b.max_natives, nl);
    a.has_pull = has_pull;
    a.c = c;
    a.tip = tip;
    if (mode == 0 && filter_rc2 > 0.0f) {
        // the first step after a rebuild, which filters the skin rows itself
        // (never a binning step: the callers bin only at a period's end)
        a.f = filter_args(b, cur, cap, tile, n_cells, fix, filter_rc2);
        if (energy)
            tile_dispatch<true, 0, true>(b, tile, a, s);
        else
            tile_dispatch<false, 0, true>(b, tile, a, s);
        return;
    }
    if (mode == 1) {
        if (energy)
            tile_dispatch<true, 1>(b, tile, a, s);
        else
            tile_dispatch<false, 1>(b, tile, a, s);
    } else {
        if (energy)
            tile_dispatch<true, 0>(b, tile, a, s);
        else
            tile_dispatch<false, 0>(b, tile, a, s);
    }
}

// Two lanes a residue for packs of 256 as long as all of them are resident at
// once so (two a CU): such packs leave most of a CU's issue slots idle.  us a
// step with one lane and two: 60 chains of 137 residues 7.7 and 6.7, 384 8.7
// and 8.2, 510 8.8 and 8.2; 250 of 250 9.4 and 8.0, 510 10.9 and 10.2; 1,000
// of 60 6.3 and 5.8.  With packs of 512 the sums fill the CU already and the
// rebuild's masks cost more than they bring (200 chains of 50-500 10.3 and
// 11.0).
bool batch_split(int n_packs, int wg) { return wg == 256 && n_packs <= 512; }

void launch_batch(const DevBufs &b, int cur, int n_packs, int wg, int cap, const StepConsts &c,
                  const FixDev &fix, const TipDev &tip, int has_pull, float rc2, int list_every, long long energy_every,
                  int n_steps, int stale, int mode, const long long *step_base, long long step_off,
                  hipStream_t s, const float *tscale)
{
    BatchArgs a{};
    a.pin = b.pos[cur];
    a.pout = b.pos[cur ^ 1];
    a.trow = b.trow;
    a.tent = b.tent;
    a.pack_off = b.pack_off;
    a.slot_res = b.slot_res;
    a.traj_lo = b.traj_lo;
    a.traj_hi = b.traj_hi;
    a.stream_ids = b.stream_ids;
    a.pull_slot = b.pull_slot;
    a.pulls = b.pulls;
    a.list = b.list16;
    a.list_cnt = b.list_cnt;
    a.place = b.place;
    a.moved = b.pack_moved;
    a.done = b.pack_done;
    a.energy = b.energy;
    a.f_ext = b.f_ext;
    a.fout = b.fout;
    a.err = b.err;
    a.step_base = step_base;
    a.step_off = step_off;
    a.energy_every = energy_every;
    a.n_steps = n_steps;
    a.list_every = list_every;
    a.stale = stale;
    a.cap = cap;
    a.has_pull = has_pull;
    a.c = c;
    a.fix = fix;
    a.tip = tip;
    a.rc2 = rc2;
    a.tscale = tscale;
    const dim3 grid(n_packs);
    auto run = [&](auto W, auto F) {
        constexpr int WGS = decltype(W)::value;
        constexpr bool FAR = decltype(F)::value;
        if (mode == 1)
            hipLaunchKernelGGL((k_batch<WGS, 1, 1, FAR>), grid, dim3(WGS), 0, s, a);
        else if (mode == 2)
            hipLaunchKernelGGL((k_batch<WGS, 2, 1, FAR>), grid, dim3(WGS), 0, s, a);
        else
            hipLaunchKernelGGL((k_batch<WGS, 0, 1, FAR>), grid, dim3(WGS), 0, s, a);
    };
    auto sized = [&](auto F) {
        switch (wg) {
        case 256: run(std::integral_constant<int, 256>{}, F); break;
        case 512: run(std::integral_constant<int, 512>{}, F); break;
        default: run(std::integral_constant<int, 1024>{}, F); break;
        }
    };
    if (fix.list_far)
        sized(std::true_type{});
    else if (mode == 0 && batch_split(n_packs, wg))
        hipLaunchKernelGGL((k_batch<256, 0, 2, false>), grid, dim3(512), 0, s, a);
    else
        sized(std::false_type{});
    const dim3 exact(std::min(n_packs, EXACT_GRID));
    if (mode == 1)
        hipLaunchKernelGGL(k_batch_exact<1>, exact, dim3(1024), 0, s, a, n_packs);
    else
        hipLaunchKernelGGL(k_batch_exact<2>, exact, dim3(1024), 0, s, a, n_packs);
}

void launch_exchange(const DevBufs &b, int n_rep, int n_groups, double kbt_ref, long long round,
                     unsigned key0, unsigned key1, hipStream_t s)
{
    const int pairs = std::max(n_rep / 2, 1);
    hipLaunchKernelGGL(k_exchange, dim3(blocks_for((long long)n_groups * pairs, WG)), dim3(WG), 0, s, b.energy,
                       b.re_kbt, n_rep, n_groups, b.re_tidx, b.re_tscale, kbt_ref, round, key0, key1, b.re_stats);
}

void launch_add_step(long long *base, long long k, hipStream_t s)
{
    hipLaunchKernelGGL(k_add_step, dim3(1), dim3(64), 0, s, base, k);
}

void launch_reduce_energy(const DevBufs &b, int n_traj, hipStream_t s)
{
    hipLaunchKernelGGL(k_reduce_chunks, dim3(b.n_chunks), dim3(WG), 0, s, b.res_energy, b.chunk_lo,
                       b.chunk_sum);
    hipLaunchKernelGGL(k_reduce_energy, dim3(blocks_for((long long)n_traj * 64, WG)), dim3(WG), 0, s,
                       b.chunk_sum, b.chunk_first, n_traj, b.energy, b.f_ext);
}

void launch_noise(const DevBufs &b, int cur, int n, const StepConsts &c, long long step, uint4 *words,
                  float4 *g, hipStream_t s)
{
    hipLaunchKernelGGL(k_noise, dim3(blocks_for(n, WG)), dim3(WG), 0, s, b.pos[cur], n, b.stream_ids,
                       c.key0, c.key1, step, words, g);
}

void launch_set_step(long long *dst, long long value, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(64), 0, s, dst, value);
}

}  // namespace sop
