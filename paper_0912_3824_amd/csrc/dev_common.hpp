#pragma once
// Device code shared by the HIP kernels of libmdx for gfx950 (wave64):
// work-item walkers, word conversions and the per-precision particle state.
//
// Overview of the kernels (step.hip, rebuild.hip, aux_kernels.hip):
//
// One MD step (Sec. 2.2, velocity Verlet with Verlet lists) is one fused
// launch of k_step plus two rebuild kernels (one, k_rebuild, in small pools of
// one slot that do not rebuild too often) that exit at once unless the
// replica's maximum displacement since its last list build exceeded skin/2:
//
//   k_step<P>    per particle: force over its Verlet list (FP32 pair term,
//                sum in the precision P), second half-kick of step n (full-
//                step velocity), first half-kick of step n+1, drift,
//                fixed-point snapshot of the new position, displacement test
//                against the list's reference position, and the count of the
//                particle's new cell (for the sort, Sec. 2.2 cell binning).
//                The sort key is the cell within the particle's species
//                plane: a binary mixture is stored as all A particles by
//                cell, then all B particles by cell.
//   k_permute<P> per cell (one wave): cell starts from the counts, then the
//                stable counting-sort scatter.  Members of a new cell come from the 27
//                surrounding old cells of the same plane (a
//                particle moves less than one cell between builds); a ballot
//                over them in old slot order gives each its new slot.  The
//                whole particle record is gathered into the scratch arena,
//                positions folded back into the box.
//   k_build<P>   per share of a cell's members (one wave): their lists over the
//                own cell and then the 13 opposite cell pairs (Sec. 4.1), the
//                distance tests on the matrix cores; the sorted records are
//                copied back from scratch.
//
// Bitwise determinism: lists are in a canonical order (own cell, then +o/-o
// pairs; inside a cell the A members, then the B members, in slot order), the sort is stable, each particle sums
// its own list sequentially, and no floating-point atomics are used.  The
// result for a replica therefore does not depend on launch shapes or on
// other replicas in the pool.
#include "md_dev.hpp"
#include "kernels.hpp"

#define LAUNCH_CHECK() return hipGetLastError()

// --------------------------------------------------------------- utilities
__device__ __forceinline__ int remap_block(int b, int nblk, int on)
{
    // Consecutive tiles to one XCD: workgroups are dealt round-robin over
    // the 8 XCDs, so block b runs on XCD b % 8.
    if (!on) return b;
    int per = nblk >> 3;
    if (b < (per << 3)) return (b & 7) * per + (b >> 3);
    return b;
}

__device__ __forceinline__ int slot_of_meta(uint32_t w) { return (int)((w & 0x7FFFFFFFu) >> SLOT_SHIFT); }

// Rank of cell c (= x + nd (y + nd z)) in the replica's cell order: itself
// in row-major order, else from the replica's rank table (a space-filling
// curve through the cells).
__device__ __forceinline__ int cell_rank(int c, const RepDev &r, const int *corder)
{
    return r.curve ? corder[r.coff + c] : c;
}

__device__ __forceinline__ int find_item_slot(const int *pref, int nslots, int item)
{
    // pref[0..nslots] non-decreasing; find s with pref[s] <= item < pref[s+1]
    int lo = 0, hi = nslots;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (pref[mid] <= item) lo = mid; else hi = mid;
    }
    return lo;
}

// Work-item walk of the rebuild kernels: the items of the slots on the
// rebuild list, which k_step writes (k_enlist for a rebuild asked for by the
// host).  items(slot) is a slot's item count, `unit` this worker's index
// among `nunits` workers; visit(slot, item) is called for each item assigned
// to it.  Consecutive slots start on different workers so that small replicas
// spread over the grid.  The slots and their item counts are read 64 at a
// time, one per lane (a few round trips to memory however many replicas
// rebuild), then walked from registers; visit is called from one place only,
// so that its code is emitted once.
template <class N, class F>
__device__ __forceinline__ void for_items(const int *rlist, N items, int unit, int nunits, F visit)
{
    const int cnt = rlist[0];
    const int lane = __lane_id();
    int cum = 0;
    for (int base = 0; base < cnt; base += 64) {
        const int li = base + lane;
        int sl = 0, its = 0;
        if (li < cnt) {
            sl = rlist[1 + li];
            its = items(sl);
        }
        const int m = min(64, cnt - base);
        for (int k = 0; k < m; ++k) {
            const int n = __builtin_amdgcn_readlane(its, k);
            const int s = __builtin_amdgcn_readlane(sl, k);
            int first = unit - cum % nunits;
            first += first < 0 ? nunits : 0;
            for (int it = first; it < n; it += nunits) visit(s, it);
            cum += n;
        }
    }
}

// A uniform index into memory that no kernel writes while this one runs:
// scalar loads.
template <class T> __device__ __forceinline__ T ld_uniform(const T *p, int k)
{
    typedef const __attribute__((address_space(4))) int CW;
    struct Words { int w[sizeof(T) / 4]; } v;
    CW *q = (CW *)(uintptr_t)(p + k);
#pragma unroll
    for (unsigned u = 0; u < sizeof(T) / 4; ++u) v.w[u] = q[u];
    T t;
    __builtin_memcpy(&t, &v, sizeof t);
    return t;
}

__device__ __forceinline__ uint4 dbl2_to_u4(double a, double b)
{
    uint4 u;
    unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    u.x = (uint32_t)x; u.y = (uint32_t)(x >> 32); u.z = (uint32_t)y; u.w = (uint32_t)(y >> 32);
    return u;
}
__device__ __forceinline__ void u4_to_dbl2(uint4 u, double &a, double &b)
{
    a = __longlong_as_double(((unsigned long long)u.y << 32) | u.x);
    b = __longlong_as_double(((unsigned long long)u.w << 32) | u.z);
}

// Order this wave's LDS accesses (no other wave shares the data).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Position relative to the centre of the particle's own cell, in units of
// 1 / CELL_UNITS of the cell edge: the fraction of X nd 2^-32 (fixed point),
// or of the double position, as the sort counted it (dbl_cell_offset1).
template <int P>
__device__ __forceinline__ void cell_units(const RepDev &r, const uint4 &a, const uint4 &b, float u[3])
{
    if constexpr (P == PREC_FP64) {
        double x[3], w;
        u4_to_dbl2(a, x[0], x[1]);
        u4_to_dbl2(b, x[2], w);
#pragma unroll
        for (int d = 0; d < 3; ++d) u[d] = (float)dbl_cell_offset1(x[d], r.L, r.invL, r.nd) * CELL_UNITS;
    } else {
        const uint32_t X[3] = {a.x, a.y, a.z};
#pragma unroll
        for (int d = 0; d < 3; ++d)
            u[d] = (float)(int)((X[d] * (uint32_t)r.nd) ^ 0x80000000u) * (CELL_UNITS / 4294967296.0f);
    }
}

// Candidate record of the list build: position in cell units and its squared
// length, each as two half-precision words (high words x, y, z, low words x,
// y, z, then the square's). 
__device__ __forceinline__ unsigned half2_bits(_Float16 a, _Float16 b)
{
    return (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
}
template <int P>
__device__ __forceinline__ uint4 cand_record(const RepDev &r, const uint4 &a, const uint4 &b)
{
    float u[3];
    cell_units<P>(r, a, b, u);
    const float s = __builtin_fmaf(u[0], u[0], __builtin_fmaf(u[1], u[1], u[2] * u[2]));
    const _Float16 xh = (_Float16)u[0], yh = (_Float16)u[1], zh = (_Float16)u[2], sh = (_Float16)s;
    const _Float16 xl = (_Float16)(u[0] - (float)xh), yl = (_Float16)(u[1] - (float)yh),
                   zl = (_Float16)(u[2] - (float)zh), sl = (_Float16)(s - (float)sh);
    return make_uint4(half2_bits(xh, yh), half2_bits(zh, xl), half2_bits(yl, zl), half2_bits(sh, sl));
}

// Cell of a position in the box (its snapshot words).
template <int P> __device__ __forceinline__ int cell_of(const RepDev &r, const uint4 &a, const uint4 &b)
{
    if constexpr (P == PREC_FP64) {
        double x, y, z, w;
        u4_to_dbl2(a, x, y);
        u4_to_dbl2(b, z, w);
        return dbl_cell(x, y, z, r.L, r.invL, r.nd);
    } else return fixed_cell(a.x, a.y, a.z, r.nd);
}

// The position in cell units of a record, to 2^-17.
__device__ __forceinline__ void record_units(const uint4 &c, float u[3])
{
    auto half = [](unsigned w) { return (float)__builtin_bit_cast(_Float16, (unsigned short)w); };
    u[0] = half(c.x) + half(c.y >> 16);
    u[1] = half(c.x >> 16) + half(c.z);
    u[2] = half(c.y) + half(c.z >> 16);
}

// ------------------------------------------------------- per-precision state
template <int P> struct State;

template <> struct State<PREC_FP32> {
    float x, y, z, vx, vy, vz;
    __device__ void load(const KArena &A, int i)
    {
        float4 a = ((const float4 *)A.st[0])[i], b = ((const float4 *)A.st[1])[i];
        x = a.x; y = a.y; z = a.z; vx = b.x; vy = b.y; vz = b.z;
    }
    __device__ void store(const KArena &A, int i) const
    {
        ((float4 *)A.st[0])[i] = make_float4(x, y, z, 0.0f);
        ((float4 *)A.st[1])[i] = make_float4(vx, vy, vz, 0.0f);
    }
};

template <> struct State<PREC_DS> {
    dsf x, y, z, vx, vy, vz;
    __device__ void load(const KArena &A, int i)
    {
        float4 a = ((const float4 *)A.st[0])[i], b = ((const float4 *)A.st[1])[i],
               c = ((const float4 *)A.st[2])[i];
        x = {a.x, a.w}; y = {a.y, b.x}; z = {a.z, b.y};
        vx = {b.z, c.y}; vy = {b.w, c.z}; vz = {c.x, c.w};
    }
    __device__ void store(const KArena &A, int i) const
    {
        ((float4 *)A.st[0])[i] = make_float4(x.hi, y.hi, z.hi, x.lo);
        ((float4 *)A.st[1])[i] = make_float4(y.lo, z.lo, vx.hi, vy.hi);
        ((float4 *)A.st[2])[i] = make_float4(vz.hi, vx.lo, vy.lo, vz.lo);
    }
};

struct StateD {
    double x, y, z, vx, vy, vz;
    __device__ void load(const KArena &A, int i)
    {
        double2 a = ((const double2 *)A.st[0])[i], b = ((const double2 *)A.st[1])[i],
                c = ((const double2 *)A.st[2])[i];
        x = a.x; y = a.y; z = b.x; vx = b.y; vy = c.x; vz = c.y;
    }
    __device__ void store(const KArena &A, int i) const
    {
        ((double2 *)A.st[0])[i] = make_double2(x, y);
        ((double2 *)A.st[1])[i] = make_double2(z, vx);
        ((double2 *)A.st[2])[i] = make_double2(vy, vz);
    }
};
template <> struct State<PREC_MIX> : StateD {};
template <> struct State<PREC_FP64> : StateD {};
