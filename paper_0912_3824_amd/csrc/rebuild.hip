// Neighbour-list rebuild kernels (cell count, stable sort, list build)
// and their launchers.
#include <type_traits>

#include "dev_common.hpp"

// ------------------------------------------------------------ k_count
// Cell counts for a rebuild forced from the host (md_rebuild_neighbours).
template <int P>
__global__ void k_count(const CountArgs a)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.P) return;
    constexpr int NS = Traits<P>::NS;
    uint4 s0 = a.snap[i];
    uint32_t meta;
    double x = 0, y = 0, z = 0, w = 0;
    if (NS == 2) {
        u4_to_dbl2(s0, x, y);
        u4_to_dbl2(a.snap[(size_t)a.P + i], z, w);
        meta = meta_of_bits(w);
    } else meta = s0.w;
    if (meta == NO_SLOT) return;
    int r = slot_of_meta(meta);
    if (r >= a.max_slots) return;
    if (!a.ctl[r].z) return;
    RepDev rp = a.rep[r];
    int cell;
    if (NS == 2) cell = dbl_cell(x, y, z, rp.L, rp.invL, rp.nd);
    else cell = rp.nd == 1 ? 0 : fixed_cell(s0.x, s0.y, s0.z, rp.nd);
    atomicAdd(a.count + rp.coff + sort_key(cell_rank(cell, rp, a.corder), meta, rp.planes, rp.nd), 1);
}

// ------------------------------------------------------------ k_enlist
// Rebuild list of a rebuild or list build asked for by the host: `slot`, unless
// its input was found wrong while it was attached, or every attached slot
// (slot < 0).
__global__ void __launch_bounds__(64) k_enlist(int *rlist, int *sync, const Ctl *ctl, const int *status,
                                               int max_slots, int slot)
{
    const int lane = threadIdx.x;
    if (lane < SYNC_WORDS / SYNC_STRIDE) sync[lane * SYNC_STRIDE] = 0;
    int cnt = 0;
    for (int base = 0; base < max_slots; base += 64) {
        const int s = base + lane;
        const bool in = s < max_slots && (slot < 0 ? ctl[s].z != 0
                                               : s == slot && !(status[s] & (ST_BAD_INPUT | ST_BAD_SPECIES)));
        const unsigned long long m = __ballot(in);
        if (in) rlist[1 + cnt + __popcll(m & ((1ull << lane) - 1ull))] = s;
        cnt += __popcll(m);
    }
    if (lane == 0) rlist[0] = cnt;
}

// Rank of the cell at an offset of at most one from cell (cx, cy, cz).
__device__ __forceinline__ int offset_rank(int cx, int cy, int cz, int dx, int dy, int dz, const RepDev &rp,
                                           const int *corder)
{
    const int nd = rp.nd;
    int x = cx + dx, y = cy + dy, z = cz + dz;
    x += x < 0 ? nd : 0; x -= x >= nd ? nd : 0;
    y += y < 0 ? nd : 0; y -= y >= nd ? nd : 0;
    z += z < 0 ? nd : 0; z -= z >= nd ? nd : 0;
    return cell_rank(x + nd * (y + nd * z), rp, corder);
}

// ------------------------------------------------------------ k_permute
// One wave per new cell: stable scatter of its members into scratch, in two
// phases.  The test phase reads the snapshots of the candidates (the members
// of the 27 neighbouring old cells, in old slot order) PERM_U x 64 at a time,
// all in flight together, and lists each member found with its destination
// in LDS; it issues no store.  The move phase then loads the listed members
// and folds and stores them.  A cell's membership is thus found in a few
// round trips to memory instead of one load-then-store pass per 256
// candidates (on this hardware one counter tracks loads and stores alike, so
// a load issued after a store also waits for that store).
#define PERM_U 8                     // candidate tests per lane in flight
#define PERM_LIST (64 + 64 * PERM_U) // listed members per wave before a move phase
#define PERM_BLOCK 256
template <int P> struct Moved {
    uint4 st[Traits<P>::NW];
    int4 meta;
    uint4 snap; // the snapshot (fixed point), or its second word (double)
};

template <int P>
__device__ __forceinline__ void move_load(const PermArgs &a, int q, Moved<P> &mv)
{
    constexpr int NW = Traits<P>::NW, NS = Traits<P>::NS;
#pragma unroll
    for (int w = 0; w < NW; ++w) mv.st[w] = a.A.st[w][q];
    mv.meta = a.A.meta[q];
    mv.snap = NS == 1 ? a.snap[q] : a.snap[(size_t)a.A.P + q];
}

__device__ __forceinline__ float4 u4_as_f4(uint4 u)
{
    return make_float4(__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w));
}
__device__ __forceinline__ uint4 f4_as_u4(float4 f)
{
    return make_uint4(__float_as_uint(f.x), __float_as_uint(f.y), __float_as_uint(f.z), __float_as_uint(f.w));
}

// Fold the member's position into [0, L) (counting the image shift in its
// meta word) and store it at scratch slot dst.
template <int P>
__device__ __forceinline__ void move_store(const PermArgs &a, const RepDev &rp, const Moved<P> &mv, int dst)
{
    constexpr int NS = Traits<P>::NS;
    int4 m = mv.meta;
    int ix = 0, iy = 0, iz = 0;
    int *im[3] = {&ix, &iy, &iz};
    if constexpr (P == PREC_FP32) {
        float4 p = u4_as_f4(mv.st[0]);
        float *c[3] = {&p.x, &p.y, &p.z};
#pragma unroll
        for (int d = 0; d < 3; ++d) { // fold by the exact edge (the box need not be a float)
            if (*c[d] < 0.0f) { *c[d] = (float)((double)*c[d] + rp.L); *im[d] -= 1; }
            if ((double)*c[d] >= rp.L) { *c[d] = (float)((double)*c[d] - rp.L); *im[d] += 1; }
        }
        a.sc_st[0][dst] = f4_as_u4(p);
        a.sc_st[1][dst] = mv.st[1];
    } else if constexpr (P == PREC_DS) {
        const float4 w0 = u4_as_f4(mv.st[0]), w1 = u4_as_f4(mv.st[1]);
        dsf x = {w0.x, w0.w}, y = {w0.y, w1.x}, z = {w0.z, w1.y};
        const dsf L = {rp.L_hi, rp.L_lo};
        dsf *c[3] = {&x, &y, &z};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (c[d]->hi < 0.0f) { *c[d] = ds_add(*c[d], L); *im[d] -= 1; }
            const dsf t = ds_sub(*c[d], L);
            if (t.hi >= 0.0f) { *c[d] = t; *im[d] += 1; }
        }
        a.sc_st[0][dst] = f4_as_u4(make_float4(x.hi, y.hi, z.hi, x.lo));
        a.sc_st[1][dst] = f4_as_u4(make_float4(y.lo, z.lo, w1.z, w1.w));
        a.sc_st[2][dst] = mv.st[2];
    } else {
        if constexpr (NS == 2) { // (of the position as the sort counted it, before the fold)
            if (rp.bmode == BUILD_CELLS) a.cand[dst] = cand_record<P>(rp, mv.st[0], mv.st[1]);
        }
        double x, y, z, w;
        u4_to_dbl2(mv.st[0], x, y);
        u4_to_dbl2(mv.st[1], z, w);
        double *c[3] = {&x, &y, &z};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (*c[d] < 0.0) { *c[d] += rp.L; *im[d] -= 1; }
            if (*c[d] >= rp.L) { *c[d] -= rp.L; *im[d] += 1; }
        }
        a.sc_st[0][dst] = dbl2_to_u4(x, y);
        a.sc_st[1][dst] = dbl2_to_u4(z, w);
        a.sc_st[2][dst] = mv.st[2];
        if constexpr (NS == 2) { // the double snapshot, from the folded state
            double zz, ww;
            u4_to_dbl2(mv.snap, zz, ww);
            a.sc_snap[dst] = dbl2_to_u4(x, y);
            a.sc_snap[(size_t)a.A.P + dst] = dbl2_to_u4(z, ww);
        }
    }
    m.x += ix; m.y += iy; m.z += iz;
    a.sc_meta[dst] = m;
    if constexpr (NS == 1) {
        a.sc_snap[dst] = mv.snap;
        if (rp.bmode == BUILD_CELLS) a.cand[dst] = cand_record<P>(rp, mv.snap, mv.snap);
    }
}

template <int P>
__device__ __forceinline__ bool in_cell(const PermArgs &a, const RepDev &rp, int q, int c)
{
    constexpr int NS = Traits<P>::NS;
    if (NS == 2) {
        double x, y, z, w;
        u4_to_dbl2(a.snap[q], x, y);
        u4_to_dbl2(a.snap[(size_t)a.A.P + q], z, w);
        return dbl_cell(x, y, z, rp.L, rp.invL, rp.nd) == c;
    }
    const uint4 X = a.snap[q];
    return fixed_cell(X.x, X.y, X.z, rp.nd) == c;
}

struct PermLds { // one per wave
    int pref[55], pst[54], srt[27];
    int2 lst[PERM_LIST]; // (old slot, scratch slot) of the members found
};

// One new cell c (rank rc): plane-0 members go to [dst0, dst0 + want0),
// plane-1 members to [dst1, dst1 + want1).
template <int P>
__device__ __forceinline__ void permute_cell(const PermArgs &a, const RepDev &rp, PermLds &W, int s, int c, int dst0,
                                             int want0, int dst1, int want1)
{
    const int lane = __lane_id();
    const int nd = rp.nd, nc = nd * nd * nd, planes = rp.planes;
    const int *cs = a.cs + rp.coff;
    // the old cells that can hold members of new cell c, in ascending
    // rank: plane 0's, then plane 1's (so that the flattened candidates
    // are in old slot order); one range per lane
    const int nold = 27, nr = planes * nold;
    // rank the 27 neighbour cells (distinct for nd >= 3)
    int orank = 0x7fffffff;
    if (lane < 27) {
        const int cx = c % nd, cy = (c / nd) % nd, cz = c / (nd * nd);
        orank = offset_rank(cx, cy, cz, lane % 3 - 1, (lane / 3) % 3 - 1, lane / 9 - 1, rp, a.corder);
    }
    int before = 0;
    for (int l = 0; l < 27; ++l) before += __shfl(orank, l, 64) < orank;
    if (lane < 27) W.srt[before] = orank;
    wave_sync();
    int len = 0, st0 = 0;
    if (lane < nr) {
        const int pl = lane >= nold, kk = lane - pl * nold;
        const int oc = pl * nc + W.srt[kk];
        st0 = cs[oc];
        len = cs[oc + 1] - st0;
    }
    int incl = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane < nr) { W.pst[lane] = st0; W.pref[lane + 1] = incl; }
    if (lane == 0) W.pref[0] = 0;
    wave_sync();
    const int tot = W.pref[nr], tot0 = W.pref[nold];
    // move phase: every listed member, loaded before any is stored
    auto move_listed = [&](int n) {
        wave_sync();
        for (int k = lane; k < n; k += 64) {
            const int2 e = W.lst[k];
            Moved<P> mv;
            move_load<P>(a, e.x, mv);
            move_store<P>(a, rp, mv, e.y);
        }
        wave_sync();
    };
    int run0 = 0, run1 = 0, nl = 0;
    int r = 0; // range of the lane's current candidate (only moves forward)
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int b = 0; b < tot; b += 64 * PERM_U) {
        int q[PERM_U];
        bool m[PERM_U];
#pragma unroll
        for (int u = 0; u < PERM_U; ++u) {
            const int e = b + 64 * u + lane;
            q[u] = -1;
            if (e < tot) {
                while (r + 1 < nr && W.pref[r + 1] <= e) ++r;
                q[u] = W.pst[r] + (e - W.pref[r]);
            }
        }
#pragma unroll
        for (int u = 0; u < PERM_U; ++u) m[u] = q[u] >= 0 && in_cell<P>(a, rp, q[u], c);
        // list the members found, in candidate order (at most 64 x
        // PERM_U, so the list, emptied below once it holds more than
        // 64, never overflows)
#pragma unroll
        for (int u = 0; u < PERM_U; ++u) {
            const bool p1 = b + 64 * u + lane >= tot0;
            const unsigned long long bal0 = __ballot(m[u] && !p1), bal1 = __ballot(m[u] && p1);
            if (m[u]) {
                const int dst = p1 ? dst1 + run1 + __popcll(bal1 & below) : dst0 + run0 + __popcll(bal0 & below);
                W.lst[nl + __popcll((bal0 | bal1) & below)] = make_int2(q[u], dst);
            }
            run0 += __popcll(bal0);
            run1 += __popcll(bal1);
            nl += __popcll(bal0 | bal1);
        }
        if (nl > PERM_LIST - 64 * PERM_U) { move_listed(nl); nl = 0; }
    }
    move_listed(nl);
    // every particle counted in this cell must have come from a
    // neighbouring old cell; a shortfall means a particle jumped further
    if (lane == 0 && (run0 != want0 || run1 != want1)) atomicOr(a.status + s, 4);
}

// Sum of count[0 .. n) over the block's threads, this thread's share; 16
// loads in flight.
__device__ __forceinline__ int thread_sum(const int *count, int n)
{
    int sum = 0;
    for (int k = threadIdx.x; k < n; k += 16 * PERM_BLOCK) {
        int v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = k + u * PERM_BLOCK < n ? count[k + u * PERM_BLOCK] : 0;
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += v[u];
    }
    return sum;
}

// A block takes a range of cells, consecutive in the cell order: it sums the
// counts of the cells before them (so no scan runs as a launch of its own:
// an idle one costs every step 1.5 us, and at 1M particles the sums take a
// block about 15 us where one block's scan took 33 us with the chip idle
// beside it), then its waves take the range's cells in turn, and it writes
// the cell starts that the list build reads.
//
// The sort waits on chains of memory round trips rather than on issue.  In
// large pools of one slot, in double-single and FP64, it is compiled for 6
// waves per SIMD (at most 80 VGPRs) instead of the 4 its unconstrained register
// use allows: 1M particles 229 -> 195 us, 250,000 69 -> 58.  Replicas of up
// to 131,072 particles have few cells a wave, and there the registers that
// spill at 80 cost more than the waves give: 256 replicas at once 131 us at 4
// waves and 170 at 6, one of 64,000 24 and 28.  The FP32 and MIXED64 forms
// spill more and keep 4.
struct PermBlockLds {
    PermLds wave[PERM_BLOCK / 64];
    int red[3][PERM_BLOCK / 64];
};

// Cells per sort unit and sort units of a replica, for a grid of nblk blocks.
// A unit of a single-cell replica is PERM_BLOCK of its particles.
__device__ __forceinline__ int perm_range(int nc, int nblk)
{
    constexpr int WPB = PERM_BLOCK / 64;
    return WPB * ((nc + WPB * nblk - 1) / (WPB * nblk));
}
__device__ __forceinline__ int perm_units(const RepDev &rp, int nblk)
{
    const int range = rp.nd == 1 ? PERM_BLOCK : perm_range(rp.items3, nblk);
    return (rp.items3 + range - 1) / range;
}

template <int P>
__device__ __forceinline__ void permute_item(const PermArgs &a, const RepDev &rp, PermBlockLds &lds, int s, int item, int nblk)
{
    constexpr int WPB = PERM_BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nd = rp.nd, nc = nd * nd * nd, range = perm_range(nc, nblk);
    const bool two = rp.planes > 1;
    const int *cnt = a.count + rp.coff;
    int *out = a.cs_new + rp.coff;
    // A single cell is sorted by plane alone: every particle keeps its place
    // (one wave listing and moving 600 particles took 9 us more).
    if (nd == 1) {
        const int k = item * PERM_BLOCK + (int)threadIdx.x;
        if (k < rp.n) {
            Moved<P> mv;
            move_load<P>(a, rp.off + k, mv);
            move_store<P>(a, rp, mv, rp.off + k);
        }
        if (k == 0) {
            const int n0 = cnt[0], n1 = two ? cnt[1] : 0;
            out[0] = rp.off;
            out[1] = rp.off + n0;
            if (two) out[2] = rp.off + n0 + n1;
            if (n0 + n1 != rp.n) atomicOr(a.status + s, 4 | 2);
            if (a.cs[rp.coff + 1] - a.cs[rp.coff] != n0) atomicOr(a.status + s, 4);
            a.nreb[s] += 1;
        }
        return;
    }
    const int c0 = item * range, c1 = min(nc, c0 + range);
    // members before the range: of plane 0; of plane 0 in all and of plane 1
    int sum[3] = {thread_sum(cnt, c0), 0, 0};
    if (two) {
        sum[1] = thread_sum(cnt + c0, nc - c0);
        sum[2] = thread_sum(cnt + nc, c0);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum[q] += __shfl_xor(sum[q], o, 64);
        if (lane == 0) lds.red[q][wv] = sum[q];
    }
    __syncthreads();
    int base[2] = {0, 0};
#pragma unroll
    for (int w = 0; w < WPB; ++w) {
        base[0] += lds.red[0][w];
        base[1] += lds.red[1][w] + lds.red[2][w];
    }
    base[1] = rp.off + base[0] + base[1];
    base[0] += rp.off;
    for (int b = c0; b < c1; b += 64) {
        const int k = b + lane;
        const int n0 = k < c1 ? cnt[k] : 0, n1 = two && k < c1 ? cnt[nc + k] : 0;
        int i0 = n0, i1 = n1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(i0, o, 64), y = __shfl_up(i1, o, 64);
            if (lane >= o) { i0 += x; i1 += y; }
        }
        const int s0 = base[0] + i0 - n0, s1 = base[1] + i1 - n1;
        if (wv == 0 && k < c1) {
            out[k] = s0;
            if (two) out[nc + k] = s1;
        }
        for (int q = wv; q < min(64, c1 - b); q += WPB) {
            const int cell = rp.curve ? a.corder_inv[rp.coff + b + q] : b + q;
            permute_cell<P>(a, rp, lds.wave[wv], s, cell, __builtin_amdgcn_readlane(s0, q),
                            __builtin_amdgcn_readlane(n0, q), __builtin_amdgcn_readlane(s1, q),
                            __builtin_amdgcn_readlane(n1, q));
        }
        base[0] += __builtin_amdgcn_readlane(i0, 63);
        base[1] += __builtin_amdgcn_readlane(i1, 63);
    }
    if (c1 == nc && threadIdx.x == 0) { // the last range knows the sum
        const int end = two ? base[1] : base[0];
        out[two ? 2 * nc : nc] = end;
        if (end - rp.off != rp.n) atomicOr(a.status + s, 4 | 2);
        a.nreb[s] += 1;
    }
    __syncthreads();
}

template <int P, int WAVES>
__global__ void __launch_bounds__(PERM_BLOCK) __attribute__((amdgpu_waves_per_eu(WAVES))) k_permute(const PermArgs a)
{
    __shared__ PermBlockLds lds;
    const int nblk = gridDim.x;
    for_items(a.rlist, [&](int sl) { return perm_units(a.rep[sl], nblk); }, blockIdx.x, nblk,
              [&](int s, int item) {
                  const RepDev rp = a.rep[s];
                  permute_item<P>(a, rp, lds, s, item, nblk);
              });
}

// ------------------------------------------------------------ k_build
// One wave per work item; the waves of a block share nothing.  An item is,
// by the replica's build mode (RepDev::bmode, build_shape() on the host):
//
//   BUILD_CELLS    a share of a cell's members against the members of the 27
//                  surrounding cells: every so many'th 32 of them on the matrix
//                  cores (build_cell_mfma), or as many consecutive ones, one
//                  lane per candidate and a loop over the members
//                  (build_by_candidates), whichever is estimated to be faster
//   BUILD_MEMBERS  64 members of a large replica of few members per cell, one
//                  lane each (build_by_members)
//   BUILD_SINGLE   members of a single-cell replica: two or eight, one lane per
//                  candidate, or 64, one lane each (single_members)
//
// Every form writes the same list: the own cell, then each half-space offset
// o followed by -o (Sec. 4.1), and within a cell the A members before the B
// members, in slot order.  The sorted records of the item's members are
// copied back from scratch, and the old cell starts retired, on the way.
#define BUILD_STRIDE 130  // stride of the members' entries buffered in LDS: members of a wave start in different banks

#define BUILD_BLOCK 256   // threads per block: four waves that share nothing

typedef int v4i_t __attribute__((ext_vector_type(4)));

struct BuildLds { // one per wave
    uint16_t lst[32][BUILD_STRIDE];
    // the chunks of 32 candidates: (slot before the chunk's first in plane 0, the
    // same in plane 1, plane-0 members left, members left and visit << 16)
    union {
        int4 tab[BUILD_SLOTS];
        struct { // more chunks (WIDE): the visits' cells, and of each chunk the visit and the place in its cell
            int4 cell[27];
            uint16_t chunk[BUILD_SLOTS_WIDE];
        } wide;
    };
    template <bool WIDE> __device__ __forceinline__ int4 chunk(int k) const
    {
        if constexpr (!WIDE) return tab[k];
        const int code = wide.chunk[k], c = 32 * (code >> 5);
        const int4 t = wide.cell[code & 31];
        return make_int4(t.x + c, t.y + c, t.z - c, t.w - c);
    }
};

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

// Offset of the v-th visit (v = 0..26) of a member: the own cell, then each
// half-space offset o followed by -o, where the half space is indices 14..26
// of the (dz, dy, dx) enumeration of the 27 offsets (odd v: +o, even v: -o).
__device__ __forceinline__ void visit_offset(int v, int &dx, int &dy, int &dz)
{
    const int q = v > 0 ? 14 + ((v - 1) >> 1) : 13;
    const int sg = (v & 1) ? 1 : -1;
    dz = sg * (q / 9 - 1);
    dy = sg * ((q / 3) % 3 - 1);
    dx = sg * (q % 3 - 1);
}

// A position as the list test reads it: the snapshot (fixed point), or its
// two words (double).
template <int P> struct Snap { uint4 a, b; };
template <int P> __device__ __forceinline__ Snap<P> ld_pos(const BuildArgs &a, int i)
{
    Snap<P> q;
    q.a = a.src_x[i];
    if constexpr (Traits<P>::NS == 2) q.b = a.src_x[(size_t)a.A.P + i];
    else q.b = q.a;
    return q;
}
template <int P> __device__ __forceinline__ int snap_species(const Snap<P> &q)
{
    return Traits<P>::NS == 2 ? (int)(q.b.z >> 31) : (int)(q.a.w >> 31);
}

// Squared list radii of a member against candidates of species A and B, in
// the units of the list test.  (Values are loaded before they are selected:
// a selected address would put the replica record in scratch memory.)
template <int P> struct ListRadii {
    typedef typename std::conditional<Traits<P>::NS == 2, double, float>::type T;
    T a, b;
    __device__ __forceinline__ ListRadii(const BuildArgs &g, const RepDev &rp, int si)
    {
        T r[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (Traits<P>::NS == 2) r[t] = g.pp.rl2d[t];
            else r[t] = rp.rl2s[t];
        }
        a = si ? r[2] : r[0];
        b = si ? r[3] : r[1];
    }
};

// The list test: is candidate q within the list radius of member x?
template <int P>
__device__ __forceinline__ bool in_list(const RepDev &rp, const Snap<P> &x, const ListRadii<P> &rl, const Snap<P> &q)
{
    const bool b = snap_species<P>(q) != 0;
    if constexpr (Traits<P>::NS == 2) {
        double xi, yi, zi, wi, xj, yj, zj, wj;
        u4_to_dbl2(x.a, xi, yi);
        u4_to_dbl2(x.b, zi, wi);
        u4_to_dbl2(q.a, xj, yj);
        u4_to_dbl2(q.b, zj, wj);
        double dx = xi - xj, dy = yi - yj, dz = zi - zj;
        dx -= rp.L * rint(dx * rp.invL);
        dy -= rp.L * rint(dy * rp.invL);
        dz -= rp.L * rint(dz * rp.invL);
        const double r2 = dx * dx + dy * dy + dz * dz;
        return r2 < (b ? rl.b : rl.a);
    } else {
        const float dx = (float)(int)(x.a.x - q.a.x), dy = (float)(int)(x.a.y - q.a.y),
                    dz = (float)(int)(x.a.z - q.a.z);
        const float r2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
        return r2 < (b ? rl.b : rl.a);
    }
}

// Entry k of slot i's list.
__device__ __forceinline__ void put_entry(const KArena &A, int i, int k, int j)
{
    A.nbr_w[4 * list_row_index(i, list_entry_row(k, A.lg), A.cap) + list_entry_col(k, A.lg)] = list_entry(j);
}

// Entries [k0, list end) up to the next multiple of four per lane: a
// particle outside the list radius at this build.  It stays beyond the force
// cutoff until the next build (each particle moves at most skin/2), so the
// force loop needs no per-entry validity test.
__device__ __forceinline__ void pad_list(const KArena &A, int i, int cnt, int k0, int pad)
{
    const int gm = (4 << A.lg) - 1;
    for (int k = max(cnt, k0); k < ((cnt + gm) & ~gm) && k < A.cap; ++k) put_entry(A, i, k, pad < 0 ? i : pad);
}

// A particle to pad the list of slot i with where every other particle of its 27
// cells is in it (a dilute gas, a small cluster): cnt are within its list
// radius, so of any cnt + 1 others one is not.  -1 where the replica has no such
// particle, or the list needs no padding.
template <int P>
__device__ __forceinline__ int far_particle(const BuildArgs &a, const RepDev &rp, int i, int cnt)
{
    if (!(cnt & ((4 << a.A.lg) - 1))) return -1;
    const Snap<P> xi = ld_pos<P>(a, i);
    const ListRadii<P> rl(a, rp, snap_species<P>(xi));
    int j = i + rp.n / 2; // (half the replica's slots away: the first one will do)
    for (int k = min(cnt + 1, rp.n - 1); k > 0; --k, ++j) {
        j -= j >= rp.off + rp.n ? rp.n : 0;
        if (j == i) ++j;
        j -= j >= rp.off + rp.n ? rp.n : 0;
        if (!in_list<P>(rp, xi, rl, ld_pos<P>(a, j))) return j;
    }
    return -1;
}

// List length of slot i, and the status bits of a list that overflowed or
// that needed padding and found none.
__device__ __forceinline__ void finish_list(const BuildArgs &a, int s, int i, int cnt, bool padded)
{
    a.A.nbr_cnt_w[i] = min(cnt, a.A.cap);
    if (cnt > a.A.cap) atomicOr(a.status + s, 1);
    if ((cnt & ((4 << a.A.lg) - 1)) && !padded) atomicOr(a.status + s, 8);
}

template <int P>
__device__ __forceinline__ void copy_back(const BuildArgs &a, int i)
{
    constexpr int NW = Traits<P>::NW, NS = Traits<P>::NS;
    const KArena &A = a.A;
    const size_t P_ = (size_t)A.P;
    if (a.from_scratch) {
#pragma unroll
        for (int w = 0; w < NW; ++w) A.st[w][i] = a.sc_st[w][i];
        A.meta[i] = a.sc_meta[i];
#pragma unroll
        for (int w = 0; w < NS; ++w) {
            uint4 x = a.src_x[w * P_ + i];
            a.snap_cur[w * P_ + i] = x;
            A.xref_w[w * P_ + i] = x;
        }
    }
}

// The members of an item: slots a0 .. a0 + na - 1, then b0 ...
struct Members {
    int a0, na, b0, n;
    __device__ __forceinline__ int slot(int m) const { return m < na ? a0 + m : b0 + (m - na); }
};

// One lane per candidate.  tab holds nr ranges of candidates in canonical
// order: (candidates before the range, first slot in plane 0, first slot in
// plane 1 less the range's plane-0 members, plane-0 members); tot candidates
// in all.  Members [m0, m1) are taken 64 at a time, each chunk of 64
// candidates tested against them in turn; a ballot keeps the order.
template <int P>
__device__ __forceinline__ void build_by_candidates(const BuildArgs &a, const RepDev &rp, int s, const int4 *tab, int nr,
                                                    int tot, const Members &mem, int m0, int m1)
{
    const KArena &A = a.A;
    const int lane = __lane_id();
    for (int g0 = m0; g0 < m1; g0 += 64) {
        const int gn = min(64, m1 - g0);
        const int mine = mem.slot(g0 + min(lane, gn - 1));
        const Snap<P> xm = ld_pos<P>(a, mine);
        int cnt = 0, pad = -1; // of this lane's member
        int r = 0;
        auto slot_at = [&](int b) { // this lane's candidate of chunk b
            const int e = min(b + lane, tot - 1);
            while (r + 1 < nr && tab[r + 1].x <= e) ++r;
            const int4 t = tab[r];
            const int x = e - t.x;
            return (x < t.w ? t.y : t.z) + x;
        };
        for (int b = 0; b < tot; b += 64) {
            const bool valid = b + lane < tot;
            const int j = slot_at(b);
            const Snap<P> q = ld_pos<P>(a, j);
            for (int m = 0; m < gn; ++m) {
                Snap<P> xi;
                xi.a.x = __builtin_amdgcn_readlane(xm.a.x, m);
                xi.a.y = __builtin_amdgcn_readlane(xm.a.y, m);
                xi.a.z = __builtin_amdgcn_readlane(xm.a.z, m);
                xi.a.w = __builtin_amdgcn_readlane(xm.a.w, m);
                if constexpr (Traits<P>::NS == 2) {
                    xi.b.x = __builtin_amdgcn_readlane(xm.b.x, m);
                    xi.b.y = __builtin_amdgcn_readlane(xm.b.y, m);
                    xi.b.z = __builtin_amdgcn_readlane(xm.b.z, m);
                    xi.b.w = __builtin_amdgcn_readlane(xm.b.w, m);
                } else xi.b = xi.a;
                const int i = __builtin_amdgcn_readlane(mine, m);
                const int base = __builtin_amdgcn_readlane(cnt, m);
                const bool other = valid && j != i;
                const bool acc = in_list<P>(rp, xi, ListRadii<P>(a, rp, snap_species<P>(xi)), q) && other;
                const unsigned long long hit = __ballot(acc), miss = __ballot(other && !acc);
                if (acc) {
                    const int k = base + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(hit >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo((unsigned)hit, 0u));
                    if (k < A.cap) put_entry(A, i, k, j);
                }
                const int found = miss ? __shfl(j, __ffsll((long long)miss) - 1, 64) : -1;
                if (lane == m) {
                    cnt += __popcll(hit);
                    pad = pad < 0 ? found : pad;
                }
            }
        }
        if (lane < gn) {
            if (pad < 0) pad = far_particle<P>(a, rp, mine, cnt);
            pad_list(A, mine, cnt, 0, pad);
            finish_list(a, s, mine, cnt, pad >= 0);
        }
    }
}

// One lane per member: each walks the candidates of its own 27 cells.
template <int P>
__device__ __forceinline__ void build_by_members(const BuildArgs &a, const RepDev &rp, int s, int i, bool live)
{
    const KArena &A = a.A;
    const int nd = rp.nd, nc = nd * nd * nd;
    const int *cs = a.cs_new + rp.coff;
    const Snap<P> xi = ld_pos<P>(a, i);
    const ListRadii<P> rl(a, rp, snap_species<P>(xi));
    const int cell = cell_of<P>(rp, xi.a, xi.b);
    int cx = cell % nd, cy = (cell / nd) % nd, cz = cell / (nd * nd);
    if constexpr (P == PREC_FP64) {
        // a member that the sort took for the last cell of an axis and folded to
        // the first's lower face (see dbl_cell_offset1): its cell is the one whose
        // slots hold it
        auto holds = [&](int x, int y, int z) {
            const int k = sort_key(cell_rank(x + nd * (y + nd * z), rp, a.corder), (uint32_t)snap_species<P>(xi) << 31,
                                   rp.planes, nd);
            return i >= cs[k] && i < cs[k + 1];
        };
        if (!holds(cx, cy, cz)) {
            const int lx = cx, ly = cy, lz = cz;
            for (int q = 1; q < 8; ++q) {
                const int x = (q & 1) && lx == 0 ? nd - 1 : lx, y = (q & 2) && ly == 0 ? nd - 1 : ly,
                          z = (q & 4) && lz == 0 ? nd - 1 : lz;
                if (holds(x, y, z)) { cx = x; cy = y; cz = z; break; }
            }
        }
    }
    int cnt = 0, pad = -1;
#pragma unroll 1
    for (int v = 0; v < 27; ++v) {
        int dx, dy, dz;
        visit_offset(v, dx, dy, dz);
        const int rk = offset_rank(cx, cy, cz, dx, dy, dz, rp, a.corder);
        const int gA = cs[rk], nA = cs[rk + 1] - gA;
        const int gB = rp.planes > 1 ? cs[nc + rk] : 0, nB = rp.planes > 1 ? cs[nc + rk + 1] - gB : 0;
        for (int e = 0; e < nA + nB; ++e) {
            const int j = e < nA ? gA + e : gB + (e - nA);
            if (j == i) continue;
            if (in_list<P>(rp, xi, rl, ld_pos<P>(a, j))) {
                if (live && cnt < A.cap) put_entry(A, i, cnt, j);
                ++cnt;
            } else pad = j;
        }
    }
    if (live) {
        if (pad < 0) pad = far_particle<P>(a, rp, i, cnt);
        pad_list(A, i, cnt, 0, pad);
        finish_list(a, s, i, cnt, pad >= 0);
    }
}

// 64 members of a single-cell replica, one lane each, against all of its
// particles, which are the same for all lanes and come by scalar loads (only
// where the sort ran in a launch of its own), a few at a time so that they are
// in flight together.  Slots are taken 32 at a time from a multiple of 32 on,
// so that no load leaves the arena.  A test of 64 members takes 14 instructions,
// against 50 for a member and 64 candidates above, where the ballot and the
// entry's place cost as much as the test; what bounds an item is its chain, 56 us
// at 700 particles (82 with each batch waited for before the next is asked for).
template <int P>
__device__ __forceinline__ void build_single_members(const BuildArgs &a, const RepDev &rp, int s, int m)
{
    constexpr int NS = Traits<P>::NS, U = NS == 2 ? 2 : 8; // (more cost scalar registers: FP64 spilled)
    struct Records { uint4 r[U]; };
    const KArena &A = a.A;
    const int end = rp.off + rp.n, lg = A.lg;
    const bool live = m < rp.n;
    const int i = rp.off + min(m, rp.n - 1);
    const Snap<P> xi = ld_pos<P>(a, i);
    const ListRadii<P> rl(a, rp, snap_species<P>(xi));
    int *list = A.nbr_w + 4 * list_row_index(i, 0, A.cap);
    int cnt = 0, pad = -1;
    auto load = [&](const uint4 *src, int j) { return ld_uniform((const Records *)(src + j), 0); };
    Records na = load(a.src_x, rp.off & ~31), nb = na;
    if constexpr (NS == 2) nb = load(a.src_x + A.P, rp.off & ~31);
    const int last = ((end + 31) & ~31) - U;
#pragma unroll 1
    for (int b = rp.off & ~31; b < end; b += 32) {
        unsigned hit = 0;
#pragma unroll 1
        for (int c = 0; c < 32; c += U) {
            const Records ra = na, rb = nb;
            // (the wait for these, then the next: scalar loads return in any order)
            asm volatile("" ::"s"(ra.r[U - 1].w), "s"(rb.r[U - 1].w));
            __builtin_amdgcn_sched_barrier(0);
            na = load(a.src_x, min(b + c + U, last));
            if constexpr (NS == 2) nb = load(a.src_x + A.P, min(b + c + U, last));
            __builtin_amdgcn_sched_barrier(0);
            unsigned h = 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                h |= in_list<P>(rp, xi, rl, Snap<P>{ra.r[u], NS == 2 ? rb.r[u] : ra.r[u]}) ? 1u << u : 0u;
            hit |= h << c;
        }
        unsigned valid = end - b >= 32 ? ~0u : (1u << (end - b)) - 1u;
        if (b < rp.off) valid &= ~0u << (rp.off - b);
        if ((unsigned)(i - b) < 32u) valid &= ~(1u << (i - b));
        const unsigned miss = valid & ~hit;
        if (miss) pad = b + __ffs(miss) - 1;
        hit = live ? hit & valid : 0u;
        for (; hit; hit &= hit - 1, ++cnt)
            if (cnt < A.cap)
                list[4 * LIST_TILE * list_entry_row(cnt, lg) + list_entry_col(cnt, lg)] = list_entry(b + __ffs(hit) - 1);
    }
    if (live) {
        pad_list(A, i, cnt, 0, pad);
        finish_list(a, s, i, cnt, pad >= 0);
    }
}

// A cell's members against its 27-cell neighbourhood on the matrix cores.
//
// Positions are taken in units of 1/CELL_UNITS of the cell edge from the
// centre of the particle's own cell (cell_units), so a candidate at w in the
// cell at offset o is w + d - u away from a member at u, d = CELL_UNITS o,
// and the list test is
//   T = |w|^2 - 2 w.u + |u|^2 - r_list^2  +  2 w.d + |d|^2 - 2 d.u < 0.
// T is a sum of products of a candidate's and a member's numbers, each split
// into two half-precision words; the products of two low words are left out.
// The first four terms (15 products) are the same for every offset, the last
// three (8 products) the same for every member up to -2 d.u: 32 candidates x
// 32 members are two v_mfma_f32_32x32x16_f16.  Lane 32 h + m gets the 16
// tests of member m and candidates 16 h .. 16 h + 15 (the candidates are
// laid over the rows of the product so that a lane's are consecutive), and
// their acceptance bits are the signs of T, one instruction each.
//
// T is off by at most 3.2e-5 of the squared edge: the products left out, the
// rounding of the low words (w and u are at most half an edge per axis; in FP64
// u is the member's own record, 2^-25 of the edge off, which moves T by 3e-7), low
// words flushed to zero, and 32 roundings of the sum.  Where some |T| is
// below BUILD_EDGE (6.1e-5 of the squared edge, about 3 % of the products),
// that candidate is tested again by the list test itself, so the lists are
// those of the list test, entry for entry.
//
// Two chunks of 32 candidates are taken at a time: the lower half of the
// wave then holds the acceptance bits of the first, the upper half those of
// the second.  The entries go to LDS as 16-bit codes (chunk, candidate), and
// from there to the list as whole rows, coalesced over the members.
//
// What bounds it is VALU issue (about 80 instructions per product of 1024
// tests, 16 of them for the acceptance bits; 10 per entry of the longest of a
// wave's lists; 4,900 per cell of 28 members, against 10,500 with a lane per
// member and 14 per test), and in small systems the chain of one cell's
// products: the visits' constants come from LDS, and the retest follows both
// products of a pair, so that nothing parts the two (through scalar loads and
// two branches a product the 1M rebuild took 555 us, 4,000 particles' 58).
// Before and after, whole rebuild group: 1M mixture in double-single 953 -> 539
// us, 200,000 particles in FP64 556 -> 167 us, an aligned rebuild of 256 small
// replicas 461 -> 354 us.
#define BUILD_EDGE (CELL_UNITS * CELL_UNITS / 16384.0f)

// Per visit, in LDS: 2 d in half precision as the candidate words multiply it
// (x y, z x, y z; for the lower half of the wave, zero for the upper), and -2 d
// and |d|^2.
struct VisitLds {
    uint4 w[2][27];
    float4 d[27];
};
__device__ __forceinline__ void fill_visits(VisitLds &V) // by threads of one block, before a barrier
{
    static_assert(CELL_UNITS == 64.0f, "2 CELL_UNITS in half precision");
    const int v = threadIdx.x;
    if (v >= 27) return;
    int o[3];
    visit_offset(v, o[0], o[1], o[2]);
    unsigned b[3];
    for (int d = 0; d < 3; ++d) b[d] = o[d] == 0 ? 0u : o[d] > 0 ? 0x5800u : 0xD800u; // +-128 = 2 CELL_UNITS
    V.w[0][v] = make_uint4(b[0] | b[1] << 16, b[2] | b[0] << 16, b[1] | b[2] << 16, 0);
    V.w[1][v] = make_uint4(0, 0, 0, 0);
    V.d[v] = make_float4(-2.0f * CELL_UNITS * o[0], -2.0f * CELL_UNITS * o[1], -2.0f * CELL_UNITS * o[2],
                         CELL_UNITS * CELL_UNITS * (o[0] * o[0] + o[1] * o[1] + o[2] * o[2]));
}

template <int P, bool WIDE>
__device__ __forceinline__ void build_cell_mfma(const BuildArgs &a, const RepDev &rp, int s, BuildLds &W,
                                                const VisitLds &V, int ns, const Members &mem, int first, int stride)
{
    const KArena &A = a.A;
    const int lane = __lane_id(), col = lane & 31, h = lane >> 5;
    const int lg = A.lg, lm = (1 << lg) - 1, cap = A.cap;
    // row `col` of the product holds this candidate of the chunk (rows 8 k +
    // 4 h + c of column m end in register 4 k + c of lane 32 h + m)
    const int ci = 16 * ((col >> 2) & 1) + 4 * (col >> 3) + (col & 3);
    // the upper half of the terms: candidate words (high words, 1, 1, B, B, 0)
    const unsigned keep1 = h ? 0x0000FFFFu : ~0u, set1 = h ? 0x3C000000u : 0u;
    const unsigned keep2 = h ? 0u : ~0u, setA = h ? 0x00003C00u : 0u, setB = h ? 0x3C003C00u : 0u;
    const unsigned setB3 = h ? 0x00003C00u : 0u, gkeep = h ? ~0u : 0u;
    auto chunk = [&](int k) { // the same for all lanes
        const int4 t = W.template chunk<WIDE>(k);
        return make_int4(__builtin_amdgcn_readfirstlane(t.x), __builtin_amdgcn_readfirstlane(t.y),
                         __builtin_amdgcn_readfirstlane(t.z), __builtin_amdgcn_readfirstlane(t.w));
    };
    auto load = [&](const int4 &t) {
        const int e = min(ci, (t.w & 0xFFFF) - 1); // past the end: the last one again, masked off below
        const unsigned j = (unsigned)((e < t.z ? t.x : t.y) + e);
        return *(const uint4 *)((const char *)a.cand + (j << 4)); // below 2^28 slots
    };
    for (int g0 = first; g0 < mem.n; g0 += stride) {
        const int m = g0 + col;
        const bool live = m < mem.n;
        const int i = mem.slot(min(m, mem.n - 1));
        const Snap<P> xi = ld_pos<P>(a, i);
        const int si = snap_species<P>(xi);
        const ListRadii<P> rl(a, rp, si);
        float u[3];
        if constexpr (P == PREC_FP64) record_units(a.cand[i], u);
        else cell_units<P>(rp, xi.a, xi.b, u);
        half8 mb; // the members' side of the terms that no offset enters
        {
            const float c0 = rp.rlc[0], c1 = rp.rlc[1], c2 = rp.rlc[2], c3 = rp.rlc[3];
            const float rlA = si ? c2 : c0, rlB = si ? c3 : c1;
            const float c = __builtin_fmaf(u[0], u[0], __builtin_fmaf(u[1], u[1], u[2] * u[2])) - rlA;
            const float px = -2.0f * u[0], py = -2.0f * u[1], pz = -2.0f * u[2], d = rlA - rlB;
            const _Float16 xh = (_Float16)px, yh = (_Float16)py, zh = (_Float16)pz, ch = (_Float16)c, dh = (_Float16)d;
            const _Float16 xl = (_Float16)(px - (float)xh), yl = (_Float16)(py - (float)yh),
                           zl = (_Float16)(pz - (float)zh), cl = (_Float16)(c - (float)ch),
                           dl = (_Float16)(d - (float)dh), one = (_Float16)1.0f, zero = (_Float16)0.0f;
            mb = h ? half8{xl, yl, zl, ch, cl, dh, dl, zero} : half8{xh, yh, zh, xh, yh, zh, one, one};
        }
        // the tests of this lane's 16 candidates of chunk t, whose record of row
        // `col` is rec
        auto product = [&](const int4 &t, const uint4 &rec) {
            const uint4 vw = V.w[h][t.w >> 16];
            const float4 vd = V.d[t.w >> 16];
            const bool isb = ci >= t.z;
            uint4 ra, ob;
            ra.x = rec.x;
            ra.y = (rec.y & keep1) | set1;
            ra.z = (rec.z & keep2) | (isb ? setB : setA);
            ra.w = (rec.w & keep2) | (isb ? setB3 : 0u);
            const float g = __builtin_fmaf(vd.x, u[0], __builtin_fmaf(vd.y, u[1], __builtin_fmaf(vd.z, u[2], vd.w)));
            const _Float16 gh = (_Float16)g;
            const unsigned gw = half2_bits((_Float16)(g - (float)gh), gh);
            ob.x = vw.x;
            ob.y = vw.y | (gw & gkeep & 0xFFFF0000u);
            ob.z = vw.z | (gw & gkeep & 0x0000FFFFu);
            ob.w = 0;
            float16v T;
#pragma unroll
            for (int q = 0; q < 16; ++q) T[q] = 0.0f;
            const half8 ca = __builtin_bit_cast(half8, ra);
            T = __builtin_amdgcn_mfma_f32_32x32x16_f16(ca, __builtin_bit_cast(half8, ob), T, 0, 0, 0);
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(ca, mb, T, 0, 0, 0);
        };
        auto signs = [&](const float16v &T) {
            unsigned hit = 0;
#pragma unroll
            for (int q = 15; q >= 0; --q) hit = __builtin_amdgcn_alignbit(hit, __float_as_uint(T[q]), 31);
            return hit;
        };
        auto nearest = [&](const float16v &T) {
            float near = fminf(fabsf(T[0]), fabsf(T[1]));
#pragma unroll
            for (int q = 2; q < 16; q += 2) near = fminf(fminf(near, fabsf(T[q])), fabsf(T[q + 1]));
            return near;
        };
        // the tests too close to call, by the list test itself
        auto retest = [&](const int4 &t, const float16v &T, unsigned &hit) {
            unsigned again = 0;
#pragma unroll
            for (int q = 0; q < 16; ++q) again |= fabsf(T[q]) < BUILD_EDGE ? 1u << q : 0u;
            for (; again; again &= again - 1) {
                const int b = __ffs(again) - 1, e = min(16 * h + b, (t.w & 0xFFFF) - 1);
                const bool in = in_list<P>(rp, xi, rl, ld_pos<P>(a, (e < t.z ? t.x : t.y) + e));
                hit = (hit & ~(1u << b)) | (in ? 1u << b : 0u);
            }
        };
        int cnt = 0, pad = -1;
        int4 t0 = chunk(0), t1 = chunk(min(1, ns - 1));
        uint4 r0 = load(t0), r1 = load(t1);
#pragma unroll 1
        for (int k = 0; k < ns; k += 2) {
            const int4 c0 = t0, c1 = t1;
            const uint4 q0 = r0, q1 = r1;
            t0 = chunk(min(k + 2, ns - 1));
            t1 = chunk(min(k + 3, ns - 1));
            r0 = load(t0);
            r1 = load(t1);
            const float16v T0 = product(c0, q0), T1 = product(c1, q1);
            unsigned h0 = signs(T0), h1 = signs(T1);
            if (fminf(nearest(T0), nearest(T1)) < BUILD_EDGE) {
                retest(c0, T0, h0);
                retest(c1, T1, h1);
            }
            // this lane's chunk: the first of the two for the lower half
            const auto sw = __builtin_amdgcn_permlane32_swap(h0, h1, false, false);
            unsigned hit = sw[0] | (sw[1] << 16);
            const int left0 = c0.w & 0xFFFF, left1 = k + 1 < ns ? c1.w & 0xFFFF : 0;
            const unsigned v0 = left0 >= 32 ? ~0u : (1u << left0) - 1u, v1 = left1 >= 32 ? ~0u : (1u << left1) - 1u;
            unsigned valid = live ? (h ? v1 : v0) : 0u;
            const int kk = k + h;
            if ((c0.w >> 16) == 0) { // the own cell's chunks come first: not the member itself
                const int self = m - 32 * kk;
                if ((unsigned)self < 32u && (c1.w >> 16 == 0 || h == 0)) valid &= ~(1u << self);
            }
            hit &= valid;
            const unsigned miss = valid & ~hit;
            const int code = kk << 5;
            if (miss) pad = code | (__ffs(miss) - 1);
            const int found = __popc(hit);
            const auto both = __builtin_amdgcn_permlane32_swap(found, found, false, false);
            int at = cnt + (h ? (int)both[0] : 0);
            cnt += (int)both[0] + (int)both[1];
            if (!__any(cnt > BUILD_WIN)) {
                uint16_t *wp = &W.lst[col][at];
                while (hit) {
                    const int b = __ffs(hit) - 1;
                    hit &= hit - 1;
                    *wp++ = (uint16_t)(code | b);
                }
            } else {
                for (; hit; ++at) { // a list beyond the buffer: its tail goes to memory at once
                    const int b = __ffs(hit) - 1;
                    hit &= hit - 1;
                    if (at < BUILD_WIN) W.lst[col][at] = (uint16_t)(code | b);
                    else if (at < cap) put_entry(A, i, at, (h ? (b < c1.z ? c1.x : c1.y) : (b < c0.z ? c0.x : c0.y)) + b);
                }
            }
        }
        // a rejected candidate of either half pads the list
        const auto pads = __builtin_amdgcn_permlane32_swap(pad, pad, false, false);
        pad = (int)pads[0] >= 0 ? (int)pads[0] : (int)pads[1];
        auto slot_of_code = [&](int code) {
            const int4 t = W.template chunk<WIDE>(code >> 5);
            const int e = code & 31;
            return (e < t.z ? t.x : t.y) + e;
        };
        const int used = min(cnt, cap), gm = (4 << lg) - 1;
        const int buffered = min(used, BUILD_WIN), filled = min((used + gm) & ~gm, BUILD_WIN);
        if (h == 0)
            for (int k = buffered; k < filled; ++k) W.lst[col][k] = (uint16_t)max(pad, 0);
        wave_sync();
        if (live) {
            const int rows = filled >> 2;
            v4i_t *dst = (v4i_t *)A.nbr_w + list_row_index(i, 0, cap);
            for (int q = h; q < rows; q += 2) { // the two halves take alternate rows
                const uint16_t *lp = &W.lst[col][((q >> lg) << (lg + 2)) | (q & lm)];
                v4i_t row;
#pragma unroll
                for (int c = 0; c < 4; ++c) row[c] = list_entry(slot_of_code(lp[c << lg]));
                dst[(size_t)q * LIST_TILE] = row;
            }
            if (h == 0) {
                if (used > BUILD_WIN && pad >= 0) pad_list(A, i, used, BUILD_WIN, slot_of_code(pad));
                finish_list(a, s, i, cnt, true);
            }
        }
        wave_sync();
        if (live && pad < 0 && (cnt & gm)) { // (apart from the rest, whose registers are free here)
            const int far = far_particle<P>(a, rp, i, cnt);
            for (int k = used; k < ((cnt + gm) & ~gm) && k < cap; ++k)
                if ((list_entry_row(k, lg) & 1) == h) put_entry(A, i, k, far < 0 ? i : far); // (the half that wrote the row)
            if (far < 0) atomicOr(a.status + s, 8);
        }
    }
}

// The sort lost a particle of slot s: the replica has stopped, and some of its
// scratch records are not its own (frames and thermostat draws pass through
// them), so nothing is copied back and it stays as the step left it.
__device__ __forceinline__ bool sort_lost(const BuildArgs &a, int s) { return (a.status[s] & 4) != 0; }

// Members per item of a single-cell replica while n replicas rebuild.  The fewer,
// the shorter the item's chain and the more work in all: the chain of 64 members
// a wave is 56 us at 700 particles.  Us a forced rebuild of 64 and 256 replicas
// of 700 with 2 members an item 187 and 510, with 8 173 and 436, with 64 174 and
// 320; of 250 82 and 206, 79 and 191, 90 and 162; 16 of 700 99, 106 and 138;
// 1,024 of 700 1,777, 1,508 and 892.
__device__ __forceinline__ int single_members(int n) { return n <= 32 ? 2 : n <= 96 ? 8 : 64; }

// Items of a replica while n replicas rebuild, and its shares per cell.
__device__ __forceinline__ bool few_rebuild(const RepDev &rp, int n) { return n <= rp.bfew_max; }
__device__ __forceinline__ int build_items(const RepDev &rp, int n)
{
    if (rp.bmode == BUILD_SINGLE) return (rp.n + single_members(n) - 1) / single_members(n);
    return few_rebuild(rp, n) ? rp.items3 * rp.bfew : rp.items4;
}

// ONE: in one launch with the sort, one replica.
template <int P, bool WIDE, bool ONE>
__device__ __forceinline__ void build_item(const BuildArgs &a, const RepDev &rp, BuildLds &W, const VisitLds &V, int s,
                                           int item, int rebuilding)
{
    const int lane = __lane_id();
    const int nd = rp.nd, nc = nd * nd * nd, planes = rp.planes;
    const bool few = few_rebuild(rp, rebuilding);
    const int items = build_items(rp, rebuilding);
    const int *cs = a.cs_new + rp.coff;
    if (a.from_scratch) { // retire this item's share of the old cell starts
        const long long all = (long long)planes * nc + 1;
        const int k1 = (int)((item + 1) * all / items);
        for (int k = (int)(item * all / items) + lane; k < k1; k += 64) a.cs[rp.coff + k] = cs[k];
    }
    if (rp.bmode == BUILD_MEMBERS) {
        const int m = item * 64 + lane;
        const int i = rp.off + min(m, rp.n - 1);
        build_by_members<P>(a, rp, s, i, m < rp.n);
        if (m < rp.n) copy_back<P>(a, i);
        return;
    }
    if (rp.bmode == BUILD_SINGLE) { // the replica's slots are one range in canonical order
        const int per = ONE ? 2 : single_members(rebuilding);
        if (!ONE && per == 64) {
            const int m = item * 64 + lane;
            build_single_members<P>(a, rp, s, m);
            if (m < rp.n) copy_back<P>(a, rp.off + m);
            return;
        }
        const Members mem = {rp.off, rp.n, 0, rp.n};
        const int m0 = item * per, m1 = min(m0 + per, rp.n);
        if (lane == 0) W.tab[0] = make_int4(0, rp.off, 0, rp.n);
        wave_sync();
        build_by_candidates<P>(a, rp, s, W.tab, 1, rp.n, mem, m0, m1);
        if (m0 + lane < m1) copy_back<P>(a, rp.off + m0 + lane);
        wave_sync();
        return;
    }
    const int parts = few ? rp.bfew : rp.bparts, cell = parts > 1 ? item / parts : item, part = item - cell * parts;
    // lane v holds the cell of visit v: its starts and members in both planes
    int gA = 0, nA = 0, gB = 0, nB = 0;
    if (lane < 27) {
        int dx, dy, dz;
        visit_offset(lane, dx, dy, dz);
        const int rk = offset_rank(cell % nd, (cell / nd) % nd, cell / (nd * nd), dx, dy, dz, rp, a.corder);
        gA = cs[rk];
        nA = cs[rk + 1] - gA;
        if (planes > 1) {
            gB = cs[nc + rk];
            nB = cs[nc + rk + 1] - gB;
        }
    }
    const int n = nA + nB;
    const Members mem = {__builtin_amdgcn_readlane(gA, 0), __builtin_amdgcn_readlane(nA, 0),
                         __builtin_amdgcn_readlane(gB, 0), __builtin_amdgcn_readlane(n, 0)};
    const int chunks = (n + 31) >> 5;
    int upto = n, chunks_upto = chunks; // inclusive sums over the visits
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const int x = __shfl_up(upto, o, 64), y = __shfl_up(chunks_upto, o, 64);
        if (lane >= o) { upto += x; chunks_upto += y; }
    }
    const int tot = __builtin_amdgcn_readlane(upto, 26), ns = __builtin_amdgcn_readlane(chunks_upto, 26);
    int m0 = 0, m1 = mem.n; // the item's share of the members
    if (parts > 1) {
        const int each = mem.n / parts, more = mem.n - each * parts;
        m0 = part * each + min(part, more);
        m1 = m0 + each + (part < more ? 1 : 0);
    }
    // A product (32 members x 32 candidates) lasts as long as two tests of a member
    // against 64 candidates, or four where the lists outgrow the buffer.  While few
    // replicas rebuild the chip is underfilled and an item's own chain counts, else
    // the sum over the cell's items.
    const int tests = few ? (mem.n + parts - 1) / parts : mem.n, groups = few ? 1 : (mem.n + 31) >> 5;
    if (ns <= (WIDE ? BUILD_SLOTS_WIDE : BUILD_SLOTS) &&
        tests * ((tot + 63) >> 6) > (ns > BUILD_SLOTS ? 4 : 2) * ns * groups) {
        if (mem.n > 32 * part) {
            const int4 t = make_int4(gA, gB - nA, nA, n | (lane << 16));
            for (int c = 0, k = chunks_upto - chunks; c < chunks; ++c, ++k) {
                if constexpr (WIDE) W.wide.chunk[k] = (uint16_t)(lane | c << 5);
                else W.tab[k] = make_int4(t.x + 32 * c, t.y + 32 * c, t.z - 32 * c, t.w - 32 * c);
            }
            if constexpr (WIDE) {
                if (lane < 27) W.wide.cell[lane] = t;
            }
            wave_sync();
            build_cell_mfma<P, WIDE>(a, rp, s, W, V, ns, mem, 32 * part, 32 * parts);
        }
    } else if (m0 < m1) {
        if (lane < 27) W.tab[lane] = make_int4(upto - n, gA, gB - nA, nA);
        wave_sync();
        build_by_candidates<P>(a, rp, s, W.tab, 27, tot, mem, m0, m1);
        wave_sync();
    }
    for (int m = m0 + lane; m < m1; m += 64) copy_back<P>(a, mem.slot(m));
}

// WIDE: for pools that hold a replica of more chunks per neighbourhood than the
// plain table takes (the second level costs the others 3 %).
template <int P, bool WIDE>
__global__ void __launch_bounds__(BUILD_BLOCK, 4) k_build(const BuildArgs a)
{
    __shared__ BuildLds lds[BUILD_BLOCK / 64];
    __shared__ VisitLds visits;
    const int cnt = a.rlist[0];
    if (cnt == 0) return;
    fill_visits(visits);
    __syncthreads();
    const int wpb = BUILD_BLOCK / 64, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for_items(a.rlist, [&](int sl) { return a.from_scratch && sort_lost(a, sl) ? 0 : build_items(a.rep[sl], cnt); },
              remap_block(blockIdx.x, gridDim.x, a.xcd) * wpb + wv, gridDim.x * wpb,
              [&](int s, int item) {
                  const RepDev rp = a.rep[s];
                  build_item<P, WIDE, false>(a, rp, lds[wv], visits, s, item, cnt);
              });
}

// ------------------------------------------------------------ k_rebuild
// The sort and the list build in one launch, for small pools of one slot.
//
// An idle launch costs every step 1.5 us, so a small system pays more for the
// second rebuild kernel than the barrier that replaces it costs the rare step
// that rebuilds: 600 particles 14.3 -> 12.9 us a step, 4,000 in FP64 12.1 ->
// 10.6, 10,000 in FP32 12.6 -> 11.2, 37,000 15.9 -> 15.2 (a rebuild there 77
// -> 95 us).  At 64,000 the two are equal, 21.8 (a rebuild 90 -> 123 us): the
// barrier's cost grows with the sort units, each of which writes its XCD's L2
// back.  (In every thread instead of one wave a block that takes 50 us more.)
//
// The barrier needs no particular number of resident blocks.  Sort units are
// taken from shared counters, by blocks that run, and no block waits while it
// holds one.  A block waits for the units done; when that takes long it takes
// what units are left itself, after which every unit is done or held by a
// block at work on it.  (A count of polls ends the wait all the same, and the
// replica is then halted.)  The counters are split over SYNC_GROUPS cache
// lines: atomics on one address take 15 to 40 ns each.
#define SYNC_POLLS 64     // polls (about 1 us each) before a waiting block helps
#define SYNC_ROUNDS 65536 // rounds of that many polls before it gives up

template <int P>
__global__ void __launch_bounds__(BUILD_BLOCK, 4) k_rebuild(const PermArgs pa, const BuildArgs ba, int *sync)
{
    static_assert(PERM_BLOCK == BUILD_BLOCK, "the sort and the list build share the block");
    constexpr int G = SYNC_GROUPS, WPB = BUILD_BLOCK / 64;
    if (ba.rlist[0] == 0) return;
    __shared__ union {
        PermBlockLds perm;
        BuildLds build[WPB];
    } lds;
    __shared__ VisitLds visits;
    __shared__ int word;
    fill_visits(visits); // (before the loop's barriers)
    const RepDev rp = ld_uniform(ba.rep, 0);
    const int lane = __lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nblk = gridDim.x;
    const int np = perm_units(rp, nblk), nb = build_items(rp, 1); // sort units, list-build items
    const int first = remap_block(blockIdx.x, nblk, ba.xcd) * WPB; // the block's first list-build item
    int g = (int)(blockIdx.x % G), left = (int)blockIdx.x < np ? 1 : 0; // groups to take units from: g and on
    for (int round = 0;;) {
        __syncthreads(); // (word)
        if (left > 0) {
            if (threadIdx.x == 0)
                word = __hip_atomic_fetch_add(sync + g * SYNC_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int unit = g + G * __builtin_amdgcn_readfirstlane(word);
            if (unit < np) {
                permute_item<P>(pa, rp, lds.perm, 0, unit, nblk);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0); // the wave's stores have reached the L2
                __syncthreads();
                if (wv == 0) { // one write-back for the block
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    if (lane == 0)
                        __hip_atomic_fetch_add(sync + (G + g) * SYNC_STRIDE, 1, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                }
                if (np <= nblk && round == 0) left = 0; // the other blocks take one each
            } else {
                --left;
                g = (g + 1) % G;
            }
            continue;
        }
        if (first >= nb) return; // nothing to build
        if (wv == 0) {
            const int want = lane < G ? (np - lane + G - 1) / G : 0; // units of group `lane`
            bool all = false;
            for (int k = 0; k < SYNC_POLLS && !all; ++k) {
                if (k > 0) __builtin_amdgcn_s_sleep(32);
                const int got = lane < G ? __hip_atomic_load(sync + (G + lane) * SYNC_STRIDE, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)
                                         : 0;
                all = __all(got >= want);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (lane == 0)
                word = !all ? 0
                       : __hip_atomic_load(ba.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 4 ? 2 : 1;
        }
        __syncthreads();
        if (word == 2) return; // (see sort_lost)
        if (word) break;
        if (round == 0) left = G;
        if (++round > SYNC_ROUNDS) {
            if (threadIdx.x == 0) atomicOr(ba.status, 4);
            return;
        }
    }
    for (int item = first + wv; item < nb; item += nblk * WPB)
        build_item<P, false, true>(ba, rp, lds.build[wv], visits, 0, item, 1);
}

// Candidate records of a slot's particles (k_permute writes those of a
// rebuild), for the first list of an attached replica.
template <int P>
__global__ void __launch_bounds__(256) k_cand(const BuildArgs a, uint4 *cand, int slot)
{
    const RepDev &rp = a.rep[slot];
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= rp.n) return;
    const Snap<P> q = ld_pos<P>(a, rp.off + k);
    cand[rp.off + k] = cand_record<P>(rp, q.a, q.b);
}
// ------------------------------------------------------------ launchers
hipError_t launch_count(int prec, const CountArgs &a, hipStream_t s)
{
    int grid = (a.P + 255) / 256;
    switch (prec) {
    case PREC_FP64: hipLaunchKernelGGL((k_count<PREC_FP64>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_count<PREC_FP32>), dim3(grid), dim3(256), 0, s, a); break;
    }
    LAUNCH_CHECK();
}

hipError_t launch_enlist(int *rlist, int *sync, const Ctl *ctl, const int *status, int max_slots, int slot,
                         hipStream_t s)
{
    hipLaunchKernelGGL(k_enlist, dim3(1), dim3(64), 0, s, rlist, sync, ctl, status, max_slots, slot);
    LAUNCH_CHECK();
}

static void (*permute_kernel(int prec, bool large))(PermArgs)
{
    switch (prec) {
    case PREC_FP32: return k_permute<PREC_FP32, 4>;
    case PREC_DS: return large ? k_permute<PREC_DS, 6> : k_permute<PREC_DS, 4>;
    case PREC_MIX: return k_permute<PREC_MIX, 4>;
    default: return large ? k_permute<PREC_FP64, 6> : k_permute<PREC_FP64, 4>;
    }
}

hipError_t launch_permute(int prec, bool large, const PermArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(permute_kernel(prec, large), dim3(grid), dim3(PERM_BLOCK), 0, s, a);
    LAUNCH_CHECK();
}

// Resident workgroups per CU of the sort and list-build kernels (their grids
// are sized to one full residency: the kernels walk their work items in a
// grid-stride loop, and a second partial round of workgroups would idle most
// of the chip while it runs).
hipError_t occupancy_permute(int prec, bool large, int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void *)permute_kernel(prec, large), PERM_BLOCK, 0);
}

static void (*build_kernel(int prec, bool wide))(BuildArgs)
{
    switch (prec) {
    case PREC_FP32: return wide ? k_build<PREC_FP32, true> : k_build<PREC_FP32, false>;
    case PREC_DS: return wide ? k_build<PREC_DS, true> : k_build<PREC_DS, false>;
    case PREC_MIX: return wide ? k_build<PREC_MIX, true> : k_build<PREC_MIX, false>;
    default: return wide ? k_build<PREC_FP64, true> : k_build<PREC_FP64, false>;
    }
}

hipError_t occupancy_build(int prec, int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void *)build_kernel(prec, false), BUILD_BLOCK, 0);
}

hipError_t launch_rebuild_one(int prec, const PermArgs &pa, const BuildArgs &ba, int *sync, int grid, hipStream_t s)
{
    const dim3 g(grid), b(BUILD_BLOCK);
    switch (prec) {
    case PREC_FP32: hipLaunchKernelGGL((k_rebuild<PREC_FP32>), g, b, 0, s, pa, ba, sync); break;
    case PREC_DS: hipLaunchKernelGGL((k_rebuild<PREC_DS>), g, b, 0, s, pa, ba, sync); break;
    case PREC_MIX: hipLaunchKernelGGL((k_rebuild<PREC_MIX>), g, b, 0, s, pa, ba, sync); break;
    default: hipLaunchKernelGGL((k_rebuild<PREC_FP64>), g, b, 0, s, pa, ba, sync); break;
    }
    LAUNCH_CHECK();
}

hipError_t launch_build(int prec, bool wide, const BuildArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(build_kernel(prec, wide), dim3(grid), dim3(BUILD_BLOCK), 0, s, a);
    LAUNCH_CHECK();
}

hipError_t launch_cand(int prec, const BuildArgs &a, uint4 *cand, int slot, int n, hipStream_t s)
{
    const int grid = (n + 255) / 256;
    if (prec == PREC_FP64) hipLaunchKernelGGL((k_cand<PREC_FP64>), dim3(grid), dim3(256), 0, s, a, cand, slot);
    else hipLaunchKernelGGL((k_cand<PREC_FP32>), dim3(grid), dim3(256), 0, s, a, cand, slot);
    LAUNCH_CHECK();
}
