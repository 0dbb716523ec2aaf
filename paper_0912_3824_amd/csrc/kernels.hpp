// Kernel argument blocks and launchers of libmdx (shared by the .hip kernel
// sources and abi.cpp).  Plain structs passed by value as kernel arguments.
#pragma once
#include <hip/hip_runtime.h>
#include "md_dev.hpp"

struct KArena {
    int P;            // arena stride (particle slots)
    int cap;          // neighbour-list capacity per particle (a multiple of 16)
    int lg;           // log2 of the lanes per particle that read a list (entry layout)
    uint4 *st[3];     // state words
    const uint4 *xref;
    uint4 *xref_w;    // same memory as xref
    int4 *meta;
    const int *nbr;
    int *nbr_w;       // same memory as nbr
    const int *nbr_cnt;
    int *nbr_cnt_w;   // same memory as nbr_cnt
};

struct StepArgs {
    KArena A;
    int cell_cap, max_slots, xcd, lpp; // lpp: lanes per particle (1, 2, 4)
    const uint4 *snap_cur;
    uint4 *snap_next;
    const RepDev *rep;
    const Ctl *ctl_cur;
    Ctl *ctl_next;
    const int *target;
    int *need_cur, *need_other;
    int *rlist_cur, *rlist_other; // [0] = count, [1..] = slots that must rebuild
    int *sync_other; // counters of the one-launch rebuild, cleared with rlist_other
    int *count_cur, *count_other;
    const int *corder; // per-replica cell rank tables (cell arena offsets)
    int *status;
    double *obs;
    PairDev pp;
    IntegDev ig;
};

// Counters of the one-launch rebuild (k_rebuild): a cache line each, SYNC_GROUPS
// of sort units taken, then SYNC_GROUPS of sort units done.
#define SYNC_GROUPS 8
#define SYNC_STRIDE 32
#define SYNC_WORDS (2 * SYNC_GROUPS * SYNC_STRIDE)

struct CountArgs {
    int P, max_slots;
    const uint4 *snap;
    const RepDev *rep;
    const Ctl *ctl;
    int *count;
    const int *corder;
};

struct PermArgs {
    KArena A;
    const RepDev *rep;
    const int *rlist;
    const int *count;  // members of each new cell
    const int *cs;     // old cell starts
    int *cs_new;
    const int *corder, *corder_inv;
    const uint4 *snap;
    uint4 *sc_st[3];
    uint4 *sc_snap;
    int4 *sc_meta;
    uint4 *cand; // candidate records of the list build
    int *status, *nreb;
};

struct BuildArgs {
    KArena A;
    int from_scratch, xcd;
    const RepDev *rep;
    const int *rlist;
    int *cs;
    const int *cs_new;
    const int *corder;
    const uint4 *src_x;
    const uint4 *cand; // candidate records (cand_record)
    uint4 *snap_cur;
    const uint4 *sc_st[3];
    const int4 *sc_meta;
    int *status;
    PairDev pp;
};

struct SlotWords;

struct ObsArgs {
    int max_slots, pad0;
    const RepDev *rep;
    const Ctl *ctl;
    const double *obs;
    const int *nbr_cnt;
    const int *chunk_pref; // per slot prefix of ceil(n / 4096) chunks
    double *partial;       // [chunks][8]
    double *out;           // [max_slots][8]
    const int *status, *nreb;
    SlotWords *words;      // [max_slots] (device or pinned host memory)
};

// What a synchronising call reads of a slot besides its sums.
struct SlotWords {
    Ctl ctl;
    int status, nreb;
};

// A replica's state or forces in particle-id order (any output may be null).
struct FrameArgs {
    KArena A;
    int off, n;
    double L;
    const double *obs;
    double *pos, *vel, *force, *energy; // [n][3], [n][3], [n][3], [n]
    int *image;                         // [n][3]
    int *bad;                           // set where a particle id is out of range
};

struct ScaleArgs {
    KArena A;
    int off, n;
    float f_hi, f_lo, ff, pad0;
    double fd;
};

// Modified Andersen thermostat (Sec. 2.3): rand48 draws, leap-frogged with
// stride n over the replica's particles.
struct ThermoArgs {
    KArena A;
    double *drawn;    // [n][3] drawn velocities, by slot (the sort's scratch state words)
    double *partial;  // chunk partial sums (8 doubles per chunk)
    int off, n, chunk0, nchunk, remove_mean;
    int levels;       // bytes of the largest particle id
    unsigned long long x0[4]; // rand48 elements n (4 call + r), r = 0..3, from the seed's
    double scale;             // sqrt(T / m)
    double temperature, mass;
};

// rand48's affine map and the element j steps from x0 (A_j x0 + C_j by
// repeated squaring).
#define R48_A 0x5DEECE66DULL
#define R48_C 0xBULL
#define R48_M ((1ULL << 48) - 1ULL)
inline unsigned long long rand48_jump(unsigned long long x0, unsigned long long j)
{
    unsigned long long A = 1, C = 0, a = R48_A, c = R48_C;
    for (; j; j >>= 1) {
        if (j & 1) { A = (a * A) & R48_M; C = (a * C + c) & R48_M; }
        c = (a * c + c) & R48_M;
        a = (a * a) & R48_M;
    }
    return (A * x0 + C) & R48_M;
}

hipError_t launch_thermostat(int prec, const ThermoArgs &a, hipStream_t s);
// Chunk rows of the allocation-free thermostat's scratch array (aux_kernels.hip):
// at most THERMO_SCRATCH_CHUNKS chunks of 4096 particles per call.
#define THERMO_SCRATCH_CHUNKS 16384
hipError_t thermo_scratch_init(int dev); // once per device, with that device current
double *thermo_scratch(int dev);         // its device address (nullptr before init)
hipError_t launch_step(int prec, const StepArgs &a, int block, int n_cu, bool obs, hipStream_t s);
hipError_t launch_count(int prec, const CountArgs &a, hipStream_t s);
hipError_t launch_enlist(int *rlist, int *sync, const Ctl *ctl, const int *status, int max_slots, int slot,
                         hipStream_t s);
hipError_t launch_permute(int prec, bool large, const PermArgs &a, int grid, hipStream_t s);
hipError_t launch_rebuild_one(int prec, const PermArgs &pa, const BuildArgs &ba, int *sync, int grid, hipStream_t s);
hipError_t launch_build(int prec, bool wide, const BuildArgs &a, int grid, hipStream_t s);
hipError_t launch_cand(int prec, const BuildArgs &a, uint4 *cand, int slot, int n, hipStream_t s);
hipError_t occupancy_permute(int prec, bool large, int *per_cu);
hipError_t occupancy_build(int prec, int *per_cu);
// A replica handed in as host arrays: by-id input rows on the device, the cell
// tables and the arrays of the slot it becomes.
struct AttachArgs {
    KArena A;
    int slot, off, n, ncell; // ncell: cells of every plane
    RepDev rep;
    const double *pos, *vel; // [n][3]
    const int *species;      // [n], or null
    int *key, *arrival;      // [n]: cell (sort key) of each particle, its place among the cell's arrivals
    int *ids;                // [n]: particle ids by slot, unordered within a cell
    const int *corder;
    int *cs, *cs_new;
    uint4 *snap0, *snap1, *cand;
    // words of the slot
    RepDev *reps;
    Ctl *ctl0, *ctl1;
    int *need0, *need1, *target, *status, *nreb, *chunks;
    int max_slots, n_species;
};
hipError_t launch_attach(int prec, const AttachArgs &a, hipStream_t s);
hipError_t launch_frame(int prec, const FrameArgs &a, hipStream_t s);
hipError_t launch_words_out(const uint4 *src, uint4 *dst, int n, hipStream_t s);
hipError_t launch_poll(const Ctl *ctl, const int *status, const int *nreb, SlotWords *out, int max_slots, hipStream_t s);
hipError_t launch_obs_reduce(const ObsArgs &a, hipStream_t s);
hipError_t launch_scale_vel(int prec, const ScaleArgs &a, hipStream_t s);
hipError_t launch_ds_eval(int op, long long n, const float *a, const float *b, float *out, hipStream_t s);
