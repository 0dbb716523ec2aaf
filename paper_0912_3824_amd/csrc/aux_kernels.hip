// Observables, velocity scaling, the double-single self-test and stream-
// ordered control writes, with their launchers.
#include <mutex>

#include "dev_common.hpp"

// ------------------------------------------------------------ k_obs_reduce
// Deterministic two-pass FP64 sums per slot of e_i, w_i, v^2, v and the list
// lengths: pass 1 reduces fixed chunks of OBS_CHUNK particles, pass 2 adds
// the chunk partials of each slot in chunk order.
#define OBS_CHUNK 4096
#define OBS_Q 7

__device__ __forceinline__ void block_sum7(double acc[OBS_Q], double (*red)[256])
{
    for (int q = 0; q < OBS_Q; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int w = blockDim.x >> 1; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < OBS_Q; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) k_obs_partial(const ObsArgs a)
{
    __shared__ double red[OBS_Q][256];
    const int total = a.chunk_pref[a.max_slots];
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const int s = find_item_slot(a.chunk_pref, a.max_slots, item);
        const RepDev rp = a.rep[s];
        const int k0 = (item - a.chunk_pref[s]) * OBS_CHUNK;
        const int k1 = min(k0 + OBS_CHUNK, rp.n);
        double acc[OBS_Q] = {0, 0, 0, 0, 0, 0, 0};
        for (int k = k0 + threadIdx.x; k < k1; k += blockDim.x) {
            const double *o = a.obs + (size_t)(rp.off + k) * 8;
            acc[0] += o[3];
            acc[1] += o[4];
            acc[2] += o[5] * o[5] + o[6] * o[6] + o[7] * o[7];
            acc[3] += o[5];
            acc[4] += o[6];
            acc[5] += o[7];
            acc[6] += (double)a.nbr_cnt[rp.off + k];
        }
        block_sum7(acc, red);
        if (threadIdx.x < OBS_Q) a.partial[(size_t)item * 8 + threadIdx.x] = red[threadIdx.x][0];
        __syncthreads();
    }
}

__device__ __forceinline__ SlotWords slot_words(const Ctl *ctl, const int *status, const int *nreb, int s)
{
    SlotWords w;
    w.ctl = ctl[s];
    w.status = status[s];
    w.nreb = nreb[s];
    return w;
}

__global__ void __launch_bounds__(256) k_obs_reduce(const ObsArgs a)
{
    const int s = blockIdx.x;
    if (s >= a.max_slots) return;
    if (threadIdx.x == 0) a.words[s] = slot_words(a.ctl, a.status, a.nreb, s);
    if (!a.ctl[s].z) return;
    __shared__ double red[OBS_Q][256];
    double acc[OBS_Q] = {0, 0, 0, 0, 0, 0, 0};
    const int c0 = a.chunk_pref[s], c1 = a.chunk_pref[s + 1];
    // chunk partials of the slot, in chunk order within each thread's stride
    for (int c = c0 + threadIdx.x; c < c1; c += blockDim.x)
        for (int q = 0; q < OBS_Q; ++q) acc[q] += a.partial[(size_t)c * 8 + q];
    block_sum7(acc, red);
    if (threadIdx.x < OBS_Q) a.out[s * 8 + threadIdx.x] = red[threadIdx.x][0];
}

__global__ void __launch_bounds__(256) k_poll(const Ctl *ctl, const int *status, const int *nreb, SlotWords *out,
                                              int max_slots)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < max_slots) out[s] = slot_words(ctl, status, nreb, s);
}

// ------------------------------------------------------------ k_frame
// A replica's state or forces by particle id, in the layout the host gets:
// positions folded into [0, L) in FP64 with the image counters that go with
// them, velocities, forces and energies.  The host used to fetch 64 to 112
// bytes a particle and decode and scatter them itself: at 1M 39 ms a frame,
// now 60 bytes a particle and 5 ms, most of it the copy to pageable memory.
// The scattered stores (24 bytes a particle at an id unrelated to its slot)
// bound the kernel: 90 us at 1M.
template <int P>
__global__ void __launch_bounds__(256) k_frame(const FrameArgs a)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    const int i = a.off + k;
    const int4 m = a.A.meta[i];
    const int id = m.w;
    if (id < 0 || id >= a.n) { // not a particle of this replica
        *a.bad = 1;
        return;
    }
    if (a.force || a.energy) {
        const double *o = a.obs + (size_t)i * 8;
        if (a.force)
#pragma unroll
            for (int d = 0; d < 3; ++d) a.force[3 * (size_t)id + d] = o[d];
        if (a.energy) a.energy[id] = o[3];
        return;
    }
    State<P> st;
    st.load(a.A, i);
    double x[3], v[3];
    if constexpr (P == PREC_DS) {
        x[0] = ds_to_double(st.x); x[1] = ds_to_double(st.y); x[2] = ds_to_double(st.z);
        v[0] = ds_to_double(st.vx); v[1] = ds_to_double(st.vy); v[2] = ds_to_double(st.vz);
    } else {
        x[0] = st.x; x[1] = st.y; x[2] = st.z;
        v[0] = st.vx; v[1] = st.vy; v[2] = st.vz;
    }
    const int img[3] = {m.x, m.y, m.z};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double f = floor(x[d] / a.L);
        double q = x[d] - f * a.L;
        // (a non-finite position counts INT_MIN boxes, as the host's conversion does)
        int im = (int)((unsigned)img[d] + (unsigned)(fabs(f) < 2147483648.0 ? (int)f : (int)0x80000000));
        if (q >= a.L) { q -= a.L; im += 1; }
        if (q < 0) { q += a.L; im -= 1; }
        if (a.pos) a.pos[3 * (size_t)id + d] = q;
        if (a.vel) a.vel[3 * (size_t)id + d] = v[d];
        if (a.image) a.image[3 * (size_t)id + d] = im;
    }
}

// Copy to pinned host memory (16-byte words, coalesced).
__global__ void __launch_bounds__(256) k_words_out(const uint4 *src, uint4 *dst, int n)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = src[k];
}

// ------------------------------------------------------------ k_scale_vel
template <int P>
__global__ void k_scale_vel(const ScaleArgs a)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    const int i = a.off + k;
    State<P> st;
    st.load(a.A, i);
    if constexpr (P == PREC_DS) {
        dsf f = {a.f_hi, a.f_lo};
        st.vx = ds_mul(st.vx, f); st.vy = ds_mul(st.vy, f); st.vz = ds_mul(st.vz, f);
    } else if constexpr (P == PREC_FP32) {
        st.vx *= a.ff; st.vy *= a.ff; st.vz *= a.ff;
    } else {
        st.vx *= a.fd; st.vy *= a.fd; st.vz *= a.fd;
    }
    st.store(a.A, i);
}

// ------------------------------------------------------------ thermostat
// rand48 (Sec. 2.3): x_{k+1} = (a x_k + c) mod 2^48.  Element j from x0 is
// A_j x0 + C_j, the j-fold composition of the affine map; particle id i at
// call k takes elements i + n (4k + r), r = 0..3 (the leap-frog of stride n
// over the particles), so no generator state is stored and the draws do not
// depend on slot order or launch shape.
//
// The host jumps to the elements n (4k + r) (rand48_jump); from there a
// particle is i steps away, one table entry per byte of i, where jumping
// from x0 by repeated squaring took 20 to 40 rounds of four products for
// each of the four elements.
#define TH_LEVELS 4 // ids are below 2^28
struct R48Map { unsigned long long a, c; };
struct R48Table { R48Map m[TH_LEVELS][256]; };
constexpr R48Map r48_then(const R48Map &f, const R48Map &g) // f, then g
{
    return {(g.a * f.a) & R48_M, (g.a * f.c + g.c) & R48_M};
}
constexpr R48Table make_r48_table()
{
    R48Table t{};
    R48Map step{R48_A, R48_C}; // 256^l steps
    for (int l = 0; l < TH_LEVELS; ++l) {
        R48Map m{1, 0};
        for (int k = 0; k < 256; ++k) {
            t.m[l][k] = m;
            m = r48_then(m, step);
        }
        step = m;
    }
    return t;
}
__device__ const R48Table r48_table = make_r48_table();

#define TH_CHUNK 4096

// The Maxwell-Boltzmann velocity of particle id at this call (Box-Muller on
// four leap-frogged rand48 elements); a pure function of (seed, call, id).
__device__ __forceinline__ void thermo_velocity(const ThermoArgs &a, int id, double v[3])
{
    unsigned long long x[4] = {a.x0[0], a.x0[1], a.x0[2], a.x0[3]};
#pragma unroll
    for (int l = 0; l < TH_LEVELS; ++l) {
        if (l >= a.levels) break;
        const R48Map m = r48_table.m[l][(id >> (8 * l)) & 255];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = m.a * x[r] + m.c; // (masked below: only the low 48 bits count)
    }
    double u[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) u[r] = (double)(x[r] & R48_M) * (1.0 / 281474976710656.0);
    const double ra = sqrt(-2.0 * log(1.0 - u[0])), rb = sqrt(-2.0 * log(1.0 - u[2]));
    const double ph = 6.283185307179586 * u[1], ph2 = 6.283185307179586 * u[3];
    v[0] = a.scale * ra * cos(ph);
    v[1] = a.scale * ra * sin(ph);
    v[2] = a.scale * rb * cos(ph2);
}

// Draw Maxwell-Boltzmann velocities into the sort's scratch state words
// (three doubles per slot), one thread a particle; a slot without a particle
// of the replica gets none.
__global__ void __launch_bounds__(256) k_thermo_draw(const ThermoArgs a)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    const int id = a.A.meta[a.off + k].w;
    double v[3] = {0, 0, 0};
    if (id >= 0 && id < a.n) thermo_velocity(a, id, v);
#pragma unroll
    for (int d = 0; d < 3; ++d) a.drawn[3 * (size_t)k + d] = v[d];
}

// sum(v) and sum(v^2) per chunk of TH_CHUNK particles into a.partial[(chunk0 +
// c) * 8 + q]: each thread adds every 256th particle in order, then a tree.
__global__ void __launch_bounds__(256) k_thermo_sum(const ThermoArgs a)
{
    __shared__ double red[4][256];
    const int c = blockIdx.x;
    const int k0 = c * TH_CHUNK, k1 = min(k0 + TH_CHUNK, a.n);
    double acc[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int k = k0 + threadIdx.x; k < k1; k += 256) {
        const int id = a.A.meta[a.off + k].w;
        const double *v = a.drawn + 3 * (size_t)k;
        const double x = v[0], y = v[1], z = v[2];
        if (id < 0 || id >= a.n) continue;
        acc[0] += x; acc[1] += y; acc[2] += z;
        acc[3] += x * x + y * y + z * z;
    }
    for (int q = 0; q < 4; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int w = blockDim.x >> 1; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 4) a.partial[(size_t)(a.chunk0 + c) * 8 + threadIdx.x] = red[threadIdx.x][0];
}

// Subtract the mean (optional), scale to exactly the bath temperature and
// store the velocities in the mode's precision.  Every workgroup adds the
// chunk partials in the same order, so all use the same factor.
template <int P>
__global__ void __launch_bounds__(256) k_thermo_apply(const ThermoArgs a)
{
    __shared__ double rows[256][4];
    double t = 0;
    for (int c0 = 0; c0 < a.nchunk; c0 += 256) {
        const int m = min(256, a.nchunk - c0);
        if ((int)threadIdx.x < m)
#pragma unroll
            for (int q = 0; q < 4; ++q) rows[threadIdx.x][q] = a.partial[(size_t)(a.chunk0 + c0 + threadIdx.x) * 8 + q];
        __syncthreads();
        if (threadIdx.x < 4)
#pragma unroll 8
            for (int c = 0; c < m; ++c) t += rows[c][threadIdx.x];
        __syncthreads();
    }
    if (threadIdx.x < 4) rows[0][threadIdx.x] = t;
    __syncthreads();
    const double *tot = rows[0];
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n) return;
    const double n = (double)a.n;
    double mean[3] = {0, 0, 0};
    if (a.remove_mean)
        for (int d = 0; d < 3; ++d) mean[d] = tot[d] / n;
    const double ss = tot[3] - n * (mean[0] * mean[0] + mean[1] * mean[1] + mean[2] * mean[2]);
    const double f = sqrt(a.temperature / (a.mass * ss / (3.0 * n)));
    const int i = a.off + k;
    const int id = a.A.meta[i].w;
    if (id < 0 || id >= a.n) return;
    const double *w = a.drawn + 3 * (size_t)k;
    const double v[3] = {(w[0] - mean[0]) * f, (w[1] - mean[1]) * f, (w[2] - mean[2]) * f};
    State<P> st;
    st.load(a.A, i);
    if constexpr (P == PREC_FP32) {
        st.vx = (float)v[0]; st.vy = (float)v[1]; st.vz = (float)v[2];
    } else if constexpr (P == PREC_DS) {
        dsf *w[3] = {&st.vx, &st.vy, &st.vz};
        for (int d = 0; d < 3; ++d) {
            w[d]->hi = (float)v[d];
            w[d]->lo = (float)(v[d] - (double)w[d]->hi);
        }
    } else {
        st.vx = v[0]; st.vy = v[1]; st.vz = v[2];
    }
    st.store(a.A, i);
}

hipError_t launch_thermostat(int prec, const ThermoArgs &a, hipStream_t s)
{
    if (a.n <= 0) return hipSuccess;
    const int grid = (a.n + 255) / 256;
    hipLaunchKernelGGL(k_thermo_draw, dim3(grid), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_thermo_sum, dim3(a.nchunk), dim3(256), 0, s, a);
    switch (prec) {
    case PREC_FP32: hipLaunchKernelGGL((k_thermo_apply<PREC_FP32>), dim3(grid), dim3(256), 0, s, a); break;
    case PREC_DS: hipLaunchKernelGGL((k_thermo_apply<PREC_DS>), dim3(grid), dim3(256), 0, s, a); break;
    case PREC_MIX: hipLaunchKernelGGL((k_thermo_apply<PREC_MIX>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_thermo_apply<PREC_FP64>), dim3(grid), dim3(256), 0, s, a); break;
    }
    LAUNCH_CHECK();
}

// ------------------------------------------- allocation-free thermostat
// For callers that cannot allocate device memory (code under graph capture,
// tight serving loops): the chunk partial sums of md_thermostat_noalloc live
// in this file-scope device array instead of the pool's workspace.  Each GPU
// holds its own copy; host code must use the address hipGetSymbolAddress
// returns for the current device, never the array's name.  Every chunk row a call reads was written by the same call, so
// nothing needs clearing; calls that overlap on one GPU race on it.
static __device__ __align__(256) double scratch[THERMO_SCRATCH_CHUNKS * 8];

#define THERMO_MAX_DEVICES 64
static double *scratch_ptr[THERMO_MAX_DEVICES];
static std::mutex scratch_mutex;

hipError_t thermo_scratch_init(int dev)
{
    if (dev < 0 || dev >= THERMO_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (scratch_ptr[dev]) return hipSuccess;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != dev) return hipErrorInvalidDevice; // must be called with that device current
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_ptr[dev] = (double *)p;
    return hipSuccess;
}

double *thermo_scratch(int dev)
{
    if (dev < 0 || dev >= THERMO_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    return scratch_ptr[dev];
}

// ------------------------------------------------------------ k_ds_eval
__global__ void k_ds_eval(int op, long long n, const float *a, const float *b, float *out)
{
    const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (op == 3) { // compensated sum of a[k].hi, single workgroup, fixed order
        if (blockIdx.x != 0 || threadIdx.x != 0) return;
        sum2f s;
        s.init();
        for (long long q = 0; q < n; ++q) s.add(a[2 * q]);
        dsf r = s.result();
        out[0] = r.hi;
        out[1] = r.lo;
        return;
    }
    if (k >= n) return;
    dsf x = {a[2 * k], a[2 * k + 1]}, y = {b[2 * k], b[2 * k + 1]}, r;
    if (op == 0) r = ds_add(x, y);
    else if (op == 1) r = ds_sub(x, y);
    else r = ds_mul(x, y);
    out[2 * k] = r.hi;
    out[2 * k + 1] = r.lo;
}

// ------------------------------------------------------------ k_attach
// A replica from host arrays: fold the positions into the box, convert them
// to the mode's words, sort the particles stably by (species plane, cell
// rank), and set the slot's words.  The conversions are those of
// oracle/upload.py, operation for operation.  The host used to do this in one
// thread: 2.6 ms at 120,000 particles, now 0.2 ms besides the copies.

// One block: the slot's words, and the chunk prefix of the observables'
// reduction (4096 particles per chunk).
__global__ void __launch_bounds__(256) k_attach_words(const AttachArgs a)
{
    __shared__ int wsum[4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (t == 0) {
        a.reps[a.slot] = a.rep;
        a.ctl0[a.slot] = a.ctl1[a.slot] = make_int4(0, 1, 1, 0);
        a.need0[a.slot] = a.need1[a.slot] = a.target[a.slot] = a.status[a.slot] = 0;
        a.nreb[a.slot] = 1;
    }
    __syncthreads();
    int carry = 0;
    if (t == 0) a.chunks[0] = 0;
    for (int base = 0; base < a.max_slots; base += 256) {
        const int s = base + t;
        const bool in = s < a.max_slots && (s == a.slot || a.ctl0[s].z || a.ctl1[s].z);
        int v = in ? ((s == a.slot ? a.n : a.reps[s].n) + OBS_CHUNK - 1) / OBS_CHUNK : 0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(v, o, 64);
            if (lane >= o) v += x;
        }
        if (lane == 63) wsum[wv] = v;
        __syncthreads();
        for (int w = 0; w < wv; ++w) v += wsum[w];
        if (s < a.max_slots) a.chunks[s + 1] = carry + v;
        int all = 0;
        for (int w = 0; w < 4; ++w) all += wsum[w];
        carry += all;
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) k_zero(int *p, int n)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = 0;
}

// Particle `id` folded into the box and converted: state words, snapshot
// words and image counters.
template <int P>
__device__ __forceinline__ void attach_encode(const AttachArgs &a, int id, State<P> &st, uint4 sn[2], int4 &meta, int &species)
{
    double x[3], v[3];
    int img[3];
    const double L = a.rep.L;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double q = a.pos[3 * (size_t)id + d];
        const double f = floor(q / L);
        x[d] = q - f * L;
        img[d] = fabs(f) < 2147483648.0 ? (int)f : (int)0x80000000;
        if (x[d] >= L) { x[d] -= L; img[d] += 1; }
        if (x[d] < 0) { x[d] += L; img[d] -= 1; }
        v[d] = a.vel[3 * (size_t)id + d];
    }
    species = a.species ? a.species[id] & 1 : 0;
    const uint32_t m = ((uint32_t)species << 31) | ((uint32_t)a.slot << SLOT_SHIFT);
    if constexpr (P == PREC_FP32) {
        float f[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            // x is in [0, L); its float may round up to L or past it, which
            // is folded by the exact edge (the box need not be a float)
            f[d] = (float)x[d];
            if ((double)f[d] >= L) { f[d] = (float)((double)f[d] - L); img[d] += 1; }
            x[d] = (double)f[d];
        }
        st.x = f[0]; st.y = f[1]; st.z = f[2];
        st.vx = (float)v[0]; st.vy = (float)v[1]; st.vz = (float)v[2];
    } else if constexpr (P == PREC_DS) {
        st.x = ds_from_double(x[0]); st.y = ds_from_double(x[1]); st.z = ds_from_double(x[2]);
        st.vx = ds_from_double(v[0]); st.vy = ds_from_double(v[1]); st.vz = ds_from_double(v[2]);
        x[0] = ds_to_double(st.x); x[1] = ds_to_double(st.y); x[2] = ds_to_double(st.z);
    } else {
        st.x = x[0]; st.y = x[1]; st.z = x[2];
        st.vx = v[0]; st.vy = v[1]; st.vz = v[2];
    }
    if constexpr (Traits<P>::NS == 2) {
        sn[0] = dbl2_to_u4(x[0], x[1]);
        sn[1] = dbl2_to_u4(x[2], bits_of_meta(m));
    } else {
        sn[0] = make_uint4(to_fixed(x[0], a.rep.fxs), to_fixed(x[1], a.rep.fxs), to_fixed(x[2], a.rep.fxs), m);
        sn[1] = sn[0];
    }
    meta = make_int4(img[0], img[1], img[2], id);
}

// The input of a slot being attached was found wrong (k_attach_count): the
// kernels that follow write nothing.
__device__ __forceinline__ bool attach_refused(const AttachArgs &a)
{
    return (a.status[a.slot] & (ST_BAD_INPUT | ST_BAD_SPECIES)) != 0;
}

// Check of the input, and of each particle its sort key and its place among
// the cell's arrivals.  Nothing of the replica is written before every particle
// has passed: non-finite positions all convert to one cell, and the passes
// over a cell's members take the square of their number.
template <int P>
__global__ void __launch_bounds__(256) k_attach_count(const AttachArgs a)
{
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= a.n) return;
    bool fine = true;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        fine = fine && isfinite(a.pos[3 * (size_t)id + d]) && isfinite(a.vel[3 * (size_t)id + d]);
    if (!fine) atomicOr(a.status + a.slot, ST_BAD_INPUT);
    if (a.species && (a.species[id] < 0 || a.species[id] >= a.n_species)) atomicOr(a.status + a.slot, ST_BAD_SPECIES);
    if (!fine) return;
    State<P> st;
    uint4 sn[2];
    int4 meta;
    int species;
    attach_encode<P>(a, id, st, sn, meta, species);
    const int nd = a.rep.nd;
    int cell = 0;
    if (nd > 1) cell = cell_of<P>(a.rep, sn[0], sn[1]);
    const int key = sort_key(cell_rank(cell, a.rep, a.corder), (uint32_t)species << 31, a.rep.planes, nd);
    a.key[id] = key;
    a.arrival[id] = atomicAdd(a.cs_new + a.rep.coff + key, 1);
}

// One block: cell starts (absolute slots) from the counts in cs_new.
__global__ void __launch_bounds__(1024) k_attach_scan(const AttachArgs a)
{
    __shared__ int wsum[16];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int *cn = a.cs_new + a.rep.coff, *cs = a.cs + a.rep.coff;
    int carry = a.off;
    for (int base = 0; base < a.ncell; base += 8 * 1024) {
        // thread t takes cells base + 1024 u + t (coalesced); rows in turn
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = base + 1024 * u + t < a.ncell ? cn[base + 1024 * u + t] : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            int incl = v[u];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int x = __shfl_up(incl, o, 64);
                if (lane >= o) incl += x;
            }
            if (lane == 63) wsum[wv] = incl;
            __syncthreads();
            int before = 0, all = 0;
            for (int w = 0; w < 16; ++w) {
                before += w < wv ? wsum[w] : 0;
                all += wsum[w];
            }
            const int k = base + 1024 * u + t;
            if (k < a.ncell) cs[k] = cn[k] = carry + before + incl - v[u];
            carry += all;
            __syncthreads();
        }
    }
    if (t == 0) cs[a.ncell] = cn[a.ncell] = carry;
}

__global__ void __launch_bounds__(256) k_attach_scatter(const AttachArgs a)
{
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id < a.n && !attach_refused(a)) a.ids[a.cs[a.rep.coff + a.key[id]] - a.off + a.arrival[id]] = id;
}

// Each particle to its slot: a cell's members in the order of their ids.
template <int P>
__global__ void __launch_bounds__(256) k_attach_place(const AttachArgs a)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.n || attach_refused(a)) return;
    const int id = a.ids[k], key = a.key[id];
    const int q0 = a.cs[a.rep.coff + key] - a.off, q1 = a.cs[a.rep.coff + key + 1] - a.off;
    int rank = 0;
    for (int q = q0; q < q1; ++q) rank += a.ids[q] < id;
    const int i = a.off + q0 + rank;
    State<P> st;
    uint4 sn[2];
    int4 meta;
    int species;
    attach_encode<P>(a, id, st, sn, meta, species);
    st.store(a.A, i);
    a.A.meta[i] = meta;
#pragma unroll
    for (int w = 0; w < Traits<P>::NS; ++w) {
        const size_t j = (size_t)w * a.A.P + i;
        a.snap0[j] = a.snap1[j] = a.A.xref_w[j] = sn[w];
    }
    if (a.rep.bmode == BUILD_CELLS) a.cand[i] = cand_record<P>(a.rep, sn[0], sn[1]);
}

template <int P> static void launch_attach_t(const AttachArgs &a, hipStream_t s)
{
    const int grid = (a.n + 255) / 256;
    hipLaunchKernelGGL((k_attach_count<P>), dim3(grid), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_attach_scan, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_attach_scatter, dim3(grid), dim3(256), 0, s, a);
    hipLaunchKernelGGL((k_attach_place<P>), dim3(grid), dim3(256), 0, s, a);
}

hipError_t launch_attach(int prec, const AttachArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_attach_words, dim3(1), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_zero, dim3((a.ncell + 255) / 256), dim3(256), 0, s, a.cs_new + a.rep.coff, a.ncell);
    switch (prec) {
    case PREC_FP32: launch_attach_t<PREC_FP32>(a, s); break;
    case PREC_DS: launch_attach_t<PREC_DS>(a, s); break;
    case PREC_MIX: launch_attach_t<PREC_MIX>(a, s); break;
    default: launch_attach_t<PREC_FP64>(a, s); break;
    }
    LAUNCH_CHECK();
}

// ------------------------------------------------------------ launchers
hipError_t launch_frame(int prec, const FrameArgs &a, hipStream_t s)
{
    const int grid = (a.n + 255) / 256;
    if (grid == 0) return hipSuccess;
    switch (prec) {
    case PREC_FP32: hipLaunchKernelGGL((k_frame<PREC_FP32>), dim3(grid), dim3(256), 0, s, a); break;
    case PREC_DS: hipLaunchKernelGGL((k_frame<PREC_DS>), dim3(grid), dim3(256), 0, s, a); break;
    case PREC_MIX: hipLaunchKernelGGL((k_frame<PREC_MIX>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_frame<PREC_FP64>), dim3(grid), dim3(256), 0, s, a); break;
    }
    LAUNCH_CHECK();
}

hipError_t launch_words_out(const uint4 *src, uint4 *dst, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_words_out, dim3((n + 255) / 256), dim3(256), 0, s, src, dst, n);
    LAUNCH_CHECK();
}

hipError_t launch_poll(const Ctl *ctl, const int *status, const int *nreb, SlotWords *out, int max_slots, hipStream_t s)
{
    hipLaunchKernelGGL(k_poll, dim3((max_slots + 255) / 256), dim3(256), 0, s, ctl, status, nreb, out, max_slots);
    LAUNCH_CHECK();
}

hipError_t launch_obs_reduce(const ObsArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_obs_partial, dim3(1024), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_obs_reduce, dim3(a.max_slots), dim3(256), 0, s, a);
    LAUNCH_CHECK();
}

hipError_t launch_scale_vel(int prec, const ScaleArgs &a, hipStream_t s)
{
    int grid = (a.n + 255) / 256;
    if (grid == 0) return hipSuccess;
    switch (prec) {
    case PREC_FP32: hipLaunchKernelGGL((k_scale_vel<PREC_FP32>), dim3(grid), dim3(256), 0, s, a); break;
    case PREC_DS: hipLaunchKernelGGL((k_scale_vel<PREC_DS>), dim3(grid), dim3(256), 0, s, a); break;
    case PREC_MIX: hipLaunchKernelGGL((k_scale_vel<PREC_MIX>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_scale_vel<PREC_FP64>), dim3(grid), dim3(256), 0, s, a); break;
    }
    LAUNCH_CHECK();
}

hipError_t launch_ds_eval(int op, long long n, const float *a, const float *b, float *out, hipStream_t s)
{
    long long grid = op == 3 ? 1 : (n + 255) / 256;
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ds_eval, dim3((unsigned)grid), dim3(256), 0, s, op, n, a, b, out);
    LAUNCH_CHECK();
}

// ------------------------------------------------------------ control pokes
// Stream-ordered writes of control words (graph- and capture-safe; no host
// buffers whose lifetime would have to outlast an asynchronous copy).
__global__ void k_add_targets(int *target, const Ctl *ctl, int max_slots, int delta)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < max_slots && ctl[s].z) target[s] += delta;
}

__global__ void k_poke(int *p, int v) { *p = v; }

// Forget the forces a finalising launch stored (control word w) for every slot.
__global__ void k_void_stored(Ctl *ctl, int max_slots)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < max_slots) ctl[s].w = 0;
}

hipError_t launch_add_targets(int *target, const Ctl *ctl, int max_slots, int delta, hipStream_t s)
{
    hipLaunchKernelGGL(k_add_targets, dim3((max_slots + 255) / 256), dim3(256), 0, s, target, ctl, max_slots, delta);
    LAUNCH_CHECK();
}

hipError_t launch_void_stored(Ctl *ctl, int max_slots, hipStream_t s)
{
    hipLaunchKernelGGL(k_void_stored, dim3((max_slots + 255) / 256), dim3(256), 0, s, ctl, max_slots);
    LAUNCH_CHECK();
}

hipError_t launch_poke(int *p, int v, hipStream_t s)
{
    hipLaunchKernelGGL(k_poke, dim3(1), dim3(1), 0, s, p, v);
    LAUNCH_CHECK();
}
