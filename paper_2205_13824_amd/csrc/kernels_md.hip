// Particle bookkeeping kernels of librbsog for gfx950: the velocity-Verlet
// kick/drift, wrap and quantise with the displacement check of the Verlet
// list, the cell list of a list build (histogram, exclusive scan, scatter,
// per-cell id sort and gather of the state into cell order), the kinetic
// energy sum and the mean-square displacement.
//
// Arrays are structure-of-arrays over all systems of the batch: component d
// of slot t is at [d*N + t].  The state is in the cell order of the latest
// list build, so these passes stream it coalesced and a re-sort moves
// particles only as far as they drifted.  The list-build kernels read the
// rebuild flag first and return at once when it is clear.
#include <type_traits>

#include "rbsog_internal.h"
#include "rbsog_math.h"
#include "rho_block.h"

namespace rbsog {

namespace {

constexpr int kBlock = 256;
inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// The cell scan works on tiles of kScanTile cells.
constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Lanes holding the same cell in a run of consecutive lanes (the state is in
// cell order, so runs are the rule) share one atomic: the run's first lane
// adds the run length and the others take their offset in the run.  Returns
// the old counter value plus the lane's offset (all lanes must be active).
__device__ __forceinline__ int32_t run_atomic_add(int32_t *ctr, int64_t cell, bool valid) {
    const int lane = threadIdx.x & 63;
    const int64_t key = valid ? cell : -1;
    const int64_t prev = __shfl_up(key, 1, 64);
    const bool head = lane == 0 || key != prev;
    const uint64_t H = __ballot(head);
    const uint64_t after = lane == 63 ? 0ull : (H >> (lane + 1)) << (lane + 1);
    const int nxt = after ? __builtin_ctzll(after) : 64;
    const int first = 63 - __clzll((long long)(H & ((2ull << lane) - 1ull)));
    int32_t base = 0;
    if (head && valid) base = atomicAdd(&ctr[cell], nxt - lane);
    base = __shfl(base, first, 64);
    return base + (lane - first);
}

// Optional kick dt/2 and drift (velocity Verlet), then wrap x into [0, L)
// (x_w = frac(x/L) L) and fixed-point coordinate u = min(2^32-1,
// floor(frac(x/L) 2^32)).  A particle farther than skin r_c / 2 from its
// position at the latest list build sets the rebuild flag: the list holds
// every pair within r_c (1 + skin) at the build, so it holds every pair
// within r_c while no particle has moved farther.
__global__ __launch_bounds__(kBlock) void k_kdq(EvalArgs a) {
    const int64_t t0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool valid = t0 < a.N;
    const int64_t t = valid ? t0 : a.N - 1;
    const int64_t N = a.N;
    double *__restrict__ x = a.cur.x;
    double *__restrict__ v = a.cur.v;
    // every load first: the system's constants and the particle's state
    const SysDev &sd = a.sys[a.sys_of[t]];
    double L[3], xs[3];
    float hf[3];
    uint32_t uref[3];
    for (int d = 0; d < 3; ++d) {
        L[d] = sd.g.L[d];
        hf[d] = sd.g.hf[d];
        xs[d] = x[d * N + t];
        uref[d] = a.u[d * N + t];
    }
    const float dthr2 = sd.g.dthr2_f;
    const double xs0[3] = {xs[0], xs[1], xs[2]};
    if (a.kick) {
        double f[3], vs[3];
        for (int d = 0; d < 3; ++d) {
            f[d] = a.Fn[d * N + t] + a.Ff[d * N + t];
            vs[d] = v[d * N + t];
        }
        if (a.nh) {
            // Nose-Hoover: xi's first half step with the kinetic energy of the
            // step's start, then v scaled by exp(-xi dt/2) (the far kernel
            // scales again after the closing kick and moves xi on)
            const int32_t s = a.sys_of[t];
            const double xh = a.nh_xi[s] + 0.5 * a.dt * (2.0 * a.kin[s] - sd.nh_nf * a.nh_T) / sd.nh_Q;
            const double sc = exp(-0.5 * a.dt * xh);
            for (int d = 0; d < 3; ++d) vs[d] *= sc;
        }
        bool bad = false;
        if (a.thermo) {
            // BAOAB: half kick, half drift, Ornstein-Uhlenbeck, half drift
            double xi[3];
            rmath::thermo_normals(a.tseed, *a.tstep, a.cur.id[t], xi);
            for (int d = 0; d < 3; ++d) {
                bad |= !isfinite(f[d]);
                vs[d] += a.hdm * f[d];
                xs[d] += 0.5 * a.dt * vs[d];
                vs[d] = fma(a.c1, vs[d], a.c2 * xi[d]);  // (rounded as where the far kernel opens the step)
                xs[d] += 0.5 * a.dt * vs[d];
                if (valid) v[d * N + t] = vs[d];
            }
        } else {
            for (int d = 0; d < 3; ++d) {
                bad |= !isfinite(f[d]);
                vs[d] += a.hdm * f[d];
                xs[d] += a.dt * vs[d];
                if (valid) v[d * N + t] = vs[d];
            }
        }
        if (bad && valid) atomicOr(a.flag, 1);
        // the step's drift, unwrapped, for the mean-square displacement
        if (valid && a.cur.dsp)
            for (int d = 0; d < 3; ++d) a.cur.dsp[d * N + t] += xs[d] - xs0[d];
    }
    uint32_t uq[3];
    const float d2 = wrap_store(a, t, valid, xs, L, hf, uref, uq);
    if (a.always_build) {
        // every evaluation builds: the cell and the histogram here (no bin pass)
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.rebuild = 1;
        int64_t c[3];
        for (int d = 0; d < 3; ++d) c[d] = (int64_t)(((uint64_t)uq[d] * (uint64_t)sd.g.nc[d]) >> 32);
        const int64_t cell = sd.c0 + c[0] + (int64_t)sd.g.nc[0] * (c[1] + (int64_t)sd.g.nc[1] * c[2]);
        if (valid) a.cell_of[t] = (int32_t)cell;
        run_atomic_add(a.cell_count, cell, valid);
    } else {
        // one atomic per wave that found a particle past the threshold
        const bool far_ = valid && !(d2 <= dthr2);
        if (__ballot(far_) != 0ull && (threadIdx.x & 63) == 0) atomicOr(a.rebuild, 1);
    }
}

// ---- exclusive scan of int32 counts: 1024 elements per block --------------

template <int BLOCK = kBlock>
__device__ int32_t block_exclusive_scan(int32_t v, int32_t *total) {
    __shared__ int32_t wsum[BLOCK / 64];
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        int32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int32_t base = 0, tot = 0;
    for (int w = 0; w < BLOCK / 64; ++w) {
        if (w < wid) base += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return base + incl - v;
}

// The kernels of a list build run at every evaluation with a kept list and
// return at once unless a build is due.  Beside the structure factor (EvalArgs::wide
// 0) their blocks are large and few: kBuildThreads threads, at most kBuildGrid
// blocks that stride, so that they pass the few wave slots that it leaves free (512
// blocks: 300,000 ions 84.8 us a step against 83.7; 64: 84.0).  A build itself takes
// longer in them, so that evaluations which build for certain, and those with
// nothing beside the build, take blocks of kWideThreads, at most kWideGrid.
constexpr int kBuildThreads = 1024;
constexpr int64_t kBuildGrid = 128;
constexpr int kWideThreads = 256;
constexpr int64_t kWideGrid = 2048;

// Exclusive scan of the counts of n cells by one block, tile after tile of four
// counts per thread: the cells' starts, the scatter's fill counters, and
// out[n] = the total.  (The last block of the bin pass did this before, after a
// device-scope fence in every block; each fence writes back its XCD's L2:
// 77,781 ions 55 us, 331,776 sites 350 us a build.)
__global__ __launch_bounds__(kBuildThreads) void k_scan_one(const int32_t *__restrict__ in, int64_t n,
                                                            int32_t *__restrict__ out, int32_t *__restrict__ fill,
                                                            const int32_t *__restrict__ cond) {
    __builtin_amdgcn_s_setprio(2);
    if (!*cond) return;
    int32_t before = 0;
    for (int64_t c0 = 0; c0 < n; c0 += 4 * kBuildThreads) {
        const int64_t c = c0 + 4 * (int64_t)threadIdx.x;
        int32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = c + k < n ? in[c + k] : 0;
            sum += v[k];
        }
        int32_t tot;
        int32_t off = before + block_exclusive_scan<kBuildThreads>(sum, &tot);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + k < n) {
                out[c + k] = off;
                fill[c + k] = off;
                off += v[k];
            }
        before += tot;
    }
    if (threadIdx.x == 0) out[n] = before;
}

// Cell c_d = (u n_d) >> 32 of slot t.
__device__ __forceinline__ int64_t cell_at(const EvalArgs &a, int64_t t) {
    const SysDev &sd = a.sys[a.sys_of[t]];
    int64_t c[3];
    int32_t nc[3];
    for (int d = 0; d < 3; ++d) {
        nc[d] = sd.g.nc[d];
        c[d] = (int64_t)(((uint64_t)a.u_tmp[d * a.N + t] * (uint64_t)nc[d]) >> 32);
    }
    return sd.c0 + c[0] + (int64_t)nc[0] * (c[1] + (int64_t)nc[1] * c[2]);
}

// Cell of each particle and the cell histogram, by block `block` of `blocks`.
__device__ __forceinline__ void bin_particles(const EvalArgs &a, int64_t block, int64_t blocks) {
    // the critical path's waves ahead of the structure factor's beside them
    __builtin_amdgcn_s_setprio(2);
    if (!*a.rebuild) return;
    const int64_t N = a.N;
    for (int64_t base = block * blockDim.x; base < N; base += blocks * blockDim.x) {
        const int64_t t0 = base + threadIdx.x;
        const bool valid = t0 < N;
        const int64_t t = valid ? t0 : N - 1;
        const int64_t cell = cell_at(a, t);
        if (valid) a.cell_of[t] = (int32_t)cell;
        run_atomic_add(a.cell_count, cell, valid);
    }
}
__global__ __launch_bounds__(kBuildThreads) void k_bin(EvalArgs a) { bin_particles(a, blockIdx.x, gridDim.x); }

__global__ void k_scan_blocks(const int32_t *__restrict__ in, int64_t n, int32_t *__restrict__ bsum,
                              const int32_t *__restrict__ cond) {
    // the critical path's waves ahead of the structure factor's beside them
    __builtin_amdgcn_s_setprio(2);
    if (!*cond) return;
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t s = 0;
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) s += in[base + k];
    int32_t tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Exclusive scan of the tile: counts in registers, the block's scan, plus
// `before` (the count of the cells before the tile).
__device__ __forceinline__ void scan_tile(const int32_t *__restrict__ in, int64_t n, int32_t before,
                                          int32_t *__restrict__ out, int32_t *__restrict__ fill) {
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t vals[kScanItems];
    int32_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        vals[k] = base + k < n ? in[base + k] : 0;
        s += vals[k];
    }
    int32_t tot;
    int32_t off = block_exclusive_scan(s, &tot) + before;
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) {
            out[base + k] = off;
            fill[base + k] = off;
        }
        off += vals[k];
        if (base + k == n - 1) out[n] = off;
    }
}

// Each block adds the totals of the tiles before it (read in parallel from
// L2 and reduced in a fixed order) to its own exclusive scan.
__global__ void k_scan_apply(const int32_t *__restrict__ in, int64_t n, const int32_t *__restrict__ bsum,
                             int32_t *__restrict__ out, int32_t *__restrict__ fill, const int32_t *__restrict__ cond) {
    // the critical path's waves ahead of the structure factor's beside them
    __builtin_amdgcn_s_setprio(2);
    if (!*cond) return;
    int32_t pre = 0;
#pragma unroll 4
    for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += kBlock) pre += bsum[b];
    int32_t before;
    block_exclusive_scan(pre, &before);
    scan_tile(in, n, before, out, fill);
}

// Each particle to a slot of its cell (atomic order), with its id beside it
// for the per-cell sort.  With SCAN each block scans the cell counts for itself
// (up to kScanLds of them, kept in LDS: a launch less, 27,000 ions 43.6 us a step
// against 47) and the fill counters start at zero; otherwise they start at the
// scan kernels' cell starts.
constexpr int kScanLds = 12 * kBuildThreads;
template <bool SCAN>
__global__ __launch_bounds__(kBuildThreads) void k_cell_scatter(EvalArgs a) {
    // the critical path's waves ahead of the structure factor's beside them
    __builtin_amdgcn_s_setprio(2);
    if (!*a.rebuild) return;
    __shared__ int32_t start[SCAN ? kScanLds : 1];
    const int64_t N = a.N;
    if constexpr (SCAN) {
        const int32_t C = (int32_t)a.C;
        for (int32_t c = threadIdx.x; c < C; c += kBuildThreads) start[c] = a.cell_count[c];
        __syncthreads();
        const int32_t per = (C + kBuildThreads - 1) / kBuildThreads, at = (int32_t)threadIdx.x * per;
        const int32_t b = at < C ? at : C, e = b + per < C ? b + per : C;
        int32_t sum = 0, tot;
        for (int32_t c = b; c < e; ++c) sum += start[c];
        int32_t off = block_exclusive_scan<kBuildThreads>(sum, &tot);
        for (int32_t c = b; c < e; ++c) {
            const int32_t v = start[c];
            start[c] = off;
            off += v;
        }
        __syncthreads();
        if (blockIdx.x == 0) {
            for (int32_t c = threadIdx.x; c < C; c += kBuildThreads) a.cell_start[c] = start[c];
            if (threadIdx.x == 0) a.cell_start[C] = tot;
        }
    }
    // grid-stride as in k_bin (the order of the atomics within a cell is
    // undone by the per-cell id sort)
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < N; base += (int64_t)gridDim.x * blockDim.x) {
        const int64_t t = base + threadIdx.x;
        const bool valid = t < N;
        const int32_t cell = valid ? a.cell_of[t] : 0;
        const int32_t key = valid ? a.cur.id[t] : 0;
        int32_t dst = run_atomic_add(a.cell_fill, cell, valid);
        if (valid) {
            if constexpr (SCAN) dst += start[cell];
            a.src[dst] = (int32_t)t;
            a.skey[dst] = key;
        }
    }
}

// Per cell: order of its slots by particle id (the order becomes (cell, id),
// independent of the scatter's atomic order), and reset of its histogram and
// fill counts for the next evaluation; then the block gathers the state of its
// cells' slots into `nxt` in the new order, one thread per slot (writes are
// coalesced, reads stay close: particles move little between builds).  The
// positions become the new list reference `u`.  A slot's place is the number
// of smaller ids in its cell.  Up to kRankMax particles: one thread per cell,
// its keys in registers.  More (water-shaped sites at r_c = 10: about 150 a
// cell): one wave per cell, a slot per lane, every key broadcast; an insertion
// sort by one thread took 2 ms a build there.
// CELLS: cells per block of THREADS, a quarter of the threads (one thread each,
// larger ones left to the waves) or one per wave.
constexpr int kRankMax = 16;

// Slots [lo, hi) of one cell ordered by a wave.
__device__ __forceinline__ void sort_cell_wave(const int32_t *__restrict__ src, const int32_t *__restrict__ skey,
                                               int32_t *__restrict__ out, int32_t lo, int32_t hi, int lane) {
    for (int32_t i0 = lo; i0 < hi; i0 += 64) {
        const int32_t i = i0 + lane;
        const int32_t key = i < hi ? skey[i] : INT32_MAX, v = i < hi ? src[i] : 0;
        int32_t rank = 0;
        for (int32_t j0 = lo; j0 < hi; j0 += 64) {
            const int32_t kj = j0 + lane < hi ? skey[j0 + lane] : INT32_MAX;
            const int m = hi - j0 < 64 ? hi - j0 : 64;
            for (int j = 0; j < m; ++j) rank += __builtin_amdgcn_readlane(kj, j) < key ? 1 : 0;
        }
        if (i < hi) out[lo + rank] = v;
    }
}

// Slots [lo, lo + cnt) of one cell, cnt <= kRankMax, ordered by a thread.
__device__ __forceinline__ void sort_cell_thread(const int32_t *__restrict__ src, const int32_t *__restrict__ skey,
                                                 int32_t *__restrict__ out, int32_t lo, int32_t cnt) {
    int32_t sv[kRankMax], key[kRankMax];
#pragma unroll
    for (int i = 0; i < kRankMax; ++i) {
        sv[i] = i < cnt ? src[lo + i] : 0;
        key[i] = i < cnt ? skey[lo + i] : INT32_MAX;
    }
#pragma unroll
    for (int i = 0; i < kRankMax; ++i) {
        int32_t rank = 0;
#pragma unroll
        for (int j = 0; j < kRankMax; ++j) rank += key[j] < key[i] ? 1 : 0;
        if (i < cnt) out[lo + rank] = sv[i];
    }
}

// Slots [k0, k1) of the new order gathered from the state by a block of THREADS:
// two slots per thread and pass, all loads issued before the stores.
template <int THREADS>
__device__ __forceinline__ void gather_slots(const EvalArgs &a, const int32_t *out, int64_t k0, int64_t k1) {
    const int64_t N = a.N;
    constexpr int U = 2;
    for (int64_t kb = k0 + threadIdx.x; kb < k1; kb += U * THREADS) {
        int64_t tt[U];
#pragma unroll
        for (int j = 0; j < U; ++j) tt[j] = kb + j * THREADS < k1 ? out[kb + j * THREADS] : -1;
        double xv[U][3], vv[U][3], qv[U];
        uint32_t uv[U][3];
        float qfv[U];
        int32_t idv[U], cv[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int64_t t = tt[j] < 0 ? 0 : tt[j];
            for (int d = 0; d < 3; ++d) {
                xv[j][d] = a.cur.x[d * N + t];
                vv[j][d] = a.cur.v[d * N + t];
                uv[j][d] = a.u_tmp[d * N + t];
            }
            qv[j] = a.cur.q[t];
            qfv[j] = a.cur.qf[t];
            idv[j] = a.cur.id[t];
            cv[j] = a.cell_of[t];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int64_t k = kb + j * THREADS;
            if (tt[j] < 0) continue;
            for (int d = 0; d < 3; ++d) {
                a.nxt.x[d * N + k] = xv[j][d];
                a.nxt.v[d * N + k] = vv[j][d];
                a.u[d * N + k] = uv[j][d];
            }
            a.nxt.q[k] = qv[j];
            a.nxt.qf[k] = qfv[j];
            a.nxt.id[k] = idv[j];
            a.cell_sorted[k] = cv[j];
        }
        if (a.cur.dsp) {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                if (tt[j] < 0) continue;
                for (int d = 0; d < 3; ++d) a.nxt.dsp[d * N + kb + j * THREADS] = a.cur.dsp[d * N + tt[j]];
            }
        }
    }
}

template <int CELLS, int THREADS>
__global__ __launch_bounds__(THREADS) void k_sort_gather(EvalArgs a) {
    // the critical path's waves ahead of the structure factor's beside them
    __builtin_amdgcn_s_setprio(2);
    if (!*a.rebuild) return;
    __shared__ int32_t nbig, big[CELLS];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    int32_t *out = a.sorted;
    for (int64_t c0 = (int64_t)blockIdx.x * CELLS; c0 < a.C; c0 += (int64_t)gridDim.x * CELLS) {
        if constexpr (CELLS == THREADS / 64) {
            const int64_t c = c0 + wave;
            if (c < a.C) {
                sort_cell_wave(a.src, a.skey, out, a.cell_start[c], a.cell_start[c + 1], lane);
                if (lane == 0) a.cell_count[c] = a.cell_fill[c] = 0;
            }
        } else {
            if (threadIdx.x == 0) nbig = 0;
            __syncthreads();
            const int64_t c = c0 + threadIdx.x;
            if (threadIdx.x < CELLS && c < a.C) {
                const int32_t lo = a.cell_start[c], cnt = a.cell_start[c + 1] - lo;
                if (cnt <= kRankMax) {
                    sort_cell_thread(a.src, a.skey, out, lo, cnt);
                } else {
                    big[atomicAdd(&nbig, 1)] = (int32_t)threadIdx.x;
                }
                a.cell_count[c] = a.cell_fill[c] = 0;
            }
            __syncthreads();
            for (int k = wave; k < nbig; k += THREADS / 64) {
                const int64_t cb = c0 + big[k];
                sort_cell_wave(a.src, a.skey, out, a.cell_start[cb], a.cell_start[cb + 1], lane);
            }
        }
        // the block's permutation entries are visible to the whole block here
        __syncthreads();
        const int64_t c1 = c0 + CELLS < a.C ? c0 + CELLS : a.C;
        gather_slots<THREADS>(a, out, a.cell_start[c0], a.cell_start[c1]);
        // the next group's permutation entries are written after every
        // thread has read this group's
        __syncthreads();
    }
}

// The whole re-sort of a small batch by one block, in steps on a kept list,
// where most launches find nothing to do: one launch (some 3 us of a step) in
// place of four.  Histogram, order and sort stay in LDS, each thread holds its
// slots' values of an array across a barrier and stores them back in place, and
// the gather records follow, so that no copy back remains.  Per step of 200
// (5 builds | 40 builds), one launch against three: 1,000 ions 37.8 | 44 us
// against 47 | 49, 8,000 ions 38.8 | 48.9 against 44.5 | 50; with twice the slots
// and the state gathered through memory it lost (16,000 ions 41 | 66 us).
constexpr int kResortSlots = 8;
constexpr int kResortMax = kResortSlots * kBuildThreads;
constexpr int kResortCells = 3072;
__device__ __forceinline__ void resort_batch(const EvalArgs &a) {
    __shared__ uint32_t ent[kResortMax];  // (id, slot) by cell
    __shared__ uint16_t ord[kResortMax];
    __shared__ int32_t cnt[kResortCells], nbig;
    __shared__ uint16_t big[kResortMax / kRankMax];
    static_assert(kResortMax <= 1 << 16 && kResortMax % kRankMax == 0, "ids and slots are packed in 16 bits");
    __builtin_amdgcn_s_setprio(2);
    if (!*a.rebuild) return;
    const int32_t N = (int32_t)a.N, C = (int32_t)a.C, tid = threadIdx.x;
    for (int32_t c = tid; c < C; c += kBuildThreads) cnt[c] = 0;
    if (tid == 0) nbig = 0;
    __syncthreads();
    int32_t cell[kResortSlots], at[kResortSlots], src[kResortSlots];
    uint32_t key[kResortSlots];
#pragma unroll
    for (int i = 0; i < kResortSlots; ++i) {
        const int32_t t = tid + i * kBuildThreads, tc = t < N ? t : 0;
        cell[i] = (int32_t)cell_at(a, tc);
        key[i] = (uint32_t)a.cur.id[tc] << 16 | (uint32_t)t;
    }
#pragma unroll
    for (int i = 0; i < kResortSlots; ++i) {
        const int32_t t = tid + i * kBuildThreads;
        if (t >= N) continue;
        at[i] = atomicAdd(&cnt[cell[i]], 1);
        a.cell_of[t] = cell[i];
    }
    __syncthreads();
    {  // each thread scans a run of cells
        const int32_t per = (C + kBuildThreads - 1) / kBuildThreads;
        const int32_t b = tid * per < C ? tid * per : C, e = b + per < C ? b + per : C;
        int32_t sum = 0, tot;
        for (int32_t c = b; c < e; ++c) sum += cnt[c];
        int32_t off = block_exclusive_scan<kBuildThreads>(sum, &tot);
        for (int32_t c = b; c < e; ++c) {
            const int32_t v = cnt[c];
            cnt[c] = off;
            a.cell_start[c] = off;
            off += v;
        }
        if (tid == 0) a.cell_start[C] = N;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kResortSlots; ++i)
        if (tid + i * kBuildThreads < N) ent[cnt[cell[i]] + at[i]] = key[i];
    __syncthreads();
    for (int32_t c = tid; c < C; c += kBuildThreads) {
        const int32_t lo = cnt[c], n = (c + 1 < C ? cnt[c + 1] : N) - lo;
        if (n > kRankMax) {
            big[atomicAdd(&nbig, 1)] = (uint16_t)c;
            continue;
        }
        uint32_t v[kRankMax];
#pragma unroll
        for (int i = 0; i < kRankMax; ++i) v[i] = i < n ? ent[lo + i] : UINT32_MAX;
#pragma unroll
        for (int i = 0; i < kRankMax; ++i) {
            int32_t rank = 0;
#pragma unroll
            for (int j = 0; j < kRankMax; ++j) rank += v[j] < v[i] ? 1 : 0;
            if (i < n) ord[lo + rank] = (uint16_t)v[i];
        }
    }
    __syncthreads();
    for (int32_t k = tid >> 6; k < nbig; k += kBuildThreads / 64) {
        const int32_t c = big[k], lo = cnt[c], hi = c + 1 < C ? cnt[c + 1] : N;
        for (int32_t i = lo + (tid & 63); i < hi; i += 64) {
            const uint32_t v = ent[i];
            int32_t rank = 0;
            for (int32_t j = lo; j < hi; ++j) rank += ent[j] < v ? 1 : 0;
            ord[lo + rank] = (uint16_t)v;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kResortSlots; ++i) src[i] = tid + i * kBuildThreads < N ? ord[tid + i * kBuildThreads] : 0;
    // charges, ids, cells and quantised coordinates, then the FP64 vectors one by one
    {
        double q[kResortSlots];
        float qf[kResortSlots];
        int32_t id[kResortSlots], cs[kResortSlots];
        uint32_t u[kResortSlots][3];
#pragma unroll
        for (int i = 0; i < kResortSlots; ++i) {
            q[i] = a.cur.q[src[i]];
            qf[i] = a.cur.qf[src[i]];
            id[i] = a.cur.id[src[i]];
            cs[i] = a.cell_of[src[i]];
            for (int d = 0; d < 3; ++d) u[i][d] = a.u_tmp[(int64_t)d * N + src[i]];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kResortSlots; ++i) {
            const int32_t k = tid + i * kBuildThreads;
            if (k >= N) continue;
            a.cur.q[k] = q[i];
            a.cur.qf[k] = qf[i];
            a.cur.id[k] = id[i];
            a.cell_sorted[k] = cs[i];
            for (int d = 0; d < 3; ++d) a.u[(int64_t)d * N + k] = a.u_tmp[(int64_t)d * N + k] = u[i][d];
            if (a.pk) a.pk[k] = make_uint4(u[i][0], u[i][1], u[i][2], __float_as_uint(qf[i]));
        }
    }
    double *const rows[3] = {a.cur.x, a.cur.v, a.cur.dsp};
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        double *__restrict__ p = rows[f];
        if (!p) continue;
        double r[kResortSlots][3];
#pragma unroll
        for (int i = 0; i < kResortSlots; ++i)
            for (int d = 0; d < 3; ++d) r[i][d] = p[(int64_t)d * N + src[i]];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kResortSlots; ++i) {
            const int32_t k = tid + i * kBuildThreads;
            if (k >= N) continue;
            for (int d = 0; d < 3; ++d) p[(int64_t)d * N + k] = r[i][d];
            if (f == 0 && a.pkx) a.pkx[k] = PosQ64{r[i][0], r[i][1], r[i][2], a.cur.q[k]};
        }
    }
}

__global__ __launch_bounds__(kBuildThreads) void k_resort_one(EvalArgs a) { resort_batch(a); }

// Evaluations on one stream: the structure factor, which reads its own copy of the
// state, in one launch with the first kernel of the list build (ONE: the re-sort of
// a small batch, else the histogram), whose blocks come first.  On the steps that
// build nothing that is a launch saved (us a step: 1,000 ions x 100 wave vectors
// 22.9 -> 20.7, 26,998 x 130 34.4 -> 32.9).
template <bool F64, bool ONE>
__global__ __launch_bounds__(1024, ONE ? 4 : 8) void k_rho_build(EvalArgs a, const RhoItem *__restrict__ items,
                                                                 int32_t nitems) {
    const int32_t first = (int32_t)gridDim.x - nitems, b = (int32_t)blockIdx.x;
    if (b >= first) rho_items<F64>(a, items, nitems, b - first, nitems);
    else if constexpr (ONE) resort_batch(a);
    else bin_particles(a, b, first);
}

// Slot of every caller index (the inverse of the id permutation of the
// current order), then the near and far forces of the requested indices.
__global__ __launch_bounds__(kBlock) void k_invert_ids(int64_t N, const int32_t *__restrict__ id,
                                                       int32_t *__restrict__ slot_of) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t < N) slot_of[id[t]] = (int32_t)t;
}

__global__ __launch_bounds__(kBlock) void k_gather_forces(int64_t N, int64_t m, const int64_t *__restrict__ ids,
                                                          const int32_t *__restrict__ slot_of,
                                                          const double *__restrict__ Fn, const double *__restrict__ Ff,
                                                          double *__restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= m) return;
    const int64_t t = slot_of[ids[k]];
    for (int d = 0; d < 3; ++d) {
        out[6 * k + d] = Fn[d * N + t];
        out[6 * k + 3 + d] = Ff[d * N + t];
    }
}

}  // namespace

void launch_subset_forces(const EvalArgs &a, int64_t m, const int64_t *ids, int32_t *slot_of, double *out,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_invert_ids, dim3(grid_for(a.N, kBlock)), dim3(kBlock), 0, s, a.N, a.cur.id, slot_of);
    if (m > 0)
        hipLaunchKernelGGL(k_gather_forces, dim3(grid_for(m, kBlock)), dim3(kBlock), 0, s, a.N, m, ids, slot_of,
                           a.Fn, a.Ff, out);
}

void launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, p, n, v);
}

void launch_kdq(const EvalArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_kdq, dim3(grid_for(a.N, kBlock)), dim3(kBlock), 0, s, a);
}

int64_t scan_blocksums_size(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

inline unsigned capped(int64_t blocks, int64_t cap) { return (unsigned)(blocks < cap ? (blocks < 1 ? 1 : blocks) : cap); }
// Threads of a build block, and the grid for n items at `per` a block.
inline int build_threads(const EvalArgs &a) { return a.wide ? kWideThreads : kBuildThreads; }
inline unsigned build_grid(const EvalArgs &a, int64_t n, int per) {
    return capped(grid_for(n, per), a.wide ? kWideGrid : kBuildGrid);
}

// More cells than the scatter scans for itself: scanned by one block up to this
// many (its 17 tiles at 68,921 cells take about 60 us of the one step in some
// thirty that builds, and one launch of some 4 us instead of two on all others), by
// two kernels (about 10 us there) above and where the evaluation builds for certain.
constexpr int64_t kScanOne = 131072;

void launch_bin(const EvalArgs &a, hipStream_t s) {
    const int threads = build_threads(a);
    hipLaunchKernelGGL(k_bin, dim3(build_grid(a, a.N, threads)), dim3((unsigned)threads), 0, s, a);
}

void launch_rho_build(const EvalArgs &a, bool f64, const RhoItem *items, int32_t nitems, bool one, hipStream_t s) {
    // (few blocks of the histogram whatever a.wide: each holds a structure-factor
    // block's place until it ends; 1,000,000 ions x 45, 977 blocks | 128: 175 | 160 us)
    const dim3 grid((unsigned)nitems + (one ? 1u : capped(grid_for(a.N, kBuildThreads), kBuildGrid))), block(kBuildThreads);
    if (f64 && one) hipLaunchKernelGGL((k_rho_build<true, true>), grid, block, 0, s, a, items, nitems);
    else if (f64) hipLaunchKernelGGL((k_rho_build<true, false>), grid, block, 0, s, a, items, nitems);
    else if (one) hipLaunchKernelGGL((k_rho_build<false, true>), grid, block, 0, s, a, items, nitems);
    else hipLaunchKernelGGL((k_rho_build<false, false>), grid, block, 0, s, a, items, nitems);
}

bool scan_apart(const EvalArgs &a) { return a.C > kScanLds; }

void launch_scan(const EvalArgs &a, hipStream_t s) {
    const int64_t n = a.C;
    if (n <= kScanOne && !a.due) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kBuildThreads), 0, s, a.cell_count, n, a.cell_start, a.cell_fill,
                           (const int32_t *)a.rebuild);
        return;
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nb), dim3(kBlock), 0, s, a.cell_count, n, a.blocksums,
                       (const int32_t *)a.rebuild);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kBlock), 0, s, a.cell_count, n, a.blocksums,
                       a.cell_start, a.cell_fill, (const int32_t *)a.rebuild);
}

void launch_cell_scatter(const EvalArgs &a, hipStream_t s) {
    const int threads = scan_apart(a) ? build_threads(a) : kBuildThreads;
    const dim3 grid(build_grid(a, a.N, threads)), block((unsigned)threads);
    if (scan_apart(a)) hipLaunchKernelGGL(k_cell_scatter<false>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(k_cell_scatter<true>, grid, block, 0, s, a);
}

// Batches that k_resort_one takes.
bool resort_in_one(const EvalArgs &a) { return a.N <= kResortMax && a.C <= kResortCells; }

void launch_resort_one(const EvalArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_resort_one, dim3(1), dim3(kBuildThreads), 0, s, a);
}

void launch_sort_gather(const EvalArgs &a, hipStream_t s) {
    auto go = [&](auto cells, auto threads) {
        constexpr int CELLS = decltype(cells)::value, THREADS = decltype(threads)::value;
        hipLaunchKernelGGL((k_sort_gather<CELLS, THREADS>), dim3(build_grid(a, a.C, CELLS)), dim3(THREADS), 0, s, a);
    };
    using std::integral_constant;
    constexpr integral_constant<int, kBuildThreads> large{};
    constexpr integral_constant<int, kWideThreads> small{};
    // one wave per cell where cells hold more than a thread ranks
    const bool waves = a.N > kRankMax * a.C;
    if (a.wide && waves) go(integral_constant<int, kWideThreads / 64>{}, small);
    else if (a.wide) go(integral_constant<int, kWideThreads / 4>{}, small);
    else if (waves) go(integral_constant<int, kBuildThreads / 64>{}, large);
    else go(integral_constant<int, kBuildThreads / 4>{}, large);
}

}  // namespace rbsog
