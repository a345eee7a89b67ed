// Transfers between the caller's arrays (row-major n x 3 in the caller's
// particle order) and the context's state (structure of arrays in cell order)
// for gfx950: the order is changed on the device, between a staging array in
// the caller's order and the state, so the host only moves one contiguous
// block each way.
//
// Bound by the link to the host (24 B per particle each way; the kernels move
// 52 B per particle of HBM beside it).  With the order changed by the host
// (ids fetched, one scattered pass over each array) 2,097,152 ions took 27.8
// ms to set positions and 50 ms to read the state.
#include <climits>

#include "rbsog_internal.h"

namespace rbsog {

namespace {

constexpr int kBlock = 256;
inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// The smallest particle index with a non-finite component into *bad (which
// holds INT32_MAX between calls).
__global__ __launch_bounds__(kBlock) void k_rows_finite(int64_t n, const double *__restrict__ rows,
                                                        int32_t *__restrict__ bad) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    if (!isfinite(rows[3 * i]) || !isfinite(rows[3 * i + 1]) || !isfinite(rows[3 * i + 2])) atomicMin(bad, (int32_t)i);
}

// Rows into the slots of the current order, unless an entry was not finite;
// the verdict goes to the host's status block.
__global__ __launch_bounds__(kBlock) void k_rows_in(int64_t n, const int32_t *__restrict__ id,
                                                    const double *__restrict__ rows, double *__restrict__ dst,
                                                    const int32_t *__restrict__ bad, int32_t *__restrict__ rebuild,
                                                    IoStat *__restrict__ st) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int32_t b = *bad;
    if (t == 0) {
        st->bad = b;
        if (b == INT_MAX && rebuild) *rebuild = 1;
    }
    if (t >= n || b != INT_MAX) return;
    const int64_t i = id[t];
    for (int d = 0; d < 3; ++d) dst[d * n + t] = rows[3 * i + d];
}

// Slots into rows.  WRAP: positions wrapped into [0, L) of their system.
template <bool WRAP>
__global__ __launch_bounds__(kBlock) void k_rows_out(int64_t n, const int32_t *__restrict__ id,
                                                     const double *__restrict__ src, const SysDev *__restrict__ sys,
                                                     const int32_t *__restrict__ sys_of, double *__restrict__ rows) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= n) return;
    const int64_t i = id[t];
    const SysDev *sp = WRAP ? sys + sys_of[t] : nullptr;
    for (int d = 0; d < 3; ++d) {
        double v = src[d * n + t];
        if constexpr (WRAP) {
            const double L = sp->g.L[d], r = v / L;
            v = (r - floor(r)) * L;
        }
        rows[3 * i + d] = v;
    }
}

// Total force F_N + F* of every slot into rows; the smallest index of a
// particle whose force is not finite into *bad.
__global__ __launch_bounds__(kBlock) void k_forces_out(int64_t n, const int32_t *__restrict__ id,
                                                       const double *__restrict__ Fn, const double *__restrict__ Ff,
                                                       double *__restrict__ rows, int32_t *__restrict__ bad) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= n) return;
    const int64_t i = id[t];
    bool ok = true;
    for (int d = 0; d < 3; ++d) {
        const double f = Fn[d * n + t] + Ff[d * n + t];
        ok = ok && isfinite(f);
        rows[3 * i + d] = f;
    }
    if (!ok) atomicMin(bad, (int32_t)i);
}

// Error flags, the largest list count, the builds made and the finiteness
// verdict to the host (one kernel in place of a copy each); *bad holds INT32_MAX
// again afterwards, whatever the host makes of the report.
__global__ void k_status(const int32_t *__restrict__ flag, const int32_t *__restrict__ pmax,
                         const int64_t *__restrict__ nbuild, int32_t *__restrict__ bad, IoStat *__restrict__ st) {
    if (threadIdx.x != 0) return;
    st->nbuild = *nbuild;
    st->flag = *flag;
    st->pmax = *pmax;
    st->bad = *bad;
    *bad = INT_MAX;
}

// Kinetic energy of the velocities as they stand: per far item and wave (a
// fixed butterfly), as the far kernel leaves it.
__global__ __launch_bounds__(256) void k_kin_items(EvalArgs a, const FarItem *__restrict__ items, int32_t nitems) {
    for (int32_t itx = blockIdx.x; itx < nitems; itx += gridDim.x) {
        const FarItem item = items[itx];
        const int64_t i = item.t0 + threadIdx.x;
        double ke = 0.0;
        if (i < item.t1) {
            const double x = a.cur.v[i], y = a.cur.v[a.N + i], z = a.cur.v[2 * a.N + i];
            ke = 0.5 * a.mass * ((x * x + y * y) + z * z);
        }
        for (int o = 32; o > 0; o >>= 1) ke += __shfl_xor(ke, o, 64);
        if ((threadIdx.x & 63) == 0) a.kpart[(int64_t)itx * 4 + (threadIdx.x >> 6)] = ke;
    }
}

// Per system: the sum of its items' partials (strided sums, then a fixed tree).
__global__ __launch_bounds__(256) void k_kin_sum(EvalArgs a) {
    __shared__ double w[256];
    const SysDev &sp = a.sys[blockIdx.x];
    double s = 0.0;
    for (int64_t i = (int64_t)sp.ft0 * 4 + threadIdx.x; i < (int64_t)sp.ft1 * 4; i += 256) s += a.kpart[i];
    w[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) w[threadIdx.x] += w[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.kin[blockIdx.x] = w[0];
}

}  // namespace

void launch_rows_in(const EvalArgs &a, const double *rows, double *dst, int32_t *bad, int32_t *rebuild, IoStat *st,
                    hipStream_t s) {
    const dim3 grid(blocks_for(a.N)), block(kBlock);
    hipLaunchKernelGGL(k_rows_finite, grid, block, 0, s, a.N, rows, bad);
    hipLaunchKernelGGL(k_rows_in, grid, block, 0, s, a.N, a.cur.id, rows, dst, (const int32_t *)bad, rebuild, st);
}

void launch_rows_out(const EvalArgs &a, const double *src, double *rows, bool wrap, hipStream_t s) {
    const dim3 grid(blocks_for(a.N)), block(kBlock);
    if (wrap) hipLaunchKernelGGL(k_rows_out<true>, grid, block, 0, s, a.N, a.cur.id, src, a.sys, a.sys_of, rows);
    else hipLaunchKernelGGL(k_rows_out<false>, grid, block, 0, s, a.N, a.cur.id, src, a.sys, a.sys_of, rows);
}

void launch_forces_out(const EvalArgs &a, double *rows, int32_t *bad, hipStream_t s) {
    hipLaunchKernelGGL(k_forces_out, dim3(blocks_for(a.N)), dim3(kBlock), 0, s, a.N, a.cur.id, a.Fn, a.Ff, rows, bad);
}

void launch_status(const EvalArgs &a, int32_t *bad, IoStat *st, hipStream_t s) {
    hipLaunchKernelGGL(k_status, dim3(1), dim3(64), 0, s, a.flag, a.pmax, a.nbuild, bad, st);
}

void launch_kinetic_now(const EvalArgs &a, const FarItem *items, int32_t nitems, int32_t block_size, hipStream_t s) {
    hipLaunchKernelGGL(k_kin_items, dim3((unsigned)nitems), dim3((unsigned)block_size), 0, s, a, items, nitems);
    hipLaunchKernelGGL(k_kin_sum, dim3((unsigned)a.nsys), dim3(256), 0, s, a);
}

}  // namespace rbsog
