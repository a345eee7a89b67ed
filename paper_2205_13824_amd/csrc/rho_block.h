// The batch's structure factor: partial sums of rho over work items, shared by its
// own kernel (kernels_far.hip) and the launches that carry the first kernel of a
// list build along (kernels_md.hip).
#pragma once

#include "rbsog_internal.h"
#include "rho_core.h"

namespace rbsog {

typedef const SysDev __attribute__((address_space(4))) CSys;

// Uniform values loaded from memory: keep them scalar.
__device__ __forceinline__ int32_t rfl(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t rfl64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// read-only within the kernels that read them uniformly: scalar loads
typedef const double __attribute__((address_space(4))) CF64;
// Particles [ja, jb) of a wave in FP64, four read at once, then used.
__device__ __forceinline__ void sum_uniform64(CF64 *x, CF64 *q, int64_t n, int64_t ja, int64_t jb, const double2 *turn,
                                              double mx, double my, double mz, double &re, double &im) {
    auto add = [&](double px, double py, double pz, double pq) {
        const double t = mx * px + my * py + mz * pz;
        double sn, cs;
        rmath::sincos2pi_tab(t, turn, &sn, &cs);
        re = fma(pq, cs, re);
        im = fma(pq, sn, im);
    };
    int64_t j = ja;
    for (; j + 4 <= jb; j += 4) {
        double p[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            p[0][g] = x[j + g];
            p[1][g] = x[n + j + g];
            p[2][g] = x[2 * n + j + g];
            p[3][g] = q[j + g];
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) add(p[0][g], p[1][g], p[2][g], p[3][g]);
    }
    for (; j < jb; ++j) add(x[j], x[n + j], x[2 * n + j], q[j]);
}

// Structure factor partial sums over the work items (grid-stride).  Item
// (s, kg, chunk, [j0, j1)): wave w handles k tile (w % kt) of group kg (one
// wave vector per lane) for particle stream (w / kt); kt * streams <= 16
// waves per block.  FP32C: the block stages kStage particles at a time in LDS (one
// coalesced load per thread) and sums them (rho_core.h).  FP64: a stream is a run
// of the chunk, its particles read as uniform (scalar) loads: the LDS, which the
// 16-byte reads of the turn table at a lane's own phase keep busy, carries nothing
// else (staged there, a particle's 32 bytes for each lane cost it as much again:
// 300,000 ions x 200 76 us against 68, 98,304 sites x 211 33 against 24).  The
// streams' sums are added in a fixed order.  Two blocks per CU (64 VGPRs).
template <bool F64>
__device__ __forceinline__ void rho_items(const EvalArgs &a, const RhoItem *__restrict__ items, int32_t nitems,
                                          int32_t block, int32_t blocks) {
    __shared__ double2 red[1024];
    __shared__ uint4 st32[F64 ? 1 : kStage];
    __shared__ int2 wcnt[F64 ? 1 : 16];
    // FP64: cos and sin of the kTurnTab turns (sincos2pi_tab)
    __shared__ double2 turn[F64 ? rmath::kTurnTab : 1];
    if constexpr (F64) fill_turns(turn);
    const int64_t n = a.N;
    // the state as the kick/drift kernel left it, in its copy: the re-sort of
    // the state into cell order may run meanwhile
    const double *__restrict__ x = a.rs_x;
    const double *__restrict__ q = a.rs_q;
    const float *__restrict__ qf = a.rs_qf;
    const uint32_t *__restrict__ u = a.rs_u;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    for (int32_t itx = block; itx < nitems; itx += blocks) {
        const RhoItem item = items[itx];
        const int32_t sys = rfl(item.sys), kg = rfl(item.kg), chunk = rfl(item.chunk);
        CSys *sp = (CSys *)(a.sys + sys);
        const int32_t P = sp->P, kt = sp->kt, streams = sp->streams;
        const int kti = wave % kt, st = wave / kt;
        const int32_t k = (kg * kt + kti) * 64 + lane;
        const bool active = k < P && st < streams;
        // the batch's wave vectors, read from the sequence at the cursor
        const int32_t *__restrict__ mk = sp->kseq + 3 * (rfl64(a.kcur[sys]) + (k < P ? k : 0));
        const int64_t j0 = rfl64(item.j0), j1 = rfl64(item.j1);
        double re = 0.0, im = 0.0;
        if constexpr (F64) {
            // the wave vectors in table units per length
            const double mx = mk[0] * (sp->g.invL[0] * rmath::kTurnTab), my = mk[1] * (sp->g.invL[1] * rmath::kTurnTab),
                         mz = mk[2] * (sp->g.invL[2] * rmath::kTurnTab);
            if (st < streams) {
                // the stream's particles, a run of the chunk
                const int64_t per = (j1 - j0 + streams - 1) / streams;
                const int64_t ja = j0 + st * per < j1 ? j0 + st * per : j1, jb = ja + per < j1 ? ja + per : j1;
                sum_uniform64((CF64 *)x, (CF64 *)q, n, ja, jb, turn, mx, my, mz, re, im);
            }
        } else {
            const uint32_t mx = (uint32_t)mk[0], my = (uint32_t)mk[1], mz = (uint32_t)mk[2];
            for (int64_t jb = j0; jb < j1; jb += kStage) {
                const int cnt = (int)(j1 - jb < kStage ? j1 - jb : kStage);
                const bool have = (int)threadIdx.x < cnt;
                uint32_t ux = 0, uy = 0, uz = 0, qb = 0;
                if (have) {
                    const int64_t j = jb + threadIdx.x;
                    ux = u[j];
                    uy = u[n + j];
                    uz = u[2 * n + j];
                    qb = __float_as_uint(qf[j]);
                }
                const int np = stage_pairs(have, ux, uy, uz, qb, st32, wcnt);
                if (st < streams) sum_staged32(st32, np, cnt - 2 * np, mx, my, mz, st, streams, re, im);
                __syncthreads();
            }
        }
        red[threadIdx.x] = make_double2(re, im);
        __syncthreads();
        if (st == 0 && active) {
            double sr = 0.0, si = 0.0;
            for (int s2 = 0; s2 < streams; ++s2) {
                const double2 v = red[(s2 * kt + kti) * 64 + lane];
                sr += v.x;
                si += v.y;
            }
            // layout [k][chunk]: the reduction reads each k's partials contiguously
            const int64_t o = sp->pofs + (int64_t)k * sp->nch + chunk;
            a.partial[2 * o] = sr;
            a.partial[2 * o + 1] = si;
        }
        __syncthreads();
        if (sp->zmode != 0 && kg == 0) {
            // dipole moment of the chunk, sum_j q_j x_j over the wrapped
            // positions, for the zero-frequency mode term (fixed order)
            double mx = 0.0, my = 0.0, mz = 0.0;
            for (int64_t j = j0 + threadIdx.x; j < j1; j += blockDim.x) {
                const double qj = q[j];
                mx = fma(qj, x[j], mx);
                my = fma(qj, x[n + j], my);
                mz = fma(qj, x[2 * n + j], mz);
            }
            red[threadIdx.x] = make_double2(mx, my);
            __syncthreads();
            for (int w = 512; w > 0; w >>= 1) {
                if ((int)threadIdx.x < w) {
                    red[threadIdx.x].x += red[threadIdx.x + w].x;
                    red[threadIdx.x].y += red[threadIdx.x + w].y;
                }
                __syncthreads();
            }
            const double2 mxy = red[0];
            __syncthreads();
            red[threadIdx.x] = make_double2(mz, 0.0);
            __syncthreads();
            for (int w = 512; w > 0; w >>= 1) {
                if ((int)threadIdx.x < w) red[threadIdx.x].x += red[threadIdx.x + w].x;
                __syncthreads();
            }
            if (threadIdx.x == 0) {
                const int64_t c = 3 * (sp->choff + chunk);
                a.dip_part[c] = mxy.x;
                a.dip_part[c + 1] = mxy.y;
                a.dip_part[c + 2] = red[0].x;
            }
            __syncthreads();
        }
    }
}

}  // namespace rbsog
