// Sums of the structure factor over particles staged in LDS (Sec. 3.1:
// rho(k) = sum_j q_j e^{i k.r_j}), shared by the batch's structure factor in FP32C
// (rho_block.h) and the context-free one (structure_factor.hip).  Blocks
// of 1024 threads, 16 waves: a wave holds one wave vector per lane and sums
// every streams-th staged particle from its stream's on, each read an LDS
// broadcast to the wave.
#pragma once

#include <type_traits>

#include "rbsog_math.h"

namespace rbsog {

// particles staged at a time: fixed-point coordinates and FP32 charge in
// FP32C, fractional coordinates (in table units) and charge in FP64
constexpr int kStage = 1024;
struct Stage64 {
    double sx, sy, sz, q;
};

// cos and sin of the kTurnTab turns in LDS for sincos2pi_tab (FP64 forms);
// all threads of the block reach the barrier.
__device__ __forceinline__ void fill_turns(double2 *turn) {
    for (int j = threadIdx.x; j < rmath::kTurnTab; j += blockDim.x) {
        const double f = (double)j / rmath::kTurnTab;
        double sn, cs;
        rmath::sincos2pi(f - rint(f), &sn, &cs);
        turn[j] = make_double2(cs, sn);
    }
    __syncthreads();
}

// FP32C staging of up to 1024 particles, one per thread (`have`: fixed-point
// coordinates u and the charge's bits qb), for the structure factor (blocks of
// 1024 threads): each wave splits its 64 particles by the sign of the charge
// and pairs consecutive ones of a sign (lane order) whose charges are equal; a
// pair (u1, u2) is written as two records, h = u1 + ((u2 - u1) >> 1) with 2q
// and d = u1 - h (so u1 = h + d and u2 = h - d up to one unit of 2^-32 of the
// box: the pair's phases are m.h +- m.d mod 2^32), the particles left single
// after all pairs as (u, q).  EVEN with `even` (the same in every thread): only
// particles whose coordinates agree in their lowest bits are paired, whose
// halves are exact, and more of them stay single.  Returns the block's number of
// pairs; the records fill st32[0, particles).  Ends with a barrier.
template <bool EVEN = false>
__device__ __forceinline__ int stage_pairs(bool have, uint32_t ux, uint32_t uy, uint32_t uz, uint32_t qb, uint4 *st32,
                                           int2 *wcnt, bool even = false) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float q = __uint_as_float(qb);
    const bool pos = q > 0.f;
    const uint64_t all = __builtin_amdgcn_ballot_w64(have), plus = __builtin_amdgcn_ballot_w64(have && pos);
    uint64_t mine = pos ? plus : (all & ~plus);
    if constexpr (EVEN) {
        if (even) {
            for (const uint32_t b : {ux, uy, uz}) {
                const uint64_t odd = __builtin_amdgcn_ballot_w64((b & 1u) != 0u);
                mine &= (b & 1u) ? odd : ~odd;
            }
        }
    }
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint64_t below = mine & lt, above = mine & ~(lt | (1ull << lane));
    const int rank = __builtin_popcountll(below), ncls = __builtin_popcountll(mine);
    const int nl = above ? __builtin_ctzll(above) : lane;        // next lane of the class
    const int pl = below ? 63 - __builtin_clzll(below) : lane;   // previous lane of the class
    const uint32_t nx = __shfl(ux, nl, 64), ny = __shfl(uy, nl, 64), nz = __shfl(uz, nl, 64);
    const uint32_t nq = __shfl(qb, nl, 64), pq = __shfl(qb, pl, 64);
    // (2 q of a pair stays finite)
    const bool twice = fabsf(q) < 0x1.0p126f;
    const bool lead = have && twice && (rank & 1) == 0 && rank + 1 < ncls && nq == qb;
    const bool follow = have && twice && (rank & 1) == 1 && pq == qb;
    const bool single = have && !lead && !follow;
    const uint64_t lm = __builtin_amdgcn_ballot_w64(lead), sm = __builtin_amdgcn_ballot_w64(single);
    if (lane == 0) wcnt[wave] = make_int2(__builtin_popcountll(lm), __builtin_popcountll(sm));
    __syncthreads();
    int pofs = 0, sofs = 0, np = 0;
    for (int w = 0; w < 16; ++w) {
        const int2 c = wcnt[w];
        np += c.x;
        if (w < wave) {
            pofs += c.x;
            sofs += c.y;
        }
    }
    if (lead) {
        const int o = 2 * (pofs + __builtin_popcountll(lm & lt));
        const uint32_t hx = ux + (uint32_t)((int32_t)(nx - ux) >> 1), hy = uy + (uint32_t)((int32_t)(ny - uy) >> 1),
                       hz = uz + (uint32_t)((int32_t)(nz - uz) >> 1);
        st32[o] = make_uint4(hx, hy, hz, __float_as_uint(2.f * q));
        st32[o + 1] = make_uint4(ux - hx, uy - hy, uz - hz, 0u);
    }
    if (single) st32[2 * np + sofs + __builtin_popcountll(sm & lt)] = make_uint4(ux, uy, uz, qb);
    __syncthreads();
    return np;
}

// The staged pairs and singles of stream st (of `streams`) for one wave
// vector per lane, added to (re, im).  A pair of equal charge q with phases
// t_m +- t_d adds 2 q cos(t_d) e^{i t_m} (cos a + cos b = 2 cos((a+b)/2)
// cos((a-b)/2), sin a + sin b = 2 sin((a+b)/2) cos((a-b)/2)): three
// transcendentals and three multiply-adds where the two particles take four
// of each.  FP32 sums over runs of 16 pairs (32 singles), then FP64.
// ROUND: phases rounded to the 2^-23 turns that the hardware sine takes (half
// a unit enters each chain as its addend) instead of truncated; the batch's
// structure factor truncates, and the far force takes the offset back.
template <bool ROUND = false>
__device__ __forceinline__ void sum_staged32(const uint4 *st32, int np, int ns, uint32_t mx, uint32_t my, uint32_t mz,
                                             int st, int streams, double &re, double &im) {
    uint64_t half = 256u;
    if constexpr (ROUND) asm volatile("" : "+v"(half));  // held in registers
    auto phase = [&](const uint4 &p) {
        if constexpr (ROUND) return rmath::phase_rev(rmath::dot3_add_mod32_v(mx, my, mz, p.x, p.y, p.z, half));
        else return rmath::phase_rev(rmath::dot3_mod32_v(mx, my, mz, p.x, p.y, p.z));
    };
    auto pairs = [&](auto one) {
        constexpr bool ONE = decltype(one)::value;
        const int sd = ONE ? 1 : streams;
        int h = st;
        for (; h + 16 * sd <= np; h += 16 * sd) {
            float rf = 0.f, fi = 0.f;
            for (int g0 = 0; g0 < 16; g0 += 4) {
                uint4 pa[4], pb[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    pa[g] = st32[2 * (h + (g0 + g) * sd)];
                    pb[g] = st32[2 * (h + (g0 + g) * sd) + 1];
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float fm = phase(pa[g]);
                    const float fd = phase(pb[g]);
                    const float w = __uint_as_float(pa[g].w) * __builtin_amdgcn_cosf(fd);
                    rf = fmaf(w, __builtin_amdgcn_cosf(fm), rf);
                    fi = fmaf(w, __builtin_amdgcn_sinf(fm), fi);
                }
            }
            re += rf;
            im += fi;
        }
        float rf = 0.f, fi = 0.f;
        for (; h < np; h += sd) {
            const uint4 pa = st32[2 * h], pb = st32[2 * h + 1];
            const float fm = phase(pa);
            const float fd = phase(pb);
            const float w = __uint_as_float(pa.w) * __builtin_amdgcn_cosf(fd);
            rf = fmaf(w, __builtin_amdgcn_cosf(fm), rf);
            fi = fmaf(w, __builtin_amdgcn_sinf(fm), fi);
        }
        re += rf;
        im += fi;
    };
    if (streams == 1) pairs(std::true_type{});
    else pairs(std::false_type{});
    // the particles left single (at most two per wave of the stage, more
    // where charges differ)
    const uint4 *sg = st32 + 2 * np;
    float rf = 0.f, fi = 0.f;
    for (int h = st; h < ns; h += streams) {
        const uint4 p = sg[h];
        const float f = phase(p);
        const float pq = __uint_as_float(p.w);
        rf = fmaf(pq, __builtin_amdgcn_cosf(f), rf);
        fi = fmaf(pq, __builtin_amdgcn_sinf(f), fi);
    }
    re += rf;
    im += fi;
}

// The staged particles of stream st in FP64: four read at once, then used.
// Phases m.s of any int32 m.
__device__ __forceinline__ void sum_staged64(const Stage64 *st64, int cnt, const double2 *turn, double mx, double my,
                                             double mz, int st, int streams, double &re, double &im) {
    auto add = [&](const Stage64 &p) {
        const double t = mx * p.sx + my * p.sy + mz * p.sz;
        double sn, cs;
        rmath::sincos2pi_tab<true>(t, turn, &sn, &cs);
        re = fma(p.q, cs, re);
        im = fma(p.q, sn, im);
    };
    int h = st;
    for (; h + 4 * streams <= cnt; h += 4 * streams) {
        Stage64 p[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) p[g] = st64[h + g * streams];
#pragma unroll
        for (int g = 0; g < 4; ++g) add(p[g]);
    }
    for (; h < cnt; h += streams) add(st64[h]);
}

}  // namespace rbsog
