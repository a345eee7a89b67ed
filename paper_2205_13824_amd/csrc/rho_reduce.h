// The structure factor's reduction by one wave per record, shared by its own
// kernel (kernels_far.hip) and the list pass that carries it along
// (kernels_near.hip).
#pragma once

#include "rbsog_internal.h"
#include "rbsog_math.h"

namespace rbsog {

// Sum over the wave in a fixed order (the same on every run).
__device__ __forceinline__ double record_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// A system's k-th wave vector of the batch and its weight (the cursor still
// points at the batch), requested ahead of the sums.
struct KVec {
    int32_t m[3];
    double w;
};
__device__ __forceinline__ KVec batch_vector(const EvalArgs &a, const SysDev &sd, int32_t sys, int32_t k) {
    const int64_t e = a.kcur[sys] + k;
    return KVec{{sd.kseq[3 * e], sd.kseq[3 * e + 1], sd.kseq[3 * e + 2]}, sd.kw ? sd.kw[e] : sd.w_rb};
}

// Record r from its wave vector and rho: rho and the per-k energy stored, and
// the amplitude-phase records of both forms written.
__device__ __forceinline__ void write_record(const EvalArgs &a, const SysDev &sd, int64_t r, const KVec &kv, double re,
                                             double im) {
    a.rho[r] = re;
    a.rho[a.K + r] = im;
    const int32_t *m = kv.m;
    const double w = kv.w;
    a.ek[r] = 0.5 * w * (re * re + im * im);
    // amplitude-phase record: phi = arg(rho) / (2 pi), a = w |rho| k
    const double phi = atan2(im, re) * (1.0 / rmath::kTwoPi);
    const double mag = hypot(re, im);
    const double c = w * mag * rmath::kTwoPi;
    KRec64 h;
    h.mx = m[0];
    h.my = m[1];
    h.mz = m[2];
    h.phi = phi * rmath::kTurnTab;
    h.ax = c * h.mx * sd.g.invL[0];
    h.ay = c * h.my * sd.g.invL[1];
    h.az = c * h.mz * sd.g.invL[2];
    h.pad = 0.0;
    a.kb64[r] = h;
    // FP32 form: phi in 2^-32 turns, plus 2^9 units: the FP32 phases of
    // the structure factor and of the far force are each truncated
    // to 2^-23 turns (half a unit of it low on average), which this
    // offset takes back
    KRec32 f;
    f.nmx = -m[0];
    f.nmy = -m[1];
    f.nmz = -m[2];
    f.phi = (uint32_t)(int64_t)rint(phi * 4294967296.0) + 512u;
    f.ax = (float)h.ax;
    f.ay = (float)h.ay;
    f.az = (float)h.az;
    f.pad = 0.f;
    a.kb32[r] = f;
}

// The structure factor's reduction.  Per k record r: rho = sum over the
// system's chunks of the partials (fixed order), the per-k energy
// 1/2 w |rho|^2, and rho written into the records.  The energies follow in
// k_kinetic, after the near part.  Nothing here waits for the near part.  (A last-block finish inside
// the reduction would need a device-scope fence in every block, a writeback
// of the XCD's L2 each: 0.3 ms for the 6,400 blocks of a 256-system batch.)
// The reduction also moves the thermostat's noise counter on: the kernel that
// drew this step's noise ran before it, the one that draws the next step's (the
// far kernel, or the next kick/drift) runs after it.  Called by one block.
__device__ __forceinline__ void advance_noise(const EvalArgs &a) {
    if (a.advance && a.kick && a.thermo && threadIdx.x == 0) *a.tstep += 1;
}

// Record r of the batch by one wave.
__device__ __forceinline__ void reduce_record(const EvalArgs &a, int64_t r) {
    const int lane = threadIdx.x & 63;
    const int32_t sys = a.ksys[r];
    const SysDev &sd = a.sys[sys];
    const int32_t k = (int32_t)(r - sd.k0);
    const double2 *pk = reinterpret_cast<const double2 *>(a.partial) + sd.pofs + (int64_t)k * sd.nch;
    const int32_t nch = sd.nch;
    const KVec kv = batch_vector(a, sd, sys, k);
    // four independent loads in flight per lane, summed in a fixed order
    double2 v0 = make_double2(0.0, 0.0), v1 = v0, v2 = v0, v3 = v0;
    int32_t c = lane;
    for (; c + 192 < nch; c += 256) {
        const double2 a0 = pk[c], a1 = pk[c + 64], a2 = pk[c + 128], a3 = pk[c + 192];
        v0.x += a0.x; v0.y += a0.y; v1.x += a1.x; v1.y += a1.y;
        v2.x += a2.x; v2.y += a2.y; v3.x += a3.x; v3.y += a3.y;
    }
    for (; c < nch; c += 64) {
        const double2 a0 = pk[c];
        v0.x += a0.x; v0.y += a0.y;
    }
    double re = (v0.x + v1.x) + (v2.x + v3.x), im = (v0.y + v1.y) + (v2.y + v3.y);
    re = record_sum(re);
    im = record_sum(im);
    if (lane == 0) write_record(a, sd, r, kv, re, im);
}

}  // namespace rbsog
