// Fourier part of the random batch sum-of-Gaussians method for gfx950
// (Sec. 3.1 eq. "fourtrans"; Sec. 3.3 eq. "approximateForce"):
//   rho(k_e) = sum_j q_j e^{i k_e.r_j}
//   F*_i     = -q_i sum_e w_e k_e (Im rho_e cos th_ie - Re rho_e sin th_ie),  th_ie = k_e.r_i
//   U*       = 1/2 sum_e w_e |rho_e|^2
// Phases are taken in revolutions of the fractional coordinate, th/(2 pi) =
// m.s with s = x/L: FP64 forms evaluate kTurnTab t = m.(kTurnTab s) in FP64
// and sin/cos of 2 pi t through a table of 1024 turns in LDS and short
// polynomials of the rest;
// FP32 forms take m.u mod 2^32 exactly on the 32-bit fixed-point coordinate
// and the hardware sin/cos of the revolution.
//
// Work split: the structure factor puts one wave vector on each lane and
// streams particles uniformly through the wave (no cross-lane reduction in
// the inner loop); the force puts one particle on each lane and streams the
// P wave-vector records uniformly.  Both walk lists of work items, each item
// within one system of the batch.  Partial sums of rho are reduced in a
// fixed order, so the result is identical from run to run.
#include "rbsog_internal.h"
#include "rbsog_math.h"
#include "rho_block.h"
#include "rho_reduce.h"

namespace rbsog {

namespace {


// k records are read-only within the kernels that stream them: reading them
// through the constant address space makes the uniform reads scalar loads
typedef const KRec64 __attribute__((address_space(4))) CRec64;
typedef const KRec32 __attribute__((address_space(4))) CRec32;
// whole records (one scalar load each)
__device__ __forceinline__ KRec64 ld(CRec64 *p) {
    KRec64 r;
    r.mx = p->mx; r.my = p->my; r.mz = p->mz;
    r.phi = p->phi;
    r.ax = p->ax; r.ay = p->ay; r.az = p->az;
    r.pad = p->pad;
    return r;
}
// the far sum's part of a record: -m and a (one 24-byte load)
struct KFar32 {
    uint32_t nmx, nmy, nmz;
    float ax, ay, az;
};
__device__ __forceinline__ KFar32 ld(CRec32 *p) {
    typedef const unsigned long long __attribute__((address_space(4))) CU64;
    const unsigned long long w0 = ((CU64 *)p)[0], w1 = ((CU64 *)p)[1], w2 = ((CU64 *)p)[2];
    KFar32 r;
    r.nmx = (uint32_t)w0; r.nmy = (uint32_t)(w0 >> 32);
    r.nmz = (uint32_t)w1; r.ax = __uint_as_float((uint32_t)(w1 >> 32));
    r.ay = __uint_as_float((uint32_t)w2); r.az = __uint_as_float((uint32_t)(w2 >> 32));
    return r;
}

template <bool F64>
__global__ __launch_bounds__(1024, 8) void k_rho(EvalArgs a, const RhoItem *__restrict__ items, int32_t nitems) {
    rho_items<F64>(a, items, nitems, (int32_t)blockIdx.x, (int32_t)gridDim.x);
}

// k_rho_reduce: one wave per record, four records per block (systems of few
// chunks, many of them in a batch).
__global__ __launch_bounds__(256) void k_rho_reduce(EvalArgs a) {
    const int64_t r = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (blockIdx.x == 0) advance_noise(a);
    if (r < a.K) reduce_record(a, r);
}

// k_rho_reduce_block: one block per record (systems of many chunks): each
// thread a fixed strided subset of the chunks with eight loads in flight,
// then a fixed butterfly across each wave and the four waves in order.
__global__ __launch_bounds__(256) void k_rho_reduce_block(EvalArgs a) {
    __shared__ double2 red[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t r = blockIdx.x;
    if (blockIdx.x == 0) advance_noise(a);
    const int32_t sys = a.ksys[r];
    const SysDev &sd = a.sys[sys];
    const int32_t k = (int32_t)(r - sd.k0);
    const double2 *pk = reinterpret_cast<const double2 *>(a.partial) + sd.pofs + (int64_t)k * sd.nch;
    const int32_t nch = sd.nch;
    const KVec kv = batch_vector(a, sd, sys, k);
    double2 v[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) v[h] = make_double2(0.0, 0.0);
    int32_t c = threadIdx.x;
    for (; c + 7 * 256 < nch; c += 8 * 256) {
        double2 w[8];
#pragma unroll
        for (int h = 0; h < 8; ++h) w[h] = pk[c + h * 256];
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            v[h].x += w[h].x;
            v[h].y += w[h].y;
        }
    }
    for (; c < nch; c += 256) {
        const double2 w = pk[c];
        v[0].x += w.x;
        v[0].y += w.y;
    }
    double re = ((v[0].x + v[1].x) + (v[2].x + v[3].x)) + ((v[4].x + v[5].x) + (v[6].x + v[7].x));
    double im = ((v[0].y + v[1].y) + (v[2].y + v[3].y)) + ((v[4].y + v[5].y) + (v[6].y + v[7].y));
    re = record_sum(re);
    im = record_sum(im);
    if (lane == 0) red[wave] = make_double2(re, im);
    __syncthreads();
    if (threadIdx.x == 0) {
        re = (red[0].x + red[1].x) + (red[2].x + red[3].x);
        im = (red[0].y + red[1].y) + (red[2].y + red[3].y);
        write_record(a, sd, r, kv, re, im);
    }
}

// Batches with a zero-frequency mode term: per system, one block, the dipole
// from the chunks' partials (strided sums, then a fixed tree).  A kernel of its
// own: the chunks' writes are visible to it without fences.
__global__ __launch_bounds__(256) void k_dipole(EvalArgs a) {
    __shared__ double si[3][256];
    const int32_t s = blockIdx.x;
    const SysDev &sd = a.sys[s];
    if (sd.zmode == 0) return;
    double m[3] = {0.0, 0.0, 0.0};
    for (int32_t ch = threadIdx.x; ch < sd.nch; ch += 256)
        for (int d = 0; d < 3; ++d) m[d] += a.dip_part[3 * (sd.choff + ch) + d];
    for (int d = 0; d < 3; ++d) si[d][threadIdx.x] = m[d];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int d = 0; d < 3; ++d) si[d][threadIdx.x] += si[d][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x < 3) a.dipole[3 * s + threadIdx.x] = si[threadIdx.x][0];
}

// The last kernel of an evaluation (nothing in it or after it reads the
// batch's place in the sequence): every system's sequence cursor moved on by P.
__device__ __forceinline__ void advance_cursors(const EvalArgs &a) {
    if (!a.advance || blockIdx.x != 0) return;
    for (int32_t s = threadIdx.x; s < a.nsys; s += blockDim.x) a.kcur[s] += a.sys[s].P;
}

// Records whose phases a wave stages at once in the FP32C far sum.
constexpr int kFarStage = 256;
// s_waitcnt lgkmcnt(0) with the other counters left alone (gfx9 encoding)
constexpr int kWaitLgkm0 = 0xC07F;

// Far force on particle i (the factor -q_i included) from `P` amplitude-phase
// records of its system, streamed as uniform loads: one sine per record,
// F_i = -q_i sum_e a_e sin(2 pi (phi_e - m_e.s_i)).  Positions and charges
// from (u, qf) in FP32C (the phase phi - m.u mod 2^32), (x, q) in FP64.
template <bool F64>
__device__ __forceinline__ void far_sum(CSys *sp, CRec64 *kb64, CRec32 *kb32, int32_t P, int64_t n, int64_t i,
                                        const uint32_t *__restrict__ u, const float *__restrict__ qf,
                                        const double *__restrict__ x, const double *__restrict__ q,
                                        const double2 *turn, uint64_t *phs, double &Fx, double &Fy, double &Fz) {
    Fx = 0.0; Fy = 0.0; Fz = 0.0;
    // records are consumed in groups so that their uniform loads overlap
    if constexpr (F64) {
        // fractional coordinates in table units, as the records' phase
        constexpr double tu = rmath::kTurnTab;
        const double sx = x[i] * (sp->g.invL[0] * tu), sy = x[n + i] * (sp->g.invL[1] * tu),
                     sz = x[2 * n + i] * (sp->g.invL[2] * tu);
        constexpr int G = 4;
        int32_t e = 0;
        for (; e + G <= P; e += G) {
            KRec64 r[G];
#pragma unroll
            for (int h = 0; h < G; ++h) r[h] = ld(kb64 + e + h);
#pragma unroll
            for (int h = 0; h < G; ++h) {
                const double t = fma(-r[h].mx, sx, fma(-r[h].my, sy, fma(-r[h].mz, sz, r[h].phi)));
                double v, cv;
                rmath::sincos2pi_tab(t, turn, &v, &cv);
                Fx = fma(r[h].ax, v, Fx);
                Fy = fma(r[h].ay, v, Fy);
                Fz = fma(r[h].az, v, Fz);
            }
        }
        for (; e < P; ++e) {
            const KRec64 r = ld(kb64 + e);
            const double t = fma(-r.mx, sx, fma(-r.my, sy, fma(-r.mz, sz, r.phi)));
            double v, cv;
            rmath::sincos2pi_tab(t, turn, &v, &cv);
            Fx = fma(r.ax, v, Fx);
            Fy = fma(r.ay, v, Fy);
            Fz = fma(r.az, v, Fz);
        }
        const double qi = q[i];
        Fx *= -qi; Fy *= -qi; Fz *= -qi;
    } else {
        const uint32_t ux = u[i], uy = u[n + i], uz = u[2 * n + i];
        // per stage of up to 256 records: each lane copies four records'
        // phases into the wave's LDS slots, from where they are read back
        // broadcast as the addends of the phase chains (phi + (-m).u = phi -
        // m.u mod 2^32, the records holding -m: the subtraction costs no
        // vector instruction).  The next stage's phases are loaded while the
        // current one is summed.  FP32 partial sums over runs of 64 records,
        // accumulated in FP64.
        const KRec32 *kg = (const KRec32 *)kb32;
        const int lane = threadIdx.x & 63;
        constexpr int G = 4;
        auto rec = [&](const KFar32 &r, uint64_t c, float &fx, float &fy, float &fz) {
            const uint32_t t = rmath::dot3_add_mod32_s(r.nmx, r.nmy, r.nmz, ux, uy, uz, c);
            const float v = __builtin_amdgcn_sinf(rmath::phase_rev(t));
            fx = fmaf(r.ax, v, fx);
            fy = fmaf(r.ay, v, fy);
            fz = fmaf(r.az, v, fz);
        };
        uint32_t nxt[kFarStage / 64];
        auto fetch = [&](int32_t e0) {
#pragma unroll
            for (int h = 0; h < kFarStage / 64; ++h) {
                const int32_t e = e0 + 64 * h + lane;
                nxt[h] = kg[e < P ? e : 0].phi;
            }
        };
        fetch(0);
        for (int32_t e0 = 0; e0 < P; e0 += kFarStage) {
            wave_sync();  // the previous stage's broadcast reads are done
#pragma unroll
            for (int h = 0; h < kFarStage / 64; ++h) phs[64 * h + lane] = (uint64_t)nxt[h];
            wave_sync();
            if (e0 + kFarStage < P) fetch(e0 + kFarStage);
            const int32_t e1 = P - e0 < kFarStage ? P : e0 + kFarStage;
            for (int32_t e = e0; e < e1; e += 64) {
                const int cnt = e1 - e < 64 ? e1 - e : 64;
                const uint64_t *ph = phs + (e - e0);
                float fx = 0.f, fy = 0.f, fz = 0.f;
                if (cnt == 64) {
                    // scalar loads and LDS reads share one wait counter, and
                    // a wait on it covers every scalar load in flight: the
                    // group's phases are read and waited for before the next
                    // group's records are requested, which then arrive while
                    // the group is summed
                    KFar32 r[G];
#pragma unroll
                    for (int h = 0; h < G; ++h) r[h] = ld(kb32 + e + h);
#pragma unroll
                    for (int h4 = 0; h4 < 64; h4 += G) {
                        const ulonglong2 w0 = *(const ulonglong2 *)(ph + h4), w1 = *(const ulonglong2 *)(ph + h4 + 2);
                        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                        __builtin_amdgcn_sched_barrier(0);
                        KFar32 rn[G];
                        if (h4 + G < 64) {
#pragma unroll
                            for (int h = 0; h < G; ++h) rn[h] = ld(kb32 + e + h4 + G + h);
                        }
                        rec(r[0], w0.x, fx, fy, fz);
                        rec(r[1], w0.y, fx, fy, fz);
                        rec(r[2], w1.x, fx, fy, fz);
                        rec(r[3], w1.y, fx, fy, fz);
                        if (h4 + G < 64) {
#pragma unroll
                            for (int h = 0; h < G; ++h) r[h] = rn[h];
                        }
                    }
                } else {
                    // a short run: the same, group by group, with the rest
                    // of up to three records one by one
                    const int full = cnt & ~(G - 1);
                    KFar32 r[G];
                    if (full) {
#pragma unroll
                        for (int h = 0; h < G; ++h) r[h] = ld(kb32 + e + h);
                    }
                    for (int h4 = 0; h4 < full; h4 += G) {
                        const ulonglong2 w0 = *(const ulonglong2 *)(ph + h4), w1 = *(const ulonglong2 *)(ph + h4 + 2);
                        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                        __builtin_amdgcn_sched_barrier(0);
                        const int nx = h4 + G < full ? h4 + G : h4;
                        KFar32 rn[G];
#pragma unroll
                        for (int h = 0; h < G; ++h) rn[h] = ld(kb32 + e + nx + h);
                        rec(r[0], w0.x, fx, fy, fz);
                        rec(r[1], w0.y, fx, fy, fz);
                        rec(r[2], w1.x, fx, fy, fz);
                        rec(r[3], w1.y, fx, fy, fz);
#pragma unroll
                        for (int h = 0; h < G; ++h) r[h] = rn[h];
                    }
                    for (int h = full; h < cnt; ++h) rec(ld(kb32 + e + h), ph[h], fx, fy, fz);
                }
                Fx += fx; Fy += fy; Fz += fz;
            }
        }
        const double qi = -(double)qf[i];
        Fx *= qi; Fy *= qi; Fz *= qi;
    }
}

// The end of an evaluation for slot i (current order) given its far force:
// the zero-frequency mode term, the far force stored, the closing half kick
// (and the second Nose-Hoover scaling) when stepping, and the kinetic energy
// of each wave's particles summed across the wave in a fixed order into
// partial `part` (k_kinetic adds them up).  FUSE: the next step
// starts here, as the kick/drift kernel would start it: its opening half kick
// with the same force, its drift (Langevin: with the noise xi between two half
// drifts), wrap and quantisation, and its displacement check.  Lanes past the item (valid false) hold slot i = t0 and
// store nothing.
constexpr int kFusePlain = 1, kFuseLangevin = 2;
template <int FUSE>
struct FarEnd {
    // loaded before the far force is stored (the stores could alias them for
    // the compiler), or before the far sum
    double vv[3], fn[3], xs[FUSE ? 3 : 1];
    uint32_t uref[FUSE ? 3 : 1];
    int32_t id;
};
template <int FUSE>
__device__ __forceinline__ FarEnd<FUSE> far_operands(const EvalArgs &a, int64_t i) {
    const int64_t n = a.N;
    FarEnd<FUSE> o;
    if constexpr (FUSE == kFuseLangevin) o.id = a.cur.id[i];
    for (int d = 0; d < 3; ++d) {
        o.vv[d] = a.cur.v[d * n + i];
        o.fn[d] = a.Fn[d * n + i];
        if constexpr (FUSE) {
            o.xs[d] = a.cur.x[d * n + i];
            o.uref[d] = a.u[d * n + i];
        }
    }
    return o;
}
template <int FUSE>
__device__ __forceinline__ void far_finish(const EvalArgs &a, CSys *sp, int32_t sys, int64_t i, bool valid,
                                           double Fx, double Fy, double Fz, int32_t part, const FarEnd<FUSE> &o,
                                           const double *xi = nullptr) {
    const int64_t n = a.N;
    double vv[3] = {o.vv[0], o.vv[1], o.vv[2]};
    const double *fn = o.fn;
    if (sp->zmode != 0) {
        const double qi = a.cur.q[i], c = sp->zf * qi;
        const double *M = a.dipole + 3 * sys;
        if (sp->zmode == 1) {
            Fx += c * M[0];
            Fy += c * M[1];
        }
        Fz += c * M[2];
    }
    if (valid) {
        a.Ff[i] = Fx;
        a.Ff[n + i] = Fy;
        a.Ff[2 * n + i] = Fz;
    }
    const double f[3] = {fn[0] + Fx, fn[1] + Fy, fn[2] + Fz};
    if (a.kick) {
        // closing half kick of the velocity-Verlet step
        bool bad = false;
        for (int d = 0; d < 3; ++d) {
            bad |= !isfinite(f[d]);
            vv[d] += a.hdm * f[d];
        }
        if (!FUSE && a.nh) {
            // Nose-Hoover: the second scaling with the step's half-step xi
            // (xi and the kinetic energy still hold the step's start)
            const double xh = a.nh_xi[sys] + 0.5 * a.dt * (2.0 * a.kin[sys] - sp->nh_nf * a.nh_T) / sp->nh_Q;
            const double sc = exp(-0.5 * a.dt * xh);
            for (int d = 0; d < 3; ++d) vv[d] *= sc;
        }
        if (!FUSE && valid)
            for (int d = 0; d < 3; ++d) a.cur.v[d * n + i] = vv[d];
        if (bad && valid) atomicOr(a.flag, 1);
    }
    double ke = valid ? 0.5 * a.mass * ((vv[0] * vv[0] + vv[1] * vv[1]) + vv[2] * vv[2]) : 0.0;
    // the wave's kinetic energy (a fixed butterfly), one partial per wave
    for (int o = 32; o > 0; o >>= 1) ke += __shfl_xor(ke, o, 64);
    if ((threadIdx.x & 63) == 0) a.kpart[part] = ke;
    if constexpr (FUSE) {
        // the next step: half kick and drift, the drift kept for the
        // mean-square displacement, then wrap and quantise
        const double xs0[3] = {o.xs[0], o.xs[1], o.xs[2]};
        double xs[3] = {o.xs[0], o.xs[1], o.xs[2]}, L[3];
        float hf[3];
        for (int d = 0; d < 3; ++d) {
            L[d] = sp->g.L[d];
            hf[d] = sp->g.hf[d];
        }
        for (int d = 0; d < 3; ++d) {
            vv[d] += a.hdm * f[d];
            if constexpr (FUSE == kFuseLangevin) {
                // half drift, Ornstein-Uhlenbeck, half drift
                xs[d] += 0.5 * a.dt * vv[d];
                vv[d] = fma(a.c1, vv[d], a.c2 * xi[d]);
                xs[d] += 0.5 * a.dt * vv[d];
            } else {
                xs[d] += a.dt * vv[d];
            }
            if (valid) a.cur.v[d * n + i] = vv[d];
        }
        if (valid && a.cur.dsp)
            for (int d = 0; d < 3; ++d) a.cur.dsp[d * n + i] += xs[d] - xs0[d];
        uint32_t uq[3];
        const float d2 = wrap_store(a, i, valid, xs, L, hf, o.uref, uq);
        // one atomic per wave that found a particle past the threshold
        const bool far_ = valid && !(d2 <= sp->g.dthr2_f);
        if (__ballot(far_) != 0ull && (threadIdx.x & 63) == 0) atomicOr(a.rebuild, 1);
    }
}

// Far force and the end of the evaluation, one particle per lane; items are
// runs of up to 256 slots of one system, in groups of 64.  W = 1: a block per
// item, a wave per group.  W > 1: a block per group, whose W waves share the
// records (in order; the partial forces meet in LDS, added in wave order) and
// whose first wave ends the evaluation, its operands requested before the sum:
// for systems with too few groups to fill the device.
// The near-list rebuild flag is cleared here (every kernel of the evaluation
// that reads it has run), unless the kernel opens the next step (FUSE), whose
// displacement check sets it: the list pass has cleared it then.
template <bool F64, int FUSE, int W>
__global__ __launch_bounds__(W == 1 ? 256 : 64 * W) void k_far(EvalArgs a, const FarItem *__restrict__ items, int32_t nitems,
                                                               int32_t groups) {
    constexpr int kWaves = W == 1 ? 4 : W;
    __shared__ double2 turn[F64 ? rmath::kTurnTab : 1];
    __shared__ uint64_t phs[F64 ? 1 : kWaves * kFarStage];  // FP32C: record phases, per wave
    __shared__ double part[W == 1 ? 1 : W][3][W == 1 ? 1 : 64];
    __shared__ double noise[W > 1 && FUSE == kFuseLangevin ? 3 : 1][W > 1 && FUSE == kFuseLangevin ? 64 : 1];
    if constexpr (F64) fill_turns(turn);
    if (!FUSE && blockIdx.x == 0 && threadIdx.x == 0 && a.rebuild) *a.rebuild = 0;
    advance_cursors(a);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    // W = 1: item = block, group = wave; W > 1: `groups` groups per item
    const int32_t itx = W == 1 ? (int32_t)blockIdx.x : (int32_t)blockIdx.x / groups;
    const int32_t grp = W == 1 ? wave : (int32_t)blockIdx.x % groups;
    if (itx >= nitems) return;
    const FarItem item = items[itx];
    const int32_t sys = rfl(item.sys);
    CSys *sp = (CSys *)(a.sys + sys);
    const int64_t t0 = rfl64(item.t0), t1 = rfl64(item.t1);
    const int64_t i0 = t0 + 64 * grp + lane;
    const bool valid = i0 < t1;
    const int64_t i = valid ? i0 : t0;
    uint64_t *ph = phs + (F64 ? 0 : wave * kFarStage);
    double Fx, Fy, Fz;
    if constexpr (W == 1) {
        far_sum<F64>(sp, (CRec64 *)(a.kb64 + sp->k0), (CRec32 *)(a.kb32 + sp->k0), sp->P, a.N, i, a.u_tmp,
                     a.cur.qf, a.cur.x, a.cur.q, turn, ph, Fx, Fy, Fz);
        const FarEnd<FUSE> o = far_operands<FUSE>(a, i);
        double xi[3];
        if constexpr (FUSE == kFuseLangevin) rmath::thermo_normals(a.tseed, *a.tstep, o.id, xi);
        far_finish<FUSE>(a, sp, sys, i, valid, Fx, Fy, Fz, itx * 4 + grp, o, xi);
    } else {
        FarEnd<FUSE> o;
        if (wave == 0) o = far_operands<FUSE>(a, i);
        // the wave's share of the records, in groups of four
        const int32_t P = sp->P, per = ((P + 4 * W - 1) / (4 * W)) * 4;
        const int32_t e0 = wave * per < P ? wave * per : P, cnt = P - e0 < per ? P - e0 : per;
        Fx = Fy = Fz = 0.0;
        if (cnt > 0)
            far_sum<F64>(sp, (CRec64 *)(a.kb64 + sp->k0 + e0), (CRec32 *)(a.kb32 + sp->k0 + e0), cnt, a.N, i, a.u_tmp,
                         a.cur.qf, a.cur.x, a.cur.q, turn, ph, Fx, Fy, Fz);
        part[wave][0][lane] = Fx;
        part[wave][1][lane] = Fy;
        part[wave][2][lane] = Fz;
        if constexpr (FUSE == kFuseLangevin) {
            // the last wave, whose share of the records is the smallest, draws the noise
            if (wave == W - 1) {
                double xi[3];
                rmath::thermo_normals(a.tseed, *a.tstep, a.cur.id[i], xi);
                for (int d = 0; d < 3; ++d) noise[d][lane] = xi[d];
            }
        }
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int w = 1; w < W; ++w) {
            Fx += part[w][0][lane];
            Fy += part[w][1][lane];
            Fz += part[w][2][lane];
        }
        double xi[3];
        if constexpr (FUSE == kFuseLangevin)
            for (int d = 0; d < 3; ++d) xi[d] = noise[d][lane];
        far_finish<FUSE>(a, sp, sys, i, valid, Fx, Fy, Fz, itx * 4 + grp, o, xi);
    }
}

// Build-every-step mode: the far force computed beside the re-sort and the
// near part, on the structure factor's stream, from the copy of the state
// that the kick/drift kernel wrote (its order: the slots before the re-sort),
// into Ff_side.
template <bool F64>
__global__ __launch_bounds__(256) void k_far_side(EvalArgs a, const FarItem *__restrict__ items, int32_t nitems) {
    __shared__ double2 turn[F64 ? rmath::kTurnTab : 1];
    __shared__ uint64_t phs[F64 ? 1 : 4 * kFarStage];  // FP32C: record phases, per wave
    if constexpr (F64) fill_turns(turn);
    const int64_t n = a.N;
    for (int32_t itx = blockIdx.x; itx < nitems; itx += gridDim.x) {
        const FarItem item = items[itx];
        CSys *sp = (CSys *)(a.sys + rfl(item.sys));
        const int64_t t0 = rfl64(item.t0), t1 = rfl64(item.t1);
        const int64_t i0 = t0 + threadIdx.x;
        const bool valid = i0 < t1;
        const int64_t i = valid ? i0 : t0;
        double Fx, Fy, Fz;
        far_sum<F64>(sp, (CRec64 *)(a.kb64 + sp->k0), (CRec32 *)(a.kb32 + sp->k0), sp->P, n, i, a.rs_u, a.rs_qf,
                     a.rs_x, a.rs_q, turn, phs + (F64 ? 0 : (threadIdx.x >> 6) * kFarStage), Fx, Fy, Fz);
        if (valid) {
            a.Ff_side[i] = Fx;
            a.Ff_side[n + i] = Fy;
            a.Ff_side[2 * n + i] = Fz;
        }
    }
}

// Build-every-step mode, after the near part: slot i of the new order takes
// the far force of its particle's slot before the re-sort (`sorted`, which
// the re-sort writes at every evaluation of this mode), then the end of the
// evaluation as in k_far.  Clears the rebuild flag.
__global__ __launch_bounds__(256) void k_far_finish(EvalArgs a, const FarItem *__restrict__ items, int32_t nitems) {
    const int64_t n = a.N;
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.rebuild) *a.rebuild = 0;
    advance_cursors(a);
    for (int32_t itx = blockIdx.x; itx < nitems; itx += gridDim.x) {
        const FarItem item = items[itx];
        const int32_t sys = rfl(item.sys);
        CSys *sp = (CSys *)(a.sys + sys);
        const int64_t t0 = rfl64(item.t0), t1 = rfl64(item.t1);
        const int64_t i0 = t0 + threadIdx.x;
        const bool valid = i0 < t1;
        const int64_t i = valid ? i0 : t0;
        const int64_t o = a.sorted[i];
        const double Fx = a.Ff_side[o], Fy = a.Ff_side[n + o], Fz = a.Ff_side[2 * n + o];
        far_finish<0>(a, sp, sys, i, valid, Fx, Fy, Fz, itx * 4 + (int32_t)(threadIdx.x >> 6),
                          far_operands<0>(a, i));
    }
}

// Per system, gridDim.x blocks: each sums a contiguous share of the far
// items' wave partials of the kinetic energy and of the near items' energy
// partials of the mode in use (eight loads in flight per thread, a fixed
// tree across the block), the first one also the far energies of the records;
// with one block it finishes alone, else the last
// block of the system (per-system counter, re-armed) adds the blocks' sums in
// block order.  The finish: U_N and the total U = U_N + U* - U_self, the
// kinetic energy after the evaluation, and for a Nose-Hoover step xi's
// second half step with it.
__global__ __launch_bounds__(256) void k_kinetic(EvalArgs a) {
    __shared__ double kw[256], ew[256], uw[256];
    const int32_t s = blockIdx.y, g = blockIdx.x, G = gridDim.x;
    const SysDev &sp = a.sys[s];
    // the block's share [lo, hi) of the partials [b0, b1)
    auto share = [&](int64_t b0, int64_t b1, int64_t &lo, int64_t &hi) {
        const int64_t per = (b1 - b0 + G - 1) / G;
        lo = b0 + (int64_t)g * per;
        hi = lo + per < b1 ? lo + per : b1;
        if (lo > hi) lo = hi;
    };
    auto sum8 = [&](const double *p, int64_t lo, int64_t hi) {
        double u8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        int64_t i = lo + threadIdx.x;
        for (; i + 7 * 256 < hi; i += 8 * 256) {
#pragma unroll
            for (int h = 0; h < 8; ++h) u8[h] += p[i + h * 256];
        }
        for (; i < hi; i += 256) u8[0] += p[i];
        return ((u8[0] + u8[1]) + (u8[2] + u8[3])) + ((u8[4] + u8[5]) + (u8[6] + u8[7]));
    };
    int64_t lo, hi;
    share((int64_t)sp.ft0 * 4, (int64_t)sp.ft1 * 4, lo, hi);
    kw[threadIdx.x] = sum8(a.kpart, lo, hi);
    const double *ep = a.always_build ? a.epart_cells : a.epart;
    share(a.always_build ? sp.jt0 : sp.it0, a.always_build ? sp.jt1 : sp.it1, lo, hi);
    ew[threadIdx.x] = sum8(ep, lo, hi);
    // the far energy of the system, summed by its first block
    double us = 0.0;
    if (g == 0)
        for (int32_t e = threadIdx.x; e < sp.P; e += 256) us += a.ek[sp.k0 + e];
    uw[threadIdx.x] = us;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            kw[threadIdx.x] += kw[threadIdx.x + o];
            ew[threadIdx.x] += ew[threadIdx.x + o];
            uw[threadIdx.x] += uw[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    double K = kw[0], un = ew[0];
    if (g == 0) {
        // U* holds the far part with the zero-frequency mode term
        double u0 = 0.0;
        if (sp.zmode != 0) {
            const double M[3] = {a.dipole[3 * s], a.dipole[3 * s + 1], a.dipole[3 * s + 2]};
            u0 = sp.zmode == 1 ? sp.zu * (M[0] * M[0] + M[1] * M[1] + M[2] * M[2]) : sp.zu * M[2] * M[2];
        }
        a.E[4 * s + 1] = uw[0] + u0;
        a.E[4 * s + 2] = sp.uself;
    }
    if (G > 1) {
        double *part = a.kin_part + (int64_t)s * 2 * G;
        part[2 * g] = K;
        part[2 * g + 1] = un;
        __threadfence();
        if (atomicAdd(&a.sys_done[s], 1u) != (uint32_t)G - 1u) return;
        __threadfence();
        K = 0.0;
        un = 0.0;
        for (int32_t b = 0; b < G; ++b) {
            K += part[2 * b];
            un += part[2 * b + 1];
        }
        a.sys_done[s] = 0u;
    }
    const double tot = un + a.E[4 * s + 1] - a.E[4 * s + 2];
    a.E[4 * s] = un;
    a.E[4 * s + 3] = tot;
    if (!isfinite(tot)) atomicOr(a.flag, 2);
    if (a.kick && a.nh) {
        const double nf = sp.nh_nf, Q = sp.nh_Q;
        const double xh = a.nh_xi[s] + 0.5 * a.dt * (2.0 * a.kin[s] - nf * a.nh_T) / Q;
        a.nh_xi[s] = xh + 0.5 * a.dt * (2.0 * K - nf * a.nh_T) / Q;
    }
    a.kin[s] = K;
}


// One block per system: sum of |dsp|^2 over its slots (strided, then a fixed
// tree), divided by n.
__global__ __launch_bounds__(256) void k_msd(EvalArgs a, double *__restrict__ msd) {
    __shared__ double w[256];
    const int32_t s = blockIdx.x;
    const SysDev &sp = a.sys[s];
    const int64_t n = a.N, p0 = sp.p0, p1 = sp.p0 + sp.g.n;
    double acc = 0.0;
    for (int64_t i = p0 + threadIdx.x; i < p1; i += 256) {
        const double dx = a.cur.dsp[i], dy = a.cur.dsp[n + i], dz = a.cur.dsp[2 * n + i];
        acc += (dx * dx + dy * dy) + dz * dz;
    }
    w[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) w[threadIdx.x] += w[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) msd[s] = w[0] / (double)sp.g.n;
}

}  // namespace

void launch_msd(const EvalArgs &a, double *msd, hipStream_t s) {
    hipLaunchKernelGGL(k_msd, dim3((unsigned)a.nsys), dim3(256), 0, s, a, msd);
}

void launch_rho(const EvalArgs &a, bool f64, const RhoItem *items, int32_t nitems, hipStream_t s) {
    dim3 grid((unsigned)nitems), block(1024);
    if (f64) hipLaunchKernelGGL(k_rho<true>, grid, block, 0, s, a, items, nitems);
    else hipLaunchKernelGGL(k_rho<false>, grid, block, 0, s, a, items, nitems);
}

void launch_rho_reduce(const EvalArgs &a, hipStream_t s) {
    if (a.K <= 0) return;
    if (a.red_waves == 4) hipLaunchKernelGGL(k_rho_reduce_block, dim3((unsigned)a.K), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_rho_reduce, dim3((unsigned)((a.K + 3) / 4)), dim3(256), 0, s, a);
    launch_dipole(a, s);
}

void launch_dipole(const EvalArgs &a, hipStream_t s) {
    if (a.zmode) hipLaunchKernelGGL(k_dipole, dim3((unsigned)a.nsys), dim3(256), 0, s, a);
}

// Waves per group of 64 particles: as many as keep the launch within 4 (FP32C) or
// 8 (FP64) waves per SIMD and leave each wave a few groups of records.  k_far at
// W = 1 and at the W taken: 1,000 ions x 100 FP32C 10.1 -> 5.8 us (16), FP64 21 ->
// 5.8; 26,998 ions x 130 11.3 -> 7.2 (8; 16: 9.4); 77,781 x 150 13.2 -> 10.5 (2);
// 98,304 x 211 FP64 40.7 -> 21.2 (4; 2: 25.8); 300,000 x 200 FP64 54 (2: 62).
// (Counted are the groups that hold particles, two for a system of 66, and no more
// are launched for an item than the fullest one has: 240 systems of 66, 264 groups
// counted and 960 launched | 480 and 480: 56.3 | 48.6 us a step.)
int32_t far_waves(const EvalArgs &a, bool f64) {
    const int64_t per = a.nsys ? a.K / a.nsys : 0;
    int32_t w = 16;
    while (w > 1 && (a.far_groups * w > (f64 ? 8192 : 4096) || per < 4 * w)) w >>= 1;
    return w;
}

template <bool F64, int FUSE>
static void far_split(const EvalArgs &a, const FarItem *items, int32_t nitems, int32_t block_size, hipStream_t s) {
    const int32_t w = far_waves(a, F64), groups = w > 1 ? a.far_span : block_size / 64;
    const dim3 grid((unsigned)(nitems * groups)), block((unsigned)(64 * w));
    switch (w) {
        case 16: hipLaunchKernelGGL((k_far<F64, FUSE, 16>), grid, block, 0, s, a, items, nitems, groups); break;
        case 8: hipLaunchKernelGGL((k_far<F64, FUSE, 8>), grid, block, 0, s, a, items, nitems, groups); break;
        case 4: hipLaunchKernelGGL((k_far<F64, FUSE, 4>), grid, block, 0, s, a, items, nitems, groups); break;
        case 2: hipLaunchKernelGGL((k_far<F64, FUSE, 2>), grid, block, 0, s, a, items, nitems, groups); break;
        default:
            hipLaunchKernelGGL((k_far<F64, FUSE, 1>), dim3((unsigned)nitems), dim3((unsigned)block_size), 0, s, a, items,
                               nitems, groups);
    }
}

void launch_far(const EvalArgs &a, bool f64, const FarItem *items, int32_t nitems, int32_t block_size,
                hipStream_t s) {
    if (a.fuse && a.thermo) {
        if (f64) far_split<true, kFuseLangevin>(a, items, nitems, block_size, s);
        else far_split<false, kFuseLangevin>(a, items, nitems, block_size, s);
    } else if (a.fuse) {
        if (f64) far_split<true, kFusePlain>(a, items, nitems, block_size, s);
        else far_split<false, kFusePlain>(a, items, nitems, block_size, s);
    } else {
        if (f64) far_split<true, 0>(a, items, nitems, block_size, s);
        else far_split<false, 0>(a, items, nitems, block_size, s);
    }
}

void launch_far_side(const EvalArgs &a, bool f64, const FarItem *items, int32_t nitems, int32_t block_size,
                     hipStream_t s) {
    dim3 grid((unsigned)nitems), block((unsigned)block_size);
    if (f64) hipLaunchKernelGGL(k_far_side<true>, grid, block, 0, s, a, items, nitems);
    else hipLaunchKernelGGL(k_far_side<false>, grid, block, 0, s, a, items, nitems);
}

void launch_far_finish(const EvalArgs &a, const FarItem *items, int32_t nitems, int32_t block_size, hipStream_t s) {
    hipLaunchKernelGGL(k_far_finish, dim3((unsigned)nitems), dim3((unsigned)block_size), 0, s, a, items, nitems);
}

void launch_kinetic(const EvalArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_kinetic, dim3((unsigned)a.kin_blocks, (unsigned)a.nsys), dim3(256), 0, s, a);
}

}  // namespace rbsog
