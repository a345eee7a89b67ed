// Stateless structure factor of one set of point charges for gfx950
// (Sec. 3.1: rho(k) = sum_j q_j e^{i k.r_j}, k = 2 pi (m_x/L_x, m_y/L_y,
// m_z/L_z); Sec. 3.4: the one reduction of the random-batch method, which a
// spatially sharded run computes per device and then sums across devices).
// Device inputs and outputs, no context: rbsog_structure_factor takes its
// partial sums in memory it allocates per call (stream ordered), and
// rbsog_structure_factor_noalloc takes them in the file-scope array `scratch`
// below, for callers that cannot allocate (graph capture, serving loops).
// Both run the same kernels with the same chunk plan, so their results are
// bitwise identical.
//
// Work split, as in the batch's structure factor (rho_core.h): a block of 16
// waves owns a chunk of particles and a group of up to 16 k tiles of 64 wave
// vectors (one per lane); the waves beyond the tiles split the chunk into
// streams.  The block wraps, quantises and stages 1024 particles at a time in
// LDS, once for all its tiles.  Bound by vector issue: FP32C sums pairs of
// equal charge (8.5 issue slots per particle and wave vector), FP64 takes its
// sines and cosines from a table of turns (20 slots).  1,999,998 particles x
// 1000 vectors FP32C: 0.62 -> 0.50 ms (0.49 at the issue rate), error against
// FP64 4.7e-7 -> 3.5e-7 with the phases rounded; 10,002 x 100 FP64: 118 -> 7
// us (before: one k tile of 256 a block and a chunk of 1024 particles, so 10
// blocks, each thread one vector, sines by polynomials).
// Each (chunk, k) partial is written once and a second kernel adds the chunks
// of every k in a fixed order; a call of one chunk writes its sums directly.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "rbsog_internal.h"
#include "rbsog_math.h"
#include "rho_core.h"

namespace rbsog {

rbsog_status fail_noctx(rbsog_status st, const char *fmt, ...);

namespace {

constexpr int kSfWaves = 16;          // waves of a block: k tiles x particle streams
constexpr int64_t kSfBlocks = 512;    // blocks of a large call: two on each of the 256 CUs
constexpr int64_t kSfMaxVectors = 65535ll * 256;  // wave vectors of a call
constexpr int64_t kSfMinChunk = 64;   // particles of a chunk at least (one wave's staging)
// Partial sums held by the no-allocation entry point: 2^20 complex FP64
// values (16 MiB per device, held until the process ends).  A call needs
// n_chunks x n_k of them; n_chunks shrinks to fit, so n_k <= 2^20.
constexpr int64_t kScratchComplex = int64_t(1) << 20;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) double2 scratch[kScratchComplex];

// FP32C pairs any two particles of equal charge while every wave vector of the
// block has |m_x| + |m_y| + |m_z| up to this.  Half a pair's difference drops its
// lowest bit, so one of the two stands a unit of 2^-32 of the box beside its place
// and its phase up to |m|_1 units off: with 256 units of rounding (half of the
// 2^-23 turns that the hardware sine takes) no more than the 512 that truncating
// every phase would cost.  Larger vectors pair where the difference is even, and
// no phase is off by more than its rounding.
constexpr uint64_t kPairAnyMax = 256;

// Shape of a call: k tiles and particle streams of a block, groups of k tiles,
// chunks and particles per chunk.
struct SfPlan {
    int32_t kt, streams;
    int64_t groups, nchunk, chunk;
};
SfPlan sf_plan(int64_t n, int64_t nk, bool f64) {
    SfPlan p;
    const int64_t tiles = (nk + 63) / 64;
    p.kt = (int32_t)(tiles < kSfWaves ? tiles : kSfWaves);
    if (tiles > kSfWaves) {
        // several groups: the k tiles of a block that take the least time over all of
        // them.  A group's time goes with the waves that a SIMD runs of it, over its
        // particle streams, and one tile's for the staging of every particle: 17
        // tiles in groups of 16 and 1 take twice the time of 16, in three groups of 6
        // (12 waves in two streams) 1.2 times (1,999,998 particles x 1025 FP32C, us:
        // 1,020 -> 700)
        int64_t best = INT64_MAX;
        for (int32_t kt = kSfWaves; kt >= 4; --kt) {
            const int64_t groups = (tiles + kt - 1) / kt, streams = kSfWaves / kt, waves = kt * streams;
            const int64_t cost = groups * ((waves + 3) / 4 * 4 * kSfWaves / streams + kSfWaves);
            if (cost < best) {
                best = cost;
                p.kt = kt;
            }
        }
    }
    p.streams = kSfWaves / p.kt;
    p.groups = (tiles + p.kt - 1) / p.kt;
    // chunks of at least kSfMinChunk particles that give two blocks per CU
    // over the groups, no more than the partial buffer holds
    int64_t want = kSfBlocks / p.groups;
    if (want > (n + kSfMinChunk - 1) / kSfMinChunk) want = (n + kSfMinChunk - 1) / kSfMinChunk;
    const int64_t fit = kScratchComplex / nk;
    if (want > fit) want = fit;
    // a small call in one chunk: the second kernel costs more (about 5 us)
    // than its particles do in one block (n x tiles x 9 issue cycles in FP32C,
    // x 20 in FP64)
    if (n * p.kt <= (f64 ? 512 : 1024)) want = 1;
    if (want < 1) want = 1;
    p.chunk = (n + want - 1) / want;
    p.nchunk = (n + p.chunk - 1) / p.chunk;
    return p;
}

// Partial structure factor of chunk c = blockIdx.x (particles [c chunk,
// (c+1) chunk)) for the k tiles of group blockIdx.y; the sums themselves into
// rho with one chunk.
template <bool F64>
__global__ __launch_bounds__(1024, F64 ? 1 : 8) void k_sf_partial(int64_t n, const double *__restrict__ x,
                                                                  const double *__restrict__ q, double Lx, double Ly,
                                                                  double Lz, int64_t nk, const int32_t *__restrict__ m,
                                                                  int32_t kt, int32_t streams, int64_t chunk,
                                                                  int64_t nchunk, double2 *__restrict__ partial,
                                                                  double *__restrict__ rho_re,
                                                                  double *__restrict__ rho_im) {
    constexpr double kTwo32 = 4294967296.0;
    __shared__ double2 red[1024];
    __shared__ uint4 st32[F64 ? 1 : kStage];
    __shared__ int2 wcnt[F64 ? 1 : 16];
    __shared__ int32_t large[F64 ? 1 : kSfWaves];  // FP32C: a wave holds a vector above kPairAnyMax
    __shared__ Stage64 st64[F64 ? kStage : 1];
    __shared__ double2 turn[F64 ? rmath::kTurnTab : 1];
    if constexpr (F64) fill_turns(turn);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int kti = wave % kt, st = wave / kt;
    const int64_t k = ((int64_t)blockIdx.y * kt + kti) * 64 + lane;
    const bool kv = k < nk;
    const int32_t mx = kv ? m[3 * k] : 0, my = kv ? m[3 * k + 1] : 0, mz = kv ? m[3 * k + 2] : 0;
    const int64_t c = blockIdx.x;
    const int64_t j0 = c * chunk;
    const int64_t j1 = j0 + chunk < n ? j0 + chunk : n;
    const double L[3] = {Lx, Ly, Lz};
    bool even = false;
    if constexpr (!F64) {
        const uint64_t l1 = (uint64_t)llabs((long long)mx) + llabs((long long)my) + llabs((long long)mz);
        const uint64_t over = __builtin_amdgcn_ballot_w64(l1 > kPairAnyMax);
        if (lane == 0) large[wave] = over != 0 ? 1 : 0;
        __syncthreads();
        even = __builtin_amdgcn_ballot_w64(large[lane & 15] != 0) != 0;
    }
    double re = 0.0, im = 0.0;
    for (int64_t jb = j0; jb < j1; jb += kStage) {
        const int cnt = (int)(j1 - jb < kStage ? j1 - jb : kStage);
        const bool have = (int)threadIdx.x < cnt;
        double s[3] = {0.0, 0.0, 0.0}, qj = 0.0;
        if (have) {
            const int64_t j = jb + threadIdx.x;
            qj = q[j];
            for (int d = 0; d < 3; ++d) {
                const double r = x[3 * j + d] / L[d];
                s[d] = r - floor(r);
            }
        }
        if constexpr (F64) {
            constexpr double tu = rmath::kTurnTab;
            if (have) st64[threadIdx.x] = Stage64{s[0] * tu, s[1] * tu, s[2] * tu, qj};
            __syncthreads();
            if (st < streams) sum_staged64(st64, cnt, turn, mx, my, mz, st, streams, re, im);
        } else {
            // fixed-point rule of the library: u = min(2^32 - 1, floor(frac(x/L) 2^32))
            uint32_t u[3];
            for (int d = 0; d < 3; ++d) {
                double w = floor(s[d] * kTwo32);
                // non-finite positions give 0 instead of an undefined conversion
                w = w >= 0.0 ? (w > kTwo32 - 1.0 ? kTwo32 - 1.0 : w) : 0.0;
                u[d] = (uint32_t)w;
            }
            const int np = stage_pairs<true>(have, u[0], u[1], u[2], __float_as_uint((float)qj), st32, wcnt, even);
            if (st < streams)
                sum_staged32<true>(st32, np, cnt - 2 * np, (uint32_t)mx, (uint32_t)my, (uint32_t)mz, st, streams, re, im);
        }
        __syncthreads();
    }
    // the streams' sums in order
    red[threadIdx.x] = make_double2(re, im);
    __syncthreads();
    if (st != 0 || !kv) return;
    double sr = 0.0, si = 0.0;
    for (int s2 = 0; s2 < streams; ++s2) {
        const double2 v = red[(s2 * kt + kti) * 64 + lane];
        sr += v.x;
        si += v.y;
    }
    if (nchunk == 1) {
        rho_re[k] = sr;
        rho_im[k] = si;
    } else {
        partial[k * nchunk + c] = make_double2(sr, si);
    }
}

// rho_k = sum over the chunks of the partials of k, one wave per k: four
// strided accumulators per lane, then a fixed butterfly across the wave.
__global__ __launch_bounds__(256) void k_sf_reduce(int64_t nk, int64_t nchunk, const double2 *__restrict__ partial,
                                                   double *__restrict__ rho_re, double *__restrict__ rho_im) {
    const int lane = threadIdx.x & 63;
    const int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= nk) return;
    const double2 *pk = partial + k * nchunk;
    double2 v0 = make_double2(0.0, 0.0), v1 = v0, v2 = v0, v3 = v0;
    int64_t c = lane;
    for (; c + 192 < nchunk; c += 256) {
        const double2 a0 = pk[c], a1 = pk[c + 64], a2 = pk[c + 128], a3 = pk[c + 192];
        v0.x += a0.x; v0.y += a0.y; v1.x += a1.x; v1.y += a1.y;
        v2.x += a2.x; v2.y += a2.y; v3.x += a3.x; v3.y += a3.y;
    }
    for (; c < nchunk; c += 64) {
        const double2 a0 = pk[c];
        v0.x += a0.x; v0.y += a0.y;
    }
    double re = (v0.x + v1.x) + (v2.x + v3.x), im = (v0.y + v1.y) + (v2.y + v3.y);
    for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o, 64);
        im += __shfl_xor(im, o, 64);
    }
    if (lane == 0) {
        rho_re[k] = re;
        rho_im[k] = im;
    }
}

rbsog_status sf_check(int64_t n, const double *x, const double *q, const double *box, int64_t nk, const int32_t *m,
                      int32_t precision, const double *rho_re, const double *rho_im, const char *who) {
    if (n < 1 || n > (int64_t)INT32_MAX) return fail_noctx(RBSOG_E_ARG, "%s: n must be in [1, 2^31-1]", who);
    if (nk < 1) return fail_noctx(RBSOG_E_ARG, "%s: n_k must be >= 1", who);
    if (nk > kSfMaxVectors) return fail_noctx(RBSOG_E_ARG, "%s: n_k above %lld", who, (long long)kSfMaxVectors);
    if (!x || !q || !box || !m || !rho_re || !rho_im) return fail_noctx(RBSOG_E_ARG, "%s: null pointer", who);
    for (int d = 0; d < 3; ++d)
        if (!(box[d] > 0.0) || !std::isfinite(box[d]))
            return fail_noctx(RBSOG_E_ARG, "%s: box sides must be finite and > 0", who);
    if (precision != RBSOG_FP64 && precision != RBSOG_FP32C)
        return fail_noctx(RBSOG_E_ARG, "%s: unknown precision %d", who, precision);
    return RBSOG_OK;
}

rbsog_status sf_launch(int64_t n, const double *x, const double *q, const double *box, int64_t nk, const int32_t *m,
                       int32_t precision, double *rho_re, double *rho_im, hipStream_t s, double2 *partial,
                       const SfPlan &p, const char *who) {
    const dim3 grid((unsigned)p.nchunk, (unsigned)p.groups), block(64 * kSfWaves);
    if (precision == RBSOG_FP64)
        hipLaunchKernelGGL(k_sf_partial<true>, grid, block, 0, s, n, x, q, box[0], box[1], box[2], nk, m, p.kt,
                           p.streams, p.chunk, p.nchunk, partial, rho_re, rho_im);
    else
        hipLaunchKernelGGL(k_sf_partial<false>, grid, block, 0, s, n, x, q, box[0], box[1], box[2], nk, m, p.kt,
                           p.streams, p.chunk, p.nchunk, partial, rho_re, rho_im);
    if (p.nchunk > 1)
        hipLaunchKernelGGL(k_sf_reduce, dim3((unsigned)((nk + 3) / 4)), dim3(256), 0, s, nk, p.nchunk,
                           (const double2 *)partial, rho_re, rho_im);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_noctx(RBSOG_E_DEVICE, "%s: launch failed: %s", who, hipGetErrorString(e));
    return RBSOG_OK;
}

// Device address of `scratch` on each device, taken once per device with the
// device current (the array's name is a host-side stand-in in host code).
std::mutex g_scratch_mu;
double2 *g_scratch_ptr[kMaxDevices] = {};

rbsog_status scratch_of_current_device(double2 **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_noctx(RBSOG_E_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail_noctx(RBSOG_E_DEVICE, "device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail_noctx(RBSOG_E_DEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = (double2 *)p;
    }
    *out = g_scratch_ptr[dev];
    return RBSOG_OK;
}

}  // namespace
}  // namespace rbsog

using namespace rbsog;

extern "C" {

rbsog_status rbsog_debug_structure_factor_plan(int64_t n, int64_t n_k, int32_t precision, int64_t *out) {
    const char *who = "rbsog_debug_structure_factor_plan";
    const double box[3] = {1.0, 1.0, 1.0};
    const int32_t m = 1;
    const rbsog_status st = sf_check(n, box, box, box, n_k, &m, precision, box, box, who);
    if (st != RBSOG_OK) return st;
    if (!out) return fail_noctx(RBSOG_E_ARG, "%s: out is null", who);
    const SfPlan p = sf_plan(n, n_k, precision == RBSOG_FP64);
    out[0] = p.kt;
    out[1] = p.streams;
    out[2] = p.groups;
    out[3] = p.nchunk;
    return RBSOG_OK;
}

rbsog_status rbsog_structure_factor(int64_t n, const double *x, const double *q, const double *box, int64_t n_k,
                                    const int32_t *m, int32_t precision, double *rho_re, double *rho_im,
                                    void *stream) {
    const char *who = "rbsog_structure_factor";
    rbsog_status st = sf_check(n, x, q, box, n_k, m, precision, rho_re, rho_im, who);
    if (st != RBSOG_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const SfPlan p = sf_plan(n, n_k, precision == RBSOG_FP64);
    void *part = nullptr;
    hipError_t e = hipSuccess;
    if (p.nchunk > 1) {
        e = hipMallocAsync(&part, (size_t)(p.nchunk * n_k) * sizeof(double2), s);
        if (e != hipSuccess)
            return fail_noctx(RBSOG_E_OOM, "%s: %lld partial sums: %s", who, (long long)(p.nchunk * n_k),
                              hipGetErrorString(e));
    }
    st = sf_launch(n, x, q, box, n_k, m, precision, rho_re, rho_im, s, (double2 *)part, p, who);
    if (part) e = hipFreeAsync(part, s);
    if (st == RBSOG_OK && e != hipSuccess) return fail_noctx(RBSOG_E_DEVICE, "%s: free: %s", who, hipGetErrorString(e));
    return st;
}

rbsog_status rbsog_structure_factor_noalloc(int64_t n, const double *x, const double *q, const double *box,
                                            int64_t n_k, const int32_t *m, int32_t precision, double *rho_re,
                                            double *rho_im, void *stream) {
    const char *who = "rbsog_structure_factor_noalloc";
    rbsog_status st = sf_check(n, x, q, box, n_k, m, precision, rho_re, rho_im, who);
    if (st != RBSOG_OK) return st;
    if (n_k > kScratchComplex)
        return fail_noctx(RBSOG_E_ARG, "%s: n_k = %lld exceeds the %lld wave vectors its scratch holds", who,
                          (long long)n_k, (long long)kScratchComplex);
    double2 *sp = nullptr;
    st = scratch_of_current_device(&sp);
    if (st != RBSOG_OK) return st;
    const SfPlan p = sf_plan(n, n_k, precision == RBSOG_FP64);
    return sf_launch(n, x, q, box, n_k, m, precision, rho_re, rho_im, (hipStream_t)stream, sp, p, who);
}

}  // extern "C"
