// Simulation-based fit of functional edges (the paper's inverse problem,
// Sections 1 and 4; its own estimator is left to later work, so this is the
// plain fit used to judge the learned scorer).
//
// For target vertex j and a hypothesised in-neighbour set G, vertex j is
// simulated with the model of the forward path (LIF Euler step, refractory
// hold, control pulses, state noise, calcium transition of Section 3.3),
// driven by its sources' activity estimated from their own observations:
// input per step in frame f = sum_{i in G} w_i e_i(f) / S(f), e_i the
// deconvolved activity in spikes, S(f) the steps of frame f.  K noise
// realisations give the mean and variance of j's frame-averaged calcium,
// and the observed fluorescence is scored with the Gaussian observation
// model F = n*cbar + b + N(0, gamma^2) (Section 3.3):
//   LL_j(G) = -1/2 sum_f [ (F_j(f) - mu(f))^2 / s2(f) + log s2(f) ],
//   mu = n*mean_k cbar + b,  s2 = gamma^2 + n^2 var_k cbar.
//
//   fitprep_kernel   e_i(f) in spikes and the control-pulse bits of every vertex
//   fitbase_kernel   per (j, f): sum_{i in G_j} w_i e_i(f) / S(f)
//   fiteval_kernel   one workgroup per target, one lane per (variant,
//                    realisation); a variant is target j with G_j, or with one
//                    candidate toggled.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "internal.h"
#include "philox.h"

namespace geonet {
namespace {

// Box-Muller in FP64 (the fit's vertex state is FP64 too): the 24-bit
// uniforms are exact, and log, sqrt and cos are correctly rounded or within
// an ulp, so a realisation's noise agrees with any other FP64 evaluation to
// about 1e-16 and cannot move a threshold crossing in practice.
__device__ __forceinline__ double gauss_fit(uint32_t a, uint32_t b) {
    const double u1 = (static_cast<double>(a >> 8) + 0.5) * 0x1p-24;
    const double u2 = (static_cast<double>(b >> 8) + 0.5) * 0x1p-24;
    return sqrt(-2.0 * log(u1)) * cos(2.0 * 3.141592653589793 * u2);
}

__device__ __forceinline__ int64_t first_step(int64_t f, int64_t num, int64_t den) { return (f * den + num - 1) / num; }

struct FitPrepArgs {
    const float* F;            // [nf][n]
    const uint32_t* drive_thr; // [n] or null
    float* e;                  // [n][nf] activity in spikes
    uint32_t* pulses;          // [n][words] bit t: control pulse at step t
    int32_t n, nf, words;
    float rho, offset, inv_jump;   // inv_jump = 1 / (gain * dt)
    int64_t frame_num, frame_den, t_end;
    uint32_t key_lo, key_hi;
};

// One thread per (vertex, 32-step word) for the pulse bits; threads with a
// word index below nf also compute e(f) for f = word index.
__global__ void __launch_bounds__(256) fitprep_kernel(FitPrepArgs a) {
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t per = a.words > a.nf ? a.words : a.nf;
    if (idx >= static_cast<int64_t>(a.n) * per) return;
    const int j = static_cast<int>(idx / per), w = static_cast<int>(idx % per);
    if (w < a.nf) {
        const int f = w;
        const float x = a.F[static_cast<int64_t>(f) * a.n + j];
        const float e = f + 1 < a.nf
                            ? fmaxf(0.0f, (a.F[static_cast<int64_t>(f + 1) * a.n + j] - a.offset) - a.rho * (x - a.offset))
                            : 0.0f;
        a.e[static_cast<int64_t>(j) * a.nf + f] = e * a.inv_jump;
    }
    if (w < a.words) {
        uint32_t bits = 0;
        const uint32_t thr = a.drive_thr ? a.drive_thr[j] : 0u;
        if (thr != 0u) {
            for (int b = 0; b < 32; ++b) {
                const int64_t t = static_cast<int64_t>(w) * 32 + b;
                if (t >= a.t_end) break;
                const uint4 r = philox4x32_10(make_uint4(static_cast<uint32_t>(j), static_cast<uint32_t>(t),
                                                      static_cast<uint32_t>(static_cast<uint64_t>(t) >> 32), 0u),
                                           a.key_lo, a.key_hi);
                bits |= (r.x < thr ? 1u : 0u) << b;
            }
        }
        a.pulses[static_cast<int64_t>(j) * a.words + w] = bits;
    }
}

struct FitBaseArgs {
    const float* e;           // [n][nf]
    const int32_t* pairs;     // [P][2]
    const int64_t* row;       // [n+1] pairs of target j are [row[j], row[j+1]) (pairs sorted by target)
    const uint8_t* member;    // [P] 1 if the pair is in G
    const float* w_src;       // [n] assumed weight of the edges out of each vertex
    double* base;             // [n][nf]
    int32_t n, nf;
    int64_t frame_num, frame_den;
};

__global__ void __launch_bounds__(256) fitbase_kernel(FitBaseArgs a) {
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= static_cast<int64_t>(a.n) * a.nf) return;
    const int j = static_cast<int>(idx / a.nf), f = static_cast<int>(idx % a.nf);
    double s = 0.0;
    for (int64_t p = a.row[j]; p < a.row[j + 1]; ++p)
        if (a.member[p]) {
            const int i = a.pairs[2 * p];
            s += static_cast<double>(a.w_src[i]) * static_cast<double>(a.e[static_cast<int64_t>(i) * a.nf + f]);
        }
    const double steps = static_cast<double>(first_step(f + 1, a.frame_num, a.frame_den) -
                                             first_step(f, a.frame_num, a.frame_den));
    a.base[idx] = s / steps;
}

struct FitEvalArgs {
    const float* F;           // [nf][n] observed
    const float* e;           // [n][nf]
    const double* base;       // [n][nf]
    const uint32_t* pulses;   // [n][words]
    const int32_t* pairs;     // [P][2]
    const int64_t* row;       // [n+1] pairs of target j
    const uint8_t* member;    // [P]
    const float* w_src;       // [n]
    double* ll;               // [P + n]: variant v < P toggles pair v; v = P + j is G_j itself
    int64_t P, t_end;
    int32_t n, nf, words, K;
    int32_t parts, per_part;  // workgroups per target, variants per workgroup
    int32_t chunk;            // steps of noise held in LDS at a time (a multiple of 32)
    float sigma;
    double decay, v_rest, v_reset, v_th, drive_amp;
    uint32_t n_ref, hold0;    // held steps after a spike and at the start
    double dt, gain, offset, gamma2;
    int64_t frame_num, frame_den;
    uint32_t key_lo, key_hi;  // fit noise key (realisation k mixed into the counter)
    // calcium over m <= 32 steps without a spike: c -> c pw[m], its sum c gs[m]
    // (pw[m] = (1 - dt/tau_c)^m, gs[m] = pw[0] + .. + pw[m - 1])
    double pw[33], gs[33];
};

constexpr int kFitMaxThreads = 1024;
constexpr int kFitNoise = 2048;    // noise values per workgroup in LDS (K x chunk)

// LDS row length of one realisation's noise: the rows of the K realisations
// that a wave reads together start 4 banks apart.
__device__ __forceinline__ int fit_ld(int chunk) { return chunk + 2; }

// The variants of one target (every single toggle, then G_j itself), one
// lane per (variant, realisation).  A realisation's noise depends on
// (target, step, k) and not on the variant, so the workgroup draws it once
// into LDS, a chunk of steps at a time, for all its variants: a Philox block
// and an FP64 Box-Muller (about 250 instructions) per lane and step become 7
// to 14 instructions and an LDS read.  Waves beyond the variants only help
// with the draws.  Spikes are collected in a 32-step mask, and the calcium
// (linear in the spikes, and nothing feeds back from it) advances once per
// mask.  Bound by VALU issue: a third of the time draws, the rest steps.
// 512 targets, 16,000 candidate pairs, K = 8, 40,000 steps: 42.8 ms -> 4.4 ms
// per evaluation of all variants.
__global__ void __launch_bounds__(kFitMaxThreads) fiteval_kernel(FitEvalArgs a) {
    __shared__ double nz[kFitNoise + 2 * 64 + 8];
    __shared__ uint32_t pulse[kFitNoise / 32 + 1];
    __shared__ double pw[33], gs[33];
    __shared__ double cbar[2][kFitMaxThreads];
    const int tid = threadIdx.x;
    const int K = a.K;
    const int j = static_cast<int>(blockIdx.x) / a.parts, part = static_cast<int>(blockIdx.x) % a.parts;
    const int64_t row0 = a.row[j];
    const int cnt = static_cast<int>(a.row[j + 1] - row0);
    const int v0 = part * a.per_part;                       // this workgroup's variants [v0, v1) of 0 .. cnt
    const int v1 = v0 + a.per_part < cnt + 1 ? v0 + a.per_part : cnt + 1;
    if (v0 >= v1) return;                                   // (the whole workgroup)
    // lane tid is realisation tid / nv of variant v0 + tid % nv: a wave's lanes
    // have two or three realisations, whose variants mostly fire together
    const int k_shift = __builtin_ctz(static_cast<unsigned>(K));      // K divides 64
    const int nv = v1 - v0;
    const bool valid = tid < nv * K;
    const int k = valid ? tid / nv : 0, v = v0 + (valid ? tid % nv : 0);
    const bool active = __ballot(valid) != 0;               // wave-uniform
    int src = -1;
    double sign = 0.0;
    if (valid && v < cnt) {
        src = a.pairs[2 * (row0 + v)];
        sign = (a.member[row0 + v] ? -1.0 : 1.0) * static_cast<double>(a.w_src[src]);
    }
    const double* bj = a.base + static_cast<int64_t>(j) * a.nf;
    const float* es = src >= 0 ? a.e + static_cast<int64_t>(src) * a.nf : nullptr;
    const uint32_t* pj = a.pulses + static_cast<int64_t>(j) * a.words;
    if (tid < 33) {
        pw[tid] = a.pw[tid];
        gs[tid] = a.gs[tid];
    }
    const int ld = fit_ld(a.chunk);
    const double* my = nz + k * ld;
    // V in FP64: the likelihood depends on V only through spike times, and
    // FP64 keeps threshold decisions aligned with the FP64 reference
    const double decay = a.decay, v_rest = a.v_rest, v_reset = a.v_reset, v_th = a.v_th;
    double V = v_rest;
    uint32_t hold = a.hold0;
    double c = 0.0, acc = 0.0, ll = 0.0;
    int64_t t = 0, c0 = 0, c1 = 0;            // the chunk in LDS holds steps [c0, c1)
    for (int f = 0; f < a.nf; ++f) {
        const int64_t t1 = first_step(f + 1, a.frame_num, a.frame_den);
        const double steps = static_cast<double>(t1 - t);
        double u = bj[f];
        if (es) u += sign * static_cast<double>(es[f]) / steps;
        const double ud = u + a.drive_amp;
        while (t < t1) {
            if (t == c1) {
                // next chunk of noise and control pulses
                c0 = c1;
                c1 = c0 + a.chunk < a.t_end ? c0 + a.chunk : a.t_end;
                const int m = static_cast<int>(c1 - c0);
                __syncthreads();               // the chunk before has been read
                for (int i = tid; i < m * K; i += static_cast<int>(blockDim.x)) {
                    const int s = i >> k_shift, q = i & (K - 1);
                    double x = 0.0;
                    if (a.sigma != 0.0f) {
                        const int64_t ts = c0 + s;
                        const uint4 r = philox4x32_10(make_uint4(static_cast<uint32_t>(j), static_cast<uint32_t>(ts),
                                                                 static_cast<uint32_t>(static_cast<uint64_t>(ts) >> 32),
                                                                 2u + static_cast<uint32_t>(q)),
                                                      a.key_lo, a.key_hi);
                        x = static_cast<double>(a.sigma) * gauss_fit(r.y, r.z);
                    }
                    nz[q * ld + s] = x;
                }
                for (int i = tid; i <= (m + 31) / 32; i += static_cast<int>(blockDim.x)) {
                    const int64_t w = (c0 >> 5) + i;
                    pulse[i] = w < a.words ? pj[w] : 0u;
                }
                __syncthreads();
            }
            // steps [t, t + m) of the frame that the chunk holds, at most 32
            const int64_t left = (t1 < c1 ? t1 : c1) - t;
            const int m = left < 32 ? static_cast<int>(left) : 32;
            const int s0 = static_cast<int>(t - c0);
            t += m;
            if (!active) continue;
            const uint64_t pp = pulse[s0 >> 5] | (static_cast<uint64_t>(pulse[(s0 >> 5) + 1]) << 32);
            const uint32_t pbits = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(pp >> (s0 & 31)));
            uint32_t fired = 0;
            auto step = [&](uint32_t& bits, int b, double x, double ub) {
                const bool spike = V >= v_th;
                const double vn = V + decay * (v_rest - V) + (ub + x);
                V = (spike | (hold != 0u)) ? v_reset : vn;      // (no branch: lanes spike at their own steps)
                hold = spike ? a.n_ref : __builtin_elementwise_sub_sat(hold, 1u);
                bits |= spike ? 1u << b : 0u;
            };
            const double* nx = my + s0;
#pragma unroll 1
            for (int g = 0; g < m; g += 8) {
                const int r = m - g < 8 ? m - g : 8;
                const uint32_t pg = pbits >> g;
                double x[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) x[b] = nx[g + b];   // (past the chunk: not used)
                // eight steps of a wave in which no lane is held or fires: half
                // the instructions; taken back when a lane did fire
                if (r == 8 && (pg & 0xFFu) == 0u && __ballot(hold != 0u) == 0) {
                    double w = V;
                    bool any = false;
#pragma unroll
                    for (int b = 0; b < 8; ++b) {
                        any |= w >= v_th;
                        w = w + decay * (v_rest - w) + (u + x[b]);
                    }
                    if (__ballot(any) == 0) {
                        V = w;
                        continue;
                    }
                }
                uint32_t bits = 0;
#pragma unroll
                for (int b = 0; b < 8; ++b)
                    if (b < r) step(bits, b, x[b], ((pg >> b) & 1u) ? ud : u);
                fired |= bits << g;
            }
            acc += c * gs[m];
            c = c * pw[m];
            while (fired != 0u) {
                const int rest = m - 1 - __builtin_ctz(fired);
                fired &= fired - 1u;
                acc += a.dt * gs[rest];
                c += a.dt * pw[rest];
            }
        }
        // frame means of all realisations to LDS; then a variant's first lane takes
        // their mean and variance (two buffers: the lanes that write frame f + 2
        // have passed the barrier of frame f + 1, behind every read of frame f)
        double* cb = cbar[f & 1];
        if (valid) cb[tid] = acc / steps;
        acc = 0.0;
        __syncthreads();
        if (tid < nv) {
            double s1 = 0.0, s2 = 0.0;
            for (int q = 0; q < K; ++q) {
                const double x = cb[q * nv + tid];
                s1 += x;
                s2 += x * x;
            }
            const double mean = s1 / K, var = fmax(s2 / K - mean * mean, 0.0);
            const double mu = a.gain * mean + a.offset;
            const double s2f = a.gamma2 + a.gain * a.gain * var;
            const double dF = static_cast<double>(a.F[static_cast<int64_t>(f) * a.n + j]) - mu;
            ll += -0.5 * (dF * dF / s2f + log(s2f));
        }
    }
    if (tid < nv) a.ll[v0 + tid < cnt ? row0 + v0 + tid : a.P + j] = ll;
}

}  // namespace

hipError_t fit_prep(const FitInputs& in, const FitWork& w, hipStream_t s) {
    FitPrepArgs a;
    a.F = in.F;
    a.drive_thr = in.drive_thr;
    a.e = w.e;
    a.pulses = w.pulses;
    a.n = in.n;
    a.nf = in.nf;
    a.words = w.words;
    a.rho = in.rho;
    a.offset = in.offset;
    a.inv_jump = in.inv_jump;
    a.frame_num = in.frame_num;
    a.frame_den = in.frame_den;
    a.t_end = in.t_end;
    a.key_lo = in.ctl_lo;
    a.key_hi = in.ctl_hi;
    const int64_t per = w.words > in.nf ? w.words : in.nf;
    const int64_t tot = static_cast<int64_t>(in.n) * per;
    hipLaunchKernelGGL(fitprep_kernel, dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t fit_eval(const FitInputs& in, const FitWork& w, hipStream_t s) {
    FitBaseArgs b;
    b.e = w.e;
    b.pairs = in.pairs;
    b.row = w.row;
    b.member = w.member;
    b.w_src = in.w_src;
    b.base = w.base;
    b.n = in.n;
    b.nf = in.nf;
    b.frame_num = in.frame_num;
    b.frame_den = in.frame_den;
    const int64_t nb = static_cast<int64_t>(in.n) * in.nf;
    hipLaunchKernelGGL(fitbase_kernel, dim3(static_cast<unsigned>((nb + 255) / 256)), dim3(256), 0, s, b);
    FitEvalArgs a;
    a.F = in.F;
    a.e = w.e;
    a.base = w.base;
    a.pulses = w.pulses;
    a.pairs = in.pairs;
    a.member = w.member;
    a.w_src = in.w_src;
    a.ll = w.ll;
    a.P = in.P;
    a.n = in.n;
    a.nf = in.nf;
    a.words = w.words;
    a.K = in.K;
    a.decay = in.decay;
    a.v_rest = in.v_rest;
    a.v_reset = in.v_reset;
    a.v_th = in.v_th;
    a.sigma = in.sigma;
    a.drive_amp = in.drive_amp;
    a.dt = in.dt;
    a.gain = in.gain;
    a.offset = in.offset;
    a.gamma2 = static_cast<double>(in.gamma) * static_cast<double>(in.gamma);
    a.frame_num = in.frame_num;
    a.frame_den = in.frame_den;
    a.key_lo = in.fit_lo;
    a.key_hi = in.fit_hi;
    a.row = w.row;
    a.t_end = in.t_end;
    // The age counter saturates at 255: a hold of 255 steps or more never
    // ends, and the vertex, whose last spike counts as 255 steps ago, starts in it.
    a.n_ref = in.n_ref >= 255 ? 0xFFFFFFFFu : static_cast<uint32_t>(in.n_ref);
    a.hold0 = in.n_ref >= 255 ? 0xFFFFFFFFu : 0u;
    const double rho = 1.0 - in.dt / in.tau_c;
    a.pw[0] = 1.0;
    a.gs[0] = 0.0;
    for (int m = 1; m <= 32; ++m) {
        a.pw[m] = a.pw[m - 1] * rho;
        a.gs[m] = a.gs[m - 1] + a.pw[m - 1];
    }
    a.chunk = std::min(256, kFitNoise / in.K);     // K <= 64: 32 steps or more
    // One workgroup per target while its variants fit in 1,024 lanes (each
    // further one draws the noise again), and at least four waves for the
    // draws of targets with few candidates.
    const int64_t most = in.max_row + 1;           // variants of the target with the most candidates
    const int64_t room = kFitMaxThreads / in.K;
    a.parts = static_cast<int32_t>((most + room - 1) / room);
    a.per_part = static_cast<int32_t>((most + a.parts - 1) / a.parts);
    const int threads = std::max(256, static_cast<int>((static_cast<int64_t>(a.per_part) * in.K + 63) / 64 * 64));
    const int64_t blocks = static_cast<int64_t>(in.n) * a.parts;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fiteval_kernel, dim3(static_cast<unsigned>(blocks)), dim3(threads), 0, s, a);
    return hipGetLastError();
}

}  // namespace geonet
