// Observation-side kernels for the inverse problem (Sections 1 and 4 of the
// paper: estimating functional connectivity from calcium observations).
//
//   pulse_kernel     number of control pulses per vertex and frame (the
//                    experimenter's own drive schedule, Philox x0).
//   prep_kernel      per vertex: deconvolved activity e(f) = max(0, (F(f+1)-b)
//                    - rho (F(f)-b)) (the calcium model of Section 3.3 sampled
//                    at frame rate, rho = (1 - dt/tau_c)^(steps per frame)) and
//                    standardised e and F.
//   popmean_kernel   mean standardised activity over vertices per frame;
//   residual_kernel  the mean and spread of each vertex's activity without it.
//   features_kernel  64 features per candidate pair (i -> j): lagged
//                    correlations of activity and fluorescence, responses of j
//                    to i's control pulses and the reverse, activity levels,
//                    distance.  Feature k is described in featureNames() of the
//                    Python binding.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "internal.h"
#include "philox.h"

namespace geonet {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

struct PrepArgs {
    const float* F;           // [nf][n]
    const uint32_t* drive_thr;  // [n] or null
    float* en;                // [n][nf] standardised activity
    float* zn;                // [n][nf] standardised fluorescence
    float* dc;                // [n][nf] control pulses per frame
    float* stats;             // [n][5]: mean e, std F, pulses, residual mean and 1 / std
    int32_t n, nf;
    float rho, offset;
    int64_t frame_num, frame_den;
    uint32_t key_lo, key_hi;
};

// Control pulses of vertex j per frame (steps first(f) .. first(f + 1) - 1):
// one wave per kPulseFrames frames of a vertex, its lanes over a frame's
// steps.  Bound by the Philox multiplies of the driven vertices (a tenth of
// them, 333 steps a frame).
constexpr int kPulseFrames = 8;
__global__ void __launch_bounds__(256) pulse_kernel(PrepArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t per = (a.nf + 4 * kPulseFrames - 1) / (4 * kPulseFrames);   // workgroups per vertex
    for (int64_t item = blockIdx.x; item < a.n * per; item += gridDim.x) {
        const int j = static_cast<int>(item / per);
        const int w = static_cast<int>(item % per) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t thr = a.drive_thr ? a.drive_thr[j] : 0u;
        float mine = 0.0f;                             // lane q: frame w kPulseFrames + q
        if (thr != 0u) {
            for (int q = 0; q < kPulseFrames; ++q) {
                const int64_t f = static_cast<int64_t>(w) * kPulseFrames + q;
                if (f >= a.nf) break;
                const int64_t t0 = (f * a.frame_den + a.frame_num - 1) / a.frame_num;
                const int64_t t1 = ((f + 1) * a.frame_den + a.frame_num - 1) / a.frame_num;
                uint32_t count = 0;
                for (int64_t t = t0 + lane; t - lane < t1; t += 64) {
                    const uint4 r = philox4x32_10(make_uint4(static_cast<uint32_t>(j), static_cast<uint32_t>(t),
                                                          static_cast<uint32_t>(static_cast<uint64_t>(t) >> 32), 0u),
                                               a.key_lo, a.key_hi);
                    count += __popcll(__ballot(t < t1 && r.x < thr));
                }
                if (lane == q) mine = static_cast<float>(count);
            }
        }
        const int f = w * kPulseFrames + lane;
        if (lane < kPulseFrames && f < a.nf) a.dc[static_cast<int64_t>(j) * a.nf + f] = mine;
    }
}

// Activity and standardisation: one wave per vertex, four vertices per
// workgroup; their fluorescence goes through LDS 512 frames at a time, since
// a vertex's frames lie n apart in F.  A first pass sums, a second one writes.
__global__ void __launch_bounds__(256) prep_kernel(PrepArgs a) {
    constexpr int kTile = 512;
    __shared__ float tile[4][kTile + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j0 = static_cast<int>(blockIdx.x) * 4, j = j0 + wave;
    const float* x = tile[wave];
    // frames f0 .. f0 + kTile of the four vertices (the last one for f + 1)
    auto load_tile = [&](int f0) {
        const int v = tid & 3;
        __syncthreads();
        for (int i = tid >> 2; i <= kTile; i += 64) {
            const int f = f0 + i;
            tile[v][i] = f < a.nf && j0 + v < a.n ? a.F[static_cast<int64_t>(f) * a.n + j0 + v] : 0.0f;
        }
        __syncthreads();
    };
    auto activity = [&](int f, int i) {
        return f + 1 < a.nf ? fmaxf(0.0f, (x[i + 1] - a.offset) - a.rho * (x[i] - a.offset)) : 0.0f;
    };
    const int64_t row = static_cast<int64_t>(j < a.n ? j : 0) * a.nf;
    float se = 0.f, see = 0.f, sf = 0.f, sff = 0.f, sp = 0.f;
    for (int f0 = 0; f0 < a.nf; f0 += kTile) {
        load_tile(f0);
        for (int i = lane; i < kTile && f0 + i < a.nf; i += 64) {
            const float e = activity(f0 + i, i);
            se += e;
            see += e * e;
            sf += x[i];
            sff += x[i] * x[i];
            sp += a.dc[row + f0 + i];
        }
    }
    se = wave_sum(se);
    see = wave_sum(see);
    sf = wave_sum(sf);
    sff = wave_sum(sff);
    sp = wave_sum(sp);
    const float inv = 1.0f / static_cast<float>(a.nf);
    const float me = se * inv, mf = sf * inv;
    const float ve = fmaxf(see * inv - me * me, 0.0f), vf = fmaxf(sff * inv - mf * mf, 0.0f);
    const float ie = ve > 1e-12f ? rsqrtf(ve) : 0.0f, iz = vf > 1e-12f ? rsqrtf(vf) : 0.0f;
    for (int f0 = 0; f0 < a.nf; f0 += kTile) {
        if (a.nf > kTile) load_tile(f0);             // (one tile: it is still there)
        if (j < a.n) {
            for (int i = lane; i < kTile && f0 + i < a.nf; i += 64) {
                a.en[row + f0 + i] = (activity(f0 + i, i) - me) * ie;
                a.zn[row + f0 + i] = (x[i] - mf) * iz;
            }
        }
    }
    if (lane == 0 && j < a.n) {
        a.stats[j * 5 + 0] = me;
        a.stats[j * 5 + 1] = sqrtf(vf);
        a.stats[j * 5 + 2] = sp;
    }
}

// Population mean of the standardised activity per frame, summed in vertex
// order: 16 frames per workgroup, whose 1,024 threads bring 512 vertices at a
// time into LDS (the next ones in flight) for 16 lanes to add up.  The chain
// of additions bounds it: 226 -> 8.7 us for 1,024 vertices, 600 frames.
__global__ void __launch_bounds__(1024) popmean_kernel(const float* en, float* pm, int32_t n, int32_t nf) {
    constexpr int kRows = 512, kPer = kRows / 64;
    __shared__ float tile[kRows][16];
    const int x = threadIdx.x & 15, y = threadIdx.x >> 4;
    const int f = static_cast<int>(blockIdx.x) * 16 + x;
    float v[kPer], s = 0.0f;
    auto load = [&](int j0) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int j = j0 + y + 64 * k;
            v[k] = j < n && f < nf ? en[static_cast<int64_t>(j) * nf + f] : 0.0f;
        }
    };
    load(0);
    for (int j0 = 0; j0 < n; j0 += kRows) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) tile[y + 64 * k][x] = v[k];
        __syncthreads();
        load(j0 + kRows);
        if (threadIdx.x < 16) {
#pragma unroll 32
            for (int r = 0; r < kRows; ++r) s += tile[r][x];     // (rows past n are zero)
        }
    }
    if (threadIdx.x < 16 && f < nf) pm[f] = s / static_cast<float>(n);
}

// Mean and 1 / std of the residual activity en - pm of every vertex (one wave
// each); the residual itself is formed where it is used.
__global__ void __launch_bounds__(256) residual_kernel(const float* en, const float* pm, float* stats, int32_t n,
                                                       int32_t nf) {
    const int lane = threadIdx.x & 63;
    const int j = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (j >= n) return;
    float s = 0.f, ss = 0.f;
    for (int f = lane; f < nf; f += 64) {
        const float r = en[static_cast<int64_t>(j) * nf + f] - pm[f];
        s += r;
        ss += r * r;
    }
    s = wave_sum(s);
    ss = wave_sum(ss);
    const float m = s / nf, v = fmaxf(ss / nf - m * m, 0.0f), iv = v > 1e-12f ? rsqrtf(v) : 0.0f;
    if (lane == 0) {
        stats[j * 5 + 3] = m;
        stats[j * 5 + 4] = iv;
    }
}

struct FeatArgs {
    const float* en;
    const float* zn;
    const float* dc;
    const float* pm;
    const float* stats;
    const int32_t* pairs;     // [P][2] (i, j)
    const float* dist;        // [P]
    float* out;               // [P][64]
    int64_t P;
    int32_t nf;
};

// Sum over the wave of 64 values per lane, value k ending in lane k: each
// level halves the values a lane still holds.  The additions are those of
// wave_sum (partners 32, 16, .. 1 apart) with 63 exchanges instead of 6 x 64.
template <int H>
__device__ __forceinline__ void fold_lanes(float (&v)[64], int lane) {
    const bool up = (lane & H) != 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const float other = __shfl_xor(up ? v[k] : v[k + H], H, 64);
        v[k] = (up ? v[k + H] : v[k]) + other;
    }
}

__device__ __forceinline__ float wave_sum_to_lane(float (&v)[64], int lane) {
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        // lanes 32..63 of v[k] change places with lanes 0..31 of v[k + 32]
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[k]), __float_as_uint(v[k + 32]), false, false);
        v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[k]), __float_as_uint(v[k + 16]), false, false);
        v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    fold_lanes<8>(v, lane);
    fold_lanes<4>(v, lane);
    fold_lanes<2>(v, lane);
    fold_lanes<1>(v, lane);
    return v[0];
}

// Orders this wave's LDS writes before its later reads of other lanes' words
// (the LDS serves a wave's operations in order; the compiler has to keep it).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per pair, all 53 sums over frames in one pass: a lane has frames
// lane, lane + 64, .. of both vertices' rows in registers and takes the rows'
// later frames, which the lags need, from LDS (64 frames and 8 more of the
// next 64, which are already in flight); a negative lag is a later frame of
// the source.  One load per value instead of one per value, lag and feature,
// and one folded reduction instead of one per feature.  Each sum takes its
// terms in the order f = lane, lane + 64, .., multiplied and added apart, then
// pairwise over the lanes: the scorer rounds features to BF16, where any other
// order would move roundings.  Workgroups that share an XCD take consecutive
// pairs, whose rows then meet in its L2.  Bound by VALU issue (106 operations
// per 64 frames).  1,024 vertices, 64,000 pairs, 600 frames: 838 -> 173 us.
__global__ void __launch_bounds__(256) features_kernel(FeatArgs a) {
    constexpr int kHalo = 8, kRow = 64 + kHalo;
    __shared__ float lds[4][5][kRow];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nb = static_cast<int>(gridDim.x), b = static_cast<int>(blockIdx.x);
    const int64_t lb = nb % 8 == 0 ? static_cast<int64_t>(b % 8) * (nb / 8) + b / 8 : b;
    const int64_t p = lb * 4 + wave;
    if (p >= a.P) return;
    const int i = __builtin_amdgcn_readfirstlane(a.pairs[2 * p]);
    const int j = __builtin_amdgcn_readfirstlane(a.pairs[2 * p + 1]);
    const int nf = a.nf;
    const float* ei = a.en + static_cast<int64_t>(i) * nf;
    const float* ej = a.en + static_cast<int64_t>(j) * nf;
    const float* zi = a.zn + static_cast<int64_t>(i) * nf;
    const float* zj = a.zn + static_cast<int64_t>(j) * nf;
    const float* di = a.dc + static_cast<int64_t>(i) * nf;
    const float* dj = a.dc + static_cast<int64_t>(j) * nf;
    const float* si = a.stats + i * 5;
    const float* sj = a.stats + j * 5;
    const float mi = si[3], vi = si[4], mj = sj[3], vj = sj[4];
    float (*row)[kRow] = lds[wave];
    struct Frame {
        float ei, ej, zi, zj, di, dj, ri, rj;
    };
    auto load = [&](int f) {
        Frame x{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};     // frames past the last one add nothing
        if (f < nf) {
            const float m = a.pm[f];
            x.ei = ei[f];
            x.ej = ej[f];
            x.zi = zi[f];
            x.zj = zj[f];
            x.di = di[f];
            x.dj = dj[f];
            x.ri = (x.ei - m - mi) * vi;
            x.rj = (x.ej - m - mj) * vj;
        }
        return x;
    };
    float acc[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) acc[k] = 0.0f;
    Frame cur = load(lane);
    for (int f = lane; f - lane < nf; f += 64) {
        const Frame nxt = load(f + 64);
        row[0][lane] = cur.ei;
        row[1][lane] = cur.ej;
        row[2][lane] = cur.zi;
        row[3][lane] = cur.zj;
        row[4][lane] = cur.rj;
        if (lane < kHalo) {
            row[0][64 + lane] = nxt.ei;
            row[1][64 + lane] = nxt.ej;
            row[2][64 + lane] = nxt.zi;
            row[3][64 + lane] = nxt.zj;
            row[4][64 + lane] = nxt.rj;
        }
        wave_lds_fence();
#pragma unroll
        for (int L = 0; L <= 8; ++L) {
            const float ejL = L ? row[1][lane + L] : cur.ej;
            acc[8 + L] += cur.ei * ejL;
            if (L < 6) acc[22 + L] += cur.di * ejL;
            if (L < 8) acc[51 + L] += cur.zi * ejL;
            const float eiL = L ? row[0][lane + L] : cur.ei;
            if (L) acc[8 - L] += eiL * cur.ej;
            if (L < 4) acc[28 + L] += cur.dj * eiL;
            if (L < 8) {
                const float zjL = L ? row[3][lane + L] : cur.zj;
                acc[43 + L] += cur.ei * zjL;
                if (L < 3) acc[19 + L] += cur.zi * zjL;
            }
            if (L == 1 || L == 2) acc[19 - L] += row[2][lane + L] * cur.zj;
            if (L < 4) acc[39 + L] += cur.ri * (L ? row[4][lane + L] : cur.rj);
        }
        wave_lds_fence();
        cur = nxt;
    }
    const float s = wave_sum_to_lane(acc, lane);
    // lane k has the sum of feature k: 0..16, 17..21, 39..42, 43..50, 51..58 are
    // lagged correlations, means over the frames that have a partner; 22..31
    // are responses per control pulse
    int L = 0;
    if (lane < 17) L = lane < 8 ? 8 - lane : lane - 8;
    else if (lane < 22) L = lane < 19 ? 19 - lane : lane - 19;
    else if (lane >= 39 && lane < 43) L = lane - 39;
    else if (lane >= 43 && lane < 51) L = lane - 43;
    else if (lane >= 51) L = lane - 51;
    const float npi = si[2], npj = sj[2];
    float val;
    if (lane < 22 || (lane >= 39 && lane < 59)) val = nf > L ? s / static_cast<float>(nf - L) : 0.0f;
    else if (lane < 28) val = s / fmaxf(1.0f, npi);
    else if (lane < 32) val = s / fmaxf(1.0f, npj);
    else if (lane < 34) val = log1pf(lane == 32 ? npi : npj);
    else if (lane < 36) val = (lane == 34 ? si : sj)[0];
    else if (lane < 38) val = (lane == 36 ? si : sj)[1];
    else if (lane == 38) val = a.dist[p] * (1.0f / 150.0f);
    else val = 0.0f;
    a.out[p * 64 + lane] = val;
}

}  // namespace

namespace {
__global__ void __launch_bounds__(256) pulse_threshold_kernel(const float* rates, int32_t n, double dt_ms,
                                                              uint32_t* thr) {
    const int32_t j = static_cast<int32_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n) return;
    // the same double-precision rule as pulse_threshold on the host
    const double t = floor(static_cast<double>(rates[j]) * (dt_ms * 1e-3) * 4294967296.0);
    thr[j] = !(t > 0.0) ? 0u : (t >= 4294967295.0 ? 0xFFFFFFFFu : static_cast<uint32_t>(t));
}
}  // namespace

hipError_t launch_pulse_thresholds(const float* rates, int32_t n, double dt_ms, uint32_t* thr, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pulse_threshold_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, rates,
                       n, dt_ms, thr);
    return hipGetLastError();
}

hipError_t launch_features(const FeatureInputs& in, const FeatureWork& w, float* out, hipStream_t s) {
    PrepArgs pa;
    pa.F = in.F;
    pa.drive_thr = in.drive_thr;
    pa.en = w.en;
    pa.zn = w.zn;
    pa.dc = w.dc;
    pa.stats = w.stats;
    pa.n = in.n;
    pa.nf = in.nf;
    pa.rho = in.rho;
    pa.offset = in.offset;
    pa.frame_num = in.frame_num;
    pa.frame_den = in.frame_den;
    pa.key_lo = in.key_lo;
    pa.key_hi = in.key_hi;
    const int64_t per = (in.nf + 4 * kPulseFrames - 1) / (4 * kPulseFrames);
    const int64_t th = static_cast<int64_t>(in.n) * 64;
    hipLaunchKernelGGL(pulse_kernel, dim3(static_cast<unsigned>(std::min<int64_t>(in.n * per, 1 << 20))),
                       dim3(256), 0, s, pa);
    hipLaunchKernelGGL(prep_kernel, dim3(static_cast<unsigned>((in.n + 3) / 4)), dim3(256), 0, s, pa);
    hipLaunchKernelGGL(popmean_kernel, dim3(static_cast<unsigned>((in.nf + 15) / 16)), dim3(1024), 0, s, w.en, w.pm,
                       in.n, in.nf);
    hipLaunchKernelGGL(residual_kernel, dim3(static_cast<unsigned>((th + 255) / 256)), dim3(256), 0, s, w.en, w.pm,
                       w.stats, in.n, in.nf);
    FeatArgs fa;
    fa.en = w.en;
    fa.zn = w.zn;
    fa.dc = w.dc;
    fa.pm = w.pm;
    fa.stats = w.stats;
    fa.pairs = in.pairs;
    fa.dist = in.dist;
    fa.out = out;
    fa.P = in.P;
    fa.nf = in.nf;
    if (in.P > 0) {
        const int64_t blocks = ((in.P + 3) / 4 + 7) / 8 * 8;      // a multiple of the XCDs
        hipLaunchKernelGGL(features_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, fa);
    }
    return hipGetLastError();
}

}  // namespace geonet
