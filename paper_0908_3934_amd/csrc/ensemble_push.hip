// Single-launch kernel: every network of a handle on one workgroup of its
// own, all steps of a call in one launch, vertex state in registers and the
// arriving input in LDS.
//
// Delivery.  Each network keeps a ring of W + 1 input slots in LDS (one word
// per vertex and slot; slot t mod (W + 1) holds the input of step t).  A spike
// of step t adds the weights of its out-edges with delays 1 .. W into the
// slots of their arrival steps during step t; where delays reach further, its
// out-edges with delays w W + 1 .. (w + 1) W follow w W steps later.  Spikes
// are kept as one bit per vertex and step.  A vertex's spike of step t + 1 is
// known as soon as step t has updated it, so at the start of a step all its
// spikes stand in LDS, every wave takes an equal share of them whatever
// vertices they belong to, and, since no push of step t touches slot t, a step
// needs one barrier.
//
// The slots hold integers: the weights of a network are multiples of its
// smallest FP16 spacing, a power of two, and are added in that unit wherever
// every row's sum of magnitudes fits 31 bits.  Such a sum is exact, so the
// order of the atomics changes no bit, and where FP32 sums are exact too it is
// the very same.  The other networks' slots hold floats, whose sums depend on
// that order where a row is not exact in FP32 (NET_W_INEXACT).  On gfx950 a 64-lane ds_add_f32 takes 80 ns of the CU's LDS, a ds_add_u32 to
// the same addresses 2.8 ns.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "philox.h"
#include "push_plan.h"
#include "vertex.h"

namespace geonet {
namespace {

// Groups up to which a wave pushes its own vertices' spikes (see push_run).  us
// per step, shared and own, quiet networks of the 2-D kind: 64 vertices 0.38 /
// 0.29, 256 0.42 / 0.34; 256 vertices of 26 out-edges each, 7 spikes a step 1.21
// / 0.89.  With one vertex a lane it still is the faster form above this line
// (320: 0.46 / 0.37, 512: 0.49 / 0.38, 512 with 15 spikes a step 1.57 / 1.35,
// 1,024: 0.59 / 0.50).
constexpr int kPushOwnGroups = 4;
static_assert(kPushThreads / 64 * kPushMaxVpt <= kWordMaxGroups && kPushThreadsFp64 / 64 * kPushMaxVptFp64 <= kWordMaxGroups,
              "word_window is exact up to so many groups");

struct PushArgs {
    const PushNet* __restrict__ nets;       // [blocks] in launch order
    const uint32_t* __restrict__ off;       // per network n x n_win + 1 edge offsets: entry s n_win + w opens
                                            // the edges of source s in window w
    const uint32_t* __restrict__ edge;      // target | (delay within the window - 1) << tbits | FP16 weight << 16
    float* __restrict__ ring;               // between launches: every network's input slots
    uint64_t* __restrict__ hist;            // between launches: every network's spike bits
    const NetParams* __restrict__ params;
    const uint32_t* __restrict__ drive_thr;
    const float* __restrict__ i_ext;
    float* __restrict__ V;
    uint16_t* __restrict__ age;
    double* __restrict__ calcium;
    double* __restrict__ frame_acc;
    float* __restrict__ frames;
    uint64_t* __restrict__ rec_raster;
    float* __restrict__ rec_v;
    float* __restrict__ rec_input;
    double* __restrict__ Vd;
    double* __restrict__ Wd;
    double* __restrict__ psc_r;
    double* __restrict__ psc_p;
    double* __restrict__ hh_m;
    double* __restrict__ hh_n;
    double* __restrict__ hh_h;
    double* __restrict__ hh_vprev;
    const int32_t* __restrict__ caller_of;
    const uint64_t* __restrict__ t_dev;     // graph replays: the step is *t_dev + t0
    // noise drawn ahead (null: drawn in the steps): [n_steps][noise_stride] values
    // and one word of control pulses per 64 of them
    double* __restrict__ noise;
    uint64_t* __restrict__ noise_pulses;
    int64_t noise_stride;
    int64_t t0, n_total, n_pad, raster_words;
    int32_t n_steps, frame_cap, frame_num, frame_den;
};

typedef const PushArgs __attribute__((address_space(4)))* const_args;

// What a wave keeps of its network while the steps run (all wave-uniform but
// `lane`).
struct PushCtx {
    const uint32_t* off;      // this network's edge offsets
    const uint32_t* edge;
    float* ring;              // W + 1 slots of `stride` words
    uint64_t* hist;           // spike bits of `buckets` steps up to the next one, one word per group
    const double* pw;         // calcium over m steps without a spike: c -> c pw[m],
    const double* gs;         // its sum c gs[m]
    uint32_t stride, slots, n_win, tbits, buckets;
    uint32_t groups_inv;      // word_inverse(groups)
    int n, groups, wave, waves, nq, node_off, lane;
    int noise_at;             // the network's first value in a row of the noise drawn ahead
    float unit, inv_unit;     // one unit of the slots' integers and its inverse (0: the slots hold floats)
    bool obs, last_net;
    bool own;                 // every wave pushes its own vertices' spikes (see push_run)
};

// Adds the edges [e0, e1) of every lane into the input slots, the
// whole wave taking 64 edges of one list at a time and eight such loads in
// flight; `slot` is the slot of the step the lists' delays count from.
__device__ __forceinline__ void push_lists(const PushCtx& c, uint32_t e0, uint32_t e1, uint32_t slot) {
    constexpr int kJobs = 8;
    uint64_t from = wave_ballot(e1 > e0);
    uint32_t e = 0, end = 0;
    while (e < end || from != 0) {
        uint32_t rec[kJobs];
        int jobs = 0;
#pragma unroll
        for (int k = 0; k < kJobs; ++k) {
            if (e >= end && from == 0) break;
            if (e >= end) {
                const int l = __builtin_ctzll(from);
                from &= from - 1;
                e = __builtin_amdgcn_readlane(e0, l);
                end = __builtin_amdgcn_readlane(e1, l);
            }
            // (weight 0 past the list's end: adds nothing)
            const uint32_t at = e + static_cast<uint32_t>(c.lane);
            rec[k] = 0u;
            if (at < end) rec[k] = c.edge[at];
            e += 64u;
            jobs = k + 1;
        }
#pragma unroll
        for (int k = 0; k < kJobs; ++k) {
            if (k >= jobs) break;
            if ((rec[k] >> 16) != 0u) {
                uint32_t s = slot + 1u + ((rec[k] & 0xFFFFu) >> c.tbits);
                s = s >= c.slots ? s - c.slots : s;
                float* to = c.ring + s * c.stride + (rec[k] & ((1u << c.tbits) - 1u));
                const float w = half_bits_to_float(rec[k] >> 16);
                if (c.inv_unit != 0.0f)
                    atomicAdd(reinterpret_cast<int*>(to), static_cast<int>(w * c.inv_unit));
                else
                    atomicAdd(to, w);
            }
        }
    }
}

// The lane's part of the vertices' state.  Lanes past the network's last
// vertex hold NaN, which never spikes.
template <int VPT, bool kFp64>
struct PushState {
    float V[VPT], iext[VPT];
    uint32_t last[VPT];                 // step of the last spike
    uint32_t jl[VPT], thr[VPT];         // index in the random streams, drive threshold
    uint32_t bits[VPT], pm[VPT];        // spikes and control pulses of the block's steps
    double cal[VPT], acc[VPT];
    HhState st[kFp64 ? VPT : 1];        // FP64 models (an Izhikevich vertex keeps its W in m)
};

// Whether vertex q of the lane spikes in the step its state stands at.
template <int kModel, class State>
__device__ __forceinline__ bool push_spikes(const State& S, int q, const NetParams& p) {
    if constexpr (kModel == NET_MODEL_LIF) return S.V[q] >= p.v_th;
    else if constexpr (kModel == NET_MODEL_IZHIKEVICH) return S.st[q].v >= static_cast<double>(p.v_th);
    else return S.st[q].v >= static_cast<double>(p.v_th) && S.st[q].vprev < static_cast<double>(p.v_th);
}

// How a network's noise comes: it has none, or every wave draws its own, or
// the draws were made ahead by noise_kernel.
enum { kQuiet = 0, kDraws = 1, kAhead = 2 };

// Steps t0 .. t1 - 1 of a network of one model.
template <int kModel, int kNoise, int VPT, bool kFp64>
__device__ __forceinline__ void push_run(const const_args ka, const PushCtx& c, const NetParams& p,
                                         PushState<VPT, kFp64>& S, const int64_t t0, const int64_t t1) {
    const int lane = c.lane;
    const bool pulses = kNoise == kQuiet && reread(ka)->drive_thr != nullptr;
    uint64_t* raster = reread(ka)->rec_raster;             // this step's row, or null
    // what a step asks about, opaque in the loop so that it is not copied for every combination
    enum { kRaster = 1, kRecords = 2 };
    const uint32_t asks = (raster ? kRaster : 0u) | (reread(ka)->rec_v || reread(ka)->rec_input ? kRecords : 0u);
    uint32_t slot = static_cast<uint32_t>(static_cast<uint64_t>(t0) % c.slots);
    uint32_t bucket = static_cast<uint32_t>(static_cast<uint64_t>(t0) % c.buckets);
    const uint32_t W = c.slots - 1u;
    const uint32_t words = c.n_win * static_cast<uint32_t>(c.groups);
    const uint32_t my_w = word_window(static_cast<uint32_t>(lane), c.groups_inv);   // window and group of the lane's
    const uint32_t my_g = static_cast<uint32_t>(lane) - my_w * static_cast<uint32_t>(c.groups);   // first word
    // Small LIF networks of one window: a wave's own spikes, which it has in
    // registers, straight away; nothing is shared.  In networks of the FP64 models
    // the spikes of a step gather in few waves (densest Izhikevich one 7.6 us a
    // step shared, above 9 so), and where a lane has several vertices the second
    // form's code alone costs 4 %.
    constexpr bool kOwn = kModel == NET_MODEL_LIF && VPT == 1;
    const bool own = kOwn && c.own;
    uint64_t spk[VPT];                       // this wave's spikes of the step to come
#pragma unroll
    for (int q = 0; q < VPT; ++q) spk[q] = c.hist[bucket * c.groups + (q < c.nq ? c.wave + q * c.waves : c.wave)];

    // noise drawn ahead: this wave's words and values of the step to come
    const double* nz = kNoise == kAhead ? reread(ka)->noise + c.noise_at + c.wave * 64 + lane : nullptr;
    const uint64_t* nz_pulse = kNoise == kAhead ? reread(ka)->noise_pulses + (c.noise_at >> 6) + c.wave : nullptr;
    const int64_t nz_row = kNoise == kAhead ? reread(ka)->noise_stride : 0;
    double ahead[VPT] = {};
    uint64_t ahead_pulse[VPT] = {};
    auto fetch_noise = [&]() {
        if constexpr (kNoise == kAhead) {
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                if (q < c.nq) {
                    ahead[q] = nz[q * c.waves * 64];
                    ahead_pulse[q] = nz_pulse[q * c.waves];
                }
            }
            nz += nz_row;
            nz_pulse += nz_row >> 6;
        }
    };
    fetch_noise();

    int64_t t = t0;
    while (t < t1) {
        // ---- a block of steps
        int m = t1 - t < 32 ? static_cast<int>(t1 - t) : 32;
        int64_t frame = 0, next = 0;
        if (c.obs) {
            const const_args a = reread(ka);
            frame = t * a->frame_num / a->frame_den;
            next = ((frame + 1) * a->frame_den + a->frame_num - 1) / a->frame_num;
            if (next - t < m) m = static_cast<int>(next - t);
        }
        if (pulses) {
            const const_args a = reread(ka);
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                if (q >= c.nq) break;
                const int j = (c.wave + q * c.waves) * 64 + lane;
                const uint32_t th = j < c.n ? a->drive_thr[c.node_off + j] : 0u;
                uint32_t pm = 0u;
                // two driven vertices by 32 steps per Philox evaluation
                for (uint64_t rem = wave_ballot(th != 0u); rem != 0;) {
                    const int l0 = __builtin_ctzll(rem);
                    rem &= rem - 1;
                    const int l1 = rem != 0 ? __builtin_ctzll(rem) : l0;
                    if (rem != 0) rem &= rem - 1;
                    const uint32_t j0 = __builtin_amdgcn_readlane(S.jl[q], l0), j1 = __builtin_amdgcn_readlane(S.jl[q], l1);
                    const uint32_t h0 = __builtin_amdgcn_readlane(th, l0), h1 = __builtin_amdgcn_readlane(th, l1);
                    const uint64_t ts = static_cast<uint64_t>(t) + (lane & 31);
                    const uint4 r = philox4x32_10(make_uint4(lane < 32 ? j0 : j1, static_cast<uint32_t>(ts),
                                                             static_cast<uint32_t>(ts >> 32), 0u),
                                                  opaque(p.key_lo), opaque(p.key_hi));
                    const uint64_t hit = wave_ballot(r.x < (lane < 32 ? h0 : h1));
                    if (lane == l0) pm = static_cast<uint32_t>(hit);
                    else if (lane == l1) pm = static_cast<uint32_t>(hit >> 32);
                }
                S.pm[q] = pm;
            }
        }
        for (int b = 0; b < m; ++b) {
            const uint32_t ask = opaque(asks);
            const int nq = static_cast<int>(opaque(static_cast<uint32_t>(c.nq)));
            const uint32_t t_lo = static_cast<uint32_t>(t + b);
            float* mine = c.ring + slot * c.stride + static_cast<uint32_t>(c.wave * 64 + lane);
            float in[VPT];
            // this step's input (the slot is cleared for step t + W + 1)
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                in[q] = 0.0f;
                if (q < nq)
                    in[q] = __hip_atomic_exchange(mine + q * c.waves * 64, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            if (c.inv_unit != 0.0f) {
#pragma unroll
                for (int q = 0; q < VPT; ++q) in[q] = static_cast<float>(__float_as_int(in[q])) * c.unit;
            }
            // the step's words of spike bits (window w's of step t - w W); the first 64 here
            uint64_t word = 0;
            if (!own && static_cast<uint32_t>(lane) < words) {
                int at = static_cast<int>(bucket) - static_cast<int>(my_w * W);
                at = at < 0 ? at + static_cast<int>(c.buckets) : at;
                word = c.hist[static_cast<uint32_t>(at * c.groups) + my_g];
            }
            if (ask & kRecords) {
                const const_args a = reread(ka);
                const int64_t row = (t + b - t0) * a->n_total + c.node_off;
#pragma unroll
                for (int q = 0; q < VPT; ++q) {
                    const int j = (c.wave + q * c.waves) * 64 + lane;
                    if (q >= nq || j >= c.n) continue;
                    if (a->rec_v) a->rec_v[row + j] = S.V[q];
                    if (a->rec_input) a->rec_input[row + j] = in[q];
                }
            }
            double drawn[VPT];
            uint64_t drawn_pulse[VPT];
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                drawn[q] = ahead[q];
                drawn_pulse[q] = ahead_pulse[q];
            }
            if (kNoise == kAhead && t + b + 1 < t1) fetch_noise();
            // ---- vertex update
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                if (q >= nq) continue;
                const bool spike = ((spk[q] >> lane) & 1u) != 0u;
                bool pulse;
                uint4 r{};
                if constexpr (kNoise == kAhead) {
                    pulse = ((drawn_pulse[q] >> lane) & 1u) != 0u;
                } else if constexpr (kNoise == kDraws) {
                    const uint32_t t_hi = static_cast<uint32_t>(static_cast<uint64_t>(t + b) >> 32);
                    r = philox4x32_10(make_uint4(S.jl[q], t_lo, t_hi, 0u), p.key_lo, p.key_hi);
                    pulse = r.x < S.thr[q];
                } else {
                    pulse = ((S.pm[q] >> b) & 1u) != 0u;
                }
                if constexpr (kModel == NET_MODEL_LIF) {
                    float u = S.iext[q];
                    u = pulse ? u + p.drive_amp : u;
                    float vn = S.V[q] + p.decay * (p.v_rest - S.V[q]) + in[q] + u;
                    if constexpr (kNoise == kDraws) vn = vn + p.sigma * gaussian(r.y, r.z);
                    if constexpr (kNoise == kAhead) vn = vn + static_cast<float>(drawn[q]);
                    const bool held = t_lo - S.last[q] - 1u < static_cast<uint32_t>(p.n_ref);
                    S.V[q] = (spike | held) ? p.v_reset : vn;
                } else {
                    double u = static_cast<double>(S.iext[q]), noise = 0.0;
                    u = pulse ? u + static_cast<double>(p.drive_amp) : u;
                    if constexpr (kNoise == kDraws) noise = static_cast<double>(p.sigma) * gaussian_d(r.y, r.z);
                    if constexpr (kNoise == kAhead) noise = drawn[q];
                    if constexpr (kModel == NET_MODEL_IZHIKEVICH) {
                        const IzhState z = izh_step(p, IzhState{S.st[q].v, S.st[q].m, S.st[q].r, S.st[q].p}, spike,
                                                    static_cast<double>(in[q]), u, noise);
                        S.st[q].v = z.v;
                        S.st[q].m = z.w;
                        S.st[q].r = z.r;
                        S.st[q].p = z.p;
                    } else {
                        S.st[q] = hh_step(p, S.st[q], static_cast<double>(in[q]), u, noise);
                    }
                    S.V[q] = static_cast<float>(S.st[q].v);
                }
                S.last[q] = spike ? t_lo : S.last[q];
                S.bits[q] |= spike ? 1u << b : 0u;
            }
            if (ask & kRaster) {
#pragma unroll
                for (int q = 0; q < VPT; ++q) {
                    if (q >= nq) break;
                    const int j0 = (c.wave + q * c.waves) * 64, u0 = c.node_off + j0, left = c.n - j0;
                    // a word of 64 vertices of this network alone is stored as it is
                    if (lane == 0) {
                        if ((u0 & 63) == 0 && (left >= 64 || c.last_net)) raster[u0 >> 6] = spk[q];
                        else put_bits_shared(raster, u0, spk[q], left >= 64 ? ~0ull : (1ull << left) - 1ull);
                    }
                }
                raster += reread(ka)->raster_words;
            }
            // ---- push: every wave takes each `waves`-th of the spikes, 64 words at a
            // time (all of this in one branch: on a step without spikes nothing
            // waits for the memory accesses in flight)
            if constexpr (kOwn) {
                if (own) {
#pragma unroll
                    for (int q = 0; q < VPT; ++q) {
                        if (q >= nq || spk[q] == 0) continue;
                        uint32_t e0 = 0u, e1 = 0u;
                        if ((spk[q] >> lane) & 1u) {
                            const uint32_t o = static_cast<uint32_t>((c.wave + q * c.waves) * 64 + lane);
                            e0 = c.off[o];
                            e1 = c.off[o + 1u];
                        }
                        push_lists(c, e0, e1, slot);
                    }
                }
            }
            for (uint32_t k0 = own ? words : 0u; k0 < words; k0 += 64u) {
                uint32_t word_w = my_w, word_g = my_g;
                if (k0 != 0u) {
                    const uint32_t k = k0 + static_cast<uint32_t>(lane);
                    word_w = word_window(k, c.groups_inv);
                    word_g = k - word_w * static_cast<uint32_t>(c.groups);
                    word = 0;
                    if (k < words) {
                        int at = static_cast<int>(bucket) - static_cast<int>(word_w * W);
                        at = at < 0 ? at + static_cast<int>(c.buckets) : at;
                        word = c.hist[static_cast<uint32_t>(at * c.groups) + word_g];
                    }
                }
                if (wave_ballot(word != 0) == 0) continue;
                uint32_t total;
                const uint32_t before = wave_prefix(static_cast<uint32_t>(__popcll(word)), &total);
                uint32_t rank = static_cast<uint32_t>(c.wave);
                while (rank < total) {
                    // the next up to 64 spikes of this wave, one per lane
                    uint32_t o = 0u, share = 0u;
                    for (; rank < total && share < 64u; rank += static_cast<uint32_t>(c.waves), ++share) {
                        const int from = 63 - __builtin_clzll(wave_ballot(before <= rank));
                        uint64_t bits = read_lane64(word, from);
                        for (uint32_t skip = rank - __builtin_amdgcn_readlane(before, from); skip != 0u; --skip) bits &= bits - 1;
                        const uint32_t src = __builtin_amdgcn_readlane(word_g, from) * 64u + static_cast<uint32_t>(__builtin_ctzll(bits));
                        const uint32_t at = src * c.n_win + __builtin_amdgcn_readlane(word_w, from);
                        o = static_cast<uint32_t>(lane) == share ? at : o;
                    }
                    uint32_t e0 = 0u, e1 = 0u;
                    if (static_cast<uint32_t>(lane) < share) {
                        e0 = c.off[o];
                        e1 = c.off[o + 1u];
                    }
                    push_lists(c, e0, e1, slot);
                }
            }
            // ---- spikes of the next step
            bucket = bucket + 1u == c.buckets ? 0u : bucket + 1u;
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                bool spike = false;
                if (q < nq) spike = push_spikes<kModel>(S, q, p);
                spk[q] = wave_ballot(spike);
                if (!own && q < nq && lane == 0) c.hist[bucket * static_cast<uint32_t>(c.groups) + c.wave + q * c.waves] = spk[q];
            }
            slot = slot + 1u == c.slots ? 0u : slot + 1u;
            lds_barrier();
        }
        t += m;
        if (c.obs) {
            const const_args a = reread(ka);
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                if (q >= c.nq) break;
                S.acc[q] += S.cal[q] * c.gs[m];
                S.cal[q] = S.cal[q] * c.pw[m];
                while (S.bits[q] != 0u) {
                    const int rest = m - 1 - __builtin_ctz(S.bits[q]);
                    S.bits[q] &= S.bits[q] - 1u;
                    S.acc[q] += p.dt_d * c.gs[rest];
                    S.cal[q] += p.dt_d * c.pw[rest];
                }
                if (t == next) {
                    const int j = (c.wave + q * c.waves) * 64 + lane;
                    if (frame < a->frame_cap && j < c.n) {
                        const int64_t first = (frame * a->frame_den + a->frame_num - 1) / a->frame_num;
                        a->frames[frame * a->n_pad + c.node_off + j] =
                            static_cast<float>(S.acc[q] / static_cast<double>(next - first));
                    }
                    S.acc[q] = 0.0;
                }
            }
        }
    }
}

// One workgroup per network; wave w has the 64-vertex groups w, w + waves, ..
// (at most VPT), each lane one vertex of each.  kModels: 0 LIF networks only,
// 1 with Izhikevich ones, 2 with Hodgkin-Huxley ones too (a network has one
// model, so the choice is the workgroup's).
//
// Steps run in blocks of at most 32 (ending with a camera frame): the control
// pulses of noise-free networks are drawn once per block, two vertices by 32
// steps at a time, and calcium, which nothing feeds back from, advances once
// per block from the block's spike bits.
//
// What bounds it: for small networks the barrier and the LDS round trip of a
// step, for large ones VALU issue on one CU and the two dependent loads of a
// spiking wave (offsets, edges).  Measured, us per step, before (two barriers,
// delivery pulled or pushed by one wave) and now: one quiet LIF network of 256
// vertices 2.46 / 0.41; 128 LIF networks of 64 .. 4096 8.9 / 1.8; 512 of them
// 8.1 / 2.3; 40 Izhikevich networks (the largest 1,000 vertices, 2e5 edges)
// 38 / 7.6; the same as Hodgkin-Huxley networks 49 / 6.1.
template <int kModels, int VPT, int kThreads>
__global__ void __launch_bounds__(kThreads) push_ensemble_kernel(PushArgs args) {
    extern __shared__ uint4 lds4[];
    (void)args;
    const const_args ka = (const_args)__builtin_amdgcn_kernarg_segment_ptr();
    const_args a = reread(ka);
    const int tid = threadIdx.x;
    const PushNet nm = load_const(a->nets + blockIdx.x);
    PushCtx c;
    c.lane = tid & 63;
    c.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    c.n = nm.n;
    c.groups = nm.groups;
    c.waves = static_cast<int>(blockDim.x >> 6) < nm.groups ? static_cast<int>(blockDim.x >> 6) : nm.groups;
    if (c.wave >= c.waves) return;                  // (barriers count the waves that are left)
    c.nq = (c.groups - c.wave + c.waves - 1) / c.waves;          // this wave's groups
    const NetParams p = load_const(a->params + nm.net);
    c.node_off = nm.node_off;
    c.noise_at = nm.noise_at;
    c.slots = static_cast<uint32_t>(nm.window) + 1u;
    c.n_win = static_cast<uint32_t>(nm.n_win);
    c.tbits = static_cast<uint32_t>(nm.tbits);
    c.buckets = (c.n_win - 1u) * static_cast<uint32_t>(nm.window) + 2u;
    c.groups_inv = word_inverse(static_cast<uint32_t>(c.groups));
    c.stride = static_cast<uint32_t>(c.groups) * 64u;
    c.obs = a->calcium != nullptr;
    c.last_net = nm.node_off + nm.n == a->n_total;
    c.own = c.n_win == 1u && c.groups <= kPushOwnGroups;
    c.unit = nm.unit;
    c.inv_unit = nm.inv_unit;
    c.off = a->off + nm.off_at;
    c.edge = a->edge;
    c.ring = reinterpret_cast<float*>(lds4);
    c.hist = reinterpret_cast<uint64_t*>(reinterpret_cast<uint8_t*>(lds4) + nm.hist_off);
    double* pw = reinterpret_cast<double*>(c.hist + static_cast<size_t>(c.buckets) * c.groups);
    c.pw = pw;
    c.gs = pw + 33;
    const int64_t t0 = a->t0 + (a->t_dev ? static_cast<int64_t>(*a->t_dev) : 0);   // graph replays read the step
    const int64_t t1 = t0 + a->n_steps;
    const int threads = c.waves * 64, me = c.wave * 64 + c.lane;
    const int ring_words = static_cast<int>(c.slots * c.stride), hist_words = static_cast<int>(c.buckets) * c.groups;
    {
        const float* from = a->ring + nm.ring_at;
        for (int i = me; i < ring_words; i += threads) c.ring[i] = from[i];
        const uint64_t* hfrom = a->hist + nm.hist_at;
        for (int i = me; i < hist_words; i += threads) c.hist[i] = hfrom[i];
        if (c.obs && me < 33) {
            const double rho = 1.0 - p.dt_d / p.tau_c_d;
            double x = 1.0, sum = 0.0;
            for (int m = 0; m < me; ++m) {
                sum += x;
                x *= rho;
            }
            pw[me] = x;
            pw[33 + me] = sum;
        }
    }
    const bool izh = kModels >= 1 && p.model == NET_MODEL_IZHIKEVICH;
    const bool hh = kModels >= 2 && p.model == NET_MODEL_HODGKIN_HUXLEY;
    PushState<VPT, (kModels >= 1)> S;
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
        const int j = (c.wave + q * c.waves) * 64 + c.lane;
        const bool valid = j < c.n;
        const int64_t u = nm.node_off + (valid ? j : 0);
        S.V[q] = valid ? a->V[u] : __builtin_nanf("");
        // (255 or more steps back: no hold reaches it.  A lane past the last vertex must never be held, which
        // would set its NaN to the reset value, and has no input of its own.)
        const uint32_t age = valid ? (a->age[u] & 0xFFu) : 255u;
        S.last[q] = static_cast<uint32_t>(t0) - age;
        S.jl[q] = static_cast<uint32_t>(a->caller_of ? a->caller_of[u] - nm.node_off : (valid ? j : 0));
        S.thr[q] = valid && a->drive_thr ? a->drive_thr[u] : 0u;
        S.iext[q] = valid && a->i_ext ? a->i_ext[u] : 0.0f;
        S.bits[q] = S.pm[q] = 0u;
        S.cal[q] = S.acc[q] = 0.0;
        if (c.obs) {
            S.cal[q] = a->calcium[u];
            S.acc[q] = a->frame_acc[u];
        }
        if constexpr (kModels >= 1) {
            S.st[q] = HhState{};
            if (izh) {
                S.st[q].v = a->Vd[u];
                S.st[q].m = a->Wd[u];
            }
            if (hh) S.st[q] = HhState{a->Vd[u], a->hh_vprev[u], a->hh_m[u], a->hh_n[u], a->hh_h[u], 0.0, 0.0};
            if (izh || hh) {
                S.st[q].r = a->psc_r[u];
                S.st[q].p = a->psc_p[u];
            }
            if (!valid) S.st[q].v = __builtin_nan("");
        }
    }
    lds_barrier();
    // the first step's spikes
    {
        const uint32_t bucket = static_cast<uint32_t>(static_cast<uint64_t>(t0) % c.buckets);
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            bool spike;
            if (kModels >= 2 && hh) spike = push_spikes<(kModels >= 2 ? NET_MODEL_HODGKIN_HUXLEY : NET_MODEL_LIF)>(S, q, p);
            else if (kModels >= 1 && izh) spike = push_spikes<(kModels >= 1 ? NET_MODEL_IZHIKEVICH : NET_MODEL_LIF)>(S, q, p);
            else spike = push_spikes<NET_MODEL_LIF>(S, q, p);
            const uint64_t spk = wave_ballot(spike);
            if (q < c.nq && c.lane == 0) c.hist[bucket * static_cast<uint32_t>(c.groups) + c.wave + q * c.waves] = spk;
        }
    }
    lds_barrier();

    const int mode = p.sigma == 0.0f ? kQuiet : (a->noise ? kAhead : kDraws);
    auto run = [&](auto model) {
        constexpr int kModel = decltype(model)::value;
        if (mode == kQuiet) push_run<kModel, kQuiet>(ka, c, p, S, t0, t1);
        else if (mode == kAhead) push_run<kModel, kAhead>(ka, c, p, S, t0, t1);
        else push_run<kModel, kDraws>(ka, c, p, S, t0, t1);
    };
    if constexpr (kModels >= 2) {
        if (hh) run(std::integral_constant<int, NET_MODEL_HODGKIN_HUXLEY>{});
    }
    if constexpr (kModels >= 1) {
        if (izh) run(std::integral_constant<int, NET_MODEL_IZHIKEVICH>{});
    }
    if (!izh && !hh) run(std::integral_constant<int, NET_MODEL_LIF>{});

    // ---- state back to memory
    a = reread(ka);
    for (int i = me; i < ring_words; i += threads) a->ring[nm.ring_at + i] = c.ring[i];
    for (int i = me; i < hist_words; i += threads) a->hist[nm.hist_at + i] = c.hist[i];
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
        const int j = (c.wave + q * c.waves) * 64 + c.lane;
        if (j >= c.n) continue;
        const int64_t u = nm.node_off + j;
        const uint32_t since = static_cast<uint32_t>(t1) - S.last[q];
        a->V[u] = S.V[q];
        a->age[u] = static_cast<uint16_t>(since < 255u ? since : 255u);
        if (c.obs) {
            a->calcium[u] = S.cal[q];
            a->frame_acc[u] = S.acc[q];
        }
        if constexpr (kModels >= 1) {
            if (izh) {
                a->Vd[u] = S.st[q].v;
                a->Wd[u] = S.st[q].m;
            }
            if (hh) {
                a->Vd[u] = S.st[q].v;
                a->hh_vprev[u] = S.st[q].vprev;
                a->hh_m[u] = S.st[q].m;
                a->hh_n[u] = S.st[q].n;
                a->hh_h[u] = S.st[q].h;
            }
            if (izh || hh) {
                a->psc_r[u] = S.st[q].r;
                a->psc_p[u] = S.st[q].p;
            }
        }
    }
}

// Noise and control pulses of `n_steps` steps drawn ahead, one wave per group
// of 64 vertices and step, for ensembles that leave most of the chip idle: a
// network's workgroup then loads what would take its CU an FP64 Box-Muller and
// a Philox block (about 1,500 cycles) per 64 vertices and step.  40 noisy
// networks of up to 1,000 vertices, us per step, drawn in the steps and ahead:
// Izhikevich 9.2 and 7.6, Hodgkin-Huxley 7.9 and 6.1.
__global__ void __launch_bounds__(256) noise_kernel(PushArgs a, const int32_t* group_net) {
    const int lane = threadIdx.x & 63;
    const int64_t per_step = a.noise_stride >> 6;
    const int64_t at = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (at >= per_step * a.n_steps) return;
    const int64_t s = at / per_step;
    const int group = static_cast<int>(at - s * per_step);
    const PushNet& nm = a.nets[group_net[group]];
    const NetParams& p = a.params[nm.net];
    if (p.sigma == 0.0f) return;
    const int j = group * 64 - nm.noise_at + lane;
    const int64_t u = nm.node_off + (j < nm.n ? j : 0);
    const uint64_t t = static_cast<uint64_t>(a.t0 + (a.t_dev ? static_cast<int64_t>(*a.t_dev) : 0) + s);
    const uint32_t jl = static_cast<uint32_t>(a.caller_of ? a.caller_of[u] - nm.node_off : u - nm.node_off);
    const uint4 r = philox4x32_10(make_uint4(jl, static_cast<uint32_t>(t), static_cast<uint32_t>(t >> 32), 0u),
                                  p.key_lo, p.key_hi);
    const double x = p.model == NET_MODEL_LIF ? static_cast<double>(p.sigma * gaussian(r.y, r.z))
                                              : static_cast<double>(p.sigma) * gaussian_d(r.y, r.z);
    a.noise[s * a.noise_stride + group * 64 + lane] = x;
    const uint64_t pulse = wave_ballot(a.drive_thr && r.x < a.drive_thr[u]);
    if (lane == 0) a.noise_pulses[s * per_step + group] = pulse;
}

typedef void (*PushKernel)(PushArgs);

PushKernel push_kernel(int models, int vpt) {
#define GEONET_PUSH(M, T) (vpt == 1 ? push_ensemble_kernel<M, 1, T> : vpt == 2 ? push_ensemble_kernel<M, 2, T> : push_ensemble_kernel<M, 4, T>)
    if (models == 2) return GEONET_PUSH(2, kPushThreadsFp64);
    if (models == 1) return GEONET_PUSH(1, kPushThreadsFp64);
    return vpt == 8 ? push_ensemble_kernel<0, 8, kPushThreads> : GEONET_PUSH(0, kPushThreads);
#undef GEONET_PUSH
}

}  // namespace

// (the same for every handle: the attribute is the kernel's)
hipError_t enable_push_ensemble(int models, int vpt) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(push_kernel(models, vpt)),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kPushMaxLds));
}

hipError_t launch_push_ensemble(const DeviceGraph& g, const EnsemblePlan& plan, int64_t t0, int32_t n_steps,
                                const net_record* rec, int32_t frame_num, int32_t frame_den, hipStream_t s,
                                hipEvent_t ev0, hipEvent_t ev1) {
    PushArgs a;
    a.nets = plan.push_nets;
    a.off = plan.push_off;
    a.edge = plan.push_edge;
    a.ring = plan.push_ring;
    a.hist = plan.push_hist;
    a.params = g.params;
    a.drive_thr = g.drive_thr;
    a.i_ext = g.i_ext;
    a.V = g.V;
    a.age = g.age;
    a.calcium = (g.calcium && frame_num > 0) ? g.calcium : nullptr;
    a.frame_acc = g.frame_acc;
    a.frames = g.frames;
    a.rec_raster = rec ? rec->raster : nullptr;
    a.rec_v = rec ? rec->v : nullptr;
    a.rec_input = rec ? rec->input : nullptr;
    a.Vd = g.Vd;
    a.Wd = g.Wd;
    a.psc_r = g.psc_r;
    a.psc_p = g.psc_p;
    a.hh_m = g.hh_m;
    a.hh_n = g.hh_n;
    a.hh_h = g.hh_h;
    a.hh_vprev = g.hh_vprev;
    a.caller_of = g.caller_of;
    a.t_dev = g.t_dev;
    a.noise = nullptr;
    a.noise_pulses = nullptr;
    a.noise_stride = plan.noise_stride;
    a.t0 = t0;
    a.n_total = g.n_total;
    a.n_pad = g.n_pad;
    a.raster_words = (g.n_total + 63) / 64;
    a.n_steps = n_steps;
    a.frame_cap = g.frame_cap;
    a.frame_num = frame_num > 0 ? frame_num : 1;
    a.frame_den = frame_den > 0 ? frame_den : 1;
    const int models = g.hh_m ? 2 : (g.Vd ? 1 : 0);
    const PushKernel kernel = push_kernel(models, plan.vpt);
    const dim3 grid(plan.blocks), block(plan.threads);
    if (!plan.noise || n_steps < kNoiseMinSteps) {
        hipExtLaunchKernelGGL(kernel, grid, block, plan.lds_bytes, s, ev0, ev1, 0, a);
        return hipGetLastError();
    }
    // the noise of as many steps as its buffer holds, then those steps
    a.noise = plan.noise;
    a.noise_pulses = plan.noise_pulses;
    for (int32_t done = 0; done < n_steps; done += plan.noise_steps) {
        const bool last = n_steps - done <= plan.noise_steps;
        a.t0 = t0 + done;
        a.n_steps = last ? n_steps - done : plan.noise_steps;
        a.rec_raster = rec && rec->raster ? rec->raster + done * a.raster_words : nullptr;
        a.rec_v = rec && rec->v ? rec->v + done * a.n_total : nullptr;
        a.rec_input = rec && rec->input ? rec->input + done * a.n_total : nullptr;
        const int64_t waves = (a.noise_stride >> 6) * a.n_steps;
        hipExtLaunchKernelGGL(noise_kernel, dim3(static_cast<unsigned>((waves + 3) / 4)), dim3(256), 0, s,
                              done == 0 ? ev0 : nullptr, nullptr, 0, a, plan.noise_nets);
        hipExtLaunchKernelGGL(kernel, grid, block, plan.lds_bytes, s, nullptr, last ? ev1 : nullptr, 0, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

}  // namespace geonet
