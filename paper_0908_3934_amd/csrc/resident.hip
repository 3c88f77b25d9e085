// One large LIF network resident on the chip for all steps of a call: every
// workgroup owns a range of vertices (state in registers, arriving input in
// LDS) and the workgroups exchange each step's spikes through memory.
//
// Exchange.  A workgroup publishes its spikes of step t + 1 as soon as step t
// has updated its vertices, before it looks at the others' spikes of step t
// (which step t + 1's input needs, but not step t's): a word with a tag of the
// step, their number and up to four vertex indices; up to three more are in a
// second word, and where still more fire, one tagged word per 32 vertices.
// Every workgroup reads every other's word, again until its tag is the step's,
// and the others as the number says.  A word is one 8-byte access, so it needs
// no order towards any other.  Four sets of words in turn are enough: a
// workgroup publishes t + 2 after it has read all words of t, whose owners had
// read all words of t - 2 before they published them.
//
// Start.  The launch is cooperative, which gives every workgroup its place on an
// idle chip, but one that another stream's kernels fill takes them in as those
// end.  So each marks a word of its own when it starts, and nothing of the state
// changes before it has seen every other's mark.  One that has waited for a
// second closes the first word that is still unmarked: if that succeeds, its
// owner cannot mark it any more and nobody sees all marks, so it does all the
// steps by itself (run_alone), and whoever meets the closed word leaves.  All
// words before a closed one are marked, so there is at most one.  (A call of 128
// steps, 256 workgroups: 2.4 us for these words; one count that all add to takes
// 5.4.)  From then on all run, and waits end within microseconds; should one
// reach its limit all the same (polls for seconds), the launch ends, what it
// leaves is marked (V and the rest of the records NaN or all ones, and every
// later read-out NaN) and the handle fails.
//
// Delivery.  Out-edges are kept by (set of workgroups, source, workgroup of the
// target), so a workgroup finds its part of a spike's edges with one load of
// two offsets.  A set is the workgroups of one XCD (block b runs on XCD b mod
// 8), next to each other in vertex order: they look up the same sources at the
// same time, and a source's offsets for all of them are one line of their L2.
// Arrivals up to W steps ahead are added into LDS as integers in units of the
// weights' smallest FP16 spacing (exact, as the FP32 sums are; see
// ensemble_push.hip for the LDS atomics' cost); later ones go into the ring of
// arrival steps in memory that push delivery uses, whose slot of step t + W
// the owner takes over at step t.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"
#include "philox.h"
#include "vertex.h"

namespace geonet {
namespace {

constexpr int kHeadIds = 4, kMoreIds = 3;         // vertex indices in the first and in the second word
// First words stand 128 bytes apart: in a shared line one workgroup's store
// waits for the others' and for every poll of them (an exchange alone among 256
// workgroups: 1.12 us against 1.67 with 16 words a line; among 32, 0.99 against
// 1.33).
constexpr int kHeadStep = 16;
constexpr int kSets = 4;                          // sets of words in turn (see above)
constexpr uint32_t kMoreTag = 0x7FFFFFFFu;        // (a second word may stand for long: a long tag)
constexpr int kListWords = 64 * kHeadIds + 128;   // a wave's list of spikes, of workgroups, and deliver_spikes' words
constexpr uint32_t kHeadMany = 15u;               // its count where they do not fit
constexpr uint32_t kFar = kResidentFar;
constexpr uint32_t kNoEdge = 0xFFFFFFFFu;
constexpr uint32_t kSpinLimit = 1u << 22;         // polls (a few seconds)
constexpr uint64_t kStartTicks = 100000000u;      // of the 100 MHz clock
// Words of `gate`, 128 bytes apart: every workgroup's start (2 x the launch's
// number, or that and 1: closed), one that nobody marks, and whether a launch
// gave up.
constexpr int kGateStep = 16;
enum { kRun = 0, kLeave = 1, kLate = 2, kAlone = 4, kLost = 8 };      // bits: what a workgroup's waves saw

struct RunArgs {
    const uint32_t* __restrict__ off;   // [sets][n_total][set_groups] and one more: first edge
    const uint2* __restrict__ edge;     // (delay n_local + target in the group, or for delays beyond the window kFar |
                                        // delay << 16 | target; weight in units)
    float* ring;                        // [ring_mask + 1][n_pad] arrivals by step
    uint64_t* head;                     // [kSets][groups] first words, kHeadStep apart
    uint64_t* more;                     // [kSets][groups] second words, then [kSets][groups][n_local / 32] words of spike bits
    uint64_t* gate;
    uint32_t* fail;                     // host memory: set where a wait reached its limit
    float* __restrict__ V;
    uint16_t* __restrict__ age;
    uint32_t* __restrict__ hist;        // pull delivery's spike history and summary (else null)
    uint32_t* __restrict__ summary;
    const uint32_t* __restrict__ drive_thr;
    const float* __restrict__ i_ext;
    double* __restrict__ calcium;
    double* __restrict__ frame_acc;
    float* __restrict__ frames;
    uint64_t* __restrict__ rec_raster;
    float* __restrict__ rec_v;
    float* __restrict__ rec_input;
    const int32_t* __restrict__ caller_of;
    const NetParams* __restrict__ params;
    // plastic networks (else null): per slot source | delay << 16 | target in its
    // group << 24 (kNoEdge: none), weights in 2^-20, each row's first slot, the
    // last kStdpHist spike steps of every vertex (kNoSpike: none) and their count
    const uint32_t* __restrict__ info;
    int32_t* wq;
    const int32_t* __restrict__ row_first;
    int32_t* spk_hist;
    int32_t* spk_cnt;
    double dt, alpha, beta;
    int64_t t0, n_total, n_pad, raster_words;
    uint64_t launch;                    // 2 x the launch's number
    uint32_t simulate;                  // NET_LOST_*
    uint32_t ring_mask, seq0;
    int32_t words;                      // of a step's arrivals, a bit per slot of the group
    int32_t n_steps, n_local, set_groups, window, max_delay, d_sum, sum_shift, frame_cap, frame_num, frame_den;
    float unit, inv_unit;
};

typedef const RunArgs __attribute__((address_space(4)))* const_args;

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Polls a published word until the low `bits` bits of it are the tag.
__device__ __forceinline__ uint64_t poll_word(const uint64_t* at, bool want, uint32_t tag, uint32_t tag_mask, bool* dead) {
    uint64_t v = tag;
    bool wait = want;
#pragma unroll 1
    for (uint32_t spin = 0; wave_ballot(wait) != 0; ++spin) {
        if (wait) {
            v = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait = (static_cast<uint32_t>(v) & tag_mask) != tag;
        }
        if (*dead || spin >= kSpinLimit) {
            *dead = true;
            break;
        }
    }
    return wait ? tag : v;       // (given up: no spikes)
}

struct RunCtx {
    const uint32_t* off;     // this workgroup's offsets, `step` apart
    uint32_t step;
    const uint2* edge;
    float* ring;             // this workgroup's first vertex in the ring's slot 0
    int* slots;
    int64_t n_pad;
    uint32_t ring_mask, size;   // (W + 1) n_local
    int lane;
    float unit;
};

// `now`: slot of step t x the slot's size (n_local, or the bits of its words)
template <bool kPlastic>
__device__ __forceinline__ void add_edge(const RunCtx& c, uint2 e, uint32_t now, uint32_t t) {
    if constexpr (kPlastic) {
        // the edge's bit in its arrival step's words
        uint32_t at = now + e.x;
        at = at < at - c.size ? at : at - c.size;
        atomicOr(reinterpret_cast<uint32_t*>(c.slots) + (at >> 5), 1u << (at & 31u));
        (void)t;
    } else if (!(e.x & kFar)) {
        const uint32_t at = now + e.x;
        atomicAdd(c.slots + (at < at - c.size ? at : at - c.size), static_cast<int>(e.y));
    } else {
        // (only this workgroup's waves touch these entries while the kernel runs)
        const uint32_t d = (e.x >> 16) & 0xFFu, to = e.x & 0xFFFFu;
        __hip_atomic_fetch_add(c.ring + static_cast<int64_t>((t + d) & c.ring_mask) * c.n_pad + to,
                               static_cast<float>(static_cast<int>(e.y)) * c.unit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Time since vertex i's last spike before step u (0 for u <= 0, u dt before any
// spike).  Its owner may be adding spikes of steps near t, which are not before
// u, in place of ones too old to be asked for.
__device__ __forceinline__ double since_spike(const int32_t* hist, int64_t i, int64_t u, double dt) {
    if (u <= 0) return 0.0;
    const uint64_t* h = reinterpret_cast<const uint64_t*>(hist + i * kStdpHist);
    uint64_t two[kStdpHist / 2];
#pragma unroll
    for (int q = 0; q < kStdpHist / 2; ++q) two[q] = __hip_atomic_load(h + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int64_t best = -1;
#pragma unroll
    for (int q = 0; q < kStdpHist / 2; ++q) {
        const int64_t a = static_cast<int32_t>(two[q]), b = static_cast<int32_t>(two[q] >> 32);
        best = a < u && a > best ? a : best;
        best = b < u && b > best ? b : best;
    }
    return best < 0 ? static_cast<double>(u) * dt : static_cast<double>(u - best - 1) * dt;
}

// Delivers this workgroup's part of up to 64 spikes, one per lane (`have`).
// Most have no edge here or a few: the edges of all lists are numbered through,
// and the wave takes 64 of them at a time, four such loads in flight (`flat`:
// 64 words of the wave's own).  With a lane per list up to four edges long and
// the wave per longer one, a step of 262,144 vertices with 11,750 spikes took
// 87 us, now 78 (65,536 vertices with 2,890 spikes: 25.3 and 19.5).
template <bool kPlastic>
__device__ __forceinline__ void deliver_spikes(const RunCtx& c, bool have, uint32_t src, uint32_t now, uint32_t t, uint32_t* flat) {
    constexpr int kLoads = 4;
    uint32_t e0 = 0u, len = 0u;
    if (have) {
        uint32_t range[2];
        __builtin_memcpy(range, c.off + static_cast<size_t>(src) * c.step, sizeof(range));
        e0 = range[0];
        len = range[1] - range[0];
    }
    const uint64_t lists = wave_ballot(len != 0u);
    if (lists == 0) return;
    uint32_t total;
    const uint32_t at = wave_prefix(len, &total);                      // the number of the list's first edge
    const bool one = (lists & (lists - 1)) == 0;
    const uint32_t e_one = __builtin_amdgcn_readlane(e0, __builtin_ctzll(lists));
    const uint32_t lane = static_cast<uint32_t>(c.lane);
    for (uint32_t n0 = 0; n0 < total; n0 += 64u * kLoads) {
        uint2 rec[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const uint32_t n = n0 + 64u * q;
            rec[q] = make_uint2(0u, 0u);
            if (n >= total) continue;
            uint32_t e = e_one + n + lane;
            if (!one) {
                // the first edge here of every list that reaches into these 64, at its place;
                // the others follow the nearest one below them
                flat[lane] = ~0u;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                const uint32_t lo = at > n ? at : n;
                if (len != 0u && lo < n + 64u && at + len > n) flat[lo - n] = e0 + (lo - at);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                const uint32_t x = flat[lane];
                const uint64_t heads = wave_ballot(x != ~0u);
                const int head = 63 - __builtin_clzll(heads & (~0ull >> (63 - c.lane)));
                e = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(head << 2, static_cast<int>(x))) + (lane - static_cast<uint32_t>(head));
            }
            if (n + lane < total) rec[q] = c.edge[e];
        }
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            if (n0 + 64u * q >= total) break;
            if (rec[q].y != 0u) add_edge<kPlastic>(c, rec[q], now, t);
        }
    }
}

// Weight e of an edge (`info`) whose spike arrived at step `now`, or whose
// target, with its last spike before at step tl (-1: none), fired there.
__device__ __forceinline__ void learn(const RunArgs __attribute__((address_space(4)))& r, int64_t e, uint32_t info, int32_t tl, int64_t now) {
    const int32_t w = r.wq[e];
    const double since = now <= 0 ? 0.0 : (tl < 0 ? static_cast<double>(now) * r.dt : static_cast<double>(now - tl - 1) * r.dt);
    const double q = since_spike(r.spk_hist, info & 0xFFFFu, now - ((info >> 16) & 0xFFu), r.dt) - since;
    const double sg = q > 0.0 ? 1.0 : (q < 0.0 ? -1.0 : 0.0);
    const double dw = r.dt * r.alpha * sg * exp(-r.beta * fabs(q));
    r.wq[e] = w + static_cast<int32_t>(rint(dw * 1048576.0));
}

// One thread, after a second: closes the first word without a mark, unless
// all words have one by now or one is closed.
__device__ uint32_t close_start(uint64_t* gate, uint64_t launch, int words) {
    for (int g = 0; g < words;) {
        uint64_t now = __hip_atomic_load(gate + g * kGateStep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (now > launch) return kLeave;
        if (now == launch) ++g;
        else if (__hip_atomic_compare_exchange_strong(gate + g * kGateStep, &now, launch + 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT))
            return kAlone;
    }
    return kRun;
}

// Marks this workgroup's start and waits for the others': what the workgroup
// has to do (`role`: a word in LDS).
__device__ __forceinline__ uint32_t start_role(const const_args a, uint32_t* role) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = static_cast<int>(blockDim.x >> 6);
    const int groups = static_cast<int>(gridDim.x);
    uint64_t* const gate = a->gate;
    const uint64_t launch = a->launch;
    const bool simulate = a->simulate == NET_LOST_AT_START;
    if (tid == 0) {
        const uint64_t was = __hip_atomic_fetch_max(gate + blockIdx.x * kGateStep, launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t lost = __hip_atomic_load(gate + (groups + 1) * kGateStep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *role = (was > launch ? kLeave : kRun) | (lost != 0 ? kLost : kRun);
    }
    lds_barrier();
    const int g = lane * waves + wave;
    const uint64_t since = wall_clock64();
    uint32_t saw = simulate ? kLate : kRun;
    while (saw == kRun) {
        const uint64_t v = g < groups ? __hip_atomic_load(gate + g * kGateStep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : launch;
        if (wave_ballot(v > launch) != 0) saw = kLeave;
        else if (wave_ballot(v < launch) == 0) break;
        else if (wall_clock64() - since >= kStartTicks) saw = kLate;
    }
    if (lane == 0 && saw != kRun) atomicOr(role, saw);
    lds_barrier();
    uint32_t r = *role;
    lds_barrier();
    if (!(r & kLeave) && (r & kLate)) {
        if (tid == 0) *role = close_start(gate, launch, groups + (simulate ? 1 : 0)) | (r & kLost);
        lds_barrier();
        r = *role;
    }
    return __builtin_amdgcn_readfirstlane(r);
}

// The launch's steps by one workgroup, for a launch whose workgroups did not
// come together: from and to the same state in memory, with the same sums.
// Vertex j is thread j mod blockDim's in every step.  us per step: 8,192 vertices
// 28, 262,144 960; 16,384 with weights that learn 2,600.
template <bool kPlastic>
__device__ __attribute__((noinline)) void run_alone(const const_args a) {
    const uint32_t groups = gridDim.x;
    const NetParams p = load_const(a->params);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, threads = blockDim.x;
    const int64_t n_total = a->n_total, n_pad = a->n_pad;
    const uint32_t sg = static_cast<uint32_t>(a->set_groups), n_local = static_cast<uint32_t>(a->n_local);
    const int32_t n_steps = a->n_steps;
    for (int32_t k = 0; k < n_steps; ++k) {
        const int64_t t64 = a->t0 + k;
        const uint32_t t = static_cast<uint32_t>(t64);
        const int64_t frame = t64 * a->frame_num / a->frame_den;
        const int64_t first = (frame * a->frame_den + a->frame_num - 1) / a->frame_num;
        const bool flush = a->calcium && ((frame + 1) * a->frame_den + a->frame_num - 1) / a->frame_num == t64 + 1;
        for (int64_t j = tid; j - lane < n_total; j += threads) {
            const bool valid = j < n_total;
            bool spike = false;
            if (valid) {
                const uint32_t ages = a->age[j], a1 = ages & 0xFFu, a2 = ages >> 8;
                const float V = a->V[j];
                spike = V >= p.v_th;
                // the step's input
                float in;
                uint32_t* const hist = a->hist ? a->hist + j : nullptr;
                [[maybe_unused]] auto arrives = [&](uint32_t info) {
                    const uint32_t ts = t - ((info >> 16) & 0xFFu);
                    return ((a->hist[static_cast<int64_t>((ts & 0xFFu) >> 5) * n_pad + (info & 0xFFFFu)] >> (ts & 31u)) & 1u) != 0u;
                };
                if constexpr (kPlastic) {
                    long long sum = 0;
                    for (int64_t e = a->row_first[j]; e < a->row_first[j + 1]; ++e) {
                        const uint32_t info = a->info[e];
                        if (info != kNoEdge && arrives(info)) sum += a->wq[e];
                    }
                    in = static_cast<float>(static_cast<double>(sum) * (1.0 / 1048576.0));
                } else {
                    // (the adds of earlier steps are in the L2)
                    in = __hip_atomic_exchange(a->ring + static_cast<int64_t>(t & a->ring_mask) * n_pad + j, 0.0f, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                }
                if (a->rec_v) a->rec_v[static_cast<int64_t>(k) * n_total + j] = V;
                if (a->rec_input) a->rec_input[static_cast<int64_t>(k) * n_total + j] = in;
                const uint32_t thr = a->drive_thr ? a->drive_thr[j] : 0u;
                float u = a->i_ext ? a->i_ext[j] : 0.0f, noise = 0.0f;
                if (thr != 0u || p.sigma != 0.0f) {
                    const uint4 r = philox4x32_10(make_uint4(static_cast<uint32_t>(a->caller_of ? a->caller_of[j] : j), t,
                                                             static_cast<uint32_t>(static_cast<uint64_t>(t64) >> 32), 0u),
                                                  p.key_lo, p.key_hi);
                    u = r.x < thr ? u + p.drive_amp : u;
                    if (p.sigma != 0.0f) noise = p.sigma * gaussian(r.y, r.z);
                }
                const float vn = V + p.decay * (p.v_rest - V) + in + u + noise;
                const bool held = a1 - 1u < static_cast<uint32_t>(p.n_ref);
                a->V[j] = (spike | held) ? p.v_reset : vn;
                const uint32_t o1 = a1 < 255u ? a1 + 1u : 255u, o2 = a2 < 255u ? a2 + 1u : 255u;
                a->age[j] = static_cast<uint16_t>(spike ? 1u | o1 << 8 : o1 | o2 << 8);
                if (a->calcium) {
                    const double cal = a->calcium[j];
                    double acc = a->frame_acc[j] + cal;
                    if (flush) {
                        if (frame < a->frame_cap) a->frames[frame * n_pad + j] = static_cast<float>(acc / static_cast<double>(t64 + 1 - first));
                        acc = 0.0;
                    }
                    a->frame_acc[j] = acc;
                    a->calcium[j] = cal + p.dt_d * (-cal / p.tau_c_d + (spike ? 1.0 : 0.0));
                }
                if (hist) {
                    uint32_t& word = hist[static_cast<int64_t>((t & 0xFFu) >> 5) * n_pad];
                    word = (word & ~(1u << (t & 31u))) | ((spike ? 1u : 0u) << (t & 31u));
                }
                if constexpr (kPlastic) {
                    const int32_t count = a->spk_cnt[j];
                    const int32_t tl = count > 0 ? __hip_atomic_load(a->spk_hist + j * kStdpHist + (count - 1) % kStdpHist, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT)
                                                 : -1;
                    if (spike) {
                        __hip_atomic_store(a->spk_hist + j * kStdpHist + count % kStdpHist, static_cast<int32_t>(t), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                        a->spk_cnt[j] = count + 1;
                    }
                    for (int64_t e = a->row_first[j]; e < a->row_first[j + 1]; ++e) {
                        const uint32_t info = a->info[e];
                        if (info != kNoEdge && (spike || arrives(info))) learn(*a, e, info, tl, t64);
                    }
                }
            }
            const uint64_t spk = wave_ballot(spike);
            if (a->rec_raster && lane == 0) a->rec_raster[static_cast<int64_t>(k) * a->raster_words + (j >> 6)] = spk;
            if constexpr (!kPlastic) {
                for (uint64_t m = spk; m != 0; m &= m - 1) {
                    const int64_t src = j - lane + __builtin_ctzll(m);
                    for (uint32_t g = lane; g < groups; g += 64u) {
                        const int64_t list = (static_cast<int64_t>(g / sg) * n_total + src) * sg + g % sg;
                        for (uint32_t e = a->off[list]; e < a->off[list + 1]; ++e) {
                            const uint2 x = a->edge[e];
                            const uint32_t d = (x.x & kFar) ? (x.x >> 16) & 0xFFu : x.x / n_local;
                            const uint32_t to = g * n_local + ((x.x & kFar) ? x.x & 0xFFFFu : x.x % n_local);
                            __hip_atomic_fetch_add(a->ring + static_cast<int64_t>((t + d) & a->ring_mask) * n_pad + to,
                                                   static_cast<float>(static_cast<int>(x.y)) * a->unit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                    }
                }
            }
        }
        // what the threads left for each other is there before the next step
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
    }
    for (int64_t j = tid; a->summary && j - lane < n_pad; j += threads) {
        const uint64_t recent = wave_ballot(j < n_total && (a->age[j] & 0xFFu) <= static_cast<uint32_t>(a->d_sum));
        if (lane == 0) put_summary(a->summary, j, recent, a->sum_shift);
    }
    // the words' tags as if they had been published: none is taken for a later step's
    const uint32_t end = a->seq0 + static_cast<uint32_t>(n_steps);
    for (uint32_t i = tid; i < kSets * groups; i += threads) {
        const uint32_t set = i / groups, next = end + (set + kSets - end % kSets) % kSets;
        a->head[static_cast<int64_t>(i) * kHeadStep] = (next - kSets) & 0xFFFFu;
    }
}

// What bounds it: the chain of a step, that is the look at the words, the two
// dependent loads of the spikes' edges, the LDS adds, two barriers and the
// update; at 1,024 vertices a CU also the noise (Philox and Box-Muller, 0.3 us a
// wave).  us per step, the per-step kernels, this kernel with the spikes of step t
// published and read within step t, and now (noise 0.05, 3-D, about 100 in-edges
// a vertex, 0.5 spikes a step and 1,000 vertices): 8,192 vertices 7.6 / 2.7 /
// 1.85; 65,536 (pull delivery before) 13.0 / 3.9 / 2.65; 262,144 (push before)
// 6.5 / 4.8 / 4.2.  At the most spikes a network can have (one in 22 vertices a
// step) 8,192: 9.2 / 6.8 / 4.1 (push 7.4), 65,536: 30 / 19.5 / 13.7 (21),
// 262,144: (81) / 78 / 76.
//
// kPlastic: a weight counts as it is when its edge's spike arrives, so a spike
// sets a bit per edge in the words of its arrival step (LDS holds all steps up to
// the largest delay), and step t adds the weights of its bits as integers and
// then, the others' words on their way, updates them and the in-edges of the
// vertices that fire: work per step for the arrivals and spikes instead of every
// edge.  16,384 vertices, 1.2e6 edges: 16.7 us a step with a kernel over all
// edges and one over all vertices, now 3.9.
template <bool kPlastic>
__global__ void __launch_bounds__(1024) run_kernel(RunArgs args) {
    extern __shared__ uint4 lds4[];
    __shared__ uint64_t s_words[2][16];
    __shared__ uint32_t s_dead, s_role;
    (void)args;
    const const_args ka = (const_args)__builtin_amdgcn_kernarg_segment_ptr();
    // ---- nothing is written before all workgroups have started
    const uint32_t role = start_role(reread(ka), &s_role);
    if (role & kLeave) return;
    if (role & kAlone) {
        run_alone<kPlastic>(reread(ka));
        return;
    }
    const_args a = reread(ka);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = static_cast<int>(blockDim.x >> 6);
    const int groups = static_cast<int>(gridDim.x), sets = groups / a->set_groups;
    const int set = static_cast<int>(blockIdx.x) % sets, in_set = static_cast<int>(blockIdx.x) / sets;
    const int b = set * a->set_groups + in_set;                        // this workgroup's place in vertex order
    const uint32_t W = static_cast<uint32_t>(a->window);
    const int n_local = a->n_local;
    const int own_words = n_local >> 6;                                 // words of 64 vertices; wave w has w, w + waves, ..
    const int64_t n_total = a->n_total, j0 = static_cast<int64_t>(b) * n_local;
    const NetParams p = load_const(a->params);
    RunCtx c;
    c.off = a->off + static_cast<int64_t>(set) * n_total * a->set_groups + in_set;
    c.step = static_cast<uint32_t>(a->set_groups);
    c.edge = a->edge;
    c.ring = a->ring + j0;
    c.slots = reinterpret_cast<int*>(lds4);
    c.n_pad = a->n_pad;
    c.ring_mask = a->ring_mask;
    const uint32_t slot_words = kPlastic ? static_cast<uint32_t>(a->words) : static_cast<uint32_t>(n_local);
    const uint32_t slot_size = kPlastic ? slot_words * 32u : slot_words;
    c.size = (W + 1u) * slot_size;
    c.lane = lane;
    c.unit = a->unit;
    const float inv_unit = a->inv_unit;
    uint32_t* const lists = reinterpret_cast<uint32_t*>(c.slots + (((W + 1u) * slot_words + 1u) & ~1u));
    uint32_t* list = lists + wave * kListWords;
    // plastic networks: the step's input sums, and each vertex's last spike before the step (-1: none)
    unsigned long long* const sums = reinterpret_cast<unsigned long long*>(lists + waves * kListWords);
    int32_t* const tlast = reinterpret_cast<int32_t*>(sums + n_local);
    const int64_t first_slot = kPlastic ? a->row_first[j0 < n_total ? j0 : n_total] : 0;
    uint32_t *who = list + 64 * kHeadIds, *flat = who + 64;
    const uint32_t many_words = static_cast<uint32_t>(n_local) >> 5;
    const int64_t t0_64 = a->t0;
    const uint32_t t0 = static_cast<uint32_t>(t0_64), seq0 = a->seq0;

    const int32_t n_steps = a->n_steps;

    // ---- state in: the arrivals of steps t0 .. t0 + W - 1 move to LDS
    if (tid == 0) s_dead = role & kLost || a->simulate == NET_LOST_IN_STEP ? 1u : 0u;
    const uint32_t slot0 = static_cast<uint32_t>(static_cast<uint64_t>(t0_64) % (W + 1u));
    const uint32_t quads = static_cast<uint32_t>(n_local) >> 2;         // (four vertices at a time, four such loads in flight)
    for (uint32_t i0 = tid; !kPlastic && i0 < (W + 1u) * quads; i0 += 4u * blockDim.x) {
        float4 x[4];
        float4* at[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t i = i0 + q * blockDim.x, k = i / quads, v = (i - k * quads) * 4u;
            x[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            at[q] = reinterpret_cast<float4*>(c.ring + static_cast<int64_t>((t0 + k) & c.ring_mask) * c.n_pad + v);
            if (k < W && j0 + v < c.n_pad) x[q] = *at[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t i = i0 + q * blockDim.x, k = i / quads, v = (i - k * quads) * 4u;
            if (k > W) continue;
            if (x[q].x != 0.0f || x[q].y != 0.0f || x[q].z != 0.0f || x[q].w != 0.0f) *at[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const uint32_t s = slot0 + k > W ? slot0 + k - (W + 1u) : slot0 + k;
            *reinterpret_cast<int4*>(c.slots + s * static_cast<uint32_t>(n_local) + v) =
                make_int4(static_cast<int>(x[q].x * inv_unit), static_cast<int>(x[q].y * inv_unit),
                          static_cast<int>(x[q].z * inv_unit), static_cast<int>(x[q].w * inv_unit));
        }
    }
    if constexpr (kPlastic) {
        // the arrivals to come, from the spikes of the last steps
        for (uint32_t i = tid; i < (W + 1u) * slot_words; i += blockDim.x) c.slots[i] = 0;
        if (tid < n_local) sums[tid] = 0u;
        lds_barrier();
        const int64_t slots_here = a->row_first[j0 + n_local < n_total ? j0 + n_local : n_total] - first_slot;
        for (int64_t rel = tid; rel < slots_here; rel += blockDim.x) {
            const uint32_t info = a->info[first_slot + rel];
            if (info == kNoEdge) continue;
            const uint32_t src = info & 0xFFFFu, d = (info >> 16) & 0xFFu;
            if ((a->age[src] & 0xFFu) > d) continue;
            for (uint32_t back = 1; back <= d; ++back) {
                const uint32_t ts = t0 - back;
                if (!((a->hist[static_cast<int64_t>((ts & 0xFFu) >> 5) * c.n_pad + src] >> (ts & 31u)) & 1u)) continue;
                add_edge<true>(c, make_uint2((d - back) * slot_size + static_cast<uint32_t>(rel), 1u), slot0 * slot_size, 0u);
            }
        }
    }
    // (255 or more steps back: as good as never)
    const bool obs = a->calcium != nullptr, pulls = a->hist != nullptr;
    const int64_t j = j0 + tid;                                         // this thread's vertex
    const bool owns = wave < own_words, valid = owns && j < n_total;
    float V = 0.0f, iext = 0.0f;
    uint32_t last = t0 - 255u, prev = t0 - 255u, thr = 0u, jl = 0u, bits = 0u;
    double cal = 0.0, acc = 0.0;
    if (valid) {
        V = a->V[j];
        const uint32_t ages = a->age[j];
        last = t0 - (ages & 0xFFu);
        prev = t0 - (ages >> 8);
        thr = a->drive_thr ? a->drive_thr[j] : 0u;
        iext = a->i_ext ? a->i_ext[j] : 0.0f;
        jl = static_cast<uint32_t>(a->caller_of ? a->caller_of[j] : j);
        if (pulls) bits = a->hist[static_cast<int64_t>((t0 & 0xFFu) >> 5) * c.n_pad + j];
        if (obs) {
            cal = a->calcium[j];
            acc = a->frame_acc[j];
        }
    }
    int32_t last_at = -1, count = 0;                                    // plastic networks: the last spike's step, spikes so far
    if (kPlastic && valid) {
        count = a->spk_cnt[j];
        for (int q = 0; q < kStdpHist && q < count; ++q) {
            const int32_t ts = a->spk_hist[j * kStdpHist + q];
            last_at = ts > last_at ? ts : last_at;
        }
    }
    uint64_t spk = wave_ballot(valid && V >= p.v_th);                   // this wave's spikes of the step to come
    const bool draws = owns && (wave_ballot(thr != 0u) != 0 || p.sigma != 0.0f);
    const bool far = static_cast<uint32_t>(a->max_delay) > W;
    uint64_t* raster = a->rec_raster && owns && lane == 0 && j < n_total ? a->rec_raster + (j >> 6) : nullptr;
    const int64_t raster_words = a->raster_words;
    const uint32_t records = a->rec_v || a->rec_input ? 1u : 0u;       // (opaque in the loop: not copied for both cases)
    uint64_t* const head = a->head;
    // the workgroup whose word this lane reads: every wave has as many, from all
    // over the network and from no regular places of it, since this one's
    // neighbours, in vertex order a power of two away, have the long lists
    const int asks = lane * waves + (wave + 5 * lane) % waves;
    const bool want = lane < (groups + waves - 1) / waves && asks < groups;
    const int my_group = want ? asks : 0;
    uint32_t slot = slot0;
    int64_t frame = 0, next_flush = INT64_MAX, frame_first = 0;
    if (obs) {
        frame = t0_64 * a->frame_num / a->frame_den;
        frame_first = (frame * a->frame_den + a->frame_num - 1) / a->frame_num;
        next_flush = ((frame + 1) * a->frame_den + a->frame_num - 1) / a->frame_num;
    }

    // this workgroup's spikes of the step whose sequence number is `seq`
    auto publish = [&](uint32_t seq) {
        const uint32_t set_of = seq % kSets;
        if (lane == 0 && owns) s_words[seq & 1u][wave] = spk;
        lds_barrier();
        if (wave != 0) return;
        const uint64_t word = lane < own_words ? s_words[seq & 1u][lane] : 0;
        uint64_t some = wave_ballot(word != 0);
        uint64_t h0 = 0, h1 = 0;                                        // count from bit 16, indices from bits 20 and 31
        uint32_t n = 0;
        for (; some != 0 && n <= kHeadIds + kMoreIds; some &= some - 1) {
            const int w = __builtin_ctzll(some);
            for (uint64_t m = read_lane64(word, w); m != 0 && n <= kHeadIds + kMoreIds; m &= m - 1, ++n) {
                const uint64_t id = static_cast<uint64_t>(w * 64 + __builtin_ctzll(m));
                if (n < kHeadIds) h0 |= id << (20 + 11 * n);
                else if (n < kHeadIds + kMoreIds) h1 |= id << (31 + 11 * (n - kHeadIds));
            }
        }
        h0 |= static_cast<uint64_t>(n > kHeadIds + kMoreIds ? kHeadMany : n) << 16;
        if (n > kHeadIds) {
            // more than the first word holds: the second, or all words
            uint64_t* const more = reread(ka)->more;
            if (n <= kHeadIds + kMoreIds) {
                if (lane == 0)
                    __hip_atomic_store(more + static_cast<int64_t>(set_of) * groups + b, h1 | (seq & kMoreTag), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            } else if (lane < own_words) {
                uint64_t* to = more + kSets * groups + (static_cast<int64_t>(set_of) * groups + b) * (n_local >> 5) + 2 * lane;
                __hip_atomic_store(to, word << 32 | (seq & kMoreTag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(to + 1, (word >> 32) << 32 | (seq & kMoreTag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (lane == 0)
            __hip_atomic_store(head + (static_cast<int>(set_of) * groups + b) * kHeadStep, h0 | (seq & 0xFFFFu), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    };
    // control pulse and noise of step t0 + k
    float noise = 0.0f;
    bool pulse = false;
    auto draw = [&](int32_t k) {
        if (!draws) return;
        const uint64_t t = static_cast<uint64_t>(t0_64 + k);
        const uint4 r = philox4x32_10(make_uint4(jl, static_cast<uint32_t>(t), static_cast<uint32_t>(t >> 32), 0u),
                                      opaque(p.key_lo), opaque(p.key_hi));
        pulse = r.x < thr;
        if (p.sigma != 0.0f) noise = p.sigma * gaussian(r.y, r.z);
    };
    draw(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                    // the ring's entries taken over are cleared
    publish(seq0);

    int32_t row = 0;
    for (int32_t k = 0; k < n_steps; ++k) {
        const uint32_t seq = seq0 + static_cast<uint32_t>(k), par = seq % kSets;
        const uint32_t t = t0 + static_cast<uint32_t>(k);
        // ---- plastic networks: the weights of this step's arrivals
        uint32_t arrived = 0u;
        if constexpr (kPlastic) {
            if (static_cast<uint32_t>(tid) < slot_words)
                arrived = __hip_atomic_exchange(reinterpret_cast<uint32_t*>(c.slots) + slot * slot_words + tid, 0u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
            const const_args r = reread(ka);
            for (uint32_t m = arrived; m != 0u; m &= m - 1u) {
                const int64_t e = first_slot + tid * 32 + __builtin_ctz(m);
                atomicAdd(sums + (r->info[e] >> 24), static_cast<unsigned long long>(static_cast<long long>(r->wq[e])));
            }
            lds_barrier();
        }
        // ---- vertex update
        if (owns) {
            float in;
            if constexpr (kPlastic) {
                const long long got = static_cast<long long>(__hip_atomic_exchange(sums + tid, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                in = static_cast<float>(static_cast<double>(got) * (1.0 / 1048576.0));
                tlast[tid] = last_at;
            } else {
            const int got = __hip_atomic_exchange(c.slots + slot * static_cast<uint32_t>(n_local) + tid, 0, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
            in = static_cast<float>(got) * c.unit;
            }
            const bool spike = ((spk >> lane) & 1u) != 0u;
            if (raster) {
                *raster = spk;
                raster += raster_words;
            }
            if (opaque(records) != 0u && valid) {
                const const_args r = reread(ka);
                if (r->rec_v) r->rec_v[static_cast<int64_t>(row) * n_total + j] = V;
                if (r->rec_input) r->rec_input[static_cast<int64_t>(row) * n_total + j] = in;
            }
            float u = iext;
            u = pulse ? u + p.drive_amp : u;
            const float vn = V + p.decay * (p.v_rest - V) + in + u + noise;
            const bool held = t - last - 1u < static_cast<uint32_t>(p.n_ref);
            V = (spike | held) ? p.v_reset : vn;
            prev = spike ? last : prev;
            last = spike ? t : last;
            bits = (bits & ~(1u << (t & 31u))) | ((spike ? 1u : 0u) << (t & 31u));
            if (obs && valid) {
                acc = acc + cal;
                if (t0_64 + k + 1 == next_flush) {
                    const const_args r = reread(ka);
                    if (frame < r->frame_cap)
                        r->frames[frame * c.n_pad + j] = static_cast<float>(acc / static_cast<double>(next_flush - frame_first));
                    acc = 0.0;
                }
                cal = cal + p.dt_d * (-cal / p.tau_c_d + (spike ? 1.0 : 0.0));
            }
            if (pulls && (t & 31u) == 31u && valid) {
                uint32_t* hist = reread(ka)->hist;
                hist[static_cast<int64_t>((t & 0xFFu) >> 5) * c.n_pad + j] = bits;
                bits = hist[static_cast<int64_t>(((t + 1u) & 0xFFu) >> 5) * c.n_pad + j];
            }
            if constexpr (kPlastic) {
                if (spk != 0) {
                    if (spike) {
                        const const_args r = reread(ka);
                        __hip_atomic_store(r->spk_hist + j * kStdpHist + (count % kStdpHist), static_cast<int32_t>(t), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                        r->spk_cnt[j] = ++count;
                        last_at = static_cast<int32_t>(t);
                    }
                    // there before the next words go out: who has read those finds it
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                }
            }
            spk = wave_ballot(valid && V >= p.v_th);
        }
        if (obs && t0_64 + k + 1 == next_flush) {
            const const_args r = reread(ka);
            frame = next_flush * r->frame_num / r->frame_den;           // (frames shorter than a step: several further)
            frame_first = next_flush;
            next_flush = ((frame + 1) * r->frame_den + r->frame_num - 1) / r->frame_num;
        }
        // the spikes of the next step are on their way while this step's are delivered
        if (k + 1 < n_steps) publish(seq + 1u);
        else if (kPlastic) lds_barrier();                               // (tlast)
        // ---- plastic networks: the edges whose spike arrived or whose target fired
        if constexpr (kPlastic) {
            const const_args r = reread(ka);
            const int64_t now = t0_64 + k;
            const uint64_t* const fired = s_words[seq & 1u];
            for (uint32_t m = arrived; m != 0u; m &= m - 1u) {
                const int64_t e = first_slot + tid * 32 + __builtin_ctz(m);
                const uint32_t info = r->info[e], to = info >> 24;
                if (!((fired[to >> 6] >> (to & 63u)) & 1u)) learn(*r, e, info, tlast[to], now);       // (else with all of its target's below)
            }
            int turn = 0;
            for (int x = 0; x < own_words; ++x) {
                for (uint64_t m = read_lane64(fired[x], 0); m != 0; m &= m - 1) {
                    if (turn++ % waves != wave) continue;
                    const int64_t to = j0 + x * 64 + __builtin_ctzll(m), e1 = r->row_first[to + 1];
                    for (int64_t e = r->row_first[to] + lane; e < e1; e += 64) {
                        const uint32_t info = r->info[e];
                        if (info != kNoEdge) learn(*r, e, info, tlast[info >> 24], now);
                    }
                }
            }
        }
        // ---- every workgroup's spikes of the step: published a step ago, so that
        // the first look mostly finds them; meanwhile the next step's noise, and the
        // ring's arrivals of step t + W (no push reaches that step's entries any more)
        bool dead = false;
        float late = 0.0f;
        {
            const uint64_t* const at = head + (static_cast<int>(par) * groups + my_group) * kHeadStep;
            uint64_t v = want ? __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            if (far && valid)
                late = __hip_atomic_exchange(c.ring + static_cast<int64_t>((t + W) & c.ring_mask) * c.n_pad + tid, 0.0f,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k + 1 < n_steps) draw(k + 1);
            const bool wait = want && (static_cast<uint32_t>(v) & 0xFFFFu) != (seq & 0xFFFFu);
            if (wave_ballot(wait) != 0) {
                const uint64_t got = poll_word(at, wait, seq & 0xFFFFu, 0xFFFFu, &dead);
                v = wait ? got : v;
            }
            const uint32_t n = want ? static_cast<uint32_t>(v >> 16) & 15u : 0u;
            const uint32_t base = static_cast<uint32_t>(my_group * n_local);
            uint32_t total = 0, r0 = 0;                     // the wave's spikes in its list, those delivered
            uint32_t asked = 0, to_ask = 0;                 // words of 32 vertices of the workgroups with too many for theirs
            uint32_t left = 0, left0 = 0;                   // such a word's spikes still to be listed, its first vertex
            bool direct = wave_ballot(n != 0u) != 0;        // a spike per lane at most: straight from the words
            if (wave_ballot(n > 1u) != 0) {
                direct = false;
                const uint32_t in_first = n == kHeadMany ? 0u : (n < kHeadIds ? n : kHeadIds);
#pragma unroll
                for (int q = 0; q < kHeadIds; ++q) {
                    const bool has = static_cast<uint32_t>(q) < in_first;
                    const uint64_t m = wave_ballot(has);
                    if (has) list[total + lanes_below(m)] = base + (static_cast<uint32_t>(v >> (20 + 11 * q)) & 0x7FFu);
                    total += static_cast<uint32_t>(__popcll(m));
                }
                const bool second = n > kHeadIds && n != kHeadMany;
                if (wave_ballot(second) != 0) {
                    const uint64_t v1 = poll_word(reread(ka)->more + static_cast<int64_t>(par) * groups + my_group, second,
                                                  seq & kMoreTag, kMoreTag, &dead);
#pragma unroll
                    for (int q = 0; q < kMoreIds; ++q) {
                        const bool has = second && !dead && q + kHeadIds < n;
                        const uint64_t m = wave_ballot(has);
                        if (has) list[total + lanes_below(m)] = base + (static_cast<uint32_t>(v1 >> (31 + 11 * q)) & 0x7FFu);
                        total += static_cast<uint32_t>(__popcll(m));
                    }
                }
                const uint64_t many = wave_ballot(n == kHeadMany);
                if (n == kHeadMany) who[lanes_below(many)] = static_cast<uint32_t>(my_group);
                to_ask = static_cast<uint32_t>(__popcll(many)) * many_words;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            }
            // up to 64 spikes at a time, one per lane
            while (true) {
                bool have;
                uint32_t src = 0u;
                if (direct) {
                    have = n != 0u;
                    src = base + (static_cast<uint32_t>(v >> 20) & 0x7FFu);
                    direct = false;
                } else if (r0 < total) {
                    have = r0 + lane < total;
                    if (have) src = list[r0 + lane];
                    r0 += 64u;
                } else if (wave_ballot(left != 0u) != 0) {
                    // up to four spikes of every lane's word
                    total = r0 = 0;
#pragma unroll
                    for (int q = 0; q < kHeadIds; ++q) {
                        const uint64_t m = wave_ballot(left != 0u);
                        if (left != 0u) list[total + lanes_below(m)] = left0 + static_cast<uint32_t>(__builtin_ctz(left));
                        left &= left - 1u;
                        total += static_cast<uint32_t>(__popcll(m));
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                    continue;
                } else if (asked < to_ask) {
                    const uint32_t x = asked + static_cast<uint32_t>(lane);
                    const bool mine = x < to_ask;
                    const uint32_t g = who[mine ? x / many_words : 0u], word = x % many_words;
                    const uint64_t w = poll_word(reread(ka)->more + kSets * groups +
                                                     (mine ? (static_cast<int64_t>(par) * groups + g) * many_words + word : 0),
                                                 mine, seq & kMoreTag, kMoreTag, &dead);
                    left = mine ? static_cast<uint32_t>(w >> 32) : 0u;
                    left0 = g * static_cast<uint32_t>(n_local) + word * 32u;
                    asked += 64u;
                    continue;
                } else {
                    break;
                }
                deliver_spikes<kPlastic>(c, have, src, slot * slot_size, t, flat);
            }
        }
        if (late != 0.0f) {
            const uint32_t to = slot == 0u ? W : slot - 1u;             // slot of step t + W
            atomicAdd(c.slots + to * static_cast<uint32_t>(n_local) + tid, static_cast<int>(late * inv_unit));
        }
        if (dead) s_dead = 1u;
        // pushes into the ring, and weights, are there before anyone goes on
        if (far || kPlastic) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        ++row;
        slot = slot == W ? 0u : slot + 1u;
        if (s_dead != 0u) {
            if (tid == 0) {
                __hip_atomic_store(reread(ka)->gate + (groups + 1) * kGateStep, uint64_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(reread(ka)->fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            break;
        }
    }
    lds_barrier();

    // ---- state out
    a = reread(ka);
    if (s_dead != 0u) {
        // no step's state: V and the records that are left say so
        const uint64_t all = wave_ballot(valid);
        const int64_t from = s_role & kLost ? 0 : row;
        for (int64_t q = from; valid && q < a->n_steps; ++q) {
            if (raster) raster[(q - row) * raster_words] = all;
            if (a->rec_v) a->rec_v[q * n_total + j] = __builtin_nanf("");
            if (a->rec_input) a->rec_input[q * n_total + j] = __builtin_nanf("");
        }
        V = __builtin_nanf("");
    }
    const uint32_t t1 = t0 + static_cast<uint32_t>(row);
    for (uint32_t i = tid; !kPlastic && i < W * quads; i += blockDim.x) {
        const uint32_t k = i / quads, v = (i - k * quads) * 4u, s = slot + k > W ? slot + k - (W + 1u) : slot + k;
        const int4 x = *reinterpret_cast<const int4*>(c.slots + s * static_cast<uint32_t>(n_local) + v);
        if ((x.x | x.y | x.z | x.w) != 0)
            *reinterpret_cast<float4*>(c.ring + static_cast<int64_t>((t1 + k) & c.ring_mask) * c.n_pad + v) =
                make_float4(static_cast<float>(x.x) * c.unit, static_cast<float>(x.y) * c.unit, static_cast<float>(x.z) * c.unit,
                            static_cast<float>(x.w) * c.unit);
    }
    if (valid) {
        const uint32_t a1 = t1 - last, a2 = t1 - prev;
        a->V[j] = V;
        a->age[j] = static_cast<uint16_t>((a1 < 255u ? a1 : 255u) | ((a2 < 255u ? a2 : 255u) << 8));
        if (pulls) a->hist[static_cast<int64_t>((t1 & 0xFFu) >> 5) * c.n_pad + j] = bits;
        if (obs) {
            a->calcium[j] = cal;
            a->frame_acc[j] = acc;
        }
    }
    if (pulls && owns) {
        const uint64_t recent = wave_ballot(valid && t1 - last <= static_cast<uint32_t>(a->d_sum));
        if (lane == 0 && j < c.n_pad) put_summary(a->summary, j, recent, a->sum_shift);
    }
}

// The ring of arrival steps from pull delivery's spike history: every edge
// adds its weight where its source fired in the last `delay` steps.
struct RebuildArgs {
    const int32_t* __restrict__ src;
    const uint16_t* __restrict__ w;
    const uint8_t* __restrict__ d;
    const uint8_t* __restrict__ rowstart;
    const int32_t* __restrict__ chunk_row0;
    const uint16_t* __restrict__ age;
    const uint32_t* __restrict__ hist;
    float* ring;
    int64_t n_chunks, n_pad;
    uint32_t t, ring_mask;
};

// f(slot, its row) for the lane's eight slots of a chunk (a wave's).
template <class F>
__device__ __forceinline__ void each_slot(const uint8_t* rowstart, const int32_t* chunk_row0, int64_t chunk, F f) {
    const int lane = threadIdx.x & 63;
    const uint32_t rs = rowstart[chunk * 64 + lane] & (lane == 0 ? ~1u : ~0u);    // (the first slot's row is chunk_row0)
    uint32_t total;
    int64_t r = chunk_row0[chunk] + wave_prefix(static_cast<uint32_t>(__popc(rs)), &total);
    for (int k = 0; k < kEdgesPerLane; ++k) {
        r += (rs >> k) & 1u;
        f(chunk * kChunkEdges + lane * kEdgesPerLane + k, r);
    }
}

__global__ void __launch_bounds__(256) rebuild_kernel(RebuildArgs a) {
    const int64_t chunk = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (chunk >= a.n_chunks) return;
    each_slot(a.rowstart, a.chunk_row0, chunk, [&](int64_t e, int64_t r) {
        const uint32_t wb = a.w[e], d = a.d[e];
        if ((wb & 0x7FFFu) == 0u) return;
        const int64_t src = a.src[e];
        if ((a.age[src] & 0xFFu) > d) return;
        for (uint32_t back = 1; back <= d; ++back) {
            const uint32_t ts = a.t - back;
            if ((a.hist[static_cast<int64_t>((ts & 0xFFu) >> 5) * a.n_pad + src] >> (ts & 31u)) & 1u)
                atomicAdd(a.ring + static_cast<int64_t>((ts + d) & a.ring_mask) * a.n_pad + r, half_bits_to_float(wb));
        }
    });
}

// The out-edge tables at net_build: count the lists' edges (kFill false: into
// off[list + 2]), prefix sums, and fill them; off[list + 1] counts up while its
// list is filled and opens the next list after.  The order within a list does
// not matter.
struct TableArgs {
    const int32_t* __restrict__ src;
    const uint16_t* __restrict__ w;
    const uint8_t* __restrict__ d;
    const uint8_t* __restrict__ rowstart;
    const int32_t* __restrict__ chunk_row0;
    uint32_t* off;
    uint2* edge;
    const int32_t* slot_orig;           // plastic networks (else null)
    const int32_t* row_first;
    uint32_t* info;
    int64_t n_chunks, n_total;
    int32_t n_local, set_groups, window, lg, words;
};

template <bool kFill>
__global__ void __launch_bounds__(256) table_kernel(TableArgs a) {
    const int64_t chunk = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (chunk >= a.n_chunks) return;
    each_slot(a.rowstart, a.chunk_row0, chunk, [&](int64_t k, int64_t r) {
        const uint32_t wb = a.w[k];
        if (a.slot_orig) {
            if (kFill) a.info[k] = kNoEdge;
            if (a.slot_orig[k] < 0) return;
        } else if ((wb & 0x7FFFu) == 0u) {
            return;
        }
        const uint32_t g = static_cast<uint32_t>(r) / static_cast<uint32_t>(a.n_local), set = g / static_cast<uint32_t>(a.set_groups);
        const int64_t list = (static_cast<int64_t>(set) * a.n_total + a.src[k]) * a.set_groups + (g - set * a.set_groups);
        if (!kFill) {
            atomicAdd(a.off + list + 2, 1u);
            return;
        }
        const uint32_t local = static_cast<uint32_t>(r) - g * static_cast<uint32_t>(a.n_local), d = a.d[k];
        if (a.slot_orig) {
            const uint32_t rel = static_cast<uint32_t>(k - a.row_first[static_cast<int64_t>(g) * a.n_local]);
            a.info[k] = static_cast<uint32_t>(a.src[k]) | d << 16 | local << 24;
            a.edge[atomicAdd(a.off + list + 1, 1u)] = make_uint2(d * static_cast<uint32_t>(a.words) * 32u + rel, 1u);
            return;
        }
        const int e = static_cast<int>((wb >> 10) & 31u);
        const int32_t units = static_cast<int32_t>((wb & 0x3FFu) | (e ? 0x400u : 0u)) << ((e > 1 ? e : 1) - 25 - a.lg);
        a.edge[atomicAdd(a.off + list + 1, 1u)] =
            make_uint2(static_cast<int>(d) <= a.window ? d * static_cast<uint32_t>(a.n_local) + local : kFar | d << 16 | local,
                       static_cast<uint32_t>((wb & 0x8000u) ? -units : units));
    });
}

// Inclusive prefix sums of x[n] in place: the sums of blocks of 4,096 values,
// their prefix sums by one workgroup, the values of each block.
constexpr int kScanBlock = 4096;
__device__ __forceinline__ uint32_t block_prefix(uint32_t x, uint32_t* total) {      // 256 threads
    __shared__ uint32_t sums[4];
    const int wave = threadIdx.x >> 6;
    uint32_t mine, before = 0, all = 0;
    const uint32_t p = wave_prefix(x, &mine);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sums[wave] = mine;
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        before += w < wave ? sums[w] : 0u;
        all += sums[w];
    }
    *total = all;
    return p + before;
}

__global__ void __launch_bounds__(256) scan_sums_kernel(const uint32_t* x, int64_t n, uint32_t* sums) {
    const int64_t at = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x * 16;
    uint32_t s = 0, total;
    for (int k = 0; k < 16; ++k) s += at + k < n ? x[at + k] : 0u;
    (void)block_prefix(s, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(256) scan_blocks_kernel(uint32_t* sums, int n) {
    uint32_t base = 0;
    for (int i0 = 0; i0 < n; i0 += 256) {
        const int i = i0 + static_cast<int>(threadIdx.x);
        const uint32_t x = i < n ? sums[i] : 0u;
        uint32_t total;
        const uint32_t before = block_prefix(x, &total);
        if (i < n) sums[i] = base + before;
        base += total;
    }
}

__global__ void __launch_bounds__(256) scan_kernel(uint32_t* x, int64_t n, const uint32_t* sums) {
    const int64_t at = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x * 16;
    uint32_t v[16], s = 0, total;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        v[k] = at + k < n ? x[at + k] : 0u;
        s += v[k];
    }
    uint32_t run = sums[blockIdx.x] + block_prefix(s, &total);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        run += v[k];
        if (at + k < n) x[at + k] = run;
    }
}

__global__ void __launch_bounds__(256) zero_kernel(float4* p, int64_t n) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * 256)
        p[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

size_t run_lds_bytes(const ResidentPlan& r) {
    const size_t lists = static_cast<size_t>(r.threads / 64) * kListWords * sizeof(uint32_t);
    const size_t slots = (static_cast<size_t>(r.window) + 1) * (r.plastic ? r.words : r.n_local);
    return ((slots + 1) & ~size_t(1)) * sizeof(int) + lists + (r.plastic ? static_cast<size_t>(r.n_local) * 12 : 0);
}

typedef void (*RunKernel)(RunArgs);
RunKernel run_for(const ResidentPlan& r) { return r.plastic ? run_kernel<true> : run_kernel<false>; }

}  // namespace

bool resident_fits(const ResidentPlan& r, int n_cu, size_t lds_max) {
    const size_t lds = run_lds_bytes(r);
    int per_cu = 0;
    return lds + 1024 <= lds_max && r.groups <= r.threads &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(run_for(r)), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(lds_max - 1024)) == hipSuccess &&
           hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, run_for(r), r.threads, lds) == hipSuccess &&
           per_cu >= 1 && r.groups <= n_cu;
}

// (`sums`: one word per 4,096 entries of the offsets)
hipError_t launch_resident_tables(const DeviceGraph& g, const ResidentPlan& r, uint32_t* off, int64_t n_off, uint2* edge, uint32_t* sums,
                                  int lg, hipStream_t s) {
    TableArgs a{g.src, g.w, g.d, g.rowstart, g.chunk_row0, off, edge, r.plastic ? g.slot_orig : nullptr, g.row_first, r.info,
                g.n_chunks, g.n_total, r.n_local, r.set_groups, r.window, lg, r.words};
    const dim3 chunks(static_cast<unsigned>((g.n_chunks + 3) / 4)), blocks(static_cast<unsigned>((n_off + kScanBlock - 1) / kScanBlock));
    table_kernel<false><<<chunks, dim3(256), 0, s>>>(a);
    scan_sums_kernel<<<blocks, dim3(256), 0, s>>>(off, n_off, sums);
    scan_blocks_kernel<<<dim3(1), dim3(256), 0, s>>>(sums, static_cast<int>(blocks.x));
    scan_kernel<<<blocks, dim3(256), 0, s>>>(off, n_off, sums);
    table_kernel<true><<<chunks, dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

size_t resident_head_words(const ResidentPlan& r) { return static_cast<size_t>(kSets) * r.groups * kHeadStep; }
size_t resident_gate_words(const ResidentPlan& r) { return (static_cast<size_t>(r.groups) + 2) * kGateStep; }
const uint64_t* resident_lost(const ResidentPlan& r) { return r.gate + (static_cast<size_t>(r.groups) + 1) * kGateStep; }
size_t resident_more_words(const ResidentPlan& r) { return static_cast<size_t>(kSets) * r.groups * (1 + r.n_local / 32); }

hipError_t launch_resident_renumber(const ResidentPlan& r, hipStream_t s) {
    zero_kernel<<<dim3(64), dim3(256), 0, s>>>(reinterpret_cast<float4*>(r.more), static_cast<int64_t>(kSets / 2) * r.groups * (1 + r.n_local / 32));
    return hipGetLastError();
}

hipError_t launch_resident_rebuild(const DeviceGraph& g, const ResidentPlan& r, int64_t t, hipStream_t s) {
    const int64_t n4 = (static_cast<int64_t>(r.ring_mask) + 1) * g.n_pad / 4;
    zero_kernel<<<dim3(2048), dim3(256), 0, s>>>(reinterpret_cast<float4*>(r.ring), n4);
    RebuildArgs a{g.src, g.w, g.d, g.rowstart, g.chunk_row0, g.age, g.ring, r.ring, g.n_chunks, g.n_pad,
                  static_cast<uint32_t>(t), r.ring_mask};
    rebuild_kernel<<<dim3(static_cast<unsigned>((g.n_chunks + 3) / 4)), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_resident(const DeviceGraph& g, const ResidentPlan& r, int64_t t0, int32_t n_steps, const net_record* rec,
                           int32_t frame_num, int32_t frame_den, hipStream_t s) {
    RunArgs a;
    a.off = r.off;
    a.edge = r.edge;
    a.ring = r.ring;
    a.head = r.head;
    a.more = r.more;
    a.gate = r.gate;
    a.fail = r.fail_dev;
    a.V = g.V;
    a.age = g.age;
    a.hist = r.push ? nullptr : g.ring;
    a.summary = r.push ? nullptr : g.summary;
    a.drive_thr = g.drive_thr;
    a.i_ext = g.i_ext;
    a.calcium = (g.calcium && frame_num > 0) ? g.calcium : nullptr;
    a.frame_acc = g.frame_acc;
    a.frames = g.frames;
    a.rec_raster = rec ? rec->raster : nullptr;
    a.rec_v = rec ? rec->v : nullptr;
    a.rec_input = rec ? rec->input : nullptr;
    a.caller_of = g.caller_of;
    a.info = r.info;
    a.wq = g.wq;
    a.row_first = g.row_first;
    a.spk_hist = g.spk_hist;
    a.spk_cnt = g.spk_cnt;
    a.dt = g.p0.dt_d;
    a.alpha = g.stdp_alpha;
    a.beta = g.stdp_beta;
    a.words = r.words;
    a.t0 = t0;
    a.n_total = g.n_total;
    a.n_pad = g.n_pad;
    a.raster_words = (g.n_total + 63) / 64;
    a.launch = 2 * (r.launches + 1);
    a.simulate = static_cast<uint32_t>(r.simulate);
    a.ring_mask = r.ring_mask;
    a.seq0 = r.seq;
    a.n_steps = n_steps;
    a.n_local = r.n_local;
    a.set_groups = r.set_groups;
    a.window = r.window;
    a.max_delay = g.max_delay;
    a.d_sum = g.d_sum;
    a.sum_shift = g.sum_shift;
    a.frame_cap = g.frame_cap;
    a.frame_num = frame_num > 0 ? frame_num : 1;
    a.frame_den = frame_den > 0 ? frame_den : 1;
    a.unit = r.unit;
    a.inv_unit = r.inv_unit;
    a.params = g.params;
    void* args[] = {&a};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(run_for(r)), dim3(r.groups), dim3(r.threads), args,
                                      static_cast<unsigned>(run_lds_bytes(r)), s);
}

}  // namespace geonet
