// Vertex models and small wave helpers shared by the simulation kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace geonet {
namespace {

// Standard normal from two 32-bit draws (Box-Muller on 24-bit uniforms).
__device__ __forceinline__ float gaussian(uint32_t a, uint32_t b) {
    const float u1 = (static_cast<float>(a >> 8) + 0.5f) * 0x1p-24f;
    const float u2 = (static_cast<float>(b >> 8) + 0.5f) * 0x1p-24f;
    return sqrtf(-2.0f * logf(u1)) * cospif(2.0f * u2);
}

// The same draw in FP64 (the Izhikevich vertex keeps its state in FP64).
__device__ __forceinline__ double gaussian_d(uint32_t a, uint32_t b) {
    const double u1 = (static_cast<double>(a >> 8) + 0.5) * 0x1p-24;
    const double u2 = (static_cast<double>(b >> 8) + 0.5) * 0x1p-24;
    return sqrt(-2.0 * log(u1)) * cos(2.0 * 3.141592653589793 * u2);
}

// One step of the Izhikevich vertex (Section 3.1, Eq. izsimple) with its
// post-synaptic current (Section 3.2, Eqs. simplepsc, alphapsc, izpsc), from
// the state at t; `spike` is spd(V(t)), `in` the delivered sum (an impulse
// into r or p, or into V without a PSC), `u` the control current and `noise`
// sigma*xi.  The expressions are evaluated in the order the header states.
struct IzhState {
    double v, w, r, p;
};

__device__ __forceinline__ IzhState izh_step(const NetParams& p, const IzhState& s, bool spike, double in, double u,
                                             double noise) {
    IzhState n = s;
    if (p.psc == NET_PSC_EXP) {
        n.r = s.r - p.dt_d * p.psc_a * s.r + in;
    } else if (p.psc == NET_PSC_ALPHA) {
        n.r = s.r + p.dt_d * s.p;
        n.p = s.p + p.dt_d * (-p.psc_a * p.psc_a * s.r - 2.0 * p.psc_a * s.p) + in;
    }
    if (spike) {
        n.v = static_cast<double>(p.v_reset);
        n.w = s.w + p.iz_d;
    } else {
        const double syn = p.psc == NET_PSC_NONE ? 0.0 : s.r;
        const double cur = p.iz_k * (s.v - p.iz_vr) * (s.v - p.iz_vt) - s.w + syn + u;
        double vn = s.v + p.dt_d * p.iz_inv_c * cur;
        if (p.psc == NET_PSC_NONE) vn = vn + in;
        n.v = vn + noise;
        n.w = s.w + p.dt_d * p.iz_a * (p.iz_b * (s.v - p.iz_vr) - s.w);
    }
    return n;
}

// Hodgkin-Huxley vertex (Section 3.1's four-state model), one Euler step
// from the state at t: the rate functions of the standard squid-axon set
// (alpha_m, alpha_n at their limits where the denominator vanishes), the PSC
// kinds as for the Izhikevich vertex.  vprev keeps V(t) for the crossing
// test of the next step.
struct HhState {
    double v, vprev, m, n, h, r, p;
};

__device__ __forceinline__ double hh_am(double V) {
    const double x = V + 40.0;
    return x == 0.0 ? 1.0 : 0.1 * x / (1.0 - exp(-x / 10.0));
}
__device__ __forceinline__ double hh_bm(double V) { return 4.0 * exp(-(V + 65.0) / 18.0); }
__device__ __forceinline__ double hh_ah(double V) { return 0.07 * exp(-(V + 65.0) / 20.0); }
__device__ __forceinline__ double hh_bh(double V) { return 1.0 / (1.0 + exp(-(V + 35.0) / 10.0)); }
__device__ __forceinline__ double hh_an(double V) {
    const double x = V + 55.0;
    return x == 0.0 ? 0.1 : 0.01 * x / (1.0 - exp(-x / 10.0));
}
__device__ __forceinline__ double hh_bn(double V) { return 0.125 * exp(-(V + 65.0) / 80.0); }

__device__ __forceinline__ HhState hh_step(const NetParams& p, const HhState& s, double in, double u, double noise) {
    HhState n = s;
    if (p.psc == NET_PSC_EXP) {
        n.r = s.r - p.dt_d * p.psc_a * s.r + in;
    } else if (p.psc == NET_PSC_ALPHA) {
        n.r = s.r + p.dt_d * s.p;
        n.p = s.p + p.dt_d * (-p.psc_a * p.psc_a * s.r - 2.0 * p.psc_a * s.p) + in;
    }
    const double syn = p.psc == NET_PSC_NONE ? 0.0 : s.r;
    const double i_na = p.hh_gna * s.m * s.m * s.m * s.h * (s.v - p.hh_ena);
    const double i_k = p.hh_gk * s.n * s.n * s.n * s.n * (s.v - p.hh_ek);
    const double i_l = p.hh_gl * (s.v - p.hh_el);
    double vn = s.v + p.dt_d * p.hh_inv_c * (-i_na - i_k - i_l + syn + u);
    if (p.psc == NET_PSC_NONE) vn = vn + in;
    n.v = vn + noise;
    n.vprev = s.v;
    n.m = s.m + p.dt_d * (hh_am(s.v) * (1.0 - s.m) - hh_bm(s.v) * s.m);
    n.h = s.h + p.dt_d * (hh_ah(s.v) * (1.0 - s.h) - hh_bh(s.v) * s.h);
    n.n = s.n + p.dt_d * (hh_an(s.v) * (1.0 - s.n) - hh_bn(s.v) * s.n);
    return n;
}

__device__ __forceinline__ float half_bits_to_float(uint32_t bits) {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(bits)));
}

__device__ __forceinline__ uint64_t wave_ballot(bool p) { return __ballot(p); }

// Write the 64 bits `bits` of local vertices [u0, u0+64) (union numbering
// u0 = first vertex) into a bit array of 64-bit words shared with other
// networks: clear this network's positions (mask), then set its bits.
__device__ __forceinline__ void put_bits_shared(uint64_t* words, int64_t u0, uint64_t bits, uint64_t mask) {
    const int64_t w0 = u0 >> 6;
    const int sh = static_cast<int>(u0 & 63);
    atomicAnd(reinterpret_cast<unsigned long long*>(words + w0), ~(mask << sh));
    atomicOr(reinterpret_cast<unsigned long long*>(words + w0), (bits & mask) << sh);
    if (sh != 0 && (mask >> (64 - sh)) != 0) {
        atomicAnd(reinterpret_cast<unsigned long long*>(words + w0 + 1), ~(mask >> (64 - sh)));
        atomicOr(reinterpret_cast<unsigned long long*>(words + w0 + 1), (bits & mask) >> (64 - sh));
    }
}

// The wave's 64 bits of the recent-spike summary (first vertex j).
__device__ __forceinline__ void put_summary(uint32_t* summary, int64_t j, uint64_t recent, int sum_shift) {
    if (sum_shift == 0) {
        reinterpret_cast<uint64_t*>(summary)[j >> 6] = recent;
    } else {
        // one bit per vertex pair: OR the pairs, then pack the even bits
        uint64_t x = (recent | (recent >> 1)) & 0x5555555555555555ull;
        x = (x | (x >> 1)) & 0x3333333333333333ull;
        x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
        x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
        x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
        x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
        summary[j >> 6] = static_cast<uint32_t>(x);
    }
}

// Barrier that orders LDS only (records on their way to memory are not waited for).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ uint64_t read_lane64(uint64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), lane);
    return lo | (static_cast<uint64_t>(hi) << 32);
}

// Memory that no kernel writes while one reads it: uniform words of it are
// scalar loads.
typedef const uint32_t __attribute__((address_space(4)))* const_words;

// A kernel's arguments, read again where they are used: a pointer the
// compiler cannot see through keeps the dozens that only the start, the end or
// a rare branch needs out of scalar registers while the steps run.
template <class P>
__device__ __forceinline__ P reread(P p) {
    asm volatile("" : "+s"(p));
    return p;
}

// A wave-uniform value that the compiler takes for a new one each time.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
    x = __builtin_amdgcn_readfirstlane(x);
    asm volatile("" : "+s"(x));
    return x;
}

// A struct in memory that no kernel writes, by scalar loads (`p` is uniform).
template <class T>
__device__ __forceinline__ T load_const(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    const const_words w = reinterpret_cast<const_words>(reinterpret_cast<uintptr_t>(p));
    uint32_t words[sizeof(T) / 4];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) words[i] = w[i];
    T v;
    __builtin_memcpy(&v, words, sizeof(T));
    return v;
}

// Sum of x over the lanes below this one; *total over all (DPP row shifts and
// row broadcasts).
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x, uint32_t* total) {
    uint32_t s = x;
    s += __builtin_amdgcn_update_dpp(0u, s, 0x111, 0xF, 0xF, false);   // row_shr:1
    s += __builtin_amdgcn_update_dpp(0u, s, 0x112, 0xF, 0xF, false);   // row_shr:2
    s += __builtin_amdgcn_update_dpp(0u, s, 0x114, 0xF, 0xF, false);   // row_shr:4
    s += __builtin_amdgcn_update_dpp(0u, s, 0x118, 0xF, 0xF, false);   // row_shr:8
    s += __builtin_amdgcn_update_dpp(0u, s, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
    s += __builtin_amdgcn_update_dpp(0u, s, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
    *total = __builtin_amdgcn_readlane(s, 63);
    return s - x;
}

}  // namespace
}  // namespace geonet
