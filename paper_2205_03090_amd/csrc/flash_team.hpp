// flash_team.hpp -- the flash's items run by a team of lanes each, for batches
// too small to fill the device.
//
// A small batch is bound by the slowest mixture's chain of steps, and a chain
// by the instructions of a step.  In a team the lanes hold the same item, run
// the same code on the same values and take the same path, except that
//   * the lane's parity is a phase (or, in the stability stages, a trial):
//     where a step evaluates the equation of state for both phases, each
//     parity evaluates one and the results are exchanged;
//   * a function applied to every component (logarithm, exponential, the
//     quotients of the compositions) is applied by one lane per component,
//     through LDS, instead of by every lane to every component.
// Nothing is summed across lanes and no expression changes, so the results
// are those of the other forms bit for bit.  A step of the split trust region at
// nc 8 issues about 2,700 instructions instead of 5,500: 100 mixtures took 0.38 ms
// with a lane pair each, 0.21 ms with a team.
#pragma once

#include "flash_group.hpp"

namespace ptf {

// A team: D lanes per parity, 2 D lanes per mixture, 32 / D mixtures per
// wavefront.  Lane l of the wavefront: parity l & 1, member (l >> 1) % D.
// WAVES: wavefronts of the block, at most.
template <int D, int WAVES = 1>
struct Team {
    static constexpr bool kTeam = true;
    static constexpr bool kShortCubic = true, kShortCut = true, kShortEnd = true;
    static constexpr int kLanes = 2 * D;
    static constexpr int kPerWave = 64 / kLanes;

    static __device__ __forceinline__ int member() { return ((int)threadIdx.x >> 1) % D; }
    static __device__ __forceinline__ bool odd() { return (threadIdx.x & 1u) != 0u; }

    // The members' exchange buffer of this parity's half of the team.
    static __device__ __forceinline__ double *buf()
    {
        __shared__ double b[WAVES * 2 * kPerWave * 2 * kMaxNc];
        const int half = 2 * ((int)threadIdx.x / kLanes) + ((int)threadIdx.x & 1);
        return b + half * 2 * kMaxNc;
    }

    // v_i = f(a_i, b_i), component i by member i mod D.
    template <int NC, class F>
    static __device__ __forceinline__ void map2(double (&v)[NC], const double (&a)[NC],
                                                const double (&b)[NC], F f)
    {
        constexpr int R = (NC + D - 1) / D;
        double *q = buf();
        if (member() == 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                q[i] = a[i];
                q[kMaxNc + i] = b[i];
            }
        }
        wave_lds_sync();
        double r[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            // members past the last component repeat it
            const int i = member() + k * D < NC ? member() + k * D : NC - 1;
            r[k] = f(q[i], q[kMaxNc + i]);
        }
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int i = member() + k * D < NC ? member() + k * D : NC - 1;
            q[i] = r[k];
        }
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < NC; ++i) v[i] = q[i];
        wave_lds_sync();
    }

    // v_i = f(v_i), component i by member i mod D.
    template <int NC, class F>
    static __device__ __forceinline__ void map(double (&v)[NC], F f)
    {
        constexpr int R = (NC + D - 1) / D;
        double *q = buf();
        if (member() == 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) q[i] = v[i];
        }
        wave_lds_sync();
        double r[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int i = member() + k * D < NC ? member() + k * D : NC - 1;
            r[k] = f(q[i]);
        }
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int i = member() + k * D < NC ? member() + k * D : NC - 1;
            q[i] = r[k];
        }
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < NC; ++i) v[i] = q[i];
        wave_lds_sync();
    }

    // The neighbour of the other parity's value.
    static __device__ __forceinline__ uint32_t other(uint32_t v)
    {
        // quad permutation (1, 0, 3, 2)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);
    }
    static __device__ __forceinline__ double other(double v)
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = other((uint32_t)u), hi = other((uint32_t)(u >> 32));
        return __builtin_bit_cast(double, lo | (hi << 32));
    }

    // first, own: the arrays of (even, odd) parity from this lane's own (in
    // place: own becomes the odd parity's).
    template <int N>
    static __device__ __forceinline__ void sort_pair(double (&first)[N], double (&own)[N])
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double x = other(own[i]);
            first[i] = odd() ? x : own[i];
            own[i] = odd() ? own[i] : x;
        }
    }

    // l0 = ln w0, l1 = ln w1: even lanes take w0, odd lanes w1.
    template <int NC>
    static __device__ __forceinline__ void log_pair(double (&l0)[NC], double (&l1)[NC],
                                                    const double (&w0)[NC],
                                                    const double (&w1)[NC])
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) l1[i] = odd() ? w1[i] : w0[i];
        map<NC>(l1, [](double v) { return log(v); });
        sort_pair<NC>(l0, l1);
    }

    // Phase evaluations of w0 (even lanes) and w1 (odd lanes): o is this
    // lane's own, r0, r1 both ln phi, z0, z1 both Z.
    template <int NC>
    static __device__ __forceinline__ void eval_pair(Phase<NC> &o, const Eos<NC> &e,
                                                     const double *__restrict__ K,
                                                     const double (&w0)[NC],
                                                     const double (&w1)[NC], double s0,
                                                     double s1, double &z0, double &z1,
                                                     double (&r0)[NC], double (&r1)[NC],
                                                     uint32_t &fl)
    {
        double w[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) w[i] = odd() ? w1[i] : w0[i];
        uint32_t f = 0;
        phase_eval_sum<NC>(o, e, K, w, odd() ? s1 : s0, f, odd() ? z1 : z0);
        fl += f + other(f);
        const double zo = other(o.Z);
        z0 = odd() ? zo : o.Z;
        z1 = odd() ? o.Z : zo;
#pragma unroll
        for (int i = 0; i < NC; ++i) r1[i] = o.lnphi[i];
        sort_pair<NC>(r0, r1);
    }
};

}  // namespace ptf
