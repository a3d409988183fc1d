// A team: blocks of one launch that go through rounds together, with a barrier between
// rounds in place of a launch.  Rounds whose work is a chain of a few dependent
// accesses cost less this way (32 blocks of one XCD: 0.4-0.9 us a barrier) than as
// launches (2-3 us from the end of one to the first access of the next).
//
// Data that blocks hand to one another is written and read with agent-scope atomics
// (they go by the CU's cache, which is not kept coherent; within one XCD they end in
// its L2) and is complete at team_sync, which waits for the caller's own.
//
// Only blocks that are running are ever waited for: a block joins while the team is
// open, the first to join closes it, and a block that comes later returns at once.
// So a team needs no number of blocks to fit the device together, beside whatever
// else runs there.
#pragma once

#include <hip/hip_runtime.h>

#include "gbp_internal.h"

constexpr int kTeamClosed = 1 << 16;
constexpr int kTeamWait = 2000;        // ticks of 10 ns the first block waits for the others

struct Team {
    TeamCtl* ctl;
    int rank, size;
};

__device__ __forceinline__ int agent_load(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float agent_load(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long agent_load(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int agent_add(int* p, int v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Floats as integers of the same order.
__device__ __forceinline__ int ordered(float x) {
    const int b = __float_as_int(x);
    return b < 0 ? b ^ 0x7fffffff : b;
}
__device__ __forceinline__ float from_ordered(int b) { return __int_as_float(b < 0 ? b ^ 0x7fffffff : b); }

// Joins the block to the launch's team (false: it is not a member and returns).
// one_xcd: the blocks of one XCD, whichever the first block runs on.  blocks: those of the
// launch that ask to join (the same on all of them).
__device__ __forceinline__ bool team_join(TeamCtl* ctl, bool one_xcd, Team& t, int blocks) {
    __shared__ int rank_sh, size_sh;
    if (threadIdx.x == 0) {
        bool mine = true;
        if (one_xcd) {
            const int me = 1 + __builtin_amdgcn_s_getreg((31 << 11) | 20);   // HW_REG_XCC_ID
            int home = 0;
            mine = __hip_atomic_compare_exchange_strong(&ctl->home, &home, me, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) ||
                   home == me;
        }
        int r = -1, n = 0;
        if (mine) {
            r = agent_add(&ctl->joined, 1);
            if (r == 0) {
                // blocks go to the 8 XCDs in turn
                const int want = min(kTeamMax, one_xcd ? (blocks + 7) / 8 : blocks);
                const long long t0 = wall_clock64();
                while (agent_load(&ctl->joined) < want && wall_clock64() - t0 < kTeamWait) {}
                n = min(kTeamMax, agent_add(&ctl->joined, kTeamClosed));
                agent_store(&ctl->size, n);
            } else if (r < kTeamMax) {
                while ((n = agent_load(&ctl->size)) == 0) {}
            }
        }
        rank_sh = r;
        size_sh = n;
    }
    __syncthreads();
    t.ctl = ctl;
    t.rank = rank_sh;
    t.size = size_sh;
    return t.rank >= 0 && t.rank < t.size;
}

__device__ __forceinline__ bool team_join(TeamCtl* ctl, bool one_xcd, Team& t) {
    return team_join(ctl, one_xcd, t, gridDim.x);
}

// The block's share [i0, i1) of n items.
__device__ __forceinline__ void team_share(const Team& t, int n, int& i0, int& i1) {
    i0 = (int)((long long)n * t.rank / t.size);
    i1 = (int)((long long)n * (t.rank + 1) / t.size);
}

// Ends round `round` (1, 2, ...) of the block, whose items are counted in *count (LDS),
// and returns once every member has: the members' counts summed, before[b] those of
// the members before b (LDS [kTeamMax + 1]), and `first` the member whose items hold
// the first of this block's share of them.
__device__ __forceinline__ int team_sync(const Team& t, int round, const int* count, int* before, int& first) {
    __shared__ int first_sh;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);   // this wave's stores and atomics are done
    __syncthreads();
    unsigned long long* flag = t.ctl->flag[round & 1];
    if (threadIdx.x < 64) {
        if (threadIdx.x == 0)
            __hip_atomic_store(flag + t.rank, ((unsigned long long)(unsigned)round << 32) | (unsigned)*count,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int run = 0;
        for (int b0 = 0; b0 < t.size; b0 += 64) {
            const int b = b0 + (int)threadIdx.x;
            unsigned long long f = 0;
            bool here;
            do {
                here = b >= t.size || (int)((f = agent_load(flag + b)) >> 32) >= round;
            } while (__ballot(!here) != 0ull);
            int inc = b < t.size ? (int)(unsigned)f : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(inc, o);
                if ((int)threadIdx.x >= o) inc += v;
            }
            if (b < t.size) before[b + 1] = run + inc;
            run += __shfl(inc, 63);
        }
        int i0, i1, m = 0;
        team_share(t, run, i0, i1);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int b0 = 0; b0 < t.size; b0 += 64) {
            const int b = b0 + (int)threadIdx.x;
            m += __popcll(__ballot(b < t.size && before[b + 1] <= i0));
        }
        if (threadIdx.x == 0) {
            before[0] = 0;
            first_sh = m;
        }
    }
    __syncthreads();
    first = first_sh;
    return before[t.size];
}
