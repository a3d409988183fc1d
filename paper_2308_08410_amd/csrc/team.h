// A team: blocks of one launch that go through rounds together, with a barrier between
// rounds in place of a launch.  Rounds whose work is a chain of a few dependent
// accesses cost less this way (32 blocks of one XCD: 0.4-0.9 us a barrier) than as
// launches (2-3 us from the end of one to the first access of the next).
//
// Data that blocks hand to one another is written and read with agent-scope atomics
// (they go by the CU's cache, which is not kept coherent; within one XCD they end in
// its L2) and is complete at team_sync, which waits for the caller's own.
//
// Only blocks that are running are ever waited for, so a team needs no number of blocks to
// fit the device together, beside whatever else runs there.  The first block to join waits
// a moment for the others; those who came found the team.  A block that comes later asks
// the first one, which takes it in at the end of a round: while there are fewer members
// than blocks, a round's end names the members of the next.  So a launch beside another
// that fills the device grows as blocks find room: the forward of 200k vertices (2.7 ms
// alone) beside 40 passes over 1 GB on another stream takes 5.4 ms, and 9.4 (up to 13)
// by its founders alone.
#pragma once

#include <hip/hip_runtime.h>

#include "gbp_internal.h"

constexpr int kTeamWait = 2000;        // ticks of 10 ns the first block waits for the others

struct Team {
    TeamCtl* ctl;
    int rank;
    int size;      // members of the current round
    int was;       // and of the last one, whose lists the current one reads
    int want;      // members it may grow to
    int late;      // the round at whose end the block joins; 0: it is a member
    double inv;    // 1 / size
};

// A member's word at a round's end (TeamCtl::flag): the round (mod 2^15), that round's
// members and the next one's, and the member's count.
__device__ __forceinline__ unsigned team_mark(int round) { return 0x8000u | ((unsigned)round & 0x7fffu); }
__device__ __forceinline__ unsigned long long team_word(int round, int size, int next, int count) {
    return (unsigned long long)(team_mark(round) << 16 | (unsigned)(size - 1) << 8 | (unsigned)(next - 1)) << 32 |
           (unsigned)count;
}
__device__ __forceinline__ unsigned word_mark(unsigned long long w) { return (unsigned)(w >> 48); }
__device__ __forceinline__ int word_size(unsigned long long w) { return (int)(w >> 40 & 255) + 1; }
__device__ __forceinline__ int word_next(unsigned long long w) { return (int)(w >> 32 & 255) + 1; }

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

// The block's share [i0, i1) of n items: at most n / size + 1.  (A product with 1 / size:
// a division takes each of a block's 16 waves some 40 operations, twice a round.)
__device__ __forceinline__ int team_first(int n, int rank, double inv) { return (int)((double)n * rank * inv); }
__device__ __forceinline__ void team_share(const Team& t, int n, int& i0, int& i1) {
    i0 = team_first(n, t.rank, t.inv);
    i1 = t.rank + 1 == t.size ? n : team_first(n, t.rank + 1, t.inv);
}

// Joins the block to the launch's team (false: it is not a member and returns).  t.late
// set: it does nothing but the team_sync of that round, and is a member from the next on.
// one_xcd: the blocks of one XCD, whichever the first block runs on.  blocks: those of the
// launch that ask to join (the same on all of them).
__device__ __forceinline__ bool team_join(TeamCtl* ctl, bool one_xcd, Team& t, int blocks, TeamLimits lim) {
    __shared__ int rank_sh, size_sh, late_sh;
    // blocks go to the 8 XCDs in turn
    int want = min(kTeamMax, one_xcd ? (blocks + 7) / 8 : blocks);
    if (lim.most > 0) want = min(want, lim.most);
    if (threadIdx.x == 0) {
        bool mine = true;
        if (one_xcd) {
            const int me = 1 + __builtin_amdgcn_s_getreg((31 << 11) | 20);   // HW_REG_XCC_ID
            int home = 0;
            mine = __hip_atomic_compare_exchange_strong(&ctl->home, &home, me, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) ||
                   home == me;
        }
        int r = -1, n = 0, late = 0;
        if (mine) {
            r = agent_add(&ctl->joined, 1);
            if (r == 0) {
                const int found = lim.found > 0 ? min(want, lim.found) : want;
                const long long t0 = wall_clock64();
                while ((n = agent_load(&ctl->joined)) < found && wall_clock64() - t0 < kTeamWait) {}
                n = min(n, found);
                agent_store(&ctl->size, n);
            } else if (r < want) {
                while ((n = agent_load(&ctl->size)) == 0) {}
                if (r >= n) {
                    // until a round's end takes it in, or the team is done (its last words
                    // are there then)
                    unsigned long long w;
                    const auto taken = [&] {
                        w = agent_load(&ctl->flag[0][0]);
                        if (word_size(w) <= r && r < word_next(w)) return true;
                        w = agent_load(&ctl->flag[1][0]);
                        return word_size(w) <= r && r < word_next(w);
                    };
                    bool in;
                    while (!(in = taken())) {
                        if (agent_load(&ctl->over)) {
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                            in = taken();
                            break;
                        }
                    }
                    n = word_size(w);
                    if (in) late = agent_load(&ctl->taken[word_mark(w) & 1]);
                    else r = -1;
                }
            } else {
                r = -1;
            }
        }
        rank_sh = r;
        size_sh = n;
        late_sh = late;
    }
    __syncthreads();
    t.ctl = ctl;
    t.rank = __builtin_amdgcn_readfirstlane(rank_sh);
    t.size = t.was = __builtin_amdgcn_readfirstlane(size_sh);
    t.want = want;
    t.late = __builtin_amdgcn_readfirstlane(late_sh);
    t.inv = 1.0 / t.size;
    return t.rank >= 0;
}

__device__ __forceinline__ bool team_join(TeamCtl* ctl, bool one_xcd, Team& t, TeamLimits lim) {
    return team_join(ctl, one_xcd, t, gridDim.x, lim);
}

// After a member's last round: blocks that still ask return.
__device__ __forceinline__ void team_leave(const Team& t) {
    if (t.rank == 0 && threadIdx.x == 0) {
        agent_store(&t.ctl->members, t.size);
        agent_store(&t.ctl->over, 1);
    }
}

// Ends round `round` (1, 2, ...) of the block, whose items are counted in *count (LDS),
// and returns once every member has: the members' counts summed, before[b] those of
// the members before b (LDS [kTeamMax + 1]), and `first` the member whose items hold
// the first of this block's share of them.  The members may be more from here on.
__device__ __forceinline__ int team_sync(Team& t, int round, const int* count, int* before, int& first) {
    __shared__ int first_sh, next_sh;
    int next = t.size;
    const bool grows = t.size < t.want;
    if (grows && t.rank == 0 && threadIdx.x == 0) {
        next = min(t.want, agent_load(&t.ctl->joined));
        if (next > t.size) agent_store(&t.ctl->taken[round & 1], round);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);   // this wave's stores and atomics are done
    __syncthreads();
    unsigned long long* flag = t.ctl->flag[round & 1];
    if (threadIdx.x < 64) {
        if (threadIdx.x == 0 && !t.late)
            __hip_atomic_store(flag + t.rank, team_word(round, t.size, next, *count), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        int run = 0;
        for (int b0 = 0; b0 < t.size; b0 += 64) {
            const int b = b0 + (int)threadIdx.x;
            unsigned long long f = 0;
            bool here;
            do {
                here = b >= t.size || word_mark(f = agent_load(flag + b)) == team_mark(round);
            } while (__ballot(!here) != 0ull);
            if (b0 == 0 && grows) next = word_next((unsigned long long)__builtin_amdgcn_readfirstlane((int)(f >> 32)) << 32);
            int inc = b < t.size ? (int)(unsigned)f : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(inc, o);
                if ((int)threadIdx.x >= o) inc += v;
            }
            if (b < t.size) before[b + 1] = run + inc;
            run += __shfl(inc, 63);
        }
        int m = 0;
        const int i0 = team_first(run, t.rank, grows ? 1.0 / next : t.inv);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int b0 = 0; b0 < t.size; b0 += 64) {
            const int b = b0 + (int)threadIdx.x;
            m += __popcll(__ballot(b < t.size && before[b + 1] <= i0));
        }
        if (threadIdx.x == 0) {
            before[0] = 0;
            first_sh = m;
            if (grows) next_sh = next;
        }
    }
    __syncthreads();
    first = first_sh;
    t.was = t.size;
    t.late = 0;
    if (grows) {
        t.size = __builtin_amdgcn_readfirstlane(next_sh);
        t.inv = 1.0 / t.size;
    }
    return before[t.was];
}
