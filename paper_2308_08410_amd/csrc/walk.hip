// Leaves-first walk of the parent graph: lambda = g + P^T lambda.
//
// Every vertex sums alpha_c lambda_c over its children c in a fixed order, so the
// result does not depend on the order in which vertices finish.  The walk goes in
// levels: a vertex is finished in the level after its last child, hands its lambda
// to its parents' entries and takes one off each parent's count of unfinished
// children; the parents whose count that brought to zero are the next level.  One
// launch walks all levels (team.h).
//
// A sum's products are exact and added in FP64, and a lambda is rounded once: with FP32
// products and sums the largest relative error over 2,704 nodes was 1.2-1.3e-7.
#include <algorithm>
#include <climits>

#include "profile.h"
#include "team.h"
#include "walk.h"

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ bool has_parent(int4 pn, int x) {
    return pn.x == x || pn.y == x || pn.z == x;
}

// The smallest vertex that a and it name each other as weighted parents, or -1.
__device__ __forceinline__ int mutual(const int4* __restrict__ pnode, int a) {
    const int4 pn = pnode[a];
    const int f[3] = {pn.x, pn.y, pn.z};
    int best = -1;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (f[k] >= 0 && has_parent(pnode[f[k]], a) && (best < 0 || f[k] < best)) best = f[k];
    return best;
}

// The vertices' records, room for the child lists, and the leaves, the first level.  a and c are partners (a two-cycle) when each is a weighted parent of
// the other (the anisotropic scheme is not causal) and each is the other's smallest
// such parent; the pair is solved jointly once both members' other children are
// finished.  A block takes the room of its vertices' lists with one atomic: where a
// list sits does not matter, only its order does (k_child_sort).
constexpr int kLinkThreads = 1024;

__global__ void __launch_bounds__(kLinkThreads) k_adj_link(AdjGraph a, const float* __restrict__ dLdT_user,
                                                           const int* __restrict__ node_user) {
    __shared__ int wsum[kLinkThreads / 64], wleaf[kLinkThreads / 64], base_sh, leaf_sh;
    const int x = blockIdx.x * kLinkThreads + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = x < a.n_v ? a.cnt[x] : 0;
    bool leaf = false;
    if (x < a.n_v) {
        const int p = mutual(a.pnode, x);
        const bool pair = p >= 0 && mutual(a.pnode, p) == x;
        const bool reached = a.T[x] < __builtin_huge_valf();
        float g = reached ? dLdT_user[node_user ? node_user[x] : x] : 0.f;
        if (g != g) g = 0.f;
        const int wait = c - (pair ? 1 : 0);   // all its children but its partner, which is one of them
        leaf = wait == 0 && reached;
        const int4 pn = a.pnode[x];
        float4* r = reinterpret_cast<float4*>(a.rec + x);   // ranks and entries: k_child_sort
        r[0] = make_float4(__int_as_float(pn.x), 0.f, 0.f, g);
        r[1] = make_float4(__int_as_float(pn.y), 0.f, 0.f, __int_as_float(c));
        r[2] = make_float4(__int_as_float(pn.z), 0.f, 0.f, __int_as_float(pair ? p : -1));
        a.rec[x].rem = wait;
        a.rec[x].pair = pair && x < p ? 2 : 0;
        a.cfill[x] = 0;
        a.g[x] = g;
        a.lam[x] = g;
        a.done[x] = reached ? 0 : 1;
    }
    int inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    const unsigned long long lm = __ballot(leaf);
    if (lane == 63) {
        wsum[wave] = inc;
        wleaf[wave] = __popcll(lm);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0, leaves = 0;
        for (int w = 0; w < kLinkThreads / 64; ++w) {
            const int t = wsum[w], u = wleaf[w];
            wsum[w] = run;
            wleaf[w] = leaves;
            run += t;
            leaves += u;
        }
        base_sh = run > 0 ? atomicAdd(&a.ctl->nchild, run) : 0;
        leaf_sh = leaves > 0 ? atomicAdd(&a.ctl->nleaf, leaves) : 0;
    }
    __syncthreads();
    if (x >= a.n_v) return;
    const int b = base_sh + wsum[wave] + inc - c;
    a.crange[x] = make_int2(b, b + c);
    a.rec[x].first = b;
    if (leaf) a.leaf[leaf_sh + wleaf[wave] + __popcll(lm & ((1ull << lane) - 1ull))] = x;
}

__global__ void k_child_fill(AdjGraph a) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.n_v) return;
    const int4 pn = a.pnode[c];
    const int f[3] = {pn.x, pn.y, pn.z};
    const float4 w = a.pa[c];
    const float al[3] = {w.x, w.y, w.z};
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (f[k] >= 0) {
            const int pos = a.crange[f[k]].x + atomicAdd(&a.cfill[f[k]], 1);
            a.cchild[pos] = (c << 2) | k;     // unpacked by k_child_sort
            a.calpha[pos] = al[k];
        }
}

// Sort each child list by child id (fixed summation order -> deterministic), then
// tell each child where its entry sits, its rank in the parent's list, and put the
// first entries' weights in the parent's record (0 where there is no entry).  They
// arrive as (child << 2 | which of the child's parents this is) from k_child_fill;
// child ids are distinct within a list, so the packed keys sort in child order, and
// the ids are written back unpacked.
constexpr int kSortRegs = 16;   // child lists up to this long are sorted in registers

__global__ void __launch_bounds__(TPB) k_child_sort(AdjGraph a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_v) return;
    const int b = a.crange[p].x, e = a.crange[p].y;
    int* cchild = a.cchild;
    float* calpha = a.calpha;
    if (e - b <= kSortRegs) {
        // the list in registers (padded with INT_MAX) through a bitonic network
        int ch[kSortRegs];
        float al[kSortRegs];
#pragma unroll
        for (int k = 0; k < kSortRegs; ++k) {
            ch[k] = b + k < e ? cchild[b + k] : INT_MAX;
            al[k] = b + k < e ? calpha[b + k] : 0.f;
        }
#pragma unroll
        for (int k = 2; k <= kSortRegs; k <<= 1)
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
                for (int i = 0; i < kSortRegs; ++i) {
                    const int l = i ^ j;
                    if (l > i) {
                        const int u = ch[i], v = ch[l];
                        const float fu = al[i], fv = al[l];
                        const bool sw = (u > v) == ((i & k) == 0);
                        ch[i] = sw ? v : u;
                        ch[l] = sw ? u : v;
                        al[i] = sw ? fv : fu;
                        al[l] = sw ? fu : fv;
                    }
                }
#pragma unroll
        for (int k = 0; k < kSortRegs; ++k)
            if (b + k < e) {
                const int c = ch[k] >> 2;
                cchild[b + k] = c;
                calpha[b + k] = al[k];
                a.rec[c].up[ch[k] & 3].rank = k < kAdjEntries ? k : b + k + kAdjEntries;
            }
        float4* r = reinterpret_cast<float4*>(a.rec[p].entry);
#pragma unroll
        for (int k = 0; k < kAdjEntries; k += 2) r[k / 2] = make_float4(0.f, al[k], 0.f, al[k + 1]);
        return;
    }
    for (int x = b + 1; x < e; ++x) {
        const int kc = cchild[x];
        const float ka = calpha[x];
        int y = x - 1;
        while (y >= b && cchild[y] > kc) {
            cchild[y + 1] = cchild[y];
            calpha[y + 1] = calpha[y];
            --y;
        }
        cchild[y + 1] = kc;
        calpha[y + 1] = ka;
    }
    for (int x = b; x < e; ++x) {
        const int v = cchild[x];
        const int c = v >> 2;
        cchild[x] = c;
        a.rec[c].up[v & 3].rank = x - b < kAdjEntries ? x - b : x + kAdjEntries;
        if (x - b < kAdjEntries) a.rec[p].entry[x - b] = {0.f, calpha[x]};
    }
}

// Data that the walk's blocks hand to one another, at the scope that holds them all: the
// block (its loads may hit the CU's cache) or the device.
template <int SCOPE, typename V>
__device__ __forceinline__ V scoped_load(const V* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, SCOPE);
}
template <int SCOPE, typename V>
__device__ __forceinline__ void scoped_store(V* p, V v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, SCOPE);
}

// Sum of a pair member's right-hand side and entries but its partner's, whose weight
// comes back in wo.
template <int SCOPE>
__device__ __forceinline__ double pair_sum(const AdjGraph& a, int v, int partner, double& wo) {
    const AdjRec* r = a.rec + v;
    double s = r->up[0].g;
    wo = 0.0;
    for (int k = 0; k < r->up[1].nchild; ++k) {
        const int at = r->first + k;
        const double w = a.calpha[at];
        if (a.cchild[at] == partner) wo = w;
        else s += w * scoped_load<SCOPE>(k < kAdjEntries ? &r->entry[k].lam : a.over + at);
    }
    return s;
}

constexpr int kWalkThreads = 8 * kWalkGroups;

// A vertex's record, by the 8 lanes of a group: lane j holds piece j (one line, one
// request; lanes 0-2 a parent each, 4-7 two entries each).
struct RecPiece {
    unsigned long long u0, u1;
};
template <int SCOPE>
__device__ __forceinline__ RecPiece walk_record(const AdjGraph& a, int x) {
    const unsigned long long* rp = reinterpret_cast<const unsigned long long*>(a.rec + x) + 2 * (threadIdx.x & 7);
    return {scoped_load<SCOPE>(rp), scoped_load<SCOPE>(rp + 1)};
}

// The value N lanes on in the row of 16 (a vector move, no trip through LDS).
template <int N>
__device__ __forceinline__ int lane_ahead(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x100 + N, 0xf, 0xf, true);
}
template <int N>
__device__ __forceinline__ double lane_ahead(double v) {
    return __hiloint2double(lane_ahead<N>(__double2hiint(v)), lane_ahead<N>(__double2loint(v)));
}

// One vertex x of the level.  ready(p): parent p's last child is finished.
template <int SCOPE, typename Ready>
__device__ __forceinline__ void walk_vertex(const AdjGraph& a, int x, RecPiece piece, Ready ready) {
    const int j = threadIdx.x & 7, g0 = threadIdx.x & 56;   // lane in the group, the group's first lane
    const unsigned long long u0 = piece.u0, u1 = piece.u1;
    const float v0 = __uint_as_float((unsigned)u0), v1 = __uint_as_float((unsigned)(u0 >> 32)),
                v2 = __uint_as_float((unsigned)u1), v3 = __uint_as_float((unsigned)(u1 >> 32));
    const float rhs = __shfl(v3, g0);
    const int nchild = __float_as_int(__shfl(v3, g0 + 1)), q = __float_as_int(__shfl(v3, g0 + 2));
    const int parent = j < 3 ? __float_as_int(v0) : -1, rank = __float_as_int(v1);
    float l, lq = 0.f;
    if (q < 0) {
        double s = (double)v0 * v1 + (double)v2 * v3;   // lanes 4-7; lane 4 gets the sum
        s += lane_ahead<2>(s);
        s += lane_ahead<1>(s);
        if (nchild > kAdjEntries) {
            // entries past the record's, each lane every eighth
            double o = 0.0;
            const int first = a.rec[x].first;
            for (int k = kAdjEntries + j; k < nchild; k += 8)
                o += (double)a.calpha[first + k] * scoped_load<SCOPE>(a.over + first + k);
            o += __shfl_xor(o, 1);
            o += __shfl_xor(o, 2);
            o += __shfl_xor(o, 4);
            s += o;
        }
        l = __shfl((float)(rhs + s), g0 + 4);
    } else {
        // a two-cycle: the second member to become ready solves the pair
        //   lam_a = S_a + w_ca lam_c,  lam_c = S_c + w_ac lam_a   (a < c)
        int second = 0;
        if (j == 0) second = __hip_atomic_fetch_add(&a.rec[min(x, q)].pair, -1, __ATOMIC_RELAXED, SCOPE) == 1;
        if (!__shfl(second, g0)) return;
        double wx, wq;   // wx: weight of x in q's parent face
        const double sx = pair_sum<SCOPE>(a, x, q, wx), sq = pair_sum<SCOPE>(a, q, x, wq);
        l = (float)((sx + wx * sq) / (1.0 - wx * wq));
        lq = (float)((sq + wq * sx) / (1.0 - wq * wx));
    }
    auto hand_on = [&](int self, float lam, int p, int rk, int skip) {
        if (p >= 0) {
            const int left = p != skip ? __hip_atomic_fetch_add(&a.rec[p].rem, -1, __ATOMIC_RELAXED, SCOPE) : 0;
            scoped_store<SCOPE>(rk < kAdjEntries ? &a.rec[p].entry[rk].lam : a.over + (rk - kAdjEntries), lam);
            if (left == 1) ready(p);
        }
        if (j == 3) {
            a.lam[self] = lam;
            a.done[self] = 1;
        }
    };
    hand_on(x, l, parent, rank, q);
    if (q >= 0) {
        const AdjParent* up = a.rec[q].up + min(j, 2);
        hand_on(q, lq, j < 3 ? up->vertex : -1, up->rank, x);
    }
}

// The walk by one block, for narrow levels: the level's list is in LDS (what does not
// fit in memory), a level ends with a block barrier.  Bound by the chain list, record,
// parents' counts, barrier, and from some 150 vertices a level on by what one CU can
// request, so the next vertex's record is on its way while one is worked on, and what
// the waves hand on goes by the CU's own cache.  An iteration on a triangle slice of
// 250k vertices (1,416 levels): 7.0 ms, of which the walk 3.4 (7.8 ms with accesses at
// the device's scope and each record loaded in its turn); 60,000: 2.71 and 2.92 ms.
constexpr int kWalkList = 8192;

constexpr int kBlock = __HIP_MEMORY_SCOPE_WORKGROUP;
__global__ void __launch_bounds__(kWalkThreads) k_adj_walk_block(AdjGraph a, int levels) {
    __shared__ int list[2][kWalkList], count[3];
    if (threadIdx.x < 3) count[threadIdx.x] = 0;
    __syncthreads();
    int n = a.ctl->nleaf, level = 0;
    while (n > 0 && level < levels) {
        const int out = (level + 1) & 1;
        int* const n_out = &count[(level + 1) % 3];
        const auto item = [&](int i) {
            return level == 0 ? a.leaf[i] : i < kWalkList ? list[level & 1][i] : scoped_load<kBlock>(a.ready[level & 1] + i);
        };
        int i = threadIdx.x >> 3, x = i < n ? item(i) : -1;
        RecPiece piece{};
        if (x >= 0) piece = walk_record<kBlock>(a, x);
        while (x >= 0) {
            // the next vertex's record loads while this one is worked on
            i += kWalkGroups;
            const int x_next = i < n ? item(i) : -1;
            RecPiece next{};
            if (x_next >= 0) next = walk_record<kBlock>(a, x_next);
            walk_vertex<kBlock>(a, x, piece, [&](int p) {
                const int at = atomicAdd(n_out, 1);
                if (at < kWalkList) list[out][at] = p;
                else scoped_store<kBlock>(a.ready[out] + at, p);
            });
            x = x_next;
            piece = next;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);   // this wave's entries are where the next level reads them
        ++level;
        if (threadIdx.x == 0) count[(level + 1) % 3] = 0;
        __syncthreads();
        n = *n_out;
    }
    if (threadIdx.x == 0) a.ctl->levels = level;
}

// The walk by a team of blocks, for wide levels: each block keeps the vertices it made
// ready in a list of its own, and the blocks share all lists of a level out evenly.
// Bound by a level's chain of dependent accesses: list 0.25 us, record 0.35, the parents'
// entries and counts, mostly lines that no child has touched before, 1.0-1.8, the next
// list written out 0.4, barrier with the wait for the slowest block 1-1.5.  500k
// vertices, 299 levels: 1.27 ms, 4.3 us a level (1.45 ms as launches over a stamp per
// vertex, and 1 us between them).  one_xcd: the team is one XCD's blocks, so that the
// chain's accesses end in one L2.
constexpr int kDevice = __HIP_MEMORY_SCOPE_AGENT;
__global__ void __launch_bounds__(kWalkThreads) k_adj_walk_team(AdjGraph a, int levels, int one_xcd) {
    __shared__ int before[kTeamMax + 1], count[3];
    if (threadIdx.x < 3) count[threadIdx.x] = 0;
    Team t;
    if (!team_join(a.team, one_xcd, t, a.limits)) return;
    int n = t.late ? 1 : a.ctl->nleaf, level = t.late ? t.late - 1 : 0, m = 0;
    size_t cap = walk_list_cap(a.n_v, t.size), cap_out = cap;
    while (n > 0 && level < levels) {
        const int* in = level == 0 ? a.leaf : a.ready[level & 1];
        int* out = a.ready[(level + 1) & 1] + cap_out * t.rank;
        int* const n_out = &count[(level + 1) % 3];
        int i0 = 0, i1 = 0;
        if (!t.late) team_share(t, n, i0, i1);
        for (int i = i0 + (threadIdx.x >> 3); i < i1; i += kWalkGroups) {
            int x;
            if (level == 0) {
                x = in[i];
            } else {
                while (before[m + 1] <= i) ++m;
                x = agent_load(in + cap * m + (i - before[m]));
            }
            walk_vertex<kDevice>(a, x, walk_record<kDevice>(a, x),
                                 [&](int p) { agent_store(out + atomicAdd(n_out, 1), p); });
        }
        ++level;
        n = team_sync(t, level, n_out, before, m);
        cap = cap_out;
        if (t.size != t.was) cap_out = walk_list_cap(a.n_v, t.size);
        if (threadIdx.x == 0) count[(level + 2) % 3] = 0;   // read by all before the sync, used after the next
    }
    team_leave(t);
    if (t.rank == 0 && threadIdx.x == 0) a.ctl->levels = level;
}

__global__ void __launch_bounds__(kLinkThreads) k_adj_remaining(AdjGraph a, int* __restrict__ list) {
    __shared__ int wsum[kLinkThreads / 64], base_sh;
    const int x = blockIdx.x * kLinkThreads + threadIdx.x;
    const bool left = x < a.n_v && !a.done[x];
    const unsigned long long m = __ballot(left);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (!__syncthreads_or(left)) return;
    if (lane == 0) wsum[wave] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int w = 0; w < kLinkThreads / 64; ++w) {
            const int t = wsum[w];
            wsum[w] = run;
            run += t;
        }
        base_sh = atomicAdd(&a.ctl->remaining, run);
    }
    __syncthreads();
    if (left) list[base_sh + wsum[wave] + __popcll(m & ((1ull << lane) - 1ull))] = x;
}

__global__ void k_sweeps_reset(TeamCtl* team, AdjCtl* ctl) {
    if (threadIdx.x < 3) ctl->diff[threadIdx.x] = ctl->lmax[threadIdx.x] = 0;
    for (int k = threadIdx.x; k < (int)(sizeof(TeamCtl) / sizeof(int)); k += blockDim.x)
        reinterpret_cast<int*>(team)[k] = 0;
}

// Gauss-Seidel sweeps (in place) over the vertices that the walk could not finish
// because of a cycle in the parent graph.  Every cycle leaks weight to parents outside
// it, so the sweeps contract to the unique solution.
//
// One sweep a launch, recording its largest |change| and |lambda| (slot it % 2; the
// other is cleared for the next).
__global__ void k_adj_sweep(AdjGraph a, const int* __restrict__ list, int it) {
    __shared__ float red[2][TPB / 64];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctl->diff[(it + 1) & 1] = 0;
        a.ctl->lmax[(it + 1) & 1] = 0;
    }
    const int n = a.ctl->remaining;
    // a block with no listed vertex has nothing to add (in a budgeted backward most
    // sweeps find the list empty: they must cost a launch, not 2 contended atomics
    // per block)
    if ((int)(blockIdx.x * blockDim.x) >= n) return;
    float d = 0.f, m = 0.f;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
        const int i = list[q];
        const int2 r = a.crange[i];
        float l = a.g[i];
        for (int k = r.x; k < r.y; ++k) l += a.calpha[k] * a.lam[a.cchild[k]];
        d = fmaxf(d, fabsf(l - a.lam[i]));
        m = fmaxf(m, fabsf(l));
        a.lam[i] = l;
    }
    for (int o = 32; o > 0; o >>= 1) {
        d = fmaxf(d, __shfl_xor(d, o));
        m = fmaxf(m, __shfl_xor(m, o));
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = d;
        red[1][threadIdx.x >> 6] = m;
    }
    __syncthreads();
    if (threadIdx.x < 2) {   // both are >= 0 and start at 0: a zero changes no maximum
        float v = 0.f;
        for (int w = 0; w < TPB / 64; ++w) v = fmaxf(v, red[threadIdx.x][w]);
        if (v > 0.f) atomicMax(threadIdx.x ? &a.ctl->lmax[it & 1] : &a.ctl->diff[it & 1], __float_as_int(v));
    }
}

__global__ void k_adj_swept(AdjCtl* ctl, int from, int count, float tol) {
    if (threadIdx.x != 0 || ctl->remaining == 0) return;
    const int slot = (from + count - 1) & 1;
    ctl->sweeps = from + count;
    ctl->settled = count > 0 && __int_as_float(ctl->diff[slot]) <= tol * __int_as_float(ctl->lmax[slot]);
}

// All sweeps in one launch, by a team: the change is looked at after every 16th (every
// 32nd of a long list) and the last; lambdas pass between the blocks as the walk's entries
// do.  A wave takes 64 neighbours in the list, most of which share lines, and the waves are
// dealt out over the blocks (one entry a block in turn: 21 us a sweep of 170 thousand).
// Short lists are one XCD's, longer ones 64 blocks of all, the longest 256.  Us a sweep by
// 8 / 64 / 256 blocks: 3 thousand 2.8 / 2.6 / 4.0, 17 thousand 8.5 / 4.7 / 6.2, 51 thousand
// 24 / 6.9 / 9.0, 77 thousand 32 / 7.8 / 8.0, 112 thousand 45 / 9.6 / 8.5, 171 thousand
// 66 / 12.5 / 8.9; as launches 5.7 at 17 thousand, 12 at 52, 17.7 at 171 (and, past the
// mesh size below, 31 us for 600 thousand, where the team's scattered requests took 70).
constexpr int kSweepThreads = 1024;
constexpr int kSweepFewBlocks = 64, kSweepBlocks = 256;
constexpr int kSweepFewList = 65536;
constexpr int kSweepOneXcd = 2048;
constexpr int kSweepTeamVerts = 1 << 18;   // mesh size, which bounds the list, up to which a team sweeps

__global__ void __launch_bounds__(kSweepThreads) k_adj_sweeps(AdjGraph a, const int* __restrict__ list,
                                                              int max_sweeps, float tol, int exhaust) {
    __shared__ int before[kTeamMax + 1], zero;
    __shared__ float red[2][kSweepThreads / 64];
    const int n = a.ctl->remaining;
    const int blocks = n <= kSweepFewList ? kSweepFewBlocks : kSweepBlocks;
    if (n == 0 || (int)blockIdx.x >= blocks) return;
    const int every = n <= kSweepFewList ? 16 : 32;
    if (threadIdx.x == 0) zero = 0;
    Team t;
    if (!team_join(a.team, n <= kSweepOneXcd, t, blocks, a.limits)) return;   // uniform over the launch
    int first, it = t.late ? t.late - 1 : 0, slot = it / every % 3;
    bool settled = false, stop = false;
    while (it < max_sweeps && !stop) {
        float d = 0.f, m = 0.f;
        int q = ((threadIdx.x >> 6) * t.size + t.rank) * 64 + (threadIdx.x & 63);
        for (q = t.late ? n : q; q < n; q += t.size * kSweepThreads) {
            const int i = list[q];
            const int2 r = a.crange[i];
            float l = a.g[i];
            const float was = agent_load(a.lam + i);
            for (int k = r.x; k < r.y; ++k) l += a.calpha[k] * agent_load(a.lam + a.cchild[k]);
            d = fmaxf(d, fabsf(l - was));
            m = fmaxf(m, fabsf(l));
            agent_store(a.lam + i, l);
        }
        ++it;
        const bool check = it % every == 0 || it == max_sweeps;
        if (check) {   // uniform over the team
            for (int o = 32; o > 0; o >>= 1) {
                d = fmaxf(d, __shfl_xor(d, o));
                m = fmaxf(m, __shfl_xor(m, o));
            }
            if ((threadIdx.x & 63) == 0) {
                red[0][threadIdx.x >> 6] = d;
                red[1][threadIdx.x >> 6] = m;
            }
            __syncthreads();
            if (threadIdx.x < 2) {
                float v = 0.f;
                for (int w = 0; w < kSweepThreads / 64; ++w) v = fmaxf(v, red[threadIdx.x][w]);
                (void)__hip_atomic_fetch_max(threadIdx.x ? &a.ctl->lmax[slot] : &a.ctl->diff[slot], __float_as_int(v),
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        team_sync(t, it, &zero, before, first);
        if (check) {
            const float ch = __int_as_float(agent_load(&a.ctl->diff[slot]));
            settled = ch <= tol * __int_as_float(agent_load(&a.ctl->lmax[slot]));
            stop = exhaust ? ch == 0.f : settled;
            // the last check's slot, which everybody has read, for the check after the next
            if (t.rank == 0 && threadIdx.x == 0) {
                agent_store(&a.ctl->diff[(slot + 2) % 3], 0);
                agent_store(&a.ctl->lmax[(slot + 2) % 3], 0);
            }
            slot = (slot + 1) % 3;
        }
    }
    team_leave(t);
    if (t.rank == 0 && threadIdx.x == 0) {
        a.ctl->sweeps += it;
        a.ctl->settled = settled;
    }
}

}  // namespace

int gbp_adj_lists(const AdjGraph& a, const float* dL_dT, const int* node_user, hipStream_t s) {
    ProfScope ps(GBP_PROF_CHILD, s);
    const int nb = gbp_blocks(a.n_v, TPB);
    k_adj_link<<<gbp_blocks(a.n_v, kLinkThreads), kLinkThreads, 0, s>>>(a, dL_dT, node_user);
    k_child_fill<<<nb, TPB, 0, s>>>(a);
    k_child_sort<<<nb, TPB, 0, s>>>(a);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

// Blocks of the team's launch, an eighth of them on one XCD.  Backward of tetrahedra,
// 16 / 32 blocks of one XCD / 64 of all: 12k vertices 256 / 275 / 290 us, 100k 887 / 894 /
// 931 us, 500k 2360 / 2250 / 2250 us; from a million on one XCD's requests bound it
// (6M: 24.4 ms by one XCD, 23.5 by all).  Another 500k mesh: 4.8 ms by 2 blocks of one
// XCD, 1.4 by 32.
constexpr int kWalkFewBlocks = 128, kWalkManyBlocks = 256;
constexpr int kWalkFewVerts = 200000;
constexpr int kWalkOneXcd = 1 << 20;

int gbp_adj_walk(const AdjGraph& a, int levels, bool narrow, hipStream_t s) {
    ProfScope ps(GBP_PROF_ADJ_LEVEL, s);
    if (narrow) {
        k_adj_walk_block<<<1, kWalkThreads, 0, s>>>(a, levels);
    } else {
        const int blocks = a.n_v < kWalkFewVerts ? kWalkFewBlocks : kWalkManyBlocks;
        k_adj_walk_team<<<blocks, kWalkThreads, 0, s>>>(a, levels, a.n_v <= kWalkOneXcd);
    }
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

int gbp_adj_sweeps(const AdjGraph& a, int* list, bool build, int from, int count, float tol, bool exhaust,
                   hipStream_t s) {
    ProfScope ps(GBP_PROF_AUX, s);
    if (build) k_adj_remaining<<<gbp_blocks(a.n_v, kLinkThreads), kLinkThreads, 0, s>>>(a, list);
    if (a.n_v <= kSweepTeamVerts) {
        k_sweeps_reset<<<1, 256, 0, s>>>(a.team, a.ctl);
        if (count > 0) k_adj_sweeps<<<kSweepBlocks, kSweepThreads, 0, s>>>(a, list, count, tol, exhaust);
    } else {
        const int grid = std::min(gbp_blocks(a.n_v, TPB), 1024);
        for (int it = from; it < from + count; ++it) k_adj_sweep<<<grid, TPB, 0, s>>>(a, list, it);
        k_adj_swept<<<1, 64, 0, s>>>(a.ctl, from, count, tol);
    }
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

int gbp_adj_sweep_batch(const AdjGraph& a) { return a.n_v > kSweepTeamVerts ? 16 : 1024; }
