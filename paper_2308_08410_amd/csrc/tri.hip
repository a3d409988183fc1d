// Geodesic-BP on triangle meshes (d = 2), the setting of the paper's 2-D study
// (Sec. 3.1): the same three steps as on tetrahedra with a segment as the local
// simplex.
//
// * forward: Alg. 2 as an active queue of vertices, a group of lanes per queued
//   vertex evaluating the local problems of its triangles (Sec. 2.2 Eq. (upwind_eq_lsqr)
//   with d = 2: two vertex candidates and one interior candidate, predicated);
// * backward: geodesic parents in FP64 (the argmin is a decision taken by
//   floating point: same precision as the reference), the adjoint
//   lambda = g + P^T lambda (Sec. 2.3 Eq. (dto_grad)) as a leaves-first walk
//   over device-built child lists in a fixed order (walk.h, the tetrahedral path's:
//   a vertex finished once all its children are, two-cycles solved as pairs),
//   Gauss-Seidel sweeps over just the vertices that longer cycles leave unfinished
//   (geometric convergence there), and the gradients w.r.t. the triangle tensors,
//   nodal velocity scales and root onsets.
//
// Meshes of the 2-D study are small (thousands of vertices) and their fronts narrow, so the
// forward's rounds run inside one launch.
#include <math.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstddef>
#include <vector>

#include "gbp_internal.h"
#include "gbp_test_hooks.h"
#include "local_solve.h"
#include "team.h"
#include "walk.h"

struct TriCtl {
    int count;           // forward: vertices around the roots
    int err;
    unsigned long long solves, updates;
    int unreached;
    AdjCtl adj;          // adjoint walk
    int rounds;          // forward: rounds with work
    int left;            // forward: queued vertices after the last
};

// Incidence of a vertex: the triangle's other two (in increasing local order) and the Q of
// the edges to them with the roots of its diagonal.
struct __align__(32) TriInc {
    int a, b;
    float qaa, qbb, qab, sa, sb;
    int pad;
};

struct gbp_tri_plan_s {
    int device = 0;
    int n_v = 0, n_t = 0;
    float2* xy = nullptr;
    int4* tri = nullptr;          // vertex ids (w unused)
    int* vptr = nullptr;          // [n_v+1] incidence: entries (tri << 2 | slot) sorted by tri
    int* vent = nullptr;
    int* nbp = nullptr;           // [n_v+1] unique neighbours
    int* nb = nullptr;
    int4* info = nullptr;         // incidence and neighbour ranges of a vertex
    int* tpos = nullptr;          // [3 n_t] position of a triangle's incidences
    TriInc* inc = nullptr;        // [3 n_t] as vent; of the forward's metric
    TeamListCap list_cap{};       // a team's lists
    int team_blocks = 0;          // its most members
    TeamLimits team_limits;       // of every team (tests)
    float* T = nullptr;
    int* now[2] = {nullptr, nullptr};   // a team's times, and each round's improvements
    unsigned long long* gain[2] = {nullptr, nullptr};
    float* troot = nullptr;
    int* q0 = nullptr;            // first queue of the forward, leaves of the adjoint
    int* q[2] = {nullptr, nullptr};   // a team's lists
    int* mark = nullptr;
    TriCtl* ctl = nullptr;
    TriCtl* ctl_host = nullptr;
    int* par = nullptr;
    int4* pnode = nullptr;        // weighted parents a, b (-1: none)
    float4* pa = nullptr;         // alpha_a, alpha_b, best, root_self
    int2* crange = nullptr;       // child lists and walk state: see AdjGraph
    int* cfill = nullptr;         // fill cursors, then the vertices the walk left
    int* done = nullptr;          // child counts, then finished flags
    AdjRec* rec = nullptr;
    float* over = nullptr;        // [2 n_v]
    int* ready[2] = {nullptr, nullptr};
    TeamCtl* team = nullptr;
    int* cchild = nullptr;        // [2 n_v]
    float* calpha = nullptr;
    float* lam = nullptr;
    float* g = nullptr;
    float* dsbar = nullptr;
    int stamp = 1;
    int last_levels = 0, last_cyclic = 0, last_sweeps = 0;   // of the last backward
    int max_rounds = 20000;
    float eps_rel = 1.0f / (1 << 20);
};

namespace {

constexpr int TPB = 256;
// Meshes whose adjoint levels one block walks.  It depends on their width, which is known
// only once walked.  Fronts about narrow levels (27 vertices at 10k, 177 at 250k, 209 at
// 900k), iteration by one block and by a team: 10k 1.20 and 1.95 ms, 60k 2.70 and 3.60,
// 250k 7.2 and 8.5, 900k 22.8 and 24.7.  About wide ones (121 at 25k, 274 at 60k, 498 at
// 250k, 1,186 at 1M), backward: 25k 0.53 and 0.77, 60k 0.88 and 0.88, 250k 3.06 and 1.96,
// 1M 11.9 and 3.5, 2M 28.2 and 10.8.
constexpr int kTriWalkBlockVerts = 1 << 20;

template <typename T>
int tri_alloc(T** p, size_t n) {
    if (n == 0) n = 1;
    if (hipMalloc((void**)p, n * sizeof(T)) != hipSuccess) {
        gbp_set_error("hipMalloc of %zu bytes failed", n * sizeof(T));
        return GBP_ERR_NOMEM;
    }
    return GBP_OK;
}

void tri_free(gbp_tri_plan p) {
    if (!p) return;
    void* ptrs[] = {p->xy,    p->tri,   p->vptr,   p->vent,   p->nbp,    p->nb,
                    p->T,     p->troot, p->q[0],   p->q[1],   p->mark,   p->ctl,    p->par,
                    p->pnode, p->pa,    p->crange, p->cfill,  p->cchild, p->calpha, p->lam,
                    p->g,     p->dsbar, p->done,   p->rec,    p->over,
                    p->ready[0], p->ready[1], p->team, p->info, p->tpos, p->inc, p->q0,
                    p->now[0], p->now[1], p->gain[0], p->gain[1]};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    if (p->ctl_host) (void)hipHostFree(p->ctl_host);
    delete p;
}

__device__ __forceinline__ bool fin(float x) { return x - x == 0.f; }

// block reductions (one atomic per block instead of one per thread)
__device__ __forceinline__ unsigned long long tri_block_sum(unsigned long long v) {
    __shared__ unsigned long long part[16];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    unsigned long long t = 0;
    for (int w = 0; w < (int)blockDim.x / 64; ++w) t += part[w];
    return t;
}

// face (a, b) of the triangle seen from its local vertex k: the other two
// vertices in increasing local order
__device__ __forceinline__ void tri_face(int4 t, int k, int& i, int& a, int& b) {
    i = k == 0 ? t.x : k == 1 ? t.y : t.z;
    a = k == 0 ? t.y : t.x;
    b = k == 2 ? t.y : t.z;
}

// d = 2 local solve in precision R: vertex a, vertex b, interior (first wins on
// ties); unreached vertices leave the other vertex's candidate.
// sa, sb: the roots of qaa and qbb.
template <typename R>
__device__ __forceinline__ R tri_local(R qaa, R qbb, R qab, R sa, R sb, R pa, R pb, R* alpha_a = nullptr) {
    const R INF = gbp_inf<R>();
    const bool fa = pa < INF, fb = pb < INF;
    R best = fa ? pa + sa : INF;
    R al = fa ? R(1) : R(0);
    const R vb = fb ? pb + sb : INF;
    if (vb < best) { best = vb; al = R(0); }
    if (fa && fb) {
        const R m = fmin(pa, pb);
        R v, ua, ub;
        edge_candidate<R>(qaa, qbb, qab, pa - m, pb - m, true, v, ua, ub);
        if (m + v < best) { best = m + v; al = ua / (ua + ub); }
    }
    if (alpha_a) *alpha_a = al;
    return best;
}

// Checks the inputs; inc (or null): the record of each of the triangle's incidences, at tpos.
__global__ void k_tri_metric(const float* __restrict__ D, const float* __restrict__ vscale,
                             const int4* __restrict__ tri, int n_t,
                             const float2* __restrict__ xy, const int* __restrict__ tpos,
                             TriInc* __restrict__ inc, TriCtl* ctl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_t) return;
    const int4 v = tri[t];
    float sbar = 1.f;
    if (vscale) {
        const float s0 = vscale[v.x], s1 = vscale[v.y], s2 = vscale[v.z];
        if (!(s0 > 0.f && s1 > 0.f && s2 > 0.f && fin(s0) && fin(s1) && fin(s2)))
            atomicOr(&ctl->err, ERRBIT_VSCALE);
        sbar = (s0 + s1 + s2) * (1.f / 3.f);
    }
    const float xx = D[3 * (size_t)t], yy = D[3 * (size_t)t + 1], dxy = D[3 * (size_t)t + 2];
    const float det = xx * yy - dxy * dxy;
    if (!(fin(xx) && fin(yy) && fin(dxy))) atomicOr(&ctl->err, ERRBIT_D_NONFINITE);
    else if (!(xx > 0.f && det > 0.f)) atomicOr(&ctl->err, ERRBIT_D_NOT_SPD);
    if (!inc) return;
    const float s = 1.f / (det * sbar * sbar);
    const float3 m = make_float3(yy * s, xx * s, -dxy * s);   // D_eff^-1
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int i, a, b;
        tri_face(v, k, i, a, b);
        const float2 xi = xy[i], xa = xy[a], xb = xy[b];
        const float ax = xa.x - xi.x, ay = xa.y - xi.y, bx = xb.x - xi.x, by = xb.y - xi.y;
        TriInc r;
        r.a = a;
        r.b = b;
        r.qaa = ax * (m.x * ax + m.z * ay) + ay * (m.z * ax + m.y * ay);
        r.qbb = bx * (m.x * bx + m.z * by) + by * (m.z * bx + m.y * by);
        r.qab = ax * (m.x * bx + m.z * by) + ay * (m.z * bx + m.y * by);
        r.sa = gbp_sqrt(r.qaa);
        r.sb = gbp_sqrt(r.qbb);
        r.pad = 0;
        inc[tpos[3 * (size_t)t + k]] = r;
    }
}

__global__ void k_tri_roots(const int* __restrict__ root_node, const float* __restrict__ root_t,
                            int n_roots, int n_v, float* __restrict__ troot, float* __restrict__ T,
                            int* __restrict__ now0, int* __restrict__ now1, int cold,
                            const int* __restrict__ nbp, const int* __restrict__ nb,
                            int* __restrict__ q0, int* __restrict__ mark, int stamp, TriCtl* ctl) {
    if (threadIdx.x == 0) {
        for (int r = 0; r < n_roots; ++r) {
            const int u = root_node[r];
            const float t = root_t[r];
            if (u < 0 || u >= n_v) { atomicOr(&ctl->err, ERRBIT_ROOT_RANGE); continue; }
            if (!fin(t)) { atomicOr(&ctl->err, ERRBIT_ROOT_NONFINITE); continue; }
            troot[u] = fminf(troot[u], t);
            if (cold) T[u] = fminf(T[u], t);
            if (now0) now0[u] = now1[u] = ordered(T[u]);
        }
    }
    __syncthreads();
    if (!cold) return;
    for (int r = threadIdx.x; r < n_roots; r += blockDim.x) {
        const int u = root_node[r];
        if (u < 0 || u >= n_v) continue;
        for (int a = nbp[u]; a < nbp[u + 1]; ++a) {
            const int w = nb[a];
            if (atomicMax(&mark[w], stamp) < stamp) q0[atomicAdd(&ctl->count, 1)] = w;
        }
    }
}

// ------------------------------------------------------------------ relaxation rounds
// One queued vertex by a group of 8 lanes, which take its triangles (and then its
// neighbours) in turn: a round is a chain of dependent loads, one triangle's and not the
// sum over the vertex's.  The chain is queue -> info -> records (the two other
// vertices and their Q, computed with the metric) -> T -> solve -> marks; the neighbours
// are read with the records.  (4 lanes: 6% slower at 2,700 nodes, 3% at 250,000.)
constexpr int kTriLanes = 8;

struct TriRelax {
    const int4* info;     // per vertex: its incidences [x, y), its neighbours [z, w)
    const TriInc* inc;
    const int* nb;
    float eps_rel;
};

// A round is a Jacobi step: all its vertices see the times of the round before, so that
// times and the parents chosen by them do not depend on which vertex was first.
template <typename Load, typename Done, typename Push>
__device__ __forceinline__ void tri_vertex(const TriRelax& g, int i, Load load, Done done, Push push,
                                           unsigned& solves, unsigned& upd) {
    const int lane = threadIdx.x & (kTriLanes - 1);
    const int4 at = g.info[i];
    const int w0 = at.z + lane < at.w ? g.nb[at.z + lane] : -1;
    const float told = load(i);
    float best = told;
    for (int e = at.x + lane; e < at.y; e += kTriLanes) {
        const int4* r = reinterpret_cast<const int4*>(g.inc + e);
        const int4 r0 = r[0], r1 = r[1];
        best = fminf(best, tri_local<float>(__int_as_float(r0.z), __int_as_float(r0.w), __int_as_float(r1.x),
                                            __int_as_float(r1.y), __int_as_float(r1.z), load(r0.x), load(r0.y)));
        ++solves;
    }
#pragma unroll
    for (int o = 1; o < kTriLanes; o <<= 1) best = fminf(best, __shfl_xor(best, o));
    if (lane == 0) done(best, best < told);
    const bool changed = (told < GBP_INF) ? (best < told - g.eps_rel * fmaxf(1.f, fabsf(told)))
                                          : (best < GBP_INF);
    if (!changed) return;
    if (lane == 0) ++upd;
    if (w0 >= 0) push(w0);
    for (int a = at.z + lane + kTriLanes; a < at.w; a += kTriLanes) push(g.nb[a]);
}

// Narrow fronts: all rounds by one block, with T, the queues and their marks in LDS and a
// block barrier between rounds.  Bound by the solves of one CU (2,704 nodes, 240 queued
// vertices a round: 3.6 us a round; as a launch a round 5.3 us and the gap to the next).
// An iteration by one block and by a team takes 666 and 755 us at 2,700 nodes, 798 and
// 770 at 4,000, 1237 and 1010 at 8,000.
constexpr int kTriBlockVerts = 4096;
constexpr int kTriThreads = 1024;

constexpr size_t tri_block_lds(int n_v) { return (size_t)n_v * 12 + 2 * (((size_t)n_v + 31) / 32) * 4 + 16; }

__global__ void __launch_bounds__(kTriThreads)
    k_tri_rounds_block(TriRelax g, int n_v, float* __restrict__ T, const int* __restrict__ q0, TriCtl* ctl, int rounds) {
    extern __shared__ float lds[];
    const int words = (n_v + 31) / 32, tid = threadIdx.x;
    float* Ts = lds;
    float* Tn = Ts + n_v;                                                            // by queue position
    unsigned* queued = reinterpret_cast<unsigned*>(Tn + n_v);                        // [2][words]
    unsigned short* q = reinterpret_cast<unsigned short*>(queued + 2 * words);       // [2][n_v]
    __shared__ int count[3];
    if (ctl->err) return;
    for (int i = tid; i < n_v; i += kTriThreads) Ts[i] = T[i];
    for (int i = tid; i < 2 * words; i += kTriThreads) queued[i] = 0;
    const int n0 = ctl->count;
    for (int i = tid; i < n0; i += kTriThreads) q[i] = (unsigned short)q0[i];
    if (tid < 3) count[tid] = tid == 0 ? n0 : 0;
    __syncthreads();
    unsigned solves = 0, upd = 0;
    unsigned long long all_solves = 0, all_upd = 0;
    int r = 0, n = n0;
    while (n > 0 && r < rounds) {
        const unsigned short* in = q + (size_t)(r & 1) * n_v;
        unsigned short* out = q + (size_t)((r + 1) & 1) * n_v;
        unsigned* mark = queued + ((r + 1) & 1) * words;
        int* n_out = &count[(r + 1) % 3];
        if (tid == 0) count[(r + 2) % 3] = 0;
        for (int i = tid; i < words; i += kTriThreads) queued[(r & 1) * words + i] = 0;
        for (int k = tid / kTriLanes; k < n; k += kTriThreads / kTriLanes)
            tri_vertex(g, in[k], [&](int x) { return Ts[x]; }, [&](float t, bool) { Tn[k] = t; },
                       [&](int x) {
                           const unsigned bit = 1u << (x & 31);
                           if (!(atomicOr(mark + (x >> 5), bit) & bit)) out[atomicAdd(n_out, 1)] = (unsigned short)x;
                       },
                       solves, upd);
        __syncthreads();
        for (int k = tid; k < n; k += kTriThreads) Ts[in[k]] = Tn[k];
        all_solves += solves;
        all_upd += upd;
        solves = upd = 0;
        __syncthreads();
        ++r;
        n = count[r % 3];
    }
    for (int i = tid; i < n_v; i += kTriThreads) T[i] = Ts[i];
    all_solves = tri_block_sum(all_solves);
    all_upd = tri_block_sum(all_upd);
    if (tid == 0) {
        ctl->solves = all_solves;
        ctl->updates = all_upd;
        ctl->rounds = r;
        ctl->left = n;
    }
}

// Wider ones: all rounds by a team of blocks; member b writes its pushes to
// list[cap * b ...], read with the prefix of the members' counts.
// Round r reads the times of `now[r & 1]` and lowers those of the other array, which holds
// the improvements of all rounds but the last; a member repeats its own of that one
// (gain, by position in the round's queue) before it adds its new ones.
// Bound by the chain of agent-scope accesses and, with many thousand vertices a round, by
// their number: 250,000 nodes (12,000 vertices a round), 8.3 us a round and 12.8 us as a
// launch a round; an iteration takes 7.6 ms with 128 blocks, 7.9 with 64, 8.1 with 256;
// at 60,000 nodes 2.99, 2.88 and 3.4; at 8,000 1011 us with 32 blocks, 1031 with 64.
// (Blocks of one XCD only: 11.6 ms at 250,000, 1087 us at 8,000.)
int tri_team_blocks(int n_v) { return n_v < 24576 ? 32 : n_v < 163840 ? 64 : 128; }

struct TriLists {
    int *now0, *now1;                    // [n_v] times, as ordered integers
    unsigned long long *gain0, *gain1;   // [n_v] vertex << 32 | its time, or all ones
    int *list0, *list1;
    const int* q0;
    int* mark;
};

__global__ void __launch_bounds__(kTriThreads)
    k_tri_rounds_team(TriRelax g, int n_v, TeamListCap list_cap, TriLists q, int stamp, TeamCtl* team, TriCtl* ctl, int rounds,
                      float* __restrict__ T, TeamLimits limits) {
    __shared__ int before[kTeamMax + 1], count[3];
    if (ctl->err) return;
    if (threadIdx.x < 3) count[threadIdx.x] = 0;
    Team t;
    if (!team_join(team, false, t, limits)) return;
    int n = t.late ? 1 : ctl->count, r = t.late ? t.late - 1 : 0, m = 0, p0 = 0, p1 = 0;
    size_t cap = list_cap(t.size), cap_out = cap;
    unsigned long long all_solves = 0, all_upd = 0;
    while (n > 0 && r < rounds) {
        const bool odd = r & 1;
        const int* in = odd ? q.list1 : q.list0;
        int* out = (odd ? q.list0 : q.list1) + cap_out * t.rank;
        int* n_out = &count[(r + 1) % 3];
        const int* T0 = odd ? q.now1 : q.now0;
        int* T1 = odd ? q.now0 : q.now1;
        const unsigned long long* last = odd ? q.gain0 : q.gain1;
        unsigned long long* gain = odd ? q.gain1 : q.gain0;
        // (the last waves, which have the fewest vertices)
        for (int k = p0 + kTriThreads - 1 - (int)threadIdx.x; k < p1; k += kTriThreads) {
            const unsigned long long v = agent_load(last + k);
            if (v != ~0ull)
                (void)__hip_atomic_fetch_min(T1 + (int)(v >> 32), (int)(unsigned)v, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        }
        const int next = stamp + r + 1;
        unsigned solves = 0, upd = 0;
        if (!t.late) team_share(t, n, p0, p1);
        for (int k = p0 + threadIdx.x / kTriLanes; k < p1; k += kTriThreads / kTriLanes) {
            int i;
            if (r == 0) {
                i = q.q0[k];
            } else {
                while (before[m + 1] <= k) ++m;
                i = agent_load(in + cap * m + (k - before[m]));
            }
            tri_vertex(g, i, [&](int x) { return from_ordered(agent_load(T0 + x)); },
                       [&](float best, bool lower) {
                           const int b = ordered(best);
                           const unsigned long long v = lower ? ((unsigned long long)(unsigned)i << 32) | (unsigned)b : ~0ull;
                           __hip_atomic_store(gain + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                           if (lower)
                               (void)__hip_atomic_fetch_min(T1 + i, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                       },
                       [&](int x) {
                           if (__hip_atomic_fetch_max(q.mark + x, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < next)
                               agent_store(out + atomicAdd(n_out, 1), x);
                       },
                       solves, upd);
        }
        all_solves += solves;
        all_upd += upd;
        ++r;
        n = team_sync(t, r, n_out, before, m);
        cap = cap_out;
        if (t.size != t.was) cap_out = list_cap(t.size);
        if (threadIdx.x == 0) count[(r + 2) % 3] = 0;   // read by all before the sync, used after the next
    }
    team_leave(t);
    const int* T0 = r & 1 ? q.now1 : q.now0;
    int i0, i1;
    team_share(t, n_v, i0, i1);
    for (int i = i0 + (int)threadIdx.x; i < i1; i += kTriThreads) T[i] = from_ordered(agent_load(T0 + i));
    all_solves = tri_block_sum(all_solves);
    all_upd = tri_block_sum(all_upd);
    if (threadIdx.x == 0) {
        atomicAdd(&ctl->solves, all_solves);
        atomicAdd(&ctl->updates, all_upd);
        if (t.rank == 0) {
            ctl->rounds = r;
            ctl->left = n;
        }
    }
}

__global__ void k_tri_ctl_reset(TriCtl* ctl, TeamCtl* team) {
    for (int k = threadIdx.x; k < (int)(sizeof(TeamCtl) / sizeof(int)); k += blockDim.x)
        reinterpret_cast<int*>(team)[k] = 0;
    if (threadIdx.x == 0) *ctl = TriCtl{};
}

__global__ void k_tri_fill(float* __restrict__ x, float v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

// No onset and, for a cold start, no time anywhere (now0, now1: a team's, or null).
__global__ void k_tri_unreached(float* __restrict__ troot, float* __restrict__ T, int* __restrict__ now0,
                                int* __restrict__ now1, int n_v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_v) return;
    troot[i] = GBP_INF;
    if (T) T[i] = GBP_INF;
    if (now0) now0[i] = now1[i] = __float_as_int(GBP_INF);
}

__global__ void k_tri_fill_i(int* __restrict__ x, int v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

__global__ void k_tri_count_inf(const float* __restrict__ T, int n_v, TriCtl* ctl) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_v && !(T[i] < GBP_INF)) atomicAdd(&ctl->unreached, 1);
}

// FP64 geodesic parent of every vertex: lowest triangle among local values
// within 1e-12 max(1, |T|) of the minimum; a vertex whose smallest onset does
// not exceed that minimum is a root (its own parent).  The parents that carry weight
// go to pnode and count the vertex among their children (ccnt, cleared before).
__global__ void k_tri_parent(const float2* __restrict__ xy, const int4* __restrict__ tri,
                             const float* __restrict__ D, const float* __restrict__ vscale,
                             const int* __restrict__ vptr, const int* __restrict__ vent,
                             const float* __restrict__ T, const float* __restrict__ troot, int n_v,
                             int* __restrict__ par, int4* __restrict__ pnode,
                             float4* __restrict__ pa, int* __restrict__ ccnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_v) return;
    par[i] = -1;
    pnode[i] = make_int4(-1, -1, -1, -1);
    pa[i] = make_float4(0.f, 0.f, GBP_INF, 0.f);
    const double Ti = T[i];
    if (!(T[i] < GBP_INF)) return;
    const double xi = xy[i].x, yi = xy[i].y;
    double best = gbp_inf<double>();
    for (int pass = 0; pass < 2; ++pass) {
        const double tol = 1e-12 * fmax(1.0, fabs(Ti));
        for (int e = vptr[i]; e < vptr[i + 1]; ++e) {
            const int code = vent[e];
            const int t = code >> 2;
            const int4 tv = tri[t];
            int ii, a, b;
            tri_face(tv, code & 3, ii, a, b);
            double sbar = 1.0;
            if (vscale) sbar = ((double)vscale[tv.x] + vscale[tv.y] + vscale[tv.z]) / 3.0;
            const double dxx = D[3 * (size_t)t], dyy = D[3 * (size_t)t + 1], dxy = D[3 * (size_t)t + 2];
            const double s = 1.0 / ((dxx * dyy - dxy * dxy) * sbar * sbar);
            const double mxx = dyy * s, myy = dxx * s, mxy = -dxy * s;
            const double ax = xy[a].x - xi, ay = xy[a].y - yi, bx = xy[b].x - xi, by = xy[b].y - yi;
            const double qaa = ax * (mxx * ax + mxy * ay) + ay * (mxy * ax + myy * ay);
            const double qbb = bx * (mxx * bx + mxy * by) + by * (mxy * bx + myy * by);
            const double qab = ax * (mxx * bx + mxy * by) + ay * (mxy * bx + myy * by);
            const double ta = T[a] < GBP_INF ? (double)T[a] : gbp_inf<double>();
            const double tb = T[b] < GBP_INF ? (double)T[b] : gbp_inf<double>();
            double al;
            const double v = tri_local<double>(qaa, qbb, qab, gbp_sqrt(qaa), gbp_sqrt(qbb), ta, tb, &al);
            if (pass == 0) {
                best = fmin(best, v);
            } else if (v <= best + tol && v < gbp_inf<double>()) {
                if (troot[i] < GBP_INF && (double)troot[i] <= best) {   // a root: its own parent
                    pa[i] = make_float4(0.f, 0.f, (float)best, 1.f);
                } else {
                    par[i] = t;
                    const float wa = (float)al, wb = (float)(1.0 - al);
                    pnode[i] = make_int4(wa > 0.f ? a : -1, wb > 0.f ? b : -1, -1, -1);
                    pa[i] = make_float4(wa, wb, (float)best, 0.f);
                    if (wa > 0.f) atomicAdd(&ccnt[a], 1);
                    if (wb > 0.f) atomicAdd(&ccnt[b], 1);
                }
                return;
            }
        }
        if (pass == 0 && !(best < gbp_inf<double>())) break;
    }
    if (troot[i] < GBP_INF) pa[i] = make_float4(0.f, 0.f, (float)best, 1.f);   // root
}

__global__ void k_tri_grad_tri(const float2* __restrict__ xy, const int4* __restrict__ tri,
                               const float* __restrict__ D, const float* __restrict__ vscale,
                               const int* __restrict__ par, const int4* __restrict__ pnode,
                               const float4* __restrict__ pa, const float* __restrict__ lam, int n_v,
                               float* __restrict__ dD, float* __restrict__ dsbar) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_v) return;
    const int t = par[i];
    const float l = lam[i];
    if (t < 0 || l == 0.f) return;
    int4 p = pnode[i];
    if (p.x < 0) p.x = i;   // no weight: any vertex does
    if (p.y < 0) p.y = i;
    const float4 w = pa[i];
    const int4 tv = tri[t];
    double sbar = 1.0;
    if (vscale) sbar = ((double)vscale[tv.x] + vscale[tv.y] + vscale[tv.z]) / 3.0;
    const double dxx = D[3 * (size_t)t], dyy = D[3 * (size_t)t + 1], dxy = D[3 * (size_t)t + 2];
    const double idet = 1.0 / (dxx * dyy - dxy * dxy);
    const double ex = w.x * ((double)xy[p.x].x - xy[i].x) + w.y * ((double)xy[p.y].x - xy[i].x);
    const double ey = w.x * ((double)xy[p.x].y - xy[i].y) + w.y * ((double)xy[p.y].y - xy[i].y);
    const double ux = (dyy * ex - dxy * ey) * idet, uy = (dxx * ey - dxy * ex) * idet;   // D^-1 e
    const double h = sqrt((ex * ux + ey * uy) / (sbar * sbar));
    if (!(h > 0.0)) return;
    if (dD) {
        const double cf = -(double)l / (2.0 * sbar * sbar * h);
        atomicAdd(&dD[3 * (size_t)t], (float)(cf * ux * ux));
        atomicAdd(&dD[3 * (size_t)t + 1], (float)(cf * uy * uy));
        atomicAdd(&dD[3 * (size_t)t + 2], (float)(2.0 * cf * ux * uy));
    }
    atomicAdd(&dsbar[t], (float)((double)l * (-h / sbar)));
}

__global__ void k_tri_grad_node(const int* __restrict__ vptr, const int* __restrict__ vent,
                                const float* __restrict__ dsbar, int n_v, float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_v) return;
    float s = 0.f;
    for (int e = vptr[i]; e < vptr[i + 1]; ++e) s += dsbar[vent[e] >> 2];
    out[i] = s * (1.f / 3.f);
}

__global__ void k_tri_grad_root(const int* __restrict__ root_node, const float* __restrict__ root_t,
                                int n_roots, int n_v, const float4* __restrict__ pa,
                                const float* __restrict__ troot, const float* __restrict__ lam,
                                float* __restrict__ out) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_roots) return;
    const int u = root_node[r];
    float v = 0.f;
    if (u >= 0 && u < n_v) {
        bool active = pa[u].w > 0.5f && root_t[r] == troot[u];
        for (int q = 0; q < r && active; ++q)
            if (root_node[q] == u && root_t[q] == root_t[r]) active = false;
        if (active) v = lam[u];
    }
    out[r] = v;
}

int tri_check(gbp_tri_plan p, const float* D, const int32_t* root_node, const float* root_t,
              int n_roots) {
    if (!p) {
        gbp_set_error("null triangle plan");
        return GBP_ERR_ARG;
    }
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev != p->device) {
        gbp_set_error("triangle plan belongs to device %d, current device is %d", p->device, dev);
        return GBP_ERR_ARG;
    }
    if (!D || n_roots < 0 || (n_roots > 0 && (!root_node || !root_t))) {
        gbp_set_error("D is required, n_roots >= 0 with root arrays");
        return GBP_ERR_ARG;
    }
    return GBP_OK;
}

int tri_read(gbp_tri_plan p, hipStream_t s) {
    GBP_HIP(hipMemcpyAsync(p->ctl_host, p->ctl, sizeof(TriCtl), hipMemcpyDeviceToHost, s));
    GBP_HIP(hipStreamSynchronize(s));
    return GBP_OK;
}

// metric, onsets and (cold) the first queue; cold = 0 leaves T alone
int tri_prepare(gbp_tri_plan p, const float* D, const float* vscale, const int32_t* root_node,
                const float* root_t, int n_roots, bool cold, hipStream_t s) {
    const int n_v = p->n_v;
    k_tri_ctl_reset<<<1, 256, 0, s>>>(p->ctl, p->team);
    if (p->stamp > (1 << 30)) {
        k_tri_fill_i<<<gbp_blocks(n_v, TPB), TPB, 0, s>>>(p->mark, 0, n_v);
        p->stamp = 1;
    }
    k_tri_metric<<<gbp_blocks(p->n_t, TPB), TPB, 0, s>>>(D, vscale, p->tri, p->n_t, p->xy, p->tpos,
                                                       cold ? p->inc : nullptr, p->ctl);
    k_tri_unreached<<<gbp_blocks(n_v, TPB), TPB, 0, s>>>(p->troot, cold ? p->T : nullptr,
                                                         cold ? p->now[0] : nullptr, p->now[1], n_v);
    k_tri_roots<<<1, TPB, 0, s>>>(root_node, root_t, n_roots, n_v, p->troot, p->T, cold ? p->now[0] : nullptr,
                                  p->now[1], cold ? 1 : 0, p->nbp, p->nb, p->q0, p->mark, p->stamp, p->ctl);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

}  // namespace

extern "C" int gbp_tri_plan_create(const float* xy, int n_v, const int32_t* tris, int n_t,
                                   gbp_tri_plan* out) {
    if (!out || !xy || !tris || n_v < 1 || n_t < 1) {
        gbp_set_error("tri_plan_create: xy, tris, out required; n_v, n_t >= 1");
        return GBP_ERR_ARG;
    }
    *out = nullptr;
    for (int i = 0; i < 2 * n_v; ++i)
        if (!std::isfinite(xy[i])) {
            gbp_set_error("non-finite coordinate at vertex %d", i / 2);
            return GBP_ERR_NONFINITE;
        }
    for (int t = 0; t < n_t; ++t) {
        const int32_t* v = tris + 3 * (size_t)t;
        for (int k = 0; k < 3; ++k)
            if (v[k] < 0 || v[k] >= n_v) {
                gbp_set_error("triangle %d: vertex id out of range", t);
                return GBP_ERR_ARG;
            }
        if (v[0] == v[1] || v[0] == v[2] || v[1] == v[2]) {
            gbp_set_error("triangle %d repeats a vertex", t);
            return GBP_ERR_ARG;
        }
        const double ax = xy[2 * v[1]] - xy[2 * v[0]], ay = xy[2 * v[1] + 1] - xy[2 * v[0] + 1];
        const double bx = xy[2 * v[2]] - xy[2 * v[0]], by = xy[2 * v[2] + 1] - xy[2 * v[0] + 1];
        const double cx = bx - ax, cy = by - ay;
        const double l2 = std::max(std::max(ax * ax + ay * ay, bx * bx + by * by), cx * cx + cy * cy);
        if (!(std::fabs(ax * by - ay * bx) > 1e-7 * l2)) {
            gbp_set_error("triangle %d is degenerate", t);
            return GBP_ERR_DEGENERATE_TET;
        }
    }
    // incidence (sorted by triangle within a vertex) and unique neighbours
    std::vector<int> vptr(n_v + 1, 0), vent((size_t)3 * n_t), tpos((size_t)3 * n_t);
    for (int t = 0; t < n_t; ++t)
        for (int k = 0; k < 3; ++k) vptr[tris[3 * (size_t)t + k] + 1]++;
    for (int i = 0; i < n_v; ++i) vptr[i + 1] += vptr[i];
    {
        std::vector<int> cur(vptr.begin(), vptr.end() - 1);
        for (int t = 0; t < n_t; ++t)
            for (int k = 0; k < 3; ++k) {
                const int e = cur[tris[3 * (size_t)t + k]]++;
                vent[e] = (t << 2) | k;
                tpos[3 * (size_t)t + k] = e;
            }
    }
    std::vector<int> nbp(n_v + 1, 0), nb;
    nb.reserve((size_t)6 * n_v);
    std::vector<int> tmp;
    for (int i = 0; i < n_v; ++i) {
        tmp.clear();
        for (int e = vptr[i]; e < vptr[i + 1]; ++e) {
            const int t = vent[e] >> 2;
            for (int k = 0; k < 3; ++k)
                if (tris[3 * (size_t)t + k] != i) tmp.push_back(tris[3 * (size_t)t + k]);
        }
        std::sort(tmp.begin(), tmp.end());
        tmp.erase(std::unique(tmp.begin(), tmp.end()), tmp.end());
        nb.insert(nb.end(), tmp.begin(), tmp.end());
        nbp[i + 1] = (int)nb.size();
    }
    std::vector<int4> info(n_v);
    std::vector<int> degree(n_v);
    for (int i = 0; i < n_v; ++i) {
        info[i] = make_int4(vptr[i], vptr[i + 1], nbp[i], nbp[i + 1]);
        degree[i] = nbp[i + 1] - nbp[i];
    }
    std::vector<float2> xy2(n_v);
    for (int i = 0; i < n_v; ++i) xy2[i] = make_float2(xy[2 * i], xy[2 * i + 1]);
    std::vector<int4> t4(n_t);
    for (int t = 0; t < n_t; ++t)
        t4[t] = make_int4(tris[3 * (size_t)t], tris[3 * (size_t)t + 1], tris[3 * (size_t)t + 2], 0);

    gbp_tri_plan p = new gbp_tri_plan_s();
    (void)hipGetDevice(&p->device);
    p->n_v = n_v;
    p->n_t = n_t;
    int rc = GBP_OK;
#define TRI_TRY(x)                  \
    if ((rc = (x)) != GBP_OK) {     \
        tri_free(p);                \
        return rc;                  \
    }
#define TRI_UP(dst, src, n)                                                                  \
    TRI_TRY(tri_alloc(&(dst), (n)));                                                        \
    if (hipMemcpy((dst), (src), (n) * sizeof(*(src)), hipMemcpyHostToDevice) != hipSuccess) { \
        gbp_set_error("upload failed");                                                      \
        tri_free(p);                                                                         \
        return GBP_ERR_HIP;                                                                  \
    }
    TRI_UP(p->xy, xy2.data(), (size_t)n_v);
    TRI_UP(p->tri, t4.data(), (size_t)n_t);
    TRI_UP(p->vptr, vptr.data(), (size_t)n_v + 1);
    TRI_UP(p->vent, vent.data(), (size_t)3 * n_t);
    TRI_UP(p->nbp, nbp.data(), (size_t)n_v + 1);
    TRI_UP(p->nb, nb.data(), nb.size());
    TRI_TRY(tri_alloc(&p->T, n_v));
    TRI_TRY(tri_alloc(&p->troot, n_v));
    TRI_UP(p->info, info.data(), (size_t)n_v);
    TRI_UP(p->tpos, tpos.data(), (size_t)3 * n_t);
    TRI_TRY(tri_alloc(&p->inc, (size_t)3 * n_t));
    TRI_TRY(tri_alloc(&p->q0, n_v));
    if (n_v > kTriBlockVerts) {
        p->team_blocks = tri_team_blocks(n_v);
        p->list_cap = team_list_cap(n_v, degree.data(), p->team_blocks);
        for (int k = 0; k < 2; ++k) {
            TRI_TRY(tri_alloc(&p->q[k], team_list_size(p->list_cap, p->team_blocks)));
            TRI_TRY(tri_alloc(&p->now[k], n_v));
            TRI_TRY(tri_alloc(&p->gain[k], n_v));
        }
    }
    TRI_TRY(tri_alloc(&p->mark, n_v));
    TRI_TRY(tri_alloc(&p->ctl, 1));
    TRI_TRY(tri_alloc(&p->par, n_v));
    TRI_TRY(tri_alloc(&p->pnode, n_v));
    TRI_TRY(tri_alloc(&p->pa, n_v));
    TRI_TRY(tri_alloc(&p->crange, n_v));
    TRI_TRY(tri_alloc(&p->cfill, n_v));
    TRI_TRY(tri_alloc(&p->done, n_v));
    TRI_TRY(tri_alloc(&p->rec, n_v));
    TRI_TRY(tri_alloc(&p->over, (size_t)2 * n_v));
    TRI_TRY(tri_alloc(&p->ready[0], walk_list_size(n_v)));
    TRI_TRY(tri_alloc(&p->ready[1], walk_list_size(n_v)));
    TRI_TRY(tri_alloc(&p->team, 1));
    TRI_TRY(tri_alloc(&p->cchild, (size_t)2 * n_v));
    TRI_TRY(tri_alloc(&p->calpha, (size_t)2 * n_v));
    TRI_TRY(tri_alloc(&p->lam, n_v));
    TRI_TRY(tri_alloc(&p->g, n_v));
    TRI_TRY(tri_alloc(&p->dsbar, n_t));
#undef TRI_UP
#undef TRI_TRY
    if (hipHostMalloc((void**)&p->ctl_host, sizeof(TriCtl)) != hipSuccess ||
        hipMemset(p->mark, 0, (size_t)n_v * sizeof(int)) != hipSuccess) {
        gbp_set_error("pinned control block or mark reset failed");
        tri_free(p);
        return GBP_ERR_HIP;
    }
    *out = p;
    return GBP_OK;
}

extern "C" void gbp_tri_plan_destroy(gbp_tri_plan p) { tri_free(p); }

extern "C" int gbp_tri_plan_set_team(gbp_tri_plan p, int founders, int most) {
    if (!p) {
        gbp_set_error("null triangle plan");
        return GBP_ERR_ARG;
    }
    return gbp_team_bounds(founders, most, p->team_limits);
}

extern "C" int gbp_tri_plan_team(gbp_tri_plan p, int* founders, int* members) {
    if (!p) {
        gbp_set_error("null triangle plan");
        return GBP_ERR_ARG;
    }
    return gbp_team_read(p->team, founders, members);
}

extern "C" int gbp_tri_backward_info(gbp_tri_plan p, int* levels, int* cyclic, int* sweeps) {
    if (!p) {
        gbp_set_error("null triangle plan");
        return GBP_ERR_ARG;
    }
    if (levels) *levels = p->last_levels;
    if (cyclic) *cyclic = p->last_cyclic;
    if (sweeps) *sweeps = p->last_sweeps;
    return GBP_OK;
}

extern "C" int gbp_tri_forward(gbp_tri_plan p, const float* D, const float* vscale,
                               const int32_t* root_node, const float* root_t, int n_roots,
                               float* T_out, gbp_stats* stats, void* stream) {
    int rc = tri_check(p, D, root_node, root_t, n_roots);
    if (rc) return rc;
    if (!T_out) {
        gbp_set_error("T_out is required");
        return GBP_ERR_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    const int n_v = p->n_v;
    if ((rc = tri_prepare(p, D, vscale, root_node, root_t, n_roots, true, s))) return rc;
    const TriRelax g{p->info, p->inc, p->nb, p->eps_rel};
    const int cap = p->max_rounds;
    if (n_v <= kTriBlockVerts) {
        k_tri_rounds_block<<<1, kTriThreads, tri_block_lds(n_v), s>>>(g, n_v, p->T, p->q0, p->ctl, cap);
    } else {
        const TriLists q{p->now[0], p->now[1], p->gain[0], p->gain[1], p->q[0], p->q[1], p->q0, p->mark};
        k_tri_rounds_team<<<p->team_blocks, kTriThreads, 0, s>>>(g, n_v, p->list_cap, q, p->stamp, p->team, p->ctl,
                                                                       cap, p->T, p->team_limits);
    }
    GBP_LAUNCH_CHECK();
    k_tri_count_inf<<<gbp_blocks(n_v, TPB), TPB, 0, s>>>(p->T, n_v, p->ctl);
    GBP_HIP(hipMemcpyAsync(T_out, p->T, (size_t)n_v * sizeof(float), hipMemcpyDeviceToDevice, s));
    if ((rc = tri_read(p, s))) return rc;
    const TriCtl& c = *p->ctl_host;
    p->stamp += c.rounds + 2;
    const bool converged = !c.err && c.left == 0;
    if (stats) {
        stats->rounds = c.rounds;
        stats->converged = converged ? 1 : 0;
        stats->face_solves = (int64_t)c.solves;
        stats->node_updates = (int64_t)c.updates;
        stats->unreached = c.unreached;
    }
    if (c.err) return gbp_err_from_bits(c.err);
    if (!converged) {
        gbp_set_error("triangle forward did not converge in %d rounds", cap);
        return GBP_ERR_NOT_CONVERGED;
    }
    return GBP_OK;
}

extern "C" int gbp_tri_backward(gbp_tri_plan p, const float* D, const float* vscale,
                                const int32_t* root_node, const float* root_t, int n_roots,
                                const float* T, const float* dL_dT, float* dL_dD,
                                float* dL_dvscale, float* dL_droot_t, void* stream) {
    int rc = tri_check(p, D, root_node, root_t, n_roots);
    if (rc) return rc;
    if (!T || !dL_dT) {
        gbp_set_error("T and dL_dT are required");
        return GBP_ERR_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    const int n_v = p->n_v, n_t = p->n_t;
    const int nb = gbp_blocks(n_v, TPB);
    GBP_HIP(hipMemcpyAsync(p->T, T, (size_t)n_v * sizeof(float), hipMemcpyDeviceToDevice, s));
    if ((rc = tri_prepare(p, D, vscale, root_node, root_t, n_roots, false, s))) return rc;
    k_tri_fill_i<<<nb, TPB, 0, s>>>(p->done, 0, n_v);
    k_tri_parent<<<nb, TPB, 0, s>>>(p->xy, p->tri, D, vscale, p->vptr, p->vent, p->T, p->troot, n_v,
                                    p->par, p->pnode, p->pa, p->done);
    GBP_LAUNCH_CHECK();
    AdjGraph a{};
    a.n_v = n_v;
    a.pnode = p->pnode;
    a.pa = p->pa;
    a.T = p->T;
    a.cnt = p->done;
    a.crange = p->crange;
    a.cfill = p->cfill;
    a.cchild = p->cchild;
    a.calpha = p->calpha;
    a.rec = p->rec;
    a.over = p->over;
    a.leaf = p->q0;
    a.ready[0] = p->ready[0];
    a.ready[1] = p->ready[1];
    a.team = p->team;
    a.limits = p->team_limits;
    a.done = p->done;
    a.g = p->g;
    a.lam = p->lam;
    a.ctl = reinterpret_cast<AdjCtl*>(reinterpret_cast<char*>(p->ctl) + offsetof(TriCtl, adj));
    if ((rc = gbp_adj_lists(a, dL_dT, nullptr, s))) return rc;
    if ((rc = gbp_adj_walk(a, INT_MAX, n_v <= kTriWalkBlockVerts, s))) return rc;
    // vertices on or above parent-graph cycles: Gauss-Seidel sweeps over just those
    // (their children outside the list are final)
    const int batch = gbp_adj_sweep_batch(a);
    if ((rc = gbp_adj_sweeps(a, p->cfill, true, 0, batch > 16 ? batch : 0, 1e-7f, false, s))) return rc;
    if ((rc = tri_read(p, s))) return rc;
    if (p->ctl_host->err) return gbp_err_from_bits(p->ctl_host->err);
    const AdjCtl& c = p->ctl_host->adj;
    const int cap = 8 * n_v + 64;
    while (c.remaining > 0 && !c.settled && c.sweeps < cap) {
        if ((rc = gbp_adj_sweeps(a, p->cfill, false, c.sweeps, batch, 1e-7f, false, s))) return rc;
        if ((rc = tri_read(p, s))) return rc;
    }
    p->last_levels = c.levels;
    p->last_cyclic = c.remaining;
    if (c.remaining > 0 && !c.settled) {
        gbp_set_error("triangle adjoint did not settle in %d sweeps", c.sweeps);
        return GBP_ERR_NOT_CONVERGED;
    }
    p->last_sweeps = c.sweeps;
    const float* lam = p->lam;
    k_tri_fill<<<gbp_blocks(n_t, TPB), TPB, 0, s>>>(p->dsbar, 0.f, n_t);
    if (dL_dD) k_tri_fill<<<gbp_blocks(3LL * n_t, TPB), TPB, 0, s>>>(dL_dD, 0.f, 3 * n_t);
    k_tri_grad_tri<<<nb, TPB, 0, s>>>(p->xy, p->tri, D, vscale, p->par, p->pnode, p->pa, lam, n_v,
                                      dL_dD, p->dsbar);
    if (dL_dvscale)
        k_tri_grad_node<<<nb, TPB, 0, s>>>(p->vptr, p->vent, p->dsbar, n_v, dL_dvscale);
    if (dL_droot_t && n_roots > 0)
        k_tri_grad_root<<<gbp_blocks(n_roots, TPB), TPB, 0, s>>>(root_node, root_t, n_roots, n_v,
                                                                 p->pa, p->troot, lam, dL_droot_t);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}
