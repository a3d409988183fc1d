// The adjoint's walk of the parent graph (Sec. 2.3 Eq. (dto_grad)), shared by
// tetrahedra and triangles: lambda = g + P^T lambda, leaves first.
#pragma once

#include "gbp_internal.h"

// One parent graph and its work arrays.  pnode names a vertex's weighted parents
// (-1: none), pa holds their weights in x, y, z (a triangle uses the first two).
struct AdjGraph {
    int n_v;
    const int4* pnode;     // [n_v]
    const float4* pa;      // [n_v]
    const float* T;        // [n_v] (+inf: unreached)
    const int* cnt;        // [n_v] children per vertex
    int2* crange;          // [n_v] child list [begin, end)
    int* cfill;            // [n_v] fill cursors
    int* cchild;           // [3 n_v] children, sorted within a list
    float* calpha;         // [3 n_v] their weights
    AdjRec* rec;           // [n_v]
    float* over;           // [3 n_v] entries past a record's, at their place in the child lists
    int* leaf;             // [n_v] the leaves
    int* ready[2];         // [walk_list_size(n_v)] the members' lists of a level
    int* done;             // [n_v] finished
    float *g, *lam;        // [n_v]
    AdjCtl* ctl;           // zeroed before gbp_adj_lists
    TeamCtl* team;         // zeroed before gbp_adj_lists
    TeamLimits limits;     // of its teams
};

// Child lists, two-cycle partners, right-hand side (node_user: internal -> caller
// vertex, or null) and leaves.  pnode, pa and cnt come from the parents' kernel.
int gbp_adj_lists(const AdjGraph& a, const float* dL_dT, const int* node_user, hipStream_t s);

// Finishes every vertex below level `levels` whose children are all finished
// (done, lam); ctl->levels receives the last level with work + 1.  Vertices on or
// above cycles longer than two stay unfinished.  narrow: levels of a few hundred
// vertices, for one block.
int gbp_adj_walk(const AdjGraph& a, int levels, bool narrow, hipStream_t s);

// Gauss-Seidel sweeps from, from + 1, ..., at most `count`, over the reached vertices
// that the walk left (ctl->remaining of them in list [n_v], listed if `build`), in place.
// ctl->sweeps: sweeps so far; ctl->settled: the last moved no lambda by more than tol
// times the largest.  exhaust: they go on to `count` unless nothing changes any more,
// else they may end once settled.
int gbp_adj_sweeps(const AdjGraph& a, int* list, bool build, int from, int count, float tol, bool exhaust,
                   hipStream_t s);
int gbp_adj_sweep_batch(const AdjGraph& a);   // sweeps worth enqueueing between the host's looks
