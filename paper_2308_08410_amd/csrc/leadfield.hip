// Lead weights on the device (Sec. 2.4): B = K Z with K the P1 stiffness of the
// plan's mesh (unit conductivity) and Z[n, l] = 1 / |x_n - e_l| the lead field of
// a point electrode, so that electrodes can move without a host assembly.
//
// Eight lanes assemble a vertex's row of K over the elements around it (the incidence
// lists of the plan), one value per neighbour, and then sum K_im Z_l(x_m) over those
// neighbours, eight leads at a time.  FP64 throughout: B is a sum of terms of both
// signs that nearly cancel away from the boundary.  Deterministic (fixed order).
#include "gbp_internal.h"
#include "local_solve.h"

namespace {

constexpr int TPB = 256;
constexpr int kLanes = 8;          // per vertex: three passes over a 24-element patch
constexpr int kVerts = TPB / kLanes;
constexpr int kSlots = 32;         // neighbours (and the vertex itself) assembled at a time
constexpr int kMaxLeads = 256;

// One vertex's row of K for the neighbours from w0 on: row[s] for neighbour w0 + s of its
// list nb (the vertex itself comes after its last neighbour).
//
// Bound by FP64 arithmetic, so it is done once per (vertex, element) and once per
// (vertex, neighbour, lead): a 24-element patch has 72 (element, other vertex) pairs
// but 14 neighbours, and the distance's reciprocal square root is the costly part.
// 500k vertices, 12 leads: 272 us; 854 us with one thread per vertex that took a square
// root and a division per (element, vertex, lead) and the geometry anew every 8 leads.
// (16 lanes per vertex: 595 us; more waves by fewer registers: 286 us and up.)
__device__ __forceinline__ void assemble_row(const int2 p, const int* __restrict__ nent,
                                             const int4* __restrict__ tetv, const float4* __restrict__ xyz,
                                             int self, const int* __restrict__ nbs, int n_nb, int w0, int lane,
                                             int* nb, double* row) {
    const int m = min(kSlots, n_nb - w0);   // neighbours in this window
    for (int s = lane; s < kSlots; s += kLanes) {
        row[s] = 0.0;
        nb[s] = s < m ? nbs[w0 + s] : self;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const float4 xi = xyz[self];
    const int c0 = p.y & 255, c1 = (p.y >> 8) & 255, c2 = (p.y >> 16) & 255, c3 = (p.y >> 24) & 255;
    const int tot = c0 + c1 + c2 + c3;
    double diag = 0.0;
    for (int b = 0; b < tot; b += kLanes) {
        const int c = b + lane;
        double k[3] = {0.0, 0.0, 0.0};
        int slot[3] = {-1, -1, -1};
        if (c < tot) {
            const int K = (c < c0) ? 0 : (c < c0 + c1) ? 1 : (c < c0 + c1 + c2) ? 2 : 3;
            int o[3];
            face_nodes_sel(tetv[nent[p.x + c]], K, o[0], o[1], o[2]);
            double e[3][3];   // edges from the vertex
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const float4 x = xyz[o[q]];
                e[q][0] = (double)x.x - xi.x;
                e[q][1] = (double)x.y - xi.y;
                e[q][2] = (double)x.z - xi.z;
            }
            // det * gradient of the other vertices' barycentric coordinates; the
            // vertex's own is minus their sum
            double n[3][3], s[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double* u = e[(q + 1) % 3];
                const double* v = e[(q + 2) % 3];
                n[q][0] = u[1] * v[2] - u[2] * v[1];
                n[q][1] = u[2] * v[0] - u[0] * v[2];
                n[q][2] = u[0] * v[1] - u[1] * v[0];
            }
#pragma unroll
            for (int z = 0; z < 3; ++z) s[z] = n[0][z] + n[1][z] + n[2][z];
            const double det = e[0][0] * n[0][0] + e[0][1] * n[0][1] + e[0][2] * n[0][2];
            const double f = -1.0 / (6.0 * fabs(det));   // volume / det^2
            diag -= f * (s[0] * s[0] + s[1] * s[1] + s[2] * s[2]);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                k[q] = f * (s[0] * n[q][0] + s[1] * n[q][1] + s[2] * n[q][2]);
                int at = 0;   // the last neighbour of the window not above o[q]
#pragma unroll
                for (int h = kSlots / 2; h > 0; h >>= 1)
                    if (at + h < m && nb[at + h] <= o[q]) at += h;
                slot[q] = m > 0 && nb[at] == o[q] ? at : -1;
            }
        }
        // the lanes in turn: elements share neighbours, and the order stays fixed
#pragma unroll
        for (int t = 0; t < kLanes; ++t)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (lane == t && slot[q] >= 0)
                    (void)__hip_atomic_fetch_add(&row[slot[q]], k[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
#pragma unroll
    for (int o = 1; o < kLanes; o <<= 1) diag += __shfl_xor(diag, o);
    if (lane == 0 && m < kSlots && n_nb - w0 >= 0) row[m] = diag;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__global__ void __launch_bounds__(TPB)
    k_lead_field(const int2* __restrict__ nptr, const int* __restrict__ nent,
                 const int4* __restrict__ tetv, const float4* __restrict__ xyz,
                 const int* __restrict__ node_user, const int* __restrict__ adj_ptr,
                 const int* __restrict__ adj, int n_v, const float* __restrict__ elec, int L,
                 float* __restrict__ W) {
    __shared__ double se[3 * kMaxLeads], row_sh[kVerts][kSlots + 1];
    __shared__ int nb_sh[kVerts][kSlots + 1];
    for (int q = threadIdx.x; q < 3 * L; q += blockDim.x) se[q] = elec[q];
    __syncthreads();
    const int lane = threadIdx.x & (kLanes - 1), v = threadIdx.x / kLanes;
    const int i = blockIdx.x * kVerts + v;
    if (i >= n_v) return;                         // uniform over the 8 lanes
    const int2 p = nptr[i];
    const int a0 = adj_ptr[i], n_nb = adj_ptr[i + 1] - a0;
    const int u = node_user[i];
    double* row = row_sh[v];
    int* nb = nb_sh[v];
    const bool one = n_nb < kSlots;               // the whole row at once
    for (int l0 = 0; l0 < L; l0 += kLanes) {
        double sum[kLanes];
#pragma unroll
        for (int q = 0; q < kLanes; ++q) sum[q] = 0.0;
        for (int w0 = 0; w0 <= n_nb; w0 += kSlots) {
            if (!one || l0 == 0) assemble_row(p, nent, tetv, xyz, i, adj + a0, n_nb, w0, lane, nb, row);
            const int m = min(kSlots, n_nb + 1 - w0);
            for (int s = lane; s < m; s += kLanes) {
                const double k = row[s];
                const float4 x = xyz[nb[s]];
#pragma unroll
                for (int q = 0; q < kLanes; ++q) {
                    const int l = l0 + q;
                    if (l >= L) break;
                    const double dx = x.x - se[3 * l], dy = x.y - se[3 * l + 1], dz = x.z - se[3 * l + 2];
                    sum[q] += k * rsqrt(dx * dx + dy * dy + dz * dz);
                }
            }
        }
        // sums over the lanes, lane j keeping lead l0 + j
#pragma unroll
        for (int o = kLanes / 2; o > 0; o >>= 1)
#pragma unroll
            for (int q = 0; q < o; ++q) {
                const bool hi = lane & o;
                const double mine = hi ? sum[q + o] : sum[q], other = hi ? sum[q] : sum[q + o];
                sum[q] = mine + __shfl_xor(other, o);
            }
        if (l0 + lane < L) W[(size_t)u * L + l0 + lane] = (float)sum[0];
    }
}

}  // namespace

extern "C" int gbp_lead_field(gbp_plan p, const float* electrodes, int n_leads, float* W,
                              void* stream) {
    int rc = gbp_plan_check(p);
    if (rc) return rc;
    if (n_leads < 1 || n_leads > kMaxLeads || !electrodes || !W) {
        gbp_set_error("lead_field: 1 <= n_leads <= %d, electrodes and W required", kMaxLeads);
        return GBP_ERR_ARG;
    }
    k_lead_field<<<gbp_blocks(p->n_v, kVerts), TPB, 0, (hipStream_t)stream>>>(
        p->nptr, p->nent, p->tetv, p->xyz, p->node_user, p->adj_ptr, p->adj, p->n_v, electrodes, n_leads, W);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}
