// Lead-field ECG (Sec. 2.4) and its backward pass on gfx950 matrix cores.
//
//   ecg[s,l] = sum_n W[n,l] U(t_s - T_n),   U(xi) = K0 + (K1-K0) sigma(4 xi / tau)
//
// The template saturates: for |4 xi / tau| >= 24, sigma equals 1 to FP32
// precision on the upper side (1 - sigma < 4e-11) and is below 4e-11 on the lower
// side.  The time axis is cut into tiles of 16 steps and the vertices into steps of 16:
// a vertex step's finite activation times span [Tmin, Tmax], so only the time tiles
// that touch [Tmin - 6 tau, Tmax + 6 tau] need the template; before them every term is
// at rest, after them at K1.  There the contraction (time x vertices) . (vertices x
// leads) runs on v_mfma_f32_16x16x16_bf16 tiles whose A operand is generated in
// registers from T.  (The K = 32 shape of gfx950 halves the matrix instructions, but 32
// vertices share a longer window, and the template's vector-ALU work is the bound.)
// Both operands are split into bf16 hi + lo parts (three products, FP32
// accumulation), since the lead weights sum to ~0 and the ECG is a cancellation.
//
// Backward:  dT_n = -sum_s U'(t_s - T_n) sum_l G[s,l] W[n,l], with U' zero outside
// the same window; R = U' G runs on MFMA (vertices x time) . (time x leads) and the
// row-wise dot with W finishes in registers.  No atomics: deterministic.
//
// A launch covers up to 32 leads (two MFMA column tiles share the template) and all
// time steps, as long as the scratch holds a row per time tile.
//
// MFMA 16x16x16 lane layout: lane l holds A[l % 16][4 (l / 16) + q] and
// B[4 (l / 16) + q][l % 16], q = 0..3, and returns D[4 (l / 16) + r][l % 16], r = 0..3.
#include <math.h>

#include <algorithm>
#include <climits>
#include <mutex>

#include "gbp_internal.h"
#include "profile.h"

namespace {

typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr float kSat = 24.f;          // |4 xi / tau| beyond which sigma is saturated
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kMaxSteps = 1 << 20;    // time steps per call
constexpr int kMaxLeads = 256;

// x = hi + lo in bf16, both rounded to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ void split_bf16(float x, float y, unsigned& hi, unsigned& lo) {
    hi = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{x, y}, bf16x2_t));
    const floatx2 rest{x - __uint_as_float(hi << 16), y - __uint_as_float(hi & 0xffff0000u)};
    lo = __builtin_bit_cast(unsigned, __builtin_convertvector(rest, bf16x2_t));
}

__device__ __forceinline__ void split4(const float (&a)[4], bf16x4_t& hi, bf16x4_t& lo) {
    uint2 h, l;
    split_bf16(a[0], a[1], h.x, l.x);
    split_bf16(a[2], a[3], h.y, l.y);
    hi = __builtin_bit_cast(bf16x4_t, h);
    lo = __builtin_bit_cast(bf16x4_t, l);
}

__device__ __forceinline__ floatx4 mfma3(bf16x4_t ah, bf16x4_t al, bf16x4_t bh, bf16x4_t bl,
                                         floatx4 acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al, bh, acc, 0, 0, 0);
    return acc;
}

struct ApDev {
    float K0, amp, c4, dudx, t0, dt, halfw;  // c4 = 4 log2(e)/tau, dudx = amp*4/tau, halfw = 6 tau
    int S;                                    // time steps of this launch
};

// Lead columns [0, Lt) of arrays whose rows are Ls floats long (W, and ecg / G per time
// step), the latter `istride` floats apart from one instance to the next.
struct LeadTile {
    int Ls, Lt;
    long long istride;
};

// Window of 16 vertices, one per lane of a group of 16, in time tiles: [lo, hi), empty
// and past the end if none is finite.  From hi on they are saturated.
__device__ __forceinline__ void step_window(float Tv, const ApDev& ap, int& lo, int& hi) {
    const bool fin = Tv < __builtin_huge_valf();
    float tmin = fin ? Tv : __builtin_huge_valf(), tmax = fin ? Tv : -__builtin_huge_valf();
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        tmin = fminf(tmin, __shfl_xor(tmin, o));
        tmax = fmaxf(tmax, __shfl_xor(tmax, o));
    }
    const int nt = (ap.S + 15) / 16;
    lo = hi = nt;
    if (!(tmin < __builtin_huge_valf())) return;
    const float S = (float)ap.S;
    const int s_lo = (int)fminf(fmaxf(ceilf((tmin - ap.halfw - ap.t0) / ap.dt), 0.f), S);
    const int s_hi = (int)fminf(fmaxf(floorf((tmax + ap.halfw - ap.t0) / ap.dt) + 1.f, 0.f), S);
    hi = (max(s_hi, s_lo) + 15) / 16;
    lo = min(s_lo / 16, hi);
}

// ------------------------------------------------------------------ forward
// A block of 16 waves takes `vb` vertices (vb / 16 steps, at most 32): their weights go to
// LDS once, split, as B operands.  The waves share out the time tiles of the block's
// window (and, where there are fewer than 16, the vertex steps of a tile); a tile is
// contracted over the steps whose window it touches and added to the ECG once.
// A step's weights' sums go to the row of g_hist of the tile from which it is saturated;
// the rows are summed over time at the end.
//
// Bound by the template (exp2, rcp and the splits, ~13 vector-ALU operations a term) and, in
// a fifth of the time, by the atomic adds.  143,564 vertices, 31 leads, 2000 steps of
// 0.1 tau: 55 us; 500,103 vertices, 12 leads, 500 steps of tau: 40 us.  With launches of 16
// leads and 992 steps, groups of 64 vertices and the window in LDS, where each group's
// tiles were added with LDS atomics: 408 us (6 launches) and 49 us.
constexpr int kFwdThreads = 1024;
constexpr int kFwdSteps = 32;         // most vertex steps of a block
constexpr int kFwdTiles = kFwdThreads / 64;         // time tiles at a time: one per wave
constexpr int kBufRow = 20;           // floats per lead of a wave's tile sums: 16 steps, padded over the banks

// Dynamic LDS: B operands, tile sums, saturated sums, times.
__host__ __device__ constexpr size_t fwd_lds(int nt, int vb) {
    return (size_t)vb * nt * 64 + (size_t)kFwdTiles * 16 * nt * kBufRow * 4 + (size_t)vb * nt * 4 + (size_t)vb * 4;
}

// Grid (blocks per instance, instances); instance i owns vertices
// [off[i], off[i+1]) (off == nullptr: one instance of n_v vertices).
template <int NT>
__global__ void __launch_bounds__(kFwdThreads)
    k_ecg_fwd(const float* __restrict__ T, const float* __restrict__ W, int n_v, LeadTile lt,
              ApDev ap, int vb, const int* __restrict__ off, double* __restrict__ g_hist_all,
              double* __restrict__ g_wsum_all, float* __restrict__ ecg_all) {
    constexpr int NL = 16 * NT;
    extern __shared__ char lds[];
    short* wf = reinterpret_cast<short*>(lds);                                  // [vb/16][NT][2][16 leads][16]
    float* buf = reinterpret_cast<float*>(lds + (size_t)vb * NT * 64);          // [waves][NL][kBufRow]
    float* ws = buf + kFwdTiles * NL * kBufRow;                                      // [vb/16][NL]
    float* Tsh = ws + (size_t)vb * NT;                                          // [vb]
    __shared__ int lo_sh[kFwdSteps], hi_sh[kFwdSteps];
    __shared__ float wtot[NL];
    const int inst = blockIdx.y;
    const int vbeg = off ? off[inst] : 0, vend = off ? off[inst + 1] : n_v;
    const int g0 = vbeg + blockIdx.x * vb;
    if (g0 >= vend) return;
    const int Ls = lt.Ls, Lt = lt.Lt, nt_all = (ap.S + 15) / 16, nk = vb / 16;
    double* g_hist = g_hist_all + (size_t)inst * (nt_all + 1) * NL;
    float* ecg = ecg_all + (size_t)inst * lt.istride;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (tid < NL) wtot[tid] = 0.f;
    if (tid < vb) {
        const float t = g0 + tid < vend ? T[g0 + tid] : __builtin_huge_valf();
        Tsh[tid] = t;
        int lo, hi;
        step_window(t, ap, lo, hi);
        if ((tid & 15) == 0) {
            lo_sh[tid >> 4] = lo;
            hi_sh[tid >> 4] = hi;
        }
    }
    for (int e = tid; e < nk * NL; e += kFwdThreads) ws[e] = 0.f;
    __syncthreads();
    // weights: two vertices a thread, split and stored as the B operand reads them, and
    // summed: over a step's finite times (saturation), over all of them (rest)
    float all = 0.f;
    for (int e = tid; e < vb / 2 * NL; e += kFwdThreads) {   // whole waves
        const int l = e % NL, n = 2 * (e / NL);
        const float* w = W + min(l, Lt - 1);
        float a = w[(size_t)min(g0 + n, vend - 1) * Ls], b = w[(size_t)min(g0 + n + 1, vend - 1) * Ls];
        a = l < Lt && g0 + n < vend ? a : 0.f;
        b = l < Lt && g0 + n + 1 < vend ? b : 0.f;
        unsigned h, r;
        split_bf16(ap.amp * a, ap.amp * b, h, r);
        short* q = wf + ((size_t)((n >> 4) * NT + (l >> 4)) * 2 * 16 + (l & 15)) * 16 + (n & 15);
        *reinterpret_cast<unsigned*>(q) = h;
        *reinterpret_cast<unsigned*>(q + 256) = r;
        const float2 t = *reinterpret_cast<const float2*>(Tsh + n);
        float fin = (t.x < __builtin_huge_valf() ? a : 0.f) + (t.y < __builtin_huge_valf() ? b : 0.f);
        all += a + b;
#pragma unroll
        for (int o = NL; o < 64; o <<= 1) fin += __shfl_xor(fin, o);   // a wave's vertices are of one step
        if (lane < NL) atomicAdd(&ws[(n >> 4) * NL + l], ap.amp * fin);
    }
#pragma unroll
    for (int o = NL; o < 64; o <<= 1) all += __shfl_xor(all, o);
    if (lane < NL) atomicAdd(&wtot[lane], all);
    __syncthreads();
    if (tid < Lt) atomicAdd(&g_wsum_all[(size_t)inst * NL + tid], (double)wtot[tid]);
    // the block's window
    const int klo = lane < nk ? lo_sh[lane] : nt_all, khi = lane < nk ? hi_sh[lane] : 0;
    int blo = klo, bhi = lane < nk && klo < nt_all ? khi : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        blo = min(blo, __shfl_xor(blo, o));
        bhi = max(bhi, __shfl_xor(bhi, o));
    }
    const int col = lane & 15, kq = lane >> 4;
    // what saturates at tile t goes to its row (one wave)
    auto saturate = [&](int t) {
        unsigned long long m = __ballot(klo < nt_all && khi == t);
        if (!m || lane >= Lt) return;
        float s = 0.f;
        for (; m; m &= m - 1) s += ws[(__ffsll(m) - 1) * NL + lane];
        atomicAdd(&g_hist[(size_t)t * NL + lane], (double)s);
    };
    for (int b0 = blo; b0 < bhi; b0 += kFwdTiles) {
        const int ntb = min(kFwdTiles, bhi - b0);
        const int parts = kFwdThreads / 64 / ntb, kpp = (nk + parts - 1) / parts;
        if (wave < ntb) saturate(b0 + wave);
        if (wave < ntb * parts) {
            const int tile = b0 + wave % ntb, part = wave / ntb;
            const float t = ap.t0 + (float)(tile * 16 + col) * ap.dt;
            floatx4 acc[NT];
#pragma unroll
            for (int z = 0; z < NT; ++z) acc[z] = floatx4{0.f, 0.f, 0.f, 0.f};
            unsigned long long m = __ballot(klo <= tile && tile < khi && lane / kpp == part);
            while (m) {
                const int k = __ffsll(m) - 1;
                m &= m - 1;
                const float4 tv = *reinterpret_cast<const float4*>(Tsh + 16 * k + 4 * kq);
                const float tr[4] = {tv.x, tv.y, tv.z, tv.w};
                float a[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    a[r] = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f((tr[r] - t) * ap.c4));
                bf16x4_t ah, al;
                split4(a, ah, al);
#pragma unroll
                for (int z = 0; z < NT; ++z) {
                    const short* q = wf + ((size_t)(k * NT + z) * 2 * 16 + col) * 16 + 4 * kq;
                    acc[z] = mfma3(ah, al, *reinterpret_cast<const bf16x4_t*>(q),
                                   *reinterpret_cast<const bf16x4_t*>(q + 256), acc[z]);
                }
            }
#pragma unroll
            for (int z = 0; z < NT; ++z)
                *reinterpret_cast<floatx4*>(buf + (wave * NL + z * 16 + col) * kBufRow + 4 * kq) = acc[z];
        }
        __syncthreads();
        for (int e = tid; e < ntb * 16 * NL; e += kFwdThreads) {
            const int l = e % NL, s = e / NL;
            const float* b = buf + ((s >> 4) * NL + l) * kBufRow + (s & 15);
            float v = 0.f;
            for (int p = 0; p < parts; ++p) v += b[p * ntb * NL * kBufRow];
            if (l < Lt && b0 * 16 + s < ap.S && v != 0.f) atomicAdd(&ecg[(size_t)(b0 * 16 + s) * Ls + l], v);
        }
        __syncthreads();
    }
    // and behind the last tile (nothing past the end)
    if (bhi < nt_all && wave == 0) saturate(bhi);
}

// ecg (columns [0, Lt)), the rows of g_hist and g_wsum cleared
__global__ void k_ecg_zero(float* __restrict__ work, int n_work, float* __restrict__ ecg_all, LeadTile lt, int S) {
    const int step = gridDim.x * blockDim.x, at = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.y == 0)
        for (int i = at; i < n_work; i += step) work[i] = 0.f;
    float* ecg = ecg_all + (size_t)blockIdx.y * lt.istride;
    const int n = S * lt.Lt;   // at most 8032 * 32 = 16096 * 16
    for (int i = at; i < n; i += step) ecg[(size_t)(i / lt.Lt) * lt.Ls + i % lt.Lt] = 0.f;
}

// ecg[s,l] += K0 * sum W + the rows of hist up to the step's tile.  Grid (blocks of
// `tpb` tiles, instances); thread (c, l) sums every (1024 / NL)-th row before the
// block's first.
template <int NL>
__global__ void __launch_bounds__(1024)
    k_ecg_finish(const double* __restrict__ g_hist_all, const double* __restrict__ g_wsum_all, int S, LeadTile lt,
                 float K0, int tpb, float* __restrict__ ecg_all) {
    constexpr int NC = 1024 / NL;
    __shared__ double part[NC][NL + 1];
    const int inst = blockIdx.y, nt = (S + 15) / 16;
    const double* g_hist = g_hist_all + (size_t)inst * (nt + 1) * NL;
    float* ecg = ecg_all + (size_t)inst * lt.istride;
    const int l = threadIdx.x % NL, c = threadIdx.x / NL;
    const int t0 = blockIdx.x * tpb, t1 = min(nt, t0 + tpb);
    double run = 0.;
    for (int t = c; t <= t0; t += NC) run += g_hist[(size_t)t * NL + l];
    part[c][l] = run;
    __syncthreads();
    if (c == 0) {
        double s = K0 * g_wsum_all[(size_t)inst * NL + l];
        for (int k = 0; k < NC; ++k) s += part[k][l];
        part[0][l] = s;
    }
    __syncthreads();
    if (l >= lt.Lt) return;
    double r = part[0][l];
    for (int t = t0; t < t1; ++t) {
        if (t > t0) r += g_hist[(size_t)t * NL + l];
        for (int s = 16 * t + c; s < min(16 * t + 16, S); s += NC) ecg[(size_t)s * lt.Ls + l] += (float)r;
    }
}

// ------------------------------------------------------------------ backward
// A block of 8 waves takes 8 steps of 16 vertices; the time tiles of the block's window
// pass through LDS as B operands, kBwdTiles at a time, and each wave contracts those of
// its own step's window.
// Bound by the template's derivative (~19 vector-ALU operations a term).  143,564 vertices,
// 31 leads, 2000 steps of 0.1 tau: 40 us (two steps a wave: 49 us); 500,103 vertices, 12
// leads, 500 steps of tau: 27 us.  With all of G in every block's LDS as rows of leads,
// windows of 64 vertices and launches of 16 leads and 992 steps: 312 us (6 launches) and 47 us.
// accumulate: add this launch's contribution to dT instead of writing it.
constexpr int kBwdThreads = 512;
constexpr int kBwdVerts = kBwdThreads / 4;
constexpr int kBwdTiles = 16;

template <int NT>
__global__ void __launch_bounds__(kBwdThreads)
    k_ecg_bwd(const float* __restrict__ T, const float* __restrict__ W,
              const float* __restrict__ G_all, int n_v, LeadTile lt, ApDev ap,
              const int* __restrict__ off, int accumulate, float* __restrict__ dT) {
    constexpr int NL = 16 * NT;
    __shared__ __align__(16) short gf[kBwdTiles][NT][2][16][16];   // tile, lead tile, hi / lo, lead, step
    __shared__ int blo_sh, bhi_sh;
    const int inst = blockIdx.y;
    const int vbeg = off ? off[inst] : 0, vend = off ? off[inst + 1] : n_v;
    const int g0 = vbeg + blockIdx.x * kBwdVerts;
    if (g0 >= vend) return;
    const int Ls = lt.Ls, Lt = lt.Lt;
    const float* G = G_all + (size_t)inst * lt.istride;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, kq = lane >> 4;
    if (tid == 0) {
        blo_sh = INT_MAX;
        bhi_sh = 0;
    }
    __syncthreads();
    const int n0 = g0 + wave * 16;
    const float tn = n0 + col < vend ? T[n0 + col] : __builtin_huge_valf();   // A row: vertex
    int lo, hi;
    step_window(tn, ap, lo, hi);
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    if (lane == 0 && lo < hi) {
        atomicMin(&blo_sh, lo);
        atomicMax(&bhi_sh, hi);
    }
    floatx4 acc[NT];
#pragma unroll
    for (int z = 0; z < NT; ++z) acc[z] = floatx4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    const int blo = blo_sh, bhi = bhi_sh;
    for (int b0 = blo; b0 < bhi; b0 += kBwdTiles) {
        const int ntb = min(kBwdTiles, bhi - b0);
        for (int e = tid; e < ntb * 8 * NL; e += kBwdThreads) {
            const int l = e % NL, s2 = 2 * (e / NL), s = b0 * 16 + s2;
            const float* g = G + (size_t)s * Ls + l;
            const float a = l < Lt && s < ap.S ? g[0] : 0.f;
            const float b = l < Lt && s + 1 < ap.S ? g[Ls] : 0.f;
            unsigned h, r;
            split_bf16(a, b, h, r);
            *reinterpret_cast<unsigned*>(&gf[s2 >> 4][l >> 4][0][l & 15][s2 & 15]) = h;
            *reinterpret_cast<unsigned*>(&gf[s2 >> 4][l >> 4][1][l & 15][s2 & 15]) = r;
        }
        __syncthreads();
        for (int t = max(lo, b0); t < min(hi, b0 + ntb); ++t) {
            float a[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float ts = ap.t0 + (float)(t * 16 + kq * 4 + r) * ap.dt;
                const float e = __builtin_amdgcn_exp2f((tn - ts) * ap.c4);
                const float q = __builtin_amdgcn_rcpf(1.f + e);
                a[r] = q * (e < 1.f ? e * q : 1.f - q);
            }
            bf16x4_t ah, al;
            split4(a, ah, al);
#pragma unroll
            for (int z = 0; z < NT; ++z)
                acc[z] = mfma3(ah, al, *reinterpret_cast<const bf16x4_t*>(&gf[t - b0][z][0][col][4 * kq]),
                               *reinterpret_cast<const bf16x4_t*>(&gf[t - b0][z][1][col][4 * kq]), acc[z]);
        }
        __syncthreads();
    }
    // acc[z][r]: R[vertex 4 kq + r of the step][lead 16 z + col]
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int n = n0 + kq * 4 + r;
        float s = 0.f;
#pragma unroll
        for (int z = 0; z < NT; ++z)
            if (n < vend && z * 16 + col < Lt) s += acc[z][r] * W[(size_t)n * Ls + z * 16 + col];
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 4);
        s += __shfl_xor(s, 8);
        if (col == 0 && n < vend) dT[n] = (accumulate ? dT[n] : 0.f) - ap.dudx * s;
    }
}

// ------------------------------------------------------------------ workspace
// Scratch of gbp_ecg_forward_noalloc: the rows per time tile and the weight sums of one
// launch for one instance (every launch of a call reuses it in stream order),
// file-scope device memory that each GPU holds until the process ends.
constexpr int kNoAllocFloats = 2 * 1008 * 16 + 16;
__device__ __align__(256) float scratch[kNoAllocFloats];

// The array's device address on the current device, looked up once per device
// (in host code the symbol's name is a host-side stand-in, not this address).
int noalloc_scratch(float** out) {
    static std::mutex mu;
    static float* addr[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        gbp_set_error("no HIP device");
        return GBP_ERR_HIP;
    }
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            gbp_set_error("hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            return GBP_ERR_HIP;
        }
        addr[dev] = (float*)p;
    }
    *out = addr[dev];
    return GBP_OK;
}

struct EcgWork {
    float* buf = nullptr;
    size_t cap = 0;
};
std::mutex g_mu;
EcgWork g_work[64];

int ecg_workspace(size_t nfloat, float** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        gbp_set_error("no HIP device");
        return GBP_ERR_HIP;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    EcgWork& w = g_work[dev];
    if (w.cap < nfloat) {
        if (w.buf) (void)hipFree(w.buf);
        w.buf = nullptr;
        w.cap = 0;
        if (hipMalloc((void**)&w.buf, nfloat * sizeof(float)) != hipSuccess) {
            gbp_set_error("ECG workspace allocation failed");
            return GBP_ERR_NOMEM;
        }
        w.cap = nfloat;
    }
    *out = w.buf;
    return GBP_OK;
}

int check_ap(const float* T, int n_v, const float* W, int L, const gbp_ap* ap) {
    if (!T || !W || !ap || n_v <= 0 || L < 1 || L > kMaxLeads) {
        gbp_set_error("ECG: need T, W, ap, n_v > 0 and 1 <= L <= %d (L=%d)", kMaxLeads, L);
        return GBP_ERR_ARG;
    }
    if (ap->n_steps < 1 || ap->n_steps > kMaxSteps || !(ap->dt > 0.f) || !(ap->tau > 0.f) ||
        !std::isfinite(ap->K0) || !std::isfinite(ap->K1) || !std::isfinite(ap->t0)) {
        gbp_set_error("ECG: bad template/time grid (n_steps in [1,%d], dt > 0, tau > 0)", kMaxSteps);
        return GBP_ERR_ARG;
    }
    return GBP_OK;
}

// the template constants for the `len` steps starting at step s0
ApDev make_ap(const gbp_ap* a, int s0, int len) {
    ApDev d;
    d.K0 = a->K0;
    d.amp = a->K1 - a->K0;
    d.c4 = 4.f * kLog2e / a->tau;
    d.dudx = (a->K1 - a->K0) * 4.f / a->tau;
    d.t0 = a->t0 + (float)s0 * a->dt;
    d.dt = a->dt;
    d.halfw = kSat * a->tau / 4.f;
    d.S = len;
    return d;
}

// Leads of a launch: the two column tiles that share the template, or one.
int lead_tiles(int left) { return left > 16 ? 2 : 1; }

// Floats of forward scratch per instance.  A launch of `len` steps takes
// (tiles + 1) * NL doubles for the rows per time tile and NL for the weight sums; what
// does not fit goes in several launches.
constexpr size_t kWorkFloats = 2 * 1008 * 16 + 16;
size_t ecg_work_floats(int n_steps) {
    return std::min<size_t>(kWorkFloats, ((size_t)(n_steps + 15) / 16 + 2) * 64);
}
int max_len(size_t work_floats, int nl) { return ((int)(work_floats / 2 / nl) - 2) * 16; }

struct EcgLaunch {
    const int* off;       // device offsets or nullptr
    int n_inst;
    int max_verts;        // largest instance
    float* work;          // n_inst * work_floats floats
    size_t work_floats;   // per instance
};

// Vertices per block of the forward: two blocks to each of the 256 CUs at a time, as the
// LDS allows, and one such round where 512 vertices a block suffice (143,564 vertices:
// 320 a block 55 us, 256 63 us, 576 66 us; 500,103: 512 a block 40 us, 256 63 us).
int fwd_verts(long long verts) {
    return (int)std::min<long long>((verts + 512 * 64 - 1) / (512 * 64) * 64, 16 * kFwdSteps);
}

template <int NT>
int ecg_forward_part(const EcgLaunch& el, const float* T, int n_v, const float* W, const LeadTile& lt, const ApDev& d,
                     float* ecg, hipStream_t s) {
    constexpr int NL = 16 * NT;
    const int tiles = (d.S + 15) / 16;
    double* g_hist = reinterpret_cast<double*>(el.work);
    double* g_wsum = g_hist + (size_t)el.n_inst * (tiles + 1) * NL;
    const int n_work = el.n_inst * (tiles + 2) * NL * 2;
    const int zb = std::min((std::max(n_work, d.S * lt.Lt) + 1023) / 1024, 512);
    k_ecg_zero<<<dim3(zb, el.n_inst), 256, 0, s>>>(el.work, n_work, ecg, lt, d.S);
    const int vb = fwd_verts((long long)el.max_verts * el.n_inst);
    {
        ProfScope ps(GBP_PROF_ECG_FWD, s);
        k_ecg_fwd<NT><<<dim3((el.max_verts + vb - 1) / vb, el.n_inst), kFwdThreads, fwd_lds(NT, vb), s>>>(
            T, W, n_v, lt, d, vb, el.off, g_hist, g_wsum, ecg);
    }
    const int tpb = std::max(8, (tiles + 63) / 64);
    k_ecg_finish<NL><<<dim3((tiles + tpb - 1) / tpb, el.n_inst), 1024, 0, s>>>(g_hist, g_wsum, d.S, lt, d.K0, tpb, ecg);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

// More LDS than the default limit of 64 KB, once per device.
int fwd_lds_limit() {
    static std::mutex mu;
    static bool set[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        gbp_set_error("no HIP device");
        return GBP_ERR_HIP;
    }
    std::lock_guard<std::mutex> lk(mu);
    if (set[dev]) return GBP_OK;
    const int most = (int)fwd_lds(2, 16 * kFwdSteps);
    GBP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ecg_fwd<1>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, most));
    GBP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ecg_fwd<2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, most));
    set[dev] = true;
    return GBP_OK;
}

// Every (leads, steps) part of the call: a part is an ECG on its own time grid (the
// instance's rows of ecg are n_steps * L floats apart).
int ecg_forward_launch(const EcgLaunch& el, const float* T, int n_v, const float* W, int L,
                       const gbp_ap* ap, float* ecg, hipStream_t s) {
    const int S = ap->n_steps;
    int rc = fwd_lds_limit();
    if (rc) return rc;
    for (int c0 = 0; c0 < L;) {
        const int nt = lead_tiles(L - c0), most = max_len(el.work_floats, 16 * nt);
        const LeadTile lt{L, std::min(16 * nt, L - c0), (long long)S * L};
        for (int s0 = 0; s0 < S; s0 += most) {
            const ApDev d = make_ap(ap, s0, std::min(most, S - s0));
            float* out = ecg + (size_t)s0 * L + c0;
            rc = nt == 2 ? ecg_forward_part<2>(el, T, n_v, W + c0, lt, d, out, s)
                         : ecg_forward_part<1>(el, T, n_v, W + c0, lt, d, out, s);
            if (rc) return rc;
        }
        c0 += 16 * nt;
    }
    return GBP_OK;
}

int ecg_backward_launch(const EcgLaunch& el, const float* T, int n_v, const float* W, int L,
                        const gbp_ap* ap, const float* G, float* dT, hipStream_t s) {
    const int S = ap->n_steps;
    const ApDev d = make_ap(ap, 0, S);
    for (int c0 = 0; c0 < L;) {
        const int nt = lead_tiles(L - c0);
        const LeadTile lt{L, std::min(16 * nt, L - c0), (long long)S * L};
        const dim3 grid((el.max_verts + kBwdVerts - 1) / kBwdVerts, el.n_inst);
        ProfScope ps(GBP_PROF_ECG_BWD, s);
        (nt == 2 ? k_ecg_bwd<2> : k_ecg_bwd<1>)<<<grid, kBwdThreads, 0, s>>>(T, W + c0, G + c0, n_v, lt, d, el.off,
                                                                            c0 > 0, dT);
        GBP_LAUNCH_CHECK();
        c0 += 16 * nt;
    }
    return GBP_OK;
}

}  // namespace

struct gbp_batch_s {
    int device = 0;
    int n_inst = 0, max_verts = 0, total = 0, max_steps = 0;
    int* off = nullptr;
    float* work = nullptr;
};

extern "C" int gbp_batch_create(const int32_t* offsets, int n_inst, int max_steps, gbp_batch* out) {
    if (!out || !offsets || n_inst < 1 || max_steps < 1 || max_steps > kMaxSteps) {
        gbp_set_error("batch: need offsets, n_inst >= 1, 1 <= max_steps <= %d", kMaxSteps);
        return GBP_ERR_ARG;
    }
    *out = nullptr;
    if (offsets[0] != 0) {
        gbp_set_error("batch: offsets[0] must be 0");
        return GBP_ERR_ARG;
    }
    int mx = 0;
    for (int i = 0; i < n_inst; ++i) {
        if (offsets[i + 1] < offsets[i]) {
            gbp_set_error("batch: offsets must be non-decreasing");
            return GBP_ERR_ARG;
        }
        mx = std::max(mx, offsets[i + 1] - offsets[i]);
    }
    gbp_batch b = new gbp_batch_s();
    (void)hipGetDevice(&b->device);
    b->n_inst = n_inst;
    b->max_verts = std::max(mx, 1);
    b->total = offsets[n_inst];
    b->max_steps = max_steps;
    const size_t nwork = (size_t)n_inst * ecg_work_floats(max_steps);
    if (hipMalloc((void**)&b->off, sizeof(int) * (n_inst + 1)) != hipSuccess ||
        hipMalloc((void**)&b->work, sizeof(float) * nwork) != hipSuccess) {
        gbp_set_error("batch: allocation failed");
        gbp_batch_destroy(b);
        return GBP_ERR_NOMEM;
    }
    if (hipMemcpy(b->off, offsets, sizeof(int) * (n_inst + 1), hipMemcpyHostToDevice) != hipSuccess) {
        gbp_set_error("batch: copy failed");
        gbp_batch_destroy(b);
        return GBP_ERR_HIP;
    }
    *out = b;
    return GBP_OK;
}

extern "C" int gbp_batch_sizes(gbp_batch b, int* n_inst, int* n_total) {
    if (!b) {
        gbp_set_error("batch is NULL");
        return GBP_ERR_ARG;
    }
    if (n_inst) *n_inst = b->n_inst;
    if (n_total) *n_total = b->total;
    return GBP_OK;
}

extern "C" void gbp_batch_destroy(gbp_batch b) {
    if (!b) return;
    if (b->off) (void)hipFree(b->off);
    if (b->work) (void)hipFree(b->work);
    delete b;
}

static int check_batch(gbp_batch b, const gbp_ap* ap) {
    if (!b) {
        gbp_set_error("batch is NULL");
        return GBP_ERR_ARG;
    }
    if (ap && ap->n_steps > b->max_steps) {
        gbp_set_error("n_steps %d exceeds the batch's max_steps %d", ap->n_steps, b->max_steps);
        return GBP_ERR_ARG;
    }
    return GBP_OK;
}

extern "C" int gbp_ecg_forward(const float* T, int n_v, const float* W, int L, const gbp_ap* ap,
                               float* ecg, void* stream) {
    int rc = check_ap(T, n_v, W, L, ap);
    if (rc) return rc;
    if (!ecg) {
        gbp_set_error("ecg is NULL");
        return GBP_ERR_ARG;
    }
    float* work;
    if ((rc = ecg_workspace(ecg_work_floats(ap->n_steps), &work))) return rc;
    return ecg_forward_launch(EcgLaunch{nullptr, 1, n_v, work, ecg_work_floats(ap->n_steps)}, T, n_v, W, L, ap, ecg,
                              (hipStream_t)stream);
}

extern "C" int gbp_ecg_forward_noalloc(const float* T, int n_v, const float* W, int L,
                                       const gbp_ap* ap, float* ecg, void* stream) {
    int rc = check_ap(T, n_v, W, L, ap);
    if (rc) return rc;
    if (!ecg) {
        gbp_set_error("ecg is NULL");
        return GBP_ERR_ARG;
    }
    float* work;
    if ((rc = noalloc_scratch(&work))) return rc;
    return ecg_forward_launch(EcgLaunch{nullptr, 1, n_v, work, kNoAllocFloats}, T, n_v, W, L, ap, ecg,
                              (hipStream_t)stream);
}

extern "C" int gbp_ecg_backward(const float* T, int n_v, const float* W, int L, const gbp_ap* ap,
                                const float* dL_decg, float* dL_dT, void* stream) {
    int rc = check_ap(T, n_v, W, L, ap);
    if (rc) return rc;
    if (!dL_decg || !dL_dT) {
        gbp_set_error("dL_decg and dL_dT are required");
        return GBP_ERR_ARG;
    }
    return ecg_backward_launch(EcgLaunch{nullptr, 1, n_v, nullptr, 0}, T, n_v, W, L, ap, dL_decg, dL_dT,
                               (hipStream_t)stream);
}

extern "C" int gbp_ecg_forward_batched(gbp_batch b, const float* T, const float* W, int L,
                                       const gbp_ap* ap, float* ecg, void* stream) {
    int rc = check_batch(b, ap);
    if (rc) return rc;
    if ((rc = check_ap(T, b->total, W, L, ap))) return rc;
    if (!ecg) {
        gbp_set_error("ecg is NULL");
        return GBP_ERR_ARG;
    }
    return ecg_forward_launch(
        EcgLaunch{b->off, b->n_inst, b->max_verts, b->work, ecg_work_floats(b->max_steps)}, T, b->total, W, L, ap, ecg,
        (hipStream_t)stream);
}

extern "C" int gbp_ecg_backward_batched(gbp_batch b, const float* T, const float* W, int L,
                                        const gbp_ap* ap, const float* dL_decg, float* dL_dT,
                                        void* stream) {
    int rc = check_batch(b, ap);
    if (rc) return rc;
    if ((rc = check_ap(T, b->total, W, L, ap))) return rc;
    if (!dL_decg || !dL_dT) {
        gbp_set_error("dL_decg and dL_dT are required");
        return GBP_ERR_ARG;
    }
    return ecg_backward_launch(EcgLaunch{b->off, b->n_inst, b->max_verts, nullptr, 0}, T, b->total, W,
                               L, ap, dL_decg, dL_dT, (hipStream_t)stream);
}
