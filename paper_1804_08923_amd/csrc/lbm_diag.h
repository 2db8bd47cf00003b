// Jet diagnostics of Sec. IV C on the current state: the leading edge of the
// jet phase and its fragments.  The paper's fragment procedure: binarise the
// order parameter (1 for the jet phase, 0 elsewhere), take the connected
// components as fragments, measure each one's volume V and convert it to the
// equivalent spherical diameter d = (6 V / pi)^(1/3); the continuous column
// attached to the nozzle is left out.
//
// Readings: the jet phase is phi > 0 (Eq. order); components are face-
// connected (6-neighbourhood) on the lattice without wrap-around; V counts
// nodes (lattice cells of volume 1); the column is every component with a node
// on the inlet plane z = 0; the leading edge is the largest z of a jet node.
//
// Connected components by lock-free union-find over node indices (the label of
// a node is a parent pointer; every union hangs the larger of two roots under
// the smaller with an atomic minimum, so parents always have smaller indices
// and every find terminates): init, merge with the -x, -y, -z neighbours,
// flatten, count per root, collect the roots.
//
// On the 128x128x512 jet the five passes took 1.13 ms of which the count, one
// atomic per node on the few roots, took 0.53 ms, the first pass, in FP64
// throughout, 0.40 ms, and the merge of every node with three neighbours 0.13 ms.
#pragma once

#include "lbm_kernels.h"

namespace cglbm {

// device work buffer: header, then labels, counts, column marks, compacted
// fragment volumes (each N int32)
struct DiagHeader {
    unsigned long long jet_nodes;
    unsigned long long column_volume;
    unsigned int n_fragments;
    int front_z;
    int overflow;  // a union-find loop hit its iteration bound (never expected)
    int pad[9];
};
static_assert(sizeof(DiagHeader) == 64, "diagnostics header layout");

struct DiagWork {
    DiagHeader* hdr;
    int* label;
    int* count;
    int* column;
    int* volume;
};

constexpr uint64_t diag_bytes(uint64_t N) { return 256 + 4 * 4 * N; }

inline DiagWork diag_layout(void* base, uint64_t N)
{
    char* p = (char*)base;
    DiagWork w;
    w.hdr = (DiagHeader*)p;
    w.label = (int*)(p + 256);
    w.count = w.label + N;
    w.column = w.count + N;
    w.volume = w.column + N;
    return w;
}

// Every union-find walk strictly decreases a node index, so it ends within N
// steps; the loops carry that bound (walk) only as a guard against a defect.

__device__ __forceinline__ int diag_load(const int* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int diag_find(const int* __restrict__ L, int x, int walk, int* overflow)
{
    for (int it = 0; it <= walk; ++it) {
        const int p = diag_load(L + x);
        if (p == x) return x;
        x = p;
    }
    *overflow = 1;
    return x;
}

__device__ __forceinline__ void diag_unite(int* __restrict__ L, int a, int b, int walk, int* overflow)
{
    for (int it = 0; it <= walk; ++it) {
        a = diag_find(L, a, walk, overflow);
        b = diag_find(L, b, walk, overflow);
        if (a == b) return;
        if (a < b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(L + a, b);  // hang root a under b
        if (old == a) return;
        a = old;  // a was hung elsewhere meanwhile: continue from its parent
    }
    *overflow = 1;
}

__device__ __forceinline__ int wave_max_int(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

__global__ void k_diag_clear(DiagWork w)
{
    if (threadIdx.x == 0) {
        w.hdr->jet_nodes = 0;
        w.hdr->column_volume = 0;
        w.hdr->n_fragments = 0;
        w.hdr->front_z = -1;
        w.hdr->overflow = 0;
    }
}

// Label of a jet node on entry to the merge: the first node of its run along x
// within the wavefront's 64 nodes of a row, so that the runs need no union-find.
// fg: lane mask of the jet nodes, i the node's index.
__device__ __forceinline__ int diag_run_label(unsigned long long fg, int i)
{
    const int lane = (int)threadIdx.x & 63;
    const unsigned long long gap = ~fg & ((1ull << lane) - 1ull);
    return i - (lane - (gap ? 64 - __clzll(gap) : 0));
}

// jet nodes and leading edge of a wavefront into the header
__device__ __forceinline__ void diag_tally(const DiagWork& w, unsigned long long fg, int z)
{
    if (!fg) return;
    const int zmax = wave_max_int(z);
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&w.hdr->jet_nodes, (unsigned long long)__popcll(fg));
        atomicMax(&w.hdr->front_z, zmax);
    }
}

// 1. order parameter of the current state, binarised; labels.  The sign of phi is
// that of rho_r rho_b0 - rho_b rho_r0.  Where the FP32 masses of the density pass
// leave no doubt about it (their error is below 1e-5) it is taken from them, else
// from the FP64 sums of lbm_macroscopic.
template <int BC, class S, class TL>
__global__ __launch_bounds__(BLOCK) void k_diag_init(const typename S::T* __restrict__ src,
                                                      const float* __restrict__ hprev, KP k, DiagWork w)
{
    __shared__ float4 win[kRecWin<TL>];
    const Tile t = state_tile<BC, TL>(k, win);
    const Node& nd = t.nd;
    bool fg = false;
    const int i = (int)((uint32_t)nd.z * k.plane + nd.q);
    if (nd.valid) {
        bool sure = false;
        if (!TL::kFlat && !k.unshifted && !(BC == LBM_BC_JET && nd.z == k.nz - 1)) {
            float d[Q], unused[Q], m0 = 0.f, x0 = 0.f, cf = 0.f, cv = 0.f;
            uint32_t bl = 0;
            pull_dirs<BC, S, false>(src, k, nd.x, nd.y, nd.z, x_offsets<BC, typename S::T>(k, nd.x), d, unused, unused);
            accum_density_win<TL::CX, TL::CY, false>(k, d, win, t.lx, t.ly, m0, x0, bl, cf, cv);
            const float rho = k.rho_b0 + m0, mk = x0 * rho + (cf + (bl ? -cv : cv));
            const float a = (bl ? rho - mk : mk) * k.rho_b0, b = (bl ? mk : rho - mk) * k.rho_r0;
            sure = fabsf(a - b) > 1e-3f * (a + b) && a + b > 0.f;
            fg = a > b;
        }
        if (!sure) {
            double m0, rr, rb, j[3];
            node_masses<BC, S, TL>(src, k, hprev, t, win, m0, rr, rb, j);
            const double a = rr / k.rho_r0, b = rb / k.rho_b0;
            fg = (float)((a - b) / (a + b)) > 0.f;  // phi as lbm_macroscopic returns it
        }
    }
    const unsigned long long m = __ballot(fg);
    const int run = TL::kFlat ? i : diag_run_label(m, i);
    if (nd.valid) w.label[i] = fg ? run : -1;
    diag_tally(w, m, fg ? nd.z : -1);
}

// 2. union with the face neighbours at -x, -y, -z.  Runs are joined where segments
// meet; towards -y and -z one union is enough for nodes whose runs go on side by
// side.  RUNS: the labels are runs (else every node has its own).
template <bool RUNS>
__global__ __launch_bounds__(BLOCK) void k_diag_merge(KP k, DiagWork w)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const int i = (int)((uint32_t)nd.z * k.plane + nd.q);
    if (diag_load(w.label + i) < 0) return;
    const int walk = (int)k.N;
    const bool begins = !RUNS || (nd.x & 63) == 0;
    const bool left = nd.x > 0 && w.label[i - 1] >= 0;
    if (left && begins) diag_unite(w.label, i, i - 1, walk, &w.hdr->overflow);
    const auto join = [&](int o) {
        if (w.label[i - o] < 0) return;
        if (left && !begins && w.label[i - o - 1] >= 0) return;  // the node to the left joins the same two runs
        diag_unite(w.label, i, i - o, walk, &w.hdr->overflow);
    };
    if (nd.y > 0) join(k.nx);
    if (nd.z > 0) join((int)k.plane);
}

// 3. every jet node points at its root; the roots' counters
__global__ __launch_bounds__(BLOCK) void k_diag_flatten(KP k, DiagWork w)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const int i = (int)((uint32_t)nd.z * k.plane + nd.q);
    if (w.label[i] < 0) return;
    const int r = diag_find(w.label, i, (int)k.N, &w.hdr->overflow);
    w.label[i] = r;
    if (r == i) {
        w.count[i] = 0;
        w.column[i] = 0;
    }
}

// 4. volumes per root; roots of components with a node on z = 0.  A thread takes
// kCountPlanes nodes along z and a wavefront adds equal roots up before its atomics:
// the column's root would otherwise serialise an atomic for every one of its nodes.
constexpr int kCountPlanes = 16;
__device__ __forceinline__ void diag_add(const DiagWork& w, int root, int n)
{
    unsigned long long left = __ballot(n > 0);
    while (left) {  // one turn per distinct root
        const int first = __ffsll((long long)left) - 1;
        const int r = __shfl(root, first, 64);
        const bool same = n > 0 && root == r;
        const unsigned long long m = __ballot(same);
        int sum = same ? n : 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (((int)threadIdx.x & 63) == first) atomicAdd(w.count + r, sum);
        left &= ~m;
    }
}
__global__ __launch_bounds__(BLOCK) void k_diag_count(KP k, DiagWork w)
{
    KP kz = k;
    kz.z0 = 0;
    const Node nd = this_node(kz);  // z: block of planes
    const int z0 = nd.z * kCountPlanes;
    int root = -1, n = 0;
#pragma unroll 4
    for (int p = 0; p < kCountPlanes; ++p) {
        const int z = z0 + p;
        const int r = nd.valid && z < k.nz ? w.label[(size_t)(uint32_t)z * k.plane + nd.q] : -1;
        if (z == 0 && r >= 0) w.column[r] = 1;
        const bool other = r >= 0 && n > 0 && r != root;
        if (__any(other)) diag_add(w, root, other ? n : 0);
        if (r >= 0) {
            n = other ? 1 : n + 1;
            root = r;
        }
    }
    diag_add(w, root, n);
}

// 5. the column volume and the list of fragment volumes
__global__ __launch_bounds__(BLOCK) void k_diag_collect(KP k, DiagWork w)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const int i = (int)((uint32_t)nd.z * k.plane + nd.q);
    if (w.label[i] != i) return;
    if (w.column[i]) {
        atomicAdd(&w.hdr->column_volume, (unsigned long long)w.count[i]);
    } else {
        const unsigned int slot = atomicAdd(&w.hdr->n_fragments, 1u);
        w.volume[slot] = w.count[i];
    }
}

// 6. the first n fragment volumes widened to int64 into out (the label and
// count arrays, free once the volumes are collected), for the host copy
__global__ __launch_bounds__(BLOCK) void k_diag_widen(DiagWork w, uint32_t n, long long* __restrict__ out)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
    if (i < n) out[i] = (long long)w.volume[i];
}

}  // namespace cglbm
