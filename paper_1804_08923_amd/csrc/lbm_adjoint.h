// Reverse (adjoint) step of the colour-gradient LBM update.
//
// The step maps the state x_t = (f^r, f^b) (54 values per node) to x_{t+1}.
// For a cotangent lambda_{t+1} of x_{t+1} the adjoint step returns
// lambda_t = (d x_{t+1} / d x_t)^T lambda_{t+1} and adds lambda_{t+1} . d x_{t+1}/dA
// and lambda_{t+1} . d x_{t+1}/d u_in (the inlet axial-velocity profile) to the
// caller's gradient accumulators.  The forward quantities of step t are
// recomputed from x_t (no tape).  Passes:
//   1. densities of x_t -> (phi, rho - rho_b0), rho_r/rho per node, and the
//      raw moments of the colour-blind deviations up to second order
//   2. (jet) outlet: the convective condition of the outlet plane depends on the
//      streamed populations of the plane below; its adjoint is formed first
//      from a forward recomputation of the three top planes
//   3. per node: reverse streaming (gather of lambda_{t+1} from x + c_i, with the
//      reflections, inlet absorption and outlet rules of the forward step),
//      then the node vector-Jacobian product (lbm_adjoint_node.h); writes the
//      cotangents of the 10 raw moments (the cotangent of deviation i is their
//      quadratic polynomial in c_i), 8 stencil/centre cotangents and a block
//      partial of dJ/dA
//   4. ghost shell of the stencil cotangents (periodic copies; jet: zero,
//      plus the sums that the mirrored ghost fields route back to the wall nodes)
//   5. per node: transpose of the gradient stencil, chain rule through
//      phi(rho_r, rho_b), rho and rho_r/rho, and the red/blue cotangents
//   6. (jet) dJ/du_in over the inlet circle; dJ/dA reduction.
#pragma once
#include "lbm_adjoint_node.h"

namespace cglbm {

// ---------------------------------------------------------------- work buffer
struct AdjWork {
    float* MOM;     // raw moments m0, j (3), P (xx yy zz xy xz yz) of the deviations [10][N]
    float* LC;      // their cotangents [10][N]
    float4* AG0;    // (L grad phi, L phi_centre) per padded node
    float4* AG1;    // (L grad rho, L rho_r/rho) per padded node
    float2* GH;     // jet: stencil cotangents gathered at ghost cells (phi, rho)
    float* PS;      // jet: post-collision populations of the top three planes [54][3][plane]
    float* ML;      // jet: cotangent of the streamed plane nz - 2 incl. the outlet condition [54][plane]
    float* DL;      // jet: direct outlet term of lambda_t at plane nz - 1 [54][plane]
    float* ST;      // jet, state from a snapshot: the outlet plane of x_t as (d, f^r) [54][plane]
    double* AP;     // dJ/dA block partials
};

inline uint64_t align256(uint64_t b) { return (b + 255) & ~(uint64_t)255; }

inline uint64_t adjoint_layout(uint64_t NP, uint64_t N, uint64_t plane, uint64_t nblk, char* base, AdjWork* w)
{
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        char* p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    };
    char* mom = take(N * 10 * 4);
    char* lc = take(N * 10 * 4);
    char* a0 = take(NP * 16);
    char* a1 = take(NP * 16);
    char* gh = take(NP * 8);
    char* ps = take(2ull * Q * 3 * plane * 4);
    char* ml = take(2ull * Q * plane * 4);
    char* dl = take(2ull * Q * plane * 4);
    char* sp = take(2ull * Q * plane * 4);
    char* ap = take((nblk + 1) * 8);
    if (w) {
        w->MOM = (float*)mom;
        w->LC = (float*)lc;
        w->AG0 = (float4*)a0;
        w->AG1 = (float4*)a1;
        w->GH = (float2*)gh;
        w->PS = (float*)ps;
        w->ML = (float*)ml;
        w->DL = (float*)dl;
        w->ST = (float*)sp;
        w->AP = (double*)ap;
    }
    return off;
}

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ uint32_t nidx(const KP& k, int x, int y, int z)
{
    return ((uint32_t)z * (uint32_t)k.ny + (uint32_t)y) * (uint32_t)k.nx + (uint32_t)x;
}

// node x of a row of nx values at a uniform address
__device__ __forceinline__ float ld_lane(const float* base, int nx, int x)
{
    return ld_row<float>(row_rsrc(base, (uint32_t)nx), (uint32_t)x * 4u, 0u);
}
template <bool NT>
__device__ __forceinline__ void st_lane(float* base, int nx, int x, float v)
{
    st_row<NT>(row_rsrc(base, (uint32_t)nx), (uint32_t)x * 4u, 0u, v);
}
// first three components of the stencil cotangents of node x, row (y, z) uniform
__device__ __forceinline__ float3 ld_cot(const float4* __restrict__ AG, const KP& k, int x, int y, int z)
{
    const auto r = row_rsrc(AG + pidx(k, -1, y, z), (uint32_t)k.px);
    const auto v = __builtin_amdgcn_raw_buffer_load_b96(r, (uint32_t)(x + 1) * 16u, 0, 0);
    return make_float3(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]));
}
__device__ __forceinline__ float3 cot_at(const float4* __restrict__ AG, const KP& k, int x, int y, int z)
{
    const float4 v = ldp(AG, pidx(k, x, y, z));
    return make_float3(v.x, v.y, v.z);
}

// 1. densities and raw moments of the deviations d_i = f^r_i + f^b_i - w_i rho_b0
// of an FP32 state (fr planes, then fb), accumulated in FP64
__global__ __launch_bounds__(BLOCK) void k_adj_density(const float* __restrict__ st, float2* __restrict__ PD,
                                                        float* __restrict__ XR, float* __restrict__ MOM, KP k)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const size_t N = k.N;
    const uint32_t n = nidx(k, nd.x, nd.y, nd.z);
    double rr = 0.0;
    MomT<double> M;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double a = st[(size_t)i * N + n], b = st[(size_t)(Q + i) * N + n];
        rr += a;
        M.add(i, (a + b) - wgtd(i) * (double)k.rho_b0);
    }
    // the adjoint passes keep the red fraction x_r = rho_r/rho in XR
    const double rho = (double)k.rho_b0 + M.m0;
    store_pd(PD, k, nd.n, M.m0, rr, rho - rr);
    stp(XR, nd.n, (float)(rr / rho));
    const double mv[10] = {M.m0, M.j[0], M.j[1], M.j[2], M.P[0], M.P[1], M.P[2], M.P[3], M.P[4], M.P[5]};
#pragma unroll
    for (int a = 0; a < 10; ++a) MOM[(size_t)a * N + n] = (float)mv[a];
}

// forward node quantities of node nd from its moments and the field stencil
template <int BC>
__device__ __forceinline__ void adj_node_fwd(const KP& k, const float* __restrict__ MOM,
                                             const float2* __restrict__ PD, const float* __restrict__ XR,
                                             const Node& nd, NodeFwdT<float>& f, float& xr)
{
    const size_t N = k.N;
    const uint32_t n = nidx(k, nd.x, nd.y, nd.z);
    MomT<float> M;
    M.m0 = MOM[n];
    for (int a = 0; a < 3; ++a) M.j[a] = MOM[(size_t)(1 + a) * N + n];
    for (int a = 0; a < 6; ++a) M.P[a] = MOM[(size_t)(4 + a) * N + n];
    const float phic = ldp(PD, nd.n).x;
    xr = ldp(XR, nd.n);
    if (k.xr_tagged) xr = frac_of(xr, 0u);
    double g[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    gradients<BC>(PD, k, nd, g);
    node_fwd<float>(k, M, phic, g, f);
}

// 2a. (jet) post-collision populations of planes nz - 3 .. nz - 1 (z0 = nz - 3)
__global__ __launch_bounds__(BLOCK) void k_adj_top_post(const float* __restrict__ MOM, const float2* __restrict__ PD,
                                                         const float* __restrict__ XR, float* __restrict__ PS, KP k)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    NodeFwdT<float> f;
    float xr;
    adj_node_fwd<LBM_BC_JET>(k, MOM, PD, XR, nd, f, xr);
    float fp[Q], V[3];
    node_post<float>(k, f, xr, fp, V);
    const int zz = nd.z - k.z0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        float fr, fb;
        recolour_dir<float>(i, xr, fp[i], V, fr, fb);
        PS[((size_t)i * 3 + zz) * k.plane + nd.q] = fr;
        PS[((size_t)(Q + i) * 3 + zz) * k.plane + nd.q] = fb;
    }
}

// 2b. (jet) outlet condition f(N) = [h + lam y] / (1 + lam), lam = max(0, u_z(y)),
// y = the streamed populations of plane nz - 2, h = the state's plane nz - 1.
// Writes ML = cotangent of y (lambda of plane nz - 2 plus the outlet terms) and
// DL = lambda of plane nz - 1 / (1 + lam) (the direct dependence on h).
// h comes as (f^r, f^b) planes of stride hs (dfr = 0) or as the (d, f^r)
// planes of stride plane that the density pass of a snapshot wrote (dfr = 1).
__device__ __forceinline__ double top_value(const KP& k, const float* __restrict__ h, size_t hs, int dfr, int j,
                                            uint32_t q)
{
    if (!dfr) return h[(size_t)j * hs + q];
    if (j < Q) return h[(size_t)(Q + j) * k.plane + q];
    const int i = j - Q;
    return ((double)h[(size_t)i * k.plane + q] + wgtd(i) * (double)k.rho_b0) - (double)h[(size_t)(Q + i) * k.plane + q];
}

__global__ __launch_bounds__(BLOCK) void k_adj_outlet(const float* __restrict__ htop, size_t hs, int dfr,
                                                       const float* __restrict__ lam_in,
                                                       const float* __restrict__ PS, float* __restrict__ ML,
                                                       float* __restrict__ DL, KP k)
{
    const uint32_t q = blockIdx.x * BLOCK + threadIdx.x;
    if (q >= k.plane) return;
    const int y = (int)(q / (uint32_t)k.nx), x = (int)(q - (uint32_t)y * k.nx);
    const int zb = k.nz - 2, zt = k.nz - 3;
    const size_t N = k.N, P = k.plane;
    float yv[2 * Q];
    double rho = 0.0, jz = 0.0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        int sx = x - kCX[j], sy = y - kCY[j], m = 0;
        if (sx < 0 || sx >= k.nx) { m |= 1; sx = x; }
        if (sy < 0 || sy >= k.ny) { m |= 2; sy = y; }
        const int jj = kMirror.v[j * 8 + m];
        const int zz = zb - kCZ[j] - zt;
        const uint32_t s = (uint32_t)sy * k.nx + (uint32_t)sx;
        yv[j] = PS[((size_t)jj * 3 + zz) * P + s];
        yv[Q + j] = PS[((size_t)(Q + jj) * 3 + zz) * P + s];
        const double f = (double)yv[j] + (double)yv[Q + j];
        rho += f;
        jz += kCZ[j] * f;
    }
    const double uz = (jz + 0.5 * (rho - (double)k.rho_b0) * (double)k.gz) / rho;
    const double lam = uz > 0.0 ? uz : 0.0;
    const double inv = 1.0 / (1.0 + lam);
    const size_t ntop = (size_t)(k.nz - 1) * P + q, nbot = (size_t)zb * P + q;
    double Llam = 0.0;
#pragma unroll
    for (int j = 0; j < 2 * Q; ++j) {
        const double L1 = lam_in[(size_t)j * N + ntop];
        const double h = top_value(k, htop, hs, dfr, j, q);
        Llam += L1 * ((double)yv[j] - h) * inv * inv;
    }
    const double Luz = uz > 0.0 ? Llam : 0.0;
#pragma unroll
    for (int j = 0; j < 2 * Q; ++j) {
        const int i = j < Q ? j : j - Q;
        const double L1 = lam_in[(size_t)j * N + ntop];
        const double L2 = lam_in[(size_t)j * N + nbot];
        ML[(size_t)j * P + q] = (float)(L2 + L1 * lam * inv + Luz * ((double)kCZ[i] + 0.5 * (double)k.gz - uz) / rho);
        DL[(size_t)j * P + q] = (float)(L1 * inv);
    }
}

// 3. reverse streaming and node VJP
// Where the cotangents of a node's post-collision populations lie.  The lattice rows
// y + c_y and z + c_z, the reflections on y and z and the planes that the outlet
// condition replaces are uniform over the wavefront (it lies in one row); along x
// a lane at the wall reads itself in the direction reversed on x.
struct GatherRows {
    const float* base[3];  // [c_z + 1] plane z + c_z of population 0
    size_t stride[3];      // from population to population
    bool lost[3];          // overwritten by the outlet condition
    uint32_t row[3];       // [c_y + 1] first node of row y + c_y in its plane
    bool my[2];            // [c_y > 0] reflected on y
    bool mz;               // reflected on z (c_z = -1)
};
template <int BC>
__device__ __forceinline__ GatherRows gather_rows(const KP& k, const float* __restrict__ lam,
                                                  const float* __restrict__ ML, int y, int z)
{
    GatherRows g;
    g.mz = BC == LBM_BC_JET && z == 0;
#pragma unroll
    for (int c = -1; c <= 1; ++c) {
        int zs = z + c, ys = y + c;
        g.lost[c + 1] = false;
        if (BC == LBM_BC_PERIODIC) {
            zs = wrapc(zs, k.nz);
            ys = wrapc(ys, k.ny);
        } else {
            if (c < 0 && g.mz) zs = 0;
            g.lost[c + 1] = c >= 0 && zs >= k.nz - 1;
            if (g.lost[c + 1]) zs = k.nz - 2;  // any plane: the value is dropped
            if (c != 0) g.my[c > 0] = ys < 0 || ys >= k.ny;
            ys = clampc(ys, k.ny);
        }
        const bool below = BC == LBM_BC_JET && zs == k.nz - 2;  // the plane under the outlet
        g.base[c + 1] = below ? ML : lam + (size_t)zs * k.plane;
        g.stride[c + 1] = below ? (size_t)k.plane : (size_t)k.N;
        g.row[c + 1] = (uint32_t)ys * (uint32_t)k.nx;
    }
    return g;
}

// lane offsets along x of c_x = +1 and -1, and (jet) the lanes at the walls
struct XSide {
    int p, m;
    bool wp, wm;
    bool inlet;  // the node below the lane is an inlet cell: overwritten by the inflow
};

// cotangents of the post-collision population I of this node, red and blue: those of
// the population it becomes after streaming (x + c_i, reversed on every axis
// that leaves the lattice), zero where the forward step overwrites it
template <int BC, int I>
__device__ __forceinline__ void adj_gather_dir(const GatherRows& g, int x, const XSide& xs, float& vr, float& vb)
{
    constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
    const float* p = g.base[cz + 1] + g.row[cy + 1];
    const size_t stride = g.stride[cz + 1];
    const int xo = cx > 0 ? xs.p : (cx < 0 ? xs.m : x);
    if constexpr (BC == LBM_BC_PERIODIC) {
        p += I * stride;
        vr = ldp(p, (uint32_t)xo);
        vb = ldp(p + Q * stride, (uint32_t)xo);
    } else {
        const bool my = cy != 0 && g.my[cy > 0], mz = cz < 0 && g.mz;
        const int j = my ? (mz ? dir_of(cx, -cy, -cz) : dir_of(cx, -cy, cz)) : (mz ? dir_of(cx, cy, -cz) : I);
        p += (size_t)j * stride;
        const float* pb = p + Q * stride;
        if constexpr (cx == 0) {
            vr = ldp(p, (uint32_t)x);
            vb = ldp(pb, (uint32_t)x);
        } else {
            const int jm = my ? (mz ? dir_of(-cx, -cy, -cz) : dir_of(-cx, -cy, cz))
                              : (mz ? dir_of(-cx, cy, -cz) : dir_of(-cx, cy, cz));
            const bool wall = cx > 0 ? xs.wp : xs.wm;
            const int64_t o = wall ? (int64_t)(jm - j) * (int64_t)stride + x : (int64_t)xo;
            vr = p[o];
            vb = pb[o];
        }
    }
}
template <int BC, int I = 0>
__device__ __forceinline__ void adj_gather(const GatherRows& g, int x, const XSide& xs, float* Lr, float* Lb)
{
    if constexpr (I < Q) {
        adj_gather_dir<BC, I>(g, x, xs, Lr[I], Lb[I]);
        adj_gather<BC, I + 1>(g, x, xs, Lr, Lb);
    }
}
// zero for the populations that the forward step overwrites: after all loads, so
// that none of them is waited for by itself
__device__ __forceinline__ void adj_drop(const GatherRows& g, const XSide& xs, float* Lr, float* Lb)
{
    if (g.mz) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (kCZ[i] >= 0) continue;
            const bool my = kCY[i] != 0 && g.my[kCY[i] > 0];
            if (!my && xs.inlet && !(kCX[i] > 0 ? xs.wp : (kCX[i] < 0 && xs.wm))) Lr[i] = Lb[i] = 0.f;
        }
    }
    if (g.lost[2]) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
            if (kCZ[i] > 0 || (kCZ[i] == 0 && g.lost[1])) Lr[i] = Lb[i] = 0.f;
    }
}

// 783 -> 540 us on the 128x128x512 jet (460 would be the traffic of 340 B per node).
// It was bound by its arithmetic at two waves per SIMD, 3600 vector instructions per
// wave on 256 registers: per-lane 64-bit addresses, mirrored directions by selects per
// lane, the node map direction by direction.  Rows by scalars and the node map by
// opposite pairs leave 2000 (620 us), by moments 1570 on 141 registers (590 us), which
// three waves per SIMD hold (540 us; four spill).  dJ/dA's terms in FP64 (perturb_vjp)
// make it 1730 on 155 registers, 16 us more.  Arithmetic takes 0.65 of the SIMDs' time
// now (by counters, at 2.4 GHz).  The loads go out before the window's barrier: 130 us
// slower with the window first.
template <int BC, class TL>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_adj_node(
    const float* __restrict__ MOM, const float* __restrict__ lam_in, const float* __restrict__ ML,
    const float2* __restrict__ PD, const float* __restrict__ XR, float* __restrict__ LC, float4* __restrict__ AG0,
    float4* __restrict__ AG1, double* __restrict__ AP, KP k)
{
    constexpr int TX = TL::CX, TY = TL::CY;
    __shared__ float2 win[TileShape<TX, TY>::W];
    const Tile t = this_tile<TX, TY>(k);
    const Node& nd = t.nd;
    double acc[1] = {0.0};
    // all global loads before the barrier of the window; lanes and blocks beyond the
    // lattice repeat its last nodes
    const size_t N = k.N;
    const int y = min(t.y0 + t.ly, k.ny - 1), z = min(t.z, k.nz - 1), x = min(nd.x, k.nx - 1);
    const size_t row = ((size_t)z * k.ny + y) * (uint32_t)k.nx;
    float Lr[Q], Lb[Q];
    XSide xs;
    xs.p = x + 1;
    xs.m = x - 1;
    xs.wp = x == k.nx - 1;
    xs.wm = x == 0;
    xs.inlet = BC == LBM_BC_JET && z == 0 && inlet_inside(k, x, y);
    if (BC == LBM_BC_PERIODIC) {
        if (xs.wp) xs.p = 0;
        if (xs.wm) xs.m = k.nx - 1;
    }
    const GatherRows rows = gather_rows<BC>(k, lam_in, ML, y, z);
    adj_gather<BC>(rows, x, xs, Lr, Lb);
    MomT<float> M;
    const float* mom = MOM + row;
    M.m0 = ldp(mom, (uint32_t)x);
    for (int a = 0; a < 3; ++a) M.j[a] = ldp(mom + (size_t)(1 + a) * N, (uint32_t)x);
    for (int a = 0; a < 6; ++a) M.P[a] = ldp(mom + (size_t)(4 + a) * N, (uint32_t)x);
    float xr = ldp(XR, nidx_of(k, x, y, z));
    stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return pd_at<BC, true>(k, PD, x, y, z); },
                         [&](int x, int y, int z) { return pd_at<BC>(k, PD, x, y, z); },
                         [&](int w, const float2& v) { win[w] = v; });
    __syncthreads();
    if (nd.valid) {
        if (BC == LBM_BC_JET) adj_drop(rows, xs, Lr, Lb);
        if (k.xr_tagged) xr = frac_of(xr, 0u);
        double g[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        gradients_win<TX, TY>(win, t.lx, t.ly, g);
        acc[0] = perturb_vjp(k, g, (double)xr, Lr, Lb);
        NodeFwdT<float> f;
        node_fwd<float>(k, M, win[wslot<TX, TY>(t.lx, t.ly, 0, 0, 0)].x, g, f);
        NodeAdjT<float> o;
        node_vjp<float>(k, f, xr, Lr, Lb, o);
        const float lc[10] = {o.Lm0, o.Lj[0], o.Lj[1], o.Lj[2], o.Lq[0], o.Lq[1], o.Lq[2], o.Lq[3], o.Lq[4], o.Lq[5]};
        float* lcr = LC + row;
#pragma unroll
        for (int a = 0; a < 10; ++a) stp(lcr + (size_t)a * N, (uint32_t)x, lc[a]);
        const uint32_t pn = pidx(k, x, y, z);
        stp(AG0, pn, make_float4(o.Lgp[0], o.Lgp[1], o.Lgp[2], o.Lphic));
        stp(AG1, pn, make_float4(o.Lgr[0], o.Lgr[1], o.Lgr[2], o.Lxr));
    }
    block_partials<1>(acc, AP, blockIdx.y * gridDim.x + blockIdx.x);
}

// 4. ghost shell of the stencil cotangents.  Periodic: copies of the wrapped
// nodes.  Jet: zero (the transpose gather then sees only interior nodes), and
// GH = the stencil cotangent that reads this ghost cell's mirrored field
// value, to be routed to the wall node it copies (zero in the inlet circle,
// where the ghost fields are constants).
template <int BC>
__global__ __launch_bounds__(BLOCK) void k_adj_ghosts(float4* __restrict__ AG0, float4* __restrict__ AG1,
                                                       float2* __restrict__ GH, KP k, uint32_t ncells)
{
    const uint32_t gidx = blockIdx.x * BLOCK + threadIdx.x;
    if (gidx >= ncells) return;
    const Ghost c = shell_cell(k, gidx);
    if (!c.valid) return;
    const uint32_t gi = pidx(k, c.x, c.y, c.z);
    if (BC == LBM_BC_PERIODIC) {
        const uint32_t wi = pidx(k, wrapc(c.x, k.nx), wrapc(c.y, k.ny), wrapc(c.z, k.nz));
        AG0[gi] = AG0[wi];
        AG1[gi] = AG1[wi];
        return;
    }
    float sp = 0.f, sr = 0.f;
    if (!(c.z < 0 && inlet_inside(k, c.x, c.y))) {
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const int x = c.x - kCX[i], y = c.y - kCY[i], z = c.z - kCZ[i];
            if (x < 0 || x >= k.nx || y < 0 || y >= k.ny || z < 0 || z >= k.nz) continue;
            const uint32_t s = pidx(k, x, y, z);
            const float4 a0 = AG0[s], a1 = AG1[s];
            const float w3 = 3.f * wgt(i);
            sp += w3 * (kCX[i] * a0.x + kCY[i] * a0.y + kCZ[i] * a0.z);
            sr += w3 * (kCX[i] * a1.x + kCY[i] * a1.y + kCZ[i] * a1.z);
        }
    }
    GH[gi] = make_float2(sp, sr);
    // only interior cells are read above, only ghost cells are written here
    AG0[gi] = make_float4(0.f, 0.f, 0.f, 0.f);
    AG1[gi] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// 5. transpose of the gradient stencil and the red / blue cotangents.  300 B of
// traffic per node, two thirds of it the 54 stores; NT (the cotangents do not fit the
// memory-side cache): non-temporal ones.  665 -> 540 us on the 128x128x512 jet with
// 24 instead of 32 B per window node, the node's own loads before the barrier and the
// stores' rows in scalar registers.
template <int BC, class TL, bool NT>
__global__ __launch_bounds__(BLOCK) void k_adj_fields(const float4* __restrict__ AG0, const float4* __restrict__ AG1,
                                                       const float2* __restrict__ GH, const float2* __restrict__ PD,
                                                       const float* __restrict__ XR, const float* __restrict__ DL,
                                                       const float* __restrict__ LC, float* __restrict__ lam_out, KP k)
{
    // the stencil cotangents of the tile and its rim from LDS windows, without the
    // fourth components, which only the node itself reads: 24 B per node, four blocks
    // per CU instead of three
    constexpr int TX = TL::CX, TY = TL::CY, W = TileShape<TX, TY>::W;
    __shared__ float2 w0[W], w1[W], w2[W];
    const Tile t = this_tile<TX, TY>(k);
    const Node& nd = t.nd;
    // the node's own values before the barrier of the window; lanes and blocks beyond
    // the lattice repeat its last nodes
    const size_t N = k.N;
    const int y = min(t.y0 + t.ly, k.ny - 1), z = min(t.z, k.nz - 1), x = min(nd.x, k.nx - 1);
    const uint32_t q0 = (uint32_t)y * (uint32_t)k.nx, nn = nidx_of(k, x, y, z), pn = pidx(k, x, y, z);
    const size_t row = (size_t)z * k.plane + q0;
    const float* lcr = LC + row;
    float lc[10];
#pragma unroll
    for (int c = 0; c < 10; ++c) lc[c] = ld_lane(lcr + (size_t)c * N, k.nx, x);
    const float2 pd = ldp(PD, nn);
    float xrn = ldp(XR, nn);
    float Lphi = ldp(AG0, pn).w, Lrf = 0.f;
    const float Lxr = ldp(AG1, pn).w;
    // batched staging (all loads before the LDS writes): 1.95 -> 1.73 ms per
    // adjoint step on the 128x128x512 jet
    stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return ld_cot(AG0, k, x, y, z); },
                         [&](int x, int y, int z) { return cot_at(AG0, k, x, y, z); },
                         [&](int w, const float3& v) { w0[w] = make_float2(v.x, v.y); w1[w].x = v.z; });
    stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return ld_cot(AG1, k, x, y, z); },
                         [&](int x, int y, int z) { return cot_at(AG1, k, x, y, z); },
                         [&](int w, const float3& v) { w1[w].y = v.x; w2[w] = make_float2(v.y, v.z); });
    __syncthreads();
    if (!nd.valid) return;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int ws = wslot<TX, TY>(t.lx, t.ly, -kCX[i], -kCY[i], -kCZ[i]);
        const float2 a = w0[ws], b = w1[ws], c = w2[ws];
        const float w3 = 3.f * wgt(i);
        Lphi += w3 * cdot(i, a.x, a.y, b.x);
        Lrf += w3 * cdot(i, b.y, c.x, c.y);
    }
    if (BC == LBM_BC_JET) {
        // ghost cells whose mirrored field value is this node's
        const int lx = nd.x == 0 ? -1 : 0, hx = nd.x == k.nx - 1 ? 1 : 0;
        const int ly = nd.y == 0 ? -1 : 0, hy = nd.y == k.ny - 1 ? 1 : 0;
        const int lz = nd.z == 0 ? -1 : 0, hz = nd.z == k.nz - 1 ? 1 : 0;
        if (lx | hx | ly | hy | lz | hz) {
            for (int sz = lz; sz <= hz; ++sz)
                for (int sy = ly; sy <= hy; ++sy)
                    for (int sx = lx; sx <= hx; ++sx) {
                        if (!(sx | sy | sz)) continue;
                        const float2 gh = GH[pidx(k, nd.x + sx, nd.y + sy, nd.z + sz)];
                        Lphi += gh.x;
                        Lrf += gh.y;
                    }
        }
    }
    // phi = (a - b)/(a + b), a = rho_r/rho_r0, b = rho_b/rho_b0; rho_r/rho; rho
    const double rho = (double)k.rho_b0 + (double)pd.y;
    if (k.xr_tagged) xrn = frac_of(xrn, 0u);
    const double rr = (double)xrn * rho, rb = rho - rr;
    const double a = rr / (double)k.rho_r0, b = rb / (double)k.rho_b0;
    const double ab2 = (a + b) * (a + b);
    const float Lrr = (float)(Lphi * 2.0 * b / (ab2 * (double)k.rho_r0) + Lrf + Lxr * rb / (rho * rho));
    const float Lrb = (float)(-Lphi * 2.0 * a / (ab2 * (double)k.rho_b0) + Lrf - Lxr * rr / (rho * rho));
    const bool top = BC == LBM_BC_JET && t.z == k.nz - 1;
    float* out = lam_out + row;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
        float Ld = lc[0];
        if (cx) Ld += cx * lc[1] + lc[4];
        if (cy) Ld += cy * lc[2] + lc[5];
        if (cz) Ld += cz * lc[3] + lc[6];
        if (cx * cy) Ld += (cx * cy) * lc[7];
        if (cx * cz) Ld += (cx * cz) * lc[8];
        if (cy * cz) Ld += (cy * cz) * lc[9];
        float r = Ld + Lrr, bl = Ld + Lrb;
        if (top) {
            r += ldp(DL + (size_t)i * k.plane + q0, (uint32_t)x);
            bl += ldp(DL + (size_t)(Q + i) * k.plane + q0, (uint32_t)x);
        }
        st_lane<NT>(out + (size_t)i * N, k.nx, x, r);
        st_lane<NT>(out + (size_t)(Q + i) * N, k.nx, x, bl);
    }
}

// 6a. (jet) dJ/du_in: the inlet ghost column (gx, gy) feeds the red populations
// with c_z = +1 of the nodes (gx + c_x, gy + c_y, 0) with its equilibrium.
template <int I = 0>
__device__ __forceinline__ void inlet_grad_dirs(const KP& k, const float* __restrict__ lam, int gx, int gy,
                                                const double (&u)[3], double& acc)
{
    if constexpr (I < Q) {
        if constexpr (kCZ[I] == 1) {
            const int x = gx + kCX[I], y = gy + kCY[I];
            if (x >= 0 && x < k.nx && y >= 0 && y < k.ny) {
                const double cu = kCX[I] * u[0] + kCY[I] * u[1] + u[2];
                const double u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
                const double dfe = (double)k.rho_r0 * wgtd(I) *
                                   ((3.0 + 9.0 * cu + 13.5 * cu * cu - 4.5 * u2) - (3.0 + 9.0 * cu) * u[2]);
                acc += (double)lam[(size_t)I * k.N + (size_t)y * k.nx + x] * dfe;
            }
        }
        inlet_grad_dirs<I + 1>(k, lam, gx, gy, u, acc);
    }
}

__global__ __launch_bounds__(BLOCK) void k_adj_inlet(const float* __restrict__ lam_in, float* __restrict__ dJ_du,
                                                      KP k)
{
    const uint32_t q = blockIdx.x * BLOCK + threadIdx.x;
    if (q >= k.plane) return;
    const int gy = (int)(q / (uint32_t)k.nx), gx = (int)(q - (uint32_t)gy * k.nx);
    if (!inlet_inside(k, gx, gy)) return;
    // inflow velocity of this column at time t (same construction as the forward step)
    const uint64_t cnt = ((uint64_t)k.t * (uint64_t)k.ny + (uint64_t)gy) * (uint64_t)k.nx + (uint64_t)gx;
    const uint64_t r = splitmix64_nth(k.seed, cnt);
    const double xi = (double)(r >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
    const float ur = (float)((double)k.noise_amp * (double)k.inlet_u * xi);
    const float dx = (float)gx - k.inlet_cx, dy = (float)gy - k.inlet_cy;
    const float rr = sqrtf(dx * dx + dy * dy);
    double u[3];
    u[0] = rr > 0.f ? ur * dx / rr : 0.f;
    u[1] = rr > 0.f ? ur * dy / rr : 0.f;
    u[2] = k.inlet_uz ? k.inlet_uz[q] : k.inlet_u;
    double acc = 0.0;
    inlet_grad_dirs(k, lam_in, gx, gy, u, acc);
    dJ_du[q] += (float)acc;
}

// 6b. dJ/dA += sum of the block partials (one block of 1024 threads)
constexpr int SUM_BLOCK = 1024;
__global__ __launch_bounds__(SUM_BLOCK) void k_adj_sumA(const double* __restrict__ AP, int nblk,
                                                         double* __restrict__ out)
{
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int b = threadIdx.x;
    for (; b + 3 * SUM_BLOCK < nblk; b += 4 * SUM_BLOCK) {
        a0 += AP[b];
        a1 += AP[b + SUM_BLOCK];
        a2 += AP[b + 2 * SUM_BLOCK];
        a3 += AP[b + 3 * SUM_BLOCK];
    }
    for (; b < nblk; b += SUM_BLOCK) a0 += AP[b];
    __shared__ double red[SUM_BLOCK / 64];
    const double s = wave_sum((a0 + a1) + (a2 + a3));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < SUM_BLOCK / 64; ++w) t += red[w];
        out[0] += t;
    }
}

}  // namespace cglbm
