// The step on the D3Q19 velocity set: the reduced lattice that Sec. II and
// Sec. IV B suggest as the way to cut the cost of the scheme, which the paper
// leaves without coefficients.  The coefficients keep every moment that the
// D3Q27 ones fix:
//   weights      1/3, 1/18 (faces), 1/36 (edges);
//   varphi_i     alpha at rest, w_i (1 - alpha) / (1 - w_0) = 1.5 w_i (1 - alpha)
//                otherwise (Eq. varphi_ik): sound speed squared (1 - alpha)/2;
//   Phi_i        -3 nu_bar u . grad rho at rest, m_i nu_bar (c.u)(c.grad rho)/4
//                with m = 2 on faces and 1 on edges (Eq. Phi): the second moment
//                nu_bar [u grad rho + grad rho u + (u . grad rho) I] of D3Q27;
//   B_i          -1/3 at rest, w_i otherwise (Eq. B_i): sum B_i = 1/3;
//   moments      the 19 rows of Eq. momentSet that are independent on D3Q19,
//                relaxed with s0, s1, s2nu, s2b, s3, s4 (Eq. scoll).
// Periodic and jet lattices, FP32 storage; the arithmetic is FP64 (the kernels are
// bound by memory traffic, and FP32 arithmetic would add about 1e-5 of the
// spurious velocity of a resting droplet to the FP32 storage floor).
// Layout, tiles, windows and walls are those of the D3Q27 kernels (rows without
// x ghosts, a wavefront inside one row but on narrow rows, the jet's ghost plane
// z = -1): against per-thread wrapped indices and neighbours through the caches the
// step on the 128x128x512 jet went from 0.61 to 0.46 ms.  The collision, by pairs of
// opposite directions, has 550 instead of 980 FP64 instructions per wave; all its
// vector instructions take half of the SIMDs' time on the 256x256x1024 jet, where it
// moves 181 B per node at 5.4 TB/s.
//
// Reduced collision.  With the paper's rates (s0 = s1 = 0, s2b = s3 = s4 = 1)
// the GMRT collision plus forcing, f - T^-1 K T (f - feq) + T^-1 (I - K/2) T F'
// with T = N(u) M, is
//     fdag = feq + F'/2 + (1 - s2nu) T(u)^-1 P T(u) g,   g = f - feq + F'/2,
// where P keeps the five deviatoric second-order central moments.  g has no
// mass and no momentum, so its central second moments are its raw ones, Pi^g.
// T(u)^-1 of a vector of second-order central moments is taken through the
// monomial moments: the central moments kappa_ab of c - u give the raw ones by
// the binomial shift (the 19 monomials x^a y^b z^c with at most two exponents
// nonzero and each <= 2 form a set closed under the shift), and the raw
// monomial moments give the populations in closed form on D3Q19.
//
// Two state forms share one buffer:
//   general  planes of N floats in node order (z ny + y) nx + x: planes 0..18 the
//            colour-blind deviations d_i = f_i - w_i rho_b0
//            after streaming at x, 19..37 the populations of the node's
//            minority colour, 38 its tag (0: red, 1: blue); the majority colour
//            is f_i minus the minority one (written by init and set_state, read
//            by the first step);
//   shifted  rows of the deviations d_i = fdag_i - w_i rho_b0 at the node
//            that produced them, direction i of row r at (r 19 + slot19(i)) rs + x,
//            then the records (x, V_x, V_y, V_z) of the nodes, V = beta (rho_r rho_b / rho)
//            (1 - alpha_bar) grad phi / |grad phi|: the red population pulled
//            from x - c_i is (rho_r / rho) f_i + varphi-weighted c_i . V (Eqs.
//            op3r/op3b), so both colours are rebuilt from 23 floats.  x holds
//            the minority colour's fraction, rho_r / rho with the sign bit clear
//            or -rho_b / rho with it set.
// Both forms keep the minority colour without the cancellation f - f^major:
// its FP32 error inside a phase would leave a noisy grad phi for the
// perturbation to turn into velocity.
#pragma once
#include "lbm_diag.h"
#include "lbm_kernels.h"

namespace cglbm {
namespace q19 {

constexpr int Q19 = 19;  // directions 0..18 of the paper's order: rest, faces, edges
constexpr int GEN_PLANES = 2 * Q19 + 1;

__host__ __device__ constexpr double w19(int i)
{
    return csq(i) == 0 ? 1.0 / 3.0 : csq(i) == 1 ? 1.0 / 18.0 : 1.0 / 36.0;
}

// varphi_i / ((1 - alpha) |c_i|): the recolouring weight of c_i . V
__host__ __device__ constexpr double krec(int i)
{
    return csq(i) == 1 ? 1.0 / 12.0 : 0.029462782549439480;  // 1 / (24 sqrt 2)
}

// byte offset of the records of a shifted form with n = rows x stride nodes
__host__ __device__ inline uint64_t rec_offset(uint64_t n) { return (76ull * n + 255ull) & ~255ull; }

// buffer bytes: the larger of the two forms
__host__ inline uint64_t pop_bytes(uint64_t N)
{
    const uint64_t general = (uint64_t)GEN_PLANES * N * 4ull, shifted = rec_offset(N) + 16ull * N;
    return general > shifted ? general : shifted;
}

// Slot of direction i within its row: the directions of a group (c_y, c_z) follow
// one another in the order of c_x; groups 00, -0, +0, 0-, 0+ of three, then --, +-,
// -+, ++ of one.
__host__ __device__ constexpr int slot19(int i)
{
    const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
    if (cy != 0 && cz != 0) return 15 + (cy > 0 ? 1 : 0) + (cz > 0 ? 2 : 0);
    return (cy < 0 ? 3 : cy > 0 ? 6 : cz < 0 ? 9 : cz > 0 ? 12 : 0) + cx + 1;
}

// the records (x, V) of the shifted form
__device__ __forceinline__ const float4* records(const float* pop, const KP& k)
{
    return (const float4*)((const char*)pop + rec_offset(k.n19));
}

// red part of a population of value f pulled along lattice direction i from a node
// with record r (mirrored at walls)
__device__ __forceinline__ double red_part(const float4& r, int i, double f)
{
    double cv = 0.0;
    if (kCX[i]) cv += kCX[i] * (double)r.y;
    if (kCY[i]) cv += kCY[i] * (double)r.z;
    if (kCZ[i]) cv += kCZ[i] * (double)r.w;
    const double rec = i ? krec(i) * cv : 0.0;
    return signbit(r.x) ? f - (-(double)r.x * f - rec) : (double)r.x * f + rec;
}

// Jet boundaries (Sec. IV A), with the rules the D3Q27 path uses: a circular
// inlet at z = -1/2 whose ghost cells hold the red equilibrium of the inflow
// (with the seeded radial noise of the time level the populations left it),
// half-way free-slip walls at x, y = -1/2, n - 1/2 and z = -1/2 (specular
// reflection: the population of the clamped node with the outside components
// reversed), and the convective outflow of the top plane.

// inlet ghost population of direction i leaving ghost column (xg, yg) at
// post-collision time tg: red equilibrium at rho_r0, alpha_r, Phi = 0
__device__ __forceinline__ double inlet_feq19(const KP& k, int i, int xg, int yg, long long tg)
{
    const uint64_t cnt = ((uint64_t)tg * (uint64_t)k.ny + (uint64_t)yg) * (uint64_t)k.nx + (uint64_t)xg;
    const uint64_t r = splitmix64_nth(k.seed, cnt);
    const double xi = (double)(r >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
    const double ur = (double)k.noise_amp * (double)k.inlet_u * xi;
    const double dx = (double)xg - (double)k.inlet_cx, dy = (double)yg - (double)k.inlet_cy;
    const double rr = sqrt(dx * dx + dy * dy);
    const double ux = rr > 0.0 ? ur * dx / rr : 0.0, uy = rr > 0.0 ? ur * dy / rr : 0.0;
    const double uz = k.inlet_uz ? (double)k.inlet_uz[yg * k.nx + xg] : (double)k.inlet_u;
    const double u2 = ux * ux + uy * uy + uz * uz;
    const double cu = kCX[i] * ux + kCY[i] * uy + kCZ[i] * uz;
    const double poly = cu * (3.0 + 4.5 * cu + 4.5 * cu * cu - 4.5 * u2) - 1.5 * u2;
    const double ph = i == 0 ? (double)k.alpha_r : 1.5 * w19(i) * (1.0 - (double)k.alpha_r);
    return (double)k.rho_r0 * (ph + w19(i) * poly);
}

// The inlet cells of the ghost plane keep their populations in FP64, as the inflow's
// equilibrium is computed: the FP32 slot of a direction that enters the lattice holds
// the rounded value, the slot of its mirror image, which nobody pulls there, the rest.
// Density, fields and state add the rests to what they pull, add(i, rest) on the
// bottom plane above the inlet (a pure red cell: the rest is red, too); the collision
// works on FP32 deviations.  The density pass takes them before its pulls: after them
// it holds 123 registers instead of 52, and the 128x128x512 jet takes 5 % longer.
template <int BC, class A>
__device__ __forceinline__ void inlet_rests(const float* __restrict__ pop, const KP& k, const Node& nd, const A& add)
{
    if (BC != LBM_BC_JET || nd.z != 0) return;
#pragma unroll
    for (int i = 1; i < Q19; ++i) {
        if (kCZ[i] != 1) continue;
        const int x = nd.x - kCX[i], y = nd.y - kCY[i];
        if (inlet_inside(k, x, y))
            add(i, (double)pop[((size_t)row_of(k, y, -1) * Q19 + slot19(mirror_dir(i, 4))) * (uint32_t)k.rs + x]);
    }
}

// Deviation of direction I streamed into node (x, y, z) of the shifted form (offsets
// xo of x; ROW: the row is uniform over the wavefront).  Not for the jet's outlet
// plane, which the convective rule fills.
template <int BC, int I, bool ROW = true>
__device__ __forceinline__ float pull19(const float* __restrict__ pop, const KP& k, int y, int z, const XOff& xo)
{
    constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
    // first of the three slots that the offsets count from
    constexpr int base = slot19(I) - cx - 1, mbase = slot19(mirror_dir(I, 2)) - cx - 1;
    bool my;
    const uint32_t row = group_row<BC, cy, cz>(k, y, z, my), rs = (uint32_t)k.rs;
    return ld_slot<ROW>(pop + (size_t)row * (Q19 * rs) + (uint32_t)(my ? mbase : base) * rs, k,
                        cx > 0 ? xo.p : (cx < 0 ? xo.m : xo.o));
}

template <int BC, bool ROW = true, int I = 0>
__device__ __forceinline__ void pull_all19(const float* __restrict__ pop, const KP& k, int y, int z, const XOff& xo,
                                           float* d)
{
    if constexpr (I < Q19) {
        d[I] = pull19<BC, I, ROW>(pop, k, y, z, xo);
        pull_all19<BC, ROW, I + 1>(pop, k, y, z, xo, d);
    }
}

// general form at the node
__device__ __forceinline__ void general_pop(const float* __restrict__ pop, const KP& k, uint32_t n, int i, double& d,
                                            double& fr)
{
    const size_t N = k.N;
    d = (double)pop[(size_t)i * N + n];
    const double mn = (double)pop[(size_t)(Q19 + i) * N + n];
    const bool blue_min = pop[(size_t)(2 * Q19) * N + n] != 0.f;
    fr = blue_min ? d + w19(i) * k.rho_b0 - mn : mn;
}

// The jet's outlet plane after streaming by the convective rule (Lou et al.):
// f(N, t) = [f(N, t - 1) + lam f(N - 1, t)] / (1 + lam), lam = max(0, u_z(N - 1, t))
// with u_z of the freshly streamed plane below (half-force term included);
// hist holds f(N, t - 1) as (d, fr) planes.  Both colours.
template <bool ROW, int I = 0>
__device__ __forceinline__ void below_dirs(const float* __restrict__ pop, const KP& k, const Node& nd, const XOff& xo,
                                           double (&d)[Q19], double (&fr)[Q19])
{
    if constexpr (I < Q19) {
        int m;
        const float4 r = pull_rec<LBM_BC_JET, I, ROW>(records(pop, k), k, nd.y, k.nz - 2, xo, m);
        d[I] = (double)pull19<LBM_BC_JET, I, ROW>(pop, k, nd.y, k.nz - 2, xo);
        fr[I] = red_part(mirror_rec(r, m), I, d[I] + w19(I) * k.rho_b0);
        below_dirs<ROW, I + 1>(pop, k, nd, xo, d, fr);
    }
}
template <bool ROW>
__device__ __forceinline__ void outlet_rule(const float* __restrict__ pop, const float* __restrict__ hist,
                                            const KP& k, const Node& nd, double (&d)[Q19], double (&fr)[Q19])
{
    below_dirs<ROW>(pop, k, nd, x_offsets<LBM_BC_JET, float>(k, nd.x), d, fr);
    double m = 0.0, jz = 0.0;
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        m += d[i];
        if (kCZ[i]) jz += kCZ[i] * d[i];
    }
    const double uz = (jz + 0.5 * m * k.gz) / (k.rho_b0 + m);
    const double lam = uz > 0.0 ? uz : 0.0, il = 1.0 / (1.0 + lam);
    const size_t P = k.plane;
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        d[i] = ((double)hist[(size_t)i * P + nd.q] + lam * d[i]) * il;
        fr[i] = ((double)hist[(size_t)(Q19 + i) * P + nd.q] + lam * fr[i]) * il;
    }
}

// the records of a tile and its rim into LDS
template <int BC, int TX, int TY>
__device__ __forceinline__ void stage_records19(const float* __restrict__ pop, const KP& k, const Tile& t,
                                                float4* __restrict__ win)
{
    const float4* R = records(pop, k);
    stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return rec_at<BC, true>(k, R, x, y, z); },
                         [&](int x, int y, int z) { return rec_at<BC>(k, R, x, y, z); },
                         [&](int w, const float4& v) { win[w] = v; });
}

// node order index
__device__ __forceinline__ uint32_t order_of(const KP& k, const Node& nd) { return (uint32_t)nd.z * k.plane + nd.q; }

// record of the source of direction I: from the window, or (NodeBlocks) through the caches
template <int BC, class TL, int TX, int TY, int I>
__device__ __forceinline__ float4 source_rec19(const float* __restrict__ pop, const KP& k, const Tile& t,
                                               const XOff& xo, const float4* __restrict__ win)
{
    if constexpr (TL::kFlat) {
        int m;
        const float4 r = pull_rec<BC, I, false>(records(pop, k), k, t.nd.y, t.nd.z, xo, m);
        return BC == LBM_BC_JET ? mirror_rec(r, m) : r;
    } else {
        return win[wslot<TX, TY>(t.lx, t.ly, -kCX[I], -kCY[I], -kCZ[I])];
    }
}

// the tile of this block with the records of its nodes and rim in the window
// (shifted form), or (NodeBlocks) this thread's node
template <bool GEN, int BC, class TL>
__device__ __forceinline__ Tile state_tile19(const float* __restrict__ pop, const KP& k, float4* __restrict__ win)
{
    if constexpr (TL::kFlat) {
        Tile t{};
        t.nd = this_node(k);
        t.z = t.nd.z;
        return t;
    } else {
        const Tile t = this_tile<TL::CX, TL::CY>(k);
        if (!GEN) {
            stage_records19<BC, TL::CX, TL::CY>(pop, k, t, win);
            __syncthreads();
        }
        return t;
    }
}

// The state at a node: the populations after streaming, (d_i, fr_i), of either form;
// the jet's outlet plane from the general form, or by the rule.
template <int BC, class TL, int I = 0>
__device__ __forceinline__ void state_dirs19(const float* __restrict__ pop, const KP& k, const Tile& t, const XOff& xo,
                                             const float4* __restrict__ win, double (&d)[Q19], double (&fr)[Q19])
{
    if constexpr (I < Q19) {
        d[I] = (double)pull19<BC, I, !TL::kFlat>(pop, k, t.nd.y, t.nd.z, xo);
        fr[I] = red_part(source_rec19<BC, TL, TL::CX, TL::CY, I>(pop, k, t, xo, win), I, d[I] + w19(I) * k.rho_b0);
        state_dirs19<BC, TL, I + 1>(pop, k, t, xo, win, d, fr);
    }
}
template <bool GEN, int BC, class TL>
__device__ __forceinline__ void node_state(const float* __restrict__ pop, const float* __restrict__ hist, const KP& k,
                                           const Tile& t, const float4* __restrict__ win, double (&d)[Q19],
                                           double (&fr)[Q19])
{
    if (GEN) {
#pragma unroll
        for (int i = 0; i < Q19; ++i) general_pop(pop, k, order_of(k, t.nd), i, d[i], fr[i]);
    } else if (BC == LBM_BC_JET && t.nd.z == k.nz - 1) {
        outlet_rule<!TL::kFlat>(pop, hist, k, t.nd, d, fr);
    } else {
        state_dirs19<BC, TL>(pop, k, t, x_offsets<BC, float>(k, t.nd.x), win, d, fr);
        inlet_rests<BC>(pop, k, t.nd, [&](int i, double e) {
            d[i] += e;
            fr[i] += e;
        });
    }
}

// Per-node fields F (field buffer, two float2 arrays): F[n] = (phi, rho - rho_b0),
// which the collision gathers from the 18 neighbours, and F[N + n] =
// (rho_r, rho_b), which it reads at the node only.
__device__ __forceinline__ void store_fields(float2* __restrict__ F, const KP& k, uint32_t n, double rr, double rb,
                                             double m)
{
    // both quotients scaled by rho_r0 rho_b0: one division
    const double a = rr * (double)k.rho_b0, b = rb * (double)k.rho_r0;
    stp(F, n, make_float2((float)div_fields(a - b, a + b), (float)m));
    stp(F + k.N, n, make_float2((float)rr, (float)rb));
}

template <int BC, class TL, int I = 0>
__device__ __forceinline__ void density_dirs(const float* __restrict__ pop, const float* d, const KP& k, const Tile& t,
                                             const XOff& xo, const float4* __restrict__ win, double& rr, double& rb,
                                             double& m)
{
    if constexpr (I < Q19) {
        const double f = (double)d[I] + w19(I) * k.rho_b0;
        const double fr = red_part(source_rec19<BC, TL, TL::DX, TL::DY, I>(pop, k, t, xo, win), I, f);
        m += (double)d[I];
        rr += fr;
        rb += f - fr;
        density_dirs<BC, TL, I + 1>(pop, d, k, t, xo, win, rr, rb, m);
    }
}

// Density pass (Eq. order): the fields F of every node, on the
// planes below the jet's outlet (all planes when periodic).
template <bool GEN, int BC, class TL>
__global__ __launch_bounds__(TL::DX* TL::DY) void k19_density(const float* __restrict__ pop, float2* __restrict__ F,
                                                              KP k)
{
    constexpr int TX = TL::DX, TY = TL::DY;
    __shared__ float4 win[GEN || TL::kFlat ? 1 : TileShape<TX, TY>::W];
    Tile t{};
    if constexpr (TL::kFlat) {
        t.nd = this_node(k);
    } else {
        t = this_tile<TX, TY>(k);
        if (!GEN) {
            stage_records19<BC, TX, TY>(pop, k, t, win);
            __syncthreads();
        }
    }
    double rr = 0.0, rb = 0.0, m = 0.0;
    if (!t.nd.valid) return;
    if (GEN) {
#pragma unroll
        for (int i = 0; i < Q19; ++i) {
            double d, fr;
            general_pop(pop, k, order_of(k, t.nd), i, d, fr);
            m += d;
            rr += fr;
            rb += d + w19(i) * k.rho_b0 - fr;
        }
    } else {
        inlet_rests<BC>(pop, k, t.nd, [&](int, double e) { m += e; });
        rr = m;
        float d[Q19];
        const XOff xo = x_offsets<BC, float>(k, t.nd.x);
        pull_all19<BC, !TL::kFlat>(pop, k, t.nd.y, t.nd.z, xo, d);
        density_dirs<BC, TL>(pop, d, k, t, xo, win, rr, rb, m);
    }
    store_fields(F, k, order_of(k, t.nd), rr, rb, m);
}

// The jet's outlet plane (grid: row segments of OBLOCK nodes): its populations after
// streaming (general form, or the convective rule from hprev) go to hcur as
// (d, fr), where the collision and the next step's rule read them, and its
// fields to F.  Also the inlet cells of the ghost plane of the state that the step
// writes (the red equilibrium at this time level, see inlet_rests, and a pure red
// record).
template <bool GEN>
__global__ __launch_bounds__(OBLOCK) void k19_outlet(const float* __restrict__ pop, float2* __restrict__ F,
                                                     const float* __restrict__ hprev, float* __restrict__ hcur,
                                                     float* __restrict__ dst, KP k)
{
    Node nd;
    nd.x = (int)(blockIdx.x * OBLOCK + threadIdx.x);
    nd.y = (int)blockIdx.y;
    nd.z = k.nz - 1;
    if (nd.x >= k.nx) return;
    nd.q = (uint32_t)nd.y * (uint32_t)k.nx + (uint32_t)nd.x;
    double d[Q19], fr[Q19];
    if (GEN) {
#pragma unroll
        for (int i = 0; i < Q19; ++i) general_pop(pop, k, order_of(k, nd), i, d[i], fr[i]);
    } else {
        outlet_rule<true>(pop, hprev, k, nd, d, fr);
    }
    double rr = 0.0, rb = 0.0, m = 0.0;
    const size_t P = k.plane;
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        m += d[i];
        rr += fr[i];
        rb += d[i] + w19(i) * k.rho_b0 - fr[i];
        hcur[(size_t)i * P + nd.q] = (float)d[i];
        hcur[(size_t)(Q19 + i) * P + nd.q] = (float)fr[i];
    }
    store_fields(F, k, order_of(k, nd), rr, rb, m);
    if (inlet_inside(k, nd.x, nd.y)) {
        const uint32_t row = row_of(k, nd.y, -1), rs = (uint32_t)k.rs;
#pragma unroll
        for (int i = 1; i < Q19; ++i) {
            if (kCZ[i] != 1) continue;
            float* cell = dst + (size_t)row * (Q19 * rs) + nd.x;
            const double v = inlet_feq19(k, i, nd.x, nd.y, k.t) - w19(i) * k.rho_b0;
            cell[(uint32_t)slot19(i) * rs] = (float)v;
            cell[(uint32_t)slot19(mirror_dir(i, 4)) * rs] = (float)(v - (double)(float)v);
        }
        const_cast<float4*>(records(dst, k))[(size_t)row * rs + nd.x] = make_float4(-0.f, 0.f, 0.f, 0.f);
    }
}

// (phi, rho - rho_b0) at (x, y, z), which may lie one node outside: periodic wrap, or
// (jet) (1, rho_r0 - rho_b0) in the inlet circle at z = -1 and the clamped
// node elsewhere outside (the mirrored field of the half-way walls and outlet).
// XIN: x lies inside.
template <int BC, bool XIN = false>
__device__ __forceinline__ float2 field_at(const float2* __restrict__ F, const KP& k, int x, int y, int z)
{
    const bool in = BC == LBM_BC_JET && z < 0 && inlet_inside(k, x, y);
    x = XIN ? x : BC == LBM_BC_PERIODIC ? wrapc(x, k.nx) : clampc(x, k.nx);
    y = BC == LBM_BC_PERIODIC ? wrapc(y, k.ny) : clampc(y, k.ny);
    z = BC == LBM_BC_PERIODIC ? wrapc(z, k.nz) : clampc(z, k.nz);
    const float2 v = ldp(F, ((uint32_t)z * (uint32_t)k.ny + (uint32_t)y) * (uint32_t)k.nx + (uint32_t)x);
    return in ? make_float2(1.f, k.rho_r0 - k.rho_b0) : v;
}

// isotropic gradients of phi and rho, 3 sum_i w_i chi(x + c_i) c_i, summed
// over the opposite pairs (i, i + 1) as differences: exactly zero on a
// uniform field, which keeps the recolouring off there
// at(dx, dy, dz): (phi, rho - rho_b0) of the neighbour
template <int I = 1, class A>
__device__ __forceinline__ void gradients(const A& at, double& gpx, double& gpy, double& gpz, double& grx, double& gry,
                                          double& grz)
{
    if constexpr (I < Q19) {
        const float2 qp = at(kCX[I], kCY[I], kCZ[I]);
        const float2 qm = at(-kCX[I], -kCY[I], -kCZ[I]);
        const double tp = 3.0 * w19(I) * ((double)qp.x - (double)qm.x);
        const double tr = 3.0 * w19(I) * ((double)qp.y - (double)qm.y);
        if (kCX[I]) { gpx += kCX[I] * tp; grx += kCX[I] * tr; }
        if (kCY[I]) { gpy += kCY[I] * tp; gry += kCY[I] * tr; }
        if (kCZ[I]) { gpz += kCZ[I] * tp; grz += kCZ[I] * tr; }
        gradients<I + 2>(at, gpx, gpy, gpz, grx, gry, grz);
    }
}

// 1/sqrt(a) of a positive normal number: the hardware estimate and two Newton steps,
// a few FP64 ulps
__device__ __forceinline__ double inv_sqrt(double a)
{
    double r = __builtin_amdgcn_rsq(a);
    r = fma(0.5 * r, fma(-a * r, r, 1.0), r);
    return fma(0.5 * r, fma(-a * r, r, 1.0), r);
}

// the model's parameters as the kernels' FP64 arithmetic takes them (FP32 values:
// converted once on the host instead of by every wavefront)
struct Consts {
    double rho_b0, alpha_b, dalpha, a_minus_w0, inv_nu_r, inv_nu_b, A, beta, eps2, g[3];
};
inline Consts consts_of(const KP& k)
{
    return Consts{k.rho_b0, k.alpha_b, k.dalpha, k.a_minus_w0, k.inv_nu_r, k.inv_nu_b, k.A, k.beta, k.eps2,
                  {k.gx, k.gy, k.gz}};
}

// Collision, perturbation, recolouring and the store of the shifted form at the
// node itself (the next step pulls from it), Sec. II: Eqs. Momentum to op3b.
template <bool GEN, int BC, class TL, bool NT>
__global__ __launch_bounds__(BLOCK) void k19_collide(const float* __restrict__ src, float* __restrict__ dst,
                                                     const float2* __restrict__ F, const float* __restrict__ hcur,
                                                     KP k, Consts c)
{
    constexpr int TX = TL::CX, TY = TL::CY;
    constexpr bool FLAT = TL::kFlat;
    __shared__ float2 win[FLAT ? 1 : TileShape<TX, TY>::W];
    Tile t{};
    if constexpr (FLAT) {
        t.nd = this_node(k);
    } else {
        t = this_tile<TX, TY>(k);
        stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return field_at<BC, true>(F, k, x, y, z); },
                             [&](int x, int y, int z) { return field_at<BC>(F, k, x, y, z); },
                             [&](int w, const float2& v) { win[w] = v; });
        __syncthreads();
    }
    const Node& nd = t.nd;
    if (!nd.valid) return;
    const size_t N = k.N;
    float d[Q19];
    if (BC == LBM_BC_JET && nd.z == k.nz - 1) {  // the outlet plane: its kernel wrote it to hcur
#pragma unroll
        for (int i = 0; i < Q19; ++i) d[i] = hcur[(size_t)i * k.plane + nd.q];
    } else if (GEN) {
#pragma unroll
        for (int i = 0; i < Q19; ++i) d[i] = src[(size_t)i * N + order_of(k, nd)];
    } else {
        pull_all19<BC, !FLAT>(src, k, nd.y, nd.z, x_offsets<BC, float>(k, nd.x), d);
    }
    const auto at = [&](int dx, int dy, int dz) -> float2 {
        if constexpr (FLAT)
            return field_at<BC>(F, k, nd.x + dx, nd.y + dy, nd.z + dz);
        else
            return win[wslot<TX, TY>(t.lx, t.ly, dx, dy, dz)];
    };
    const float2 P = at(0, 0, 0), Q = ldp(F + k.N, order_of(k, nd));
    const double phi = P.x, m = P.y, rr = Q.x, rb = Q.y;
    double gpx = 0, gpy = 0, gpz = 0, grx = 0, gry = 0, grz = 0;
    gradients(at, gpx, gpy, gpz, grx, gry, grz);
    // interpolated properties, body force, velocity (Eqs. bodyForceJet, Momentum)
    const double rho = c.rho_b0 + m;
    const double hp = 0.5 * (1.0 + phi);
    const double ab = c.alpha_b + hp * c.dalpha;
    const double amw = c.a_minus_w0 + hp * c.dalpha;  // alpha_bar - 1/3
    const double nub = div_fields(1.0, hp * c.inv_nu_r + (1.0 - hp) * c.inv_nu_b);
    const double s2 = div_fields(1.0, 3.0 * nub + 0.5);
    const double Fx = m * c.g[0], Fy = m * c.g[1], Fz = m * c.g[2];
    // momentum and second moments of d over opposite pairs (i, i + 1)
    double jx = 0, jy = 0, jz = 0, pxx = 0, pyy = 0, pzz = 0, pxy = 0, pxz = 0, pyz = 0;
#pragma unroll
    for (int i = 1; i < Q19; i += 2) {
        const double sp = (double)d[i] + (double)d[i + 1], df = (double)d[i] - (double)d[i + 1];
        if (kCX[i]) { jx += kCX[i] * df; pxx += sp; }
        if (kCY[i]) { jy += kCY[i] * df; pyy += sp; }
        if (kCZ[i]) { jz += kCZ[i] * df; pzz += sp; }
        if (kCX[i] * kCY[i]) pxy += (kCX[i] * kCY[i]) * sp;
        if (kCX[i] * kCZ[i]) pxz += (kCX[i] * kCZ[i]) * sp;
        if (kCY[i] * kCZ[i]) pyz += (kCY[i] * kCZ[i]) * sp;
    }
    const double irho = div_fields(1.0, rho);
    const double ux = (jx + 0.5 * Fx) * irho, uy = (jy + 0.5 * Fy) * irho, uz = (jz + 0.5 * Fz) * irho;
    const double u2 = ux * ux + uy * uy + uz * uz;
    const double udr = ux * grx + uy * gry + uz * grz;
    const double uF = ux * Fx + uy * Fy + uz * Fz;
    const double kap = 1.5 * (1.0 - ab) * m - 1.5 * amw * c.rho_b0;  // 1.5 (1 - ab) rho - rho_b0
    // Pi^g of g = f - feq + F'/2 from closed forms of the moments of feq and F'
    // (both lattices' coefficients give them): sum feq c c = rho [(1 - ab)/2 I
    // + u u] + nu_bar [u grad rho + grad rho u + (u . grad rho) I] (Eqs. EES,
    // Phi), sum F' c c = u F + F u (Eq. ketFd), sum w_i rho_b0 c c = rho_b0/3 I.
    // Only the deviatoric part is used, so the isotropic terms are left out:
    // dev Pi^g = dev [sum d c c - rho u u - nu_bar (u grad rho + grad rho u)
    //                 + (u F + F u)/2]
    pxx += -rho * ux * ux - 2.0 * nub * ux * grx + ux * Fx;
    pyy += -rho * uy * uy - 2.0 * nub * uy * gry + uy * Fy;
    pzz += -rho * uz * uz - 2.0 * nub * uz * grz + uz * Fz;
    pxy += -rho * ux * uy - nub * (ux * gry + uy * grx) + 0.5 * (ux * Fy + uy * Fx);
    pxz += -rho * ux * uz - nub * (ux * grz + uz * grx) + 0.5 * (ux * Fz + uz * Fx);
    pyz += -rho * uy * uz - nub * (uy * grz + uz * gry) + 0.5 * (uy * Fz + uz * Fy);
    // (1 - s2nu) times the deviatoric central second moments
    const double om = 1.0 - s2, tr3 = (pxx + pyy + pzz) * (1.0 / 3.0);
    const double k200 = om * (pxx - tr3), k020 = om * (pyy - tr3), k002 = om * (pzz - tr3);
    const double k110 = om * pxy, k101 = om * pxz, k011 = om * pyz;
    // raw monomial moments of h = T(u)^-1 of them (binomial shift)
    const double m210 = uy * k200 + 2.0 * ux * k110, m120 = ux * k020 + 2.0 * uy * k110;
    const double m201 = uz * k200 + 2.0 * ux * k101, m102 = ux * k002 + 2.0 * uz * k101;
    const double m021 = uz * k020 + 2.0 * uy * k011, m012 = uy * k002 + 2.0 * uz * k011;
    const double m220 = uy * uy * k200 + ux * ux * k020 + 4.0 * ux * uy * k110;
    const double m202 = uz * uz * k200 + ux * ux * k002 + 4.0 * ux * uz * k101;
    const double m022 = uz * uz * k020 + uy * uy * k002 + 4.0 * uy * uz * k011;
    // perturbation (Eq. perturb, Eq. B_i) and recolouring record (Eqs. op3r/op3b)
    const double G2 = gpx * gpx + gpy * gpy + gpz * gpz;
    const bool on = G2 > c.eps2;
    const double ign = on ? inv_sqrt(G2) : 0.0;
    const double Agn = c.A * G2 * ign, Aign = c.A * ign;  // A |grad phi|, A / |grad phi|
    const double irc = div_fields(1.0, rr + rb);
    const double vs = c.beta * rr * rb * irc * (1.0 - ab) * ign;
    // jet, bottom plane: the ghost cell below mirrors this node outside the inlet
    const uint32_t row = row_of(k, nd.y, nd.z), rsB = 4u * (uint32_t)k.rs, xB = 4u * (uint32_t)nd.x;
    const bool bottom = BC == LBM_BC_JET && nd.z == 0;
    const bool gcell = bottom && !inlet_inside(k, nd.x, nd.y);
    const uint32_t grow = BC == LBM_BC_JET ? row_of(k, nd.y, -1) : 0u;
    const auto put = [&](uint32_t r, int slot, float v) {
        float* b = dst + (size_t)r * (uint32_t)(Q19 * k.rs);
        if constexpr (!FLAT)
            st_row<NT>(row_rsrc(b, (uint32_t)(Q19 * k.rs)), xB, (uint32_t)slot * rsB, v);
        else if constexpr (NT)
            __builtin_nontemporal_store(v, b + (uint32_t)slot * (uint32_t)k.rs + nd.x);
        else
            b[(uint32_t)slot * (uint32_t)k.rs + nd.x] = v;
    };
    const auto store = [&](int i, double f) {
        const float v = (float)f;
        put(row, slot19(i), v);
        if (BC == LBM_BC_JET && kCZ[i] < 0 && bottom) {  // uniform: leaves downwards
            if (gcell) put(grow, slot19(mirror_dir(i, 4)), v);
        }
    };
    // rest population
    store(0, rho * amw + m * (1.0 / 3.0) - 0.5 * rho * u2 - 3.0 * nub * udr - 0.5 * uF + Agn * (1.0 / 3.0) +
                 (m220 + m202 + m022) - (k200 + k020 + k002));
    // Opposite pairs: with m_i / 4 = 9 w_i the terms of feq, F'/2 and the perturbation
    // share one factor w_i,
    //   even = kappa' - 1.5 rho u^2 - 1.5 u.F - A |g| + cu (4.5 rho cu + 9 nu cr + 4.5 cF) + A/|g| cg^2,
    //   odd  = cu (rho (3 - 4.5 u^2) + 4.5 rho cu^2) + 1.5 cF
    // (cu = c.u, cr = c.grad rho, cF = c.F, cg = c.grad phi); h, the part of the
    // relaxed moments, splits the same way.
    const double K0 = kap - 1.5 * rho * u2 - 1.5 * uF - Agn, K1 = rho * (3.0 - 4.5 * u2), r45 = 4.5 * rho;
    const double nub9 = 9.0 * nub;
    // 9 nu grad rho + 4.5 F and 1.5 F
    const double qx = nub9 * grx + 4.5 * Fx, qy = nub9 * gry + 4.5 * Fy, qz = nub9 * grz + 4.5 * Fz;
    const double sx = 1.5 * Fx, sy = 1.5 * Fy, sz = 1.5 * Fz;
#pragma unroll
    for (int i = 1; i < Q19; i += 2) {
        const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
        double he, ho;
        if (cx && cy) {
            he = 0.25 * (m220 + (cx * cy) * k110);
            ho = 0.25 * (cx * m120 + cy * m210);
        } else if (cx && cz) {
            he = 0.25 * (m202 + (cx * cz) * k101);
            ho = 0.25 * (cx * m102 + cz * m201);
        } else if (cy && cz) {
            he = 0.25 * (m022 + (cy * cz) * k011);
            ho = 0.25 * (cy * m012 + cz * m021);
        } else if (cx) {
            he = 0.5 * (k200 - m220 - m202);
            ho = -0.5 * cx * (m120 + m102);
        } else if (cy) {
            he = 0.5 * (k020 - m220 - m022);
            ho = -0.5 * cy * (m210 + m012);
        } else {
            he = 0.5 * (k002 - m202 - m022);
            ho = -0.5 * cz * (m201 + m021);
        }
        const double cu = cdot(i, ux, uy, uz), cg = cdot(i, gpx, gpy, gpz);
        const double v = r45 * cu;
        const double even = he + w19(i) * (K0 + cu * (v + cdot(i, qx, qy, qz)) + (Aign * cg) * cg);
        const double odd = ho + w19(i) * (cu * (K1 + v * cu) + cdot(i, sx, sy, sz));
        store(i, even + odd);
        store(i + 1, even - odd);
    }
    // minority fraction: rho_r / rho, or -rho_b / rho (sign bit set, also for 0)
    const float xm = rr <= rb ? (float)(rr * irc) : -(float)(rb * irc);
    const float4 rv = make_float4(xm, (float)(vs * gpx), (float)(vs * gpy), (float)(vs * gpz));
    float4* R = const_cast<float4*>(records(dst, k));
    if constexpr (FLAT) {
        R[(size_t)row * (uint32_t)k.rs + nd.x] = rv;
        if (gcell) R[(size_t)grow * (uint32_t)k.rs + nd.x] = mirror_rec(rv, 4);
    } else {
        st_rec(R, k, row, nd.x, rv);
        if (gcell) st_rec(R, k, grow, nd.x, mirror_rec(rv, 4));
    }
}

// Macroscopic fields (node order) and FP64 audit partial sums, one slot per block.
template <bool GEN, int BC, class TL>
__global__ __launch_bounds__(BLOCK) void k19_macro(const float* __restrict__ pop, const float* __restrict__ hist, KP k,
                                                   float* __restrict__ o_rr, float* __restrict__ o_rb,
                                                   float* __restrict__ o_u, float* __restrict__ o_phi,
                                                   double* __restrict__ partials)
{
    __shared__ float4 win[GEN ? 1 : kRecWin<TL>];
    const Tile t = state_tile19<GEN, BC, TL>(pop, k, win);
    double acc[5] = {0, 0, 0, 0, 0};
    if (t.nd.valid) {
        double d[Q19], fv[Q19];
        node_state<GEN, BC, TL>(pop, hist, k, t, win, d, fv);
        double m0 = 0.0, rr = 0.0, rb = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
        for (int i = 0; i < Q19; ++i) {
            m0 += d[i];
            rr += fv[i];
            rb += d[i] + w19(i) * k.rho_b0 - fv[i];
            if (kCX[i]) jx += kCX[i] * d[i];
            if (kCY[i]) jy += kCY[i] * d[i];
            if (kCZ[i]) jz += kCZ[i] * d[i];
        }
        const double rho = (double)k.rho_b0 + m0;
        const double px = jx + 0.5 * m0 * k.gx, py = jy + 0.5 * m0 * k.gy, pz = jz + 0.5 * m0 * k.gz;
        const size_t n = order_of(k, t.nd);
        if (o_rr) o_rr[n] = (float)rr;
        if (o_rb) o_rb[n] = (float)rb;
        if (o_u) {
            o_u[3 * n] = (float)(px / rho);
            o_u[3 * n + 1] = (float)(py / rho);
            o_u[3 * n + 2] = (float)(pz / rho);
        }
        if (o_phi) {
            const double a = rr / k.rho_r0, b = rb / k.rho_b0;
            o_phi[n] = (float)((a - b) / (a + b));
        }
        acc[0] = rr;
        acc[1] = rb;
        acc[2] = px;
        acc[3] = py;
        acc[4] = pz;
    }
    if (partials) block_partials<5>(acc, partials, blockIdx.y * gridDim.x + blockIdx.x);
}

// the state fr[i N + n], fb[(19 + i) N + n] of either form
template <bool GEN, int BC, class TL>
__global__ __launch_bounds__(BLOCK) void k19_get_state(const float* __restrict__ pop, const float* __restrict__ hist,
                                                       KP k, float* __restrict__ st)
{
    __shared__ float4 win[GEN ? 1 : kRecWin<TL>];
    const Tile t = state_tile19<GEN, BC, TL>(pop, k, win);
    if (!t.nd.valid) return;
    const size_t N = k.N, n = order_of(k, t.nd);
    double d[Q19], fr[Q19];
    node_state<GEN, BC, TL>(pop, hist, k, t, win, d, fr);
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        st[(size_t)i * N + n] = (float)fr[i];
        st[(size_t)(Q19 + i) * N + n] = (float)(d[i] + w19(i) * k.rho_b0 - fr[i]);
    }
}

// Jet diagnostics (Sec. IV C), first pass on D3Q19: the order parameter of the
// current state binarised (phi as lbm_macroscopic returns it) and labels; the
// union-find passes that follow are those of the D3Q27 path.
template <bool GEN, int BC, class TL>
__global__ __launch_bounds__(BLOCK) void k19_diag_init(const float* __restrict__ pop, const float* __restrict__ hist,
                                                       KP k, DiagWork w)
{
    __shared__ float4 win[GEN ? 1 : kRecWin<TL>];
    const Tile t = state_tile19<GEN, BC, TL>(pop, k, win);
    bool fg = false;
    if (t.nd.valid) {
        double d[Q19], fr[Q19];
        node_state<GEN, BC, TL>(pop, hist, k, t, win, d, fr);
        double rr = 0.0, rb = 0.0;
#pragma unroll
        for (int i = 0; i < Q19; ++i) {
            rr += fr[i];
            rb += d[i] + w19(i) * k.rho_b0 - fr[i];
        }
        const double a = rr / k.rho_r0, b = rb / k.rho_b0;
        fg = (float)((a - b) / (a + b)) > 0.f;
    }
    const unsigned long long m = __ballot(fg);
    const int i = (int)order_of(k, t.nd), run = TL::kFlat ? i : diag_run_label(m, i);
    if (t.nd.valid) w.label[i] = fg ? run : -1;
    diag_tally(w, m, fg ? t.nd.z : -1);
}

// general form of one node from FP64 colour populations: the deviations rounded
// once, the minority colour kept as given
__device__ __forceinline__ void put_general(float* __restrict__ dst, const KP& k, uint32_t n, const double (&fr)[Q19],
                                            const double (&fb)[Q19])
{
    const size_t N = k.N;
    double rr = 0.0, rb = 0.0;
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        rr += fr[i];
        rb += fb[i];
    }
    const bool blue_min = rr > rb;
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        dst[(size_t)i * N + n] = (float)(fr[i] + fb[i] - w19(i) * k.rho_b0);
        dst[(size_t)(Q19 + i) * N + n] = (float)(blue_min ? fb[i] : fr[i]);
    }
    dst[(size_t)(2 * Q19) * N + n] = blue_min ? 1.f : 0.f;
}

// a caller state (lbm_get_state layout) into the general form
__global__ __launch_bounds__(BLOCK) void k19_set_state(float* __restrict__ dst, KP k, const float* __restrict__ st)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const size_t N = k.N, n = order_of(k, nd);
    double fr[Q19], fb[Q19];
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        fr[i] = st[(size_t)i * N + n];
        fb[i] = st[(size_t)(Q19 + i) * N + n];
    }
    put_general(dst, k, (uint32_t)n, fr, fb);
}

// Initial state (general form): per-colour equilibria rho_k {varphi_i(alpha_k) +
// w_i [velocity terms of Eq. EES]} of the droplet preset or of caller fields,
// in FP64.
__global__ __launch_bounds__(BLOCK) void k19_init(float* __restrict__ dst, KP k, int kind,
                                                  const float* __restrict__ frr, const float* __restrict__ frb,
                                                  const float* __restrict__ fu, double dcx, double dcy, double dcz,
                                                  double R, double W, double rho_r0, double rho_b0, double alpha_r,
                                                  double alpha_b)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const uint32_t n = order_of(k, nd);
    double rr, rb, ux = 0, uy = 0, uz = 0;
    if (kind == LBM_INIT_DROPLET) {
        const double dx = nd.x - dcx, dy = nd.y - dcy, dz = nd.z - dcz;
        const double th = tanh(2.0 * (sqrt(dx * dx + dy * dy + dz * dz) - R) / W);
        rr = 0.5 * rho_r0 * (1.0 - th);
        rb = 0.5 * rho_b0 * (1.0 + th);
    } else if (kind == LBM_INIT_JET) {
        rr = 0.0;
        rb = rho_b0;
    } else {
        rr = frr[n];
        rb = frb[n];
        if (fu) {
            ux = fu[3 * (size_t)n];
            uy = fu[3 * (size_t)n + 1];
            uz = fu[3 * (size_t)n + 2];
        }
    }
    const double u2 = ux * ux + uy * uy + uz * uz;
    double fr[Q19], fb[Q19];
#pragma unroll
    for (int i = 0; i < Q19; ++i) {
        const double cu = kCX[i] * ux + kCY[i] * uy + kCZ[i] * uz;
        const double wp = w19(i) * (3.0 * cu + 4.5 * cu * cu - 1.5 * u2 + 4.5 * cu * cu * cu - 4.5 * cu * u2);
        const double phr = i == 0 ? alpha_r : 1.5 * w19(i) * (1.0 - alpha_r);
        const double phb = i == 0 ? alpha_b : 1.5 * w19(i) * (1.0 - alpha_b);
        fr[i] = rr * (phr + wp);
        fb[i] = rb * (phb + wp);
    }
    put_general(dst, k, n, fr, fb);
}

}  // namespace q19
}  // namespace cglbm
