// HIP kernels of the colour-gradient D3Q27 central-moment LBM step for gfx950.
//
// Design (one MI355X, one process):
//  * Rows: a row is the nx nodes (y, z), stored with stride rs >= nx elements;
//    rs is nx rounded up to the widest alignment (a cache line, if it fits) that
//    the buffers hold.  Row r = (z + zg) ny + y; node index n = r rs + x for the
//    per-node arrays.  There are no ghost cells along x and y and, on periodic
//    lattices, none along z: a wavefront works inside one row, so the row that a
//    direction is pulled from is a scalar, wrapped or mirrored with scalar
//    selects, and the two lanes at the ends of the row take their offset by one
//    select shared by all directions.  The jet keeps one ghost plane z = -1
//    (zg = 1): the mirrored bottom plane, and the inlet equilibria inside the
//    inlet circle.
//  * Populations: A-B buffers; the 27 directions of a row follow one another,
//    slot s = 9 (c_z + 1) + 3 (c_y + 1) + (c_x + 1) of row r at (r 27 + s) rs + x.
//    Mirroring a velocity on an axis moves its slot by a constant (2, 6, 18), so
//    that a free-slip wall costs no more than a periodic one.  What bounds the
//    step is this traffic, and aligned rows without x ghosts carry it faster: a
//    probe of 27 shifted reads and 27 writes per node on 256x256x512 nodes ran
//    1.90 ms with padded plane-major rows, 1.48 ms with aligned plane-major rows,
//    1.45 ms with aligned interleaved rows.
//    The slots hold the colour-blind deviation d_i = f_i - w_i rho_b0; d is
//    small in both pure phases (rho_r0 varphi_i(alpha_r) = rho_b0 w_i for
//    |c_i| >= 1 because gamma = (1 - alpha_b)/(1 - alpha_r)), so FP32 and
//    16-bit storage keep the momentum sum_i d_i c_i well conditioned.
//  * Colour populations: after recolouring (Eqs. op3r/op3b) with
//    varphi_i = w_i kappa(alpha_bar) for |c_i| >= 1 and cos(theta_i) linear in
//    c_i, the post-collision populations of either colour are
//        f^r*_i = x_r f'_i + (w_i / |c_i|) c_i . V,   f^b*_i = x_b f'_i - (same),
//        x_k = rho_k/rho,  V = beta (rho_r rho_b / rho) kappa grad phi / |grad phi|,
//    affine functions of the colour-blind post-collision f' with four
//    per-node scalars.  The fused kernel therefore stores only d' and the
//    float4 R = (x*, V) of every node, x* the fraction of the kept colour
//    (the one of smaller reference density, see kept_sgn); readers rebuild
//    f^* of direction i at x from d_i and R at the source node x - c_i, and
//    the other colour as f - f^*.  A general state (after initialisation or
//    set_state) is kept on a padded lattice in 54 planes at the node itself
//    ("unshifted": deviations, then the kept colour's populations) and is read
//    that way by the first step.
//  * A step: density pass (phi, rho - rho_b0, x* per node), then the fused
//    collide-perturb-recolour-stream kernel (reads 27 deviations and the
//    (phi, rho) stencil, writes 27 deviations and R).  The jet's outlet plane
//    z = nz - 1 (convective condition) and the inlet cells of the ghost plane
//    have a small kernel of their own before them; the fused kernel writes the
//    mirrored part of the ghost plane.
//  * Launch geometry: see "stencil tiles"; a wavefront takes 64 consecutive nodes of
//    one row, but for the kernels that take blocks of nodes on narrow rows
//    (NodeBlocks) and the ones that only write the general form.
//  * Collision: with s0 = s1 = 0 and s2b = s3..s6 = 1 (Sec. II) the GMRT
//    collision (Eq. scoll) leaves every central moment at its equilibrium
//    value plus half the forcing moment, except the five deviatoric second-
//    order moments, which relax with s2nu.  The kernel therefore needs only
//    the raw moments of d up to second order, uses the closed-form moments of
//    f^(e) and F' (Eq. EES with Eq. Phi; Eq. ketFd) and maps the relaxed
//    deviatoric central moments back to populations through the tensor-product
//    inverse of the one-dimensional central-moment transform.  This equals
//    f^(e) + F'/2 + (1 - s2nu) T(u)^-1 P T(u) (f - f^(e) + F'/2), P the
//    projector on rows 4..8 of Eq. momentSet.
#pragma once
#include "lbm_lattice.h"

#include <math.h>
#include <stdio.h>
#include <type_traits>
#include <stdlib.h>
#include <string.h>

#include "cglbm.h"

namespace cglbm {

// ---------------------------------------------------------------- storage codecs
// kEqRef: the "equilibrium-referenced" 16-bit forms store the moving
// populations relative to a per-node reference equilibrium (see "16-bit
// storage" below) and the rest population exactly, split over two 16-bit
// planes; the plain 16-bit forms store the deviation d_i itself.
struct StF32 {
    typedef float T;
    static constexpr bool kEqRef = false;
    static __device__ __forceinline__ float dec(T v) { return v; }
    static __device__ __forceinline__ T enc(float v) { return v; }
};
// bfloat16: upper half of the FP32 pattern; encoded round-to-nearest-even by
// the gfx950 conversion instruction (v_cvt_pk_bf16_f32)
template <bool EQ>
struct StBF16T {
    typedef uint16_t T;
    static constexpr bool kEqRef = EQ;
    static __device__ __forceinline__ float dec(T v) { return __uint_as_float((uint32_t)v << 16); }
    static __device__ __forceinline__ T enc(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
    static __device__ __forceinline__ float dec_bits(uint32_t b) { return __uint_as_float(b << 16); }
    static __device__ __forceinline__ uint32_t enc_bits(float v) { return enc(v); }
};
// IEEE binary16, hardware conversion (round to nearest even)
template <bool EQ>
struct StF16T {
    typedef _Float16 T;
    static constexpr bool kEqRef = EQ;
    static __device__ __forceinline__ float dec(T v) { return (float)v; }
    static __device__ __forceinline__ T enc(float v) { return (T)v; }
    static __device__ __forceinline__ float dec_bits(uint32_t b)
    {
        return (float)__builtin_bit_cast(_Float16, (uint16_t)b);
    }
    static __device__ __forceinline__ uint32_t enc_bits(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }
};
using StBF16 = StBF16T<false>;
using StF16 = StF16T<false>;
using StBF16Eq = StBF16T<true>;
using StF16Eq = StF16T<true>;

// ---------------------------------------------------------------- parameters
struct KP {
    int nx, ny, nz;    // interior lattice
    int rs;            // row stride in elements (rs >= nx)
    int zg;            // stored planes below z = 0 (jet: 1)
    uint32_t n19;      // D3Q19: rows x stride
    int px, py;        // padded lattice (general state, adjoint's stencil cotangents): nx + 2, ny + 2
    uint32_t NP;       // its node count px * py * (nz + 2)
    uint32_t N;        // interior node count nx * ny * nz
    uint32_t plane;    // nx * ny
    uint32_t nx_mul;   // p / nx = (p * nx_mul) >> nx_sh, exact for p < 2^31
    int nx_sh;
    int z0;            // first interior plane of the launch
    int planes;        // planes of the launch (tiled kernels)
    float rho_r0, rho_b0, alpha_r, alpha_b;
    float dalpha;      // alpha_r - alpha_b
    float a_minus_w0;  // alpha_b - w_0
    float kappa_b_m1;  // 27 (1 - alpha_b) / 19 - 1
    float inv_nu_r, inv_nu_b, A, beta, eps2;
    float gx, gy, gz;
    float inlet_cx, inlet_cy, inlet_r2, inlet_u, noise_amp;
    uint64_t seed;
    long long t;       // time level of the state that is read
    int unshifted;     // general state (54 padded planes) stored without the streaming shift
    int xr_tagged;     // adjoint passes: XR holds the tagged minority fraction (else rho_r / rho)
    const float* inlet_uz;
    const float4* R;   // (tagged minority fraction, V) of the state that is read
    const uint4* Qrec; // referenced 16-bit storage: reference record of the state that is read
};

struct MirrorTable {
    int8_t v[Q * 8];
};
constexpr MirrorTable make_mirror()
{
    MirrorTable t{};
    for (int i = 0; i < Q; ++i)
        for (int m = 0; m < 8; ++m) t.v[i * 8 + m] = (int8_t)mirror_dir(i, m);
    return t;
}
// direction i with the components in mask m (bit 0: x, 1: y, 2: z) reversed
__constant__ MirrorTable kMirror = make_mirror();

// index on the padded lattice (one ghost cell on every side): the general state
// and the adjoint's stencil cotangents
__device__ __forceinline__ uint32_t pidx(const KP& k, int x, int y, int z)
{
    return ((uint32_t)(z + 1) * (uint32_t)k.py + (uint32_t)(y + 1)) * (uint32_t)k.px + (uint32_t)(x + 1);
}

// row (y, z) and index of node (x, y, z) in the per-node arrays
__device__ __forceinline__ uint32_t row_of(const KP& k, int y, int z)
{
    return (uint32_t)(z + k.zg) * (uint32_t)k.ny + (uint32_t)y;
}
__device__ __forceinline__ uint32_t nidx_of(const KP& k, int x, int y, int z)
{
    return row_of(k, y, z) * (uint32_t)k.rs + (uint32_t)x;
}

__device__ __forceinline__ int wrapc(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }
__device__ __forceinline__ int clampc(int a, int n) { return a < 0 ? 0 : (a >= n ? n - 1 : a); }

// slot of direction i within its row (see the layout above)
__host__ __device__ constexpr int slot_of(int i) { return 9 * (kCZ[i] + 1) + 3 * (kCY[i] + 1) + (kCX[i] + 1); }

// interior node of this thread: z = blockIdx.y + z0
struct Node {
    int x, y, z;
    uint32_t n;  // index in the per-node arrays
    uint32_t q;  // y nx + x (index within an interior plane)
    bool valid;
};

__device__ __forceinline__ Node this_node(const KP& k)
{
    Node d;
    const uint32_t p = blockIdx.x * 256u + threadIdx.x;
    d.valid = p < k.plane;
    d.z = (int)blockIdx.y + k.z0;
    d.y = (int)(((uint64_t)p * k.nx_mul) >> k.nx_sh);
    d.x = (int)p - d.y * k.nx;
    d.q = p;
    d.n = nidx_of(k, d.x, d.y, d.z);
    return d;
}

// element idx of a plane, addressed as uniform base + byte offset (32-bit for
// elements of up to 8 bytes: at most 2^29 padded nodes)
template <class T>
__device__ __forceinline__ T ldp(const T* __restrict__ base, uint32_t idx)
{
    if constexpr (sizeof(T) >= 16)  // 16-byte records: 64-bit offsets (more than 2^28 nodes)
        return *(const T*)((const char*)base + (size_t)idx * sizeof(T));
    else
        return *(const T*)((const char*)base + (idx * (uint32_t)sizeof(T)));
}
template <class T>
__device__ __forceinline__ void stp(T* __restrict__ base, uint32_t idx, T v)
{
    if constexpr (sizeof(T) >= 16)
        *(T*)((char*)base + (size_t)idx * sizeof(T)) = v;
    else
        *(T*)((char*)base + (idx * (uint32_t)sizeof(T))) = v;
}

// Populations through buffer resources: the base address of a row sits in
// scalar registers and the lane supplies only its byte offset within the row (one
// of three for all 27 directions), so a pull costs no per-lane address
// arithmetic.  The record count bounds every access to the row (out-of-range
// loads read 0 and out-of-range stores are dropped).
template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const T* base, uint32_t elems)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), (short)0, (int)(elems * (uint32_t)sizeof(T)),
                                             0x00020000);
}
// 2- or 4-byte value at byte offset voff + soff (soff uniform)
template <class T>
__device__ __forceinline__ T ld_row(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    static_assert(sizeof(T) == 2 || sizeof(T) == 4, "population slots hold 2- or 4-byte values");
    if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
}
// NT: a non-temporal store
template <bool NT, class T>
__device__ __forceinline__ void st_row(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, T v)
{
    if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, NT ? 2 : 0);
    else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, voff, soff, NT ? 2 : 0);
}

// 16-byte record (R, reference record) of node x of row `row` (uniform)
template <class T>
__device__ __forceinline__ void st_rec(T* __restrict__ base, const KP& k, uint32_t row, int x, T v)
{
    static_assert(sizeof(T) == 16, "16-byte records");
    const auto r = row_rsrc(base + (size_t)row * (uint32_t)k.rs, (uint32_t)k.rs);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) uint32_t, v), r,
                                           (uint32_t)x * 16u, 0, 0);
}

// ---------------------------------------------------------------- 16-bit storage
// In the plain 16-bit forms the stored deviation d_i = f_i - w_i rho_b0 of a
// moving direction carries the velocity part of the equilibrium,
// w_i rho (3 c.u + ...), and at interfaces its phase part w_i (rho kappa -
// rho_b0); their 16-bit rounding feeds an O(2^-9 |u|) momentum error into
// every step.  The equilibrium-referenced forms remove both: the collision
// writes, per node, a reference record (rho~, u~, E~) rounded to the storage
// format, E = rho kappa(alpha_bar) - rho_b0, and stores
//   e_i = d'_i - w_i (E~ + rho~ P_i(u~)),
//   P_i(u) = c.u (3 + 4.5 (c.u)^2 - 4.5 u^2) + 4.5 (c.u)^2 - 1.5 u^2;
// readers add the same term computed from the same rounded record, so only
// the rounding of the small remainder e_i is lost.  The rest population (O(1)
// in the red phase) is kept exactly: its FP32 bits are split over its own slot
// (high half) and a 28th slot of the row (low half).
__device__ __forceinline__ float eq_poly(float cu, float u2)
{
    return cu * (3.f + 4.5f * cu * cu - 4.5f * u2) + (4.5f * cu * cu - 1.5f * u2);
}

struct RefRec {
    float rho, ux, uy, uz, e;
};

template <class S>
__device__ __forceinline__ RefRec dec_ref(uint4 q)
{
    RefRec r;
    r.rho = S::dec_bits(q.x & 0xffffu);
    r.ux = S::dec_bits(q.x >> 16);
    r.uy = S::dec_bits(q.y & 0xffffu);
    r.uz = S::dec_bits(q.y >> 16);
    r.e = S::dec_bits(q.z & 0xffffu);
    return r;
}

template <class S>
__device__ __forceinline__ uint4 enc_ref(float rho, float ux, float uy, float uz, float e)
{
    return make_uint4(S::enc_bits(rho) | (S::enc_bits(ux) << 16), S::enc_bits(uy) | (S::enc_bits(uz) << 16),
                      S::enc_bits(e), 0u);
}

// the records of a node mirrored across the walls in mask m (bit 0: x, 1: y, 2: z)
__device__ __forceinline__ float4 mirror_rec(float4 r, int m)
{
    if (m & 1) r.y = -r.y;
    if (m & 2) r.z = -r.z;
    if (m & 4) r.w = -r.w;
    return r;
}
__device__ __forceinline__ uint4 mirror_ref(uint4 q, int m)
{
    if (m & 1) q.x ^= 0x80000000u;
    if (m & 2) q.y ^= 0x00008000u;
    if (m & 4) q.y ^= 0x80000000u;
    return q;
}

// slots of a row in the shifted form
template <class S>
constexpr int kSlots = S::kEqRef ? Q + 1 : Q;

__device__ __forceinline__ bool inlet_inside(const KP& k, int xg, int yg)
{
    if (xg < 0 || xg >= k.nx || yg < 0 || yg >= k.ny) return false;
    const float dx = (float)xg - k.inlet_cx, dy = (float)yg - k.inlet_cy;
    return dx * dx + dy * dy < k.inlet_r2;
}

// n-th output of SplitMix64 seeded with `seed` (Steele, Lea and Flood 2014)
__device__ __forceinline__ uint64_t splitmix64_nth(uint64_t seed, uint64_t n)
{
    uint64_t z = seed + (n + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// inlet ghost population of direction I leaving ghost column (xg, yg) at
// post-collision time tg: red equilibrium at rho_r0, alpha_r, Phi = 0, with the
// uniform axial inflow plus the radial noise (Sec. IV A).  Returns f^e_I.
template <int I>
__device__ __forceinline__ float inlet_feq_dir(const KP& k, int xg, int yg, long long tg)
{
    const uint64_t cnt = ((uint64_t)tg * (uint64_t)k.ny + (uint64_t)yg) * (uint64_t)k.nx + (uint64_t)xg;
    const uint64_t r = splitmix64_nth(k.seed, cnt);
    const double xi = (double)(r >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
    const float ur = (float)((double)k.noise_amp * (double)k.inlet_u * xi);
    const float dx = (float)xg - k.inlet_cx, dy = (float)yg - k.inlet_cy;
    const float rr = sqrtf(dx * dx + dy * dy);
    const float ux = rr > 0.f ? ur * dx / rr : 0.f, uy = rr > 0.f ? ur * dy / rr : 0.f;
    const float uz = k.inlet_uz ? k.inlet_uz[yg * k.nx + xg] : k.inlet_u;
    // fused multiply-adds written out, so that the inflow does not depend on the
    // code that this is inlined into
    const float u2 = fmaf(uz, uz, fmaf(ux, ux, uy * uy));
    const float cu = kCX[I] * ux + kCY[I] * uy + kCZ[I] * uz;
    const float poly = cu * (3.f + 4.5f * cu + 4.5f * cu * cu - 4.5f * u2) - 1.5f * u2;
    // |c_I| >= 1 here: varphi_I = w_I kappa_r, kappa_r = 27/19 (1 - alpha_r)
    return k.rho_r0 * wgt(I) * fmaf(27.f / 19.f, 1.f - k.alpha_r, poly);
}

// ---------------------------------------------------------------- colour fractions
// The recolouring of a node needs x_r = rho_r/rho and x_b = 1 - x_r.  FP32
// keeps a fraction near 1 only to an absolute 2^-24, which leaves the other
// colour a relative error 2^-24/x, and Eq. order multiplies the error of
// rho_k by rho/rho_k0 (up to gamma where the dense colour dominates).  A node
// therefore keeps the fraction of its minority colour, with full relative
// precision at both ends, and marks which colour that is in the lowest
// mantissa bit: 0 red (the value is x_r), 1 blue (the value is x_b).  The
// mark costs one bit of the fraction: the value is the FP32 number nearest to
// the fraction among those with the right lowest bit (an unbiased rounding to
// a grid of two ulps, so colour masses do not drift).  The other colour is
// always formed as the colour-blind value minus the kept one.
__device__ __forceinline__ uint32_t blue_kept(float s) { return __float_as_uint(s) & 1u; }
__device__ __forceinline__ float frac_tag(double x, uint32_t blue)
{
    const float f = (float)x;
    uint32_t b = __float_as_uint(f);
    if ((b & 1u) != blue) {
        if ((b & 0x7fffffffu) == 0u)
            b |= 1u;  // +-0: the smallest magnitude that carries the mark
        else
            b += fabs(x) > fabs((double)f) ? 1u : 0xffffffffu;  // one ulp towards x (in magnitude)
    }
    return __uint_as_float(b);
}
// the fraction of colour `blue` (0 red, 1 blue) from a tagged value s
__device__ __forceinline__ float frac_of(float s, uint32_t blue) { return blue_kept(s) == blue ? s : 1.f - s; }

// ---------------------------------------------------------------- pull
// Where a node (x, y, z) pulls from.  Along x the lane holds three byte offsets
// into the three slots c_x = -1, 0, 1 of a group (c_y, c_z): the source x - c_x,
// wrapped, or (jet) at the wall the node itself in the slot of the reversed
// velocity.  The group's row is uniform over the wavefront (y and z are).
struct XOff {
    uint32_t p, o, m;     // c_x = +1, 0, -1
    uint32_t rp, ro, rm;  // the same sources in a row of 16-byte records
    bool wp, wm;          // jet: the source lies beyond the wall
};
template <int BC, class T>
__device__ __forceinline__ XOff x_offsets(const KP& k, int x)
{
    constexpr uint32_t B = sizeof(T);
    const uint32_t rs = (uint32_t)k.rs, nx = (uint32_t)k.nx, ux = (uint32_t)x;
    XOff o;
    o.o = (rs + ux) * B;
    o.p = (2 * rs + ux - 1u) * B;
    o.m = (ux + 1u) * B;
    o.ro = ux * 16u;
    o.rp = o.ro - 16u;
    o.rm = o.ro + 16u;
    o.wp = x == 0;
    o.wm = x == k.nx - 1;
    if (o.wp) {
        o.p = BC == LBM_BC_PERIODIC ? (2 * rs + nx - 1u) * B : 0u;
        o.rp = BC == LBM_BC_PERIODIC ? (nx - 1u) * 16u : 0u;
    }
    if (o.wm) {
        o.m = BC == LBM_BC_PERIODIC ? 0u : (2 * rs + nx - 1u) * B;
        o.rm = BC == LBM_BC_PERIODIC ? 0u : (nx - 1u) * 16u;
    }
    return o;
}

// The row that the group (CY, CZ) of node row (y, z) is pulled from: (y - CY,
// z - CZ), wrapped; jet: at a side wall the node's own row, mirrored (my), below
// the bottom the ghost plane (which holds the mirrored populations and the
// inflow).  The jet's outlet plane is never pulled into; its row above is clamped
// to stay inside the buffer.
template <int BC, int CY, int CZ>
__device__ __forceinline__ uint32_t group_row(const KP& k, int y, int z, bool& my)
{
    int ys = y - CY, zs = z - CZ;
    my = false;
    if (BC == LBM_BC_PERIODIC) {
        if (CY) ys = wrapc(ys, k.ny);
        if (CZ) zs = wrapc(zs, k.nz);
    } else {
        if (CY && (ys < 0 || ys >= k.ny)) {
            ys = y;
            my = true;
        }
        if (CZ < 0 && zs >= k.nz) zs = k.nz - 1;
    }
    return row_of(k, ys, zs);
}

// element offset of the group in its row; a mirrored row gives the mirrored group
template <int BC, int SL, int CY, int CZ>
__device__ __forceinline__ size_t group_off(const KP& k, int y, int z)
{
    bool my;
    const uint32_t row = group_row<BC, CY, CZ>(k, y, z, my);
    const int g = 9 * (CZ + 1) + 3 * (CY + 1) - (my ? 6 * CY : 0);
    return ((size_t)row * SL + g) * (uint32_t)k.rs;
}

// Value at byte offset x of the slots (or records) that begin at `row`.  ROW: the
// pointer is uniform over the wavefront; else each lane has its own.
template <bool ROW, class T>
__device__ __forceinline__ T ld_slot(const T* __restrict__ row, const KP& k, uint32_t x)
{
    if constexpr (!ROW)
        return *(const T*)((const char*)row + x);
    else if constexpr (sizeof(T) == 16)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(row_rsrc(row, (uint32_t)k.rs), x, 0, 0));
    else
        return ld_row<T>(row_rsrc(row, 3u * (uint32_t)k.rs), x, 0u);
}

// stored value of direction I pulled into node row (y, z); ROW: the row is uniform
// over the wavefront (else every lane has its own)
template <int BC, class S, int I, bool ROW = true>
__device__ __forceinline__ typename S::T pull_raw(const typename S::T* __restrict__ src, const KP& k, int y, int z,
                                                  const XOff& xo)
{
    constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
    return ld_slot<ROW>(src + group_off<BC, kSlots<S>, cy, cz>(k, y, z), k, cx > 0 ? xo.p : (cx < 0 ? xo.m : xo.o));
}

// A per-node record at (x, y, z), which may lie one node outside: wrapped, or
// (jet) the wall node's record mirrored.  z = -1 is the jet's ghost plane.
// XIN: x lies inside.
template <int BC, bool XIN>
__device__ __forceinline__ uint32_t rec_index(const KP& k, int x, int y, int z, int& mask)
{
    mask = 0;
    if (BC == LBM_BC_PERIODIC) return nidx_of(k, XIN ? x : wrapc(x, k.nx), wrapc(y, k.ny), wrapc(z, k.nz));
    if (!XIN && (x < 0 || x >= k.nx)) {
        mask |= 1;
        x = clampc(x, k.nx);
    }
    if (y < 0 || y >= k.ny) {
        mask |= 2;
        y = clampc(y, k.ny);
    }
    if (z >= k.nz) z = k.nz - 1;
    return nidx_of(k, x, y, z);
}
template <int BC, bool XIN = false>
__device__ __forceinline__ float4 rec_at(const KP& k, const float4* __restrict__ R, int x, int y, int z)
{
    int m;
    const float4 r = ldp(R, rec_index<BC, XIN>(k, x, y, z, m));
    return BC == LBM_BC_JET ? mirror_rec(r, m) : r;
}
template <int BC, bool XIN = false>
__device__ __forceinline__ uint4 ref_at(const KP& k, int x, int y, int z)
{
    int m;
    const uint4 q = ldp(k.Qrec, rec_index<BC, XIN>(k, x, y, z, m));
    return BC == LBM_BC_JET ? mirror_ref(q, m) : q;
}
// (phi, rho - rho_b0) at (x, y, z), which may lie one node outside: wrapped, or
// (jet) the wall node's value, and (1, rho_r0 - rho_b0) in the inlet circle
template <int BC, bool XIN = false>
__device__ __forceinline__ float2 pd_at(const KP& k, const float2* __restrict__ PD, int x, int y, int z)
{
    if (BC == LBM_BC_PERIODIC) return ldp(PD, nidx_of(k, XIN ? x : wrapc(x, k.nx), wrapc(y, k.ny), wrapc(z, k.nz)));
    const float2 v = ldp(PD, nidx_of(k, XIN ? x : clampc(x, k.nx), clampc(y, k.ny), clampc(z, k.nz)));
    return z < 0 && inlet_inside(k, x, y) ? make_float2(1.f, k.rho_r0 - k.rho_b0) : v;
}

// the part of d_I that the referenced 16-bit forms keep in the record of the
// source node (zero in the other forms)
template <int I>
__device__ __forceinline__ float ref_part(const RefRec& r)
{
    const float cu = kCX[I] * r.ux + kCY[I] * r.uy + kCZ[I] * r.uz;
    const float u2 = r.ux * r.ux + r.uy * r.uy + r.uz * r.uz;
    return wgt(I) * (r.e + r.rho * eq_poly(cu, u2));
}

// 16-byte record of the source of direction I; m: the axes it has to be mirrored on
template <int BC, int I, bool ROW = true, class T>
__device__ __forceinline__ T pull_rec(const T* __restrict__ base, const KP& k, int y, int z, const XOff& xo, int& m)
{
    static_assert(sizeof(T) == 16, "16-byte records");
    constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
    bool my;
    const uint32_t row = group_row<BC, cy, cz>(k, y, z, my);
    m = (BC == LBM_BC_JET && ((cx > 0 && xo.wp) || (cx < 0 && xo.wm)) ? 1 : 0) | (my ? 2 : 0);
    return ld_slot<ROW>(base + (size_t)row * (uint32_t)k.rs, k,
                        cx > 0 ? xo.rp : (cx < 0 ? xo.rm : xo.ro));
}

// pre-collision deviation d_I pulled into node (x, y, z)
template <int BC, class S, int I, bool ROW = true>
__device__ __forceinline__ float pull_dev(const typename S::T* __restrict__ src, const KP& k, int x, int y, int z,
                                          const XOff& xo)
{
    if constexpr (!S::kEqRef) {
        return S::dec(pull_raw<BC, S, I, ROW>(src, k, y, z, xo));
    } else if constexpr (I == 0 && !ROW) {
        const typename S::T* b = src + (size_t)row_of(k, y, z) * (kSlots<S> * (uint32_t)k.rs) + x;
        const uint32_t hi = __builtin_bit_cast(uint16_t, b[slot_of(0) * (uint32_t)k.rs]);
        const uint32_t lo = __builtin_bit_cast(uint16_t, b[Q * (uint32_t)k.rs]);
        return __uint_as_float((hi << 16) | lo);
    } else if constexpr (I == 0) {
        const auto r = row_rsrc(src + (size_t)row_of(k, y, z) * (kSlots<S> * (uint32_t)k.rs),
                                kSlots<S> * (uint32_t)k.rs);
        const uint32_t B = sizeof(typename S::T), rs = (uint32_t)k.rs;
        const uint32_t hi = __builtin_bit_cast(uint16_t, ld_row<typename S::T>(r, (uint32_t)x * B, slot_of(0) * rs * B));
        const uint32_t lo = __builtin_bit_cast(uint16_t, ld_row<typename S::T>(r, (uint32_t)x * B, Q * rs * B));
        return __uint_as_float((hi << 16) | lo);
    } else {
        int m;
        const uint4 q = pull_rec<BC, I, ROW>(k.Qrec, k, y, z, xo, m);
        return S::dec(pull_raw<BC, S, I, ROW>(src, k, y, z, xo)) + ref_part<I>(dec_ref<S>(mirror_ref(q, m)));
    }
}

// Pre-collision value of direction I at a node of a post-collision (shifted)
// state: d, and both colours rebuilt from the source's R (Eqs. op3r/op3b):
//   f^k*_i = x_k f'_i +- (w_i/|c_i|) c_i . V   (+ red, - blue),
// the kept colour from its fraction, the other as f - f^k (formed in FP64,
// rounded once).
__device__ __forceinline__ float other_colour(const KP& k, int i, float d, float fk)
{
    return (float)(((double)d + wgtd(i) * (double)k.rho_b0) - (double)fk);
}

template <int I>
__device__ __forceinline__ void colours_of(const KP& k, float d, const float4& r, float& fr, float& fb)
{
    const float f = d + wgt(I) * k.rho_b0;
    const float vt = I == 0 ? 0.f : (wgt(I) * inv_len(I)) * cdot(I, r.y, r.z, r.w);
    const uint32_t bl = blue_kept(r.x);
    const float fk = r.x * f + (bl ? -vt : vt);
    const float fo = other_colour(k, I, d, fk);
    fr = bl ? fo : fk;
    fb = bl ? fk : fo;
}

template <int BC, class S, bool WANT_F, bool ROW = true, int I = 0>
__device__ __forceinline__ void pull_dirs(const typename S::T* __restrict__ src, const KP& k, int x, int y, int z,
                                          const XOff& xo, float* d, float* fr, float* fb)
{
    if constexpr (I < Q) {
        d[I] = pull_dev<BC, S, I, ROW>(src, k, x, y, z, xo);
        if constexpr (WANT_F) {
            int m;
            const float4 r = pull_rec<BC, I, ROW>(k.R, k, y, z, xo, m);
            colours_of<I>(k, d[I], mirror_rec(r, m), fr[I], fb[I]);
        }
        pull_dirs<BC, S, WANT_F, ROW, I + 1>(src, k, x, y, z, xo, d, fr, fb);
    }
}

// General state, stored at the node itself on the padded lattice: planes 0..26
// hold the deviations, planes 27..53 the populations of the colour that the flag
// of the node's R names (its R sits at the padded index, too).
template <class T>
__device__ __forceinline__ T ld_general(const T* __restrict__ src, const KP& k, int i, uint32_t pn, bool kept)
{
    return ldp(src + (size_t)((kept ? Q : 0) + i) * k.NP, pn);
}

template <class S, bool WANT_F, int I = 0>
__device__ __forceinline__ void general_dirs(const typename S::T* __restrict__ src, const KP& k, uint32_t pn,
                                             uint32_t bl, float* d, float* fr, float* fb)
{
    if constexpr (I < Q) {
        d[I] = S::dec(ld_general(src, k, I, pn, false));
        if constexpr (WANT_F) {
            const float fk = S::dec(ld_general(src, k, I, pn, true));
            const float fo = other_colour(k, I, d[I], fk);
            fr[I] = bl ? fo : fk;
            fb[I] = bl ? fk : fo;
        }
        general_dirs<S, WANT_F, I + 1>(src, k, pn, bl, d, fr, fb);
    }
}

// the 27 pre-collision deviations (and colour populations) of a node
template <int BC, class S, bool WANT_F, bool ROW = true>
__device__ __forceinline__ void pull_all(const typename S::T* __restrict__ src, const KP& k, int x, int y, int z,
                                         float* d, float* fr, float* fb)
{
    if (k.unshifted) {
        const uint32_t pn = pidx(k, x, y, z);
        general_dirs<S, WANT_F>(src, k, pn, WANT_F ? blue_kept(ldp(k.R, pn).x) : 0u, d, fr, fb);
    } else {
        pull_dirs<BC, S, WANT_F, ROW>(src, k, x, y, z, x_offsets<BC, typename S::T>(k, x), d, fr, fb);
    }
}

// Pre-collision state of an outlet node (x, y, nz - 1) by the convective
// condition f(N) = [f_prev(N) + lam f(N - 1)] / (1 + lam), lam = max(0, u_z(N - 1))
// evaluated on the freshly streamed populations of the node below; hprev holds
// the outlet plane of the previous step (d, then f^r); blue is formed as f - f^r.
template <class S, bool ROW = true>
__device__ void outlet_state(const typename S::T* __restrict__ src, const KP& k, const float* __restrict__ hprev,
                             const Node& nd, float* d, float* fr, float* fb)
{
    if (k.unshifted) {
        pull_all<LBM_BC_JET, S, true, ROW>(src, k, nd.x, nd.y, nd.z, d, fr, fb);
        return;
    }
    pull_all<LBM_BC_JET, S, true, ROW>(src, k, nd.x, nd.y, nd.z - 1, d, fr, fb);
    float m0 = 0.f, jz = 0.f;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        m0 += d[i];
        if (kCZ[i]) jz += kCZ[i] * d[i];
    }
    const float rho = k.rho_b0 + m0;
    const float uz = (jz + 0.5f * m0 * k.gz) / rho;
    const float lam = uz > 0.f ? uz : 0.f;
    const float inv = 1.f / (1.f + lam);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        d[i] = (hprev[(size_t)i * k.plane + nd.q] + lam * d[i]) * inv;
        fr[i] = (hprev[(size_t)(Q + i) * k.plane + nd.q] + lam * fr[i]) * inv;
        fb[i] = other_colour(k, i, d[i], fr[i]);
    }
}

// ---------------------------------------------------------------- block reduction (FP64 audit)
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NV>
__device__ void block_partials(double (&v)[NV], double* __restrict__ out, uint32_t slot)
{
    __shared__ double red[NV][4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < NV; ++a) {
        const double s = wave_sum(v[a]);
        if (lane == 0) red[a][wv] = s;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        const int a = threadIdx.x;
        out[(size_t)slot * NV + a] = red[a][0] + red[a][1] + red[a][2] + red[a][3];
    }
}

constexpr int BLOCK = 256;

// ---------------------------------------------------------------- stencil tiles
// The step's kernels take a tile of TX x TY nodes of one plane per block, a
// wavefront 64 nodes of one row, and stage the neighbour data they gather 26
// times per node (the recolouring float4 R of the density pass, the (phi, rho)
// fields of the gradient) once into LDS: a window of the tile plus a one-node
// rim in x and y, over planes z - 1, z, z + 1, loaded row by row.
// Tiles of the step kernels: CX x CY nodes in the fused kernel, DX x DY in the
// density pass.
template <int X, int D>
struct StepTiles {
    static constexpr int CX = X, CY = BLOCK / X, DX = X, DY = D / X;
    static constexpr bool kFlat = false;
};
// no tiles: blocks of 256 consecutive nodes of a plane, neighbours through the caches
struct NodeBlocks {
    static constexpr int CX = BLOCK, CY = 1, DX = BLOCK, DY = 1;
    static constexpr bool kFlat = true;
};
using WideTiles = StepTiles<128, 512>;
using NarrowTiles = StepTiles<64, 256>;
using RefTiles = StepTiles<64, 512>;  // referenced 16-bit forms

template <int TX, int TY>
struct TileShape {
    static constexpr int WX = TX + 2, WY = TY + 2, W = 3 * WX * WY, NT = TX * TY;
};

struct Tile {
    int x0, y0, z, lx, ly;
    Node nd;
};

// Order of the tiles.  Workgroups go round-robin to the 8 XCDs, so a plane's
// neighbouring tiles would sit on different L2s, each fetching the halo
// rows they share and each writing a part of the lines in which two
// unaligned rows meet.  With T tiles in a plane XCD j takes the contiguous
// band of tiles [(j T + z mod 8) / 8, ((j + 1) T + z mod 8) / 8): T tiles in
// any eight planes, and where T is a multiple of 8 the same ones in each.
// Against the plain order where T is no multiple of 8: 0.78 -> 0.70 ms on
// 154x120x422 nodes (FP32), 0.90 -> 0.78 ms on 144x183x488 (FP16).
//
// Grid of a launch over `planes` planes of T tiles: (T, planes) where T is a
// multiple of 8 or below 8, else the blocks of the planes rounded up to a
// multiple of 8 in one row.  A row of 2^32 lanes or more cannot be launched (thin
// lattices: from 2^25 rows of nodes with 128x2 tiles); these keep (T, planes) in the
// plain order (with more than one plane: a plane has fewer than 2^21 tiles).
template <int TX, int TY>
__host__ __device__ __forceinline__ uint32_t tiles_in_plane(int nx, int ny)
{
    return (uint32_t)((nx + TX - 1) / TX) * (uint32_t)((ny + TY - 1) / TY);
}
template <int TX, int TY>
inline dim3 tile_grid(int nx, int ny, int planes)
{
    const uint64_t T = tiles_in_plane<TX, TY>(nx, ny), row = T * (uint64_t)((planes + 7) / 8 * 8);
    if (T % 8 == 0 || T < 8 || row * (TX * TY) >= (1ull << 32)) return dim3((unsigned)T, planes);
    return dim3((unsigned)row);
}

// tile b and plane z of block (bx, by) of such a grid (gx, gy) of T tiles a plane; not
// live: beyond the planes
struct TileOrder {
    int b, z;
    bool live;
};
__host__ __device__ __forceinline__ TileOrder tile_of_block(uint32_t gx, uint32_t gy, uint32_t bx, uint32_t by, int T,
                                                            int planes)
{
    int b = (int)bx, z = (int)by;
    bool live = true;
    if (gy == 1 && gx > 8) {
        const int j = b & 7, i = b >> 3, q = i / T;
        b = i - q * T;  // the band's tiles of planes 8 q .. 8 q + 7, plane by plane
        z = 8 * q;
        int lo = j * T;
        for (int r = 0; r < 7; ++r) {
            const int n = ((lo + T) >> 3) - (lo >> 3);
            if (b < n) break;
            b -= n;
            ++lo;
            ++z;
        }
        b += lo >> 3;
        live = z < planes;
    } else if ((gx & 7u) == 0) {
        b = (b & 7) * (int)(gx >> 3) + (b >> 3);
    }
    return TileOrder{b, z, live};
}

template <int TX, int TY>
__device__ __forceinline__ Tile this_tile(const KP& k)
{
    static_assert(TX % 64 == 0, "a wavefront lies in one row");
    Tile t;
    const int ntx = (k.nx + TX - 1) / TX;
    const TileOrder o = tile_of_block(gridDim.x, gridDim.y, blockIdx.x, blockIdx.y,
                                      ntx * ((k.ny + TY - 1) / TY), k.planes);
    t.z = o.z + k.z0;
    const int ty = o.live ? o.b / ntx : (k.ny + TY) / TY + 1, tx = o.live ? o.b - ty * ntx : 0;  // idle: beyond every row
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);  // uniform, and so are y and the row
    t.x0 = tx * TX;
    t.y0 = ty * TY;
    t.lx = (wave % (TX / 64)) * 64 + ((int)threadIdx.x & 63);
    t.ly = wave / (TX / 64);
    Node& d = t.nd;
    d.x = t.x0 + t.lx;
    d.y = t.y0 + t.ly;
    d.z = t.z;
    d.valid = d.x < k.nx && d.y < k.ny;
    d.q = (uint32_t)d.y * (uint32_t)k.nx + (uint32_t)d.x;
    d.n = nidx_of(k, d.x, d.y, d.z);
    return t;
}

// window slot of the node at offset (dx, dy, dz) from local node (lx, ly)
template <int TX, int TY>
__device__ __forceinline__ int wslot(int lx, int ly, int dx, int dy, int dz)
{
    using TS = TileShape<TX, TY>;
    return ((dz + 1) * TS::WY + (ly + 1 + dy)) * TS::WX + (lx + 1 + dx);
}

// Stage a per-node array over the window of tile t by put(slot, value).  A
// wavefront takes whole row segments of 64 nodes, so the source row is a scalar
// and only the x offset is per lane: fetch_row(x, y, z), x inside the lattice;
// the two rim columns, 2 x 3 (TY + 2) nodes, are gathered by one wavefront with
// fetch(x, y, z).  Nodes beyond the rim of a ragged last tile are skipped: no
// valid node reads them.  All of a lane's loads are issued before its LDS
// writes: one memory latency for the window instead of one per element.
template <int TX, int TY, class F, class G, class P>
__device__ __forceinline__ void stage_window(const KP& k, const Tile& t, F&& fetch_row, G&& fetch, P&& put)
{
    using TS = TileShape<TX, TY>;
    constexpr int NW = TX * TY / 64, SEG = TX / 64, ROWS = 3 * TS::WY, NIT = (ROWS * SEG + NW - 1) / NW;
    static_assert(2 * ROWS <= 64, "one wavefront gathers the rim columns");
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    decltype(fetch(0, 0, 0)) v[NIT], e;
    bool ok[NIT];
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
        const int s = wave + j * NW, r = s / SEG, wz = r / TS::WY;
        const int x = t.x0 + (s % SEG) * 64 + lane, y = t.y0 - 1 + (r - wz * TS::WY);
        ok[j] = s < ROWS * SEG && y <= k.ny && x < k.nx;
        if (ok[j]) v[j] = fetch_row(x, y, t.z - 1 + wz);
    }
    const int er = lane >> 1, ez = er / TS::WY, ex = (lane & 1) ? min(TX, k.nx - t.x0) : -1, ey = er - ez * TS::WY;
    const bool eok = wave == NW - 1 && er < ROWS && t.y0 - 1 + ey <= k.ny;
    if (eok) e = fetch(t.x0 + ex, t.y0 - 1 + ey, t.z - 1 + ez);
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
        const int s = wave + j * NW, r = s / SEG;
        if (ok[j]) put(r * TS::WX + 1 + (s % SEG) * 64 + lane, v[j]);
    }
    if (eok) put(er * TS::WX + 1 + ex, e);
}

// LDS window of the reference records of the 16-bit forms that have them,
// unpacked once for their 26 readers: a = (u, rho), b = (u^2, E).  It takes 24 B per
// node, which is why these forms run on tiles of 64 nodes: with 128 the windows
// leave too few waves (0.81 against 1.16 ms per step on the 128x128x512 jet; 0.87 ms
// with 128 and the records from the caches).
template <class S, int W>
struct RefWin {
    float4 a[S::kEqRef ? W : 1];
    float2 b[S::kEqRef ? W : 1];
};

template <class S, int W>
__device__ __forceinline__ void put_ref(RefWin<S, W>& rw, int w, uint4 q)
{
    const RefRec r = dec_ref<S>(q);
    rw.a[w] = make_float4(r.ux, r.uy, r.uz, r.rho);
    rw.b[w] = make_float2(r.ux * r.ux + r.uy * r.uy + r.uz * r.uz, r.e);
}

// the 27 pre-collision deviations of a node, the references from the window
template <int BC, class S, int TX, int TY, int W, int I = 0>
__device__ __forceinline__ void pull_win(const typename S::T* __restrict__ src, const KP& k, const Tile& t,
                                         const XOff& xo, const RefWin<S, W>& rw, float* d)
{
    if constexpr (I < Q) {
        if constexpr (!S::kEqRef || I == 0) {
            d[I] = pull_dev<BC, S, I>(src, k, t.nd.x, t.nd.y, t.nd.z, xo);
        } else {
            const int w = wslot<TX, TY>(t.lx, t.ly, -kCX[I], -kCY[I], -kCZ[I]);
            const float4 a = rw.a[w];
            const float2 b = rw.b[w];
            const float cu = kCX[I] * a.x + kCY[I] * a.y + kCZ[I] * a.z;
            d[I] = S::dec(pull_raw<BC, S, I>(src, k, t.nd.y, t.nd.z, xo))
                   + wgt(I) * (b.y + a.w * eq_poly(cu, b.x));
        }
        pull_win<BC, S, TX, TY, W, I + 1>(src, k, t, xo, rw, d);
    }
}

// ---------------------------------------------------------------- density pass
// n / d for the O(1), positive denominators of the fields (a density, a sum
// of two): the hardware reciprocal refined by two Newton steps and one
// residual correction, a few FP64 ulps from the rounded quotient, which the
// callers then round to FP32.  Saves the scaling and fix-up steps of the IEEE
// division, which these operands need no cover for (no zero, denormal or
// infinite values).
__device__ __forceinline__ double div_fields(double n, double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double q = n * r;
    return fma(fma(-d, q, n), r, q);
}

// fields: PD = (phi, rho - rho_b0) per padded node and XR = the minority
// colour's fraction, tagged (see "colour fractions"), from the mass sum
// m0 = rho - rho_b0 and the two colour masses.  phi = (rho_r/rho_r0 -
// rho_b/rho_b0) / (rho_r/rho_r0 + rho_b/rho_b0) (Eq. order) with both
// quotients scaled by rho_r0 rho_b0: one division.
__device__ __forceinline__ float2 store_pd(float2* __restrict__ PD, const KP& k, uint32_t n, double m0, double rr,
                                           double rb)
{
    const double a = rr * (double)k.rho_b0, b = rb * (double)k.rho_r0;
    const float2 v = make_float2((float)div_fields(a - b, a + b), (float)m0);
    stp(PD, n, v);
    return v;
}

__device__ __forceinline__ float2 store_fields_sums(float2* __restrict__ PD, float* __restrict__ XR, const KP& k,
                                                    uint32_t n, double m0, double rr, double rb)
{
    const double rho = (double)k.rho_b0 + m0;
    const float2 v = store_pd(PD, k, n, m0, rr, rb);
    const uint32_t bl = rr > rb;
    stp(XR, n, frac_tag(div_fields(bl ? rb : rr, rho), bl));
    return v;
}

__device__ __forceinline__ float2 store_fields(float2* __restrict__ PD, float* __restrict__ XR, const KP& k,
                                               uint32_t n, const float* d, const float* fr)
{
    double m0 = 0.0, rr = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        m0 += (double)d[i];
        rr += (double)fr[i];
    }
    return store_fields_sums(PD, XR, k, n, m0, rr, (double)k.rho_b0 + m0 - rr);
}

__host__ __device__ constexpr double inv_lend(int i)
{
    return csq(i) == 1 ? 1.0 : csq(i) == 2 ? 0.70710678118654752440 : 0.57735026918962576451;
}

// Mass and colour masses of a general state at a node.  The mass sum m0 runs in
// FP64 (an exact sum of the stored deviations: mass is conserved up to the
// storage rounding); mk is the mass of the colour the planes Q..2Q-1 hold.
template <class S, int I = 0>
__device__ __forceinline__ void accum_general(const typename S::T* __restrict__ src, const KP& k, uint32_t pn,
                                              double& m0, double& mk)
{
    if constexpr (I < Q) {
        m0 += (double)S::dec(ld_general(src, k, I, pn, false));
        mk += (double)S::dec(ld_general(src, k, I, pn, true));
        accum_general<S, I + 1>(src, k, pn, m0, mk);
    }
}

// Mass and minority-colour mass of a shifted state at n, from the pulled
// deviations d and the R of the source nodes in the LDS window.  The colour m
// is the one node n kept in the previous step (its own R, direction 0); its
// mass is written
//   rho_m = x_m(x) rho + sum_{i>=1} [(x_m(x - c_i) - x_m(x)) f_i +- (w_i/|c_i|) c_i . V(x - c_i)],
// an FP64 main term plus FP32 corrections (cf: fractions, cv: recolouring
// vectors, + for red, - for blue) that vanish wherever x_m and V are uniform,
// so pure phases carry no rounding bias.  CDOT: without the products with 0 (the plain
// 16-bit density pass gains 2 %, the others lose as much by the schedule).
template <int TX, int TY, bool CDOT, class M, int I = 0>
__device__ __forceinline__ void accum_density_win(const KP& k, const float* d, const float4* __restrict__ win,
                                                  int lx, int ly, M& m0, float& x0, uint32_t& bl, float& cf,
                                                  float& cv)
{
    if constexpr (I < Q) {
        constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
        const float4 r = win[wslot<TX, TY>(lx, ly, -cx, -cy, -cz)];
        m0 += (M)d[I];
        if (I == 0) {
            x0 = r.x;
            bl = blue_kept(r.x);
        } else {
            cf += (frac_of(r.x, bl) - x0) * (d[I] + wgt(I) * k.rho_b0);
            cv += (wgt(I) * inv_len(I)) * (CDOT ? cdot(I, r.y, r.z, r.w) : cx * r.y + cy * r.z + cz * r.w);
        }
        accum_density_win<TX, TY, CDOT, M, I + 1>(k, d, win, lx, ly, m0, x0, bl, cf, cv);
    }
}

// Raw moments of the deviations up to second order -- m0, j (3), P (xx, yy,
// zz, xy, xz, yz) -- as 10 planes of N floats at node index nn (z plane + q),
// for the adjoint step; j and P are FP32 sums over opposite pairs.
__device__ __forceinline__ void store_moments(float* __restrict__ MOM, const KP& k, uint32_t nn, float m0,
                                              const float* d)
{
    float jx = 0.f, jy = 0.f, jz = 0.f, pxx = 0.f, pyy = 0.f, pzz = 0.f, pxy = 0.f, pxz = 0.f, pyz = 0.f;
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const float sp = d[i] + d[i + 1], df = d[i] - d[i + 1];
        if (kCX[i]) { jx += kCX[i] * df; pxx += sp; }
        if (kCY[i]) { jy += kCY[i] * df; pyy += sp; }
        if (kCZ[i]) { jz += kCZ[i] * df; pzz += sp; }
        if (kCX[i] * kCY[i]) pxy += (kCX[i] * kCY[i]) * sp;
        if (kCX[i] * kCZ[i]) pxz += (kCX[i] * kCZ[i]) * sp;
        if (kCY[i] * kCZ[i]) pyz += (kCY[i] * kCZ[i]) * sp;
    }
    const float mv[10] = {m0, jx, jy, jz, pxx, pyy, pzz, pxy, pxz, pyz};
    const size_t N = k.N;
#pragma unroll
    for (int a = 0; a < 10; ++a) MOM[(size_t)a * N + nn] = mv[a];
}

// Waves per SIMD the density pass is compiled for: eight for the plain 16-bit
// forms, the compiler's choice for 512-lane blocks in the others (on the 128x128x512
// jet, in the plane-major layout before the rows: 177 against 184 us in BF16, 281
// against 271 us in FP32).
template <class S>
constexpr int kDensityWaves = (sizeof(typename S::T) == 2 && !S::kEqRef) ? 8 : 2;

// Density pass over the planes of the grid (for the jet all but the outlet
// plane, which k_outlet takes: its branch would double this kernel's
// register count and halve its occupancy).
// MOMS (the adjoint step from a snapshot): also the raw moments of the pulled
// deviations into MOM.  A compile-time switch: the moment code would raise the step's
// registers (FP32: to 90) and with them lower its waves.  335 us on the 128x128x512
// jet, 176 B of traffic per node at 4.4 TB/s (518 us in the plane-major layout).
template <int BC, class S, class TL, bool MOMS = false>
__global__ __launch_bounds__(TL::DX* TL::DY) __attribute__((amdgpu_waves_per_eu(kDensityWaves<S>, 8))) void k_density(
    const typename S::T* __restrict__ src, float2* __restrict__ PD, float* __restrict__ XR, KP k,
    float* __restrict__ MOM)
{
    constexpr int TX = TL::DX, TY = TL::DY, W = TileShape<TX, TY>::W;
    __shared__ float4 win[W];
    __shared__ RefWin<S, W> rw;
    const Tile t = this_tile<TX, TY>(k);
    const Node& nd = t.nd;
    double m0 = 0.0, mk = 0.0;
    if (k.unshifted) {
        if (!nd.valid) return;
        const uint32_t pn = pidx(k, nd.x, nd.y, nd.z);
        accum_general<S>(src, k, pn, m0, mk);
        const double mo = (double)k.rho_b0 + m0 - mk;
        const bool bl = blue_kept(ldp(k.R, pn).x);
        store_fields_sums(PD, XR, k, nd.n, m0, bl ? mo : mk, bl ? mk : mo);
        return;
    }
    stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return rec_at<BC, true>(k, k.R, x, y, z); },
                                 [&](int x, int y, int z) { return rec_at<BC>(k, k.R, x, y, z); },
                           [&](int w, const float4& v) { win[w] = v; });
    if constexpr (S::kEqRef)
        stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return ref_at<BC, true>(k, x, y, z); },
                                     [&](int x, int y, int z) { return ref_at<BC>(k, x, y, z); },
                               [&](int w, const uint4& v) { put_ref<S, W>(rw, w, v); });
    __syncthreads();
    if (!nd.valid) return;
    float d[Q];
    pull_win<BC, S, TX, TY, W>(src, k, t, x_offsets<BC, typename S::T>(k, nd.x), rw, d);
    float x0 = 0.f, cf = 0.f, cv = 0.f;
    uint32_t bl = 0;
    // mass: exact FP64 sum of FP32 deviations; with 16-bit storage an FP32 sum
    // (its rounding is far below the storage rounding, and it is exact in the
    // pure phases, where the deviations vanish)
    using MassT = typename std::conditional<sizeof(typename S::T) == 4, double, float>::type;
    MassT ms = 0;
    accum_density_win<TX, TY, sizeof(typename S::T) == 2 && !S::kEqRef>(k, d, win, t.lx, t.ly, ms, x0, bl, cf, cv);
    m0 = (double)ms;
    const double rho = (double)k.rho_b0 + m0;
    mk = (double)x0 * rho + (double)(cf + (bl ? -cv : cv));
    store_fields_sums(PD, XR, k, nd.n, m0, bl ? rho - mk : mk, bl ? mk : rho - mk);
    if constexpr (MOMS) store_moments(MOM, k, (uint32_t)nd.z * k.plane + nd.q, (float)m0, d);
}

// Ends a basic block (the time level is never negative).  With contraction on the
// compiler chooses which product of a sum goes into a fused multiply-add, by what else
// the block holds; in a block of their own the pairs of directions kept that choice
// when the stores between them changed.  That is what one compiler does, not a property
// of the code: another may round differently, which is no less exact, but in 16-bit
// storage moves the fields of a run by up to 1e-3 of their size within 20 steps.
// Scalar branches, 10 per wave: no time that could be measured.
__device__ __forceinline__ void end_block(const KP& k)
{
    if (k.t < 0) asm volatile("s_nop 0");
}

// inlet cell (x, y) of the ghost plane of dst: the red equilibrium of the
// inflow in the directions that enter the lattice (c_z = 1), a pure red record
template <class S, int I = 0>
__device__ __forceinline__ void store_inlet(typename S::T* __restrict__ dst, const KP& k, int x, int y)
{
    if constexpr (I < Q) {
        if constexpr (kCZ[I] == 1)
            dst[((size_t)row_of(k, y, -1) * kSlots<S> + slot_of(I)) * (uint32_t)k.rs + x] =
                S::enc(inlet_feq_dir<I>(k, x, y, k.t) - wgt(I) * k.rho_b0);
        store_inlet<S, I + 1>(dst, k, x, y);
    }
}

// Jet: the outlet plane (z = nz - 1) by the convective condition, recorded in
// hcur for the collision, and (dst) the inlet cells of the ghost plane of the
// state the step writes, which depend on the time level only.  One plane, so
// the launch uses small blocks (OBLOCK lanes of one row) to spread the
// latency-bound work over many CUs.
constexpr int OBLOCK = 64;

template <class S>
__global__ __launch_bounds__(OBLOCK) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_outlet(const typename S::T* __restrict__ src, float2* __restrict__ PD,
                                                   float* __restrict__ XR, const float* __restrict__ hprev,
                                                   float* __restrict__ hcur, KP k, float* __restrict__ MOM,
                                                   typename S::T* __restrict__ dst, float4* __restrict__ Rout,
                                                   uint4* __restrict__ Qout)
{
    Node nd;
    nd.x = (int)(blockIdx.x * OBLOCK + threadIdx.x);
    nd.y = (int)blockIdx.y;
    nd.z = k.nz - 1;
    if (nd.x >= k.nx) return;
    nd.q = (uint32_t)nd.y * (uint32_t)k.nx + (uint32_t)nd.x;
    nd.valid = true;
    nd.n = nidx_of(k, nd.x, nd.y, nd.z);
    float d[Q], fr[Q], fb[Q];
    outlet_state<S>(src, k, hprev, nd, d, fr, fb);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        hcur[(size_t)i * k.plane + nd.q] = d[i];
        hcur[(size_t)(Q + i) * k.plane + nd.q] = fr[i];
    }
    const float2 v = store_fields(PD, XR, k, nd.n, d, fr);
    if (MOM) store_moments(MOM, k, (uint32_t)nd.z * k.plane + nd.q, v.y, d);
    if (dst && inlet_inside(k, nd.x, nd.y)) {
        store_inlet<S>(dst, k, nd.x, nd.y);
        const uint32_t g = nidx_of(k, nd.x, nd.y, -1);
        Rout[g] = make_float4(frac_tag(0.0, 1u), 0.f, 0.f, 0.f);  // pure red: x_b = 0
        if (S::kEqRef) Qout[g] = make_uint4(0u, 0u, 0u, 0u);  // zero record: the stored value is the deviation
    }
}

// ---------------------------------------------------------------- ghost shell
// Ghost cell g of the shell of a padded lattice (the adjoint's stencil
// cotangents): z faces (all x, y incl. ghosts), then y faces (z interior), then
// x faces (y, z interior).
struct Ghost {
    int x, y, z;
    bool valid;
};

__device__ __forceinline__ Ghost shell_cell(const KP& k, uint32_t g)
{
    Ghost c;
    const uint32_t A = (uint32_t)k.px * k.py, B = (uint32_t)k.px * k.nz, C = (uint32_t)k.ny * k.nz;
    c.valid = true;
    if (g < 2 * A) {
        const uint32_t f = g / A, r = g - f * A;
        c.x = (int)(r % k.px) - 1;
        c.y = (int)(r / k.px) - 1;
        c.z = f ? k.nz : -1;
    } else if (g < 2 * A + 2 * B) {
        const uint32_t h = g - 2 * A, f = h / B, r = h - f * B;
        c.x = (int)(r % k.px) - 1;
        c.z = (int)(r / k.px);
        c.y = f ? k.ny : -1;
    } else if (g < 2 * A + 2 * B + 2 * C) {
        const uint32_t h = g - 2 * A - 2 * B, f = h / C, r = h - f * C;
        c.y = (int)(r % k.ny);
        c.z = (int)(r / k.ny);
        c.x = f ? k.nx : -1;
    } else {
        c.valid = false;
        c.x = c.y = c.z = 0;
    }
    return c;
}

// ---------------------------------------------------------------- stencil
// isotropic gradients 3 sum_i w_i chi(x + c_i) c_i of phi and rho - rho_b0 at a
// node, accumulated over opposite pairs (i, i + 1) in FP64: g = (dphi[3], drho[3])
template <int BC, int I = 1>
__device__ __forceinline__ void gradients(const float2* __restrict__ pd, const KP& k, const Node& nd, double (&g)[6])
{
    if constexpr (I < Q) {
        constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
        const float2 a = pd_at<BC>(k, pd, nd.x + cx, nd.y + cy, nd.z + cz);
        const float2 b = pd_at<BC>(k, pd, nd.x - cx, nd.y - cy, nd.z - cz);
        const double dp = (double)a.x - (double)b.x, dr = (double)a.y - (double)b.y;
        constexpr double w3 = 3.0 * wgtd(I);
        if (cx) { g[0] += (w3 * cx) * dp; g[3] += (w3 * cx) * dr; }
        if (cy) { g[1] += (w3 * cy) * dp; g[4] += (w3 * cy) * dr; }
        if (cz) { g[2] += (w3 * cz) * dp; g[5] += (w3 * cz) * dr; }
        gradients<BC, I + 2>(pd, k, nd, g);
    }
}

// the same gradients from the LDS window of the (phi, rho) fields, in FP32 in the
// step: each pair difference chi(x + c_i) - chi(x - c_i) is exact for nearly equal
// values, the weighted sum of 13 of them is well conditioned
template <int TX, int TY, class T, int I = 1>
__device__ __forceinline__ void gradients_win(const float2* __restrict__ win, int lx, int ly, T (&g)[6])
{
    if constexpr (I < Q) {
        constexpr int cx = kCX[I], cy = kCY[I], cz = kCZ[I];
        const float2 a = win[wslot<TX, TY>(lx, ly, cx, cy, cz)];
        const float2 b = win[wslot<TX, TY>(lx, ly, -cx, -cy, -cz)];
        const T dp = (T)a.x - (T)b.x, dr = (T)a.y - (T)b.y;
        constexpr T w3 = T(3) * (std::is_same<T, double>::value ? (T)wgtd(I) : (T)wgt(I));
        if (cx) { g[0] += (w3 * cx) * dp; g[3] += (w3 * cx) * dr; }
        if (cy) { g[1] += (w3 * cy) * dp; g[4] += (w3 * cy) * dr; }
        if (cz) { g[2] += (w3 * cz) * dp; g[5] += (w3 * cz) * dr; }
        gradients_win<TX, TY, T, I + 2>(win, lx, ly, g);
    }
}

// one-dimensional inverse central-moment basis: for shift u, the vectors
// h0, h1 (and the constant h2 = (1/2, -1, 1/2)) over c = -1, 0, 1 whose
// central moments sum_c h_a(c) (c - u)^b are delta_ab (a, b = 0, 1, 2).
struct Basis1D {
    float h0[3], h1[3];  // index c + 1
    __device__ __forceinline__ explicit Basis1D(float u)
    {
        h0[1] = 1.f - u * u;
        h0[2] = 0.5f * (u * u + u);
        h0[0] = 0.5f * (u * u - u);
        h1[1] = -2.f * u;
        h1[2] = u + 0.5f;
        h1[0] = u - 0.5f;
    }
};
__device__ __forceinline__ constexpr float h2(int c) { return c == 0 ? -1.f : 0.5f; }

// Jet, bottom plane: the populations that left downwards since the last call
// (pair i ends a group of pairs), in the slots of their mirror images in the ghost
// cell below; not in the inlet.
template <int BC, class S, bool NT>
__device__ __forceinline__ void store_down(int i, const KP& k, uint32_t grow, bool gcell, const uint32_t (&vo)[3],
                                           uint32_t rsB, typename S::T* __restrict__ dst,
                                           const typename S::T (&down)[9])
{
    if (BC != LBM_BC_JET || !gcell) return;
    const auto rg = row_rsrc(dst + (size_t)grow * (kSlots<S> * (uint32_t)k.rs), kSlots<S> * (uint32_t)k.rs);
    const int first = i == 7 ? 3 : (i == 15 ? 11 : i);  // pairs 3..7 and 11..15 end together
#pragma unroll
    for (int p = 1; p < Q; p += 2) {
        if (p < first || p > i || kCZ[p] == 0) continue;
        const int s = kCZ[p] < 0 ? slot_of(p) : slot_of(p + 1);  // 3 (c_y + 1) + (c_x + 1), c_z = -1
        st_row<NT>(rg, vo[s % 3], (uint32_t)(s - s % 3 + 18) * rsB, down[s]);
    }
}

// Collision, perturbation and recolouring of one node from its pre-collision
// colour-blind deviations d, the centre values phic and xk (the tagged
// minority-colour fraction) and the gradients; writes the 27 post-collision
// colour-blind deviations to dst and (xk, V) of the recolouring to Rout (jet, on
// the bottom plane: also the mirrored ghost cell below).  FP64 only where a
// sum must be exact or an O(1) cancellation happens: the mass m0 and the
// equilibrium offsets E0, E1 (zero in the pure phases).  The momentum and the
// second moments are FP32 sums over opposite pairs (pair differences are exact
// for nearly equal populations, so the momentum of a fluid at rest is exactly
// zero).
template <int BC, class S, bool NT>
__device__ __forceinline__ void collide_store(const KP& k, const Node& nd, const float* d, float phic, float xk,
                                              const float (&g)[6], typename S::T* __restrict__ dst,
                                              float4* __restrict__ Rout, uint4* __restrict__ Qout)
{
    // the node's row, and lane offsets into the slots c_x = -1, 0, 1 of a group
    constexpr uint32_t B = sizeof(typename S::T);
    const uint32_t row = row_of(k, nd.y, nd.z), rsB = (uint32_t)k.rs * B;
    const auto rd = row_rsrc(dst + (size_t)row * (kSlots<S> * (uint32_t)k.rs), kSlots<S> * (uint32_t)k.rs);
    const uint32_t vo[3] = {(uint32_t)nd.x * B, rsB + (uint32_t)nd.x * B, 2 * rsB + (uint32_t)nd.x * B};
    // jet, bottom plane: the ghost cell below mirrors this node outside the inlet
    const bool bottom = BC == LBM_BC_JET && nd.z == 0;
    const uint32_t grow = BC == LBM_BC_JET ? row_of(k, nd.y, -1) : 0u;
    const bool gcell = bottom && !inlet_inside(k, nd.x, nd.y);
    // Scalar precision: FP64 for the mass sum and the equilibrium offsets with
    // FP32 storage (exact mass, no rounding bias in the pure phases at the
    // 1e-5 parity level); FP32 with 16-bit storage, whose own rounding is four
    // orders larger (the sum of 27 16-bit values is exact in FP32 but for the
    // widest exponent spreads).  It saved about 70 VALU
    // instructions per wave of the 16-bit kernels (858 now).
    using H = typename std::conditional<sizeof(typename S::T) == 4, double, float>::type;
    // raw moments of d up to second order
    H m0s = (H)d[0];
    float jx = 0.f, jy = 0.f, jz = 0.f;
    float pxx = 0.f, pyy = 0.f, pzz = 0.f, pxy = 0.f, pxz = 0.f, pyz = 0.f;
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        m0s += (H)d[i] + (H)d[i + 1];
        const float sp = d[i] + d[i + 1], df = d[i] - d[i + 1];
        if (kCX[i]) { jx += kCX[i] * df; pxx += sp; }
        if (kCY[i]) { jy += kCY[i] * df; pyy += sp; }
        if (kCZ[i]) { jz += kCZ[i] * df; pzz += sp; }
        if (kCX[i] * kCY[i]) pxy += (kCX[i] * kCY[i]) * sp;
        if (kCX[i] * kCZ[i]) pxz += (kCX[i] * kCZ[i]) * sp;
        if (kCY[i] * kCZ[i]) pyz += (kCY[i] * kCZ[i]) * sp;
    }
    const H m0d = m0s;
    const float m0 = (float)m0d;
    const float rhof = (float)((H)k.rho_b0 + m0d);
    // hardware reciprocals (1 ulp): the node quantities need no correctly
    // rounded division, and each IEEE division costs about ten instructions
    const float inv_rho = __builtin_amdgcn_rcpf(rhof);
    // interpolated properties (Sec. II): alpha_bar, harmonic nu_bar, s2nu
    const float hpf = 0.5f * (1.f + phic), hmf = 0.5f * (1.f - phic);
    const float nubf = __builtin_amdgcn_rcpf(hpf * k.inv_nu_r + hmf * k.inv_nu_b);
    const float s2 = __builtin_amdgcn_rcpf(3.f * nubf + 0.5f);
    const H hp = (H)0.5 * ((H)1 + (H)phic);
    const H abar = (H)k.alpha_b + hp * (H)k.dalpha;
    const H kap = (H)(27.0 / 19.0) * ((H)1 - abar);
    // equilibrium offsets in deviation form: E0 = rho abar - w_0 rho_b0, E1 = rho kappa - rho_b0
    const H E0 = (H)k.rho_b0 * (hp * (H)k.dalpha + (H)k.a_minus_w0) + m0d * abar;
    const H E1 = (H)k.rho_b0 * (-(H)(27.0 / 19.0) * hp * (H)k.dalpha + (H)k.kappa_b_m1) + m0d * kap;
    // body force (Eq. bodyForceJet) and velocity with the half-force term (Eq. Momentum)
    const float Fxf = m0 * k.gx, Fyf = m0 * k.gy, Fzf = m0 * k.gz;
    const float uxf = (jx + 0.5f * Fxf) * inv_rho, uyf = (jy + 0.5f * Fyf) * inv_rho, uzf = (jz + 0.5f * Fzf) * inv_rho;
    const float grxf = g[3], gryf = g[4], grzf = g[5];
    // second moments of f - f^(e) + F'/2 (its zeroth and first moments vanish, so
    // these are its central moments): sum f^(e) c_a c_b = iso + rho u_a u_b +
    // nu_bar (u_a dr_b + dr_a u_b); sum F' c_a c_b = u_a F_b + u_b F_a
    const float cxy = pxy - rhof * uxf * uyf - nubf * (uxf * gryf + grxf * uyf) + 0.5f * (uxf * Fyf + uyf * Fxf);
    const float cxz = pxz - rhof * uxf * uzf - nubf * (uxf * grzf + grxf * uzf) + 0.5f * (uxf * Fzf + uzf * Fxf);
    const float cyz = pyz - rhof * uyf * uzf - nubf * (uyf * grzf + gryf * uzf) + 0.5f * (uyf * Fzf + uzf * Fyf);
    const float cxx = pxx - rhof * uxf * uxf - 2.f * nubf * uxf * grxf + uxf * Fxf;
    const float cyy = pyy - rhof * uyf * uyf - 2.f * nubf * uyf * gryf + uyf * Fyf;
    const float czz = pzz - rhof * uzf * uzf - 2.f * nubf * uzf * grzf + uzf * Fzf;
    const float tr3 = (cxx + cyy + czz) * (1.f / 3.f);
    const float om = 1.f - s2;
    // relaxed deviatoric central moments, scaled by (1 - s2nu)
    const float kxy = om * cxy, kxz = om * cxz, kyz = om * cyz;
    const float kxx = om * (cxx - tr3), kyy = om * (cyy - tr3), kzz = om * (czz - tr3);
    const float u2 = uxf * uxf + uyf * uyf + uzf * uzf;
    const float udr = uxf * grxf + uyf * gryf + uzf * grzf;
    const float uF = uxf * Fxf + uyf * Fyf + uzf * Fzf;

    // FP32 per-direction part
    const float E1f = (float)E1;
    const float gpx = g[0], gpy = g[1], gpz = g[2];
    // back-projection of the relaxed moments: Delta(c) = sum_a U_a(cy, cz) h_a(cx, ux),
    // contracted axis by axis (z, then y, then x)
    const Basis1D bx(uxf), by(uyf), bz(uzf);
    float U0[3][3], U1[3][3], U2[3][3];
#pragma unroll
    for (int jz2 = 0; jz2 < 3; ++jz2) {
        const float A_ = kxy * bz.h0[jz2], B_ = kxz * bz.h1[jz2], C_ = kyz * bz.h1[jz2];
        const float D_ = kxx * bz.h0[jz2], E_ = kyy * bz.h0[jz2], G_ = kzz * h2(jz2 - 1);
#pragma unroll
        for (int jy2 = 0; jy2 < 3; ++jy2) {
            U1[jy2][jz2] = A_ * by.h1[jy2] + B_ * by.h0[jy2];
            U0[jy2][jz2] = C_ * by.h1[jy2] + E_ * h2(jy2 - 1) + G_ * by.h0[jy2];
            U2[jy2][jz2] = D_ * by.h0[jy2];
        }
    }
    // perturbation (squared projection, prefactor A) and recolouring weights
    const float G2 = gpx * gpx + gpy * gpy + gpz * gpz;
    const bool on = G2 > k.eps2;
    const float inv_gn = on ? __builtin_amdgcn_rsqf(G2) : 0.f;
    const float gn = G2 * inv_gn;
    const float Agn = k.A * gn, Aign = k.A * inv_gn;
    // recolouring vector V = beta (rho_r rho_b / rho) kappa n (x_r x_b = xk (1 - xk))
    const float rec = k.beta * xk * (1.f - xk) * rhof * (float)kap * inv_gn;
    const float4 rv = make_float4(xk, rec * gpx, rec * gpy, rec * gpz);
    st_rec(Rout, k, row, nd.x, rv);
    if (gcell) st_rec(Rout, k, grow, nd.x, mirror_rec(rv, 4));
    end_block(k);
    const float nub9 = 9.f * nubf;
    // referenced 16-bit storage: reference record of this node, rounded as stored
    float rt = 0.f, uxt = 0.f, uyt = 0.f, uzt = 0.f, et = 0.f;
    if constexpr (S::kEqRef) {
        const uint4 qr = enc_ref<S>(rhof, uxf, uyf, uzf, (float)E1);
        st_rec(Qout, k, row, nd.x, qr);
        if (gcell) st_rec(Qout, k, grow, nd.x, mirror_ref(qr, 4));
        end_block(k);
        const RefRec r = dec_ref<S>(qr);
        rt = r.rho;
        uxt = r.ux;
        uyt = r.uy;
        uzt = r.uz;
        et = r.e;
    }
    const float u2t = uxt * uxt + uyt * uyt + uzt * uzt;

    // rest population
    {
        const float w = wgt(0);
        const float de = (float)E0 - 1.5f * w * rhof * u2 - 3.f * nubf * udr;
        const float Fp = -3.f * w * uF;
        const float pert = on ? k.A * (10.f / 27.f) * gn : 0.f;
        const float delta = U0[1][1] * bx.h0[1] + U1[1][1] * bx.h1[1] + U2[1][1] * h2(0);
        const float dd = de + 0.5f * Fp + delta + pert;
        if constexpr (S::kEqRef) {
            const uint32_t b = __float_as_uint(dd);
            st_row<NT>(rd, vo[1], 12 * rsB, __builtin_bit_cast(typename S::T, (uint16_t)(b >> 16)));
            st_row<NT>(rd, vo[0], Q * rsB, __builtin_bit_cast(typename S::T, (uint16_t)(b & 0xffffu)));
        } else {
            st_row<NT>(rd, vo[1], 12 * rsB, S::enc(dd));
        }
    }
    // opposite pairs (i, i + 1): shared even parts, odd parts change sign.
    // Per direction (w_i factored out; cu = c.u, cr = c.grad rho, cF = c.F,
    // cg = c.grad phi):
    //   even = f^(e) even part + F'/2 even part + perturbation
    //        = K0 + cu (4.5 rho cu + 9 nu cr + 4.5 cF) + A/|g| cg^2,
    //          K0 = E1 - 1.5 rho u^2 - 1.5 u.F - A |g|,
    //   odd  = cu (K1 + 4.5 rho cu^2) + 1.5 cF,  K1 = rho (3 - 4.5 u^2)
    const float K0 = E1f - 1.5f * rhof * u2 - 1.5f * uF - Agn;
    const float K1 = rhof * (3.f - 4.5f * u2);
    const float r45 = 4.5f * rhof;
    typename S::T down[9];  // the populations that leave downwards (slots 0..8)
    // the order of one sum, for the same reason as end_block: which of its two terms is
    // rounded by itself follows what the compiler chose before the sum was written out
    constexpr bool kForceLast = sizeof(typename S::T) == 4 || S::kEqRef || BC == LBM_BC_PERIODIC;
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
        const float w = wgt(i);
        const float cu = cdot(i, uxf, uyf, uzf);
        const float cr = cdot(i, grxf, gryf, grzf);
        const float cF = cdot(i, Fxf, Fyf, Fzf);
        const float cg = cdot(i, gpx, gpy, gpz);
        const float t = r45 * cu + (kForceLast ? fmaf(4.5f, cF, nub9 * cr) : fmaf(nub9, cr, 4.5f * cF));
        const float even = w * (K0 + cu * t + (Aign * cg) * cg);
        const float odd = w * (cu * (K1 + r45 * (cu * cu)) + 1.5f * cF);
        // direction i (+c) and i + 1 (-c)
        const float dl_p = U0[cy + 1][cz + 1] * bx.h0[cx + 1] + U1[cy + 1][cz + 1] * bx.h1[cx + 1]
                           + U2[cy + 1][cz + 1] * h2(cx);
        const float dl_m = U0[1 - cy][1 - cz] * bx.h0[1 - cx] + U1[1 - cy][1 - cz] * bx.h1[1 - cx]
                           + U2[1 - cy][1 - cz] * h2(-cx);
        float dp = even + odd + dl_p;
        float dm = even - odd + dl_m;
        if constexpr (S::kEqRef) {
            // remove the reference's velocity part (even and odd in c)
            const float cut = cdot(i, uxt, uyt, uzt);
            const float re = w * (et + rt * (4.5f * cut * cut - 1.5f * u2t));
            const float ro = w * rt * cut * (3.f + 4.5f * cut * cut - 4.5f * u2t);
            dp -= re + ro;
            dm -= re - ro;
        }
        const uint32_t gp = (uint32_t)(9 * (cz + 1) + 3 * (cy + 1)), gm = (uint32_t)(9 * (1 - cz) + 3 * (1 - cy));
        const typename S::T ep = S::enc(dp), em = S::enc(dm);
        st_row<NT>(rd, vo[cx + 1], gp * rsB, ep);
        st_row<NT>(rd, vo[1 - cx], gm * rsB, em);
        if (cz < 0) down[slot_of(i)] = ep;
        if (cz > 0) down[slot_of(i + 1)] = em;
        if (cx != 0) {
            end_block(k);
            if (bottom) store_down<BC, S, NT>(i, k, grow, gcell, vo, rsB, dst, down);  // uniform
        }
    }
}


// ---------------------------------------------------------------- fused collide-recolour-stream
// A state above this size (the 256 MB memory-side cache), populations and recolouring
// records, has its populations written with non-temporal stores (the records with plain
// ones: no difference): nothing of it will be read from a cache in the next step, and
// the lines that the pulls share stay longer.  FP32 step 4.78 -> 4.68 ms (256x256x1024)
// and 0.584 -> 0.561 ms (128x128x512); 100^3 nodes (124 MB) keep the plain stores,
// 0.077 against 0.079 ms.  The reference records are not counted: BF16_EQ, 150^3 nodes,
// 359 us a step with plain stores, 366 without.
constexpr uint64_t kCacheBytes = 256ull << 20;

// waves per SIMD, measured on MI355X: four (at most 128 VGPRs) in FP32 and
// the referenced forms, 7 % faster than three in FP32 (five spill there);
// five for plain BF16 and FP16 (96 VGPRs, no spill), up to 9 % faster than
// four.  Jet: the outlet plane's pre-collision state is the one the density
// pass recorded.
// NT (non-temporal population stores): for states larger than the memory-side
// cache, see kCacheBytes.
template <class S>
constexpr int kCollideWaves = (sizeof(typename S::T) == 2 && !S::kEqRef) ? 5 : 4;

template <int BC, class S, class TL, bool NT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(kCollideWaves<S>, kCollideWaves<S>))) void
k_collide(
    const typename S::T* __restrict__ src, typename S::T* __restrict__ dst, const float2* __restrict__ PD,
    const float* __restrict__ XR, const float* __restrict__ hcur, float4* __restrict__ Rout, uint4* __restrict__ Qout,
    KP k)
{
    // the (phi, rho) stencil from an LDS window (measured faster than through
    // the caches, for the 16-bit forms too at their present occupancy)
    constexpr int TX = TL::CX, TY = TL::CY, W = TileShape<TX, TY>::W;
    __shared__ float2 win[W];
    __shared__ RefWin<S, W> rw;
    const Tile t = this_tile<TX, TY>(k);
    const Node& nd = t.nd;
    stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return pd_at<BC, true>(k, PD, x, y, z); },
                                 [&](int x, int y, int z) { return pd_at<BC>(k, PD, x, y, z); },
                           [&](int w, const float2& v) { win[w] = v; });
    if constexpr (S::kEqRef) {
        if (!k.unshifted)
            stage_window<TX, TY>(k, t, [&](int x, int y, int z) { return ref_at<BC, true>(k, x, y, z); },
                                         [&](int x, int y, int z) { return ref_at<BC>(k, x, y, z); },
                                   [&](int w, const uint4& v) { put_ref<S, W>(rw, w, v); });
    }
    __syncthreads();
    if (!nd.valid) return;
    float d[Q];
    if (BC == LBM_BC_JET && t.z == k.nz - 1) {
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = hcur[(size_t)i * k.plane + nd.q];
    } else if (k.unshifted) {
        float unused[Q];
        general_dirs<S, false>(src, k, pidx(k, nd.x, nd.y, nd.z), 0u, d, unused, unused);
    } else {
        pull_win<BC, S, TX, TY, W>(src, k, t, x_offsets<BC, typename S::T>(k, nd.x), rw, d);
    }
    const float xk = ldp(XR, nd.n);
    float g[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const float phic = win[wslot<TX, TY>(t.lx, t.ly, 0, 0, 0)].x;
    gradients_win<TX, TY>(win, t.lx, t.ly, g);
    collide_store<BC, S, NT>(k, nd, d, phic, xk, g, dst, Rout, Qout);
}


// ---------------------------------------------------------------- state in and out
// Initial state (general form): per-colour equilibria f^k_i = rho_k {varphi_i(alpha_k)
// + w_i [velocity terms of Eq. EES]} of the droplet / jet preset or of caller
// fields (node order), evaluated in FP64 and rounded once to the storage format.
template <class S>
__global__ __launch_bounds__(BLOCK) void k_init(typename S::T* __restrict__ dst, float4* __restrict__ Rw, KP k,
                                                 int kind,
                                                 const float* __restrict__ frr, const float* __restrict__ frb,
                                                 const float* __restrict__ fu, double dcx, double dcy, double dcz,
                                                 double R, double W, double rho_r0, double rho_b0, double alpha_r,
                                                 double alpha_b, double rho_ref)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const uint32_t u_idx = (uint32_t)nd.z * k.plane + nd.q;
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
        rr = frr[u_idx];
        rb = frb[u_idx];
        if (fu) {
            ux = fu[3 * (size_t)u_idx];
            uy = fu[3 * (size_t)u_idx + 1];
            uz = fu[3 * (size_t)u_idx + 2];
        }
    }
    const double u2 = ux * ux + uy * uy + uz * uz;
    const double kap_r = 27.0 * (1.0 - alpha_r) / 19.0, kap_b = 27.0 * (1.0 - alpha_b) / 19.0;
    const uint32_t bl = rr > rb;  // planes Q..2Q-1 keep the minority colour
    const uint32_t pn = pidx(k, nd.x, nd.y, nd.z);
    stp(Rw, pn, make_float4(frac_tag(0.0, bl), 0.f, 0.f, 0.f));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double w = wgtd(i);
        const double cu = kCX[i] * ux + kCY[i] * uy + kCZ[i] * uz;
        const double poly = 3.0 * cu + 4.5 * cu * cu - 1.5 * u2 + 4.5 * cu * cu * cu - 4.5 * cu * u2;
        double fv, fb;
        if (i == 0) {
            fv = rr * (alpha_r + w * poly);
            fb = rb * (alpha_b + w * poly);
        } else {
            fv = rr * w * (kap_r + poly);
            fb = rb * w * (kap_b + poly);
        }
        const double dv = (fv + fb) - w * rho_ref;  // deviation from the kernels' reference density
        stp(dst + (size_t)i * k.NP, pn, S::enc((float)dv));
        stp(dst + (size_t)(Q + i) * k.NP, pn, S::enc((float)(bl ? fb : fv)));
    }
}

// set an explicit (fr, fb) FP32 state (node order), general form: d formed in
// FP64 and rounded once, and the populations of the node's minority colour
// (flagged in Rw)
template <class S>
__global__ __launch_bounds__(BLOCK) void k_set_state(typename S::T* __restrict__ dst, float4* __restrict__ Rw, KP k,
                                                      const float* __restrict__ st, double rho_b0)
{
    const Node nd = this_node(k);
    if (!nd.valid) return;
    const size_t N = k.N;
    const uint32_t u_idx = (uint32_t)nd.z * k.plane + nd.q;
    double rr = 0.0, rb = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        rr += (double)st[(size_t)i * N + u_idx];
        rb += (double)st[(size_t)(Q + i) * N + u_idx];
    }
    const uint32_t bl = rr > rb;
    const uint32_t pn = pidx(k, nd.x, nd.y, nd.z);
    stp(Rw, pn, make_float4(frac_tag(0.0, bl), 0.f, 0.f, 0.f));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const float fr = st[(size_t)i * N + u_idx], fb = st[(size_t)(Q + i) * N + u_idx];
        const double dv = ((double)fr + (double)fb) - wgtd(i) * rho_b0;
        stp(dst + (size_t)i * k.NP, pn, S::enc((float)dv));
        stp(dst + (size_t)(Q + i) * k.NP, pn, S::enc(bl ? fb : fr));
    }
}

// The kernels that read a state node by node (macroscopic fields, get_state, the first
// pass of the diagnostics) take the tiles of the fused collision, the records R of the
// neighbours from an LDS window, or NodeBlocks, where every lane has a row of its own
// and the records come through the caches, for rows that leave too many lanes of a tile
// idle (see read_form).
template <class TL>
constexpr int kRecWin = TL::kFlat ? 1 : TileShape<TL::CX, TL::CY>::W;

// the tile of this block and its window, or this thread's node
template <int BC, class TL>
__device__ __forceinline__ Tile state_tile(const KP& k, float4* __restrict__ win)
{
    if constexpr (TL::kFlat) {
        Tile t{};
        t.nd = this_node(k);
        t.z = t.nd.z;
        return t;
    } else {
        const Tile t = this_tile<TL::CX, TL::CY>(k);
        if (!k.unshifted)
            stage_window<TL::CX, TL::CY>(k, t, [&](int x, int y, int z) { return rec_at<BC, true>(k, k.R, x, y, z); },
                                         [&](int x, int y, int z) { return rec_at<BC>(k, k.R, x, y, z); },
                                   [&](int w, const float4& v) { win[w] = v; });
        __syncthreads();
        return t;
    }
}

// record R of the source of direction I
template <int BC, class TL, int I>
__device__ __forceinline__ float4 source_rec(const KP& k, const Tile& t, const XOff& xo, const float4* __restrict__ win)
{
    if constexpr (TL::kFlat) {
        int m;
        const float4 r = pull_rec<BC, I, false>(k.R, k, t.nd.y, t.nd.z, xo, m);
        return BC == LBM_BC_JET ? mirror_rec(r, m) : r;
    } else {
        return win[wslot<TL::CX, TL::CY>(t.lx, t.ly, -kCX[I], -kCY[I], -kCZ[I])];
    }
}

template <int BC, class S, class TL, int I = 0>
__device__ __forceinline__ void state_dirs(const typename S::T* __restrict__ src, const KP& k, const Tile& t,
                                           const XOff& xo, const float4* __restrict__ win, float* d, float* fr,
                                           float* fb)
{
    if constexpr (I < Q) {
        d[I] = pull_dev<BC, S, I, !TL::kFlat>(src, k, t.nd.x, t.nd.y, t.nd.z, xo);
        colours_of<I>(k, d[I], source_rec<BC, TL, I>(k, t, xo, win), fr[I], fb[I]);
        state_dirs<BC, S, TL, I + 1>(src, k, t, xo, win, d, fr, fb);
    }
}

template <int BC, class S, class TL>
__device__ __forceinline__ void read_state(const typename S::T* __restrict__ src, const KP& k,
                                           const float* __restrict__ hprev, const Tile& t,
                                           const float4* __restrict__ win, float* d, float* fr, float* fb)
{
    const Node& nd = t.nd;
    if (BC == LBM_BC_JET && nd.z == k.nz - 1)
        outlet_state<S, !TL::kFlat>(src, k, hprev, nd, d, fr, fb);
    else if (k.unshifted)
        pull_all<BC, S, true, !TL::kFlat>(src, k, nd.x, nd.y, nd.z, d, fr, fb);
    else
        state_dirs<BC, S, TL>(src, k, t, x_offsets<BC, typename S::T>(k, nd.x), win, d, fr, fb);
}

// current state as (fr, fb) FP32 in node order
template <int BC, class S, class TL>
__global__ __launch_bounds__(BLOCK) void k_get_state(const typename S::T* __restrict__ src,
                                                      const float* __restrict__ hprev, KP k, float* __restrict__ st,
                                                      double rho_b0)
{
    __shared__ float4 win[kRecWin<TL>];
    const Tile t = state_tile<BC, TL>(k, win);
    const Node& nd = t.nd;
    if (!nd.valid) return;
    const size_t N = k.N;
    const uint32_t u_idx = (uint32_t)nd.z * k.plane + nd.q;
    float d[Q], fr[Q], fb[Q];
    read_state<BC, S, TL>(src, k, hprev, t, win, d, fr, fb);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        st[(size_t)i * N + u_idx] = fr[i];
        st[(size_t)(Q + i) * N + u_idx] = fb[i];
    }
}

// FP64 sums over the directions of a shifted state: the mass m0 = rho - rho_b0, the
// momentum and the kept colour's mass mk; marks has bit 0 set where every source
// kept blue, bit 1 where any did.
template <int BC, class TL, int I = 0>
__device__ __forceinline__ void mass_dirs(const KP& k, const Tile& t, const XOff& xo, const float4* __restrict__ win,
                                          const float* d, double& m0, double& mk, double (&j)[3], uint32_t& marks)
{
    if constexpr (I < Q) {
        const float4 r = source_rec<BC, TL, I>(k, t, xo, win);
        const uint32_t bl = blue_kept(r.x);
        const float f = d[I] + wgt(I) * k.rho_b0;
        const float vt = I == 0 ? 0.f : (wgt(I) * inv_len(I)) * cdot(I, r.y, r.z, r.w);
        mk += (double)(r.x * f + (bl ? -vt : vt));
        marks = (marks & (bl | 2u)) | (bl << 1);
        m0 += (double)d[I];
        if (kCX[I]) j[0] += kCX[I] * (double)d[I];
        if (kCY[I]) j[1] += kCY[I] * (double)d[I];
        if (kCZ[I]) j[2] += kCZ[I] * (double)d[I];
        if (!TL::kFlat && I % 3 == 2) __builtin_amdgcn_sched_barrier(0);
        mass_dirs<BC, TL, I + 1>(k, t, xo, win, d, m0, mk, j, marks);
    }
}

template <int BC, class TL, int I = 0>
__device__ __forceinline__ void mixed_masses(const KP& k, const Tile& t, const XOff& xo,
                                             const float4* __restrict__ win, const float* d, double& rr, double& rb)
{
    if constexpr (I < Q) {
        float fr, fb;
        colours_of<I>(k, d[I], source_rec<BC, TL, I>(k, t, xo, win), fr, fb);
        rr += (double)fr;
        rb += (double)fb;
        if (I % 3 == 2) __builtin_amdgcn_sched_barrier(0);
        mixed_masses<BC, TL, I + 1>(k, t, xo, win, d, rr, rb);
    }
}

// Masses (m0 = rho - rho_b0, rho_r, rho_b) and momentum of a node in FP64.  Where all
// sources kept the same colour, which is everywhere but next to phi = 0, its mass is
// the sum of the kept values and the other colour the rest; else both colours are
// rebuilt direction by direction.
template <int BC, class S, class TL>
__device__ __forceinline__ void node_masses(const typename S::T* __restrict__ src, const KP& k,
                                            const float* __restrict__ hprev, const Tile& t,
                                            const float4* __restrict__ win, double& m0, double& rr, double& rb,
                                            double (&j)[3])
{
    m0 = rr = rb = j[0] = j[1] = j[2] = 0.0;
    const Node& nd = t.nd;
    if (!TL::kFlat && !k.unshifted && !(BC == LBM_BC_JET && nd.z == k.nz - 1)) {
        float d[Q], unused[Q];
        double mk = 0.0;
        uint32_t marks = 1u;
        const XOff xo = x_offsets<BC, typename S::T>(k, nd.x);
        pull_dirs<BC, S, false, !TL::kFlat>(src, k, nd.x, nd.y, nd.z, xo, d, unused, unused);
        mass_dirs<BC, TL>(k, t, xo, win, d, m0, mk, j, marks);
        const double other = (double)k.rho_b0 + m0 - mk;
        rr = marks ? other : mk;
        rb = marks ? mk : other;
        if (marks == 2u) {  // mixed
            rr = rb = 0.0;
            mixed_masses<BC, TL>(k, t, xo, win, d, rr, rb);
        }
        return;
    }
    float d[Q], fr[Q], fb[Q];
    read_state<BC, S, TL>(src, k, hprev, t, win, d, fr, fb);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        m0 += (double)d[i];
        rr += (double)fr[i];
        rb += (double)fb[i];
        if (kCX[i]) j[0] += kCX[i] * (double)d[i];
        if (kCY[i]) j[1] += kCY[i] * (double)d[i];
        if (kCZ[i]) j[2] += kCZ[i] * (double)d[i];
    }
}

// macroscopic fields (node order) and FP64 audit partial sums (one slot per block)
template <int BC, class S, class TL>
__global__ __launch_bounds__(BLOCK) void k_macro(const typename S::T* __restrict__ src,
                                                  const float* __restrict__ hprev, KP k, float* __restrict__ o_rr,
                                                  float* __restrict__ o_rb, float* __restrict__ o_u,
                                                  float* __restrict__ o_phi, double* __restrict__ partials)
{
    __shared__ float4 win[kRecWin<TL>];
    const Tile t = state_tile<BC, TL>(k, win);
    const Node& nd = t.nd;
    double acc[5] = {0, 0, 0, 0, 0};
    if (nd.valid) {
        double m0, rr, rb, j[3];
        node_masses<BC, S, TL>(src, k, hprev, t, win, m0, rr, rb, j);
        const double rho = (double)k.rho_b0 + m0;
        const double px = j[0] + 0.5 * m0 * k.gx, py = j[1] + 0.5 * m0 * k.gy, pz = j[2] + 0.5 * m0 * k.gz;
        const size_t n = (size_t)nd.z * k.plane + nd.q;
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

__global__ __launch_bounds__(BLOCK) void k_audit_final(const double* __restrict__ partials, int nblk,
                                                        double* __restrict__ out)
{
    double acc[5] = {0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < nblk; b += BLOCK)
#pragma unroll
        for (int a = 0; a < 5; ++a) acc[a] += partials[(size_t)b * 5 + a];
    __shared__ double red[5][4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < 5; ++a) {
        const double s = wave_sum(acc[a]);
        if (lane == 0) red[a][wv] = s;
    }
    __syncthreads();
    if (threadIdx.x < 5)
        out[threadIdx.x] = red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] + red[threadIdx.x][3];
}

}  // namespace cglbm
