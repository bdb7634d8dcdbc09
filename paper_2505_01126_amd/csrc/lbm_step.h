#pragma once

// Device code of one accLB time step (arXiv 2505.01126, Secs. 2-3): the fused
// step kernel and everything it is built from.
//
// k_step fuses, per lattice site and time step:
//   pull-streaming of the 27 D3Q27 populations (structure of arrays, one
//   coalesced row per direction), their moments, the phase-field stencils (LDS-staged phi tile),
//   the forces of Eq. (8), the regularised collision of Eqs. (6)-(7) rebuilt
//   from p*, u and a^(2) (each site writes only its own slots, Sec. 3), and the
//   conservative Allen-Cahn update of Eq. (3).
//
// Populations are stored as h_i = f_i / w_i - P0 in FP32, FP16 or BF16, plane
// by plane: population i of site (x, y, z) at ((z * 27 + i) * ny + y) * nx + x,
// so the 27 rows a site reads or writes lie within 3 x 27 planes and are
// addressed from one per-plane base pointer with 32-bit offsets; all
// arithmetic is FP32.  Each phase-field flux through a face or lattice link is
// evaluated by contraction-free code from identical operands on both sides of
// the link (or once, shared through LDS), so the two sites see bit-identical
// values; the fluxes are accumulated in FP64 into the FP64 phi, so sum phi is
// conserved to FP64 round-off, or, with the int32 fixed-point phi, rounded
// once each to the fixed-point grid and summed exactly, so sum phi is
// conserved bit for bit.
//
// Instruction economy: the D3Q27 weights are a tensor product,
// w(c) = w1(cx) w1(cy) w1(cz) with w1(0) = 2/3, w1(+-1) = 1/6, so the moments
// up to second order (of the populations and of the phi stencil) are computed
// axis by axis, and the post-collision populations, a quadratic polynomial in
// c, are generated the same way.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm_internal.h"
#include "lbm_mlp_device.h"

namespace lbm {

// ------------------------------------------------------------------ lattice
// D3Q27 velocity i: c = (i % 3 - 1, (i / 3) % 3 - 1, i / 9 - 1); rest = 13; -c_i = c_{26-i}
__host__ __device__ constexpr int CX(int i) { return i % 3 - 1; }
__host__ __device__ constexpr int CY(int i) { return (i / 3) % 3 - 1; }
__host__ __device__ constexpr int CZ(int i) { return i / 9 - 1; }
__host__ __device__ constexpr int C2(int i) { return CX(i) * CX(i) + CY(i) * CY(i) + CZ(i) * CZ(i); }
__host__ __device__ constexpr float WT(int i)
{
    return C2(i) == 0 ? 8.0f / 27.0f : C2(i) == 1 ? 2.0f / 27.0f : C2(i) == 2 ? 1.0f / 54.0f : 1.0f / 216.0f;
}
__host__ __device__ constexpr double WTD(int i)
{
    return C2(i) == 0 ? 8.0 / 27.0 : C2(i) == 1 ? 2.0 / 27.0 : C2(i) == 2 ? 1.0 / 54.0 : 1.0 / 216.0;
}

// ----------------------------------------------------------------- storage
template <int S> struct Pop;
// enc: round to nearest even (the initial state); enc_step: the encode of the
// step's post-collision values, given the bits of another population of the
// same site as a source of dither (used by BF16 only).
template <> struct Pop<0> {
    using T = float;
    __device__ static float dec(T v) { return v; }
    __device__ static T enc(float v) { return v; }
    __device__ static T enc_step(float v, uint32_t) { return v; }
};
template <> struct Pop<1> {
    using T = _Float16;
    __device__ static float dec(T v) { return (float)v; }
    __device__ static T enc(float v)  // round to nearest even
    {
        // the conversion is an instruction of its own: the compiler could
        // otherwise fuse the multiply-add that produced v into it (one
        // rounding instead of two) in some template variants and not in
        // others, and the variants would no longer agree bit for bit
        uint32_t r;
        asm("v_cvt_f16_f32 %0, %1" : "=v"(r) : "v"(v));
        return __builtin_bit_cast(T, (uint16_t)r);
    }
    __device__ static T enc_step(float v, uint32_t) { return enc(v); }
};
template <> struct Pop<2> {
    using T = __bf16;
    __device__ static float dec(T v) { return (float)v; }
    __device__ static T enc(float v)  // round to nearest even
    {
        // an instruction of its own, as for FP16 (the low half of the packed
        // conversion of (v, 0))
        uint32_t r;
        asm("v_cvt_pk_bf16_f32 %0, %1, 0" : "=v"(r) : "v"(v));
        return __builtin_bit_cast(T, (uint16_t)r);
    }
    // Stochastic rounding: a BF16 ulp of a shifted population (|h| ~ 0.03) is
    // about 1e-4, far above the change that a weak body force makes in one
    // step, so rounding to nearest drops that change at every step and the
    // flow drifts.  Adding 16 dither bits below the kept mantissa before
    // cutting them off rounds up with probability equal to the cut fraction,
    // so the change survives in expectation.  The dither is the low 16 bits
    // of another population of the site (their low mantissa bits are close to
    // uniform): deterministic, with no state, the same bits in every kernel
    // variant.  A NaN stays a NaN; a value within a dither of the largest
    // finite one may round to infinity.
    __device__ static T enc_step(float v, uint32_t dither)
    {
        const uint32_t b = __builtin_bit_cast(uint32_t, v) + (dither & 0xffffu);
        return __builtin_bit_cast(T, (uint16_t)(b >> 16));
    }
};

__device__ __forceinline__ int wrapi(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }
__device__ __forceinline__ int modi(int v, int n)
{
    v %= n;
    return v < 0 ? v + n : v;
}

// Pointers into global memory.  Kernel arguments are known to be global; a
// pointer read from a descriptor table (the batch kernel) is generic, and
// generic (flat) accesses also count against the LDS wait counter, so every
// LDS wait would then wait for the prefetches too.  These casts restore global
// addressing.
#define LBM_GLOBAL __attribute__((address_space(1)))
template <class T> __device__ __forceinline__ const LBM_GLOBAL T *gconst(const T *p)
{
    return (const LBM_GLOBAL T *)p;
}
template <class T> __device__ __forceinline__ LBM_GLOBAL T *gmut(T *p) { return (LBM_GLOBAL T *)p; }

// Phase-field storage of the step: FP64 (fluxes summed in FP64), or int32
// fixed point q = phi 2^30 (each flux rounded to nearest on that grid, summed
// in wrapping 32-bit integers, so the two sites of a link add and subtract
// exactly the same integer).
template <bool FX> struct PhiStore;
template <> struct PhiStore<false> {
    using T = double;    // stored value
    using Acc = double;  // flux accumulator
    __device__ static float f32(T v) { return (float)v; }
    __device__ static Acc flux(float f) { return (double)f; }
    __device__ static T add(T phi, Acc d) { return phi + d; }
};
template <> struct PhiStore<true> {
    using T = int32_t;
    using Acc = uint32_t;
    __device__ static float f32(T q) { return (float)q * 0x1p-30f; }
    __device__ static Acc flux(float f) { return (uint32_t)(int32_t)__builtin_rintf(f * 0x1p30f); }
    __device__ static T add(T q, Acc d) { return (int32_t)((uint32_t)q + d); }
};

// Raw buffer access to one z plane of a field (of populations: 27 rows of
// nx * ny): row offsets go in the scalar offset, the offset in the row in the
// vector offset, so no vector address arithmetic is needed.  (Global loads with
// the same scalar base took a 64-bit vector addition and two registers per
// address: the compiler extends the offsets to 64 bits outside the loop.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <class T> __device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
}
// Stores of the step's outputs may be non-temporal (cache policy nt): nothing
// reads them before the next launch, by which time a 512^3 state has long left
// L2 and the Infinity Cache, so caching them only evicts input lines that
// neighbouring work items still fetch (measured 2-4 % faster per step on
// 512^3).  The step uses them for the boxes whose tile rows cover whole 128-byte
// lines (a partial line written past the caches measured slower: a batch of
// boxes with edges 32-96, 8 %) where the batch's populations exceed the Infinity
// Cache, which otherwise holds them for the next step.  (In a batch with both kinds
// of box each kind is a launch of its own: a policy per box inside one launch
// doubles the plane loop, which then spilled 20-80 registers.)  Loads keep the default
// policy: non-temporal loads measured slower.
constexpr int STORE_NT = 2;
template <class T, int AUX = 0>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, T v)
{
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, AUX);
    else if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, voff, soff, AUX);
}
// ------------------------------------------------------ separable moments
// Ten sums M_abc = 216 sum_c w(c) v(c) cx^a cy^b cz^c (a + b + c <= 2) of 27
// lattice-ordered values, taken axis by axis (x, then y, then z); along each
// axis the weights are (1, 4, 1) = 6 w1.
struct M10 {
    float m000, m100, m010, m001, m200, m020, m002, m110, m101, m011;
};

// The sums over one z plane of the 3 x 3 x 3 stencil (rows of cy = -1, 0, 1):
// p_ab = sum over the plane with weights cx^a cy^b.
struct P6 {
    float p00, p01, p02, p10, p11, p20;
};
__device__ __forceinline__ void plane6(const float *v, P6 &p)
{
    float r0[3], r1[3], r2[3];
#pragma unroll
    for (int row = 0; row < 3; row++) {
        const float vm = v[3 * row], v0 = v[3 * row + 1], vp = v[3 * row + 2];
        r2[row] = vp + vm;
        r1[row] = vp - vm;
        r0[row] = fmaf(4.0f, v0, r2[row]);
    }
    p.p02 = r0[2] + r0[0];
    p.p00 = fmaf(4.0f, r0[1], p.p02);
    p.p01 = r0[2] - r0[0];
    p.p10 = fmaf(4.0f, r1[1], r1[2] + r1[0]);
    p.p11 = r1[2] - r1[0];
    p.p20 = fmaf(4.0f, r2[1], r2[2] + r2[0]);
}
// the ten sums from the plane sums below (a), at (b) and above (c)
__device__ __forceinline__ void planes10(const P6 &a, const P6 &b, const P6 &c, M10 &M)
{
    M.m002 = c.p00 + a.p00;
    M.m000 = fmaf(4.0f, b.p00, M.m002);
    M.m001 = c.p00 - a.p00;
    M.m010 = fmaf(4.0f, b.p01, c.p01 + a.p01);
    M.m011 = c.p01 - a.p01;
    M.m020 = fmaf(4.0f, b.p02, c.p02 + a.p02);
    M.m100 = fmaf(4.0f, b.p10, c.p10 + a.p10);
    M.m101 = c.p10 - a.p10;
    M.m110 = fmaf(4.0f, b.p11, c.p11 + a.p11);
    M.m200 = fmaf(4.0f, b.p20, c.p20 + a.p20);
}
__device__ __forceinline__ void moments10(const float (&v)[27], M10 &M)
{
    P6 p[3];
#pragma unroll
    for (int z = 0; z < 3; z++) plane6(v + 9 * z, p[z]);
    planes10(p[0], p[1], p[2], M);
}

// ------------------------------------------------------- per-site physics
struct Macro {
    float dp;     // p* - P0
    float rho;
    float u[3];   // u = j + a/2
    float a[3];   // F / rho
    float S[6];   // Pi - p* c_s^2 I  (xx yy zz xy xz yz)
    float omega;  // 1 / tau at this site
};

// Phase-field stencil quantities at a site: g = grad phi, H = Hessian (lattice
// stencils of Sec. 2.3): g = M1 / 72, H_aa = (M_aa - M000/3) / 24, H_ab = M_ab / 24.
struct PhiGrad {
    float phi, g[3], H[6];
};

__device__ __forceinline__ void phi_grad(const M10 &M, float phi, PhiGrad &G)
{
#pragma clang fp contract(off)
    const float k1 = 1.0f / 72.0f, k2 = 1.0f / 24.0f, third = -1.0f / 3.0f;
    G.phi = phi;
    G.g[0] = M.m100 * k1;
    G.g[1] = M.m010 * k1;
    G.g[2] = M.m001 * k1;
    G.H[0] = fmaf(third, M.m000, M.m200) * k2;
    G.H[1] = fmaf(third, M.m000, M.m020) * k2;
    G.H[2] = fmaf(third, M.m000, M.m002) * k2;
    G.H[3] = M.m110 * k2;
    G.H[4] = M.m101 * k2;
    G.H[5] = M.m011 * k2;
}
__device__ __forceinline__ void phi_stencil(const float (&ph)[27], M10 &M, PhiGrad &G)
{
    moments10(ph, M);
    phi_grad(M, ph[13], G);
}

// Surface-tension force with the finite-difference curvature (Sec. 2.3 CSF
// form): F^s = -(3 delta/2) sigma K |g| g, with K |g| = tr H - g.H.g / |g|^2
// (K = div n, n = g/|g| toward phi = 1); zero where |g| <= 1e-12.
// surface_coef gives the factor of g.
// The roundings are written out (contraction-free), so that every kernel forms
// the same bits; with the learned curvature (ML) |g|^2 and tr H are those of
// its criterion.
template <bool ML> __device__ __forceinline__ float surface_coef(const M10 &M, const PhiGrad &G, const Params &P)
{
#pragma clang fp contract(off)
    const float *g = G.g, *H = G.H;
    const float k2 = 1.0f / 24.0f, third = -1.0f / 3.0f;
    const float g2 = ML ? g[0] * g[0] + g[1] * g[1] + g[2] * g[2] : fmaf(g[2], g[2], fmaf(g[0], g[0], g[1] * g[1]));
    float cs = 0.f;
    if (g2 > 1e-24f) {
        const float trH = ML ? (H[0] + H[1]) + H[2]
                             : fmaf(k2, fmaf(third, M.m000, M.m002), fmaf(k2, fmaf(third, M.m000, M.m200), H[1]));
        const float hx = fmaf(H[4], g[2], fmaf(H[3], g[1], H[0] * g[0]));
        const float hy = fmaf(H[5], g[2], fmaf(H[3], g[0], H[1] * g[1]));
        const float hz = fmaf(H[2], g[2], fmaf(H[4], g[0], H[5] * g[1]));
        const float gHg = fmaf(g[2], hz, fmaf(g[0], hx, g[1] * hy));
        cs = -P.fs_coef * fmaf(-__builtin_amdgcn_rcpf(g2), gHg, trH);
    }
    return cs;
}
// Learned curvature: K_FD and |g| at the site, and whether the network is
// consulted (interface cell 0.02 < phi < 0.98 with |K_FD| > k_lo).
// (The learned-curvature helpers are contraction-free, so that every inlined
// copy -- single-box and batch kernels -- rounds identically.)
__device__ __forceinline__ float grad_norm(const PhiGrad &G)
{
#pragma clang fp contract(off)
    return sqrtf(G.g[0] * G.g[0] + G.g[1] * G.g[1] + G.g[2] * G.g[2]);
}
__device__ __forceinline__ bool mlp_select(const PhiGrad &G, const Params &P, float &kfd, float &gn)
{
#pragma clang fp contract(off)
    const float *g = G.g, *H = G.H;
    const float g2 = g[0] * g[0] + g[1] * g[1] + g[2] * g[2];
    kfd = 0.f;
    gn = 0.f;
    if (!(g2 > 1e-24f)) return false;
    const float trH = H[0] + H[1] + H[2];
    const float gHg = g[0] * (H[0] * g[0] + H[3] * g[1] + H[4] * g[2]) +
                      g[1] * (H[3] * g[0] + H[1] * g[1] + H[5] * g[2]) +
                      g[2] * (H[4] * g[0] + H[5] * g[1] + H[2] * g[2]);
    gn = sqrtf(g2);
    kfd = (trH - gHg / g2) / gn;
    return G.phi > 0.02f && G.phi < 0.98f && fabsf(kfd) > P.k_lo;
}

// Blend of the network output y = (K, n) with the finite-difference K and n:
// s = smoothstep((|K_FD| - k_lo) / (k_hi - k_lo)), K = s K_net + (1 - s) K_FD,
// n_s = normalise(s n_net/|n_net| + (1 - s) g/|g|), F^s = -(3 delta/2) sigma K |g|^2 n_s;
// the finite-difference force (cs_fd g) is kept when the output is non-finite
// or |n_net| is outside [0.5, 1.5].
__device__ __forceinline__ void surface_blend(const PhiGrad &G, float cs_fd, const Params &P, float kfd, float gn,
                                              const float (&y)[4], float (&fs)[3])
{
#pragma clang fp contract(off)
    const float nn = sqrtf(y[1] * y[1] + y[2] * y[2] + y[3] * y[3]);
    if (!(isfinite(y[0]) && isfinite(nn) && nn >= 0.5f && nn <= 1.5f)) {
#pragma unroll
        for (int a = 0; a < 3; a++) fs[a] = cs_fd * G.g[a];
        return;
    }
    const float t = fminf((fabsf(kfd) - P.k_lo) / (P.k_hi - P.k_lo), 1.0f);
    const float sw = t * t * (3.0f - 2.0f * t);
    const float K = sw * y[0] + (1.0f - sw) * kfd;
    float b[3], bn2 = 0.f;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        b[a] = sw * y[1 + a] / nn + (1.0f - sw) * G.g[a] / gn;
        bn2 += b[a] * b[a];
    }
    const float bn = sqrtf(bn2);
    const float c = -P.fs_coef * K * gn * gn;
#pragma unroll
    for (int a = 0; a < 3; a++) fs[a] = c * (bn > 1e-12f ? b[a] / bn : G.g[a] / gn);
}

// Forces of Eq. (8) and the velocity u = j + a/2 from the moments M of the
// pulled populations h_i = f_i / w_i - P0 (Sec. 2.2); fs is the surface-tension force.
//   F^p = -p* c_s^2 grad rho,  grad rho = (rho_l - rho_g) g
//   F^b = rho a_ext
//   F^nu = -(nu / (tau c_s^2)) (Pi - p* c_s^2 I - u0 u0) grad rho, u0 = j + (F^s + F^p + F^b)/(2 rho)
// PH: buoyancy and the phase-dependent relaxation time are compiled in (each
// still switched by its parameter); without them the step keeps one tau.
template <bool TP, bool PH = true>
__device__ __forceinline__ void site_macro(const M10 &M, const PhiGrad &G, const float (&fs)[3],
                                           const float (&aext)[3], const Params &P, Macro &m)
{
    const float r = 1.0f / 216.0f;
    m.dp = M.m000 * r;
    float j[3] = {M.m100 * r, M.m010 * r, M.m001 * r};
    const float pc = m.dp * (1.0f / 3.0f);
    m.S[0] = fmaf(M.m200, r, -pc);
    m.S[1] = fmaf(M.m020, r, -pc);
    m.S[2] = fmaf(M.m002, r, -pc);
    m.S[3] = M.m110 * r;
    m.S[4] = M.m101 * r;
    m.S[5] = M.m011 * r;
    if constexpr (TP) {
        const float rho = P.rho_g + (P.rho_l - P.rho_g) * G.phi;
        const float *g = G.g;
        const float drho = P.rho_l - P.rho_g;
        const float cp = -(P.p0 + m.dp) * (1.0f / 3.0f) * drho;  // F^p = cp * g
        const float inv_rho = __builtin_amdgcn_rcpf(rho);
        float F[3], u0[3];
#pragma unroll
        for (int a = 0; a < 3; a++) F[a] = fs[a] + cp * g[a] + rho * aext[a];
        if (PH && P.gravity_on) {  // buoyancy against the box-mean hydrostatic balance
            const float dr = rho - P.rho_mean;
#pragma unroll
            for (int a = 0; a < 3; a++) F[a] += dr * P.grav[a];
        }
#pragma unroll
        for (int a = 0; a < 3; a++) u0[a] = j[a] + 0.5f * F[a] * inv_rho;
        // relaxation rate and viscous-correction coefficient nu / (tau c_s^2) = 1 - omega / 2
        float omega = P.omega, fnu = P.fnu_coef;
        if (PH && P.tau_g > 0.0f) {
            const float c = fminf(fmaxf(G.phi, 0.0f), 1.0f);
            omega = 1.0f / fmaf(c, P.tau_l - P.tau_g, P.tau_g);
            fnu = 1.0f - 0.5f * omega;
        }
        m.omega = omega;
        const float n0 = m.S[0] - u0[0] * u0[0], n1 = m.S[1] - u0[1] * u0[1], n2 = m.S[2] - u0[2] * u0[2];
        const float n3 = m.S[3] - u0[0] * u0[1], n4 = m.S[4] - u0[0] * u0[2], n5 = m.S[5] - u0[1] * u0[2];
        const float cnu = -fnu * drho;
        F[0] += cnu * (n0 * g[0] + n3 * g[1] + n4 * g[2]);
        F[1] += cnu * (n3 * g[0] + n1 * g[1] + n5 * g[2]);
        F[2] += cnu * (n4 * g[0] + n5 * g[1] + n2 * g[2]);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            m.a[a] = F[a] * inv_rho;
            m.u[a] = j[a] + 0.5f * m.a[a];
        }
        m.rho = rho;
    } else {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            m.a[a] = aext[a];
            m.u[a] = j[a] + 0.5f * aext[a];
        }
        m.rho = P.rho_l;
        m.omega = P.omega;
    }
}

// Regularised post-collision h_i = f^post_i / w_i - P0,
//   f^post = f^eq(p*, u) + (1 - omega) w H : a2 / (2 c_s^4) + S/2,
//   a2 = Pi - p* c_s^2 I - u u + (u a + a u)/2  (closed form of Eq. (7)),
// which is the quadratic polynomial h(c) = base + b.c + c.B.c with
//   b = 3 (u + a/2), B = (9/4)(u w + w u) + (9/2)(1 - omega) a2, w = u + a,
//   base = p* - P0 - (3/2)(u.u + u.a) - (3/2)(1 - omega) tr a2,
// evaluated on the 27 velocities axis by axis.
__device__ __forceinline__ void collide(const Macro &m, float omega, float (&h)[27])
{
    const float ux = m.u[0], uy = m.u[1], uz = m.u[2];
    const float ax = m.a[0], ay = m.a[1], az = m.a[2];
    const float wx = ux + ax, wy = uy + ay, wz = uz + az;
    const float k = 4.5f * (1.0f - omega);
    const float Axx = m.S[0] - ux * ux + ux * ax;
    const float Ayy = m.S[1] - uy * uy + uy * ay;
    const float Azz = m.S[2] - uz * uz + uz * az;
    const float Axy = m.S[3] - ux * uy + 0.5f * (ux * ay + ax * uy);
    const float Axz = m.S[4] - ux * uz + 0.5f * (ux * az + ax * uz);
    const float Ayz = m.S[5] - uy * uz + 0.5f * (uy * az + ay * uz);
    const float Bxx = fmaf(k, Axx, 4.5f * ux * wx);
    const float Byy = fmaf(k, Ayy, 4.5f * uy * wy);
    const float Bzz = fmaf(k, Azz, 4.5f * uz * wz);
    const float Bxy2 = 2.0f * fmaf(k, Axy, 2.25f * (ux * wy + wx * uy));
    const float Bxz2 = 2.0f * fmaf(k, Axz, 2.25f * (ux * wz + wx * uz));
    const float Byz2 = 2.0f * fmaf(k, Ayz, 2.25f * (uy * wz + wy * uz));
    const float bx = 3.0f * ux + 1.5f * ax, by = 3.0f * uy + 1.5f * ay, bz = 3.0f * uz + 1.5f * az;
    const float u2 = ux * ux + uy * uy + uz * uz, ua = ux * ax + uy * ay + uz * az;
    const float base = m.dp - 1.5f * (u2 + ua) - (k * (1.0f / 3.0f)) * (Axx + Ayy + Azz);
    const float gz = base + Bzz;
    const float G[3] = {gz - bz, base, gz + bz};
    const float Y[3] = {by - Byz2, by, by + Byz2};
    const float X[3] = {bx - Bxz2, bx, bx + Bxz2};
#pragma unroll
    for (int z = 0; z < 3; z++) {
        const float ty = G[z] + Byy;
        const float T[3] = {ty - Y[z], G[z], ty + Y[z]};
        const float Xc[3] = {X[z] - Bxy2, X[z], X[z] + Bxy2};
#pragma unroll
        for (int y = 0; y < 3; y++) {
            const int row = 3 * z + y;
            const float tx = T[y] + Bxx;
            h[3 * row] = tx - Xc[y];
            h[3 * row + 1] = T[y];
            h[3 * row + 2] = tx + Xc[y];
        }
    }
}

// ----------------------------------------------------- phase-field fluxes
// WENO-5 (Jiang & Shu) value at the face right of cell c from the upwind-biased
// cells (a, b, c, d, e) = (c-2 .. c+2): candidates q_k, smoothness beta_k with
// the 13/12 and 1/4 factors, linear weights (1/10, 6/10, 3/10), eps = 1e-6,
// p = 2; the nonlinear weights d_k / (eps + beta_k)^2 are taken with one
// reciprocal after scaling by the product of the three denominators.
// Contraction-free (explicit fma only) so both cells of a face get the same bits.
__device__ __forceinline__ float weno5(float a, float b, float c, float d, float e)
{
#pragma clang fp contract(off)
    const float q0 = fmaf(11.0f / 6.0f, c, fmaf(-7.0f / 6.0f, b, (1.0f / 3.0f) * a));
    const float q1 = fmaf(1.0f / 3.0f, d, fmaf(5.0f / 6.0f, c, (-1.0f / 6.0f) * b));
    const float q2 = fmaf(-1.0f / 6.0f, e, fmaf(5.0f / 6.0f, d, (1.0f / 3.0f) * c));
    const float t0 = fmaf(-2.0f, b, a + c), r0 = fmaf(-4.0f, b, fmaf(3.0f, c, a));
    const float t1 = fmaf(-2.0f, c, b + d), r1 = b - d;
    const float t2 = fmaf(-2.0f, d, c + e), r2 = fmaf(3.0f, c, fmaf(-4.0f, d, e));
    float s0 = fmaf((13.0f / 12.0f) * t0, t0, fmaf(0.25f * r0, r0, 1e-6f));
    float s1 = fmaf((13.0f / 12.0f) * t1, t1, fmaf(0.25f * r1, r1, 1e-6f));
    float s2 = fmaf((13.0f / 12.0f) * t2, t2, fmaf(0.25f * r2, r2, 1e-6f));
    s0 = s0 * s0;
    s1 = s1 * s1;
    s2 = s2 * s2;
    const float w0 = 0.1f * (s1 * s2), w1 = 0.6f * (s0 * s2), w2 = 0.3f * (s0 * s1);
    const float num = fmaf(w2, q2, fmaf(w1, q1, w0 * q0));
    return num * __builtin_amdgcn_rcpf((w0 + w1) + w2);
}

// Advective flux ubar * phi_face through the face between cells l and l+1:
// v0..v5 = phi at l-2 .. l+3, ul / ur = velocity component at l / l+1;
// upwinded by the sign of ubar, zero when ubar == 0.
__device__ __forceinline__ float face_flux(float v0, float v1, float v2, float v3, float v4, float v5, float ul,
                                           float ur)
{
#pragma clang fp contract(off)
    const float ub = 0.5f * (ul + ur);
    const bool pos = ub > 0.0f;
    const float a = pos ? v0 : v5, b = pos ? v1 : v4, c = pos ? v2 : v3, d = pos ? v3 : v2, e = pos ? v4 : v1;
    const float h = weno5(a, b, c, d, e);
    return ub == 0.0f ? 0.0f : ub * h;
}

// Diffusion + sharpening flux leaving a toward b = a + c_I (canonical I > 13):
// w_I [6 D (phi_a - phi_b) + 3 kappa (Q_a + Q_b) . c_I]; the projection on c_I
// takes the nonzero components in x, y, z order.
template <int I>
__device__ __forceinline__ float link_flux(float pa, float pb, const float (&qa)[3], const float (&qb)[3], float d6w,
                                           float k3w)
{
#pragma clang fp contract(off)
    constexpr int cx = CX(I), cy = CY(I), cz = CZ(I);
    const float tx = qa[0] + qb[0], ty = qa[1] + qb[1], tz = qa[2] + qb[2];
    float s;
    if constexpr (cx != 0) {
        s = cx > 0 ? tx : -tx;
        if constexpr (cy != 0) s = cy > 0 ? s + ty : s - ty;
        if constexpr (cz != 0) s = cz > 0 ? s + tz : s - tz;
    } else if constexpr (cy != 0) {
        s = cy > 0 ? ty : -ty;
        if constexpr (cz != 0) s = cz > 0 ? s + tz : s - tz;
    } else {
        s = cz > 0 ? tz : -tz;
    }
    return fmaf(k3w, s, d6w * (pa - pb));
}

// Q = phi (1 - phi) n, n = g / |g| (zero where |g| <= 1e-12), from the first
// moments M1 of the phi stencil (g = M1 / 72; n needs only M1).  Neighbouring
// workgroups, and the prologue and body of one workgroup, evaluate Q at the
// same point from different inlined copies: contraction-free, so every copy
// rounds identically.
__device__ __forceinline__ void q_of(float Mx, float My, float Mz, float phi, float (&q)[3])
{
#pragma clang fp contract(off)
    const float m2 = fmaf(Mx, Mx, fmaf(My, My, Mz * Mz));
    const float c = phi * (1.0f - phi);
    const float s = m2 > 5.184e-21f ? c * __frsqrt_rn(m2) : 0.0f;  // |g| > 1e-12 <=> |M1| > 7.2e-11
    q[0] = s * Mx;
    q[1] = s * My;
    q[2] = s * Mz;
}
// plane sums for the first moments alone
struct P3 {
    float p00, p01, p10;
};
__device__ __forceinline__ void plane3(const float *v, P3 &p)
{
    float r0[3], r1[3];
#pragma unroll
    for (int row = 0; row < 3; row++) {
        const float vm = v[3 * row], v0 = v[3 * row + 1], vp = v[3 * row + 2];
        r1[row] = vp - vm;
        r0[row] = fmaf(4.0f, v0, vp + vm);
    }
    p.p00 = fmaf(4.0f, r0[1], r0[2] + r0[0]);
    p.p01 = r0[2] - r0[0];
    p.p10 = fmaf(4.0f, r1[1], r1[2] + r1[0]);
}

// ----------------------------------------------------------------- forcing
// Time-independent body acceleration (Sec. 5.1 uses a fixed large-scale
// field).  k_forcing groups the modes by |kx| and folds the y and z phases into
// per-row coefficients (see lbm_internal.h); a site combines its row's 15
// coefficients with the x twiddles ex = (cos t, sin t, cos 2t, sin 2t).
// UNIFORM: the row is the same in every lane of the wave (one x-row per wave);
// its coefficients are then read with scalar loads through the constant
// address space (the table is read-only while a step runs), which the scalar
// data cache serves and which leave the vector-memory counter to the
// population loads.
#define LBM_CONST __attribute__((address_space(4)))
template <bool UNIFORM>
__device__ __forceinline__ void forcing_at(const Params &P, float4 ex, uint32_t row, float (&a)[3])
{
    float c[15];
    if constexpr (UNIFORM) {
        const LBM_CONST float *r = (const LBM_CONST float *)P.frow + (size_t)row * FROW;
#pragma unroll
        for (int k = 0; k < 15; k++) c[k] = r[k];
    } else {
        const LBM_GLOBAL float *r = gconst(P.frow) + (size_t)row * FROW;
#pragma unroll
        for (int k = 0; k < 15; k++) c[k] = r[k];
    }
#pragma unroll
    for (int d = 0; d < 3; d++)
        a[d] = c[d] + (c[3 + d] * ex.x + c[6 + d] * ex.y) + (c[9 + d] * ex.z + c[12 + d] * ex.w);
}

// ------------------------------------------------------------ fused step
constexpr int HX = 3, HY = 3;                  // phi tile halo (WENO-5 needs 3)
constexpr int NRING = 7;                       // phi planes z-3 .. z+3

// Workgroup tile of TW x (256 / TW) sites: TW = 64 is one wave per x-row;
// TW = 32 puts two rows in a wave (boxes of 32 or 96 sites in x waste no lanes).
// LDS tiles and per-thread work rounds derive from it.
template <int TW> struct Tile {
    static constexpr int X = TW, Y = NTHREADS / TW;
    static constexpr int PX = X + 2 * HX, PY = Y + 2 * HY;
    static constexpr int PLANE = PX * PY;         // phi values per staged plane
    static constexpr int QX = X + 2, QY = Y + 2;  // Q tile (halo 1)
    static constexpr int LOADS = (PLANE + NTHREADS - 1) / NTHREADS;
    static constexpr int QHALO = QX * QY - NTHREADS;  // points of the Q tile's halo ring
    // Q, x faces and y faces are held with the row stride of the phi tile, so
    // that one LDS address per thread (its phi tile index) serves all of them:
    // rows HY-1 .. of the tile for Q, rows HY .. for the faces
    static constexpr int Q0 = (HY - 1) * PX, QN = QY * PX;
    static constexpr int F0 = HY * PX, NXF = Y * PX, NYF = (Y + 1) * PX;
};

__device__ __forceinline__ int ring(int z) { return (z + 4 * NRING) % NRING; }

// Workgroup barrier for LDS traffic only: waits for this wave's LDS operations,
// not for its outstanding global loads, so prefetches stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), vmcnt / expcnt untouched
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// No instruction moves across: the scheduler otherwise starts the LDS reads of
// many links and faces at once, for which the step has no registers, and a
// spilled register read back waits for every load in flight before it.
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Software pipeline over the z planes of a chunk: while plane z is processed,
// the phi plane z+4, the face velocities of plane z+1, the 27 populations of
// plane z+1 and the site's own phi and u_z ahead are already being fetched.
//
// What bounds it: with 16-bit populations the vector instructions (934 per site
// and plane, issued 90 % of the time with three waves per SIMD), with FP32 ones
// the memory traffic.  Hence: the phi stencil is summed plane by plane, each
// plane once for the Q, the gradient and the Hessian of the three planes it
// enters (summed anew for each, they were 110 instructions more); every address
// is a scalar base plus one of three 32-bit columns; and the wait counts are
// exact, so that neither the stores of a plane nor the loads of the next are
// waited for before they are needed.  512^3 bubbly HIT, per step: FP16 5.0 ->
// 4.6 ms; 256^3 single phase FP16 0.575 -> 0.47 ms; Runge-Kutta stage at 256^3
// 0.385 -> 0.35 ms; FP32 at 512^3 as before.
// One work item: the xy tile and z chunk with linear index L (x tile fastest,
// then y tile, then z chunk) of one box.  Every thread of the workgroup calls
// it; it leaves no LDS state that the next call relies on.
//
// ACO (Allen-Cahn only): one Runge-Kutta stage of the phase field and nothing
// else: phi_out = rk_a phi^n + rk_b (phi_in + L(phi_in)) with phi_in staged in
// the LDS ring (B.phin), phi^n read at the site (B.phin0), FP64 phi.
template <int S, bool TP, bool FRC, bool ML, int TW = TX, bool NT = false, bool FX = false, bool ACO = false,
          bool PH = false>
__device__ __forceinline__ void step_tile(const Params &P, const Buffers &B, const uint32_t L, double rk_a = 0.0,
                                          double rk_b = 1.0)
{
    static_assert(!ACO || (TP && !FX && !ML), "a Runge-Kutta stage needs the FP64 phase field");
    // ML: the learned curvature.  The network pass (pass_tile) that runs
    // before the step leaves in B.mlpy the network output at every interface
    // cell that the curvature criterion selects (NaN at the other interface
    // cells); the step reads it where its own criterion selects the cell (the
    // same test on the same stencil, so the pass has written there) and falls
    // back to finite differences on NaN, so the network's registers and LDS
    // are not part of the step kernel.
    constexpr bool LBM = !ACO;  // the populations are streamed and collided
    using T = typename Pop<S>::T;
    using PS = PhiStore<FX>;
    using PT = typename PS::T;
    using AT = typename PS::Acc;
    using TL = Tile<TW>;
    constexpr int TXW = TL::X, TYW = TL::Y, PX = TL::PX, PLANE = TL::PLANE, QX = TL::QX, LOADS = TL::LOADS,
                  QHALO = TL::QHALO, Q0 = TL::Q0, F0 = TL::F0;
    constexpr uint32_t ES = sizeof(T);
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const uint32_t N = plane * (uint32_t)nz;
    const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * TXW + tx;
    const int bx = (int)(L % (uint32_t)P.gx), by = (int)((L / (uint32_t)P.gx) % (uint32_t)P.gy);
    const int bz = (int)(L / ((uint32_t)P.gx * (uint32_t)P.gy));
    const int x0 = bx * TXW, y0 = by * TYW, z0 = bz * P.zchunk;
    const int zend = min(z0 + P.zchunk, nz);
    // Lanes past the box's edge (a ragged last tile) step the periodic image of
    // their site: the same inputs give the same bits, so their writes repeat
    // the owner's.  Keeping every lane busy keeps every memory operation
    // unconditional, so the compiler counts the loads in flight exactly instead
    // of draining all of them (stores included) before the next plane.
    const int xg = (x0 + tx) % nx, yg = (y0 + ty) % ny;
    const T *__restrict__ fin = (const T *)B.fin;
    T *__restrict__ fout = (T *)B.fout;
    const float *__restrict__ uin = B.uin;  // component a at a * N
    const PT *__restrict__ phin = (const PT *)B.phin;

    // The periodic neighbours' columns xs and rows ys (k = 1 + offset).  With
    // one x-row per wave (TW = 64) the row is wave-uniform: it goes into the
    // scalar part of every address, and the vector part is one of three
    // columns.  Two rows per wave (TW = 32) take the row in the vector part.
    constexpr bool ROW = TW == 64;
    const int yw = ROW ? __builtin_amdgcn_readfirstlane(yg) : yg;
    uint32_t xs[3], ys[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        xs[k] = (uint32_t)wrapi(xg + k - 1, nx);
        ys[k] = (uint32_t)wrapi(yw + k - 1, ny) * (uint32_t)nx;
    }
    auto srow = [&](int k) { return ROW ? ys[k] : 0u; };                            // scalar part
    auto vcol = [&](int ky, int kx) { return ROW ? xs[kx] : ys[ky] + xs[kx]; };  // vector part
    const uint32_t own_v = vcol(1, 1);
    auto zp = [&](int z) { return (uint32_t)z * plane; };  // first site of plane z (below 2^30)
    // buffer over plane z of a field of one value per site
    auto field = [&](auto *base, int z) { return plane_rsrc(base + zp(z), plane * (uint32_t)sizeof(*base)); };
    // element of a field at plane z, row ky and column kx of the neighbourhood
    auto at = [&](auto *base, int z, int ky, int kx) {
        using E = std::remove_cv_t<std::remove_reference_t<decltype(*base)>>;
        return bload<E>(field(base, z), vcol(ky, kx) * (uint32_t)sizeof(E), srow(ky) * (uint32_t)sizeof(E));
    };
    auto put = [&](auto *base, int z, auto v) {  // own site
        bstore<decltype(v), NT ? STORE_NT : 0>(field(base, z), own_v * (uint32_t)sizeof(v),
                                               srow(1) * (uint32_t)sizeof(v), v);
    };

    // The x twiddles of the body force: in LDS with the phase field (read once
    // per plane there; four registers less to carry through it), in registers
    // without
    __shared__ float4 sex[FRC && TP ? TXW : 1];
    float4 ex = {0.f, 0.f, 0.f, 0.f};
    if constexpr (FRC) {
        const LBM_GLOBAL float *fx = gconst((const float *)P.fx) + 4 * xg;
        ex = make_float4(fx[0], fx[1], fx[2], fx[3]);
        if (TP && ty == 0) sex[tx] = ex;
    }
    const uint32_t yrow = (uint32_t)yw;

    // pull-stream of plane z into hv: h_i(x) = h^post_i(x - c_i)
    // raw storage values: decoded only where they are consumed, so the loads of
    // the next plane stay in flight (a decode right after the load would wait for it)
    // 16-bit values are held zero-extended in full registers: packed two to a
    // register, each pair would wait for its loads on arrival (a 16-bit load
    // into half a register depends on the other half), which would make the
    // prefetch synchronous
    using HT = std::conditional_t<sizeof(T) == 2, uint32_t, T>;
    HT hv[27];
    const uint32_t pbytes = 27u * plane * ES;   // bytes per z plane of populations
    // steps of the row offset from one population to the next: the next x, and
    // from the last x of row y + 1, y, y - 1 to the first of the row after it
    const uint32_t pstep = plane * ES, rstep01 = pstep + (srow(1) - srow(2)) * ES,
                   rstep10 = pstep + (srow(0) - srow(1)) * ES, rstep12 = pstep + (srow(2) - srow(0)) * ES;
    auto fetch_pops = [&](int z) {
        const __amdgpu_buffer_rsrc_t zsrc[3] = {plane_rsrc(fin + (size_t)zp(wrapi(z + 1, nz)) * 27, pbytes),
                                                plane_rsrc(fin + (size_t)zp(z) * 27, pbytes),
                                                plane_rsrc(fin + (size_t)zp(wrapi(z - 1, nz)) * 27, pbytes)};
        // running offset of the population's row, kept opaque so that the 27
        // offsets are not all precomputed into scalar registers
        uint32_t soff = srow(2) * ES;
#pragma unroll
        for (int i = 0; i < 27; i++) {
            const uint32_t v = vcol(1 - CY(i), 1 - CX(i)) * ES;
            if constexpr (std::is_same_v<HT, T>)
                hv[i] = bload<T>(zsrc[CZ(i) + 1], v, soff);
            else
                hv[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(zsrc[CZ(i) + 1], v, soff, 0);
            soff += CX(i) < 1 ? pstep : (CY(i) < 0 ? rstep01 : (CY(i) < 1 ? rstep10 : rstep12));
            asm volatile("" : "+s"(soff));
        }
    };

    // LDS: phi ring (FP32), Q of planes z-1..z+1, x/y advective face fluxes of plane z
    __shared__ float sphi[TP ? NRING : 1][TP ? PLANE : 1];
    constexpr int QN = TP ? TL::QN : 1;
    __shared__ float sq[TP ? 3 : 1][3][QN];
    __shared__ float sjx[TP ? TL::NXF : 1];
    __shared__ float sjy[TP ? TL::NYF : 1];
    // plane sums of the halo points: each point's three sums of the last two
    // planes, read and written by its own thread only (kept in registers they
    // made the step spill)
    __shared__ float sh[TP ? 2 : 1][3][TP ? QHALO : 1];
    const int lc = (ty + HY) * PX + (tx + HX);  // own phi tile index
    PT phn[LOADS];          // prefetched phi plane
    uint32_t p_off[LOADS];  // byte offsets of its points in a plane
    // Q is evaluated at the own site by every thread and at the halo ring of
    // the tile by the waves after the first; the first wave has the y faces
    // above the top row instead, so that no SIMD of the CU (wave i of a
    // workgroup runs on SIMD i) has both.
    static_assert(QHALO <= NTHREADS - 64, "one halo point per thread");
    const int hp = tid - 64;
    const bool halo = TP && hp >= 0 && hp < QHALO;
    int h_lc = lc;
    if (halo) {
        const int k = hp - 2 * QX;
        const int qy = hp < QX ? 0 : (hp < 2 * QX ? TYW + 1 : 1 + (k >> 1));
        const int qx = hp < QX ? hp : (hp < 2 * QX ? hp - QX : (k & 1) * (QX - 1));
        h_lc = (qy + HY - 1) * PX + (qx + HX - 1);
    }
    // The x and y faces of a plane tile are evaluated in three rounds, each
    // wave taking one direction in each: (A) the x face left of every site,
    // (B) the y face below every site, (C) the y faces above the top row
    // (threads 0 .. TXW-1, the first wave) and the x faces right of the last
    // column (the first threads of the last wave).  c_lc: the phi tile
    // index of the left (lower) cell of a round-C face.
    constexpr int RIGHT0 = NTHREADS - 64;
    const bool c_top = tid < TXW, c_right = tid >= RIGHT0 && tid < RIGHT0 + TYW;
    const int c_lc = c_top ? (TYW - 1 + HY) * PX + tid + HX : (tid - RIGHT0 + HY) * PX + (TXW - 1 + HX);
    float fa_l, fa_r, fb_l, fb_r, fc_l = 0.f, fc_r = 0.f;  // prefetched face velocities
    // the round-C face's velocities in plane 0 (per-lane pointers: the two kinds
    // of face read different components)
    const LBM_GLOBAL float *c_l = nullptr, *c_r = nullptr;
    float jz_left = 0.f, uz_c = 0.f, uz_n = 0.f;
    PT po = 0;              // prefetched own phi
    // carried from plane to plane: the phi stencil's plane sums of the two
    // planes below the next one (own site), so that every plane is summed once
    // for the Q, the gradient and the Hessian of three planes
    P6 pa, pb;
    // the phi gradient and curvature (its coefficient in the force; with the
    // learned curvature K_FD) of the current and the next plane, read and
    // written by its own thread only (in registers they made the step spill)
    __shared__ float4 sg[LBM && TP ? 2 : 1][LBM && TP ? NTHREADS : 1];
    float cs = 0.f, csn = 0.f;        // learned curvature: the coefficient ...
    bool sel = false, seln = false;   // ... and whether the network is consulted

    // in-plane offset of position e of the phi tile
    auto tile_xy = [&](int e) {
        const int ly = e / PX, lx = e - ly * PX;
        return (uint32_t)modi(y0 + ly - HY, ny) * nx + (uint32_t)modi(x0 + lx - HX, nx);
    };
    auto fetch_plane = [&](PT(&r)[LOADS], int z) {
        const __amdgpu_buffer_rsrc_t src = field(phin, wrapi(z, nz));
#pragma unroll
        for (int k = 0; k < LOADS; k++) r[k] = bload<PT>(src, p_off[k], 0);
    };
    auto store_plane = [&](const PT(&r)[LOADS], int z) {
        float *dst = sphi[ring(z)];
#pragma unroll
        for (int k = 0; k < LOADS; k++) {
            const int e = tid + k * NTHREADS;
            if (e < PLANE) dst[e] = PS::f32(r[k]);
        }
    };
    auto fetch_face_u = [&](int z) {
        const __amdgpu_buffer_rsrc_t ux = field(uin, z), uy = field(uin + N, z);
        fa_l = bload<float>(ux, vcol(1, 0) * 4u, srow(1) * 4u);
        fa_r = bload<float>(ux, own_v * 4u, srow(1) * 4u);
        fb_l = bload<float>(uy, vcol(0, 1) * 4u, srow(0) * 4u);
        fb_r = bload<float>(uy, own_v * 4u, srow(1) * 4u);
        if (c_top || c_right) {
            fc_l = c_l[zp(z)];
            fc_r = c_r[zp(z)];
        }
    };
    auto load9 = [&](const float *p, float (&v)[9]) {
#pragma unroll
        for (int i = 0; i < 9; i++) v[i] = p[(i / 3 - 1) * PX + i % 3 - 1];
    };
    auto put3 = [&](int z, const P3 &n) {
        auto &h = sh[z & 1];
        h[0][hp] = n.p00;
        h[1][hp] = n.p01;
        h[2][hp] = n.p10;
    };
    // q of plane z (phi planes z-1 .. z+1: the carried sums and the newest
    // plane) and, from the same moments, the own site's phi gradient and Hessian
    auto compute_q = [&](int z) {
        const float *pc = sphi[ring(z)], *pn = sphi[ring(z + 1)];
        float(*q)[QN] = sq[(z + 3) % 3];
        float v[9], qv[3];
        {
            P6 n;
            M10 M;
            load9(pn + lc, v);
            plane6(v, n);
            planes10(pa, pb, n, M);
            pa = pb;
            pb = n;
            const float c = pc[lc];
            q_of(M.m100, M.m010, M.m001, c, qv);
#pragma unroll
            for (int a = 0; a < 3; a++) q[a][lc - Q0] = qv[a];
            if constexpr (LBM) {
                PhiGrad G;
                phi_grad(M, c, G);
                csn = surface_coef<ML>(M, G, P);
                float w = csn;
                if constexpr (ML) {
                    float gn;
                    seln = mlp_select(G, P, w, gn);
                }
                sg[z & 1][tid] = make_float4(G.g[0], G.g[1], G.g[2], w);
            }
        }
        if (halo) {
            P3 n;
            load9(pn + h_lc, v);
            plane3(v, n);
            const auto &a3 = sh[(z + 1) & 1], &b3 = sh[z & 1];
            q_of(fmaf(4.0f, b3[2][hp], n.p10 + a3[2][hp]), fmaf(4.0f, b3[1][hp], n.p01 + a3[1][hp]),
                 n.p00 - a3[0][hp], pc[h_lc], qv);
            put3(z + 1, n);
#pragma unroll
            for (int a = 0; a < 3; a++) q[a][h_lc - Q0] = qv[a];
        }
    };
    // advective x and y fluxes of plane z through the faces of the tile, each
    // face once, held at the tile index of the cell right of (above) it
    auto compute_faces = [&](int z) {
        const float *pl = sphi[ring(z)];
        {
            const float *p = pl + lc - 3;  // cells x-3 .. x+2 of the row
            sjx[lc - F0] = face_flux(p[0], p[1], p[2], p[3], p[4], p[5], fa_l, fa_r);
        }
        sched_fence();
        {
            const float *p = pl + lc - 3 * PX;  // cells y-3 .. y+2 of the column
            sjy[lc - F0] = face_flux(p[0], p[PX], p[2 * PX], p[3 * PX], p[4 * PX], p[5 * PX], fb_l, fb_r);
        }
        if (c_top) {
            const float *p = pl + c_lc - 2 * PX;
            sjy[c_lc + PX - F0] = face_flux(p[0], p[PX], p[2 * PX], p[3 * PX], p[4 * PX], p[5 * PX], fc_l, fc_r);
        } else if (c_right) {
            const float *p = pl + c_lc - 2;
            sjx[c_lc + 1 - F0] = face_flux(p[0], p[1], p[2], p[3], p[4], p[5], fc_l, fc_r);
        }
    };
    if (LBM && !TP) fetch_pops(z0);
    if constexpr (TP) {
#pragma unroll
        for (int k = 0; k < LOADS; k++) {
            const int e = tid + k * NTHREADS;
            p_off[k] = tile_xy(e < PLANE ? e : PLANE - 1) * (uint32_t)sizeof(PT);  // spare lanes re-read the last
        }
        const LBM_GLOBAL float *uc = gconst(uin) + (c_top ? (size_t)N : 0);
        c_l = uc + tile_xy(c_lc);
        c_r = uc + tile_xy(c_top ? c_lc + PX : c_lc + 1);
        {
            // the six planes below the loop's first one, all in flight at once
            PT r[6][LOADS];
#pragma unroll
            for (int j = 0; j < 6; j++) fetch_plane(r[j], z0 - 3 + j);
            fetch_plane(phn, z0 + 3);
            fetch_face_u(z0);
#pragma unroll
            for (int j = 0; j < 6; j++) store_plane(r[j], z0 - 3 + j);
        }
        if (LBM) fetch_pops(z0);
        lds_barrier();
        {
            float v[9];
            load9(sphi[ring(z0 - 2)] + lc, v);
            plane6(v, pa);
            load9(sphi[ring(z0 - 1)] + lc, v);
            plane6(v, pb);
            if (halo)
                for (int z = z0 - 2; z < z0; z++) {
                    P3 n;
                    load9(sphi[ring(z)] + h_lc, v);
                    plane3(v, n);
                    put3(z, n);
                }
            compute_q(z0 - 1);
            compute_q(z0);
            cs = csn;
            sel = seln;
            // z face below the first plane: cells z0-3 .. z0+2, velocities at z0-1, z0
            const float um = at(uin + 2 * (size_t)N, wrapi(z0 - 1, nz), 1, 1);
            uz_c = at(uin + 2 * (size_t)N, z0, 1, 1);
            uz_n = at(uin + 2 * (size_t)N, wrapi(z0 + 1, nz), 1, 1);
            po = at(phin, z0, 1, 1);
            float c[6];
#pragma unroll
            for (int k = 0; k < 6; k++) c[k] = sphi[ring(z0 - 3 + k)][lc];
            jz_left = face_flux(c[0], c[1], c[2], c[3], c[4], c[5], um, uz_c);
        }
    }
    // Every load of the prologue is complete when the loop begins.  The compiler
    // counts the operations issued since a load on the way into the loop and
    // around it and waits for the smaller number; on the way in no stores
    // follow the population loads, so without this wait every plane of the
    // loop waited for the stores of the plane before.
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), expcnt / lgkmcnt untouched
    for (int z = z0; z < zend; z++) {
        const bool more = z + 1 < zend;
        // The prefetches for the next plane run in the last plane of the chunk
        // too, re-reading the current plane's data (in L2, valid addresses): an
        // unconditional load keeps the prefetched values in the same registers
        // on every path, where a skipped one made the compiler copy all 27
        // populations and the other prefetched values on both sides of the branch.
        const int zn = more ? z + 1 : z;
        if constexpr (TP) {
            store_plane(phn, z + 3);
            fetch_plane(phn, zn + 3);
            lds_barrier();
            compute_q(z + 1);
            sched_fence();
            compute_faces(z);
            sched_fence();
            fetch_face_u(zn);
            lds_barrier();
        }
        M10 M;
        float aext[3] = {0.f, 0.f, 0.f};
        float y[4] = {0.f, 0.f, 0.f, 0.f};  // learned curvature: network output at a selected cell
        {
            if constexpr (LBM) {
                float hf[27];
#pragma unroll
                for (int i = 0; i < 27; i++) {
                    if constexpr (std::is_same_v<HT, T>) hf[i] = Pop<S>::dec(hv[i]);
                    else hf[i] = Pop<S>::dec(__builtin_bit_cast(T, (uint16_t)hv[i]));
                }
                moments10(hf, M);
            }
            if (LBM && !TP) fetch_pops(zn);
            if constexpr (TP) {
                // Allen-Cahn: phi^{n+1} = phi^n - sum (outgoing - incoming) face and link fluxes
                // four independent partial sums keep the dependent add chains short
                AT acc[4];
                acc[0] = PS::flux(sjx[lc - F0]) - PS::flux(sjx[lc - F0 + 1]);
                acc[0] += PS::flux(sjy[lc - F0]) - PS::flux(sjy[lc - F0 + PX]);
                {
                    float v[6];
#pragma unroll
                    for (int k = 0; k < 6; k++) v[k] = sphi[ring(z - 2 + k)][lc];
                    const float jr = face_flux(v[0], v[1], v[2], v[3], v[4], v[5], uz_c, uz_n);
                    acc[1] = PS::flux(jz_left) - PS::flux(jr);
                    jz_left = jr;
                    uz_c = uz_n;
                    uz_n = at(uin + 2 * (size_t)N, wrapi(zn + 1, nz), 1, 1);
                }
                sched_fence();
                {
                    const float *pm = sphi[ring(z - 1)] + lc, *pc = sphi[ring(z)] + lc, *pp = sphi[ring(z + 1)] + lc;
                    auto q_at = [&](int k, int off, float(&q)[3]) {
#pragma unroll
                        for (int a = 0; a < 3; a++) q[a] = sq[(z + k + 3) % 3][a][lc - Q0 + off];
                    };
                    float qo[3];
                    q_at(0, 0, qo);
                    const float p0 = pc[0];
                    const float d6w[4] = {0.f, P.d6 * WT(14), P.d6 * WT(15), P.d6 * WT(26)};
                    const float k3w[4] = {0.f, P.k3 * WT(14), P.k3 * WT(15), P.k3 * WT(26)};
                    // links 14 and 15 open the partial sums 2 and 3
#define LB_LINK(I)                                                                                    \
    {                                                                                                 \
        constexpr int off = CY(I) * PX + CX(I), up = CZ(I) > 0;                                       \
        float qn[3], qs[3];                                                                           \
        q_at(up, off, qn);                                                                            \
        q_at(-up, -off, qs);                                                                          \
        const float fo = link_flux<I>(p0, (up ? pp : pc)[off], qo, qn, d6w[C2(I)], k3w[C2(I)]);       \
        const float fi = link_flux<I>((up ? pm : pc)[-off], p0, qs, qo, d6w[C2(I)], k3w[C2(I)]);      \
        const AT d = PS::flux(fi) - PS::flux(fo);                                                     \
        if constexpr (I == 14 || I == 15) acc[I & 3] = d;                                             \
        else acc[I & 3] += d;                                                                         \
    }
                    LB_LINK(14) LB_LINK(15) LB_LINK(16) LB_LINK(17)
                    sched_fence();
                    LB_LINK(18) LB_LINK(19) LB_LINK(20) LB_LINK(21) LB_LINK(22)
                    sched_fence();
                    LB_LINK(23) LB_LINK(24) LB_LINK(25) LB_LINK(26)
                    sched_fence();
#undef LB_LINK
                }
                PT pnew;
                if constexpr (ACO)
                    pnew = rk_a * at((const double *)B.phin0, z, 1, 1) +
                           rk_b * (po + ((acc[0] + acc[1]) + (acc[2] + acc[3])));
                else
                    pnew = PS::add(po, (acc[0] + acc[1]) + (acc[2] + acc[3]));
                put((PT *)B.phout, z, pnew);
                if constexpr (ML || ACO) {
                    // interface flags of the new phi, as the next network pass
                    // will see it (its FP32 value): one byte per 32-lane half
                    // of the wave, each half one 32-site segment of one row
                    if (B.iflag) {
                        const float pf = PS::f32(pnew);
                        const uint64_t m = __ballot(pf > 0.02f && pf < 0.98f);
                        const int lane = tid & 63;
                        if ((lane & 31) == 0 && x0 + tx < nx && y0 + ty < ny)
                            B.iflag[((size_t)z * ny + yg) * flag_segments(nx) + xg / 32] =
                                (uint8_t)(((lane < 32 ? m : m >> 32) & 0xffffffffull) != 0);
                    }
                }
                po = at(phin, zn, 1, 1);
            }
            // Every other load of this plane is issued before the populations of
            // the next one: loads complete in order, so waiting for a load
            // issued after the 27 prefetches would wait for them as well.
            if constexpr (FRC && LBM) forcing_at<TW == 64>(P, TP ? sex[tx] : ex, (uint32_t)z * ny + yrow, aext);
            if constexpr (ML) {
                if (sel) {  // the network output that the learned-curvature pass left here
                    const LBM_GLOBAL float *yi = gconst((const float *)B.mlpy) + 4 * (size_t)(zp(z) + srow(1) + own_v);
                    y[0] = yi[0];
                    y[1] = yi[1];
                    y[2] = yi[2];
                    y[3] = yi[3];
                }
            }
            if (LBM && TP) fetch_pops(zn);
        }
        if constexpr (ACO) continue;
        // surface tension: finite differences, or blended with the network
        // output that the learned-curvature pass left for the selected cells
        PhiGrad G;
        float fs[3] = {0.f, 0.f, 0.f};
        if constexpr (TP) {
            const float4 g = sg[z & 1][tid];
            G.phi = sphi[ring(z)][lc];
            G.g[0] = g.x;
            G.g[1] = g.y;
            G.g[2] = g.z;
            const float c = ML ? cs : g.w;
#pragma unroll
            for (int a = 0; a < 3; a++) fs[a] = c * G.g[a];
            if constexpr (ML) {
                if (sel) surface_blend(G, cs, P, g.w, grad_norm(G), y, fs);
                cs = csn;
                sel = seln;
            }
        }
        {
            // moments -> forces, velocity
            Macro m;
            site_macro<TP, PH>(M, G, fs, aext, P, m);

            // regularised collision, written to this site's own slots
            float h[27];
            collide(m, m.omega, h);
            const __amdgpu_buffer_rsrc_t dst = plane_rsrc(fout + (size_t)zp(z) * 27, pbytes);
            uint32_t soff = srow(1) * ES;
#pragma unroll
            for (int i = 0; i < 27; i++) {
                bstore<T, NT ? STORE_NT : 0>(dst, own_v * ES, soff,
                                             Pop<S>::enc_step(h[i], __builtin_bit_cast(uint32_t, h[(i + 1) % 27])));
                soff += pstep;
                asm volatile("" : "+s"(soff));
            }

            if constexpr (TP) {  // velocity of this step, advects phi in the next one
                put(B.uout, z, m.u[0]);
                put(B.uout + N, z, m.u[1]);
                put(B.uout + 2 * (size_t)N, z, m.u[2]);
            }
        }
    }
}

// The learned-curvature pass over one work item, ahead of the step: at every
// interface cell (0.02 < phi < 0.98) it leaves in B.mlpy (float4 per site) the
// network output where the curvature criterion selects the cell and NaN
// elsewhere.  The 3^3 stencil needs phi at halo 1 only, so the pass stages a
// (TW + 2) x (256/TW + 2) tile in a four-plane ring (the step stages halo 3 and
// seven planes for WENO-5): half the phi bytes per item.  The staged values,
// the stencil and the criterion are the step's, so the step selects exactly
// the cells written here.  A work item none of whose sites is an interface
// cell is skipped: its flags are the x-segments of its rows in its planes.
// W: the weights in LDS; *loaded: the weights W holds (reloaded when a box of
// the batch brings others).
template <int TW, bool FX>
__device__ __forceinline__ void pass_tile(const Params &P, const Buffers &B, const uint32_t L, MlpW &W,
                                          MlpWave *wave_lds, const void *&loaded)
{
    using PS = PhiStore<FX>;
    using PT = typename PS::T;
    constexpr int TXW = TW, TYW = NTHREADS / TW;
    constexpr int PX = TXW + 2, PY = TYW + 2, PLANE = PX * PY;
    constexpr int LOADS = (PLANE + NTHREADS - 1) / NTHREADS;
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * TXW + tx;
    const int bx = (int)(L % (uint32_t)P.gx), by = (int)((L / (uint32_t)P.gx) % (uint32_t)P.gy);
    const int bz = (int)(L / ((uint32_t)P.gx * (uint32_t)P.gy));
    const int x0 = bx * TXW, y0 = by * TYW, z0 = bz * P.zchunk;
    const int zend = min(z0 + P.zchunk, nz);
    // lanes past a ragged box edge evaluate the periodic image of their site
    // and write the owner's bits again
    const int xg = (x0 + tx) % nx, yg = (y0 + ty) % ny;
    // planes zs .. ze-1 of the chunk hold every interface cell of the item:
    // the first and last planes with a flag set (a candidate cell of plane z
    // sets its segment's flag of plane z)
    int zs = z0, ze = zend;
    if (B.iflag) {
        __shared__ int s_kmin, s_kmax;
        const int nseg = flag_segments(nx);
        const int s0 = x0 / 32, ns = min((x0 + TXW + 31) / 32, nseg) - s0;
        const int nr = min(TYW, ny - y0), np = zend - z0;
        if (tid == 0) {
            s_kmin = np;
            s_kmax = -1;
        }
        __syncthreads();
        int kmin = np, kmax = -1;
        for (int e = tid; e < ns * nr * np; e += NTHREADS) {
            const int si = e % ns, r = (e / ns) % nr, k = e / (ns * nr);
            if (B.iflag[((size_t)(z0 + k) * ny + (y0 + r)) * nseg + s0 + si] != 0) {
                kmin = min(kmin, k);
                kmax = max(kmax, k);
            }
        }
        if (kmax >= 0) {
            atomicMin(&s_kmin, kmin);
            atomicMax(&s_kmax, kmax);
        }
        __syncthreads();
        if (s_kmax < 0) return;  // uniform: no interface cell in the item
        zs = z0 + s_kmin;
        ze = z0 + s_kmax + 1;
    }
    if (P.mlp != loaded) {  // uniform: one box per work item
        load_weights(gconst((const uint16_t *)P.mlp), W, tid);
        loaded = P.mlp;
    }
    const LBM_GLOBAL PT *__restrict__ phin = gconst((const PT *)B.phin);
    LBM_GLOBAL float *__restrict__ yout = gmut((float *)B.mlpy);
    __shared__ float sphi[4][PLANE];
    __shared__ uint32_t sxy[PLANE];
#pragma unroll
    for (int k = 0; k < LOADS; k++) {
        const int e = tid + k * NTHREADS;
        const int ly = e / PX, lx = e - ly * PX;
        if (e < PLANE) sxy[e] = (uint32_t)modi(y0 + ly - 1, ny) * nx + (uint32_t)modi(x0 + lx - 1, nx);
    }
    __syncthreads();
    // phi planes in flight: three register sets, each fetched three planes
    // ahead of its store into the ring (one plane of work is too short to
    // hide a load from memory); every fetch and store is unconditional (a
    // plane past the chunk re-reads a valid plane) so that the compiler waits
    // for exactly the set it stores
    PT ra[LOADS], rb[LOADS], rc[LOADS];
    auto fetch_plane = [&](PT(&r)[LOADS], int z) {
        const LBM_GLOBAL PT *src = phin + (uint32_t)wrapi(z, nz) * plane;
#pragma unroll
        for (int k = 0; k < LOADS; k++) {
            const int e = tid + k * NTHREADS;
            r[k] = src[sxy[e < PLANE ? e : PLANE - 1]];  // spare lanes re-read the last point
        }
    };
    auto store_plane = [&](const PT(&r)[LOADS], int z) {
        float *dst = sphi[(z + 4) & 3];
#pragma unroll
        for (int k = 0; k < LOADS; k++) {
            const int e = tid + k * NTHREADS;
            if (e < PLANE) dst[e] = PS::f32(r[k]);
        }
    };
    const int lc = (ty + 1) * PX + (tx + 1);  // own phi tile index
    const uint32_t own_xy = (uint32_t)yg * nx + xg;
    // stencil, criterion and network of plane z (planes z-1 .. z+1 in the ring)
    auto compute = [&](int z) {
        const float *pm = sphi[(z + 3) & 3];
        const float *pc = sphi[z & 3];
        const float *pp = sphi[(z + 1) & 3];
        const float c0 = pc[lc];
        const bool cand = c0 > 0.02f && c0 < 0.98f;
        if (__ballot(cand) == 0ull) return;  // most waves hold no interface cell
        float ph[27];
        float y[4] = {0.f, 0.f, 0.f, 0.f};
        bool sel = false;
        if (cand) {
#pragma unroll
            for (int i = 0; i < 27; i++) {
                const float *pl = CZ(i) < 0 ? pm : (CZ(i) > 0 ? pp : pc);
                ph[i] = pl[lc + CY(i) * PX + CX(i)];
            }
            PhiGrad G;
            float kfd, gn;
            M10 M;
            phi_stencil(ph, M, G);
            sel = mlp_select(G, P, kfd, gn);
        }
        mlp_wave(W, wave_lds[tid >> 6], sel, ph, y, tid & 63);
        if (cand) {
            const float nan = __builtin_nanf("");
            LBM_GLOBAL float *yo = yout + 4 * (size_t)((uint32_t)z * plane + own_xy);
            yo[0] = sel ? y[0] : nan;
            yo[1] = sel ? y[1] : nan;
            yo[2] = sel ? y[2] : nan;
            yo[3] = sel ? y[3] : nan;
        }
    };
    // plane z: plane z+1 into the ring (its slot held z-3, last read two
    // planes ago), plane z+4 into the freed register set, one barrier
    auto plane_step = [&](int z, PT(&r)[LOADS]) {
        store_plane(r, z + 1);
        fetch_plane(r, z + 4);
        lds_barrier();
        if (z < ze) compute(z);
    };
    fetch_plane(ra, zs - 1);
    store_plane(ra, zs - 1);
    fetch_plane(ra, zs);
    store_plane(ra, zs);
    // issued in this order (the compiler would otherwise reorder the three
    // sets, and the first wait of every pass through the loop would then
    // cover all of them)
    fetch_plane(ra, zs + 1);
    asm volatile("" ::: "memory");
    fetch_plane(rb, zs + 2);
    asm volatile("" ::: "memory");
    fetch_plane(rc, zs + 3);
    for (int z = zs; z < ze; z += 3) {
        plane_step(z, ra);
        plane_step(z + 1, rb);
        plane_step(z + 2, rc);
    }
}

// ------------------------------------------------------------ work queue
// The persistent loop of a batched launch over the boxes of a batch: a
// workgroup takes the next work item from one queue counter per launch, so the
// load stays balanced to the last item; item k belongs to the box b with
// first[b] <= k < first[b + 1].  The counter of this launch is counter[parity];
// the launch clears the other one for the next launch on the stream.
// body(b, item within the box) runs with every thread of the workgroup.
// (Per-die queues, each die draining a contiguous range of items first so that
// neighbouring tiles share its L2, cut the L2-miss reads by a fifth (FP32) to a
// third (FP16) but made the FP32 step 2.5 % slower and left FP16 unchanged: the
// step is not bound by the L2-miss traffic, and one queue keeps all dies on the
// same z range.)
// A workgroup's first item is its own index in the grid, the queue hands out
// the items after those, and a launch of no more items than workgroups does
// without it: the atomic additions of a whole grid on one counter take about
// 10 ns each (a single-phase step of an 8^3 box, 1792 resident workgroups,
// 26 us).
template <int TW, class Body>
__device__ __forceinline__ void batch_loop(const uint32_t *__restrict__ first, int nbox, uint32_t *counter,
                                           int parity, Body body)
{
    __shared__ uint32_t s_item;
    const int tid = threadIdx.y * TW + threadIdx.x;
    const uint32_t total = first[nbox];
    if (blockIdx.x == 0 && tid == 0) counter[parity ^ 1] = 0u;
    for (uint32_t item = blockIdx.x; item < total;) {
        int lo = 0, hi = nbox - 1;  // last box with first[b] <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (first[mid] <= item) lo = mid;
            else hi = mid - 1;
        }
        const int b = __builtin_amdgcn_readfirstlane(lo);
        body(b, item - first[b]);
        if (total <= gridDim.x) break;
        if (tid == 0) s_item = gridDim.x + atomicAdd(&counter[parity], 1u);
        __syncthreads();  // the item's LDS traffic is over
        item = (uint32_t)__builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();  // s_item read by all
    }
}

// One Runge-Kutta stage of the phase field of one or many boxes, on the same
// work items as the step (buf[b].phin: the stage input, buf[b].phin0: phi^n,
// buf[b].phout: the stage output).  Bound by vector issue and its latency, so
// by the waves per SIMD: four fit (107 registers, 40,608 bytes of LDS per
// workgroup with two planes of halo sums instead of three) where three did, and
// a 256^3 time step of two stages, step and network passes went from 1.72 to
// 1.65 ms.
template <int TW>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(4)))
k_ac_stage_batch(const Params *__restrict__ tab, const Buffers *__restrict__ buf, const uint32_t *__restrict__ first,
                 int nbox, uint32_t *counter, int parity, double rk_a, double rk_b)
{
    batch_loop<TW>(first, nbox, counter, parity, [&](int b, uint32_t L) {
        step_tile<0, true, false, false, TW, false, false, true>(tab[b], buf[b], L, rk_a, rk_b);
    });
}

// The learned-curvature pass of one or many boxes ahead of their step, on the
// same work items (buf[b].phin: phi^n; buf[b].mlpy: the network outputs the
// step reads).
template <int TW, bool FX>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3)))
k_mlp_pass_batch(const Params *__restrict__ tab, const Buffers *__restrict__ buf, const uint32_t *__restrict__ first,
                 int nbox, uint32_t *counter, int parity)
{
    __shared__ MlpW w_lds;
    __shared__ MlpWave wave_lds[NTHREADS / 64];
    const void *loaded = nullptr;
    batch_loop<TW>(first, nbox, counter, parity, [&](int b, uint32_t L) {
        pass_tile<TW, FX>(tab[b], buf[b], L, w_lds, wave_lds, loaded);
    });
}

// The time step of one or many independent boxes in one launch (a single box
// is a batch of one); tab[b] and buf[b] are the box's parameters and this
// step's buffers.
template <int S, bool TP, bool FRC, bool ML, int TW, bool FX, bool PH, bool NT>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3)))
k_step_batch(const Params *__restrict__ tab, const Buffers *__restrict__ buf, const uint32_t *__restrict__ first,
             int nbox, uint32_t *counter, int parity)
{
    batch_loop<TW>(first, nbox, counter, parity, [&](int b, uint32_t L) {
        step_tile<S, TP, FRC, ML, TW, NT, FX, false, PH>(tab[b], buf[b], L);
    });
}

// ------------------------------------------------------- step dispatch
// template dispatch: storage x two-phase x forcing x learned curvature
// (the learned curvature exists only with the phase field)
#define LBM_DISPATCH_S(S_, tp, frc, ml, CALL)                                  \
    do {                                                                       \
        if (tp) {                                                              \
            if (ml) { if (frc) CALL(S_, true, true, true) else CALL(S_, true, false, true) } \
            else { if (frc) CALL(S_, true, true, false) else CALL(S_, true, false, false) }  \
        } else {                                                               \
            if (frc) CALL(S_, false, true, false) else CALL(S_, false, false, false)        \
        }                                                                      \
    } while (0)
#define LBM_DISPATCH(storage, tp, frc, ml, CALL)                               \
    do {                                                                       \
        if (storage == 0) LBM_DISPATCH_S(0, tp, frc, ml, CALL);                \
        else if (storage == 1) LBM_DISPATCH_S(1, tp, frc, ml, CALL);           \
        else LBM_DISPATCH_S(2, tp, frc, ml, CALL);                             \
    } while (0)

// Non-temporal stores are a template parameter: chosen at run time inside the
// kernel, the two store sequences made the compiler's counting of the
// operations in flight lose the 27 stores, and every plane then waited for the
// previous plane's stores before it used its populations.
// the step kernel also takes the phi storage and whether buoyancy or a
// viscosity contrast is compiled in (both exist only with the phase field)
#define LBM_STEP_CALL(S_, TP_, F_, M_)                                                               \
    {                                                                                                \
        if constexpr (TP_) {                                                                         \
            if (fix) {                                                                               \
                if (phys) STEP_CALL(S_, TP_, F_, M_, true, true) else STEP_CALL(S_, TP_, F_, M_, true, false) \
            } else {                                                                                 \
                if (phys) STEP_CALL(S_, TP_, F_, M_, false, true) else STEP_CALL(S_, TP_, F_, M_, false, false) \
            }                                                                                        \
        } else                                                                                       \
            STEP_CALL(S_, TP_, F_, M_, false, false)                                                 \
    }

// Occupancy-sized persistent grid and launch of the step kernel for one
// population storage S; each storage is instantiated in a translation unit
// of its own (lbm_step_s0/s1/s2.hip) so that the build compiles them in parallel.
// nt: non-temporal stores (tile 64, and with FP32 populations 32, whose rows are whole lines too)
#define LBM_STEP_TILE(S_, TP_, F_, M_, X_, H_, CALL)                                   \
    {                                                                                  \
        if (tile == 32) {                                                              \
            if (S_ == 0 && nt) CALL((k_step_batch<S_, TP_, F_, M_, 32, X_, H_, S_ == 0>)) \
            else CALL((k_step_batch<S_, TP_, F_, M_, 32, X_, H_, false>))              \
        } else if (nt) CALL((k_step_batch<S_, TP_, F_, M_, 64, X_, H_, true>))         \
        else CALL((k_step_batch<S_, TP_, F_, M_, 64, X_, H_, false>))                  \
    }
template <int S>
int step_grid(bool tp, bool frc, bool ml, bool fix, bool phys, int tile, bool nt)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
#define STEP_GRID(K) (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, K, NTHREADS, 0);
#define STEP_CALL(S_, TP_, F_, M_, X_, H_) LBM_STEP_TILE(S_, TP_, F_, M_, X_, H_, STEP_GRID)
    LBM_DISPATCH_S(S, tp, frc, ml, LBM_STEP_CALL);
#undef STEP_CALL
#undef STEP_GRID
    return per_cu * cus;
}

template <int S>
hipError_t step_launch(const Params *tab, const Buffers *buf, const uint32_t *first, int nbox, uint32_t *counter,
                       int parity, bool tp, bool frc, bool ml, bool fix, bool phys, int tile, bool nt, int grid,
                       hipStream_t s)
{
    dim3 g(grid), block(tile, NTHREADS / tile, 1);
#define STEP_LAUNCH(K) hipLaunchKernelGGL(K, g, block, 0, s, tab, buf, first, nbox, counter, parity);
#define STEP_CALL(S_, TP_, F_, M_, X_, H_) LBM_STEP_TILE(S_, TP_, F_, M_, X_, H_, STEP_LAUNCH)
    LBM_DISPATCH_S(S, tp, frc, ml, LBM_STEP_CALL);
#undef STEP_CALL
#undef STEP_LAUNCH
    return hipGetLastError();
}

}  // namespace lbm
