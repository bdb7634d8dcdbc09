// Hand-written gfx950 kernels of one accLB time step (arXiv 2505.01126, Secs. 2-3)
// other than the step itself (whose device code is in lbm_step.h): the initial
// state, field read-out, reductions, the Runge-Kutta phase-field stage, and the
// host launchers.
#include "lbm_step.h"

namespace lbm {

extern template int step_grid<0>(bool, bool, bool, bool, bool, int, bool);
extern template int step_grid<1>(bool, bool, bool, bool, bool, int, bool);
extern template int step_grid<2>(bool, bool, bool, bool, bool, int, bool);
extern template hipError_t step_launch<0>(const Params *, const Buffers *, const uint32_t *, int, uint32_t *, int, bool,
                                          bool, bool, bool, bool, int, bool, int, hipStream_t);
extern template hipError_t step_launch<1>(const Params *, const Buffers *, const uint32_t *, int, uint32_t *, int, bool,
                                          bool, bool, bool, bool, int, bool, int, hipStream_t);
extern template hipError_t step_launch<2>(const Params *, const Buffers *, const uint32_t *, int, uint32_t *, int, bool,
                                          bool, bool, bool, bool, int, bool, int, hipStream_t);

// ------------------------------------------------------------- row marches
// The marches below walk a box as the step does: a workgroup takes 256 sites of
// a plane through a chunk of z planes, one site per lane, so that the sums over a
// plane of a stencil are formed once and carried to the two planes above, and
// the addresses are 32-bit offsets in one plane (a thread per site, gathering
// its whole stencil through 64-bit addresses, spent its time on those: 624
// vector instructions per site in the FP16 read-out, and 27 phi loads).
//
// wx > 0: each wave takes 64 sites of one x-row, so that rows are wave-uniform
// (scalar offsets), and wx waves stand side by side in x: the lines that a
// shifted row of populations shares with the next 64 sites are then fetched
// once.  With the phase field and 16-bit populations the waves
// take four rows instead, which then share their phi rows (512^3 FP16 read-out:
// 2.62 ms against 2.77).  Lanes past the box's edge repeat a periodic image and
// its writes (the same bits), so that no memory operation is conditional and the
// compiler counts those in flight exactly.
// wx = 0: 256 consecutive sites of the plane, in boxes too small for chunks of
// three planes on every compute unit and where nx is no multiple of 64: rows then
// end inside a wave and inside a memory line (190^3: reduction of FP16 133 us
// against 145 by rows, read-out of FP32 197 us against 231; 300^3: 496 and 534,
// 752 and 849).
inline int march_wx(const Params &p, bool rows)
{
    auto fits = [&](int w) { return (p.nx + w - 1) / w * w * 10 <= p.nx * 11; };
    if (p.nx % 64 != 0 || (int64_t)p.nx * p.ny * p.nz < (int64_t)NTHREADS * 6 * RED_BLOCKS) return 0;
    return rows || !fits(128) ? 1 : (fits(256) ? 4 : 2);
}
template <bool ROW> struct RowMarch {
    int nx, ny, nz, y, z0, zend;
    uint32_t plane, xs[3], ys[3];  // periodic neighbours' columns and row offsets (k = 1 + offset)
    bool in_row, in_box;           // the wave has sites of the box; so has the lane
    __device__ __forceinline__ RowMarch(const Params &P, uint32_t L, int chunk, int wx)
    {
        nx = P.nx;
        ny = P.ny;
        nz = P.nz;
        plane = (uint32_t)nx * (uint32_t)ny;
        int x;
        if constexpr (ROW) {
            const int wy = 4 / wx, wave = (int)(threadIdx.x >> 6);
            const uint32_t gx = (nx + 64 * wx - 1) / (64 * wx), gy = (ny + wy - 1) / wy;
            x = ((int)(L % gx) * wx + wave % wx) * 64 + (int)(threadIdx.x & 63);
            y = __builtin_amdgcn_readfirstlane((int)(L / gx % gy) * wy + wave / wx);
            z0 = (int)(L / (gx * gy)) * chunk;
            in_row = y < ny;
            in_box = in_row && x < nx;
            x %= nx;
            y = in_row ? y : 0;
        } else {
            const uint32_t gp = (plane + NTHREADS - 1) / NTHREADS, e = L % gp * NTHREADS + threadIdx.x;
            z0 = (int)(L / gp) * chunk;
            in_row = true;
            in_box = e < plane;
            x = (int)((in_box ? e : plane - 1) % (uint32_t)nx);
            y = (int)((in_box ? e : plane - 1) / (uint32_t)nx);
        }
        zend = min(z0 + chunk, nz);
#pragma unroll
        for (int k = 0; k < 3; k++) {
            xs[k] = (uint32_t)wrapi(x + k - 1, nx);
            ys[k] = (uint32_t)wrapi(y + k - 1, ny) * (uint32_t)nx;
        }
    }
    __device__ __forceinline__ uint32_t srow(int ky) const { return ROW ? ys[ky] : 0u; }
    __device__ __forceinline__ uint32_t vcol(int ky, int kx) const { return ROW ? xs[kx] : ys[ky] + xs[kx]; }
    template <class E> __device__ __forceinline__ __amdgpu_buffer_rsrc_t field(const E *base, int z) const
    {
        return plane_rsrc(base + (uint32_t)z * plane, plane * (uint32_t)sizeof(E));
    }
    template <class E> __device__ __forceinline__ E at(const E *base, int z, int ky, int kx) const
    {
        return bload<E>(field(base, z), vcol(ky, kx) * (uint32_t)sizeof(E), srow(ky) * (uint32_t)sizeof(E));
    }
    // the nine values of plane z (periodic) around the site
    template <class E> __device__ __forceinline__ void at9(const E *base, int z, E (&v)[9]) const
    {
        const __amdgpu_buffer_rsrc_t r = field(base, wrapi(z, nz));
#pragma unroll
        for (int i = 0; i < 9; i++)
            v[i] = bload<E>(r, vcol(i / 3, i % 3) * (uint32_t)sizeof(E), srow(i / 3) * (uint32_t)sizeof(E));
    }
    // base may be null: a buffer of no bytes, whose stores the hardware drops.
    // Its scalar offset is zero then: the range check is vector offset >= bytes -
    // scalar offset, a difference that must not go below zero.
    template <bool NT, class E> __device__ __forceinline__ void put(E *base, int z, E v) const
    {
        const uint32_t bytes = base ? plane * (uint32_t)sizeof(E) : 0u;
        bstore<E, NT ? STORE_NT : 0>(plane_rsrc(base ? base + (uint32_t)z * plane : base, bytes),
                                     vcol(1, 1) * (uint32_t)sizeof(E), base ? srow(1) * (uint32_t)sizeof(E) : 0u, v);
    }
};
int64_t march_tiles(const Params &p, int wx)
{
    if (wx == 0) return ((int64_t)p.nx * p.ny + NTHREADS - 1) / NTHREADS;
    const int wy = 4 / wx;
    return (int64_t)((p.nx + 64 * wx - 1) / (64 * wx)) * ((p.ny + wy - 1) / wy);
}
// planes per workgroup: `rounds` workgroups for each that is resident, at most 16
// (the chunk's first two planes of sums are extra work)
int march_chunk(const Params &p, int wx, int rounds = 2)
{
    const int64_t c = march_tiles(p, wx) * p.nz / (rounds * RED_BLOCKS);
    return (int)(c < 1 ? 1 : (c < 16 ? c : 16));
}
// The same for the reduction of a box whose launch has few rounds of workgroups
// (up to 2^21 sites): the length that brings it through them soonest, a workgroup
// costing its planes and the two before them (80^3 FP32: 28.2 -> 23.3 us, a thread
// per site 25; 128^3: 52 -> 48).  A larger box is bound by memory and not by its
// rounds (150 x 141 x 203: 114 us by this rule, 110 by the one above).
int even_chunk(const Params &p, int wx)
{
    const int64_t tiles = march_tiles(p, wx);
    int best = 1;
    int64_t cost = 0;
    for (int c = 1; c <= 16; c++) {
        const int64_t items = tiles * ((p.nz + c - 1) / c), t = (items + RED_BLOCKS - 1) / RED_BLOCKS * (c + 2);
        if (c == 1 || t < cost) {
            best = c;
            cost = t;
        }
    }
    return best;
}

// How a kernel goes through a box: by sites, one thread per site, or by a march.
struct Plan {
    bool sites;
    int wx, chunk;
    bool nt = false;  // a march's fields are stored non-temporally
};
// The plane's sites fill less than `tenths` tenths of the lanes that a march puts
// on it: 256 lanes walk z for 64 sites of 8 x 8, 512 for 289 of 17 x 17.
bool thin(const Params &p, int tenths)
{
    return (int64_t)p.nx * p.ny * 10 < march_tiles(p, 0) * NTHREADS * tenths;
}
// Fields too large to stay in the caches until they are read are stored
// non-temporally.  The initial phi and u of a box from 1.18 M sites on: set-up and
// first step of 400 x 400 x 60 1.14 ms, 1.19 cached; of 32^3 to 64^3 up to 10 us
// less cached.  The fields of a read-out whose rows are whole lines (512^3: 4.00 ms, 4.13
// cached), and those that do not fit the 256 MB Infinity Cache together with the
// state they are read from: cached, they push out what the next step or read-out
// needs (268 x 40 x 207 FP32, set-up and read-out: 227 us, 237 cached; 190 x 130 x 170
// FP16, read-outs alone: 85 us, 94 cached; a pass over u and phi after each costs 2-5 %
// more then, up to 250^3, where it gains 10).  Below, cached fields are as fast to
// write and 2-4 % faster to use (129 x 120 x 116 FP32: 72 us with the pass, 75).
bool large(const Params &p, int64_t sites) { return (int64_t)p.nx * p.ny * p.nz >= sites; }
// Set-up.  By sites on thin planes (8 x 8 x 65536: 321 us against 570; 17 x 17 x
// 4000: 127 and 140); 20 x 20, which fills 0.78 of the lanes, is even, and full
// planes gain by the march (256^3: 0.80 against 1.1 ms).
Plan plan_init(const Params &p)
{
    const int wx = march_wx(p, false);
    return {thin(p, 6), wx, march_chunk(p, wx), large(p, (int64_t)NTHREADS * 6 * RED_BLOCKS)};
}
// Read-out (fields) and reduction.  In single phase there is no stencil whose sums
// a march could carry, and a thread per site reads its 27 populations as fast or
// faster: FP16 reduction of 190^3 in 96 us against 230, of 256^3 in 203 against
// 266; FP32 read-out of 190^3 in 176 us against 195, of 257 x 255 x 256 in 393
// against 454. With the phase field the march wins except on thin planes (8 x 8 x
// 65536: FP32 read-out 151 us by sites against 255; 17 x 17 x 4000: 35 and 42, but
// with the fixed-point phi 46 and 34). With the learned curvature a wave with many
// selected cells runs the network for them plane after plane: the march needs six
// workgroups for each resident one to hide that, and planes that fill the lanes
// (40 x 17 x 2000 FP16 read-out: 68 us by sites, 93 in chunks of 3; reduction of
// 13 x 200 x 500: 72 us in chunks of 1, 111 of 3).  A read-out of less than two
// planes per workgroup goes by sites (64^3: 22 us against 25); the reduction gains
// from the first plane on (64^3: 29 and 35).
Plan plan_read(const Params &p, int storage, bool fields)
{
    if (!p.two_phase) return {true, 0, 0};
    const int wx = march_wx(p, storage != 0);
    const bool nt = wx || large(p, 256000000 / (27 * (storage ? 2 : 4) + 36));
    if (p.curv_mode == 1) {
        const int c = march_chunk(p, wx, 6);
        return {thin(p, 8) || (fields && c < 2), wx, c, nt};
    }
    const bool few = !fields && (int64_t)p.nx * p.ny * p.nz <= 1 << 21;
    return {thin(p, p.phi_fix ? 5 : 6), wx, few ? even_chunk(p, wx) : march_chunk(p, wx), nt};
}
uint32_t site_blocks(const Params &p) { return ((uint32_t)p.nx * p.ny * p.nz + NTHREADS - 1) / NTHREADS; }
uint32_t march_items(const Params &p, int chunk, int wx)
{
    return (uint32_t)(march_tiles(p, wx) * ((p.nz + chunk - 1) / chunk));
}

// ----------------------------------------------------------- initial state
// f^0 = f^eq(p*0, u0) + w H : A0 / (2 c_s^4), A0 = -c_s^2 tau (grad u0 + grad u0^T),
// written pre-shifted (slot of x - c_i) so that the first pull yields f^0 at x.
// FP64 throughout.
//
// The populations h_i of a site with velocity u, its gradient G[a][b] = d_b u_a,
// phase field ph and pressure ps: put(i, h_i)
template <class Put>
__device__ __forceinline__ void init_pops(const Params &P, const double (&u)[3], const double (&G)[3][3], double ph,
                                          double ps, Put put)
{
    double tau = 1.0 / (double)P.omega;
    if (P.two_phase && P.tau_g > 0.0f) {  // relaxation time of the initial phase field
        const double c = fmin(fmax(ph, 0.0), 1.0);
        tau = c * (double)P.tau_l + (1.0 - c) * (double)P.tau_g;
    }
    double A[3][3];
#pragma unroll
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) A[a][b] = -(tau / 3.0) * (G[a][b] + G[b][a]);
    const double dp = ps - (double)P.p0;
    const double u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
#pragma unroll
    for (int i = 0; i < 27; i++) {
        const double c[3] = {(double)CX(i), (double)CY(i), (double)CZ(i)};
        const double cu = c[0] * u[0] + c[1] * u[1] + c[2] * u[2];
        double hA = 0.0;
        for (int a = 0; a < 3; a++)
            for (int b = 0; b < 3; b++) hA += (c[a] * c[b] - (a == b ? 1.0 / 3.0 : 0.0)) * A[a][b];
        put(i, (float)(dp + 3.0 * cu + 4.5 * cu * cu - 1.5 * u2 + 4.5 * hA));
    }
}
// nearest point of the fixed-point grid, clamped to its range [-2, 2)
__device__ __forceinline__ int32_t phi_to_fix(double ph)
{
    return (int32_t)__builtin_rint(fmin(fmax(ph * 0x1p30, -0x1p31), 0x1p31 - 1.0));
}

// by sites
template <int S>
__global__ void __launch_bounds__(NTHREADS) k_init_site(Params P, void *fout_, void *phi_out, float *u_out,
                                                        const double *phi0, const double *u0, const double *ps0)
{
    using T = typename Pop<S>::T;
    T *fout = (T *)fout_;
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    const uint32_t plane = (uint32_t)nx * ny, N = plane * (uint32_t)nz;
    const uint32_t s = blockIdx.x * NTHREADS + threadIdx.x;
    if (s >= N) return;
    const int x = s % nx, y = (s / nx) % ny, z = s / plane;
    double u[3] = {0, 0, 0}, G[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    if (u0) {
        for (int a = 0; a < 3; a++) u[a] = u0[(size_t)a * N + s];
#pragma unroll
        for (int i = 0; i < 27; i++) {
            const uint32_t t = (uint32_t)wrapi(z + CZ(i), nz) * plane + (uint32_t)wrapi(y + CY(i), ny) * nx +
                               (uint32_t)wrapi(x + CX(i), nx);
            for (int a = 0; a < 3; a++) {
                const double v = 3.0 * WTD(i) * u0[(size_t)a * N + t];
                G[a][0] += v * CX(i);
                G[a][1] += v * CY(i);
                G[a][2] += v * CZ(i);
            }
        }
    }
    const double ph = P.two_phase ? phi0[s] : 0.0;
    init_pops(P, u, G, ph, ps0 ? ps0[s] : (double)P.p0, [&](int i, float h) {
        const size_t slot = ((size_t)wrapi(z - CZ(i), nz) * 27 + i) * plane + (uint32_t)wrapi(y - CY(i), ny) * nx +
                            (uint32_t)wrapi(x - CX(i), nx);
        fout[slot] = Pop<S>::enc(h);
    });
    if (phi_out) {
        if (P.phi_fix) ((int32_t *)phi_out)[s] = phi_to_fix(ph);
        else ((double *)phi_out)[s] = ph;
    }
    if (u_out)
        for (int a = 0; a < 3; a++) u_out[(size_t)a * N + s] = (float)u[a];
}

// The march: each plane of u0 is loaded once, for the gradients of the three
// planes it enters (27 loads per site instead of 81): the sums of site z+1 and
// z+2 are under way while those of z are completed, each in the order of the
// velocities.
template <int S, bool ROW, bool NT>
__global__ void __launch_bounds__(NTHREADS) k_init(Params P, void *fout_, void *phi_out, float *u_out,
                                                   const double *phi0, const double *u0, const double *ps0, int chunk,
                                                   int wx)
{
    using T = typename Pop<S>::T;
    constexpr uint32_t ES = sizeof(T);
    T *fout = (T *)fout_;
    const RowMarch<ROW> R(P, blockIdx.x, chunk, wx);
    if (!R.in_row) return;
    const uint32_t plane = R.plane;
    const size_t N = (size_t)plane * (uint32_t)R.nz;
    // G[b] += d_b u terms of the velocities i0 .. i0 + 8, v: u there
    auto grad = [](auto i0, const double (&v)[9], double (&G)[3]) {
#pragma unroll
        for (int j = 0; j < 9; j++) {
            constexpr int I0 = decltype(i0)::value;
            const double t = 3.0 * WTD(I0 + j) * v[j];
            if (CX(I0 + j)) G[0] += t * CX(I0 + j);
            if (CY(I0 + j)) G[1] += t * CY(I0 + j);
            if (CZ(I0 + j)) G[2] += t * CZ(I0 + j);
        }
    };
    using Low = std::integral_constant<int, 0>;
    using Mid = std::integral_constant<int, 9>;
    using Top = std::integral_constant<int, 18>;
    double G[3][3], Gn[3][3];  // d_b u_a at z and z+1: the planes up to z
    double u[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) G[a][b] = Gn[a][b] = 0.0;
    if (u0) {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            double v[9];
            R.at9(u0 + a * N, R.z0 - 1, v);
            grad(Low{}, v, G[a]);
            R.at9(u0 + a * N, R.z0, v);
            grad(Mid{}, v, G[a]);
            grad(Low{}, v, Gn[a]);
            u[a] = v[4];
        }
    }
    for (int z = R.z0; z < R.zend; z++) {
        double un[3] = {0, 0, 0}, Gnn[3][3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            for (int b = 0; b < 3; b++) Gnn[a][b] = 0.0;
            if (u0) {
                double v[9];
                R.at9(u0 + a * N, z + 1, v);
                grad(Top{}, v, G[a]);
                grad(Mid{}, v, Gn[a]);
                grad(Low{}, v, Gnn[a]);
                un[a] = v[4];
            }
        }
        const double ph = P.two_phase ? R.at(phi0, z, 1, 1) : 0.0;
        __amdgpu_buffer_rsrc_t dst[3];  // slots of z - cz: row y - cy, column x - cx of population i
#pragma unroll
        for (int k = 0; k < 3; k++)
            dst[k] = plane_rsrc(fout + (size_t)((uint32_t)wrapi(z + 1 - k, R.nz) * plane) * 27, 27u * plane * ES);
        init_pops(P, u, G, ph, ps0 ? R.at(ps0, z, 1, 1) : (double)P.p0, [&](int i, float h) {
            bstore<T>(dst[CZ(i) + 1], R.vcol(1 - CY(i), 1 - CX(i)) * ES, ((uint32_t)i * plane + R.srow(1 - CY(i))) * ES,
                      Pop<S>::enc(h));
        });
        if (P.phi_fix) R.template put<NT>((int32_t *)phi_out, z, phi_to_fix(ph));
        else R.template put<NT>((double *)phi_out, z, ph);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            R.template put<NT>(u_out ? u_out + a * N : u_out, z, (float)u[a]);
            u[a] = un[a];
            for (int b = 0; b < 3; b++) {
                G[a][b] = Gn[a][b];
                Gn[a][b] = Gnn[a][b];
            }
        }
    }
}

// -------------------------------------------------- fields and reductions
// By sites: macroscopic state at time n of site s (pull + stencils from global
// memory).  Every lane of the wave calls this together (the network stage is a
// wave-wide MFMA); lanes with valid == false only take part in that stage.
template <int S, bool TP, bool FRC, bool ML>
__device__ __forceinline__ void site_state(const Params &P, const void *fin_, const void *phi, uint32_t s, bool valid,
                                           Macro &m, const MlpW &W, MlpWave &wv)
{
    using T = typename Pop<S>::T;
    const T *fin = (const T *)fin_;
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    const uint32_t plane = (uint32_t)nx * ny;
    const int x = s % nx, y = (s / nx) % ny, z = s / plane;
    // the periodic neighbours' coordinates, once per site: index k = 1 + offset
    const uint32_t xk[3] = {(uint32_t)wrapi(x - 1, nx), (uint32_t)x, (uint32_t)wrapi(x + 1, nx)};
    const uint32_t yk[3] = {(uint32_t)wrapi(y - 1, ny) * nx, (uint32_t)y * nx, (uint32_t)wrapi(y + 1, ny) * nx};
    const uint32_t zk[3] = {(uint32_t)wrapi(z - 1, nz), (uint32_t)z, (uint32_t)wrapi(z + 1, nz)};
    M10 M;
    PhiGrad G;
    float ph[27];
    float kfd = 0.f, gn = 0.f, cs = 0.f;
    bool sel = false;
    if (valid) {
        float hv[27];
#pragma unroll
        for (int i = 0; i < 27; i++)  // population i of site s - c_i
            hv[i] = Pop<S>::dec(fin[((size_t)zk[1 - CZ(i)] * 27 + i) * plane + yk[1 - CY(i)] + xk[1 - CX(i)]]);
        moments10(hv, M);
        if constexpr (TP) {
            M10 Mp;
#pragma unroll
            for (int i = 0; i < 27; i++)
                ph[i] = (float)phi_load(phi, zk[1 + CZ(i)] * plane + yk[1 + CY(i)] + xk[1 + CX(i)], P.phi_fix);
            phi_stencil(ph, Mp, G);
            cs = surface_coef<ML>(Mp, G, P);
            if constexpr (ML) sel = mlp_select(G, P, kfd, gn);
        }
    }
    float fs[3] = {0.f, 0.f, 0.f};
    if constexpr (TP) {
        if (valid)
#pragma unroll
            for (int a = 0; a < 3; a++) fs[a] = cs * G.g[a];
    }
    if constexpr (ML) {
        float yv[4] = {0.f, 0.f, 0.f, 0.f};
        mlp_wave(W, wv, sel, ph, yv, threadIdx.x & 63);
        if (sel) surface_blend(G, cs, P, kfd, gn, yv, fs);
    }
    if (valid) {
        float aext[3] = {0.f, 0.f, 0.f};
        if constexpr (FRC) forcing_at<false>(P, P.fx[x], (uint32_t)z * ny + y, aext);
        site_macro<TP>(M, G, fs, aext, P, m);
    }
}

template <int S, bool TP, bool FRC, bool ML>
__global__ void __launch_bounds__(NTHREADS) k_moments_site(Params P, const void *fin, const void *phi, float *rho,
                                                           float *pr, float *u, double *phi_out)
{
    __shared__ __align__(16) char mlp_raw[ML ? sizeof(MlpW) + (NTHREADS / 64) * sizeof(MlpWave) : 1];
    MlpW &W = *(MlpW *)mlp_raw;
    MlpWave *wv = (MlpWave *)(mlp_raw + (ML ? sizeof(MlpW) : 0));
    if constexpr (ML) {
        load_weights((const uint16_t *)P.mlp, W, threadIdx.x);
        __syncthreads();
    }
    const uint32_t N = (uint32_t)P.nx * P.ny * P.nz;
    const uint32_t s = blockIdx.x * NTHREADS + threadIdx.x;
    const bool valid = s < N;
    Macro m;
    site_state<S, TP, FRC, ML>(P, fin, phi, valid ? s : 0u, valid, m, W, wv[ML ? threadIdx.x >> 6 : 0]);
    if (!valid) return;
    if (rho) rho[s] = m.rho;
    if (pr) pr[s] = (P.p0 + m.dp) * m.rho * (1.0f / 3.0f);
    if (u) {
        u[s] = m.u[0];
        u[(size_t)N + s] = m.u[1];
        u[2 * (size_t)N + s] = m.u[2];
    }
    if (phi_out) phi_out[s] = TP ? phi_load(phi, s, P.phi_fix) : 0.0;
}

// The march: macroscopic state at time n of the sites of item L (pull + stencils
// from global memory): use(z, state, phi, R) for each site of the box.  In the marches
// by rows (the long ones) and without the network, the populations and the phi
// plane of the next site are in flight while this one is worked on.  Bound by
// memory: 512^3 read-out, FP16 4.03 -> 2.6 ms, FP32 4.46 -> 4.0 ms (4.8 TB/s);
// reduction, FP32 4.53 -> 3.33 ms (4.7 TB/s).
template <int S, bool FRC, bool ML, bool FX, bool ROW, class Use>
__device__ __forceinline__ void read_tile(const Params &P, const void *fin_, const void *phi_, uint32_t L, int chunk,
                                          int wx, const MlpW &W, MlpWave &wv, Use use)
{
    using T = typename Pop<S>::T;
    using PS = PhiStore<FX>;
    using PT = typename PS::T;
    constexpr uint32_t ES = sizeof(T);
    const RowMarch<ROW> R(P, L, chunk, wx);
    if (!R.in_row) return;
    const T *fin = (const T *)fin_;
    const PT *phi = (const PT *)phi_;
    const uint32_t plane = R.plane;
    T hv[27];
    auto fetch_pops = [&](int z) {
        const int zs[3] = {wrapi(z + 1, R.nz), z, wrapi(z - 1, R.nz)};
#pragma unroll
        for (int i = 0; i < 27; i++) {
            const __amdgpu_buffer_rsrc_t src =
                plane_rsrc(fin + (size_t)((uint32_t)zs[CZ(i) + 1] * plane) * 27, 27u * plane * ES);
            hv[i] = bload<T>(src, R.vcol(1 - CY(i), 1 - CX(i)) * ES, ((uint32_t)i * plane + R.srow(1 - CY(i))) * ES);
        }
    };
    auto f32 = [&](const PT(&r)[9], float (&v)[9]) {
#pragma unroll
        for (int i = 0; i < 9; i++) v[i] = PS::f32(r[i]);
    };
    float4 ex = {0.f, 0.f, 0.f, 0.f};
    if constexpr (FRC) ex = P.fx[R.xs[1]];
    P6 pa, pb;  // plane sums of phi at z-1 and z ...
    float ph[27];  // ... or, for the network's inputs, the three planes themselves
    PT c = 0, r[9];
    float v[9];
    {
        PT ra[9], rb[9];
        R.at9(phi, R.z0 - 1, ra);
        R.at9(phi, R.z0, rb);
        f32(ra, v);
        plane6(v, pa);
        if constexpr (ML)
            for (int i = 0; i < 9; i++) ph[9 + i] = v[i];
        f32(rb, v);
        plane6(v, pb);
        if constexpr (ML)
            for (int i = 0; i < 9; i++) ph[18 + i] = v[i];
        c = rb[4];
    }
    auto fetch = [&](int z) {
        fetch_pops(z);
        R.at9(phi, z + 1, r);
    };
    constexpr bool AHEAD = ROW && !ML;
    auto site = [&](int z, int zn) {
        M10 M;
        PhiGrad G;
        float cs = 0.f, kfd = 0.f, gn = 0.f;
        bool sel = false;
        PT c_next = 0;
        {
            float hf[27];
#pragma unroll
            for (int i = 0; i < 27; i++) hf[i] = Pop<S>::dec(hv[i]);
            moments10(hf, M);
        }
        {
            M10 Mp;
            f32(r, v);
            c_next = r[4];
            if constexpr (ML) {
                for (int i = 0; i < 18; i++) ph[i] = ph[9 + i];
                for (int i = 0; i < 9; i++) ph[18 + i] = v[i];
                moments10(ph, Mp);
            } else {
                P6 n;
                plane6(v, n);
                planes10(pa, pb, n, Mp);
                pa = pb;
                pb = n;
            }
            phi_grad(Mp, PS::f32(c), G);
            cs = surface_coef<ML>(Mp, G, P);
            if constexpr (ML) sel = mlp_select(G, P, kfd, gn);  // images too: they write what the owner writes
        }
        if constexpr (AHEAD) fetch(zn);
        float fs[3];
#pragma unroll
        for (int a = 0; a < 3; a++) fs[a] = cs * G.g[a];
        if constexpr (ML) {
            if (__ballot(sel)) {  // the network: a wave-wide MFMA, so every lane takes part
                float y[4] = {0.f, 0.f, 0.f, 0.f};
                mlp_wave(W, wv, sel, ph, y, threadIdx.x & 63);
                if (sel) surface_blend(G, cs, P, kfd, gn, y, fs);
            }
        }
        float aext[3] = {0.f, 0.f, 0.f};
        if constexpr (FRC) forcing_at<ROW>(P, ex, (uint32_t)z * R.ny + R.y, aext);
        Macro m;
        site_macro<true>(M, G, fs, aext, P, m);
        use(z, m, FX ? (double)c * 0x1p-30 : (double)c, R);
        c = c_next;
    };
    if constexpr (AHEAD) {
        fetch(R.z0);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): exact counts in the loop, as in the step
        for (int z = R.z0; z < R.zend; z++) site(z, z + 1 < R.zend ? z + 1 : z);
    } else {
        for (int z = R.z0; z < R.zend; z++) {
            fetch(z);
            site(z, z);
        }
    }
}

template <int S, bool FRC, bool ML, bool FX, bool ROW, bool NT>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(ML || !ROW ? 3 : 4)))
k_moments(Params P, const void *fin, const void *phi, float *rho, float *pr, float *u, double *phi_out, int chunk,
          int wx)
{
    __shared__ __align__(16) char mlp_raw[ML ? sizeof(MlpW) + (NTHREADS / 64) * sizeof(MlpWave) : 1];
    MlpW &W = *(MlpW *)mlp_raw;
    MlpWave *wv = (MlpWave *)(mlp_raw + (ML ? sizeof(MlpW) : 0));
    if constexpr (ML) {
        load_weights((const uint16_t *)P.mlp, W, threadIdx.x);
        __syncthreads();
    }
    const size_t N = (size_t)P.nx * P.ny * P.nz;
    read_tile<S, FRC, ML, FX, ROW>(P, fin, phi, blockIdx.x, chunk, wx, W, wv[ML ? threadIdx.x >> 6 : 0],
                                   [&](int z, const Macro &m, double ph, const RowMarch<ROW> &R) {
        R.template put<NT>(rho, z, m.rho);
        R.template put<NT>(pr, z, (P.p0 + m.dp) * m.rho * (1.0f / 3.0f));
#pragma unroll
        for (int a = 0; a < 3; a++) R.template put<NT>(u ? u + a * N : u, z, m.u[a]);
        R.template put<NT>(phi_out, z, ph);
    });
}

// Wavefront reductions in FP64: a butterfly over the 64 lanes (xor
// partners 32, 16, .., 1).  Each lane combines the same two operands in the same
// order as its partner, so all lanes end with the same bits, and the pattern is
// fixed, so the result does not depend on scheduling.
constexpr bool red_is_max(int k) { return k == 7 || k == 8; }
template <int K> __device__ __forceinline__ double wave_reduce(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double w = __shfl_xor(v, o, 64);
        v = red_is_max(K) ? fmax(v, w) : v + w;
    }
    return v;
}
__device__ __forceinline__ long long wave_sum_i64(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// the NRED statistics of this workgroup: one wavefront reduction per
// statistic, then lane 0 of every wave writes its value and thread k < NRED
// combines the NTHREADS / 64 wave values of statistic k in a fixed order
__device__ __forceinline__ void block_reduce(const double (&acc)[NRED], double (&wred)[NTHREADS / 64][NRED],
                                            double &res)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[NRED];
    v[0] = wave_reduce<0>(acc[0]);
    v[1] = wave_reduce<1>(acc[1]);
    v[2] = wave_reduce<2>(acc[2]);
    v[3] = wave_reduce<3>(acc[3]);
    v[4] = wave_reduce<4>(acc[4]);
    v[5] = wave_reduce<5>(acc[5]);
    v[6] = wave_reduce<6>(acc[6]);
    v[7] = wave_reduce<7>(acc[7]);
    v[8] = wave_reduce<8>(acc[8]);
    v[9] = wave_reduce<9>(acc[9]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NRED; k++) wred[wave][k] = v[k];
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < NRED) {
        res = wred[0][k];
#pragma unroll
        for (int w = 1; w < NTHREADS / 64; w++) res = red_is_max(k) ? fmax(res, wred[w][k]) : res + wred[w][k];
    }
}

// The ten statistics of one site added to a thread's; phi_sum: phi, or with the
// fixed-point phi the integer q
template <bool TP>
__device__ __forceinline__ void accumulate(const Params &P, const Macro &m, double ph, double phi_sum,
                                           double (&acc)[NRED])
{
    const double r = m.rho, pstar = (double)P.p0 + (double)m.dp;
    const double ux = m.u[0], uy = m.u[1], uz = m.u[2];
    const bool bad = !isfinite(pstar) || !isfinite(ux) || !isfinite(uy) || !isfinite(uz) || !isfinite(ph);
    if (bad) {
        acc[9] += 1.0;
        return;
    }
    const double u2 = ux * ux + uy * uy + uz * uz;
    acc[0] += phi_sum;
    acc[1] += r;
    acc[2] += pstar;
    acc[3] += r * ux;
    acc[4] += r * uy;
    acc[5] += r * uz;
    acc[6] += 0.5 * r * u2;
    acc[7] = fmax(acc[7], u2);  // the root of the largest at the end
    acc[8] = TP ? fmax(acc[8], fmax(ph - 1.0, fmax(-ph, 0.0))) : 0.0;
}
__device__ __forceinline__ void put_partials(double (&acc)[NRED], double *partials)
{
    acc[7] = sqrt(acc[7]);
    __shared__ double wred[NTHREADS / 64][NRED];
    double res = 0.0;
    block_reduce(acc, wred, res);
    if (threadIdx.x < NRED) partials[(size_t)blockIdx.x * NRED + threadIdx.x] = res;
}

// FP64 partial sums per block over a fixed partition of the sites or items,
// combined in a fixed order: the result does not depend on scheduling.  With the
// fixed-point phi, sum phi is accumulated as the integer sum of q (exact in
// the FP64 block partials, which stay below 2^53, and in the final int64 sum),
// so it is a function of that integer alone.
template <int S, bool TP, bool FRC, bool ML>
__global__ void __launch_bounds__(NTHREADS) k_reduce_site(Params P, const void *fin, const void *phi, double *partials)
{
    __shared__ __align__(16) char mlp_raw[ML ? sizeof(MlpW) + (NTHREADS / 64) * sizeof(MlpWave) : 1];
    MlpW &W = *(MlpW *)mlp_raw;
    MlpWave *wv = (MlpWave *)(mlp_raw + (ML ? sizeof(MlpW) : 0));
    if constexpr (ML) {
        load_weights((const uint16_t *)P.mlp, W, threadIdx.x);
        __syncthreads();
    }
    const uint32_t N = (uint32_t)P.nx * P.ny * P.nz;
    double acc[NRED];
#pragma unroll
    for (int k = 0; k < NRED; k++) acc[k] = 0.0;
    // uniform trip count across the block (the network stage is wave-wide)
    for (uint32_t base = blockIdx.x * NTHREADS; base < N; base += gridDim.x * NTHREADS) {
        const uint32_t s = base + threadIdx.x;
        const bool valid = s < N;
        Macro m;
        site_state<S, TP, FRC, ML>(P, fin, phi, valid ? s : 0u, valid, m, W, wv[ML ? threadIdx.x >> 6 : 0]);
        if (!valid) continue;
        const double ph = TP ? phi_load(phi, s, P.phi_fix) : 0.0;
        accumulate<TP>(P, m, ph, P.phi_fix ? ph * 0x1p30 : ph, acc);
    }
    put_partials(acc, partials);
}

template <int S, bool FRC, bool ML, bool FX, bool ROW>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3)))
k_reduce(Params P, const void *fin, const void *phi, double *partials, uint32_t items, int chunk, int wx)
{
    __shared__ __align__(16) char mlp_raw[ML ? sizeof(MlpW) + (NTHREADS / 64) * sizeof(MlpWave) : 1];
    MlpW &W = *(MlpW *)mlp_raw;
    MlpWave *wv = (MlpWave *)(mlp_raw + (ML ? sizeof(MlpW) : 0));
    if constexpr (ML) {
        load_weights((const uint16_t *)P.mlp, W, threadIdx.x);
        __syncthreads();
    }
    double acc[NRED];
#pragma unroll
    for (int k = 0; k < NRED; k++) acc[k] = 0.0;
    for (uint32_t L = blockIdx.x; L < items; L += gridDim.x)
        read_tile<S, FRC, ML, FX, ROW>(P, fin, phi, L, chunk, wx, W, wv[ML ? threadIdx.x >> 6 : 0],
                                       [&](int, const Macro &m, double ph, const RowMarch<ROW> &R) {
            if (R.in_box) accumulate<true>(P, m, ph, FX ? ph * 0x1p30 : ph, acc);
        });
    put_partials(acc, partials);
}

// one wave per statistic over the RED_BLOCKS partials
__global__ void __launch_bounds__(64 * NRED) k_reduce_final(const double *partials, int fix, double *out)
{
    const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
    double v[RED_BLOCKS / 64];
#pragma unroll
    for (int j = 0; j < RED_BLOCKS / 64; j++) v[j] = partials[(size_t)(64 * j + lane) * NRED + k];
    if (fix && k == 0) {  // fixed-point phi: integer sum of q
        long long q = 0;
#pragma unroll
        for (int j = 0; j < RED_BLOCKS / 64; j++) q += (long long)v[j];
        q = wave_sum_i64(q);
        if (lane == 0) out[0] = (double)q * 0x1p-30;
        return;
    }
    double s = 0.0, m = 0.0;  // the maxima are of values >= 0
#pragma unroll
    for (int j = 0; j < RED_BLOCKS / 64; j++) {
        s += v[j];
        m = fmax(m, v[j]);
    }
    s = red_is_max(k) ? wave_reduce<7>(m) : wave_reduce<0>(s);
    if (lane == 0) out[k] = s;
}

// --------------------------------------------------------------- launchers
int batch_grid(int storage, bool tp, bool frc, bool ml, bool fix, bool phys, int tile, bool nt)
{
    if (storage == 0) return step_grid<0>(tp, frc, ml, fix, phys, tile, nt);
    if (storage == 1) return step_grid<1>(tp, frc, ml, fix, phys, tile, nt);
    return step_grid<2>(tp, frc, ml, fix, phys, tile, nt);
}

hipError_t launch_step_batch(const Params *tab, const Buffers *buf, const uint32_t *first, int nbox,
                             uint32_t *counter, int parity, int storage, bool tp, bool frc, bool ml, bool fix,
                             bool phys, int tile, bool nt, int grid, hipStream_t s)
{
    if (storage == 0)
        return step_launch<0>(tab, buf, first, nbox, counter, parity, tp, frc, ml, fix, phys, tile, nt, grid, s);
    if (storage == 1)
        return step_launch<1>(tab, buf, first, nbox, counter, parity, tp, frc, ml, fix, phys, tile, nt, grid, s);
    return step_launch<2>(tab, buf, first, nbox, counter, parity, tp, frc, ml, fix, phys, tile, nt, grid, s);
}

int mlp_pass_grid(bool fix, int tile)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (tile == 32) {
        if (fix) (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_pass_batch<32, true>, NTHREADS, 0);
        else (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_pass_batch<32, false>, NTHREADS, 0);
    } else {
        if (fix) (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_pass_batch<64, true>, NTHREADS, 0);
        else (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_pass_batch<64, false>, NTHREADS, 0);
    }
    return per_cu * cus;
}

hipError_t launch_mlp_pass_batch(const Params *tab, const Buffers *buf, const uint32_t *first, int nbox,
                                 uint32_t *counter, int parity, bool fix, int tile, int grid, hipStream_t s)
{
    dim3 g(grid), block(tile, NTHREADS / tile, 1);
#define PASS(TW_, X_) hipLaunchKernelGGL((k_mlp_pass_batch<TW_, X_>), g, block, 0, s, tab, buf, first, nbox, counter, parity)
    if (tile == 32) {
        if (fix) PASS(32, true);
        else PASS(32, false);
    } else {
        if (fix) PASS(64, true);
        else PASS(64, false);
    }
#undef PASS
    return hipGetLastError();
}

int ac_stage_grid(int tile)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (tile == 32)
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_ac_stage_batch<32>, NTHREADS, 0);
    else
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_ac_stage_batch<64>, NTHREADS, 0);
    return per_cu * cus;
}

hipError_t launch_ac_stage_batch(const Params *tab, const Buffers *buf, const uint32_t *first, int nbox,
                                 uint32_t *counter, int parity, double rk_a, double rk_b, int tile, int grid,
                                 hipStream_t s)
{
    dim3 g(grid), block(tile, NTHREADS / tile, 1);
    if (tile == 32)
        hipLaunchKernelGGL(k_ac_stage_batch<32>, g, block, 0, s, tab, buf, first, nbox, counter, parity, rk_a, rk_b);
    else
        hipLaunchKernelGGL(k_ac_stage_batch<64>, g, block, 0, s, tab, buf, first, nbox, counter, parity, rk_a, rk_b);
    return hipGetLastError();
}

hipError_t launch_init(const Params &p, int storage, void *fout, void *phi_out, float *u_out, const double *phi0,
                       const double *u0, const double *ps0, hipStream_t s)
{
    const dim3 block(NTHREADS);
    const Plan plan = plan_init(p);
    if (plan.sites) {
        const dim3 grid(site_blocks(p));
#define INIT(S_) hipLaunchKernelGGL(k_init_site<S_>, grid, block, 0, s, p, fout, phi_out, u_out, phi0, u0, ps0)
        if (storage == 0) INIT(0);
        else if (storage == 1) INIT(1);
        else INIT(2);
#undef INIT
        return hipGetLastError();
    }
    const int wx = plan.wx, c = plan.chunk;
    const dim3 grid(march_items(p, c, wx));
#define INIT_AS(S_, R_, NT_) \
    hipLaunchKernelGGL((k_init<S_, R_, NT_>), grid, block, 0, s, p, fout, phi_out, u_out, phi0, u0, ps0, c, wx)
#define INIT(S_)                                 \
    {                                            \
        if (wx) INIT_AS(S_, true, true);         \
        else if (plan.nt) INIT_AS(S_, false, true); \
        else INIT_AS(S_, false, false);          \
    }
    if (storage == 0) INIT(0)
    else if (storage == 1) INIT(1)
    else INIT(2)
#undef INIT
#undef INIT_AS
    return hipGetLastError();
}

// the marches of the read-out also take the phi storage and the kind of march
#define LBM_MARCH_CALL(S_, TP_, F_, M_)                 \
    {                                                   \
        if constexpr (TP_) {                            \
            if (p.phi_fix) {                            \
                if (wx) MARCH(S_, F_, M_, true, true);  \
                else MARCH(S_, F_, M_, true, false);    \
            } else {                                    \
                if (wx) MARCH(S_, F_, M_, false, true); \
                else MARCH(S_, F_, M_, false, false);   \
            }                                           \
        }                                               \
    }

// ------------------------------------------------------------ body force
// Row and column tables of the body force.  Per mode B = A e^{i (ky ty + kz tz)}
// is folded into the row coefficients of cos(|kx| t) (Re B) and sin(|kx| t)
// (-sign(kx) Im B), t = 2 pi x / nx, modes in table order; one thread per row,
// FP64, contraction-free: the bits of the same loop on the host, which took
// 5.6 ms for the 65,536 rows and 32 modes of a 256^3 box (its whole set-up:
// 7.3 -> 1.7 ms).
struct Cplx {
    double c, s;
};
__device__ __forceinline__ Cplx circle(const double *e, int k, int v, int n)
{
    const uint32_t kn = (uint32_t)(k % n + n) % (uint32_t)n;  // exact phase index k v mod n
    const uint32_t f = n <= 65536 ? kn * (uint32_t)v % (uint32_t)n
                                  : (uint32_t)((uint64_t)kn * (uint32_t)v % (uint32_t)n);
    return {e[2 * f], e[2 * f + 1]};
}
__global__ void __launch_bounds__(256) k_forcing(const double *__restrict__ in, int nm, int nx, int ny, int nz,
                                                 float *__restrict__ frow, float4 *__restrict__ fx)
{
#pragma clang fp contract(off)
    const double *ex = in + 9 * (size_t)nm, *ey = ex + 2 * (size_t)nx, *ez = ey + 2 * (size_t)ny;
    const uint32_t r = blockIdx.x * 256 + threadIdx.x, rows = (uint32_t)ny * (uint32_t)nz;
    if (r < (uint32_t)nx) {
        const Cplx a = circle(ex, 1, (int)r, nx), b = circle(ex, 2, (int)r, nx);
        fx[r] = make_float4((float)a.c, (float)a.s, (float)b.c, (float)b.s);
    }
    if (r >= rows) return;
    const int y = (int)(r % (uint32_t)ny), z = (int)(r / (uint32_t)ny);
    double p[3][3] = {}, q[3][3] = {};  // of cos and sin, by |kx| and component (q[0] unused)
    for (int m = 0; m < nm; m++) {
        const double *t = in + 9 * m;
        const int kx = (int)t[0], kk = kx < 0 ? -kx : kx;
        const Cplx cy = circle(ey, (int)t[1], y, ny), cz = circle(ez, (int)t[2], z, nz);
        const double pc = cy.c * cz.c - cy.s * cz.s, ps = cy.c * cz.s + cy.s * cz.c;
        const double sg = kx < 0 ? -1.0 : 1.0;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const double ar = t[3 + 2 * a], ai = t[4 + 2 * a];
            const double br = ar * pc - ai * ps, bi = ar * ps + ai * pc;
#pragma unroll
            for (int k = 0; k < 3; k++)
                if (k == kk) {
                    p[k][a] += br;
                    q[k][a] -= sg * bi;
                }
        }
    }
    float v[FROW];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        v[a] = (float)p[0][a];
        v[3 + a] = (float)p[1][a];
        v[6 + a] = (float)q[1][a];
        v[9 + a] = (float)p[2][a];
        v[12 + a] = (float)q[2][a];
    }
    v[15] = 0.f;
    float4 *out = (float4 *)(frow + (size_t)r * FROW);
#pragma unroll
    for (int i = 0; i < 4; i++) out[i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
}
hipError_t launch_forcing(const double *in, int nm, int nx, int ny, int nz, float *frow, float4 *fx, hipStream_t s)
{
    const size_t n = std::max((size_t)ny * nz, (size_t)nx);
    hipLaunchKernelGGL(k_forcing, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, in, nm, nx, ny, nz, frow, fx);
    return hipGetLastError();
}

hipError_t launch_moments(const Params &p, int storage, const void *fin, const void *phi, float *rho, float *pr,
                          float *u, double *phi_out, hipStream_t s)
{
    const bool tp = p.two_phase != 0, frc = p.n_modes > 0, ml = p.curv_mode == 1;
    const dim3 block(NTHREADS);
    const Plan plan = plan_read(p, storage, true);
    if (plan.sites) {
        const dim3 grid(site_blocks(p));
#define SITE(S_, TP_, F_, M_) \
    hipLaunchKernelGGL((k_moments_site<S_, TP_, F_, M_>), grid, block, 0, s, p, fin, phi, rho, pr, u, phi_out);
        LBM_DISPATCH(storage, tp, frc, ml, SITE);
#undef SITE
        return hipGetLastError();
    }
    const int wx = plan.wx, c = plan.chunk;
    const dim3 grid(march_items(p, c, wx));
#define MARCH_AS(S_, F_, M_, X_, R_, NT_)                                                                           \
    hipLaunchKernelGGL((k_moments<S_, F_, M_, X_, R_, NT_>), grid, block, 0, s, p, fin, phi, rho, pr, u, phi_out, c, \
                       wx)
#define MARCH(S_, F_, M_, X_, R_)                                \
    do {                                                         \
        if (R_ || plan.nt) MARCH_AS(S_, F_, M_, X_, R_, true);   \
        else MARCH_AS(S_, F_, M_, X_, R_, R_);                   \
    } while (0)
    LBM_DISPATCH(storage, tp, frc, ml, LBM_MARCH_CALL);
#undef MARCH
#undef MARCH_AS
    return hipGetLastError();
}

hipError_t launch_reduce(const Params &p, int storage, const void *fin, const void *phi, double *partials,
                         double *out, hipStream_t s)
{
    const bool tp = p.two_phase != 0, frc = p.n_modes > 0, ml = p.curv_mode == 1;
    const Plan plan = plan_read(p, storage, false);
    const dim3 block(NTHREADS), grid(RED_BLOCKS);
    if (plan.sites) {
#define SITE(S_, TP_, F_, M_) \
    hipLaunchKernelGGL((k_reduce_site<S_, TP_, F_, M_>), grid, block, 0, s, p, fin, phi, partials);
        LBM_DISPATCH(storage, tp, frc, ml, SITE);
#undef SITE
    } else {
        const int wx = plan.wx, c = plan.chunk;
        const uint32_t items = march_items(p, c, wx);
#define MARCH(S_, F_, M_, X_, R_) \
    hipLaunchKernelGGL((k_reduce<S_, F_, M_, X_, R_>), grid, block, 0, s, p, fin, phi, partials, items, c, wx)
        LBM_DISPATCH(storage, tp, frc, ml, LBM_MARCH_CALL);
#undef MARCH
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(64 * NRED), 0, s, partials, p.phi_fix, out);
    return hipGetLastError();
}

}  // namespace lbm
