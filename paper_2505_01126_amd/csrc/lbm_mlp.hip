// Learned curvature network on gfx950 FP16 MFMA: forward, backward (MSE),
// Adam, and the harvest of training samples from a phase field.
//
// Network 27 -> 64 -> 64 -> 4 with tanh hidden layers; fp16 weights and
// activations, FP32 accumulation (v_mfma_f32_16x16x32_f16).  One wave handles
// a tile of 16 samples.  Operand layouts of the 16x16x32 MFMA (lane l):
//   A: row l % 16, k = 8 (l / 16) + j, j = 0..7
//   B: column l % 16, k = 8 (l / 16) + j
//   C: column l % 16, rows 4 (l / 16) + i, i = 0..3
#include <hip/hip_runtime.h>

#include <mutex>

#include "lbm.h"
#include "lbm_internal.h"
#include "lbm_mlp_device.h"

namespace lbm {

constexpr int CHUNK = 64;  // samples per workgroup pass of the backward (4 waves x 16)

__device__ __forceinline__ half8 load_x(const uint16_t *__restrict__ x, int64_t row, int64_t B, int kq)
{
    half8 v;
    if (row < B) {
        const uint4 raw = *(const uint4 *)(x + row * KIN + 8 * kq);
        v = __builtin_bit_cast(half8, raw);
    } else {
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = (_Float16)0.0f;
    }
    return v;
}

__global__ void __launch_bounds__(256) k_mlp_forward(const uint16_t *__restrict__ w, const uint16_t *__restrict__ x,
                                                     int64_t B, float *__restrict__ y)
{
    __shared__ MlpW L;
    __shared__ __align__(16) _Float16 hbuf[4][16][HP];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t ntiles = (B + 15) / 16, t0 = (int64_t)blockIdx.x * 4 + wave;
    half8 xa = load_x(x, t0 * 16 + (lane & 15), B, lane >> 4);  // in flight while the weights are staged
    load_weights(w, L, tid);
    __syncthreads();
    for (int64_t t = t0; t < ntiles; t += (int64_t)gridDim.x * 4) {
        const int64_t s0 = t * 16;
        const half8 xn = load_x(x, (t + (int64_t)gridDim.x * 4) * 16 + (lane & 15), B, lane >> 4);
        const f32x4 o = forward_tile(L, xa, hbuf[wave], hbuf[wave], lane);
        xa = xn;
        const int col = lane & 15, kq = lane >> 4;
        if (col < NOUT)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int64_t s = s0 + 4 * kq + i;
                if (s < B) y[s * NOUT + col] = o[i];
            }
    }
}

// ------------------------------------------------------------- backward
// Per workgroup: a fixed set of 64-sample chunks (chunk c -> block c % grid);
// forward with saved activations, then
//   d3 = 2 (y - t)               (the 1/B is applied at the end)
//   d2 = (d3 W3) * (1 - h2^2),   d1 = (d2 W2) * (1 - h1^2)
//   gW3 = d3^T h2, gW2 = d2^T h1, gW1 = d1^T x, gb = column sums,
// accumulated over the block's chunks; block partials are summed in a fixed
// order by k_mlp_reduce.
//
// A batch of 16384 is one chunk for each of 256 workgroups, so what counts is
// the length of the chain through one chunk, not any rate.  The C layout of an
// MFMA holds four consecutive samples of one neuron per lane: h1, h2, d2 and
// d1 go from there to LDS both by sample (the next layer's A operand) and, 8
// bytes at a time, by neuron, which is what both operands of the weight
// gradients read 16 bytes at a time (gathered from the layout by sample, sample
// by sample, they took 128 reads of 2 bytes per lane).  gW3 = d3^T h2 keeps d3 in
// FP32 on the FP32 MFMA; the bias gradients are one more column of ones in the
// products.  The weights are read 16 bytes at a time.  16384 samples: 23.1 ->
// 14.6 us.
struct BLds {
    WLds W;
    _Float16 h[4][16][HP];  // each wave's activations, then its d2, by sample
    _Float16 xt[KIN][HP];   // by input or neuron, then by sample of the chunk
    _Float16 h1t[NH][HP], h2t[NH][HP], d2t[NH][HP], d1t[NH][HP];
    float d3[CHUNK][NOUT];
    float d3t[NOUT][CHUNK + 4];
};
static_assert(HP >= CHUNK && HP % 8 == 0, "a row by neuron holds the samples of a chunk");

typedef _Float16 half4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) k_mlp_backward(const uint16_t *__restrict__ w, const uint16_t *__restrict__ x,
                                                      const float *__restrict__ tgt, int64_t B,
                                                      float *__restrict__ partial)
{
    extern __shared__ __align__(16) char lds_raw[];
    BLds &S = *(BLds *)lds_raw;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, kq = lane >> 4;
    const int64_t nchunks = (B + CHUNK - 1) / CHUNK;
    // inputs and targets of a chunk's 16 samples of this wave, fetched one chunk ahead
    auto fetch = [&](int64_t c, half8 &xa, float (&t)[4]) {
        const int64_t s0 = c * CHUNK + 16 * wave;
        xa = load_x(x, s0 + r, B, kq);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t s = s0 + 4 * kq + i;
            t[i] = r < NOUT && s < B ? tgt[s * NOUT + r] : 0.0f;
        }
    };
    half8 xa;
    float t[4];
    fetch(blockIdx.x, xa, t);
    load_weights(w, S.W, tid);
    // accumulators: wave owns neuron tile n = 16 wave .. +15 of gW2 (4 column
    // tiles and one of ones, its bias), of gW1 (2 column tiles, input 27 the
    // ones of its bias) and the columns 16 wave .. +15 of gW3
    f32x4 acc2[5], acc1[2], acc3 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 5; k++) acc2[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 2; k++) acc1[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    half8 ones;
#pragma unroll
    for (int j = 0; j < 8; j++) ones[j] = (_Float16)(r == 0 ? 1.0f : 0.0f);
    float gb3 = 0.f, loss = 0.f;
    __syncthreads();
    float w3[4][NOUT];  // of this lane's neurons 16 nt + r
#pragma unroll
    for (int nt = 0; nt < 4; nt++)
#pragma unroll
        for (int o = 0; o < NOUT; o++) w3[nt][o] = (float)S.W.w3[o][16 * nt + r];
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const int64_t s0 = c * CHUNK + 16 * wave;
        const int sw = 16 * wave + 4 * kq;  // this lane's four samples of the chunk
        _Float16(*h)[HP] = S.h[wave];
#pragma unroll
        for (int j = 0; j < 8; j++) S.xt[8 * kq + j][16 * wave + r] = 8 * kq + j == NIN ? (_Float16)1.0f : xa[j];
        _Float16 h1[16], h2[16];
        const f32x4 y = forward_tile(S.W, xa, h, h, lane, h1, h2);
        if (r < NOUT) {
            f32x4 d;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float e = s0 + 4 * kq + i < B ? y[i] - t[i] : 0.0f;
                loss += e * e;
                d[i] = 2.0f * e;
                S.d3[sw + i][r] = d[i];
            }
            *(f32x4 *)&S.d3t[r][sw] = d;
        }
        fetch(c + gridDim.x, xa, t);
        wave_lds_sync();
        // d2 in the C layout of h2
        {
            f32x4 d3[4];
#pragma unroll
            for (int i = 0; i < 4; i++) d3[i] = *(const f32x4 *)&S.d3[sw + i][0];
#pragma unroll
            for (int nt = 0; nt < 4; nt++) {
                half4 v2, a1, a2;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    float v = 0.f;
#pragma unroll
                    for (int o = 0; o < NOUT; o++) v += d3[i][o] * w3[nt][o];
                    const float hv = (float)h2[4 * nt + i];
                    v2[i] = (_Float16)(v * (1.0f - hv * hv));
                    a1[i] = h1[4 * nt + i];
                    a2[i] = h2[4 * nt + i];
                    h[4 * kq + i][16 * nt + r] = v2[i];
                }
                *(half4 *)&S.h1t[16 * nt + r][sw] = a1;
                *(half4 *)&S.h2t[16 * nt + r][sw] = a2;
                *(half4 *)&S.d2t[16 * nt + r][sw] = v2;
            }
        }
        wave_lds_sync();
        // d1 = (d2 W2) (1 - h1^2)
        {
            const half8 a0 = ld8(&h[r][8 * kq]), a1 = ld8(&h[r][32 + 8 * kq]);
#pragma unroll
            for (int nt = 0; nt < 4; nt++) {
                f32x4 cc = {0.f, 0.f, 0.f, 0.f};
                cc = mfma(a0, ld8(&S.W.w2t[16 * nt + r][8 * kq]), cc);
                cc = mfma(a1, ld8(&S.W.w2t[16 * nt + r][32 + 8 * kq]), cc);
                half4 v1;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float hv = (float)h1[4 * nt + i];
                    v1[i] = (_Float16)(cc[i] * (1.0f - hv * hv));
                }
                *(half4 *)&S.d1t[16 * nt + r][sw] = v1;
            }
        }
        __syncthreads();
        // weight gradients over the 64 samples of the chunk (K = 2 x 32)
        {
            const int n = 16 * wave + r;  // A row (neuron) of this lane
#pragma unroll
            for (int ks = 0; ks < 2; ks++) {
                const int sb = 32 * ks + 8 * kq;
                const half8 a2 = ld8(&S.d2t[n][sb]), a1 = ld8(&S.d1t[n][sb]);
#pragma unroll
                for (int nt = 0; nt < 4; nt++) acc2[nt] = mfma(a2, ld8(&S.h1t[16 * nt + r][sb]), acc2[nt]);
                acc2[4] = mfma(a2, ones, acc2[4]);
#pragma unroll
                for (int nt = 0; nt < 2; nt++) acc1[nt] = mfma(a1, ld8(&S.xt[16 * nt + r][sb]), acc1[nt]);
            }
            // FP32 MFMA 16x16x4 (A: row l % 16, k = l / 16; B: column l % 16,
            // k = l / 16; C as above): step j takes sample 16 (l / 16) + j, so
            // that a lane reads its operands of all steps contiguously
            f32x4 a[4];
#pragma unroll
            for (int q = 0; q < 4; q++)
                a[q] = r < NOUT ? *(const f32x4 *)&S.d3t[r][16 * kq + 4 * q] : f32x4{0.f, 0.f, 0.f, 0.f};
            const half8 b0 = ld8(&S.h2t[n][16 * kq]), b1 = ld8(&S.h2t[n][16 * kq + 8]);
#pragma unroll
            for (int j = 0; j < 16; j++) {
                const float av = a[j / 4][j % 4];
                acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(av, (float)(j < 8 ? b0[j % 8] : b1[j % 8]), acc3, 0, 0, 0);
                gb3 += av;
            }
        }
        __syncthreads();
    }
    // block partial: [NPARAM + 1] floats (gradient, then the loss)
    float *P = partial + (size_t)blockIdx.x * (NPARAM + 1);
    {
        const int n0 = 16 * wave + 4 * kq;
#pragma unroll
        for (int nt = 0; nt < 4; nt++)
#pragma unroll
            for (int i = 0; i < 4; i++) P[OW2 + (n0 + i) * NH + 16 * nt + r] = acc2[nt][i];
#pragma unroll
        for (int nt = 0; nt < 2; nt++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int k = 16 * nt + r;
                if (k < NIN) P[OW1 + (n0 + i) * NIN + k] = acc1[nt][i];
                else if (k == NIN) P[OB1 + n0 + i] = acc1[nt][i];
            }
        if (r == 0)
#pragma unroll
            for (int i = 0; i < 4; i++) P[OB2 + n0 + i] = acc2[4][i];
        if (kq == 0)
#pragma unroll
            for (int i = 0; i < 4; i++) P[OW3 + i * NH + 16 * wave + r] = acc3[i];
        gb3 += __shfl_xor(gb3, 16, 64);
        gb3 += __shfl_xor(gb3, 32, 64);
        if (wave == 0 && lane < NOUT) P[OB3 + lane] = gb3;
    }
    // loss: fixed-order sum over the lanes that hold outputs
    __shared__ float lsum[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
    if (lane == 0) lsum[wave] = loss;
    __syncthreads();
    if (tid == 0) P[NPARAM] = (lsum[0] + lsum[1]) + (lsum[2] + lsum[3]);
}

// Sums of the block partials: 32 values per workgroup, 16 threads to a value,
// each every 16th partial, then a tree in a fixed order.  Bound by the latency
// of its loads (6.4 MB for 256 partials): one thread per value, adding them one
// after the other, took 58.7 us, this 4.3 us.
constexpr int RED_VALS = 32, RED_THREADS = 16;
__global__ void __launch_bounds__(RED_VALS *RED_THREADS)
    k_mlp_reduce(const float *__restrict__ partial, int nblocks, float inv_b, float *__restrict__ grad,
                 float *__restrict__ loss)
{
    __shared__ float sum[RED_THREADS][RED_VALS];
    const int v = threadIdx.x % RED_VALS, g = threadIdx.x / RED_VALS, p = blockIdx.x * RED_VALS + v;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (p <= NPARAM) {
        int b = g;
        for (; b + 3 * RED_THREADS < nblocks; b += 4 * RED_THREADS)
#pragma unroll
            for (int k = 0; k < 4; k++) s[k] += partial[(size_t)(b + k * RED_THREADS) * (NPARAM + 1) + p];
        for (int k = 0; b < nblocks; b += RED_THREADS, k++) s[k] += partial[(size_t)b * (NPARAM + 1) + p];
    }
    sum[g][v] = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int h = RED_THREADS / 2; h > 0; h /= 2) {
        __syncthreads();
        if (g < h) sum[g][v] += sum[g + h][v];
    }
    if (g != 0 || p > NPARAM) return;
    if (p < NPARAM) grad[p] = sum[0][v] * inv_b;
    else loss[0] = sum[0][v] * inv_b;
}

// ----------------------------------------------------------------- Adam
__global__ void __launch_bounds__(256) k_mlp_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                                  const float *__restrict__ g, uint16_t *__restrict__ w16, float lr,
                                                  float b1, float b2, float eps, float c1, float c2)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= NPARAM) return;
    const float gi = g[p];
    const float mi = b1 * m[p] + (1.0f - b1) * gi;
    const float vi = b2 * v[p] + (1.0f - b2) * gi * gi;
    m[p] = mi;
    v[p] = vi;
    const float wi = w[p] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    w[p] = wi;
    w16[p] = __builtin_bit_cast(uint16_t, (_Float16)wi);
}

// -------------------------------------------------------------- harvest
// Interface cells (0.02 < phi < 0.98) in site order: pass 1 counts them per
// workgroup range, pass 2 sums the counts of the ranges before its own (at most
// 1024 of them, 4 per thread) and writes its rows there.  The counts stay on
// the device and the spheres of an ordinary box come as kernel arguments, so
// the call waits for the stream once.  Interface cells are few and scattered,
// so pass 2 first lists the cells of a block of sites in LDS and then spreads
// the list over the threads: one thread per column of a row (a row is one
// 64-byte store, and the loads of 64 rows are in flight at once) and one thread
// per label.  Bound by those chains of loads: 4096 rows of a 48^3 box of four
// spheres took 12.9 us with one thread per row, 7.4 us here, and the call, with
// one wait and no upload, 79 -> 56 us.
__device__ __forceinline__ bool is_interface(double p) { return p > 0.02 && p < 0.98; }

__global__ void __launch_bounds__(256) k_harvest_count(const void *__restrict__ phi, int fix, uint32_t N,
                                                       uint32_t chunk, long long *__restrict__ counts)
{
    __shared__ int wsum[4];
    const uint32_t b0 = blockIdx.x * chunk, b1 = min(b0 + chunk, N);
    int cnt = 0;
    for (uint32_t s = b0 + threadIdx.x; s < b1; s += 256) cnt += is_interface(phi_load(phi, s, fix)) ? 1 : 0;
    // wave sums then fixed-order block sum
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_down(cnt, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = (long long)wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// counts: one per workgroup; *total gets their sum
template <int FIX>
__global__ void __launch_bounds__(256) k_harvest_write(Params P, const void *__restrict__ phi, uint32_t chunk,
                                                       const long long *__restrict__ counts,
                                                       long long *__restrict__ total, SphereArgs few,
                                                       const Sphere *__restrict__ many, int nb,
                                                       uint16_t *__restrict__ X, float *__restrict__ Y, int64_t cap)
{
    constexpr int SITES = 1024, PER = SITES / 256, FLY = 8;
    __shared__ int wcnt[PER][4];
    __shared__ long long wsum[4];
    __shared__ uint32_t ls[SITES];
    __shared__ int ly[SITES], lz[SITES];
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    const uint32_t plane = (uint32_t)nx * ny, N = plane * (uint32_t)nz;
    const uint32_t b0 = blockIdx.x * chunk, b1 = min(b0 + chunk, N);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = tid & 31, cell = min(col, 26);
    const int dx = cell % 3 - 1, dy = (cell / 3) % 3 - 1, dz = cell / 9 - 1;
    long long base = 0;
    for (uint32_t b = tid; b < blockIdx.x; b += 256) base += counts[b];
    for (int off = 32; off > 0; off >>= 1) base += __shfl_down(base, off, 64);
    if (lane == 0) wsum[wave] = base;
    __syncthreads();
    base = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (blockIdx.x == gridDim.x - 1 && tid == 0) *total = base + counts[blockIdx.x];
    // (base is the same in every thread; without the second condition a call that
    // only counts, cap = 0, read the phase field twice: 256^3 84 us, now 54)
    for (uint32_t s0 = b0; s0 < b1 && base < cap; s0 += SITES) {
        unsigned long long ballot[PER];
#pragma unroll
        for (int j = 0; j < PER; j++) {
            const uint32_t s = s0 + 256 * j + tid;
            ballot[j] = __ballot(s < b1 && is_interface(phi_load(phi, s, FIX)));
            if (lane == 0) wcnt[j][wave] = __popcll(ballot[j]);
        }
        __syncthreads();
        int n = 0;  // cells listed so far, in site order
#pragma unroll
        for (int j = 0; j < PER; j++) {
            int i = n;
#pragma unroll
            for (int w = 0; w < 4; w++) {
                i += w < wave ? wcnt[j][w] : 0;
                n += wcnt[j][w];
            }
            if (ballot[j] >> lane & 1)
                ls[i + __popcll(ballot[j] & ((1ull << lane) - 1ull))] = s0 + 256 * j + tid;
        }
        __syncthreads();
        const int rows = (int)min((long long)n, (long long)cap - base);
        for (int i = tid; i < rows; i += 256) {
            const uint32_t s = ls[i], row = s / (uint32_t)nx;
            ls[i] = s - row * nx;
            ly[i] = (int)(row % (uint32_t)ny);
            lz[i] = (int)(row / (uint32_t)ny);
        }
        __syncthreads();
        for (int i0 = tid >> 5; i0 < rows; i0 += 8 * FLY) {
            double p[FLY];
#pragma unroll
            for (int f = 0; f < FLY; f++) {  // FLY loads in flight; past the end the last row again
                const int i = min(i0 + 8 * f, rows - 1);
                int x = (int)ls[i] + dx, y = ly[i] + dy, z = lz[i] + dz;
                x += x < 0 ? nx : x >= nx ? -nx : 0;
                y += y < 0 ? ny : y >= ny ? -ny : 0;
                z += z < 0 ? nz : z >= nz ? -nz : 0;
                p[f] = phi_load(phi, (uint32_t)z * plane + (uint32_t)y * nx + x, FIX);
            }
#pragma unroll
            for (int f = 0; f < FLY; f++)
                if (i0 + 8 * f < rows)
                    X[(base + i0 + 8 * f) * KIN + col] =
                        col < 27 ? __builtin_bit_cast(uint16_t, (_Float16)(2.0 * p[f] - 1.0)) : 0;  // one rounding
        }
        for (int i = tid; i < rows; i += 256) {
            // nearest sphere surface (periodic minimum image)
            const int x = (int)ls[i], y = ly[i], z = lz[i];
            int best = -1;
            double bestd = 1e300, bd[3] = {0, 0, 0}, br = 0, bR = 0;
#pragma unroll 1
            for (int k = 0; k < nb; k++) {
                const Sphere c = many ? many[k] : few.s[k];
                double d[3] = {x - c.x, y - c.y, z - c.z};
                const double L[3] = {(double)nx, (double)ny, (double)nz};
                for (int a = 0; a < 3; a++) d[a] -= L[a] * rint(d[a] / L[a]);
                const double rr = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
                const double gap = fabs(rr - fabs(c.r));
                if (gap < bestd) {
                    bestd = gap;
                    best = k;
                    br = rr;
                    bR = c.r;
                    bd[0] = d[0];
                    bd[1] = d[1];
                    bd[2] = d[2];
                }
            }
            float4 yr = make_float4(0.f, 0.f, 0.f, 0.f);
            if (best >= 0 && br > 1e-12) {
                const double sg = bR > 0 ? -1.0 : 1.0;  // toward phi = 1
                yr.x = (float)(bR > 0 ? -2.0 / bR : 2.0 / (-bR));
                yr.y = (float)(sg * bd[0] / br);
                yr.z = (float)(sg * bd[1] / br);
                yr.w = (float)(sg * bd[2] / br);
            }
            float *y4 = Y + (base + i) * 4;  // any alignment of a float
            y4[0] = yr.x;
            y4[1] = yr.y;
            y4[2] = yr.z;
            y4[3] = yr.w;
        }
        base += n;
        __syncthreads();
    }
}

// --------------------------------------------------------------- launchers
int mlp_backward_blocks(int64_t B)
{
    const int64_t nchunks = (B + CHUNK - 1) / CHUNK;
    return (int)(nchunks < 512 ? (nchunks > 0 ? nchunks : 1) : 512);
}

hipError_t launch_mlp_forward(const uint16_t *w, const uint16_t *x, int64_t B, float *y, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    const int64_t ntiles = (B + 15) / 16;
    const int grid = (int)((ntiles + 3) / 4 < 4096 ? (ntiles + 3) / 4 : 4096);
    hipLaunchKernelGGL(k_mlp_forward, dim3(grid), dim3(256), 0, s, w, x, B, y);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(const uint16_t *w, const uint16_t *x, const float *t, int64_t B, float *grad,
                               float *loss, float *partial, hipStream_t s)
{
    const int blocks = mlp_backward_blocks(B);
    const size_t lds = sizeof(BLds);
    hipError_t e = hipFuncSetAttribute((const void *)k_mlp_backward, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_backward, dim3(blocks), dim3(256), lds, s, w, x, t, B, partial);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const float inv_b = B > 0 ? 1.0f / (float)B : 0.0f;
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NPARAM + RED_VALS) / RED_VALS), dim3(RED_VALS * RED_THREADS), 0, s,
                       partial, blocks, inv_b, grad, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *w, float *m, float *v, const float *g, uint16_t *w16, float lr, float b1, float b2,
                           float eps, float c1, float c2, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, s, w, m, v, g, w16, lr, b1, b2, eps, c1,
                       c2);
    return hipGetLastError();
}

hipError_t launch_harvest_count(const void *phi, int fix, uint32_t N, uint32_t chunk, int blocks, long long *counts,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_harvest_count, dim3(blocks), dim3(256), 0, s, phi, fix, N, chunk, counts);
    return hipGetLastError();
}

hipError_t launch_harvest_write(const Params &p, const void *phi, uint32_t chunk, int blocks,
                                const long long *counts, long long *total, const SphereArgs &few, const Sphere *many,
                                int nb, uint16_t *X, float *Y, int64_t cap, hipStream_t s)
{
    hipLaunchKernelGGL(p.phi_fix ? k_harvest_write<1> : k_harvest_write<0>, dim3(blocks), dim3(256), 0, s, p, phi, chunk, counts, total, few, many, nb, X,
                       Y, cap);
    return hipGetLastError();
}

// ------------------------------------------- backward without a workspace
// The block partials of lbm_mlp_backward_static live in a file-scope device
// array sized for LBM_MLP_STATIC_MAX_BATCH samples, one instance per GPU for
// the life of the process.  On the host the array's name is only a stand-in
// for the symbol: kernels get the device address that hipGetSymbolAddress
// returns, looked up once per device (the first call on that device).
constexpr int STATIC_BLOCKS = (LBM_MLP_STATIC_MAX_BATCH + CHUNK - 1) / CHUNK;
static_assert(STATIC_BLOCKS <= 512, "the backward grid is capped at 512 blocks");
static __device__ __align__(256) float scratch[(size_t)STATIC_BLOCKS * (NPARAM + 1)];
constexpr int MAX_DEVICES = 64;

hipError_t mlp_static_scratch(float **out)
{
    static std::mutex mu;
    static float *addr[MAX_DEVICES] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = (float *)p;
    }
    *out = addr[dev];
    return hipSuccess;
}

}  // namespace lbm

int lbm_mlp_backward_static(const uint16_t *d_w, const uint16_t *d_x, const float *d_t, int64_t batch, float *d_grad,
                            float *d_loss, void *stream)
{
    if (!d_w || batch < 0 || !d_grad || !d_loss || (batch > 0 && (!d_x || !d_t))) return LBM_EINVAL;
    if (batch > LBM_MLP_STATIC_MAX_BATCH) return LBM_ERANGE;
    float *partial = nullptr;
    if (lbm::mlp_static_scratch(&partial) != hipSuccess) return LBM_EHIP;
    return lbm::launch_mlp_backward(d_w, d_x, d_t, batch, d_grad, d_loss, partial, (hipStream_t)stream) ==
                   hipSuccess
               ? LBM_OK
               : LBM_EHIP;
}
