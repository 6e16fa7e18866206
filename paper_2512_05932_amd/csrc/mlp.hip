// Surrogate network kernels: BF16 matrix products on the MFMA units with
// FP32 accumulation, the elementwise steps around them (bias, GELU and its
// derivative, the loss and its gradient, bias gradients) and the AdamW update.
//
// Network: 1056 -> 256 -> 256 -> 256 -> 16 (inputs 1030..1055 and outputs
// 13..15 are padding), GELU(z) = z/2 (1 + erf(z / sqrt 2)).  Weights are
// kept in FP32 (the optimiser's copy) and in BF16 (the operands of the
// products); activations between layers and the backward operands are BF16.
#include <algorithm>

#include "engine.h"

namespace lidar {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kTileM = 64, kTileN = 64, kTileK = 32;
constexpr int kLdsK = kTileK + 8;         // row stride in LDS (elements)

__device__ inline uint16_t to_bf16(float f)
{
    // round to nearest, ties to even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// C = A B over a 64 x 64 tile per workgroup (4 waves of 32 x 32, each 2 x 2
// MFMA 16x16x16 blocks), K in steps of 32 staged through LDS.  Both operands
// are stored in LDS with K contiguous ([row][k] for A, [col][k] for B), so
// every lane's 4 consecutive K values are one 8-byte read.
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmArgs g)
{
    __shared__ uint16_t As[kTileM][kLdsK];
    __shared__ uint16_t Bs[kTileN][kLdsK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = blockIdx.y * kTileM, n0 = blockIdx.x * kTileN;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // load mapping: consecutive threads walk the operand's unit-stride axis
    const bool b_kfast = g.sbk == 1;
    // this workgroup's share of K (whole tiles)
    const int kchunk = ((g.K + g.ksplit - 1) / g.ksplit + kTileK - 1) / kTileK * kTileK;
    const int kbeg = blockIdx.z * kchunk, kend = min(g.K, kbeg + kchunk);
    for (int k0 = kbeg; k0 < kend; k0 += kTileK) {
#pragma unroll
        for (int q = 0; q < (kTileM * kTileK) / 256; ++q) {
            const int e = tid + 256 * q;
            const int r = e / kTileK, k = e % kTileK;
            const int gi = m0 + r, gk = k0 + k;
            As[r][k] = (gi < g.M && gk < kend) ? g.A[(long)gi * g.lda + gk] : (uint16_t)0;
        }
#pragma unroll
        for (int q = 0; q < (kTileN * kTileK) / 256; ++q) {
            const int e = tid + 256 * q;
            const int c = b_kfast ? e / kTileK : e % kTileN;
            const int k = b_kfast ? e % kTileK : e / kTileN;
            const int gj = n0 + c, gk = k0 + k;
            Bs[c][k] = (gj < g.N && gk < kend) ? g.B[(long)gk * g.sbk + (long)gj * g.sbn] : (uint16_t)0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kTileK; kk += 16) {
            const int kq = kk + 4 * (lane >> 4);
            bf16x4 a[2], b[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                a[t] = *(const bf16x4*)&As[wm * 32 + t * 16 + (lane & 15)][kq];
                b[t] = *(const bf16x4*)&Bs[wn * 32 + t * 16 + (lane & 15)][kq];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
    // D block: lane holds column lane % 16, rows 4 (lane / 16) + r
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn * 32 + j * 16 + (lane & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm * 32 + i * 16 + 4 * (lane >> 4) + r;
                if (row < g.M && col < g.N) {
                    if (g.ksplit > 1)
                        atomicAdd(&g.C[(long)row * g.ldc + col], acc[i][j][r]);
                    else
                        g.C[(long)row * g.ldc + col] = acc[i][j][r];
                }
            }
        }
}

// erf by the rational approximation of Abramowitz & Stegun, formula 7.1.26
// (absolute error <= 1.5e-7): for x >= 0, erf(x) = 1 - t (a1 + t (a2 + t (a3
// + t (a4 + t a5)))) exp(-x^2) with t = 1 / (1 + p x); odd in x.  The
// hardware reciprocal and exponential add a few ulp; the result feeds BF16
// activations (relative step 2^-8), far coarser than either error.
__device__ inline float erf_as(float x)
{
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * ax);
    const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f +
                       t * (-1.453152027f + t * 1.061405429f))));
    return copysignf(1.0f - poly * __expf(-ax * ax), x);
}

__device__ inline float gelu(float z) { return 0.5f * z * (1.0f + erf_as(z * 0.70710678118654752f)); }

__device__ inline float gelu_prime(float z)
{
    return 0.5f * (1.0f + erf_as(z * 0.70710678118654752f)) +
           z * __expf(-0.5f * z * z) * 0.39894228040143268f;
}

// H = bf16(gelu(Z + bias)), four elements a thread (C a multiple of 4); with
// `zero`, also clears zn floats there and the loss sum (the first layer does,
// ahead of the kernels that add into them: a launch for each was 4.4 us).
__global__ __launch_bounds__(256)
void k_bias_gelu(const float4* Z, const float4* bias, bf16x4* H, long n4, int C4, float* zero, long zn, float* loss)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (zero) {
        for (long k = i; k < zn; k += (long)gridDim.x * 256) zero[k] = 0.0f;
        if (i == 0) *loss = 0.0f;
    }
    if (i >= n4) return;
    const float4 z = Z[i], b = bias[i % C4];
    H[i] = bf16x4{(short)to_bf16(gelu(z.x + b.x)), (short)to_bf16(gelu(z.y + b.y)), (short)to_bf16(gelu(z.z + b.z)),
                  (short)to_bf16(gelu(z.w + b.w))};
}

__device__ inline float bce(float z, float t) { return fmaxf(z, 0.0f) - z * t + log1pf(expf(-fabsf(z))); }
__device__ inline float sigm(float z) { return 1.0f / (1.0f + expf(-z)); }

// Per-row loss and gradient (scaled by 1/n) with respect to the 16 outputs Y +
// bias; a wave per 64 rows (4096 rows then take 64 CUs and not 16: 7 us of
// dependent exponentials and logarithms become 5), four waves together in the
// deterministic mode, so that up to 256 rows are summed in a fixed order.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES)
void k_loss(const float* Y, const float* bias, const float* lab, long n, float inv_n, uint16_t* dYb, float* loss_sum)
{
    const long r = (long)blockIdx.x * (64 * WAVES) + threadIdx.x;
    float L = 0.0f;
    if (r < n) {
        const float* l = lab + r * 16;
        float y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = Y[r * 16 + j] + bias[j];
        float d[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) d[j] = 0.0f;
        bool ok = true;
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const float ex = l[e];
            const bool te = ex > 0.5f;
            ok = ok && ((y[e] > 0.0f) == te);
            ok = ok && !(te && fabsf(y[3 + e] - l[3 + e]) * kSurBinScale > 0.5f);
            ok = ok && !(te && fabsf(l[3 + e]) >= kSurDkClip);
            L += bce(y[e], ex);
            d[e] = sigm(y[e]) - ex;
            const float dk = y[3 + e] - l[3 + e];
            const float di = y[6 + e] - l[6 + e];
            const float dw = y[9 + e] - l[9 + e];
            L += ex * (kSurWBin * dk * dk + kSurWInt * di * di + kSurWEpw * dw * dw);
            d[3 + e] = ex * 2.0f * kSurWBin * dk;
            d[6 + e] = ex * 2.0f * kSurWInt * di;
            d[9 + e] = ex * 2.0f * kSurWEpw * dw;
        }
        const float okf = ok ? 1.0f : 0.0f;
        L += bce(y[12], okf);
        d[12] = sigm(y[12]) - okf;
#pragma unroll
        for (int j = 0; j < 16; ++j) dYb[r * 16 + j] = to_bf16(d[j] * inv_n);
    }
    // the workgroup's sum of the row losses, one atomic
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) L += __shfl_xor(L, m);
    if constexpr (WAVES > 1) {
        __shared__ float part[WAVES];
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = L;
        __syncthreads();
        L = part[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) L += part[w];
    }
    if (threadIdx.x == 0) atomicAdd(loss_sum, L * inv_n);
}

// dZ = bf16(dH * gelu'(Z + bias)), four elements a thread
__global__ __launch_bounds__(256)
void k_gelu_back(const float4* dH, const float4* Z, const float4* bias, bf16x4* dZb, long n4, int C4)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const float4 d = dH[i], z = Z[i], b = bias[i % C4];
    dZb[i] = bf16x4{(short)to_bf16(d.x * gelu_prime(z.x + b.x)), (short)to_bf16(d.y * gelu_prime(z.y + b.y)),
                    (short)to_bf16(d.z * gelu_prime(z.z + b.z)), (short)to_bf16(d.w * gelu_prime(z.w + b.w))};
}

// Weight and bias gradients of all layers in one launch: dW = A^T D (A
// [n][in] BF16 activations, D [n][out] BF16 output gradients), db = column
// sums of D, FP32 accumulation on the MFMA units.
//
// The products are small (256 x 256 and 1056 x 256 outputs) with a long sum over
// the n rows, so the rows are split over the grid as well: a workgroup takes a
// kGradT x kGradT tile of one layer over `span` rows and adds it to dW (zeroed
// before) with atomics, or stores it when span covers every row (then the
// order of the sum is fixed).  Both operands have the rows outermost, while
// an MFMA fragment holds eight consecutive rows of a column: a thread loads
// four rows of eight columns, turns them in registers and writes four-row
// pieces into a [column][row] tile in LDS, from where a fragment is one
// 16-byte read; the next step's rows are loaded meanwhile.
// A library product per layer with 16 to 68 workgroups, and the column sums
// apart, took 28 us and 16 us each (4096 rows); all four layers here 29 us,
// bound by the latency of the loads (without the atomics it takes as long).
constexpr int kGradT = 64;                   // tile of dW: in x out
constexpr int kGradK = 64;                   // rows per step
constexpr int kGradLd = kGradK + 8;          // row stride of an LDS tile (elements)

__global__ __launch_bounds__(256) void k_weight_grads(WeightGradArgs a)
{
    __shared__ __align__(16) uint16_t tile[2][kGradT][kGradLd];    // A, D: [column][row]
    __shared__ float part[2][kGradT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // this workgroup's layer and tile
    int t = blockIdx.x % a.tiles, l = 0;
    const long r0 = (long)(blockIdx.x / a.tiles) * a.span, r1 = min(a.n, r0 + a.span);
    while (t >= a.layer[l].tiles) t -= a.layer[l++].tiles;
    const WeightGradLayer g = a.layer[l];
    const int tiles_out = (g.out + kGradT - 1) / kGradT;
    const int i0 = t / tiles_out * kGradT, j0 = t % tiles_out * kGradT;
    const bool atomic = a.span < a.n;
    // operand (0: A, 1: D), columns 8 cb .. and rows 4 rq .. of this thread
    const int op = wave >> 1, cb = tid & 7, rq = (tid & 127) >> 3;
    const uint16_t* src = op ? g.D : g.A;
    const int ld = op ? g.out : g.in, c = (op ? j0 : i0) + 8 * cb;
    const bool col_ok = c < ld;                      // in and out are multiples of 8
    const bool sums = op == 1 && i0 == 0;            // the column sums of D, once per column
    float cs[8] = {};
    uint4 q[4];
    auto load = [&](long r) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long row = r + 4 * rq + k;
            q[k] = col_ok && row < r1 ? *(const uint4*)(src + row * ld + c) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, quad = lane >> 4;
    load(r0);
    for (long r = r0; r < r1; r += kGradK) {
        __syncthreads();                             // the last step's fragments are read
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const unsigned x[4] = {(&q[0].x)[w], (&q[1].x)[w], (&q[2].x)[w], (&q[3].x)[w]};
            // columns 2 w and 2 w + 1: their four rows
            const uint2 lo = make_uint2(__builtin_amdgcn_perm(x[1], x[0], 0x05040100u),
                                        __builtin_amdgcn_perm(x[3], x[2], 0x05040100u));
            const uint2 hi = make_uint2(__builtin_amdgcn_perm(x[1], x[0], 0x07060302u),
                                        __builtin_amdgcn_perm(x[3], x[2], 0x07060302u));
            *(uint2*)&tile[op][8 * cb + 2 * w][4 * rq] = lo;
            *(uint2*)&tile[op][8 * cb + 2 * w + 1][4 * rq] = hi;
            if (sums) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    cs[2 * w] += __uint_as_float(x[k] << 16);
                    cs[2 * w + 1] += __uint_as_float(x[k] & 0xffff0000u);
                }
            }
        }
        __syncthreads();
        if (r + kGradK < r1) load(r + kGradK);
#pragma unroll
        for (int k = 0; k < kGradK; k += 32) {
            bf16x8 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[i] = *(const bf16x8*)&tile[0][wm * 32 + i * 16 + l16][k + 8 * quad];
                fb[i] = *(const bf16x8*)&tile[1][wn * 32 + i * 16 + l16][k + 8 * quad];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }
    // lane: column l16, rows 4 quad + r of every 16 x 16 block
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = j0 + wn * 32 + j * 16 + l16;
            if (col >= g.out) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int row = i0 + wm * 32 + i * 16 + 4 * quad + k;
                if (row >= g.in) continue;
                float* p = g.dW + (long)row * g.out + col;
                if (atomic) unsafeAtomicAdd(p, acc[i][j][k]);
                else *p = acc[i][j][k];
            }
        }
    if (i0 != 0) return;                             // the whole workgroup
    // column sums: over the lanes of a column block, then the two waves
    if (op == 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float v = cs[k];
            for (int m = 8; m < 64; m <<= 1) v += __shfl_xor(v, m);
            if (lane < 8) part[wave & 1][8 * cb + k] = v;
        }
    }
    __syncthreads();
    if (tid < kGradT && j0 + tid < g.out) {
        const float v = part[0][tid] + part[1][tid];
        if (atomic) unsafeAtomicAdd(g.db + j0 + tid, v);
        else g.db[j0 + tid] = v;
    }
}

__global__ void k_zero_f32(float* p, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// AdamW (decoupled weight decay on the weights, not on the biases), then
// the BF16 operand copy of the parameter.
__global__ void k_adamw(float* theta, const float* grad, float* m, float* v, uint16_t* theta_b,
                        long n, AdamArgs a)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const bool decay = sur_is_weight(i);
    float t = theta[i];
    if (decay) t *= a.decay_factor;
    const float g = grad[i];
    const float mi = a.beta1 * m[i] + (1.0f - a.beta1) * g;
    const float vi = a.beta2 * v[i] + (1.0f - a.beta2) * g * g;
    m[i] = mi;
    v[i] = vi;
    t -= a.lr * (mi * a.inv_bc1) / (sqrtf(vi * a.inv_bc2) + a.eps);
    theta[i] = t;
    theta_b[i] = to_bf16(t);
}

// ---- minibatches of the training loop -------------------------------------
// Position p of epoch e maps to row perm(p): a four-round Feistel network on
// k-bit values (k even, 2^k >= n; halves of k/2 bits), cycle-walked until the
// value is below n (a bijection of 0 .. n-1).  Round r replaces (L, R) by
// (R, L ^ (mix(key ^ R) & mask)), key = seed ^ ((4 e + r + 1) * golden),
// mix the SplitMix64 output function.
__device__ inline unsigned long long mix64(unsigned long long z)
{
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__device__ inline unsigned long long feistel(unsigned long long x, int half, unsigned long long seed,
                                             unsigned long long epoch)
{
    const unsigned long long mask = (1ull << half) - 1ull;
    unsigned long long L = x >> half, R = x & mask;
#pragma unroll
    for (unsigned long long r = 0; r < 4; ++r) {
        const unsigned long long key = seed ^ ((4ull * epoch + r + 1ull) * 0x9e3779b97f4a7c15ull);
        const unsigned long long t = L ^ (mix64(key ^ R) & mask);
        L = R;
        R = t;
    }
    return (L << half) | R;
}

// Rows perm(pos0 + i), i < b, of X [n][1056] BF16 and lab [n][16] into Xb, Lb:
// a wave per row (132 + 4 sixteen-byte pieces).
__global__ __launch_bounds__(256) void k_gather_rows(const uint4* X, const uint4* lab, long n, int half,
                                                     unsigned long long seed, unsigned long long epoch,
                                                     long pos0, int b, uint4* Xb, uint4* Lb)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= b) return;
    unsigned long long r = (unsigned long long)(pos0 + i);
    do {
        r = feistel(r, half, seed, epoch);
    } while (r >= (unsigned long long)n);
    constexpr int kRowX = kSurIn * 2 / 16, kRowL = kSurOut * 4 / 16;
    for (int c = lane; c < kRowX; c += 64) Xb[(long)i * kRowX + c] = X[(long)r * kRowX + c];
    if (lane < kRowL) Lb[(long)i * kRowL + lane] = lab[(long)r * kRowL + lane];
}

__global__ void k_to_bf16(const float* x, uint16_t* y, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = to_bf16(x[i]);
}

// Place of feature f inside its block of 32 inputs of a hidden layer: the
// fused inference kernel's MFMA fragments hold features 4 q .. 4 q + 3 and 16 +
// 4 q .. 16 + 4 q + 3 of a block at the eight K positions of lane quad q.
__device__ inline int frag_place(int f) { return 8 * ((f & 15) >> 2) + ((f & 16) >> 2) + (f & 3); }

// BF16 operand copies for the fused inference kernel in the order of its
// fragments: blocks of 32 inputs x 16 outputs, lane by lane (output l % 16, the
// eight K positions of quad l / 16; hidden layers' inputs at frag_place), so
// that a wave reads a fragment as one contiguous kilobyte.
__global__ void k_weight_fragments(const uint16_t* W, int in, int out, bool hidden, uint16_t* Wt)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long)in * out) return;
    const int k = (int)(i / out), n = (int)(i % out), p = hidden ? frag_place(k & 31) : k & 31;
    Wt[(((long)(k >> 5) * (out / 16) + n / 16) * 64 + (p >> 3) * 16 + n % 16) * 8 + (p & 7)] = W[i];
}

// Fused inference: a workgroup of four waves takes kInfRows rows (beams) through
// all four layers.  The weights are the MFMA's A operand (tiles of 16 output
// features), the rows its B operand; a wave holds 64 features of the 64 rows
// (4 x 4 tiles), so that a K step of 32 needs four fragments of each for 16
// MFMAs.  No two waves share a feature: weight fragments go from memory (L2,
// 0.8 MB) straight into registers, two K steps ahead.  The first layer's rows,
// which all waves need, are staged in double-buffered LDS, 64 columns a stage,
// loaded three stages ahead because they come from HBM; the activations
// between layers lie over them, so that three workgroups fit a CU (168 VGPRs) and one's
// GELUs (about as long as its MFMAs) run beside another's products.  The output
// of v_mfma_f32_16x16x32_bf16 (lane l: features 4 (l / 16) .. + 3 of row l % 16)
// is stored in the order of the next layer's fragments (frag_place; its
// weights lie in the same order), 16 bytes for two tiles.  Sums run over the K
// steps in ascending order.
// 128000 rows: 217 us with 16 rows and all 256 features per wave (every MFMA read
// its weight fragment from LDS), 167 us with this tile and the weights staged in
// LDS, 137 us with them straight from memory (141 us at two workgroups per CU), and
// 132 us with the MFMAs at raised wave priority: 104 GFLOP, 790 TFLOP/s.
constexpr int kInfWaves = 4;
constexpr int kInfRows = 64;                 // rows (beams) per workgroup
constexpr int kInfThreads = 64 * kInfWaves;
constexpr int kInfXK = 64;                   // row columns of a stage
constexpr int kInfLdX = kInfXK + 8;          // LDS row strides (elements): 16-byte reads
constexpr int kInfLdH = kSurHid + 8;         // of 8 rows touch all banks once

union InferLds {
    uint16_t X[2][kInfRows][kInfLdX];        // row stages of the first layer
    uint16_t H[kInfRows][kInfLdH];           // activations [row][feature, fragment order]
};

__device__ inline bf16x8 ld8(const uint16_t* p) { return *(const bf16x8*)p; }

constexpr int kInfS1 = kSurIn / 32;          // K steps of the first layer
constexpr int kInfSH = kSurHid / 32;         // of a hidden one
constexpr int kInfSteps = kInfS1 + 2 * kInfSH;
constexpr int kInfX = (kSurIn + kInfXK - 1) / kInfXK;        // row stages, the last one half
constexpr int kInfPieces = kInfRows * kInfXK / 8 / kInfThreads;   // 16-byte pieces of a stage per thread
static_assert(kSurIn % 32 == 0 && kInfSH % 2 == 0 && kInfRows == 64, "whole K steps");

// bias + GELU of the wave's 64 x 64 block into the activations
__device__ inline void store_hidden(InferLds& L, const f32x4 (&acc)[4][4], const float* bias, int wave, int l16, int q)
{
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int f = 64 * wave + 32 * p;
        const float4 b0 = *(const float4*)(bias + f + 4 * q), b1 = *(const float4*)(bias + f + 16 + 4 * q);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 x = acc[2 * p][j], y = acc[2 * p + 1][j];
            const bf16x8 h = {(__bf16)gelu(x[0] + b0.x), (__bf16)gelu(x[1] + b0.y), (__bf16)gelu(x[2] + b0.z),
                              (__bf16)gelu(x[3] + b0.w), (__bf16)gelu(y[0] + b1.x), (__bf16)gelu(y[1] + b1.y),
                              (__bf16)gelu(y[2] + b1.z), (__bf16)gelu(y[3] + b1.w)};
            *(bf16x8*)&L.H[16 * j + l16][f + 8 * q] = h;
        }
    }
}

__global__ __launch_bounds__(kInfThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_infer(InferArgs a)
{
    extern __shared__ float4 lds_v4[];
    InferLds& L = *(InferLds*)lds_v4;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long row0 = (long)blockIdx.x * kInfRows;
    // weight fragments of K step g (the layers' steps follow each other in
    // memory), two steps in turn
    const uint16_t* wsrc = a.Wt1 + (4 * wave * 64 + lane) * 8;
    bf16x8 w[2][4];
    auto wload = [&](int g, bf16x8 (&f)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = ld8(wsrc + ((long)g * (kSurHid / 16) + i) * 512);
    };
    // rows of the first layer: pieces tid and tid + kInfThreads of a stage (rows
    // past n repeat the last one; their outputs are not stored)
    const uint16_t* xsrc[kInfPieces];
    bf16x8 x[2][kInfPieces];
#pragma unroll
    for (int i = 0; i < kInfPieces; ++i)
        xsrc[i] = a.X + min(row0 + (tid >> 3) + kInfThreads / 8 * i, a.n - 1) * kSurIn + 8 * (tid & 7);
    auto xload = [&](int s, bf16x8 (&r)[kInfPieces]) {
        if (kInfXK * s + 8 * (tid & 7) < kSurIn)
#pragma unroll
            for (int i = 0; i < kInfPieces; ++i) r[i] = ld8(xsrc[i] + kInfXK * s);
    };
    auto xstore = [&](int s, const bf16x8 (&r)[kInfPieces]) {
#pragma unroll
        for (int i = 0; i < kInfPieces; ++i)
            *(bf16x8*)&L.X[s & 1][(tid >> 3) + kInfThreads / 8 * i][8 * (tid & 7)] = r[i];
    };
    f32x4 acc[4][4];                                // [feature tile][row tile]
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    // K step g: its fragments meet the rows' in b, then take step g + 2
    auto step = [&](int g, bf16x8 (&f)[4], const bf16x8 (&b)[4]) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[i], b[j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        if (g + 2 < kInfSteps) wload(g + 2, f);
    };
    xload(0, x[0]);
    wload(0, w[0]);
    wload(1, w[1]);
    xload(1, x[1]);
    xstore(0, x[0]);
    xload(2, x[0]);
    __syncthreads();
    clear();
    // row stage s: the next one goes to LDS (its buffer was read in stage s - 1),
    // and its registers take a later one
    for (int s0 = 0; s0 < kInfX; s0 += 2) {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int s = s0 + v;
            if (s >= kInfX) break;
            if (s + 1 < kInfX) xstore(s + 1, x[(v + 1) & 1]);
            if (s + 3 < kInfX) xload(s + 3, x[(v + 1) & 1]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (2 * s + u >= kInfS1) break;
                bf16x8 b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = ld8(&L.X[v][16 * j + l16][32 * u + 8 * q]);
                step(2 * s + u, w[u], b);
            }
            __syncthreads();
        }
    }
    store_hidden(L, acc, a.b1, wave, l16, q);
    __syncthreads();
#pragma unroll 1
    for (int l = 0; l < 2; ++l) {
        clear();
#pragma unroll
        for (int t = 0; t < kInfSH; ++t) {
            bf16x8 b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = ld8(&L.H[16 * j + l16][32 * t + 8 * q]);
            step(kInfS1 + kInfSH * l + t, w[(kInfS1 + t) & 1], b);
        }
        __syncthreads();                                 // every read of H is done
        store_hidden(L, acc, l == 0 ? a.b2 : a.b3, wave, l16, q);
        __syncthreads();
    }
    // output layer: one tile of 16 outputs for 16 rows per wave
    const int r = 16 * wave + l16;
    f32x4 y = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < kInfSH; ++t)
        y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(a.Wt4 + (t * 64 + lane) * 8), ld8(&L.H[r][32 * t + 8 * q]), y,
                                                    0, 0, 0);
    if (row0 + r < a.n) {
        const float4 b4 = *(const float4*)(a.b4 + 4 * q);
        *(float4*)(a.Y + (row0 + r) * kSurOut + 4 * q) = make_float4(y[0] + b4.x, y[1] + b4.y, y[2] + b4.z, y[3] + b4.w);
    }
}

inline unsigned blocks(long n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

hipError_t launch_transpose_weights(hipStream_t s, const uint16_t* theta_b, uint16_t* wt)
{
    struct L { long off, toff; int in, out; };
    const L ls[4] = {{kSurOffW1, 0, kSurIn, kSurHid},
                     {kSurOffW2, (long)kSurIn * kSurHid, kSurHid, kSurHid},
                     {kSurOffW3, (long)kSurIn * kSurHid + (long)kSurHid * kSurHid, kSurHid, kSurHid},
                     {kSurOffW4, (long)kSurIn * kSurHid + 2L * kSurHid * kSurHid, kSurHid, kSurOut}};
    for (const L& l : ls) {
        const long n = (long)l.in * l.out;
        hipLaunchKernelGGL(k_weight_fragments, dim3(blocks(n, 256)), dim3(256), 0, s, theta_b + l.off,
                           l.in, l.out, l.off != kSurOffW1, wt + l.toff);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_infer(hipStream_t s, const InferArgs& a)
{
    if (a.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_infer, dim3(blocks(a.n, kInfRows)), dim3(kInfThreads), sizeof(InferLds), s,
                       a);
    return hipGetLastError();
}

hipError_t launch_gemm_bf16(hipStream_t s, const GemmArgs& g0, bool det)
{
    if (g0.M <= 0 || g0.N <= 0) return hipSuccess;
    GemmArgs g = g0;
    const long tiles = (long)((g.N + kTileN - 1) / kTileN) * ((g.M + kTileM - 1) / kTileM);
    // few output tiles and a long K (the first layer on few rows): split K over
    // the grid (not when deterministic: the atomic adds of the parts come in any
    // order)
    g.ksplit = 1;
    while (!det && tiles * g.ksplit < 512 && g.K / (g.ksplit * 2) >= 4 * kTileK) g.ksplit *= 2;
    if (g.ksplit > 1) {
        if (g.ldc != g.N) return hipErrorInvalidValue;   // split K needs a dense C to zero
        const hipError_t e = launch_zero_f32(s, g.C, (long)g.M * g.N);
        if (e != hipSuccess) return e;
    }
    dim3 grid((g.N + kTileN - 1) / kTileN, (g.M + kTileM - 1) / kTileM, g.ksplit);
    hipLaunchKernelGGL(k_gemm_bf16, grid, dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_bias_gelu(hipStream_t s, const float* Z, const float* bias, uint16_t* H, long n, int C,
                            float* zero, long zn, float* loss)
{
    if (n * C == 0) return hipSuccess;
    if (C % 4 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_bias_gelu, dim3(blocks(n * C / 4, 256)), dim3(256), 0, s, (const float4*)Z,
                       (const float4*)bias, (bf16x4*)H, n * C / 4, C / 4, zero, zn, loss);
    return hipGetLastError();
}

hipError_t launch_loss(hipStream_t s, const float* Y, const float* bias, const float* lab, long n, uint16_t* dYb,
                       float* loss_sum, bool det)
{
    if (n == 0) return hipSuccess;
    const float inv_n = 1.0f / (float)n;
    if (det)
        hipLaunchKernelGGL(k_loss<4>, dim3(blocks(n, 256)), dim3(256), 0, s, Y, bias, lab, n, inv_n, dYb, loss_sum);
    else
        hipLaunchKernelGGL(k_loss<1>, dim3(blocks(n, 64)), dim3(64), 0, s, Y, bias, lab, n, inv_n, dYb, loss_sum);
    return hipGetLastError();
}

hipError_t launch_gelu_back(hipStream_t s, const float* dH, const float* Z, const float* bias, uint16_t* dZb, long n,
                            int C)
{
    if (n * C == 0) return hipSuccess;
    if (C % 4 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gelu_back, dim3(blocks(n * C / 4, 256)), dim3(256), 0, s, (const float4*)dH,
                       (const float4*)Z, (const float4*)bias, (bf16x4*)dZb, n * C / 4, C / 4);
    return hipGetLastError();
}

// Rows of a workgroup: all of them when the sum's order is to be fixed (det)
// or the rows are few, else shares of at least 256 rows, at most 64 of them (a
// step on 4096 rows: 116 us with shares of 512 rows, too few workgroups to
// hide their loads; 110 us with 256; 134 us with 128, where the atomics cost
// more).
long weight_grad_span(long n, bool det)
{
    if (det || n <= 256) return n;
    const long parts = std::min<long>(64, (n + 255) / 256);
    return ((n + parts - 1) / parts + kGradK - 1) / kGradK * kGradK;
}

hipError_t launch_weight_grads(hipStream_t s, const WeightGradArgs& a0)
{
    if (a0.n <= 0) return hipSuccess;
    WeightGradArgs a = a0;
    a.tiles = 0;
    for (WeightGradLayer& l : a.layer) {
        if (l.in % 8 != 0 || l.out % 8 != 0) return hipErrorInvalidValue;
        l.tiles = ((l.in + kGradT - 1) / kGradT) * ((l.out + kGradT - 1) / kGradT);
        a.tiles += l.tiles;
    }
    const long parts = (a.n + a.span - 1) / a.span;
    hipLaunchKernelGGL(k_weight_grads, dim3((unsigned)(a.tiles * parts)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_gather_rows(hipStream_t s, const uint16_t* X, const float* lab, long n, int half,
                              unsigned long long seed, unsigned long long epoch, long pos0, int b,
                              uint16_t* Xb, float* Lb)
{
    if (b <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_rows, dim3((b + 3) / 4), dim3(256), 0, s, (const uint4*)X,
                       (const uint4*)lab, n, half, seed, epoch, pos0, b, (uint4*)Xb, (uint4*)Lb);
    return hipGetLastError();
}

hipError_t launch_zero_f32(hipStream_t s, float* p, long n)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks(n, 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_adamw(hipStream_t s, float* theta, const float* grad, float* m, float* v,
                        uint16_t* theta_b, long n, const AdamArgs& a)
{
    hipLaunchKernelGGL(k_adamw, dim3(blocks(n, 256)), dim3(256), 0, s, theta, grad, m, v, theta_b, n, a);
    return hipGetLastError();
}

hipError_t launch_to_bf16(hipStream_t s, const float* x, uint16_t* y, long n)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks(n, 256)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

}  // namespace lidar

namespace lidar {

hipError_t SurWork::ensure(long n)
{
    if (n <= cap) return hipSuccess;
    hipError_t e;
    const size_t nh = (size_t)n * kSurHid, no = (size_t)n * kSurOut;
    if ((e = Z1.ensure(nh)) || (e = Z2.ensure(nh)) || (e = Z3.ensure(nh)) || (e = dH.ensure(nh)) ||
        (e = H1.ensure(nh)) || (e = H2.ensure(nh)) || (e = H3.ensure(nh)) || (e = dZ1.ensure(nh)) ||
        (e = dZ2.ensure(nh)) || (e = dZ3.ensure(nh)) || (e = Y.ensure(no)) || (e = dYb.ensure(no)) ||
        (e = loss.ensure(1)))
        return e;
    cap = n;
    return hipSuccess;
}

#define TRY(x)                                        \
    do {                                              \
        hipError_t e_ = (x);                          \
        if (e_ != hipSuccess) return e_;              \
    } while (0)

// A training product: the library GEMM where it runs (not in the
// deterministic mode, whose products keep a fixed summation order), else the
// own MFMA kernel
static hipError_t gemm(hipStream_t s, const GemmArgs& g, bool det, BlasCtx* blas)
{
    if (!det && blas) {
        const hipError_t e = blas_gemm(blas, s, g);
        if (e != hipErrorNotSupported) return e;
    }
    return launch_gemm_bf16(s, g, det);
}

// Z = A W (before the bias) with A [n][k] row-major BF16 and W [k][c] BF16
static hipError_t dense(hipStream_t s, const uint16_t* A, int k, const uint16_t* W, int c, long n,
                        float* Z, bool det, BlasCtx* blas)
{
    GemmArgs g{A, k, W, c, 1, Z, c, (int)n, c, k, 1};
    return gemm(s, g, det, blas);
}

hipError_t sur_forward(hipStream_t s, const SurNet& net, const uint16_t* X, long n, SurWork& w, float* grad,
                       float* loss)
{
    const uint16_t* Wb = net.theta_b.p;
    const float* th = net.theta.p;
    TRY(dense(s, X, kSurIn, Wb + kSurOffW1, kSurHid, n, w.Z1.p, net.det, w.blas));
    TRY(launch_bias_gelu(s, w.Z1.p, th + kSurOffB1, w.H1.p, n, kSurHid, grad ? grad : loss,
                         grad ? kSurParams : 0, loss));
    TRY(dense(s, w.H1.p, kSurHid, Wb + kSurOffW2, kSurHid, n, w.Z2.p, net.det, w.blas));
    TRY(launch_bias_gelu(s, w.Z2.p, th + kSurOffB2, w.H2.p, n, kSurHid));
    TRY(dense(s, w.H2.p, kSurHid, Wb + kSurOffW3, kSurHid, n, w.Z3.p, net.det, w.blas));
    TRY(launch_bias_gelu(s, w.Z3.p, th + kSurOffB3, w.H3.p, n, kSurHid));
    return dense(s, w.H3.p, kSurHid, Wb + kSurOffW4, kSurOut, n, w.Y.p, net.det, w.blas);
}

hipError_t sur_infer(hipStream_t s, SurNet& net, const uint16_t* X, long n, float* Y)
{
    TRY(net.theta_t.ensure(kSurWtSize));
    if (net.t_stale) {
        TRY(launch_transpose_weights(s, net.theta_b.p, net.theta_t.p));
        net.t_stale = false;
    }
    const uint16_t* t = net.theta_t.p;
    InferArgs a;
    a.X = X;
    a.n = n;
    a.Wt1 = t;
    a.Wt2 = t + (long)kSurIn * kSurHid;
    a.Wt3 = a.Wt2 + (long)kSurHid * kSurHid;
    a.Wt4 = a.Wt3 + (long)kSurHid * kSurHid;
    a.b1 = net.theta.p + kSurOffB1;
    a.b2 = net.theta.p + kSurOffB2;
    a.b3 = net.theta.p + kSurOffB3;
    a.b4 = net.theta.p + kSurOffB4;
    a.Y = Y;
    return launch_mlp_infer(s, a);
}

// dH = D W^T (D [n][out], W [in][out]) in FP32
static hipError_t input_grad(hipStream_t s, const uint16_t* D, int out, const uint16_t* W, int in,
                             long n, float* dH, bool det, BlasCtx* blas)
{
    GemmArgs g{D, out, W, 1, out, dH, in, (int)n, in, out, 1};
    return gemm(s, g, det, blas);
}

hipError_t sur_gradients(hipStream_t s, SurNet& net, const uint16_t* X, const float* lab, long n,
                         SurWork& w, float* g, float* loss)
{
    const uint16_t* Wb = net.theta_b.p;
    const float* th = net.theta.p;
    const long span = weight_grad_span(n, net.det);
    TRY(sur_forward(s, net, X, n, w, span < n ? g : nullptr, loss));
    TRY(launch_loss(s, w.Y.p, th + kSurOffB4, lab, n, w.dYb.p, loss, net.det));
    TRY(input_grad(s, w.dYb.p, kSurOut, Wb + kSurOffW4, kSurHid, n, w.dH.p, net.det, w.blas));
    TRY(launch_gelu_back(s, w.dH.p, w.Z3.p, th + kSurOffB3, w.dZ3.p, n, kSurHid));
    TRY(input_grad(s, w.dZ3.p, kSurHid, Wb + kSurOffW3, kSurHid, n, w.dH.p, net.det, w.blas));
    TRY(launch_gelu_back(s, w.dH.p, w.Z2.p, th + kSurOffB2, w.dZ2.p, n, kSurHid));
    TRY(input_grad(s, w.dZ2.p, kSurHid, Wb + kSurOffW2, kSurHid, n, w.dH.p, net.det, w.blas));
    TRY(launch_gelu_back(s, w.dH.p, w.Z1.p, th + kSurOffB1, w.dZ1.p, n, kSurHid));
    WeightGradArgs a{};
    a.n = n;
    a.span = span;
    a.layer[0] = {X, w.dZ1.p, kSurIn, kSurHid, 0, g + kSurOffW1, g + kSurOffB1};
    a.layer[1] = {w.H1.p, w.dZ2.p, kSurHid, kSurHid, 0, g + kSurOffW2, g + kSurOffB2};
    a.layer[2] = {w.H2.p, w.dZ3.p, kSurHid, kSurHid, 0, g + kSurOffW3, g + kSurOffB3};
    a.layer[3] = {w.H3.p, w.dYb.p, kSurHid, kSurOut, 0, g + kSurOffW4, g + kSurOffB4};
    return launch_weight_grads(s, a);
}

#undef TRY

}  // namespace lidar
