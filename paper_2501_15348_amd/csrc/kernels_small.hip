// Dense steps of few rows, a call of their own: a product or a recurrent step that does not fill the chip.
//   gemm_small   out[n,M] = act((row_scale .* A)[n,K] * W[K,M] + b)
//   rnn_small    one GRU / LSTM step
//
// The kernels for many rows stage or prepare the weights once per block and walk through row tiles; with a few tiles that
// leaves most compute units without work and each busy one with a chain of staging, waiting and many matrix instructions.
// Here a block makes ONE tile of 32 rows by 32 columns (units): its waves split the terms (gemm_small: quarters; rnn_small:
// a wave per gate and source), request all they need at once, straight from memory, multiply with the fp32 matrix
// instructions, and add their parts through LDS.  Bound by latency: one round of loads, a quarter of the matrix instructions,
// one exchange.  The parts are short sums in fp32: the error is below that of the kernels for many rows (root mean square
// against 64 bits: 128 -> 128 7.3e-8 against 9.9e-8, 602 -> 128 1.3e-7 against 2.5e-7, GRU 128/128 5.7e-8 against 7.2e-8).
// Measured, kernel, before and now: 200 rows 64 -> 64 6.9 -> 3.5 us, 3200 rows 8.2 -> 3.6; 800 rows 128 -> 128 13.4 -> 4.4;
// 200 rows 1433 -> 16 146 -> 24; 800 rows GRU 64/64 16.1 -> 8.1, GRU 128/128 23.4 -> 13.0, LSTM 128/64 21.5 -> 11.8.
#include "ctx.h"

namespace reinc {

namespace {

typedef float acc16 __attribute__((ext_vector_type(16)));

constexpr int kGroups = 8;  // groups of eight terms a wave requests at once

// Where the kernels for many rows take over, in tiles: four blocks per compute unit (64 -> 64 at 800 tiles 5.8 against 8.5 us,
// at 1600 9.1 against 9.1; 256 -> 256 at 800 13.1 against 20.9, at 1600 20.6 against 21.9; bf16 256 -> 256 at 1600 22.4
// against 19.9), and one of the six or eight waves of a recurrent step (GRU 128/128 at 200 tiles 13.4 against 24.2, at 400 25
// against 24; LSTM 128/128 at 200 15.8 against 18.7, at 400 28 against 21).  Products deeper than the plane kernels take have
// only kernels that walk the terms block by block against them: up to twice the tiles, of columns that give those few
// blocks (602 -> 128 at 2000 tiles 81 against 199; 1024 -> 512 85 against 78), and recurrent steps of any size (GRU 512/64 at
// 500 tiles 52 against 167, at 2000 197 against 203; LSTM 602/128 at 8000 1297 against 2335; GRU 300/300 at 20000 1658
// against 3064).
constexpr int kSmallGemmTiles = 1024, kSmallRnnTiles = 256;

// four values at p, of which the first `count` (may be <= 0) exist
template <bool BF16>
__device__ inline void load_four(const void *base, int64_t at, int count, bool vec, float (&v)[4])
{
    if (BF16) {
        const uint16_t *p = static_cast<const uint16_t *>(base) + at;
        if (vec && count >= 4) {
            const uint2 x = *reinterpret_cast<const uint2 *>(p);
            v[0] = __uint_as_float(x.x << 16), v[1] = __uint_as_float(x.x & 0xFFFF0000u);
            v[2] = __uint_as_float(x.y << 16), v[3] = __uint_as_float(x.y & 0xFFFF0000u);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = e < count ? __uint_as_float(uint32_t(p[e]) << 16) : 0.0f;
        }
    } else {
        const float *p = static_cast<const float *>(base) + at;
        if (vec && count >= 4) {
            const float4 x = *reinterpret_cast<const float4 *>(p);
            v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = e < count ? p[e] : 0.0f;
        }
    }
}

__device__ inline acc16 none()
{
    acc16 z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.0f;
    return z;
}

// the terms [k0, k1) of 32 rows of A (rows of K values; `row`: the lane's) with 32 columns of W (`col`: the lane's;
// element (k, col) at W[k * ldw + col]).  Of a group of eight terms a lane holds four, of its half; the groups go to CHAINS
// sums in turn (the longer a chain, the larger its error: one of 128 terms had 1.06 times that of the kernels for many rows).
template <bool BF16, int CHAINS>
__device__ inline acc16 tile_terms(const void *A, int64_t row, int K, bool vec, float scale, const float *W, int ldw, int col, int k0, int k1)
{
    const int kk = (threadIdx.x >> 5) & 1;
    acc16 acc[CHAINS];
#pragma unroll
    for (int c = 0; c < CHAINS; ++c) acc[c] = none();
#pragma unroll 1
    for (int kb = k0; kb < k1; kb += 8 * kGroups) {
        float a[kGroups][4], b[kGroups][4];
#pragma unroll
        for (int u = 0; u < kGroups; ++u) {
            if (kb + 8 * u >= k1) break;  // (the same for the whole wave)
            const int k = kb + 8 * u + 4 * kk;
            load_four<BF16>(A, row * K + k, k1 - k, vec, a[u]);
            const float *w = W + int64_t(k) * ldw + col;
#pragma unroll
            for (int e = 0; e < 4; ++e, w += ldw) b[u][e] = k + e < k1 ? *w : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kGroups; ++u) {
            if (kb + 8 * u >= k1) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // (a term past the end stays 0 under a scale that is not finite)
                const float ae = kb + 8 * u + 4 * kk + e < k1 ? a[u][e] * scale : 0.0f;
                acc[u % CHAINS] = __builtin_amdgcn_mfma_f32_32x32x2f32(ae, b[u][e], acc[u % CHAINS], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int c = CHAINS / 2; c > 0; c /= 2)
#pragma unroll
        for (int q = 0; q < c; ++q) acc[q] += acc[q + c];
    return acc[0];
}

// a wave's part of the tile to LDS
__device__ inline void put_part(float (&part)[32][33], const acc16 &acc)
{
    const int i = threadIdx.x & 31, kk = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int e = 0; e < 16; ++e) part[8 * (e / 4) + 4 * kk + e % 4][i] = acc[e];
}

struct SmallGemmArgs {
    const void *A;
    int64_t n;
    int K, M;
    const float *row_scale, *W, *bias;
    int relu, vec;
    float *out;
};

template <bool BF16>
__global__ void __launch_bounds__(256) gemm_small(SmallGemmArgs g)
{
    __shared__ float part[4][32][33];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 31;
    const int64_t row0 = int64_t(blockIdx.x) * 32, row = min(row0 + i, g.n - 1);
    const int c0 = blockIdx.y * 32;
    const int quarter = (g.K + 31) / 32 * 8, k0 = w * quarter, k1 = min(g.K, k0 + quarter);
    const float scale = g.row_scale ? g.row_scale[row] : 1.0f;
    put_part(part[w], tile_terms<BF16, 1>(g.A, row, g.K, g.vec, scale, g.W, g.M, min(c0 + i, g.M - 1), k0, k1));
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = (threadIdx.x >> 5) + 8 * q, c = c0 + i;
        if (row0 + r >= g.n || c >= g.M) continue;
        float v = (part[0][r][i] + part[1][r][i]) + (part[2][r][i] + part[3][r][i]);
        if (g.bias) v += g.bias[c];
        if (g.relu) v = fmaxf(v, 0.0f);
        g.out[(row0 + r) * g.M + c] = v;
    }
}

struct SmallRnnArgs {
    const float *x;
    int64_t n;
    int d, H;
    const float *h_prev, *carry;  // carry: GRU the state, LSTM c_prev; null: zero
    const float *W_i, *W_h, *b_i, *b_h;
    float *h_out, *c_out, *saved;
    int vec_x, vec_h;
};

// (as in the other recurrent kernels: the hardware's exp2 and reciprocal)
__device__ inline float sigmoid(float v) { return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * v)); }
__device__ inline float hyperbolic(float v) { return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(2.88539008f * v)); }

template <bool LSTM>
__global__ void __launch_bounds__(LSTM ? 512 : 384) rnn_small(SmallRnnArgs g)
{
    constexpr int KG = LSTM ? 4 : 3;
    __shared__ float part[2 * KG][32][33];  // per gate the terms of x, then those of h
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 31;
    const int64_t row0 = int64_t(blockIdx.x) * 32, row = min(row0 + i, g.n - 1);
    const int u0 = blockIdx.y * 32, H = g.H, gate = w % KG;
    const int col = gate * H + min(u0 + i, H - 1);
    if (w < KG)
        put_part(part[w], tile_terms<false, 4>(g.x, row, g.d, g.vec_x, 1.0f, g.W_i, KG * H, col, 0, g.d));
    else
        put_part(part[w], g.h_prev ? tile_terms<false, 4>(g.h_prev, row, H, g.vec_h, 1.0f, g.W_h, KG * H, col, 0, H) : none());
    __syncthreads();
    const int j = u0 + i;
    if (j >= H) return;
    float bi[KG], bh[KG];
#pragma unroll
    for (int t = 0; t < KG; ++t) {
        bi[t] = g.b_i ? g.b_i[t * H + j] : 0.0f;
        bh[t] = g.b_h ? g.b_h[t * H + j] : 0.0f;
    }
    for (int r = threadIdx.x >> 5; r < 32; r += 2 * (2 * KG)) {
        if (row0 + r >= g.n) break;
        const int64_t o = (row0 + r) * H + j;
        const float prev = g.carry ? g.carry[o] : 0.0f;
        auto sum = [&](int t) { return (part[t][r][i] + part[KG + t][r][i]) + (bi[t] + bh[t]); };
        const float k0 = sigmoid(sum(0)), k1 = sigmoid(sum(1));
        float k2, k3, hn;
        if (LSTM) {
            k2 = hyperbolic(sum(2));
            k3 = sigmoid(sum(KG - 1));
            const float cn = k1 * prev + k0 * k2;
            g.c_out[o] = cn;
            hn = k3 * hyperbolic(cn);
        } else {
            k3 = part[KG + 2][r][i] + bh[2];
            k2 = hyperbolic(part[2][r][i] + bi[2] + k0 * k3);
            hn = k2 + k1 * (prev - k2);
        }
        g.h_out[o] = hn;
        if (g.saved) {
            float *sv = g.saved + (row0 + r) * 4 * H + j;
            sv[0] = k0;
            sv[H] = k1;
            sv[2 * H] = k2;
            sv[3 * H] = k3;
        }
    }
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

int64_t tiles(int64_t n, int M) { return ((n + 31) / 32) * ((M + 31) / 32); }

// a block writes before another one has read the row: outputs that lie in an input are left to the kernels for many rows
bool apart(const float *out, int64_t out_count, const void *in, int64_t in_bytes)
{
    const uintptr_t o = reinterpret_cast<uintptr_t>(out), i = reinterpret_cast<uintptr_t>(in);
    return !out || !in || o + uintptr_t(4 * out_count) <= i || i + uintptr_t(in_bytes) <= o;
}

}  // namespace

bool launch_gemm_small(const void *A, int a_bf16, int64_t n, int32_t K, int32_t M, const float *row_scale, const float *W,
                       const float *bias, int relu, float *out, hipStream_t s)
{
    if (n <= 0 || M > 32 * 65535 || tiles(n, M) > (K > kMaxPlaneK && M <= 128 ? 2 : 1) * kSmallGemmTiles) return false;
    if (!apart(out, n * M, A, n * K * (a_bf16 ? 2 : 4))) return false;
    const SmallGemmArgs g{A, n, K, M, row_scale, W, bias, relu, aligned16(A) && K % 4 == 0, out};
    const dim3 grid(unsigned((n + 31) / 32), unsigned((M + 31) / 32));
    if (a_bf16)
        gemm_small<true><<<grid, 256, 0, s>>>(g);
    else
        gemm_small<false><<<grid, 256, 0, s>>>(g);
    return true;
}

bool launch_rnn_small(int lstm, const float *x, int64_t n, int32_t d_in, int32_t H, const float *h_prev, const float *c_prev,
                      const float *W_i, const float *W_h, const float *b_i, const float *b_h, float *h_out, float *c_out, float *saved,
                      hipStream_t s)
{
    if (n <= 0 || H > 32 * 65535 || (plane_pad(d_in) + plane_pad(H) <= kMaxPlaneK && tiles(n, H) > kSmallRnnTiles)) return false;
    for (const float *in : {x, h_prev})
        for (const float *out : {h_out, c_out, saved})
            if (!apart(out, n * H * (out == saved ? 4 : 1), in, 4 * n * (in == x ? d_in : H))) return false;
    const SmallRnnArgs g{x, n, d_in, H, h_prev, lstm ? c_prev : h_prev, W_i, W_h, b_i, b_h, h_out, c_out, saved,
                         aligned16(x) && d_in % 4 == 0, aligned16(h_prev) && H % 4 == 0};
    const dim3 grid(unsigned((n + 31) / 32), unsigned((H + 31) / 32));
    if (lstm)
        rnn_small<true><<<grid, 512, 0, s>>>(g);
    else
        rnn_small<false><<<grid, 384, 0, s>>>(g);
    return true;
}

}  // namespace reinc
