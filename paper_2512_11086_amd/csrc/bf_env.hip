// bf_env.hip -- envelope detection and display compression of beamformed
// images (the stage after DAS: the paper's Hilbert transform and its log /
// power display scales).
//
// A real (RF) image is [n_cols][N] with depth fastest; the envelope of a
// column is |x_a| with x_a its analytic signal along depth:
//     X = DFT_N(x),  X_a[k] = h[k] X[k]  (h = 1 at DC and Nyquist, 2 for
//     positive, 0 for negative frequencies),  x_a = IDFT_N(X_a).
// Power-of-two N from 64 to 256: env_fft_tile_kernel, two columns packed as one
// complex sequence, N = R L with R values in each of L lanes, FFTs inside the
// lanes and one transposition through LDS each way.  N = 512 and 1024: one
// wavefront per two columns (packed alike, env_fft_reg_kernel), FFT held in
// registers (four-step split N = 64 M: a 64-point FFT across the lanes by
// xor-partner exchanges, a twiddle, an M-point FFT inside each lane, then the
// mirror image for the inverse); no LDS passes and no barriers.  Other power-of-two N: one
// workgroup per column, radix-2 FFT in LDS (forward decimation-in-time from a
// bit-reversed load, spectrum weighting, inverse decimation-in-frequency, read
// back in bit-reversed order).  Twiddles come from a host-FP64, stage-major
// table in global memory (stage len holds exp(-j 2 pi pos / len) for pos <
// len / 2 at offset len / 2 - 1), so the lanes of a stage read consecutive
// entries (cached; no LDS bank conflicts).  Other N: Re x_a = x exactly, and
// Im x_a is the circular convolution of x with q = Im IDFT(h) (host FP64): a
// circulant product on the matrix cores (env_circ_kernel), or summed directly
// below 24 and above 1000 samples.
// IQ images already are analytic: the envelope is |z|.
//
// Compression (ref > 0 is fused into the store; ref <= 0 uses the image
// maximum: every workgroup writes the maximum of its envelope values to a
// partial-max buffer, one workgroup reduces it in a fixed order, and a second
// pass applies the compression -- no atomics, so repeated calls agree):
//     log:   y = max(20 log10(env / ref), -param)
//     power: y = min(env / ref, 1)^param
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "bf.h"
#include "bf_common.h"
#include "bf_plan.h"

namespace bf {

constexpr int ENV_MAX_N = 4096;

struct EnvArgs {
    const float *img;        // [n_cols][N] real, or [n_cols][N][2] complex (iq)
    float *out;              // [n_cols][N]
    const float2 *tw;        // FFT: [N - 1] stage-major twiddles (see above)
    const float2 *tw_lane;   // register FFT: [6][64] W_{2d}^{l mod d}, d = 32, 16, .., 1
    const float2 *tw_mid;    // register FFT: [64][M] W_N^{r bitrev6(l)}; tile FFT: [R][L] W_N^{k l}
    float2 wm[8];            // register FFT: W_M^j, j < M / 2
    const float *q;          // direct path: [N] Im IDFT(h)
    float *part_max;         // [n_parts] per-workgroup maxima (ref <= 0)
    float *img_max;          // reduced maximum (ref <= 0)
    int n_parts;             // partial maxima the compression pass reduces itself (0: img_max)
    int given;               // ref is the maximum of part_max (second pass of the tile FFT)
    int vec;                 // out holds whole 16-byte groups (compression pass)
    long n_cols;
    int N, log2n;
    int compress;
    float ref, param;
    float inv_ref;           // 1 / ref (ref > 0)
};

// Compression with the hardware base-2 logarithm and exponential (about 1 ulp
// each): 20 log10(x) = (20 log10 2) log2(x) and x^p = 2^(p log2 x); x = 0
// gives log2 = -inf, i.e. -param dB and 0 (param > 0).  inv_ref = 1 / ref.
__device__ inline float compress_value(float env, int mode, float inv_ref, float param)
{
    const float x = env * inv_ref;
    if (mode == BF_COMPRESS_LOG)
        return fmaxf(6.0205999132796239f * __builtin_amdgcn_logf(x), -param);
    if (mode == BF_COMPRESS_POWER)
        return __builtin_amdgcn_exp2f(param * __builtin_amdgcn_logf(fminf(x, 1.f)));
    return env;
}

// Store one envelope value: compressed now (ref given), or raw with the
// running maximum (compression pass follows).
__device__ inline void store_env(const EnvArgs &a, long idx, float env, float &local_max)
{
    if (a.compress != BF_COMPRESS_NONE && a.ref > 0.f) {
        a.out[idx] = compress_value(env, a.compress, a.inv_ref, a.param);
    } else {
        a.out[idx] = env;
        local_max = fmaxf(local_max, env);
    }
}

// Maximum of the workgroup's envelope values to part_max[blockIdx.x]
// (wavefront shuffles, then LDS across wavefronts; blockDim <= 256).
__device__ inline void publish_max(const EnvArgs &a, float local_max)
{
    if (!(a.compress != BF_COMPRESS_NONE && a.ref <= 0.f)) return;
    __shared__ float s_max[4];
    for (int o = 32; o > 0; o >>= 1) local_max = fmaxf(local_max, __shfl_xor(local_max, o, 64));
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = local_max;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = s_max[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmaxf(m, s_max[w]);
        a.part_max[blockIdx.x + gridDim.x * blockIdx.y] = m;
    }
}

// The image maximum from the partial maxima, by every workgroup for itself (at
// most ENV_FEW_PARTS of them).
constexpr int ENV_FEW_PARTS = 2048;
__device__ inline float max_of_parts(const EnvArgs &a)
{
    __shared__ float s[4];
    float m = 0.f;
    for (int i = threadIdx.x; i < a.n_parts; i += blockDim.x) m = fmaxf(m, a.part_max[i]);
    for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
    __syncthreads();
    m = s[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmaxf(m, s[w]);
    return m;
}

// One value compressed by the image maximum a.ref (an all-zero image gives
// -param or 0).
__device__ inline float compress_by_max(const EnvArgs &a, float env)
{
    return a.ref > 0.f ? compress_value(env, a.compress, a.inv_ref, a.param)
                       : a.compress == BF_COMPRESS_LOG ? -a.param : 0.f;
}

__device__ inline float2 cmul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

__device__ inline unsigned bitrev(unsigned v, int bits) { return __brev(v) >> (32 - bits); }

// grid: n_cols workgroups of T threads; LDS: N float2 data
__global__ __launch_bounds__(256) void env_fft_kernel(EnvArgs a)
{
    extern __shared__ float2 sm[];
    float2 *d = sm;
    const float2 *__restrict__ tw = a.tw;
    const int N = a.N, half_n = N >> 1, T = blockDim.x, t = threadIdx.x;
    const long col = blockIdx.x;
    const float *x = a.img + col * N;
    for (int n = t; n < N; n += T) d[bitrev(n, a.log2n)] = make_float2(x[n], 0.f);
    __syncthreads();
    // forward DIT: butterflies (i, i + h) with twiddle exp(-j 2 pi pos / len)
    for (int len = 2; len <= N; len <<= 1) {
        const int h = len >> 1;
        const float2 *twl = tw + (h - 1);
        for (int b = t; b < half_n; b += T) {
            const int pos = b & (h - 1);
            const int i = ((b - pos) << 1) + pos;
            const float2 u = d[i], v = cmul(d[i + h], twl[pos]);
            d[i] = make_float2(u.x + v.x, u.y + v.y);
            d[i + h] = make_float2(u.x - v.x, u.y - v.y);
        }
        __syncthreads();
    }
    // analytic-signal weights: 1 at DC and Nyquist, 2 positive, 0 negative
    for (int k = t; k < N; k += T) {
        const float w = (k == 0 || k == half_n) ? 1.f : (k < half_n ? 2.f : 0.f);
        d[k] = make_float2(d[k].x * w, d[k].y * w);
    }
    __syncthreads();
    // inverse DIF: butterflies (i, i + h), (u + v, (u - v) exp(+j 2 pi pos / len))
    for (int len = N; len >= 2; len >>= 1) {
        const int h = len >> 1;
        const float2 *twl = tw + (h - 1);
        for (int b = t; b < half_n; b += T) {
            const int pos = b & (h - 1);
            const int i = ((b - pos) << 1) + pos;
            const float2 u = d[i], v = d[i + h];
            const float2 w = twl[pos];
            d[i] = make_float2(u.x + v.x, u.y + v.y);
            d[i + h] = cmul(make_float2(u.x - v.x, u.y - v.y), make_float2(w.x, -w.y));
        }
        __syncthreads();
    }
    const float inv_n = 1.f / (float)N;
    float local_max = 0.f;
    for (int n = t; n < N; n += T) {
        const float2 z = d[bitrev(n, a.log2n)];
        store_env(a, col * N + n, sqrtf(z.x * z.x + z.y * z.y) * inv_n, local_max);
    }
    publish_max(a, local_max);
}

// Any N: y = Im x_a = sum_k q[k] x[(n - k) mod N]; env = sqrt(x^2 + y^2).
// LDS holds the column twice (no modulo in the sum) and q.
__global__ __launch_bounds__(256) void env_direct_kernel(EnvArgs a)
{
    extern __shared__ float sf[];
    const int N = a.N, T = blockDim.x, t = threadIdx.x;
    float *x2 = sf;            // [2N]: x2[i] = x[i mod N]
    float *q = sf + 2 * N;     // [N]
    const long col = blockIdx.x;
    const float *x = a.img + col * N;
    for (int i = t; i < N; i += T) {
        const float v = x[i];
        x2[i] = v;
        x2[i + N] = v;
        q[i] = a.q[i];
    }
    __syncthreads();
    float local_max = 0.f;
    for (int n = t; n < N; n += T) {
        // x[(n - k) mod N] = x2[n - k + N] for 0 <= k < N
        float y = 0.f;
        for (int k = 0; k < N; ++k) y = fmaf(q[k], x2[n - k + N], y);
        const float xv = x2[n];
        store_env(a, col * N + n, sqrtf(fmaf(xv, xv, y * y)), local_max);
    }
    publish_max(a, local_max);
}

// ---------------------------------------------------------------------------
// Any N up to ENV_CIRC_MAX on the FP32 matrix cores: y = Im x_a of 16 columns
// is a circulant matrix of q times the columns (v_mfma_f32_16x16x4_f32, tiles of
// 16 outputs x 16 columns).  For even N, q is 0 at even distances, so even
// outputs read odd samples only and odd outputs even ones: two products of
// half the size (P = 2 phases of H = N / P outputs).
//
// The direct sum reads two LDS words per FMA and thread and wastes the lanes
// past N; here one word of q and one of x feed 16 FMAs.  us, direct and here:
// 96 x 96 columns of 192 43.7, 13.6; 60 x 70 of 251 34.2, 20.0; 128 x 128 of 300
// 181, 45.
//
// Few columns (less than a workgroup per CU) spread their tiles over several
// workgroups, which then store their outputs from the accumulators; every one
// of them reads whole columns, so an envelope that overwrites its image keeps
// one workgroup per group of columns.
//
// An infinite or NaN sample leaves its column no finite envelope.  At an odd N
// every output reads every sample; at an even N the zeros of q keep a sample out
// of half of the outputs, so there a column with such a sample gets 1e-30 times
// its sum added to all (as with the rounded zeros of a summed q).  Finite columns
// skip the sum: taken for each, its shuffles cost 0.9 us of the 8 to 21 us of
// 96 x 96 columns of 192 and fewer; the test of the bits costs 0.1 us.
//
// LDS: the columns by phase ([16][stride], phase pe at pe H4; stride = 4 modulo
// 64 words, so 16 columns x 4 samples fall in different banks), their
// envelopes (same shape), and q by distance: entry d + H4 + 3 holds the q of
// outputs o and samples m of a phase with d = o - m (+ the phase's shift).
// ---------------------------------------------------------------------------
constexpr int ENV_CIRC_MIN = 24, ENV_CIRC_MAX = 1000;
typedef float env_v4f __attribute__((ext_vector_type(4)));

struct EnvCirc {
    int P, H, H4;         // phases, outputs (= samples) per phase, rounded up to 4
    int tiles;            // 16-output tiles per phase
    int stride;           // words per column
    int nq;               // entries of the q table
};
static EnvCirc env_circ(int n)
{
    EnvCirc c;
    c.P = n % 2 == 0 ? 2 : 1;
    c.H = n / c.P;
    c.H4 = (c.H + 3) & ~3;
    c.tiles = (c.H + 15) / 16;
    c.stride = ((c.P * c.H4 + 63) & ~63) + 4;
    c.nq = c.H4 + 16 * c.tiles + 4;
    return c;
}
static size_t env_circ_lds(const EnvCirc &c) { return ((size_t)2 * 16 * c.stride + c.nq) * sizeof(float); }

__global__ __launch_bounds__(256) void env_circ_kernel(EnvArgs a, EnvCirc c)
{
    extern __shared__ float sf[];
    __shared__ float s_rest[16];
    float *xs = sf, *env = sf + 16 * c.stride, *qs = env + 16 * c.stride;
    const int N = a.N, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long col0 = (long)blockIdx.x * 16;
    const int cols = (int)min(16L, a.n_cols - col0);
    for (int i = threadIdx.x; i < 16 * c.stride; i += 256) xs[i] = 0.f;
    // distance d = i - (H4 + 3) between output o and sample m of a phase's
    // product: q index 2 d + 1 (even N: odd output 2 o + 1, even sample 2 m;
    // the even outputs 2 o and odd samples 2 m + 1 are one step nearer) or d
    for (int i = threadIdx.x; i < c.nq; i += 256) {
        int k = c.P == 2 ? 2 * (i - c.H4 - 3) + 1 : i - c.H4 - 3;
        k %= N;
        qs[i] = a.q[k < 0 ? k + N : k];
    }
    __syncthreads();
    const float *img = a.img + col0 * N;
    float rest = 0.f;            // of column wave + 4 lane, for lanes 0 to 3
    if (c.P == 1) {
        for (int g = wave; g < cols; g += 4)
            for (int n = lane; n < N; n += 64) xs[g * c.stride + n] = img[(long)g * N + n];
    } else {
        unsigned top = 0;        // largest magnitude, as bits
        for (int g = wave; g < cols; g += 4)
            for (int n = lane; n < N; n += 64) {
                const float x = img[(long)g * N + n];
                xs[g * c.stride + (n & 1) * c.H4 + (n >> 1)] = x;
                top = max(top, __float_as_uint(x) & 0x7fffffffu);
            }
        if (__any(top >= 0x7f800000u))
            for (int i = 0; i < 4 && wave + 4 * i < cols; ++i) {
                float sum = 0.f;
                for (int n = lane; n < N; n += 64)
                    sum = fmaf(img[(long)(wave + 4 * i) * N + n], 1e-30f, sum);
                for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
                if (lane == i) rest = sum;
            }
    }
    if (lane < 4) s_rest[wave + 4 * lane] = rest;
    __syncthreads();
    const int col = lane & 15, kq = lane >> 4;
    const int total = c.P * c.tiles;
    rest = s_rest[col];
    float local_max = 0.f;
    for (int t = blockIdx.y * 4 + wave; t < total; t += 4 * gridDim.y) {
        const int ph = t / c.tiles;                         // parity of the outputs (P = 2)
        const int o0 = 16 * (t - ph * c.tiles);
        // row i = col of the operand: q at o0 + i - m, m = 4 s + kq
        const int shift = c.P == 2 && ph == 0 ? 1 : 0;
        const float *qp = qs + (c.H4 + 3) + o0 + col - kq - shift;
        const float *xp = xs + col * c.stride + (c.P == 2 ? (1 - ph) * c.H4 : 0) + kq;
        // four accumulators: independent products, and chains a quarter as
        // long (relative error 6.5e-8 at N = 192, 1.0e-7 of the direct sum)
        env_v4f acc[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        int m = 0;
        for (; m + 16 <= c.H4; m += 16) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(qp[-m - 4 * u], xp[m + 4 * u], acc[u], 0, 0, 0);
        }
        for (; m < c.H4; m += 4)
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(qp[-m], xp[m], acc[0], 0, 0, 0);
        // accumulator: outputs o0 + 4 kq + r of column col
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = o0 + 4 * kq + r;
            if (o >= c.H) continue;
            const int w = col * c.stride + ph * (c.P == 2 ? c.H4 : 0) + o;
            const float x = xs[w], y = ((acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r])) + rest;
            const float e = sqrtf(fmaf(x, x, y * y));
            if (gridDim.y == 1)
                env[w] = e;
            else if (col < cols)
                store_env(a, (col0 + col) * N + c.P * o + (c.P == 2 ? ph : 0), e, local_max);
        }
    }
    if (gridDim.y == 1) {        // whole columns: contiguous stores
        __syncthreads();
        for (int g = wave; g < cols; g += 4)
            for (int n = lane; n < N; n += 64)
                store_env(a, (col0 + g) * N + n,
                          env[g * c.stride + (c.P == 2 ? (n & 1) * c.H4 + (n >> 1) : n)], local_max);
    }
    publish_max(a, local_max);
}

// ---------------------------------------------------------------------------
// Register FFT (N = 64 M = 512 or 1024): sample n = M l + r lives in lane l,
// register r.  X[k1 + 64 k2] = sum_r W_M^{r k2} W_N^{r k1} [sum_l x[M l + r] W_64^{l k1}].
// ---------------------------------------------------------------------------
// Value of lane l ^ m (m a power of two, constant after unrolling).  Lane
// distances 1 and 2 move through DPP quad permutes and 32 through the gfx950
// half-swap (permlane32_swap: lanes 32-63 of the first operand trade places
// with lanes 0-31 of the second), all in the VALU; 4, 8 and 16 go through the
// LDS crossbar (ds_bpermute), so both pipes share the exchanges.
__device__ inline float xor_lane(float x, int m, int lane)
{
    const int xi = __float_as_int(x);
    if (m == 1) return __int_as_float(__builtin_amdgcn_update_dpp(0, xi, 0xB1, 0xF, 0xF, false));
    if (m == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, xi, 0x4E, 0xF, 0xF, false));
    if (m == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
        return __int_as_float(lane < 32 ? r[1] : r[0]);
    }
    return __shfl_xor(x, m, 64);
}

__device__ inline float2 shfl_xor2(float2 v, int m, int lane)
{
    return make_float2(xor_lane(v.x, m, lane), xor_lane(v.y, m, lane));
}

// 64-point DIF across lanes for each register (sign -1: forward); lane l ends
// with the bin bitrev6(l).  Pairs (l, l ^ d): lower l gets v + p, upper gets
// (p - v) W_{2d}^{l mod d}, both as (sigma v + p) w with sigma = +-1 and w = 1
// on the lower lane (no selects).  tw_l[s] = W_{2d}^{l mod d} for every lane.
template <int M>
__device__ inline void lane_dif(float2 (&v)[M], const float2 *tw_l, int lane)
{
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        const int d = 32 >> s;
        const bool up = (lane & d) != 0;
        const float sg = up ? -1.f : 1.f;
        const float2 w = up ? tw_l[s] : make_float2(1.f, 0.f);
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const float2 p = shfl_xor2(v[r], d, lane);
            v[r] = cmul(make_float2(fmaf(sg, v[r].x, p.x), fmaf(sg, v[r].y, p.y)), w);
        }
    }
}

// 64-point inverse DIT across lanes from bit-reversed bins back to natural
// order (sign +1): lower l gets v + W p, upper gets p - W v, W = conj(W_{2d}^{l mod d}).
// The upper lane multiplies its own value by W before the exchange, so both
// results are sigma u + p with u the lane's (weighted) value, sigma = +-1.
template <int M>
__device__ inline void lane_dit_inv(float2 (&v)[M], const float2 *tw_l, int lane)
{
#pragma unroll
    for (int s = 5; s >= 0; --s) {
        const int d = 32 >> s;
        const bool up = (lane & d) != 0;
        const float sg = up ? -1.f : 1.f;
        const float2 w = up ? make_float2(tw_l[s].x, -tw_l[s].y) : make_float2(1.f, 0.f);
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const float2 u = cmul(v[r], w);
            const float2 p = shfl_xor2(u, d, lane);
            v[r] = make_float2(fmaf(sg, u.x, p.x), fmaf(sg, u.y, p.y));
        }
    }
}

// In-register M-point DFT, natural order in and out; sign -1 forward, +1 inverse.
template <int M>
__device__ inline void reg_fft(float2 (&v)[M], const float2 *wm, float sign)
{
    if constexpr (M > 1) {
        // bit-reverse permutation, then iterative DIT
        constexpr int L = M == 2 ? 1 : M == 4 ? 2 : M == 8 ? 3 : 4;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            int j = 0;
#pragma unroll
            for (int b = 0; b < L; ++b) j |= ((i >> b) & 1) << (L - 1 - b);
            if (j > i) {
                const float2 t = v[i];
                v[i] = v[j];
                v[j] = t;
            }
        }
#pragma unroll
        for (int h = 1; h < M; h <<= 1) {
#pragma unroll
            for (int i0 = 0; i0 < M; i0 += 2 * h) {
#pragma unroll
                for (int j = 0; j < h; ++j) {
                    const float2 w0 = wm[j * (M / (2 * h))];
                    const float2 w = make_float2(w0.x, sign < 0.f ? w0.y : -w0.y);
                    const float2 t = cmul(v[i0 + j + h], w);
                    const float2 u = v[i0 + j];
                    v[i0 + j] = make_float2(u.x + t.x, u.y + t.y);
                    v[i0 + j + h] = make_float2(u.x - t.x, u.y - t.y);
                }
            }
        }
    }
}

// Two real columns per wavefront, 8 per 256-thread workgroup.  The Hilbert
// transform H is linear with a real kernel, so for z = x1 + j x2 the inverse
// DFT of -j sgn(k) DFT(z) (sgn = 0 at DC and Nyquist, +1 for positive and -1
// for negative frequencies) is H{x1} + j H{x2}, and each envelope is
// |x_a| = sqrt(x^2 + H{x}^2): the analytic signal of both columns for one
// complex FFT pair (half the work of one pair per column).
template <int M>
__global__ __launch_bounds__(256) void env_fft_reg_kernel(EnvArgs a)
{
    constexpr int N = 64 * M;
    const int lane = threadIdx.x & 63;
    const long col = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 2;
    float local_max = 0.f;
    if (col < a.n_cols) {
        const bool has2 = col + 1 < a.n_cols;
        const float *x = a.img + col * N + M * lane;
        float x1[M], x2[M];
        float2 v[M];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            x1[r] = x[r];
            x2[r] = has2 ? x[N + r] : 0.f;
            v[r] = make_float2(x1[r], x2[r]);
        }
        float2 twl[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) twl[s] = a.tw_lane[s * 64 + lane];
        lane_dif<M>(v, twl, lane);
        // lane holds bin k1 = bitrev6(lane) of each register's 64-point DFT
        const float2 *tm = a.tw_mid + lane * M;
#pragma unroll
        for (int r = 0; r < M; ++r) v[r] = cmul(v[r], tm[r]);
        reg_fft<M>(v, a.wm, -1.f);
        // -j sgn(k) on Z[k1 + 64 k2] (register k2): -j s (a + j b) = s (b - j a)
        const int k1 = (int)(__brev((unsigned)lane) >> 26);
#pragma unroll
        for (int k2 = 0; k2 < M; ++k2) {
            const int k = k1 + 64 * k2;
            const float sg = (k == 0 || 2 * k == N) ? 0.f : (2 * k < N ? 1.f : -1.f);
            v[k2] = make_float2(sg * v[k2].y, -sg * v[k2].x);
        }
        reg_fft<M>(v, a.wm, 1.f);
#pragma unroll
        for (int r = 0; r < M; ++r) v[r] = cmul(v[r], make_float2(tm[r].x, -tm[r].y));
        lane_dit_inv<M>(v, twl, lane);
        const float inv_n = 1.f / (float)N;
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const float h1 = v[r].x * inv_n, h2 = v[r].y * inv_n;
            store_env(a, col * N + M * lane + r,
                      __builtin_amdgcn_sqrtf(fmaf(x1[r], x1[r], h1 * h1)), local_max);
            if (has2)
                store_env(a, (col + 1) * N + M * lane + r,
                          __builtin_amdgcn_sqrtf(fmaf(x2[r], x2[r], h2 * h2)), local_max);
        }
    }
    publish_max(a, local_max);
}

// ---------------------------------------------------------------------------
// Tile FFT (64 <= N <= 256, N = R L, R >= L): sample n = n1 L + n2 lives in
// register n1 of lane n2; L lanes hold one pair of columns, so a wavefront
// holds 64 / L pairs.
//   X[k1 + R k2] = sum_n2 W_L^{n2 k2} [ W_N^{n2 k1} sum_n1 W_R^{n1 k1} x[n1 L + n2] ]
// The inner sum is an R-point FFT inside the lane; after a transposition
// through LDS a lane holds the R / L bins k1 = u L + lane with all their n2,
// and the outer sum is R / L FFTs of L points inside the lane.  The inverse
// retraces the steps.
//
// The 128 x 128 x 256 volume: 17.8 us with a 64-point FFT across the lanes
// (exchanges of every value in each of its 12 stages, about 700 vector
// instructions per pair of columns, VALU-bound), 9.6 us here with about 240 per
// pair (reading and writing the volume takes 6.6 us).  N = 512 and 1024 stay
// with the FFT across the lanes: 32 values per lane unroll to code that a
// wavefront runs once, bound by its instruction fetch (1 x 400 columns of 512
// 15.8 us against 8.4, 64 x 64 17.5 against 13.7).
// ---------------------------------------------------------------------------
// cos(pi k / 16)
__device__ constexpr float COS16[17] = {1.0000000000f, 0.9807852804f, 0.9238795325f, 0.8314696123f, 0.7071067812f, 0.5555702330f, 0.3826834324f, 0.1950903220f, 0.0000000000f, -0.1950903220f, -0.3826834324f, -0.5555702330f, -0.7071067812f, -0.8314696123f, -0.9238795325f, -0.9807852804f, -1.0000000000f};

// v times exp(-+ j 2 pi J / M) (M a power of two up to 32, J < M / 2): forward
// - (INV = false), inverse +.  Quarter and eighth turns without a full product.
template <int M, int J, bool INV>
__device__ inline float2 turn(float2 v)
{
    if constexpr (J == 0) {
        return v;
    } else if constexpr (4 * J == M) {
        return INV ? make_float2(-v.y, v.x) : make_float2(v.y, -v.x);
    } else {
        constexpr int K = 32 / M * J;                       // 16ths of a half turn
        constexpr float c = COS16[K];
        constexpr float s0 = K <= 8 ? COS16[8 - K] : COS16[K - 8];    // sin(pi K / 16)
        constexpr float s = INV ? s0 : -s0;
        if constexpr (8 * J == M || 8 * J == 3 * M) {       // |c| = |s|
            constexpr float h = 0.70710678118654752f;
            const float sum = v.x + v.y, dif = v.x - v.y;
            if constexpr (8 * J == M) return INV ? make_float2(h * dif, h * sum) : make_float2(h * sum, -h * dif);
            return INV ? make_float2(-h * sum, h * dif) : make_float2(-h * dif, -h * sum);
        }
        return make_float2(fmaf(v.x, c, -v.y * s), fmaf(v.x, s, v.y * c));
    }
}

__host__ __device__ constexpr int log2_of(int m) { return m <= 1 ? 0 : 1 + log2_of(m / 2); }
__host__ __device__ constexpr int bit_reverse(int v, int bits)
{
    return bits == 0 ? 0 : ((v & 1) << (bits - 1)) | bit_reverse(v >> 1, bits - 1);
}

// M-point DFT of v[0 .. M): decimation in frequency, natural order in, bin
// bit_reverse(p) in register p out.
template <int M, int J = 0>
__device__ inline void fft_dif(float2 *v)
{
    if constexpr (M > 1) {
        if constexpr (J < M / 2) {
            const float2 a = v[J], b = v[J + M / 2];
            v[J] = make_float2(a.x + b.x, a.y + b.y);
            v[J + M / 2] = turn<M, J, false>(make_float2(a.x - b.x, a.y - b.y));
            fft_dif<M, J + 1>(v);
        } else {
            fft_dif<M / 2>(v);
            fft_dif<M / 2>(v + M / 2);
        }
    }
}
// The inverse (unscaled): bit-reversed bins in, natural order out.
template <int M, int J>
__device__ inline void fft_dit_stage(float2 *v)
{
    if constexpr (J < M / 2) {
        const float2 a = v[J], b = turn<M, J, true>(v[J + M / 2]);
        v[J] = make_float2(a.x + b.x, a.y + b.y);
        v[J + M / 2] = make_float2(a.x - b.x, a.y - b.y);
        fft_dit_stage<M, J + 1>(v);
    }
}
template <int M>
__device__ inline void fft_dit(float2 *v)
{
    if constexpr (M > 1) {
        fft_dit<M / 2>(v);
        fft_dit<M / 2>(v + M / 2);
        fft_dit_stage<M, 0>(v);
    }
}

// Between a wavefront's LDS writes and its other lanes' reads of them: keeps
// the compiler from moving either across (LDS accesses of one wavefront run in
// order, so no instruction is needed).
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Pairs of columns of a wavefront, LDS float2 of a wavefront.
template <int R, int L> struct EnvTile {
    static constexpr int pairs = 64 / L;
    static constexpr int lds = pairs * R * (L + 1);
};

// Two real columns per lane group.  The Hilbert transform H is linear with a
// real kernel, so for z = x1 + j x2 the inverse DFT of -j sgn(k) DFT(z) (sgn =
// 0 at DC and Nyquist, +1 for positive and -1 for negative frequencies) is
// H{x1} + j H{x2}, and each envelope is |x_a| = sqrt(x^2 + H{x}^2): the
// analytic signal of both columns for one complex FFT pair.  A wavefront uses
// its own part of LDS only: no barriers.
// MAX: the maximum alone, nothing is stored.  a.given: ref is the maximum that
// pass left in part_max.
template <int R, int L, bool MAX>
__global__ __launch_bounds__(256) void env_fft_tile_kernel(EnvArgs a)
{
    extern __shared__ float2 sm[];
    constexpr int N = R * L, U = R / L, B = log2_of(R), BL = log2_of(L);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l = lane % L, g = lane / L;
    float2 *buf = sm + wave * EnvTile<R, L>::lds + g * R * (L + 1);
    const long col =
        (((long)blockIdx.x * (blockDim.x >> 6) + wave) * EnvTile<R, L>::pairs + g) * 2;
    const bool has1 = col < a.n_cols, has2 = col + 1 < a.n_cols;
    const float *x = a.img + col * N + l;
    const float2 *tw = a.tw_mid + l;
    float x1[R], x2[R];
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        x1[r] = has1 ? x[r * L] : 0.f;
        x2[r] = has2 ? x[N + r * L] : 0.f;
        v[r] = make_float2(x1[r], x2[r]);
    }
    fft_dif<R>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        constexpr int b = B;
        const int k1 = bit_reverse(r, b);
        buf[k1 * (L + 1) + l] = cmul(v[r], tw[k1 * L]);
    }
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float2 w[L];
        float2 *row = buf + (u * L + l) * (L + 1);
#pragma unroll
        for (int n2 = 0; n2 < L; ++n2) w[n2] = row[n2];
        fft_dif<L>(w);
        // -j sgn(k) on X[k1 + R k2], k1 = u L + l: k is positive for k2 < L / 2,
        // negative above, DC and Nyquist at k1 = 0 of k2 = 0 and L / 2
        const float edge = u == 0 && l == 0 ? 0.f : 1.f;
#pragma unroll
        for (int r = 0; r < L; ++r) {
            const int k2 = bit_reverse(r, BL);
            float2 z = 2 * k2 < L ? make_float2(w[r].y, -w[r].x) : make_float2(-w[r].y, w[r].x);
            if (k2 == 0 || 2 * k2 == L) z = make_float2(edge * z.x, edge * z.y);
            w[r] = z;
        }
        fft_dit<L>(w);
#pragma unroll
        for (int n2 = 0; n2 < L; ++n2) row[n2] = w[n2];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k1 = bit_reverse(r, B);
        const float2 t = tw[k1 * L];
        v[r] = cmul(buf[k1 * (L + 1) + l], make_float2(t.x, -t.y));
    }
    fft_dit<R>(v);
    const float inv_n = 1.f / (float)N;
    float local_max = 0.f;
    if (!MAX && a.given) {
        a.ref = max_of_parts(a);
        a.inv_ref = a.ref > 0.f ? 1.f / a.ref : 0.f;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float h1 = v[r].x * inv_n, h2 = v[r].y * inv_n;
        const float e1 = __builtin_amdgcn_sqrtf(fmaf(x1[r], x1[r], h1 * h1));
        const float e2 = __builtin_amdgcn_sqrtf(fmaf(x2[r], x2[r], h2 * h2));
        if constexpr (MAX) {
            local_max = fmaxf(local_max, fmaxf(e1, e2));     // (columns outside the image are 0)
        } else if (a.given) {
            if (has1) a.out[col * N + r * L + l] = compress_by_max(a, e1);
            if (has2) a.out[(col + 1) * N + r * L + l] = compress_by_max(a, e2);
        } else {
            if (has1) store_env(a, col * N + r * L + l, e1, local_max);
            if (has2) store_env(a, (col + 1) * N + r * L + l, e2, local_max);
        }
    }
    if (!a.given) publish_max(a, local_max);
}

__global__ __launch_bounds__(256) void env_iq_kernel(EnvArgs a)
{
    const long total = a.n_cols * a.N;
    float local_max = 0.f;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const float2 z = reinterpret_cast<const float2 *>(a.img)[i];
        store_env(a, i, sqrtf(fmaf(z.x, z.x, z.y * z.y)), local_max);
    }
    publish_max(a, local_max);
}

// One workgroup: img_max = max of part_max[0 .. n) (fixed order per thread,
// then a tree over threads).
__global__ __launch_bounds__(256) void env_reduce_kernel(const float *part_max, long n,
                                                         float *img_max)
{
    __shared__ float s[256];
    float m = 0.f;
    for (long i = threadIdx.x; i < n; i += 256) m = fmaxf(m, part_max[i]);
    s[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] = fmaxf(s[threadIdx.x], s[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *img_max = s[0];
}

// Compression by the image maximum: reduced by env_reduce_kernel, or, from at
// most ENV_FEW_PARTS partial maxima, by every workgroup for itself (a launch
// less).
__global__ __launch_bounds__(256) void env_compress_kernel(EnvArgs a)
{
    const long total = a.n_cols * a.N;
    const long step = (long)gridDim.x * 256, first = (long)blockIdx.x * 256 + threadIdx.x;
    // the thread's first two groups of four are loaded before the maxima
    constexpr int F = 2;
    float4 *o = reinterpret_cast<float4 *>(a.out);
    const long groups = a.vec ? total / 4 : 0;
    float4 y[F];
#pragma unroll
    for (int u = 0; u < F; ++u)
        y[u] = first + u * step < groups ? o[first + u * step] : make_float4(0.f, 0.f, 0.f, 0.f);
    a.ref = a.n_parts > 0 ? max_of_parts(a) : *a.img_max;
    a.inv_ref = a.ref > 0.f ? 1.f / a.ref : 0.f;
    auto value = [&](float v) { return compress_by_max(a, v); };
    auto put = [&](long i, float4 v) { o[i] = make_float4(value(v.x), value(v.y), value(v.z), value(v.w)); };
#pragma unroll
    for (int u = 0; u < F; ++u)
        if (first + u * step < groups) put(first + u * step, y[u]);
    for (long i = first + F * step; i < groups; i += step) put(i, o[i]);
    if (!a.vec)
        for (long i = first; i < total; i += step) a.out[i] = value(a.out[i]);
}

}  // namespace bf

using namespace bf;

struct bf_env_s {
    uint32_t magic = 0xBFE7E701u;
    long n_cols = 0;
    int N = 0, iq = 0, log2n = -1;
    long n_parts = 0;
    int tile = 0;                 // tile FFT (N = 64, 128, 256)
    int circ = 0;                 // circulant product on the matrix cores
    int split = 1;                // workgroups a group of 16 columns is spread over (out apart from img)
    int waves = 1;                // wavefronts per workgroup of the tile FFT
    int reg_m = 0;                // register FFT: M = N / 64 (N = 512, 1024)
    float2 wm[8] = {};
    float2 *d_tw = nullptr;
    float2 *d_tw_lane = nullptr;  // [6][64]
    float2 *d_tw_mid = nullptr;   // [64][M] or [R][L]
    float *d_q = nullptr;
    float *d_part = nullptr;      // [n_parts] per-workgroup maxima, then the maximum
    ~bf_env_s()
    {
        if (d_tw) (void)hipFree(d_tw);
        if (d_tw_lane) (void)hipFree(d_tw_lane);
        if (d_tw_mid) (void)hipFree(d_tw_mid);
        if (d_q) (void)hipFree(d_q);
        if (d_part) (void)hipFree(d_part);
    }
};

// Lanes per pair of columns of the tile FFT (R = n / L values per lane).
static int env_tile_lanes(int n) { return n <= 128 ? 8 : 16; }

template <int R, int L>
static void launch_tile(const EnvArgs &a, unsigned blocks, int waves, bool max_only, hipStream_t s)
{
    const size_t shm = (size_t)waves * EnvTile<R, L>::lds * sizeof(float2);
    if (max_only)
        hipLaunchKernelGGL((env_fft_tile_kernel<R, L, true>), dim3(blocks), dim3(64 * waves), shm, s, a);
    else
        hipLaunchKernelGGL((env_fft_tile_kernel<R, L, false>), dim3(blocks), dim3(64 * waves), shm, s, a);
}

static void launch_tile_n(const EnvArgs &a, unsigned blocks, int waves, bool max_only, hipStream_t s)
{
    switch (a.N) {
        case 64: launch_tile<8, 8>(a, blocks, waves, max_only, s); break;
        case 128: launch_tile<16, 8>(a, blocks, waves, max_only, s); break;
        default: launch_tile<16, 16>(a, blocks, waves, max_only, s); break;
    }
}

static bool live(bf_env e) { return e && e->magic == 0xBFE7E701u; }

extern "C" {

int bf_env_create(int64_t n_cols, int32_t n, int32_t iq, bf_env *out)
{
    clear_err();
    if (!out) return fail(BF_ERR_NULL, "out is NULL");
    *out = nullptr;
    if (n_cols < 1) return fail(BF_ERR_SHAPE, "n_cols=%lld < 1", (long long)n_cols);
    if (n < 1 || n > ENV_MAX_N) return fail(BF_ERR_SHAPE, "n=%d not in [1,%d]", n, ENV_MAX_N);
    if (iq != 0 && iq != 1) return fail(BF_ERR_UNSUPPORTED, "iq must be 0 or 1");
    if (n_cols >= (int64_t(1) << 31) || n_cols * n * (iq ? 2 : 1) >= (int64_t(1) << 31))
        return fail(BF_ERR_TOO_LARGE, "image exceeds 2^31 elements");
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count < 1) {
        (void)hipGetLastError();
        return fail(BF_ERR_NO_DEVICE, "no HIP device available");
    }
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
        return fail(BF_ERR_HIP, "device query failed");
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(BF_ERR_NO_DEVICE, "device %d is %s, libbf is built for gfx950", dev,
                    prop.gcnArchName);
    bf_env e = new bf_env_s();
    e->n_cols = n_cols;
    e->N = n;
    e->iq = iq;
    // workgroups of the envelope pass: the grid-stride launch of the IQ path,
    // one per column, eight columns each (register FFT), 16 (circulant), or 2 * 64 / L columns per wavefront of the tile FFT (four
    // wavefronts per workgroup, one where that leaves fewer workgroups than CUs)
    if (!iq && (n & (n - 1)) == 0 && n >= 64 && n <= 256) {
        e->tile = 1;
        const long per_wave = 2 * (64 / env_tile_lanes(n));
        const long waves = (n_cols + per_wave - 1) / per_wave;
        e->waves = waves >= 4 * 256 ? 4 : 1;
        e->n_parts = (waves + e->waves - 1) / e->waves;
    } else if (!iq && (n == 512 || n == 1024)) {
        e->reg_m = n / 64;
        e->n_parts = (n_cols + 7) / 8;
    } else {
        e->circ = !iq && (n & (n - 1)) != 0 && n >= ENV_CIRC_MIN && n <= ENV_CIRC_MAX;
        e->n_parts = iq ? std::min<long>((n_cols * n + 1023) / 1024, ENV_FEW_PARTS)
                        : e->circ ? (n_cols + 15) / 16 : n_cols;
        if (e->circ) {
            const EnvCirc c = env_circ(n);
            const long groups = e->n_parts;
            e->split = groups >= 256 ? 1 : (int)std::min<long>((c.P * c.tiles + 3) / 4, 512 / groups);
            e->n_parts = groups * e->split;
        }
    }
    hipError_t err = hipMalloc(&e->d_part, (e->n_parts + 1) * sizeof(float));
    if (err == hipSuccess && !iq) {
        if ((n & (n - 1)) == 0 && n >= 2) {
            int l = 0;
            while ((1 << l) < n) ++l;
            e->log2n = l;
            // stage-major: stage len (h = len / 2) at offset h - 1, pos < h
            std::vector<float2> tw(n - 1);
            for (int h = 1; h < n; h <<= 1)
                for (int pos = 0; pos < h; ++pos) {
                    const double ph = -M_PI * pos / h;      // -2 pi pos / len
                    tw[h - 1 + pos] = make_float2((float)cos(ph), (float)sin(ph));
                }
            err = hipMalloc(&e->d_tw, tw.size() * sizeof(float2));
            if (err == hipSuccess)
                err = hipMemcpy(e->d_tw, tw.data(), tw.size() * sizeof(float2), hipMemcpyHostToDevice);
            if (err == hipSuccess && e->reg_m) {
                const int M = e->reg_m;
                // lane stage twiddles W_{2d}^{l mod d}, d = 32 >> s
                std::vector<float2> tl(6 * 64), tm((size_t)64 * M);
                for (int st = 0; st < 6; ++st) {
                    const int d = 32 >> st;
                    for (int l = 0; l < 64; ++l) {
                        const double ph = -M_PI * (l % d) / d;
                        tl[st * 64 + l] = make_float2((float)cos(ph), (float)sin(ph));
                    }
                }
                // W_N^{r bitrev6(l)}
                for (int l = 0; l < 64; ++l) {
                    int br = 0;
                    for (int b = 0; b < 6; ++b) br |= ((l >> b) & 1) << (5 - b);
                    for (int r = 0; r < M; ++r) {
                        const double ph = -2.0 * M_PI * (double)((long)r * br % n) / n;
                        tm[(size_t)l * M + r] = make_float2((float)cos(ph), (float)sin(ph));
                    }
                }
                for (int j = 0; j < M / 2; ++j) {
                    const double ph = -2.0 * M_PI * j / M;
                    e->wm[j] = make_float2((float)cos(ph), (float)sin(ph));
                }
                err = hipMalloc(&e->d_tw_lane, tl.size() * sizeof(float2));
                if (err == hipSuccess) err = hipMalloc(&e->d_tw_mid, tm.size() * sizeof(float2));
                if (err == hipSuccess)
                    err = hipMemcpy(e->d_tw_lane, tl.data(), tl.size() * sizeof(float2),
                                    hipMemcpyHostToDevice);
                if (err == hipSuccess)
                    err = hipMemcpy(e->d_tw_mid, tm.data(), tm.size() * sizeof(float2),
                                    hipMemcpyHostToDevice);
            }
            if (err == hipSuccess && e->tile) {
                const int L = env_tile_lanes(n), R = n / L;
                std::vector<float2> tm(n);
                for (int l = 0; l < L; ++l)
                    for (int k = 0; k < R; ++k) {
                        const double ph = -2.0 * M_PI * (double)(l * k) / n;
                        tm[(size_t)k * L + l] = make_float2((float)cos(ph), (float)sin(ph));
                    }
                err = hipMalloc(&e->d_tw_mid, tm.size() * sizeof(float2));
                if (err == hipSuccess)
                    err = hipMemcpy(e->d_tw_mid, tm.data(), tm.size() * sizeof(float2),
                                    hipMemcpyHostToDevice);
            }
        } else {
            // q[k] = Im IDFT(h)[k] = (1/N) sum_k' h[k'] sin(2 pi k' k / N)
            std::vector<float> q(n);
            for (int k = 0; k < n; ++k) {
                double s = 0.0;
                // weight 2 for 0 < k' < N/2; DC and Nyquist add sin(0) = sin(pi k) = 0
                for (int kk = 1; 2 * kk < n; ++kk)
                    s += 2.0 * sin(2.0 * M_PI * (double)((long)kk * k % n) / n);
                q[k] = (float)(s / n);
            }
            err = hipMalloc(&e->d_q, n * sizeof(float));
            if (err == hipSuccess)
                err = hipMemcpy(e->d_q, q.data(), n * sizeof(float), hipMemcpyHostToDevice);
        }
    }
    if (err != hipSuccess) {
        delete e;
        return hip_fail(err, "envelope tables");
    }
    *out = e;
    return BF_OK;
}

int bf_env_destroy(bf_env e)
{
    clear_err();
    if (!e) return BF_OK;
    if (!live(e)) return fail(BF_ERR_STATE, "not a live envelope plan");
    (void)hipDeviceSynchronize();
    e->magic = 0;
    delete e;
    return BF_OK;
}

int bf_envelope(bf_env e, const float *img, float *out, int32_t compress, double ref,
                double param, void *stream)
{
    clear_err();
    if (!e) return fail(BF_ERR_NULL, "envelope plan is NULL");
    if (!live(e)) return fail(BF_ERR_STATE, "not a live envelope plan");
    if (!img || !out) return fail(BF_ERR_NULL, "img and out must be non-NULL");
    if (compress < BF_COMPRESS_NONE || compress > BF_COMPRESS_POWER)
        return fail(BF_ERR_UNSUPPORTED, "unknown compression %d", compress);
    if (!isfinite(ref)) return fail(BF_ERR_GEOMETRY, "ref must be finite");
    if (compress != BF_COMPRESS_NONE && !(isfinite(param) && param > 0.0))
        return fail(BF_ERR_GEOMETRY, "param must be finite and > 0");
    EnvArgs a;
    a.img = img;
    a.out = out;
    a.tw = e->d_tw;
    a.tw_lane = e->d_tw_lane;
    a.tw_mid = e->d_tw_mid;
    for (int j = 0; j < 8; ++j) a.wm[j] = e->wm[j];
    a.q = e->d_q;
    a.part_max = e->d_part;
    a.img_max = e->d_part + e->n_parts;
    a.n_cols = e->n_cols;
    a.N = e->N;
    a.log2n = e->log2n;
    a.compress = compress;
    a.ref = (float)ref;
    a.param = (float)param;
    // (a ref below 2^-128 keeps a finite reciprocal: env = 0 still maps to 0)
    a.inv_ref = ref > 0.0 ? (float)std::min(1.0 / ref, 3.4028234663852886e38) : 0.f;
    hipStream_t s = (hipStream_t)stream;
    const bool two_pass = compress != BF_COMPRESS_NONE && ref <= 0.0;
    const long total = e->n_cols * e->N;
    const bool apart = out + total <= img || img + total <= out;
    const int split = apart ? e->split : 1;
    const long n_parts = e->n_parts / e->split * split;      // (split divides n_parts)
    a.n_parts = n_parts <= ENV_FEW_PARTS ? (int)n_parts : 0;
    a.given = 0;
    // From 2^21 points on the tile FFT runs twice, first for the maximum alone,
    // instead of storing the envelope and reading it back: the 128 x 128 x 256
    // volume moves 50 MB instead of 67 (22.5 -> 17.8 us); smaller images are
    // bound by the latency of a pass.
    const bool twice = e->tile && two_pass && a.n_parts > 0 && total >= (1L << 21);
    a.vec = total % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    if (e->iq) {
        hipLaunchKernelGGL(env_iq_kernel, dim3((unsigned)e->n_parts), dim3(256), 0, s, a);
    } else if (e->tile) {
        const unsigned g = (unsigned)e->n_parts;
        launch_tile_n(a, g, e->waves, twice, s);
        if (twice) {
            a.given = 1;
            launch_tile_n(a, g, e->waves, false, s);
        }
    } else if (e->reg_m) {
        const dim3 g((unsigned)e->n_parts), b(256);
        if (e->reg_m == 8)
            hipLaunchKernelGGL(env_fft_reg_kernel<8>, g, b, 0, s, a);
        else
            hipLaunchKernelGGL(env_fft_reg_kernel<16>, g, b, 0, s, a);
    } else if (e->log2n > 0) {
        const int T = std::min(256, std::max(64, e->N / 2));
        hipLaunchKernelGGL(env_fft_kernel, dim3((unsigned)e->n_cols), dim3(T),
                           (size_t)e->N * 8, s, a);
    } else if (e->circ) {
        const EnvCirc c = env_circ(e->N);
        const size_t shm = env_circ_lds(c);
        if (shm > 65536) {
            const hipError_t he = hipFuncSetAttribute(reinterpret_cast<const void *>(&env_circ_kernel),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
            if (he != hipSuccess) return hip_fail(he, "envelope LDS size");
        }
        hipLaunchKernelGGL(env_circ_kernel, dim3((unsigned)(n_parts / split), split), dim3(256),
                           shm, s, a, c);
    } else {
        hipLaunchKernelGGL(env_direct_kernel, dim3((unsigned)e->n_cols), dim3(256),
                           (size_t)3 * e->N * sizeof(float), s, a);
    }
    if (two_pass && !twice) {
        if (a.n_parts == 0)
            hipLaunchKernelGGL(env_reduce_kernel, dim3(1), dim3(256), 0, s, e->d_part, n_parts,
                               e->d_part + e->n_parts);
        const long items = a.vec ? total / 4 : total;
        const unsigned eblocks = (unsigned)std::min<long>((items + 511) / 512, 2048);
        hipLaunchKernelGGL(env_compress_kernel, dim3(eblocks), dim3(256), 0, s, a);
    }
    hipError_t err = hipGetLastError();
    return err == hipSuccess ? BF_OK : hip_fail(err, "envelope launch");
}

}  // extern "C"
