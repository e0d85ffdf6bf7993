// bf_adjoint.hip -- adjoint of DAS and the image-sharpness loss.
//
// DAS is linear in the decoded data e for a fixed sound speed c, so its
// adjoint scatters dL/d(out) back along the same delays and interpolation
// weights.  The sound speed enters only through the delay:
//   s = (tof - t0) fs,  tof = path / c   =>   ds/dc = -tof fs / c
// and the apodization does not depend on c, so
//   dL/dc = sum_p G(p) sum_ij a(p,i,j) v'_ij(s) ds/dc.
// The cubic Hermite read has a continuous derivative (Sec. IV-B), which is
// what makes this gradient usable for sound-speed autofocus.
#include "bf_common.h"

namespace bf {

// One (point, trace) term of the adjoint.  ga = G(p) * a(p,i,j).
// Adds ga * w_k(t) to grad_e taps (if GE) and returns a * v'(s) (if GC).
template <int ET, int IP, bool GE, bool GC>
__device__ inline float adjoint_term(const void *tr, float *ge, int S, int nB, float s, float ga,
                                     float a_w)
{
    if constexpr (IP == IN_NEAREST) {
        if constexpr (GE) {
            const int n = nB + (int)floorf(s + 0.5f);
            if ((unsigned)n < (unsigned)S) atomicAdd(ge + n, ga);
        }
        return 0.f;
    } else {
        const float fl = floorf(s);
        const float t = s - fl;
        const int n = nB + (int)fl;
        float d = 0.f;
        if constexpr (IP == IN_LINEAR) {
            if constexpr (GC) {
                const float p0 = ((unsigned)n < (unsigned)S) ? load_e<ET>(tr, n) : 0.f;
                const float p1 = ((unsigned)(n + 1) < (unsigned)S) ? load_e<ET>(tr, n + 1) : 0.f;
                d = a_w * (p1 - p0);
            }
            if constexpr (GE) {
                if ((unsigned)n < (unsigned)S) atomicAdd(ge + n, ga * (1.f - t));
                if ((unsigned)(n + 1) < (unsigned)S) atomicAdd(ge + n + 1, ga * t);
            }
        } else {
            if constexpr (GC) {
                const float pm = ((unsigned)(n - 1) < (unsigned)S) ? load_e<ET>(tr, n - 1) : 0.f;
                const float p0 = ((unsigned)n < (unsigned)S) ? load_e<ET>(tr, n) : 0.f;
                const float p1 = ((unsigned)(n + 1) < (unsigned)S) ? load_e<ET>(tr, n + 1) : 0.f;
                const float p2 = ((unsigned)(n + 2) < (unsigned)S) ? load_e<ET>(tr, n + 2) : 0.f;
                const float c1 = 0.5f * (p1 - pm);
                const float c2 = pm - 2.5f * p0 + 2.0f * p1 - 0.5f * p2;
                const float c3 = 0.5f * (p2 - pm) + 1.5f * (p0 - p1);
                d = a_w * fmaf(t, fmaf(2.f, c2, 3.f * t * c3), c1);
            }
            if constexpr (GE) {
                const float t2 = t * t, t3 = t2 * t;
                const float w[4] = {-0.5f * t + t2 - 0.5f * t3, 1.f - 2.5f * t2 + 1.5f * t3,
                                    0.5f * t + 2.f * t2 - 1.5f * t3, -0.5f * t2 + 0.5f * t3};
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((unsigned)(n - 1 + q) < (unsigned)S) atomicAdd(ge + n - 1 + q, ga * w[q]);
            }
        }
        return d;
    }
}

// Per lane: returns sum_ij a v'(s) ds/dc (if GC); scatters into grad_e (if GE).
template <int MODE, int ET, int IP, bool GE, bool GC>
__device__ inline float adjoint_point(const DasArgs &a, const Lane &L, float G)
{
    const float kf = (float)a.k;
    const float kc = (float)(a.k / a.c);     // d/dc of (path * fs / c) = -path * k / c
    const bool live = L.active && (GC || G != 0.f);
    float acc = 0.f;
    const float xr = rx_coord<MODE>(L.x, L.y);
    for (int j = 0; j < a.n_ch; ++j) {
        const float cj = a.rx_c[j];
        if constexpr (MODE != MODE_HERCULES) {
            // separable modes: transmit path z + Et, receive path z + Er
            const float dxr = xr - cj;
            const float r2 = dxr * dxr;
            const bool act = live && r2 < L.thr;
            if (!__any(act)) continue;
            const float Er = excess(r2, L.z, L.z2);
            const float Rj = fmaf(Er, kf, L.fB);
            const float aj = act ? hann_u2(r2 * L.wsc) : 0.f;
            for (int i = 0; i < a.n_tx; ++i) {
                if (act) {
                    const float Et = tx_excess<MODE>(a, L.x, L.z, L.z2, i);
                    const float s = fmaf(Et, kf, Rj);
                    const long trace = (long)i * a.n_ch + j;
                    const float d = adjoint_term<ET, IP, GE, GC>(
                        trace_ptr<ET>(a.e, trace, a.S), a.grad_e + trace * a.S, a.S, L.nB, s,
                        G * aj, aj);
                    if constexpr (GC) acc = fmaf(d, -(2.f * L.z + Er + Et) * kc, acc);
                }
            }
        } else {
            const float dy = L.y - cj;
            const float dy2 = dy * dy;
            if (!__any(live && dy2 < L.thr)) continue;
            for (int i = 0; i < a.n_tx; ++i) {
                const float dx = L.x - a.tx_x[i];
                const float rho2 = fmaf(dx, dx, dy2);
                const bool act = live && rho2 < L.thr;
                if (!__any(act)) continue;
                if (act) {
                    const float E = excess(rho2, L.z, L.z2);
                    const float s = fmaf(E, kf, L.fB);
                    const float w = hann_u2(rho2 * L.wsc);
                    const long trace = (long)i * a.n_ch + j;
                    const float d = adjoint_term<ET, IP, GE, GC>(
                        trace_ptr<ET>(a.e, trace, a.S), a.grad_e + trace * a.S, a.S, L.nB, s,
                        G * w, w);
                    // path = transmit path of the point (plane or diverging) + z + E
                    if constexpr (GC) acc = fmaf(d, -(L.ptx + L.z + E) * kc, acc);
                }
            }
        }
    }
    return acc;
}

// grid: ceil(n_waves / 4) blocks of 256; writes one FP64 partial of
// sum_p G(p) dout(p)/dc per block (deterministic order).
template <int MODE, int ET, int IP, bool GE, bool GC>
__global__ __launch_bounds__(256) void das_adjoint_kernel(DasArgs a)
{
    __shared__ double red[4];
    const int wave_id = blockIdx.x * 4 + (threadIdx.x >> 6);
    double contrib = 0.0;
    if (wave_id < a.n_waves) {
        const Lane L = lane_setup(a, wave_id, threadIdx.x & 63);
        const float G = L.active ? a.grad_out[L.out_idx] : 0.f;
        const float d = adjoint_point<MODE, ET, IP, GE, GC>(a, L, G);
        contrib = (double)G * (double)d;
    }
    if constexpr (GC) {
        for (int off = 32; off > 0; off >>= 1) contrib += __shfl_down(contrib, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = contrib;
        __syncthreads();
        if (threadIdx.x == 0) a.partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// Sum of the per-block partials in a fixed order -> grad_c.
// out[b] = sum of partial[b * n .. b * n + n) in a fixed order (one
// workgroup per frame b).
__global__ __launch_bounds__(256) void reduce_partials_kernel(const double *partial, int n,
                                                             float *out)
{
    __shared__ double red[256];
    partial += (long)blockIdx.x * n;
    out += blockIdx.x;
    double s = 0.0;
    for (int q = threadIdx.x; q < n; q += 256) s += partial[q];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = (float)red[0];
}

hipError_t launch_reduce_partials(const double *partial, int n, float *out, hipStream_t s,
                                  int n_frames)
{
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(n_frames), dim3(256), 0, s, partial, n, out);
    return hipGetLastError();
}

__global__ void fill_kernel(float *p, long n, float v)
{
    for (long q = (long)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (long)gridDim.x * blockDim.x)
        p[q] = v;
}

template <int MODE, int ET, int IP>
static hipError_t launch_adj3(const DasArgs &a, bool ge, bool gc, hipStream_t s)
{
    dim3 grid((a.n_waves + 3) / 4);
    if (ge && gc)
        hipLaunchKernelGGL((das_adjoint_kernel<MODE, ET, IP, true, true>), grid, dim3(256), 0, s, a);
    else if (ge)
        hipLaunchKernelGGL((das_adjoint_kernel<MODE, ET, IP, true, false>), grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((das_adjoint_kernel<MODE, ET, IP, false, true>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int MODE, int ET>
static hipError_t launch_adj2(const DasArgs &a, int ip, bool ge, bool gc, hipStream_t s)
{
    switch (ip) {
        case IN_NEAREST: return launch_adj3<MODE, ET, IN_NEAREST>(a, ge, gc, s);
        case IN_LINEAR: return launch_adj3<MODE, ET, IN_LINEAR>(a, ge, gc, s);
        case IN_CUBIC: return launch_adj3<MODE, ET, IN_CUBIC>(a, ge, gc, s);
        default: return hipErrorInvalidValue;
    }
}

template <int MODE>
static hipError_t launch_adj1(const DasArgs &a, int et, int ip, bool ge, bool gc, hipStream_t s)
{
    switch (et) {
        case ET_F32: return launch_adj2<MODE, ET_F32>(a, ip, ge, gc, s);
        case ET_BF16: return launch_adj2<MODE, ET_BF16>(a, ip, ge, gc, s);
        case ET_I32: return launch_adj2<MODE, ET_I32>(a, ip, ge, gc, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fill(float *p, long n, float v, hipStream_t s)
{
    long blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_das_adjoint(const DasArgs &a, int mode, int et, int ip, float *grad_c,
                              hipStream_t s)
{
    const bool ge = a.grad_e != nullptr, gc = grad_c != nullptr;
    if (!ge && !gc) return hipSuccess;
    hipError_t err;
    if (ge) {
        err = launch_fill(a.grad_e, (long)a.n_tx * a.n_ch * a.S, 0.f, s);
        if (err != hipSuccess) return err;
    }
    switch (mode) {
        case MODE_FORCES: err = launch_adj1<MODE_FORCES>(a, et, ip, ge, gc, s); break;
        case MODE_HERCULES: err = launch_adj1<MODE_HERCULES>(a, et, ip, ge, gc, s); break;
        case MODE_TPW: err = launch_adj1<MODE_TPW>(a, et, ip, ge, gc, s); break;
        case MODE_VLS: err = launch_adj1<MODE_VLS>(a, et, ip, ge, gc, s); break;
        default: return hipErrorInvalidValue;
    }
    if (err != hipSuccess || !gc) return err;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(256), 0, s, a.partial,
                       (a.n_waves + 3) / 4, grad_c);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Sharpness: L = -sum I^4 / (sum I^2)^2 per image, FP64 sums in a fixed order,
// then dL/dI in a second sweep.
//
// One workgroup per image is bound by the latency of its loads: it keeps eight
// 16-byte loads per thread in flight (eight 256 x 256 images 32 -> 9.3 us;
// one load in flight before).  From SHARP_SPLIT points on an image is spread
// over workgroups of SHARP_CHUNK points in three launches: the chunks' sums go
// to the head of the image's gradient (which is written last, by the third
// launch), so no scratch memory is needed; without a gradient to write, one
// workgroup sums the image (48 x 48 x 96 points: 98 -> 14.5 us with the split;
// one workgroup 18.7 us at 131 071 points, 9.1 at 65 536).
// ---------------------------------------------------------------------------
constexpr int SHARP_CHUNK = 8192;            // points per workgroup of a split image
constexpr long SHARP_SPLIT = 131072;

// Adds the fourth and second powers of img[beg .. end) to the thread's sums.
template <int T>
__device__ inline void sharp_sums(const float *img, long beg, long end, double &P, double &Q)
{
    auto add = [&](float v) {
        const double x = v, x2 = x * x;
        Q += x2;
        P += x2 * x2;
    };
    long q = beg;
    if ((reinterpret_cast<uintptr_t>(img + beg) & 15) == 0) {
        for (; q + 32L * T <= end; q += 32L * T) {
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = *reinterpret_cast<const float4 *>(img + q + 4L * (u * T + threadIdx.x));
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                add(v[u].x); add(v[u].y); add(v[u].z); add(v[u].w);
            }
        }
    }
    for (; q + 8L * T <= end; q += 8L * T) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = img[q + u * T + threadIdx.x];
#pragma unroll
        for (int u = 0; u < 8; ++u) add(v[u]);
    }
    for (q += threadIdx.x; q < end; q += T) add(img[q]);
}

// Sums of the workgroup in a fixed order, to every thread.
template <int T>
__device__ inline void sharp_total(double &P, double &Q)
{
    __shared__ double s[2][T / 64];
    for (int o = 32; o > 0; o >>= 1) {
        P += __shfl_down(P, o, 64);
        Q += __shfl_down(Q, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s[0][threadIdx.x >> 6] = P;
        s[1][threadIdx.x >> 6] = Q;
    }
    __syncthreads();
    P = Q = 0.0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
        P += s[0][w];
        Q += s[1][w];
    }
}

// Gradient of img[beg .. end) from the image's sums.
template <int T>
__device__ inline void sharp_grad(const float *img, float *grad, long beg, long end, double P, double Q)
{
    const double a = (Q > 0.0) ? -4.0 / (Q * Q) : 0.0;
    const double b = (Q > 0.0) ? 4.0 * P / (Q * Q * Q) : 0.0;
    auto slope = [&](float v) {
        const double x = v;
        return (float)(a * x * x * x + b * x);
    };
    long q = beg;
    if (((reinterpret_cast<uintptr_t>(img + beg) | reinterpret_cast<uintptr_t>(grad + beg)) & 15) == 0) {
        for (; q + 16L * T <= end; q += 16L * T) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v[u] = *reinterpret_cast<const float4 *>(img + q + 4L * (u * T + threadIdx.x));
#pragma unroll
            for (int u = 0; u < 4; ++u)
                *reinterpret_cast<float4 *>(grad + q + 4L * (u * T + threadIdx.x)) =
                    make_float4(slope(v[u].x), slope(v[u].y), slope(v[u].z), slope(v[u].w));
        }
    }
    for (q += threadIdx.x; q < end; q += T) grad[q] = slope(img[q]);
}

__device__ inline float sharp_loss(double P, double Q) { return (Q > 0.0) ? (float)(-P / (Q * Q)) : 0.f; }

__global__ __launch_bounds__(1024) void sharpness_kernel(const float *img, long n, float *loss,
                                                         float *grad)
{
    const float *I = img + (long)blockIdx.x * n;
    double P = 0.0, Q = 0.0;
    sharp_sums<1024>(I, 0, n, P, Q);
    sharp_total<1024>(P, Q);
    if (threadIdx.x == 0) loss[blockIdx.x] = sharp_loss(P, Q);
    if (grad) sharp_grad<1024>(I, grad + (long)blockIdx.x * n, 0, n, P, Q);
}

// Split image, launch 1: sums of chunk blockIdx.x of image blockIdx.y as four
// words at the head of the image's gradient.
__global__ __launch_bounds__(256) void sharp_part_kernel(const float *img, long n, float *grad)
{
    const long beg = (long)blockIdx.x * SHARP_CHUNK;
    double P = 0.0, Q = 0.0;
    sharp_sums<256>(img + (long)blockIdx.y * n, beg, min(beg + SHARP_CHUNK, n), P, Q);
    sharp_total<256>(P, Q);
    if (threadIdx.x == 0) {
        uint32_t *w = reinterpret_cast<uint32_t *>(grad + (long)blockIdx.y * n) + 4 * blockIdx.x;
        const uint64_t p = __double_as_longlong(P), q = __double_as_longlong(Q);
        w[0] = (uint32_t)p; w[1] = (uint32_t)(p >> 32);
        w[2] = (uint32_t)q; w[3] = (uint32_t)(q >> 32);
    }
}

// The image's sums from the chunks' words.
__device__ inline void sharp_read_parts(const float *grad, int chunks, double &P, double &Q)
{
    const uint32_t *w = reinterpret_cast<const uint32_t *>(grad);
    P = Q = 0.0;
    for (int k = threadIdx.x; k < chunks; k += 256) {
        P += __longlong_as_double((uint64_t)w[4 * k] | ((uint64_t)w[4 * k + 1] << 32));
        Q += __longlong_as_double((uint64_t)w[4 * k + 2] | ((uint64_t)w[4 * k + 3] << 32));
    }
    sharp_total<256>(P, Q);
}

// Launch 2 (head = 0): the gradient past the chunks' words, chunk by chunk.
// Launch 3 (head = 1, one workgroup per image): the loss, and the gradient
// over the words once every thread has read them.
__global__ __launch_bounds__(256) void sharp_grad_kernel(const float *img, long n, int chunks,
                                                         float *loss, float *grad, int head)
{
    const float *I = img + (long)blockIdx.y * n;
    float *g = grad + (long)blockIdx.y * n;
    double P, Q;
    sharp_read_parts(g, chunks, P, Q);
    if (head) {
        __syncthreads();
        if (threadIdx.x == 0) loss[blockIdx.y] = sharp_loss(P, Q);
        sharp_grad<256>(I, g, 0, 4L * chunks, P, Q);
    } else {
        const long beg = (long)blockIdx.x * SHARP_CHUNK;
        sharp_grad<256>(I, g, max(beg, 4L * chunks), min(beg + SHARP_CHUNK, n), P, Q);
    }
}

hipError_t launch_sharpness(const float *img, long n, int n_images, float *loss, float *grad,
                            hipStream_t s)
{
    // (a gradient over the image itself leaves no room for the chunks' words;
    // grid.y is at most 65535)
    const long chunks = (n + SHARP_CHUNK - 1) / SHARP_CHUNK, total = n * n_images;
    const bool apart = grad && (grad + total <= img || img + total <= grad);
    if (apart && n >= SHARP_SPLIT && n_images <= 65535) {
        hipLaunchKernelGGL(sharp_part_kernel, dim3((unsigned)chunks, n_images), dim3(256), 0, s, img, n,
                           grad);
        hipLaunchKernelGGL(sharp_grad_kernel, dim3((unsigned)chunks, n_images), dim3(256), 0, s, img, n,
                           (int)chunks, loss, grad, 0);
        hipLaunchKernelGGL(sharp_grad_kernel, dim3(1, n_images), dim3(256), 0, s, img, n, (int)chunks,
                           loss, grad, 1);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(sharpness_kernel, dim3(n_images), dim3(1024), 0, s, img, n, loss, grad);
    return hipGetLastError();
}

}  // namespace bf
