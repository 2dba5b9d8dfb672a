// Unit-wise natural gradient for BatchNorm (Sec. 4.2, Eq. 15-17).
//   bn_reduce_kernel: per-sample gradients of gamma/beta from dy and xhat ([N, C, HW]):
//     pure streaming, HBM-bound.
//   bn_unit_kernel: the 2x2 Fisher block (3 unique numbers) of a channel from the [N, C] per-sample gradients
//     (coalesced over channels), folded into the running average, and the closed-form 2x2 inverse applied to the
//     mean gradient.  Latency bound (a few MB): 64 channels per workgroup, its four wavefronts take a quarter of
//     the samples each.
#include "kfac_internal.h"

namespace kfac {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// NCHW: a row is the plane of one (sample, channel).  HBM bound (8 bytes per position); what kept it from the rate of a
// plain read (5.3 of 6.2 TB/s over ResNet-50's 53 layers) were wavefronts that lived for one short row: the job search and
// twelve dependent shuffles around a single load.  So a workgroup takes bn_rows(HW) rows:
//   HW <= 128        they are one contiguous block of at most 4096 elements, loaded in 16-byte pieces whatever the row
//                    length, multiplied, and summed per row out of LDS (256 / rows threads each);
//   128 < HW <= 256  four rows per wavefront, all loads ahead of the sums;
//   else             one row per wavefront, 1024 positions in flight.
// Loads need element alignment only.
typedef float bn_vec4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void bn_add4(float &sg, float &sb, const bn_vec4 &a, const bn_vec4 &b)
{
    sg += (a[0] * b[0] + a[1] * b[1]) + (a[2] * b[2] + a[3] * b[3]);
    sb += (a[0] + a[1]) + (a[2] + a[3]);
}

__global__ __launch_bounds__(256) void bn_reduce_kernel(const BnReduceJob *__restrict__ jobs, int n_jobs, int N)
{
    __shared__ __attribute__((aligned(16))) float block[2][4096];
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const BnReduceJob J = jobs[lo];
    const int HW = J.HW, R = bn_rows(HW), tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long rows = (long long)N * J.C, row0 = (long long)(wg - J.wg_start) * R;
    const int here = (int)(rows - row0 < R ? rows - row0 : R);        // rows of this workgroup
    const bn_vec4 zero = {0.f, 0.f, 0.f, 0.f};
    if (HW <= 128) {
        const Global<const float> dy = global(J.dy) + row0 * HW, xh = global(J.xhat) + row0 * HW;
        const int total = here * HW;                                  // <= 4096
        bn_vec4 a[4], b[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e = 4 * (tid + 256 * g);
            a[g] = b[g] = zero;
            if (e + 4 <= total) {
                a[g] = __builtin_nontemporal_load((Global<const bn_vec4>)(dy + e));
                b[g] = __builtin_nontemporal_load((Global<const bn_vec4>)(xh + e));
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (e + q < total) { a[g][q] = dy[e + q]; b[g][q] = xh[e + q]; }
            }
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e = 4 * (tid + 256 * g);
            *(floatx4 *)(block[0] + e) = (floatx4)(a[g] * b[g]);
            *(floatx4 *)(block[1] + e) = (floatx4)a[g];
        }
        __syncthreads();
        // T threads per row; row r starts r steps into its round, so that the banks differ where HW is even
        const int T = 256 / R, r = tid / T, j = tid & (T - 1), K = (HW + T - 1) / T;
        float sg = 0.f, sb = 0.f;
        if (r < here) {
            int k = r % K;
            for (int q = 0; q < K; ++q) {
                const int e = j + T * k;
                if (e < HW) { sg += block[0][r * HW + e]; sb += block[1][r * HW + e]; }
                k = k + 1 == K ? 0 : k + 1;
            }
        }
        for (int o = T >> 1; o > 0; o >>= 1) { sg += __shfl_xor(sg, o, 64); sb += __shfl_xor(sb, o, 64); }
        if (r < here && j == 0) {
            global(J.g_gamma)[row0 + r] = sg;
            global(J.g_beta)[row0 + r] = sb;
        }
        return;
    }
    const int per_wave = R >> 2;                                      // 4 (HW <= 256) or 1
    const int first = wave * per_wave;
    if (first >= here) return;
    const int n4 = HW & ~3;
    if (per_wave == 4) {
        const Global<const float> dy = global(J.dy) + (row0 + first) * HW, xh = global(J.xhat) + (row0 + first) * HW;
        bn_vec4 a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = b[q] = zero;
            if (first + q < here && 4 * lane < n4) {
                a[q] = __builtin_nontemporal_load((Global<const bn_vec4>)(dy + q * HW + 4 * lane));
                b[q] = __builtin_nontemporal_load((Global<const bn_vec4>)(xh + q * HW + 4 * lane));
            }
        }
        float sg[4] = {0.f, 0.f, 0.f, 0.f}, sb[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (first + q < here && n4 + lane < HW) {                 // the last HW % 4 positions
                sb[q] = dy[q * HW + n4 + lane];
                sg[q] = sb[q] * xh[q * HW + n4 + lane];
            }
            bn_add4(sg[q], sb[q], a[q], b[q]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int q = 0; q < 4; ++q) { sg[q] += __shfl_xor(sg[q], off, 64); sb[q] += __shfl_xor(sb[q], off, 64); }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (lane == 0 && first + q < here) {
                global(J.g_gamma)[row0 + first + q] = sg[q];
                global(J.g_beta)[row0 + first + q] = sb[q];
            }
        return;
    }
    const long long row = row0 + first;
    const Global<const float> dy = global(J.dy) + row * HW, xh = global(J.xhat) + row * HW;
    float sg = 0.f, sb = 0.f;
    for (int t = 4 * lane; t < n4; t += 1024) {
        bn_vec4 a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = b[q] = zero;
            if (t + 256 * q < n4) {
                a[q] = __builtin_nontemporal_load((Global<const bn_vec4>)(dy + t + 256 * q));
                b[q] = __builtin_nontemporal_load((Global<const bn_vec4>)(xh + t + 256 * q));
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) bn_add4(sg, sb, a[q], b[q]);
    }
    if (n4 + lane < HW) {
        const float a = dy[n4 + lane];
        sg += a * xh[n4 + lane];
        sb += a;
    }
    sg = wave_sum(sg);
    sb = wave_sum(sb);
    if (lane == 0) {
        global(J.g_gamma)[row] = sg;
        global(J.g_beta)[row] = sb;
    }
}

// The same from NHWC tensors ([N, HW, C]): a workgroup takes 64 channels of one sample, lanes along the channels
// (16 lanes x 16 bytes per position when C % 4 == 0, else 64 lanes x 4 bytes), 16 (4) positions at a time; the
// partial sums of the threads that share a channel are added through LDS in a fixed order.
__global__ __launch_bounds__(256) void bn_reduce_nhwc_kernel(const BnReduceJob *__restrict__ jobs, int n_jobs, int N)
{
    __shared__ float red[2][16][64];
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const BnReduceJob J = jobs[lo];
    const int chunks = (J.C + 63) / 64;
    const int local = wg - J.wg_start;
    const int n = local / chunks, c0 = (local - n * chunks) * 64;
    const Global<const float> dy = global(J.dy) + (long long)n * J.HW * J.C;
    const Global<const float> xh = global(J.xhat) + (long long)n * J.HW * J.C;
    const bool vec = ((J.C & 3) == 0) && ((((uintptr_t)J.dy | (uintptr_t)J.xhat) & 15) == 0);
    const int tid = threadIdx.x;
    if (vec) {
        const int c = c0 + 4 * (tid & 15), part = tid >> 4;   // 16 parts
        floatx4 sg = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
        if (c < J.C)
            for (int t = part; t < J.HW; t += 16) {
                const floatx4 a = *(Global<const floatx4>)(dy + (long long)t * J.C + c);
                const floatx4 b = *(Global<const floatx4>)(xh + (long long)t * J.C + c);
                sg += a * b;
                sb += a;
            }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            red[0][part][4 * (tid & 15) + e] = sg[e];
            red[1][part][4 * (tid & 15) + e] = sb[e];
        }
    } else {
        const int c = c0 + (tid & 63), part = tid >> 6;       // 4 parts
        float sg = 0.f, sb = 0.f;
        if (c < J.C)
            for (int t = part; t < J.HW; t += 4) {
                const float a = dy[(long long)t * J.C + c];
                sg += a * xh[(long long)t * J.C + c];
                sb += a;
            }
        red[0][part][tid & 63] = sg;
        red[1][part][tid & 63] = sb;
    }
    __syncthreads();
    if (tid < 128) {
        const int which = tid >> 6, cl = tid & 63;
        const int parts = vec ? 16 : 4;
        float sum = 0.f;
        for (int q = 0; q < parts; ++q) sum += red[which][q][cl];
        if (c0 + cl < J.C) global(which ? J.g_beta : J.g_gamma)[(long long)n * J.C + c0 + cl] = sum;
    }
}

__global__ __launch_bounds__(256) void bn_unit_kernel(const BnJob *__restrict__ jobs, int n_jobs, int N,
                                                      float decay, float lambda)
{
    __shared__ float red[4][5][64];
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const BnJob J = jobs[lo];
    const int ch = threadIdx.x & 63, part = threadIdx.x >> 6, i = (wg - J.wg_start) * 64 + ch;
    float a = 0.f, b = 0.f, d = 0.f, mg = 0.f, mb = 0.f;
    if (i < J.C) {
#pragma unroll 8
        for (int n = part; n < N; n += 4) {
            const float gg = global(J.g_gamma)[(long long)n * J.C + i];
            const float gb = global(J.g_beta)[(long long)n * J.C + i];
            a = fmaf(gg, gg, a); b = fmaf(gg, gb, b); d = fmaf(gb, gb, d);
            mg += gg; mb += gb;
        }
    }
    red[part][0][ch] = a; red[part][1][ch] = b; red[part][2][ch] = d; red[part][3][ch] = mg; red[part][4][ch] = mb;
    __syncthreads();
    if (part || i >= J.C) return;
    auto sum = [&](int k) { return (red[0][k][ch] + red[1][k][ch]) + (red[2][k][ch] + red[3][k][ch]); };
    a = sum(0); b = sum(1); d = sum(2); mg = sum(3); mb = sum(4);
    const float inv_n = 1.0f / (float)N;
    a *= inv_n; b *= inv_n; d *= inv_n; mg *= inv_n; mb *= inv_n;
    const Global<float> F = global(J.F_ema) + (long long)3 * i;
    float f0 = (1.0f - decay) * a, f1 = (1.0f - decay) * b, f2 = (1.0f - decay) * d;
    if (decay != 0.0f) { f0 += decay * F[0]; f1 += decay * F[1]; f2 += decay * F[2]; }
    F[0] = f0; F[1] = f1; F[2] = f2;
    // (F + lambda I)^-1 [mg, mb]^T with [[a,b],[c,d]]^-1 = 1/(ad - bc) [[d,-b],[-c,a]]
    const float fa = f0 + lambda, fd = f2 + lambda;
    const float det = fa * fd - f1 * f1;
    global(J.out_gamma)[i] = (fd * mg - f1 * mb) / det;
    global(J.out_beta)[i] = (fa * mb - f1 * mg) / det;
}

hipError_t launch_bn(const BnJob *jobs_dev, int n_jobs, int total_wgs, int N, float decay, float lambda,
                     hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    bn_unit_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs, N, decay, lambda);
    return hipGetLastError();
}

hipError_t launch_bn_reduce(const BnReduceJob *jobs_dev, int n_jobs, int total_wgs, int N, int nhwc, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    if (nhwc) bn_reduce_nhwc_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs, N);
    else      bn_reduce_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs, N);
    return hipGetLastError();
}

}  // namespace kfac
