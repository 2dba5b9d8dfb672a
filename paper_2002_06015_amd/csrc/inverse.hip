// Kernels of the damped inversion (Sec. 3.3, Eq. 12) other than the GEMMs:
//   - trace_kernel:  pi^2 = (tr A / dA) / (tr G / dG) and the two damping values per layer;
//   - copy_damp_kernel: dst = src + damp * I (start of the blocked inversion), optionally with the
//     bias border of an A factor eliminated on the way (Schur complement), and border_kernel,
//     which puts the border back into the finished inverse;
//   - leaf_block_kernel: (X + damp I)^-1 for n <= 288 by a blocked symmetric sweep held in the
//     registers of one 1024-thread workgroup, block products on the matrix cores (one matrix per
//     workgroup, many matrices per launch).
#include "kfac_internal.h"


namespace kfac {

// ------------------------------------------------------------------ trace / pi / damping
__global__ __launch_bounds__(256) void trace_kernel(const TraceJob *__restrict__ jobs, float gamma,
                                                    float *__restrict__ damp, float *__restrict__ pi_out)
{
    __shared__ double red[2][256];
    const TraceJob J = jobs[blockIdx.x];
    double sa = 0.0, sg = 0.0;
    for (int i = threadIdx.x; i < J.dA; i += 256) sa += (double)J.A[(long long)i * J.dA + i];
    for (int i = threadIdx.x; i < J.dG; i += 256) sg += (double)J.G[(long long)i * J.dG + i];
    red[0][threadIdx.x] = sa;
    red[1][threadIdx.x] = sg;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double trA = red[0][0], trG = red[1][0];
        double pi = 1.0;
        if (trA > 0.0 && trG > 0.0) pi = sqrt((trA / J.dA) / (trG / J.dG));
        damp[3 * J.idx + 0] = (float)pi;
        damp[3 * J.idx + 1] = (float)(pi * (double)gamma);   // added to A
        damp[3 * J.idx + 2] = (float)((double)gamma / pi);   // added to G
        if (pi_out) pi_out[J.idx] = (float)pi;
    }
}

hipError_t launch_trace(const TraceJob *jobs_dev, int n_layers, float gamma, float *damp_dev,
                        float *pi_out, hipStream_t s)
{
    if (n_layers <= 0) return hipSuccess;
    trace_kernel<<<dim3(n_layers), dim3(256), 0, s>>>(jobs_dev, gamma, damp_dev, pi_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ dst = src + damp I
// Bandwidth bound.  The recursion reads the lower triangle of a source only, except inside the diagonal blocks that are
// inverted as leaves: a row is copied up to kLeafMax columns past the diagonal (ResNet-50's factors: 232 -> 153 us).
constexpr int COPY_ROWS = 8;

__global__ __launch_bounds__(256) void copy_damp_kernel(const CopyJob *__restrict__ jobs, int n_jobs,
                                                        const float *__restrict__ damp)
{
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const CopyJob J = jobs[lo];
    const float d = (J.damp_idx >= 0) ? damp[J.damp_idx] : 0.f;
    const int r0 = (wg - J.wg_start) * COPY_ROWS;
    const float *last = J.src + (long long)J.n * J.lds;   // the border row u^T, c (if any)
    const float ic = J.border ? 1.f / (last[J.n] + d) : 0.f;
    const int r1 = min(J.n, r0 + COPY_ROWS);
    // four adjacent columns per thread (16-byte accesses that only need element alignment: the
    // leading dimensions are odd for bordered factors), all rows of the workgroup in flight at once
    typedef float vec4 __attribute__((ext_vector_type(4), aligned(4)));
    const int n4 = min(J.n & ~3, (r1 + kLeafMax + 3) & ~3);
    for (int c = 4 * (int)threadIdx.x; c < n4; c += 1024) {
        vec4 v[COPY_ROWS];
#pragma unroll
        for (int q = 0; q < COPY_ROWS; ++q)
            if (r0 + q < r1) v[q] = *(const vec4 *)(J.src + (long long)(r0 + q) * J.lds + c);
        vec4 u = {0.f, 0.f, 0.f, 0.f};
        if (J.border) u = *(const vec4 *)(last + c);
#pragma unroll
        for (int q = 0; q < COPY_ROWS; ++q) {
            const int r = r0 + q;
            if (r >= r1) break;
            vec4 x = v[q];
            if (r >= c && r < c + 4) x[r - c] += d;
            if (J.border) {
                const float ur = last[r] * ic;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = fmaf(-ur, u[e], x[e]);
            }
            *(vec4 *)(J.dst + (long long)r * J.ldd + c) = x;
        }
    }
    for (int r = r0; r < r1; ++r) {
        const float ur = J.border ? last[r] * ic : 0.f;
        for (int c = n4 + (int)threadIdx.x; c < min(J.n, n4 + 4); c += 256) {
            float v = J.src[(long long)r * J.lds + c];
            if (r == c) v += d;
            if (J.border) v = fmaf(-ur, last[c], v);
            J.dst[(long long)r * J.ldd + c] = v;
        }
    }
}

hipError_t launch_copy_damp(const CopyJob *jobs_dev, int n_jobs, int total_wgs, const float *damp_dev,
                            hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    copy_damp_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs, damp_dev);
    return hipGetLastError();
}

// ------------------------------------------------------------------ border of a bordered inverse
__global__ __launch_bounds__(256) void border_kernel(const BorderJob *__restrict__ jobs, int n_jobs, int pass,
                                                     const float *__restrict__ damp, int32_t *__restrict__ info)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (pass == 0) {
        // one wavefront per row i: w_i = sum_j X[i][j] u_j
        const int wg = blockIdx.x;
        int lo = 0, hi = n_jobs;
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
        }
        const BorderJob J = jobs[lo];
        const int i = (wg - J.wg_start) * 4 + wave;
        if (i >= J.n) return;
        const float *u = J.src + (long long)J.n * J.lds;
        const float *x = J.X + (long long)i * J.ldx;
        // 16-byte accesses that only need element alignment (the leading dimensions are odd)
        typedef float vec4 __attribute__((ext_vector_type(4), aligned(4)));
        float a4[4] = {0.f, 0.f, 0.f, 0.f};
        const int n4 = J.n & ~3;
        for (int j = 4 * lane; j < n4; j += 256) {
            const vec4 xv = *(const vec4 *)(x + j), uv = *(const vec4 *)(u + j);
#pragma unroll
            for (int e = 0; e < 4; ++e) a4[e] = fmaf(xv[e], uv[e], a4[e]);
        }
        float acc = (a4[0] + a4[1]) + (a4[2] + a4[3]);
        for (int j = n4 + lane; j < J.n; j += 64) acc = fmaf(x[j], u[j], acc);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (lane == 0) {
            const float c = u[J.n] + ((J.damp_idx >= 0) ? damp[J.damp_idx] : 0.f);
            const float v = -acc / c;
            J.X[(long long)i * J.ldx + J.n] = v;
            J.X[(long long)J.n * J.ldx + i] = v;
        }
        return;
    }
    // corner: X[n][n] = (1 - sum_i u_i X[n][i]) / c   (X[n][i] = -w_i / c from pass 0)
    __shared__ float red[4];
    const BorderJob J = jobs[blockIdx.x];
    const float *u = J.src + (long long)J.n * J.lds;
    const float *xr = J.X + (long long)J.n * J.ldx;
    float acc = 0.f;
    for (int i = threadIdx.x; i < J.n; i += 256) acc = fmaf(u[i], xr[i], acc);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float c = u[J.n] + ((J.damp_idx >= 0) ? damp[J.damp_idx] : 0.f);
        const float q = (red[0] + red[1]) + (red[2] + red[3]);
        J.X[(long long)J.n * J.ldx + J.n] = (1.f - q) / c;
        if (!(c > 0.f) && info && J.info_idx >= 0) atomicCAS(&info[J.info_idx], 0, J.n + 1);
    }
}

hipError_t launch_border(const BorderJob *jobs_dev, int n_jobs, int total_wgs, int pass, const float *damp_dev,
                         int32_t *info, hipStream_t s)
{
    if (n_jobs <= 0) return hipSuccess;
    border_kernel<<<dim3(pass == 0 ? total_wgs : n_jobs), dim3(256), 0, s>>>(jobs_dev, n_jobs, pass, damp_dev, info);
    return hipGetLastError();
}

__global__ void zero_i32_kernel(int32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_zero_i32(int32_t *p, int n, hipStream_t s)
{
    if (n <= 0 || !p) return hipSuccess;
    zero_i32_kernel<<<dim3((n + 255) / 256), dim3(256), 0, s>>>(p, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------ blocked leaf inverse on the matrix cores
// (X + damp I)^-1 for n <= 288 by one 1024-thread workgroup, as a symmetric block sweep with 32x32 blocks.  The matrix
// is first scaled to unit diagonal (s_i = 1/sqrt(x_ii), undone at the end), which makes every pivot of the elimination
// lie in (0, 1].  The workgroup holds N = -(scaled matrix), one 32x32 tile per unordered pair of block indices, in the
// accumulator layout of the 32x32 matrix instructions in the registers of one wavefront.  Sweeping block k
// (D = (-N_kk)^-1; R_i = N_ik, the column panel):
//     P_i   = R_i D             ->  new N_ik
//     N_ij += P_i R_j^T         (i, j != k)
//     N_kk  = D
// After all blocks N = X^-1 (the usual sweep operator, written for -X so that every update is an accumulation).
//
// The kernel is a latency chain on one compute unit: 9 dependent blocks for n = 288.  What it does about that:
//   - One wavefront (the chain wavefront) holds no tile.  In step k it takes R_{k+1} and the diagonal tile of block
//     k + 1 as the previous step left them, forms P_{k+1}, brings that tile up to date and sweeps it, all out of its own
//     registers, while the other fifteen do the rest of step k.  D of the next block is ready when they are.
//   - The tiles are dealt out as stars: a wavefront's tiles (at most three) share one block index v, so it needs one
//     P_v only and forms it itself.  It forms the transpose, D R_v^T: its accumulator layout (lane: row of block v,
//     registers: k) is, split into planes, the operand layout of the update R_j P_v^T, with the contraction index in the
//     order the registers have.  Every operand uses that order; P never goes through LDS and one barrier per step is left.
//   - A tile is (registers: row of block j, lanes: row of block v).  For the panel of step k a tile with j = k is stored
//     as the fragments its readers load (three planes, 16 bytes a lane: form F), a tile with v = k as [k][row] rows that
//     are read with the transposing LDS read (form T); no 2-byte stores.  The panels of two steps alternate.
// n = 288: 49 us (77 us with two barriers per step, P and R through LDS and the sweep between the products of its
// wavefront); 224: 33 (51), 160: 20.5 (31), 64: 8.5 (15).  In-kernel times at n = 288, cycles a block: the chain 8800 to 9700
// (sweep 3500 alone on its SIMD, 6000 to 7300 beside the others; D into planes 900, operand reads 300, P and update 1300), the
// other wavefronts up to 10900, most of it the 192 matrix instructions of a SIMD (6100) and the conversions around them.
// Loads and stores: 6 us.
//
// Products are in the three-plane mode (x = h + m + l exactly, see split_pair; six bf16 matrix instructions per
// 16-wide step, fp32 accumulation).
typedef float lb_floatx16 __attribute__((ext_vector_type(16)));
typedef float lb_floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 lb_bf16x8 __attribute__((ext_vector_type(8)));
typedef short lb_shortx4 __attribute__((ext_vector_type(4)));
typedef short lb_shortx8 __attribute__((ext_vector_type(8)));
typedef lb_shortx4 __attribute__((address_space(3))) *lb_lds_shortx4_ptr;
constexpr int LB_MAXT = 9;
constexpr int LB_CHAIN = 15;                            // the chain wavefront
constexpr int LB_TROW = 72;                             // bytes per k row of form T (32 bf16 + 8 bytes: spreads the banks)
constexpr int LB_BLK = 32 * LB_TROW;                    // bytes of one plane of one panel block (form F needs 2048)
constexpr int LB_IDENT = LB_MAXT;                       // a panel block that always holds the identity, form F
constexpr int LB_PLANE = (LB_MAXT + 1) * LB_BLK;        // bytes of one plane of a panel
constexpr int LB_PANEL = 3 * LB_PLANE;                  // one panel: [plane][block]
constexpr int LB_DP = 3 * 2048;                         // planes of D, form F
constexpr int LB_LDS_D = 2 * LB_PANEL, LB_LDS_DIAG = LB_LDS_D + 2 * LB_DP,
              LB_LDS_SC = LB_LDS_DIAG + 2 * 4096, LB_LDS_BYTES = LB_LDS_SC + 32 * LB_MAXT * 4;
static_assert(LB_LDS_BYTES <= 160 * 1024 - 64, "one compute unit's LDS");
static_assert(LB_LDS_D >= 15 * 32 * 33 * 4, "the staging tiles of the final store fit into the panels");

// Tiles of 6 .. 9 blocks dealt to the wavefronts as stars {v; j, j, j} (-1: none), found by a search that minimises the
// matrix instructions of the busiest SIMD (wavefront % 4, the chain's included) summed over the steps, with v = k + 1 for
// the tile of blocks k + 1 and k (the chain reads form F only).  Up to 5 blocks: one tile per wavefront, v the larger index.
__constant__ signed char kLeafStar[4][15][4] = {
    {{2, 1, 4, -1}, {3, 5, 1, -1}, {1, 1, 0, -1}, {5, 4, -1, -1}, {5, 5, 0, -1}, {4, 4, 3, -1}, {2, 2, 0, -1},
     {4, 0, -1, -1}, {3, 3, 2, -1}, {0, 0, 3, -1}, {1, 5, 4, -1}, {2, 5, -1, -1}, {-1, -1, -1, -1}, {-1, -1, -1,
     -1}, {-1, -1, -1, -1}},
    {{5, 2, 3, -1}, {0, 0, 6, -1}, {4, 0, 1, -1}, {3, 0, 1, -1}, {6, 1, 4, -1}, {3, 3, 2, -1}, {6, 5, 3, -1},
     {4, 4, 3, -1}, {2, 0, 1, -1}, {5, 5, 4, -1}, {1, 1, 5, -1}, {2, 2, 4, -1}, {5, 0, -1, -1}, {1, 0, -1, -1},
     {6, 6, 2, -1}},
    {{4, 4, 0, 6}, {6, 0, 1, -1}, {7, 3, 0, -1}, {3, 6, 2, -1}, {0, 0, 5, 2}, {5, 5, 7, 2}, {1, 7, 0, -1}, {2,
     2, 6, 7}, {6, 6, 5, -1}, {1, 1, 5, -1}, {5, 4, 3, -1}, {7, 7, 6, -1}, {2, 4, 1, -1}, {4, 3, 7, 1}, {3, 3,
     1, 0}},
    {{4, 4, 3, 0}, {1, 1, 0, 3}, {6, 6, 0, 4}, {2, 4, 0, 7}, {1, 6, 7, 4}, {8, 0, 7, 2}, {7, 0, 3, 4}, {0, 0, 3,
     5}, {8, 8, 6, 1}, {2, 2, 5, 1}, {7, 7, 6, 5}, {8, 5, 3, 4}, {5, 5, 4, 1}, {6, 5, 2, 3}, {3, 3, 2, 5}},
};
// bit i of [blocks - 6][k]: the tile of blocks i and k is held with v = i (panel form F in step k), else with v = k (T)
__constant__ unsigned short kLeafForm[4][9] = {
    {0x36, 0xc, 0x8, 0x11, 0x26, 0xe, 0x0, 0x0, 0x0},
    {0x3e, 0x5c, 0x68, 0x70, 0x64, 0x42, 0x1, 0x0, 0x0},
    {0xda, 0x5c, 0x29, 0xb0, 0x24, 0x43, 0x9c, 0x36, 0x0},
    {0x1d6, 0x124, 0x148, 0x1d3, 0x1e6, 0x1cd, 0x182, 0x106, 0x0},
};

__device__ __forceinline__ float lb_readlane(float x, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

struct LbFrag { lb_bf16x8 h, m, l; };

// eight accumulator registers (8 u .. 8 u + 7) of a tile as an operand fragment of step u
__device__ __forceinline__ LbFrag lb_split8(const lb_floatx16 &t, int u)
{
    uint4 h, m, l;
    split_pair(t[8 * u + 0], t[8 * u + 1], h.x, m.x, l.x);
    split_pair(t[8 * u + 2], t[8 * u + 3], h.y, m.y, l.y);
    split_pair(t[8 * u + 4], t[8 * u + 5], h.z, m.z, l.z);
    split_pair(t[8 * u + 6], t[8 * u + 7], h.w, m.w, l.w);
    return {__builtin_bit_cast(lb_bf16x8, h), __builtin_bit_cast(lb_bf16x8, m), __builtin_bit_cast(lb_bf16x8, l)};
}
__device__ __forceinline__ void lb_mma(lb_floatx16 &acc, const LbFrag &a, const LbFrag &b)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, acc, 0, 0, 0);
}
// form F: fragments as they are read, plane stride given; [u][lane] 16 bytes each
__device__ __forceinline__ LbFrag lb_read_f(const char *blk, int plane, int u, int lane)
{
    auto rd = [&](int q) { return __builtin_bit_cast(lb_bf16x8, *(const lb_shortx8 *)(blk + q * plane + u * 1024 + lane * 16)); };
    return {rd(0), rd(1), rd(2)};
}
__device__ __forceinline__ void lb_store_f(char *blk, int plane, int u, const LbFrag &f, int lane)
{
    *(lb_shortx8 *)(blk + u * 1024 + lane * 16) = __builtin_bit_cast(lb_shortx8, f.h);
    *(lb_shortx8 *)(blk + plane + u * 1024 + lane * 16) = __builtin_bit_cast(lb_shortx8, f.m);
    *(lb_shortx8 *)(blk + 2 * plane + u * 1024 + lane * 16) = __builtin_bit_cast(lb_shortx8, f.l);
}
// form T: [k][row]; the tile's lanes are k and its registers rows.  The transposing read gives lane i of 16 element i % 4
// of the 8-byte groups addressed by lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12: four adjacent k of row i.
__device__ __forceinline__ LbFrag lb_read_t(const char *blk, int u, int lane)
{
    const int i = lane & 15, row0 = lane & 16, half = lane >> 5;
    const char *p = blk + (16 * u + 4 * half + (i >> 2)) * LB_TROW + 2 * (row0 + 4 * (i & 3));
    auto rd = [&](int q) {
        const lb_shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lb_lds_shortx4_ptr)(p + q * LB_PLANE));
        const lb_shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lb_lds_shortx4_ptr)(p + q * LB_PLANE + 8 * LB_TROW));
        return __builtin_bit_cast(lb_bf16x8, lb_shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    };
    return {rd(0), rd(1), rd(2)};
}
__device__ __forceinline__ void lb_store_t(char *blk, const lb_floatx16 &t, int lane)
{
    char *d = blk + (lane & 31) * LB_TROW + 8 * (lane >> 5);
#pragma unroll
    for (int g = 0; g < 4; ++g) {   // rows 8 g + 4 half .. + 3
        uint2 h, m, l;
        split_pair(t[4 * g], t[4 * g + 1], h.x, m.x, l.x);
        split_pair(t[4 * g + 2], t[4 * g + 3], h.y, m.y, l.y);
        *(uint2 *)(d + 16 * g) = h;
        *(uint2 *)(d + LB_PLANE + 16 * g) = m;
        *(uint2 *)(d + 2 * LB_PLANE + 16 * g) = l;
    }
}
// both fragments of panel block i
__device__ __forceinline__ void lb_read_panel(LbFrag (&f)[2], const char *panel, int i, bool form_f, int lane)
{
    const char *blk = panel + i * LB_BLK;
    if (form_f) {
        f[0] = lb_read_f(blk, LB_PLANE, 0, lane);
        f[1] = lb_read_f(blk, LB_PLANE, 1, lane);
    } else {
        f[0] = lb_read_t(blk, 0, lane);
        f[1] = lb_read_t(blk, 1, lane);
    }
}

// The chain wavefront keeps the diagonal tile in an order that puts consecutive pivots 2 m, 2 m + 1 into the two half-waves
// of one accumulator register: tile row (and column) 8 g + 4 h + e holds row 8 g + 2 e + h of the block.
__device__ __forceinline__ int lb_row(int q, int h) { return 8 * (q >> 2) + 2 * (q & 3) + h; }              // of register q
__device__ __forceinline__ int lb_row_of(int r) { return (r & 24) | ((r & 3) << 1) | ((r >> 2) & 1); }       // of tile row r
__device__ __forceinline__ int lb_tile_row(int m) { return (m & 24) | ((m & 1) << 2) | ((m >> 1) & 3); }     // its inverse
// register q of that order -> the accumulator layout of the plain order (rows only): registers 4 g + e and 4 g + e + 2
// exchange half-waves (swap(x, y): upper half of x with the lower half of y)
__device__ __forceinline__ lb_floatx16 lb_plain_rows(const lb_floatx16 &t)
{
    lb_floatx16 o;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[4 * g + e]), __float_as_uint(t[4 * g + e + 2]), false, false);
            o[4 * g + 2 * e] = __uint_as_float(s[0]);
            o[4 * g + 2 * e + 1] = __uint_as_float(s[1]);
        }
    return o;
}

// Scalar sweep of a 32x32 diagonal tile N (symmetric, negative definite, unit-diagonal scale) inside one wavefront, on the
// matrix core, two pivots per instruction: register v holds both pivot rows, one in each half-wave, and a half-wave is one
// k slot of the fp32 instruction, which takes its pivot's rank-1 update.  The pivots are eliminated one after the other:
// with x0, x1 their rows in the tile as it stands and a = x0[0], b = x0[1] = x1[0], c = x1[1] (index: the pivot),
//     q0 = -1 / a,  u0 = x0 with 1 + a at the first pivot,
//     d1 = c + q0 b b (the second pivot after the first one),  q1 = -1 / d1,
//     u1 = (x1 with 1 + c at the second pivot) + q0 b u0,
// and N += q0 u0 u0^T + q1 u1 u1^T.  That adds the two terms of the elimination, leaves the rows and columns of the pivots
// as those of the swept tile and their block as Q - 2 I, Q = -[[a, b], [b, c]]^-1.  (Pivots lie in [-1, 0): the patches are
// sums of equal-signed terms.)  No later pivot reads the block (pivot q reads row q only, and adds to it), so the 2 is put
// back once, at the end.
// u1 has to be formed before it is used: it is small where the rows are nearly parallel (neighbouring taps of a patch), so
// that q1 = O(1 / d1) meets a small vector only.  Solving the pair by its determinant and adding terms in the full rows is
// the same in exact arithmetic and one reciprocal shorter, but its rounding errors are 2^-24 / d1 instead of 2^-24: pairs
// correlated by 0.9995 (0.99995) came out 12 (150) times less accurate, and by 0.99999 as not positive definite.
// What bounds it is the issue of one wavefront, 28 vector instructions for two pivots.  The chain from one pair to the next
// (two dependent reciprocals) does not go through the matrix instruction of its own pair: the next rows are brought up to
// date with fmas from the tile as it was before.  The products in one fp32 instruction (64 cycles) are exact; as eight bf16
// terms of their planes (32 cycles, 14 instructions to make them) they cost 23.6 us at n = 160 instead of 22.8.
// On return the tile is (-N)^-1.  Returns the 1-based index of the first non-positive pivot of -N, or 0.
__device__ __forceinline__ int leaf_chain_sweep(lb_floatx16 &t, int lane)
{
    const int z = (lane & 31) - 4 * (lane >> 5);
    const bool h = lane >= 32;
    float pa[16], pd[16], worst = -1.f;             // the pivots
    float x = t[0];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int p = 8 * (v >> 2) + (v & 3);       // tile row of the first pivot; the second one is p + 4
        const float a = lb_readlane(x, p), b = lb_readlane(x, p + 4), c = lb_readlane(x, p + 36);
        const float q0 = -__builtin_amdgcn_rcpf(a), m = q0 * b;
        const float d1 = fmaf(m, b, c), q1 = -__builtin_amdgcn_rcpf(d1);
        const float y = z == p ? x + 1.f : x;
        // both patched rows in both half-waves (swap(x, y) exchanges the upper half of x with the lower half of y)
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
        const float u0 = __uint_as_float(s[0]), u1 = fmaf(m, u0, __uint_as_float(s[1]));
        const float fb = h ? u1 : u0;
        const float fa = (h ? q1 : q0) * fb;
        float next = 0.f;
        if (v + 1 < 16) {
            const int q = 8 * ((v + 1) >> 2) + ((v + 1) & 3);
            const float n0 = fmaf(lb_readlane(fa, q + 32), u1, fmaf(lb_readlane(fa, q), u0, t[v + 1]));
            const float n1 = fmaf(lb_readlane(fa, q + 36), u1, fmaf(lb_readlane(fa, q + 4), u0, t[v + 1]));
            next = h ? n1 : n0;
        }
        pa[v] = a;
        pd[v] = d1;
        worst = fmaxf(fmaxf(worst, a), d1);
        t = __builtin_amdgcn_mfma_f32_32x32x2f32(fa, fb, t, 0, 0, 0);
        x = next;
    }
    // register v holds the diagonal element of its lane where z is 8 (v / 4) + v % 4
#pragma unroll
    for (int v = 0; v < 16; ++v) t[v] += z == 8 * (v >> 2) + (v & 3) ? 2.f : 0.f;
    // (a NaN anywhere has reached the last pivot)
    if (__builtin_amdgcn_readfirstlane((int)(worst < 0.f && pd[15] < 0.f))) return 0;
    int first = 0;
#pragma unroll
    for (int v = 15; v >= 0; --v) first = !(pa[v] < 0.f) ? 2 * v + 1 : !(pd[v] < 0.f) ? 2 * v + 2 : first;
    return first;
}

template <int NSLOT>
__global__ __launch_bounds__(1024) void leaf_block_kernel(const LeafJob *__restrict__ jobs,
                                                          const float *__restrict__ damp,
                                                          int32_t *__restrict__ info)
{
    extern __shared__ __attribute__((aligned(16))) char lb_lds[];
    float *sc = (float *)(lb_lds + LB_LDS_SC);       // [32 T] diagonal scaling

    const LeafJob J = jobs[blockIdx.x];
    const int n = J.n;
    const int T = (n + 31) >> 5;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32_ = lane & 31, h_ = lane >> 5;
    const float d = (J.damp_idx >= 0) ? damp[J.damp_idx] : 0.f;
    const unsigned lds = (unsigned)J.lds, ldd = (unsigned)J.ldd;

    // my tiles: (rows of block j[s]: registers, rows of block v: lanes)
    int v_ = -1, j_[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) j_[s] = -1;
    if (NSLOT == 1 || T < 6) {
        int r = 0;
        while ((r + 1) * (r + 2) / 2 <= w) ++r;
        if (w < T * (T + 1) / 2 && w != LB_CHAIN) { v_ = r; j_[0] = w - r * (r + 1) / 2; }
    } else if (w != LB_CHAIN) {
        v_ = kLeafStar[T - 6][w][0];
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) j_[s] = kLeafStar[T - 6][w][1 + s];
    }
    // bit i: the panel block i of step k is in form F
    auto form_mask = [&](int k) { return (NSLOT == 1 || T < 6) ? ~((2u << k) - 1u) : (unsigned)kLeafForm[T - 6][k]; };

    // the chain wavefront loads the first diagonal tile, the others their tiles; the scaling needs the diagonal
    auto load_tile = [&](lb_floatx16 &t, int bi, int bj, bool chain) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int i = 32 * bi + (chain ? lb_row(q, h_) : 8 * (q >> 2) + 4 * h_ + (q & 3)), j = 32 * bj + (chain ? lb_row_of(l32_) : l32_);
            t[q] = J.src[(unsigned)min(i, n - 1) * lds + (unsigned)min(j, n - 1)];   // (outside: replaced when it is scaled)
        }
    };
    // scales of the tile's rows (by register) and of its lane's column
    auto tile_scales = [&](float (&si)[16], float &sj, int bi, int bj, bool chain) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (chain) {
#pragma unroll
                for (int e = 0; e < 4; ++e) si[4 * g + e] = sc[32 * bi + 8 * g + 2 * e + h_];
            } else {
                const lb_floatx4 x = *(const lb_floatx4 *)(sc + 32 * bi + 8 * g + 4 * h_);
#pragma unroll
                for (int e = 0; e < 4; ++e) si[4 * g + e] = x[e];
            }
        }
        sj = sc[32 * bj + (chain ? lb_row_of(l32_) : l32_)];
    };
    auto whole = [&](int bi, int bj) { return 32 * (max(bi, bj) + 1) <= n; };
    auto scale_tile = [&](lb_floatx16 &t, int bi, int bj, bool chain) {
        float si[16], sj;
        tile_scales(si, sj, bi, bj, chain);
        const float dd = bi == bj ? d : 0.f;
        // (the diagonal lies at the same registers and lanes in either order)
#pragma unroll
        for (int q = 0; q < 16; ++q) t[q] = -(t[q] + (8 * (q >> 2) + 4 * h_ + (q & 3) == l32_ ? dd : 0.f)) * si[q] * sj;
        if (!whole(bi, bj)) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int i = 32 * bi + (chain ? lb_row(q, h_) : 8 * (q >> 2) + 4 * h_ + (q & 3)), j = 32 * bj + (chain ? lb_row_of(l32_) : l32_);
                t[q] = (i < n && j < n) ? t[q] : (i == j ? -1.f : 0.f);     // identity padding (of -X)
            }
        }
    };
    auto scales = [&]() {
        if (tid < 32 * T) {
            float v = 1.f;
            if (tid < n) {
                const float a = J.src[(unsigned)tid * lds + (unsigned)tid] + d;
                v = a > 0.f ? rsqrtf(a) : 1.f;   // a non-positive diagonal shows up as a non-positive pivot
            }
            sc[tid] = v;
        }
    };

    // The two roles run loops of their own with the same barriers: one after the scales, one per step, one at the end.
    if (w == LB_CHAIN) {
        lb_floatx16 t;
        load_tile(t, 0, 0, true);
        __syncthreads();
        scale_tile(t, 0, 0, true);
        __builtin_amdgcn_s_setprio(3);
        int bad = 0;
        for (int k = 0; k < T; ++k) {
            // t: the diagonal tile of block k, up to date
            int l64 = lane;
            asm volatile("" : "+v"(l64));
            const int b = leaf_chain_sweep(t, l64);
            if (bad == 0 && b != 0) bad = 32 * k + b;
            char *Dq = lb_lds + LB_LDS_D + (k & 1) * LB_DP;
            {
                const lb_floatx16 dt = lb_plain_rows(t);       // lanes (D is symmetric: its rows) in the chain's order yet
                const int at = (l64 & 32) | lb_row_of(l64 & 31);
                lb_store_f(Dq, 2048, 0, lb_split8(dt, 0), at);
                lb_store_f(Dq, 2048, 1, lb_split8(dt, 1), at);
            }
            __syncthreads();   // D and panel of step k, diagonal tile of block k + 1
            if (k + 1 == T) break;
            // rows of R in the chain's order (lanes), its columns and D in the plain one
            const char *blk = lb_lds + (k & 1) * LB_PANEL + (k + 1) * LB_BLK;
            const int from = (l64 & 32) | lb_row_of(l64 & 31);
            const LbFrag r[2] = {lb_read_f(blk, LB_PLANE, 0, from), lb_read_f(blk, LB_PLANE, 1, from)};
            const LbFrag d0 = lb_read_f(Dq, 2048, 0, l64), d1 = lb_read_f(Dq, 2048, 1, l64);
            const lb_floatx4 *o = (const lb_floatx4 *)(lb_lds + LB_LDS_DIAG + ((k + 1) & 1) * 4096);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const lb_floatx4 x = o[g * 64 + l64];
#pragma unroll
                for (int e = 0; e < 4; ++e) t[4 * g + e] = x[e];
            }
            lb_floatx16 p;
#pragma unroll
            for (int q = 0; q < 16; ++q) p[q] = 0.f;
            lb_mma(p, d0, r[0]);      // P^T = D R^T
            lb_mma(p, d1, r[1]);
            lb_mma(t, r[0], lb_split8(p, 0));
            lb_mma(t, r[1], lb_split8(p, 1));
        }
        if (bad != 0 && lane == 0 && info && J.info_idx >= 0) atomicCAS(&info[J.info_idx], 0, J.pivot_base + bad);
        __syncthreads();
        return;
    }

    lb_floatx16 acc[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s)
        if (j_[s] >= 0) load_tile(acc[s], j_[s], v_, false);
    scales();
    if (w < 12) {   // the identity: wavefront w writes step fragments w % 2 of plane (w / 2) % 3 of panel w / 6
        const int u = w & 1, q = (w >> 1) % 3;
        lb_shortx8 e;
#pragma unroll
        for (int x = 0; x < 8; ++x) e[x] = (q == 0 && 16 * u + 8 * (x >> 2) + 4 * h_ + (x & 3) == l32_) ? (short)0x3F80 : (short)0;
        *(lb_shortx8 *)(lb_lds + (w / 6) * LB_PANEL + q * LB_PLANE + LB_IDENT * LB_BLK + u * 1024 + lane * 16) = e;
    }
    __syncthreads();
    // panel of step kk from the tiles that have an index kk, and the diagonal tile of block kk + 1 for the chain
    auto publish = [&](int kk, int l64) {
        char *panel = lb_lds + (kk & 1) * LB_PANEL;
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) {
            const int j = j_[s];
            if (j < 0) continue;
            if (v_ == kk && j != kk) lb_store_t(panel + j * LB_BLK, acc[s], l64);
            else if (j == kk && v_ != kk) {
                lb_store_f(panel + v_ * LB_BLK, LB_PLANE, 0, lb_split8(acc[s], 0), l64);
                lb_store_f(panel + v_ * LB_BLK, LB_PLANE, 1, lb_split8(acc[s], 1), l64);
            }
            if (j == v_ && v_ == kk + 1) {
                // in the chain's order: row 8 g + 4 half + e is its register 4 g + 2 half + e / 2 of half-wave e % 2
                float *o = (float *)(lb_lds + LB_LDS_DIAG + ((kk + 1) & 1) * 4096) + 4 * lb_tile_row(l64 & 31) + 2 * (l64 >> 5);
#pragma unroll
                for (int q = 0; q < 16; ++q) o[(q >> 2) * 256 + 128 * (q & 1) + ((q >> 1) & 1)] = acc[s][q];
            }
        }
    };
#pragma unroll
    for (int s = 0; s < NSLOT; ++s)
        if (j_[s] >= 0) scale_tile(acc[s], j_[s], v_, false);
    publish(0, lane);

    for (int k = 0; k < T; ++k) {
        // (per-step copy of the lane index: as loop invariants, LDS addresses would be kept live throughout)
        int l64 = lane;
        asm volatile("" : "+v"(l64));
        const unsigned fm = form_mask(k);
        const char *panel = lb_lds + (k & 1) * LB_PANEL, *Dq = lb_lds + LB_LDS_D + (k & 1) * LB_DP;
        __syncthreads();   // D and panel of step k
        __builtin_amdgcn_s_sleep(2);   // the chain's reads first
        if (v_ >= 0) {
            // One path for all tiles: N_jv (+)= R_j P_v^T with the identity for R_v where v = k (P = D) and for R_j where
            // j = k, and a zero start for the tiles of block k (I P = P_v^T, R_j D, I D: exact, h + m + l).  The diagonal
            // tile of block k + 1 is the chain's: what is left in it here is replaced in the next step.
            LbFrag f[2], dq[2];
            lb_read_panel(f, panel, v_ == k ? LB_IDENT : v_, v_ == k || ((fm >> v_) & 1), l64);
            dq[0] = lb_read_f(Dq, 2048, 0, l64);
            dq[1] = lb_read_f(Dq, 2048, 1, l64);
            lb_floatx16 p;
#pragma unroll
            for (int q = 0; q < 16; ++q) p[q] = 0.f;
            lb_mma(p, dq[0], f[0]);
            lb_mma(p, dq[1], f[1]);
            const LbFrag p0 = lb_split8(p, 0), p1 = lb_split8(p, 1);
#pragma unroll
            for (int s = 0; s < NSLOT; ++s) {
                const int j = j_[s];
                if (j < 0) break;                       // (the slots of a star are filled from the front)
                lb_read_panel(f, panel, j == k ? LB_IDENT : j, j == k || ((fm >> j) & 1), l64);
                if (v_ == k || j == k) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[s][q] = 0.f;
                }
                lb_mma(acc[s], f[0], p0);
                lb_mma(acc[s], f[1], p1);
            }
        }
        if (k + 1 < T) publish(k + 1, l64);
    }
    __syncthreads();   // the panels are dead: staging tiles

    // undo the scaling; every off-diagonal tile is written twice, as it is and (through a per-wavefront 32x33 LDS tile, so
    // that it goes along rows as well) transposed; of a diagonal tile the lower half is written and mirrored: exactly symmetric
    if (v_ < 0) return;
    float *stage = (float *)lb_lds + w * (32 * 33);
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
        const int bi = j_[s], bj = v_;
        if (bi < 0) continue;
        float si[16], sj;
        tile_scales(si, sj, bi, bj, false);
        lb_floatx16 x, y;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            x[q] = acc[s][q] * si[q] * sj;
            stage[l32_ * 33 + 8 * (q >> 2) + 4 * h_ + (q & 3)] = x[q];          // transposed
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) y[q] = stage[(8 * (q >> 2) + 4 * h_ + (q & 3)) * 33 + l32_];
        float *dx = J.dst + (unsigned)(32 * bi) * ldd + (unsigned)(32 * bj + l32_);   // rows of block bi
        float *dy = J.dst + (unsigned)(32 * bj) * ldd + (unsigned)(32 * bi + l32_);   // the mirror image
        if (bi != bj && whole(bi, bj)) {
#pragma unroll
            for (int q = 0; q < 16; ++q) dx[(unsigned)(8 * (q >> 2) + 4 * h_ + (q & 3)) * ldd] = x[q];
#pragma unroll
            for (int q = 0; q < 16; ++q) dy[(unsigned)(8 * (q >> 2) + 4 * h_ + (q & 3)) * ldd] = y[q];
        } else {
            const int room_i = n - 32 * bi, room_j = n - 32 * bj;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int r = 8 * (q >> 2) + 4 * h_ + (q & 3);
                // of a diagonal tile the elements below and on the diagonal, and those above from their mirror image
                const float z = (bi != bj || l32_ <= r) ? x[q] : y[q];
                if (r < room_i && l32_ < room_j) dx[(unsigned)(8 * (q >> 2) + 4 * h_ + (q & 3)) * ldd] = z;
                if (bi != bj && r < room_j && l32_ < room_i) dy[(unsigned)(8 * (q >> 2) + 4 * h_ + (q & 3)) * ldd] = y[q];
            }
        }
    }
}

template <int NSLOT>
static hipError_t launch_leaf_block(const LeafJob *jobs_dev, int n_jobs, const float *damp_dev, int32_t *info,
                                    hipStream_t s)
{
    constexpr size_t lds_bytes = LB_LDS_BYTES;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void *)leaf_block_kernel<NSLOT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        configured = true;
    }
    leaf_block_kernel<NSLOT><<<dim3(n_jobs), dim3(1024), lds_bytes, s>>>(jobs_dev, damp_dev, info);
    return hipGetLastError();
}

hipError_t launch_leaf(const LeafJob *jobs_dev, int n_jobs, int size_class, const float *damp_dev,
                       int32_t *info, hipStream_t s)
{
    if (n_jobs <= 0) return hipSuccess;
    switch (kLeafClasses[size_class]) {   // class value = n_max / 32: one, two or three tiles for each of fifteen wavefronts
        case 5: return launch_leaf_block<1>(jobs_dev, n_jobs, damp_dev, info, s);
        case 7: return launch_leaf_block<2>(jobs_dev, n_jobs, damp_dev, info, s);
        case 9: return launch_leaf_block<3>(jobs_dev, n_jobs, damp_dev, info, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kfac
