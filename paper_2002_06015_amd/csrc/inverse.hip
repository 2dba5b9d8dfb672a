// Kernels of the damped inversion (Sec. 3.3, Eq. 12) other than the GEMMs:
//   - trace_kernel:  pi^2 = (tr A / dA) / (tr G / dG) and the two damping values per layer;
//   - copy_damp_kernel: dst = src + damp * I (start of the blocked inversion), optionally with the
//     bias border of an A factor eliminated on the way (Schur complement), and border_kernel,
//     which puts the border back into the finished inverse;
//   - leaf_block_kernel: (X + damp I)^-1 for n <= 288 by a blocked symmetric sweep held in the
//     registers of one 768-thread workgroup, block products on the matrix cores (one matrix per
//     workgroup, many matrices per launch).
#include "kfac_internal.h"


namespace kfac {

// ------------------------------------------------------------------ trace / pi / damping
__device__ __forceinline__ double pi_of(const TraceJob &J, double trA, double trG)
{
    return trA > 0.0 && trG > 0.0 ? sqrt((trA / J.dA) / (trG / J.dG)) : 1.0;
}
__device__ __forceinline__ void write_damping(const TraceJob &J, double pi, float gamma, float *damp, float *pi_out)
{
    damp[3 * J.idx + 0] = (float)pi;
    damp[3 * J.idx + 1] = (float)(pi * (double)gamma);   // added to A
    damp[3 * J.idx + 2] = (float)((double)gamma / pi);   // added to G
    if (pi_out) pi_out[J.idx] = (float)pi;
}
// The traces of a layer over the THREADS threads of a workgroup, in two halves: their parts per wavefront into parts[2][THREADS / 64]
// (then a barrier), and the damping of A or G from these.  Layers of up to kInlineTrace rows in both factors: one memory latency in
// the place of a launch of its own.  (The order of the sums is that of the workgroup: A and G of a layer, and a launch of its own, may
// differ in the last place of pi as a double.)
template <int THREADS>
__device__ __forceinline__ void trace_parts(const TraceJob &J, double *parts)
{
    const Global<const float> A = global(J.A), G = global(J.G);
    const int tid = threadIdx.x;
    double sa = 0.0, sg = 0.0;
    for (int i = tid; i < J.dA; i += THREADS) sa += (double)A[(long long)i * J.dA + i];
    for (int i = tid; i < J.dG; i += THREADS) sg += (double)G[(long long)i * J.dG + i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { sa += __shfl_xor(sa, o); sg += __shfl_xor(sg, o); }
    if ((tid & 63) == 0) { parts[tid >> 6] = sa; parts[THREADS / 64 + (tid >> 6)] = sg; }
}
template <int THREADS>
__device__ __forceinline__ double pi_from_parts(const TraceJob &J, const double *parts)
{
    double sa = 0.0, sg = 0.0;
    for (int w = 0; w < THREADS / 64; ++w) { sa += parts[w]; sg += parts[THREADS / 64 + w]; }
    return pi_of(J, sa, sg);
}

__global__ __launch_bounds__(256) void trace_kernel(const TraceJob *__restrict__ jobs, float gamma,
                                                    float *__restrict__ damp, float *__restrict__ pi_out)
{
    __shared__ double red[2][256];
    const TraceJob J = jobs[blockIdx.x];
    const Global<const float> A = global(J.A), G = global(J.G);
    double sa = 0.0, sg = 0.0;
    for (int i = threadIdx.x; i < J.dA; i += 256) sa += (double)A[(long long)i * J.dA + i];
    for (int i = threadIdx.x; i < J.dG; i += 256) sg += (double)G[(long long)i * J.dG + i];
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
    if (threadIdx.x == 0) write_damping(J, pi_of(J, red[0][0], red[1][0]), gamma, damp, pi_out);
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

__global__ __launch_bounds__(256) void copy_damp_kernel(const CopyJob *__restrict__ jobs, int n_jobs, Damping D)
{
    __shared__ double parts[2 * 4];
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const CopyJob J = jobs[lo];
    float d = 0.f;
    if (D.layers) {
        const TraceJob L = D.layers[J.layer];
        trace_parts<256>(L, parts);
        __syncthreads();
        const double pi = pi_from_parts<256>(L, parts);
        const bool of_A = J.damp_idx == 3 * L.idx + 1;
        d = (float)(of_A ? pi * (double)D.gamma : (double)D.gamma / pi);
        if (of_A && wg == J.wg_start && threadIdx.x == 0) write_damping(L, pi, D.gamma, D.damp, D.pi_out);
    } else if (J.damp_idx >= 0) {
        d = D.damp[J.damp_idx];
    }
    const int r0 = (wg - J.wg_start) * COPY_ROWS;
    const Global<const float> src = global(J.src);
    const Global<float> dst = global(J.dst);
    const Global<const float> last = src + (long long)J.n * J.lds;   // the border row u^T, c (if any)
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
            if (r0 + q < r1) v[q] = *(Global<const vec4>)(src + (long long)(r0 + q) * J.lds + c);
        vec4 u = {0.f, 0.f, 0.f, 0.f};
        if (J.border) u = *(Global<const vec4>)(last + c);
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
            *(Global<vec4>)(dst + (long long)r * J.ldd + c) = x;
        }
    }
    for (int r = r0; r < r1; ++r) {
        const float ur = J.border ? last[r] * ic : 0.f;
        for (int c = n4 + (int)threadIdx.x; c < min(J.n, n4 + 4); c += 256) {
            float v = src[(long long)r * J.lds + c];
            if (r == c) v += d;
            if (J.border) v = fmaf(-ur, last[c], v);
            dst[(long long)r * J.ldd + c] = v;
        }
    }
}

hipError_t launch_copy_damp(const CopyJob *jobs_dev, int n_jobs, int total_wgs, const Damping &damping, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    copy_damp_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs, damping);
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
        const Global<const float> u = global(J.src) + (long long)J.n * J.lds;
        const Global<float> X = global(J.X), x = X + (long long)i * J.ldx;
        // 16-byte accesses that only need element alignment (the leading dimensions are odd)
        typedef float vec4 __attribute__((ext_vector_type(4), aligned(4)));
        float a4[4] = {0.f, 0.f, 0.f, 0.f};
        const int n4 = J.n & ~3;
        for (int j = 4 * lane; j < n4; j += 256) {
            const vec4 xv = *(Global<const vec4>)(x + j), uv = *(Global<const vec4>)(u + j);
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
            X[(long long)i * J.ldx + J.n] = v;
            X[(long long)J.n * J.ldx + i] = v;
        }
        return;
    }
    // corner: X[n][n] = (1 - sum_i u_i X[n][i]) / c   (X[n][i] = -w_i / c from pass 0)
    __shared__ float red[4];
    const BorderJob J = jobs[blockIdx.x];
    const Global<const float> u = global(J.src) + (long long)J.n * J.lds;
    const Global<float> xr = global(J.X) + (long long)J.n * J.ldx;
    float acc = 0.f;
    for (int i = threadIdx.x; i < J.n; i += 256) acc = fmaf(u[i], xr[i], acc);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float c = u[J.n] + ((J.damp_idx >= 0) ? damp[J.damp_idx] : 0.f);
        const float q = (red[0] + red[1]) + (red[2] + red[3]);
        xr[J.n] = (1.f - q) / c;
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
// (X + damp I)^-1 for n <= 288 by one 768-thread workgroup, as a symmetric block sweep with 32x32 blocks.  The matrix
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
//     registers, while the others do the rest of step k.  D of the next block is ready when they are.  It has a SIMD for
//     itself: beside it, the tiles' wavefronts waited for its issue slots and finished last.
//   - The tiles are dealt to nine wavefronts, three on each other SIMD, as stars: the five tiles of wavefront v share the
//     block index v, so it needs one P_v only and forms it itself.  It forms the transpose, D R_v^T: its accumulator layout
//     (lane: row of block v, registers: k) is, split into planes, the operand layout of the update R_j P_v^T, with the
//     contraction index in the order the registers have.  Every operand uses that order; P never goes through LDS and one
//     barrier per step is left.  (Twelve wavefronts with four tiles: more P's, and registers that spill.)
//   - A tile is (registers: row of block j, lanes: row of block v).  For the panel of step k a tile with j = k is stored
//     as the fragments its readers load (two planes, 16 bytes a lane: form F), a tile with v = k as [k][row] rows that
//     are read with the transposing LDS read (form T); no 2-byte stores.  The panels of two steps alternate.  The wavefront
//     that stores most of the next panel goes first in its SIMD.
//
// Products are through two fp16 planes (x s = h + l, three instructions per 16-wide step instead of six; see gemm_nt.hip), with
// scales that are exact: a panel block and D take the power of two that brings their largest element to [2^14, 2^15), P_v one per
// row (a lane).  Nothing overflows, and elements down to 2^-16 of the largest of their block lose nothing.  The sum of a product
// is scaled back into the tile with one fma, so a tile is rounded once per step (six times as the accumulator of bf16 planes):
// inverses of 5 to 288 rows err 0.65 of what they did with three bf16 planes, those of 289 to 4609 rows 0.52 (127 and 87 factors of
// random layers).  P also takes the product of the low planes (two instructions a step more, 36 before; 0.5 us at n = 288): where rows
// are nearly parallel D is large and its products with R cancel, and what that product leaves out does not.  Pairs correlated by 0.9995,
// 288 rows: 1.0e-3 with it, 2.9e-3 without, 1.2e-3 with three bf16 planes; 0.95^|i-j| 1.7e-5, 3.1e-5, 3.4e-5; patches of smooth
// images 2.6e-5, 5.1e-5, 4.5e-5; 0.999^|i-j| 0.21, 0.49, 0.21.
//
// n = 288: 42 us (52 with fifteen wavefronts, three bf16 planes and an address per element), 224: 30.4 (36.3), 160: 20.4
// (23.8), 64: 11.2 (11.3), 42: 12.0 (11.4: stores of partial tiles).  In-kernel cycles, before the product of the low planes at n = 288: loads and scales 8400, a step 7650, stores 9000.  Of a step, the chain
// needs 5600 (sweep 3640, D into planes 850, operand reads 260, P and update 900); a SIMD with three stars 3460 for its matrix
// instructions and 5800 for the vector ones.
typedef float lb_floatx16 __attribute__((ext_vector_type(16)));
typedef float lb_floatx4 __attribute__((ext_vector_type(4)));
typedef float lb_floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef short lb_shortx4 __attribute__((ext_vector_type(4)));
typedef short lb_shortx8 __attribute__((ext_vector_type(8)));
typedef lb_shortx4 __attribute__((address_space(3))) *lb_lds_shortx4_ptr;
constexpr int LB_MAXT = 9;
constexpr int LB_THREADS = 768;                         // three wavefronts a SIMD
constexpr int LB_CHAIN = 11;                            // the chain wavefront
constexpr int LB_TROW = 72;                             // bytes per k row of form T (32 bf16 + 8 bytes: spreads the banks)
constexpr int LB_BLK = 32 * LB_TROW;                    // bytes of one plane of one panel block (form F needs 2048)
constexpr int LB_IDENT = LB_MAXT;                       // a panel block that always holds the identity, form F
constexpr int LB_PLANE = (LB_MAXT + 1) * LB_BLK;        // bytes of one plane of a panel
constexpr int LB_PANEL = 2 * LB_PLANE;                  // one panel: [plane][block]
constexpr int LB_DP = 2 * 2048;                         // planes of D, form F
constexpr int LB_TOP = 14;                              // a scaled block has its largest element in [2^14, 2^15)
constexpr int LB_LDS_D = 2 * LB_PANEL, LB_LDS_DIAG = LB_LDS_D + 2 * LB_DP,
              LB_LDS_SC = LB_LDS_DIAG + 2 * 4096, LB_LDS_UN = LB_LDS_SC + 32 * LB_MAXT * 4,
              LB_LDS_BYTES = LB_LDS_UN + 2 * LB_THREADS / 64 * 8;   // UN: reciprocal scales of two panels' blocks, of I and (LB_UN_D) of D
constexpr int LB_UN_D = LB_IDENT + 1;
static_assert(2 * 16 * 4 <= 2 * LB_THREADS / 64 * 8 && LB_LDS_UN % 8 == 0, "the traces' parts lie in the same place");
static_assert(LB_LDS_BYTES <= 160 * 1024 - 64, "one compute unit's LDS");
constexpr int LB_STAGE = 36;                            // row length of the staging tiles (16-byte accesses spread over the banks)
static_assert(LB_LDS_D >= LB_MAXT * 2 * 32 * LB_STAGE * 4, "the staging tiles of the final store fit into the panels");

// Of T blocks in a circle, the tile of blocks v and j is held as (v, j) where v is at most half a circle ahead of j (exactly
// half of it: where v > j): star v is {v; v, v - 1, ..., v - T / 2}, the same number of tiles for every wavefront.
constexpr int LB_SLOTS = LB_MAXT / 2 + 1;
__device__ __forceinline__ int lb_star(int T, int v, int s)   // tile s of star v: its j, or -1
{
    return 2 * s < T || (2 * s == T && 2 * v >= T) ? (v >= s ? v - s : v - s + T) : -1;
}
__device__ __forceinline__ bool lb_form_f(int T, int i, int k)   // in step k: block i of the panel comes from star i
{
    const int d = i >= k ? i - k : i - k + T;
    return 2 * d < T || (2 * d == T && i > k);
}

__device__ __forceinline__ float lb_readlane(float x, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

struct LbFrag { halfx8 h, l; };

// eight accumulator registers (8 u .. 8 u + 7) of a tile, scaled, as an operand fragment of step u
__device__ __forceinline__ LbFrag lb_split8(const lb_floatx16 &t, int u, float scale)
{
    uint4 h, l;
    split_half_pair(t[8 * u + 0], t[8 * u + 1], scale, h.x, l.x);
    split_half_pair(t[8 * u + 2], t[8 * u + 3], scale, h.y, l.y);
    split_half_pair(t[8 * u + 4], t[8 * u + 5], scale, h.z, l.z);
    split_half_pair(t[8 * u + 6], t[8 * u + 7], scale, h.w, l.w);
    return {__builtin_bit_cast(halfx8, h), __builtin_bit_cast(halfx8, l)};
}
// product of two blocks (fragments of both 16-wide steps), the small terms first; FOUR: with the product of the low planes
template <bool FOUR>
__device__ __forceinline__ lb_floatx16 lb_mma(const LbFrag (&a)[2], const LbFrag (&b)[2])
{
    lb_floatx16 c;
#pragma unroll
    for (int q = 0; q < 16; ++q) c[q] = 0.f;
    if constexpr (FOUR) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0].l, b[0].l, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1].l, b[1].l, c, 0, 0, 0);
    }
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0].l, b[0].h, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0].h, b[0].l, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1].l, b[1].h, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1].h, b[1].l, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0].h, b[0].h, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1].h, b[1].h, c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ float lb_max_abs(const lb_floatx16 &t)
{
    float m = fmaxf(fabsf(t[0]), fabsf(t[1]));
#pragma unroll
    for (int q = 2; q < 16; q += 2) m = fmaxf(fmaxf(m, fabsf(t[q])), fabsf(t[q + 1]));
    return m;
}
// (magnitudes compare as unsigned numbers, which have no quiet form to be brought into)
template <int CTRL>
__device__ __forceinline__ unsigned lb_max_dpp(unsigned x)
{
    return max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ unsigned lb_max_halves(unsigned x)   // of lanes l and l + 32
{
    const auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return max(s[0], s[1]);
}
// the largest magnitudes of the lanes' parts of N tiles -> the scales of the tiles (uniform)
template <int N>
__device__ __forceinline__ void lb_tile_scales(float (&most)[N])
{
    unsigned m[N];
#pragma unroll
    for (int n = 0; n < N; ++n) m[n] = lb_max_dpp<0xB1>(__float_as_uint(most[n]));   // quad_perm 1 0 3 2
#pragma unroll
    for (int n = 0; n < N; ++n) m[n] = lb_max_dpp<0x4E>(m[n]);                       // quad_perm 2 3 0 1
#pragma unroll
    for (int n = 0; n < N; ++n) m[n] = lb_max_dpp<0x141>(m[n]);                      // row_half_mirror
#pragma unroll
    for (int n = 0; n < N; ++n) m[n] = lb_max_dpp<0x140>(m[n]);                      // row_mirror
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const auto s = __builtin_amdgcn_permlane16_swap(m[n], m[n], false, false);
        m[n] = max(s[0], s[1]);
    }
#pragma unroll
    for (int n = 0; n < N; ++n) most[n] = half_scale(__uint_as_float(__builtin_amdgcn_readfirstlane(lb_max_halves(m[n]))), LB_TOP);
}
__device__ __forceinline__ float lb_tile_scale(const lb_floatx16 &t)
{
    float m[1] = {lb_max_abs(t)};
    lb_tile_scales(m);
    return m[0];
}
__device__ __forceinline__ float lb_reciprocal(float s) { return __uint_as_float((254u << 23) - __float_as_uint(s)); }   // of a power of two
// form F: fragments as they are read, plane stride given; [u][lane] 16 bytes each
__device__ __forceinline__ LbFrag lb_read_f(const char *blk, int plane, int u, int lane)
{
    auto rd = [&](int q) { return __builtin_bit_cast(halfx8, *(const lb_shortx8 *)(blk + q * plane + u * 1024 + lane * 16)); };
    return {rd(0), rd(1)};
}
__device__ __forceinline__ void lb_store_f(char *blk, int plane, int u, const LbFrag &f, int lane)
{
    *(lb_shortx8 *)(blk + u * 1024 + lane * 16) = __builtin_bit_cast(lb_shortx8, f.h);
    *(lb_shortx8 *)(blk + plane + u * 1024 + lane * 16) = __builtin_bit_cast(lb_shortx8, f.l);
}
// form T: [k][row]; the tile's lanes are k and its registers rows.  The transposing read gives lane i of 16 element i % 4
// of the 8-byte groups addressed by lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12: four adjacent k of row i.
__device__ __forceinline__ LbFrag lb_read_t(const char *blk, int u, int lane)
{
    const int i = lane & 15, row0 = lane & 16, half = lane >> 5;
    const char *p = blk + __umul24(16 * u + 4 * half + (i >> 2), LB_TROW) + 2 * (row0 + 4 * (i & 3));
    auto rd = [&](int q) {
        const lb_shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lb_lds_shortx4_ptr)(p + q * LB_PLANE));
        const lb_shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lb_lds_shortx4_ptr)(p + q * LB_PLANE + 8 * LB_TROW));
        return __builtin_bit_cast(halfx8, lb_shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    };
    return {rd(0), rd(1)};
}
__device__ __forceinline__ void lb_store_t(char *blk, const lb_floatx16 &t, float scale, int lane)
{
    char *d = blk + (lane & 31) * LB_TROW + 8 * (lane >> 5);
#pragma unroll
    for (int g = 0; g < 4; ++g) {   // rows 8 g + 4 half .. + 3
        uint2 h, l;
        split_half_pair(t[4 * g], t[4 * g + 1], scale, h.x, l.x);
        split_half_pair(t[4 * g + 2], t[4 * g + 3], scale, h.y, l.y);
        *(uint2 *)(d + 16 * g) = h;
        *(uint2 *)(d + LB_PLANE + 16 * g) = l;
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

__global__ __launch_bounds__(LB_THREADS) void leaf_block_kernel(const LeafJob *__restrict__ jobs, Damping D,
                                                               int32_t *__restrict__ info)
{
    extern __shared__ __attribute__((aligned(16))) char lb_lds[];
    float *sc = (float *)(lb_lds + LB_LDS_SC);       // [32 T] diagonal scaling
    float *unscale = (float *)(lb_lds + LB_LDS_UN);  // [2][16]

    const LeafJob J = jobs[blockIdx.x];
    const int n = J.n;
    const int T = (n + 31) >> 5;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32_ = lane & 31, h_ = lane >> 5;
    float d = 0.f;
    const bool find_damping = D.layers && J.layer >= 0;
    const TraceJob *layer = D.layers + max(J.layer, 0);
    double *parts = (double *)(lb_lds + LB_LDS_UN);   // (until the first scale is written there)
    if (find_damping) trace_parts<LB_THREADS>(*layer, parts);
    else if (J.damp_idx >= 0) d = D.damp[J.damp_idx];
    // called by all wavefronts once their loads are under way
    auto wait_for_damping = [&]() {
        if (!find_damping) return;
        __syncthreads();
        const double pi = pi_from_parts<LB_THREADS>(*layer, parts);
        const bool of_A = J.damp_idx == 3 * layer->idx + 1;
        d = (float)(of_A ? pi * (double)D.gamma : (double)D.gamma / pi);
        if (of_A && tid == 0) write_damping(*layer, pi, D.gamma, D.damp, D.pi_out);
        __syncthreads();
    };
    const unsigned lds = (unsigned)J.lds, ldd = (unsigned)J.ldd;
    const Global<const float> src = global(J.src);
    const Global<float> dst = global(J.dst);

    // my tiles: (rows of block j[s]: registers, rows of block v: lanes)
    const int worker = (w & 3) == 3 ? LB_MAXT : w - (w >> 2);   // (the chain's SIMD has no other)
    const int v_ = worker < T ? worker : -1;
    int j_[LB_SLOTS];
#pragma unroll
    for (int s = 0; s < LB_SLOTS; ++s) j_[s] = v_ >= 0 ? lb_star(T, v_, s) : -1;

    // the chain wavefront loads the first diagonal tile, the others their tiles; the scaling needs the diagonal
    // (row pointers of whole tiles are uniform, with one offset per lane: as an address per element, the vector instructions for
    // them took most of the loads' time, and of the stores')
    auto whole = [&](int bi, int bj) { return 32 * (max(bi, bj) + 1) <= n; };
    auto load_tile = [&](lb_floatx16 &t, int bi, int bj, bool chain) {
        if (whole(bi, bj)) {
            const Global<const char> row = (Global<const char>)(src + (long long)(32 * bi) * lds + 32 * bj);
            const unsigned at = 4u * (chain ? h_ * lds + lb_row_of(l32_) : 4 * h_ * lds + l32_);
#pragma unroll
            for (int q = 0; q < 16; ++q) t[q] = *(Global<const float>)(row + (long long)(chain ? lb_row(q, 0) : 8 * (q >> 2) + (q & 3)) * lds * 4 + at);
            return;
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int i = 32 * bi + (chain ? lb_row(q, h_) : 8 * (q >> 2) + 4 * h_ + (q & 3)), j = 32 * bj + (chain ? lb_row_of(l32_) : l32_);
            t[q] = src[(unsigned)min(i, n - 1) * lds + (unsigned)min(j, n - 1)];   // (outside: replaced when it is scaled)
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
    auto scale_tile = [&](lb_floatx16 &t, int bi, int bj, bool chain, bool diagonal) {
        float si[16], sj;
        tile_scales(si, sj, bi, bj, chain);
        if (diagonal) {   // (at the same registers and lanes in either order)
#pragma unroll
            for (int q = 0; q < 16; ++q) t[q] += 8 * (q >> 2) + 4 * h_ + (q & 3) == l32_ ? d : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) t[q] = t[q] * si[q] * -sj;
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
                const float a = src[(unsigned)tid * lds + (unsigned)tid] + d;
                v = a > 0.f ? rsqrtf(a) : 1.f;   // a non-positive diagonal shows up as a non-positive pivot
            }
            sc[tid] = v;
        }
    };

    // The two roles run loops of their own with the same barriers: one after the scales, one per step, one at the end.
    if (w == LB_CHAIN) {
        lb_floatx16 t;
        load_tile(t, 0, 0, true);
        wait_for_damping();
        __syncthreads();
        scale_tile(t, 0, 0, true, true);
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
                const float scale = lb_tile_scale(t);
                const lb_floatx16 dt = lb_plain_rows(t);       // lanes (D is symmetric: its rows) in the chain's order yet
                const int at = (l64 & 32) | lb_row_of(l64 & 31);
                lb_store_f(Dq, 2048, 0, lb_split8(dt, 0, scale), at);
                lb_store_f(Dq, 2048, 1, lb_split8(dt, 1, scale), at);
                if (l64 == 0) unscale[16 * (k & 1) + LB_UN_D] = lb_reciprocal(scale);
            }
            __syncthreads();   // D and panel of step k, diagonal tile of block k + 1
            if (k + 1 == T) break;
            // rows of R in the chain's order (lanes), its columns and D in the plain one
            const char *blk = lb_lds + (k & 1) * LB_PANEL + (k + 1) * LB_BLK;
            const int from = (l64 & 32) | lb_row_of(l64 & 31);
            const LbFrag r[2] = {lb_read_f(blk, LB_PLANE, 0, from), lb_read_f(blk, LB_PLANE, 1, from)};
            const LbFrag d[2] = {lb_read_f(Dq, 2048, 0, l64), lb_read_f(Dq, 2048, 1, l64)};
            const float un_r = unscale[16 * (k & 1) + k + 1], un_d = unscale[16 * (k & 1) + LB_UN_D];
            const lb_floatx4 *o = (const lb_floatx4 *)(lb_lds + LB_LDS_DIAG + ((k + 1) & 1) * 4096);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const lb_floatx4 x = o[g * 64 + l64];
#pragma unroll
                for (int e = 0; e < 4; ++e) t[4 * g + e] = x[e];
            }
            const lb_floatx16 p = lb_mma<true>(d, r);      // P^T = D R^T
            const float scale = half_scale(__uint_as_float(lb_max_halves(__float_as_uint(lb_max_abs(p)))), LB_TOP), un = lb_reciprocal(scale) * un_d * un_r * un_r;
            const LbFrag pf[2] = {lb_split8(p, 0, scale), lb_split8(p, 1, scale)};
            const lb_floatx16 c = lb_mma<false>(r, pf);
#pragma unroll
            for (int q = 0; q < 16; ++q) t[q] = fmaf(c[q], un, t[q]);
        }
        if (lane == 0 && info && J.info_idx >= 0) {
            if (J.pivot_base == 0) info[J.info_idx] = bad;
            else if (bad != 0) atomicCAS(&info[J.info_idx], 0, J.pivot_base + bad);
        }
        __syncthreads();
        return;
    }

    lb_floatx16 acc[LB_SLOTS];
#pragma unroll
    for (int s = 0; s < LB_SLOTS; ++s) {
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[s][q] = 0.f;
        if (j_[s] >= 0) load_tile(acc[s], j_[s], v_, false);
    }
    wait_for_damping();
    scales();
    if (w < 8) {   // the identity: wavefront w writes step fragments w % 2 of plane (w / 2) % 2 of panel w / 4
        const int u = w & 1, q = (w >> 1) & 1;
        lb_shortx8 e;
#pragma unroll
        for (int x = 0; x < 8; ++x) e[x] = (q == 0 && 16 * u + 8 * (x >> 2) + 4 * h_ + (x & 3) == l32_) ? (short)0x3C00 : (short)0;
        *(lb_shortx8 *)(lb_lds + (w >> 2) * LB_PANEL + q * LB_PLANE + LB_IDENT * LB_BLK + u * 1024 + lane * 16) = e;
        if (lane == 0) unscale[16 * (w >> 2) + LB_IDENT] = 1.f;
    }
    __syncthreads();
    // panel of step kk from the tiles that have an index kk, and the diagonal tile of block kk + 1 for the chain
    auto publish = [&](int kk, int l64) {
        char *panel = lb_lds + (kk & 1) * LB_PANEL;
        float *un = unscale + 16 * (kk & 1);
        if (v_ == kk) {
            // all tiles but the diagonal one, their scales side by side (a lone reduction over the lanes is latency)
            float scale[LB_SLOTS - 1];
#pragma unroll
            for (int s = 1; s < LB_SLOTS; ++s) scale[s - 1] = lb_max_abs(acc[s]);
            lb_tile_scales(scale);
#pragma unroll
            for (int s = 1; s < LB_SLOTS; ++s) {
                if (j_[s] < 0) break;
                lb_store_t(panel + j_[s] * LB_BLK, acc[s], scale[s - 1], l64);
                if (l64 == 0) un[j_[s]] = lb_reciprocal(scale[s - 1]);
            }
            return;
        }
#pragma unroll
        for (int s = 1; s < LB_SLOTS; ++s) {
            if (j_[s] != kk) continue;
            const float scale = lb_tile_scale(acc[s]);
            lb_store_f(panel + v_ * LB_BLK, LB_PLANE, 0, lb_split8(acc[s], 0, scale), l64);
            lb_store_f(panel + v_ * LB_BLK, LB_PLANE, 1, lb_split8(acc[s], 1, scale), l64);
            if (l64 == 0) un[v_] = lb_reciprocal(scale);
        }
        if (v_ == kk + 1) {
            // in the chain's order: row 8 g + 4 half + e is its register 4 g + 2 half + e / 2 of half-wave e % 2
            float *o = (float *)(lb_lds + LB_LDS_DIAG + ((kk + 1) & 1) * 4096) + 4 * lb_tile_row(l64 & 31) + 2 * (l64 >> 5);
#pragma unroll
            for (int q = 0; q < 16; ++q) o[(q >> 2) * 256 + 128 * (q & 1) + ((q >> 1) & 1)] = acc[0][q];
        }
    };
#pragma unroll
    for (int s = 0; s < LB_SLOTS; ++s)
        if (j_[s] >= 0) scale_tile(acc[s], j_[s], v_, false, s == 0);
    publish(0, lane);

    for (int k = 0; k < T; ++k) {
        // (per-step copy of the lane index: as loop invariants, LDS addresses would be kept live throughout)
        int l64 = lane;
        asm volatile("" : "+v"(l64));
        const char *panel = lb_lds + (k & 1) * LB_PANEL, *Dq = lb_lds + LB_LDS_D + (k & 1) * LB_DP;
        __syncthreads();   // D and panel of step k
        __builtin_amdgcn_s_sleep(2);   // the chain's reads first
        // the star whose whole panel is published at the end of the step goes first, then those that publish one tile
        if (v_ == k + 1) __builtin_amdgcn_s_setprio(3);
        else if (k + 1 < T && lb_form_f(T, v_, k + 1)) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
        if (v_ >= 0) {
            // N_jv += R_j P_v^T with the identity for R_v where v = k (P = D); of the tiles of block k, N_kv = P_v^T (j = k) and
            // N_jk = R_j D (v = k).  The diagonal tile of block k + 1 is the chain's: what is left in it here is replaced in the
            // next step.
            LbFrag f[2][2], dq[2];
            const float *un = unscale + 16 * (k & 1);
            const int iv = v_ == k ? LB_IDENT : v_;
            lb_read_panel(f[1], panel, iv, v_ == k || lb_form_f(T, v_, k), l64);
            dq[0] = lb_read_f(Dq, 2048, 0, l64);
            dq[1] = lb_read_f(Dq, 2048, 1, l64);
            const float un_p = un[LB_UN_D] * un[iv];
            float un_j[LB_SLOTS];
#pragma unroll
            for (int s = 0; s < LB_SLOTS; ++s) un_j[s] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(un[max(j_[s], 0)])));
            // the fragments of a tile are requested ahead of the products of the one before (those of tile (v, v) are at hand)
            auto read_tile = [&](int s) {
                if (j_[s] >= 0 && j_[s] != k) lb_read_panel(f[(s + 1) & 1], panel, j_[s], lb_form_f(T, j_[s], k), l64);
            };
            read_tile(1);
            const lb_floatx16 p = lb_mma<true>(dq, f[1]);
            const float scale = half_scale(__uint_as_float(lb_max_halves(__float_as_uint(lb_max_abs(p)))), LB_TOP), un_v = lb_reciprocal(scale) * un_p;
            dq[0] = lb_split8(p, 0, scale);
            dq[1] = lb_split8(p, 1, scale);
#pragma unroll
            for (int s = 0; s < LB_SLOTS; ++s)
                if (j_[s] == k) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[s][q] = p[q] * un_p;
                }
#pragma unroll
            for (int s = 0; s < LB_SLOTS; ++s) {
                const int j = j_[s];
                if (j < 0) break;                       // (the slots of a star are filled from the front)
                if (s > 0 && s + 1 < LB_SLOTS) read_tile(s + 1);
                __builtin_amdgcn_sched_barrier(0);
                if (j == k) continue;
                const float u = un_v * un_j[s];
                const lb_floatx16 c = lb_mma<false>(f[(s + 1) & 1], dq);
                __builtin_amdgcn_sched_barrier(0);
                if (v_ == k) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[s][q] = c[q] * u;
                } else {
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[s][q] = fmaf(c[q], u, acc[s][q]);
                }
            }
        }
        if (k + 1 < T) publish(k + 1, l64);
    }
    __syncthreads();   // the panels are dead: staging tiles

    // undo the scaling; every off-diagonal tile is written twice, as it is and transposed, both through LDS tiles of the wavefront,
    // so that a store is 16 bytes a lane along rows; of a diagonal tile the lower half is written and mirrored: exactly symmetric
    if (v_ < 0) return;
    float *st = (float *)lb_lds + worker * (2 * 32 * LB_STAGE), *stt = st + 32 * LB_STAGE;
#pragma unroll
    for (int s = 0; s < LB_SLOTS; ++s) {
        const int bi = j_[s], bj = v_;
        if (bi < 0) break;
        float si[16], sj;
        tile_scales(si, sj, bi, bj, false);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            lb_floatx4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = acc[s][4 * g + e] * si[4 * g + e] * sj;
                st[(8 * g + 4 * h_ + e) * LB_STAGE + l32_] = x[e];
            }
            *(lb_floatx4 *)(stt + l32_ * LB_STAGE + 8 * g + 4 * h_) = x;
        }
        const int c4 = 4 * (lane & 7), r8 = lane >> 3;
        const bool inside = whole(bi, bj);
        auto store = [&](const float *from, int br, int bc) {   // rows of block br
            const Global<char> to = (Global<char>)(dst + (long long)(32 * br) * ldd + 32 * bc);
            const unsigned at = 4u * (r8 * ldd + c4);
            lb_floatx4 x[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                x[g] = *(const lb_floatx4 *)(from + (8 * g + r8) * LB_STAGE + c4);
                if (s == 0) {   // above the diagonal: from the mirror image
                    const lb_floatx4 y = *(const lb_floatx4 *)(stt + (8 * g + r8) * LB_STAGE + c4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[g][e] = c4 + e <= 8 * g + r8 ? x[g][e] : y[e];
                }
            }
            if (inside) {
#pragma unroll
                for (int g = 0; g < 4; ++g) *(Global<lb_floatx4_u>)(to + (long long)(8 * g) * ldd * 4 + at) = x[g];
            } else {
                const int cols = n - 32 * bc, rows = n - 32 * br;
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (8 * g + r8 < rows && c4 + e < cols) *(Global<float>)(to + (long long)(8 * g) * ldd * 4 + at + 4 * e) = x[g][e];
            }
        };
        store(st, bi, bj);
        if (s > 0) store(stt, bj, bi);
    }
}

hipError_t launch_leaf(const LeafJob *jobs_dev, int n_jobs, const Damping &damping, int32_t *info, hipStream_t s)
{
    if (n_jobs <= 0) return hipSuccess;
    constexpr size_t lds_bytes = LB_LDS_BYTES;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void *)leaf_block_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        configured = true;
    }
    leaf_block_kernel<<<dim3(n_jobs), dim3(LB_THREADS), lds_bytes, s>>>(jobs_dev, damping, info);
    return hipGetLastError();
}

}  // namespace kfac
