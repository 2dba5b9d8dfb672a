// Grouped NT GEMM for small products of plain fp32 matrices: the Schur-complement products of the blocked inverse
// at its lower levels and the preconditioning of small layers.
//     C[i][j] = alpha * sum_m a(i, m) * b(j, m) + beta * C[i][j]
// in the product mode of three bf16 planes (see gemm_nt.hip: x = h + m + l exactly, six bf16 matrix instructions per
// block product, fp32 accumulation), same problem table, same epilogue rules.
//
// What bounds such a product is latency, not throughput: 288 x 288 x 288 is 48 MFLOP, 0.3 us of the chip, but the
// kernel of gemm_nt.hip needs 13-19 us for it (a K loop of 9 tiles, each global load -> LDS -> barrier -> fragments,
// by 25 workgroups).  Here
//   - a tile is 32 TM x 32 TN, so that a product of a few hundred rows has enough workgroups,
//   - the four wavefronts of a workgroup share the tile and split the contraction (16-wide steps dealt out in turn,
//     so that together they read whole 256-byte row segments),
//   - a lane loads its fragments straight from global memory in the layout the matrix instruction wants (8 adjacent
//     k of one row), RING steps ahead, and splits them in registers: no LDS and no barrier before the end,
//   - the four partial tiles are added in a fixed order through LDS in the epilogue (bitwise reproducible).
//
// Splitting the contraction this way also splits neighbouring steps, and where those cancel (products with the inverse of a
// factor whose neighbouring variables are correlated) a wavefront's sum is far larger than the result.  Rounded six times a
// step, once per plane product and not to nearest, such sums were up to 3 times less accurate than those of the staged kernel,
// and inverses of smooth images' factors 1.2 to 1.3 times.  So the five low-order plane products, 2^-8 of the sum, have an
// accumulator of their own and the sum is rounded once a step: 0.7 of the staged kernel's error, inverses 0.6 to 0.9 of it.
// Runs of adjacent steps per wavefront on top of that: 0.4, but 1 to 3 % slower (a row's 256 bytes are read in four places).
#include "gemm_tiles.h"

namespace kfac {

typedef float gd_floatx16 __attribute__((ext_vector_type(16)));
typedef float gd_floatx4 __attribute__((ext_vector_type(4)));
typedef float gd_floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 gd_bf16x8 __attribute__((ext_vector_type(8)));
typedef const float __attribute__((address_space(1))) *gd_gptr;
typedef const gd_floatx4_u __attribute__((address_space(1))) *gd_gptr4;

struct GdPlanes { gd_bf16x8 h, m, l; };

__device__ __forceinline__ GdPlanes gd_split(const gd_floatx4 &x, const gd_floatx4 &y)
{
    uint4 h, m, l;
    split_pair(x[0], x[1], h.x, m.x, l.x);
    split_pair(x[2], x[3], h.y, m.y, l.y);
    split_pair(y[0], y[1], h.z, m.z, l.z);
    split_pair(y[2], y[3], h.w, m.w, l.w);
    return {__builtin_bit_cast(gd_bf16x8, h), __builtin_bit_cast(gd_bf16x8, m), __builtin_bit_cast(gd_bf16x8, l)};
}

// 32 rows of a plain operand as the lanes of a wavefront see them: lane % 32 is the row (clamped to the last one:
// rows outside the operand only feed elements of C that are not stored), lane / 32 the half of a 16-wide step.
struct GdRows {
    gd_gptr p;
    __device__ __forceinline__ void init(const Operand &op, int row0, int lane)
    {
        p = (gd_gptr)op.base + (long long)min(row0 + (lane & 31), op.rows - 1) * op.row_stride + 8 * (lane >> 5);
    }
    __device__ __forceinline__ void load(int k, gd_floatx4 &x, gd_floatx4 &y) const
    {
        x = *(gd_gptr4)(p + k);
        y = *(gd_gptr4)(p + k + 4);
    }
    // the last, partial step: only elements below K are read
    __device__ __forceinline__ void load_tail(int k, int kend, int lane, gd_floatx4 &x, gd_floatx4 &y) const
    {
        const int first = k + 8 * (lane >> 5);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] = 0.f; y[e] = 0.f;
            if (first + e < kend) x[e] = p[k + e];
            if (first + 4 + e < kend) y[e] = p[k + 4 + e];
        }
    }
};

// low: the products with a middle or last plane
template <int TM, int TN>
__device__ __forceinline__ void gd_mma(gd_floatx16 (&acc)[TM][TN], gd_floatx16 (&low)[TM][TN], const gd_floatx4 (&f)[TM + TN][2])
{
    GdPlanes a[TM], b[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = gd_split(f[i][0], f[i][1]);
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = gd_split(f[TM + j][0], f[TM + j][1]);
    auto mm = [&](gd_floatx16 (&c)[TM][TN], auto pa, auto pb) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa(a[i]), pb(b[j]), c[i][j], 0, 0, 0);
    };
    auto H = [](const GdPlanes &x) { return x.h; };
    auto M = [](const GdPlanes &x) { return x.m; };
    auto L = [](const GdPlanes &x) { return x.l; };
    mm(low, L, H); mm(low, M, M); mm(low, H, L); mm(acc, H, H); mm(low, M, H); mm(low, H, M);
}

// partial sums of four wavefronts in LDS, [wave][v][lane] per 32 x 32 block in the accumulator layout
// (column = lane % 32, row = 8 * (v / 4) + 4 * (lane / 32) + v % 4)
__device__ __forceinline__ int gd_place(int blk, int r, int c)
{
    return blk * 1024 + (4 * (r >> 3) + (r & 3)) * 64 + c + 32 * ((r >> 2) & 1);
}
template <int BLOCKS>
__device__ __forceinline__ float gd_sum(const float *part, int e)
{
    constexpr int W = BLOCKS * 1024;
    return (part[e] + part[e + W]) + (part[e + 2 * W] + part[e + 3 * W]);
}

template <int TM, int TN, int RING>
__global__ __launch_bounds__(256, TM == 2 ? 2 : 1) void gemm_direct_kernel(const GemmProblem *__restrict__ probs,
                                                          const int *__restrict__ tile_start, int n_probs)
{
    constexpr int BLOCKS = TM * TN;
    __shared__ __attribute__((aligned(16))) float part[4 * BLOCKS * 1024];
    const int wg = blockIdx.x;
    const int pi = find_problem(tile_start, n_probs, wg);
    const GemmProblem &P = probs[pi];
    const int tile = xcd_remap(wg - tile_start[pi], P.n_tiles);
    int tm, tn;
    decode_tile(P, tile, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = tm * 32 * TM, j0 = tn * 32 * TN;
    const int K = P.K;

    GdRows rows[TM + TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) rows[i].init(P.a, i0 + 32 * i, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) rows[TM + j].init(P.b, j0 + 32 * j, lane);

    gd_floatx16 acc[TM][TN], low[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;

    // wavefront w takes a run of the 16-wide steps, the last one also the partial step
    const int full = K >> 4;
    const int mine = (full - w + 3) >> 2;
    if (mine > 0) {
        // loads past this wavefront's last step repeat it (always valid addresses, no branches around loads)
        gd_floatx4 f[RING][TM + TN][2];
        auto load = [&](int idx, gd_floatx4 (&d)[TM + TN][2]) {
            const int k = 16 * (w + 4 * min(idx, mine - 1));
#pragma unroll
            for (int q = 0; q < TM + TN; ++q) rows[q].load(k, d[q][0], d[q][1]);
        };
#pragma unroll
        for (int u = 0; u < RING; ++u) load(u, f[u]);
        for (int s = 0; s < mine; s += RING) {
#pragma unroll
            for (int u = 0; u < RING; ++u) {
                if (s + u < mine) gd_mma<TM, TN>(acc, low, f[u]);
                if (s + RING < mine) load(s + RING + u, f[u]);
            }
        }
    }
    if ((K & 15) && w == (full & 3)) {
        gd_floatx4 f[TM + TN][2];
#pragma unroll
        for (int q = 0; q < TM + TN; ++q) rows[q].load_tail(16 * full, K, lane, f[q][0], f[q][1]);
        gd_mma<TM, TN>(acc, low, f);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) part[((w * BLOCKS + i * TN + j) * 16 + v) * 64 + lane] = acc[i][j][v] + low[i][j][v];
    __syncthreads();
    const bool sym = (P.flags & GEMM_SYM) != 0;
    const bool diag_tile = sym && tm == tn;
    const float alpha = P.alpha, beta = P.beta;
    // direct pass: a thread owns 4 adjacent columns of one row of every block; old values of all blocks requested first
    const int q8 = 4 * (tid & 7), r32 = tid >> 3;
    const Global<float> C = global(P.C), mbase = global(!sym ? P.Ct : i0 - j0 - (32 * TN - 1) < P.mirror_band ? P.C : nullptr);
    const long long ldm = sym ? P.ldc : P.ldct;
    gd_floatx4 old[BLOCKS];
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b) old[b] = gd_floatx4{0.f, 0.f, 0.f, 0.f};
    if (beta != 0.0f) {
#pragma unroll
        for (int b = 0; b < BLOCKS; ++b) {
            const int i = i0 + 32 * (b / TN) + r32, j = j0 + 32 * (b % TN) + q8;
            if (i < P.M && j + 3 <= min(diag_tile ? i : P.N - 1, P.N - 1)) old[b] = *(Global<const gd_floatx4_u>)(C + (long long)i * P.ldc + j);
        }
    }
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b) {
        const int i = i0 + 32 * (b / TN) + r32, j = j0 + 32 * (b % TN) + q8;
        const int jmax = min(diag_tile ? i : P.N - 1, P.N - 1);   // last column this row may write
        if (i >= P.M || j > jmax) continue;
        const Global<float> dst = C + (long long)i * P.ldc + j;
        gd_floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = alpha * gd_sum<BLOCKS>(part, gd_place(b, r32, q8 + e));
        if (beta != 0.0f) {
            if (j + 3 <= jmax)
                for (int e = 0; e < 4; ++e) v[e] = fmaf(beta, old[b][e], v[e]);
            else
                for (int e = 0; e < 4 && j + e <= jmax; ++e) v[e] = fmaf(beta, dst[e], v[e]);
        }
        if (C) {
            if (j + 3 <= jmax) *(Global<gd_floatx4_u>)dst = v;
            else
                for (int e = 0; e < 4 && j + e <= jmax; ++e) dst[e] = v[e];
        }
        if (mbase)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[gd_place(b, r32, q8 + e)] = v[e];
    }
    // mirrored / transposed pass over the values of the direct pass, left in the first wavefront's place: a thread owns 4
    // adjacent rows of one column, which are adjacent in the mirror image
    if (mbase) {
        __syncthreads();
#pragma unroll
        for (int b = 0; b < BLOCKS; ++b) {
            const int i = i0 + 32 * (b / TN) + q8, j = j0 + 32 * (b % TN) + r32;
            const int e0 = diag_tile ? max(0, j + 1 - i) : 0, e1 = min(4, P.M - i);
            if (j >= P.N || e0 >= e1) continue;
            const Global<float> dst = mbase + (long long)j * ldm + i;
            gd_floatx4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = part[gd_place(b, q8 + e, r32)];
            if (e0 == 0 && e1 == 4) *(Global<gd_floatx4_u>)dst = v;
            else
                for (int e = e0; e < e1; ++e) dst[e] = v[e];
        }
    }
}

hipError_t launch_gemm_direct(const GemmProblem *probs_dev, const int *tile_start_dev, int n_probs, int total_wgs,
                              int tile_cfg, int k_max, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    // A wavefront's share of up to 320 columns is 5 steps, all requested at once (142 registers, 3 workgroups a compute unit);
    // longer contractions go round the ring anyway and are better off with 4 (126 registers, 4 workgroups).
    if (tile_cfg == 2 && k_max <= 320) gemm_direct_kernel<1, 1, 5><<<dim3(total_wgs), dim3(256), 0, s>>>(probs_dev, tile_start_dev, n_probs);
    else if (tile_cfg == 2)            gemm_direct_kernel<1, 1, 4><<<dim3(total_wgs), dim3(256), 0, s>>>(probs_dev, tile_start_dev, n_probs);
    else                               gemm_direct_kernel<2, 2, 2><<<dim3(total_wgs), dim3(256), 0, s>>>(probs_dev, tile_start_dev, n_probs);
    return hipGetLastError();
}

}  // namespace kfac
