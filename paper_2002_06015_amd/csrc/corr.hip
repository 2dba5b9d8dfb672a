// The A factor of a 3x3 / stride 1 / pad 1 convolution without the patch matrix (Sec. 3.3,
// Eq. 10 and 11 define A = 1/(N hw) sum_n M_A M_A^T with M_A = im2col).  Entry
// ((c,ky,kx), (c',ky',kx')) of the sum is
//     sum_n sum_{(y,x)} a_c(n, y+ky-1, x+kx-1) a_c'(n, y+ky'-1, x+kx'-1)     (a = 0 outside)
// and, with u = (y+ky-1, x+kx-1) and D = (ky'-ky, kx'-kx), equals the full spatial
// cross-correlation  C_D[c,c'] = sum_n sum_u a_c(n,u) a_c'(n,u+D)  except that
//     ky = ky' = 2 leaves out the image row u_y = 0,   ky = ky' = 0 the row u_y = H-1,
//     kx = kx' = 2 leaves out the column u_x = 0,      kx = kx' = 0 the column u_x = W-1
// (every other bound on u coincides with u and u+D lying in the image).  So instead of the
// 81 C^2 products of the patch Gram matrix, 13 displacements D (the other 12 are transposes)
// are contracted over the image, plus corrections from the four border lines (1-D
// correlations) and the four corners (inclusion-exclusion), all by the grouped GEMM kernel:
//   - pad_kernel rewrites the activations as planes of Hp x Wp with (at least) two zero rows on
//     top and two zero columns on the left of each plane.  Because the planes follow each
//     other in memory, every position just outside an image (up to 2 away) is a zero of the
//     same or the next plane, and a(n, u+D) is simply the element dy*Wp+dx further on: a
//     shifted operand is the same buffer with an offset base pointer, no masks.
//     It also extracts the border lines [C][N][L+pad] and corners [C][N] for the corrections.
//   - assemble_kernel combines the 13 + 12 + 4 small Gram matrices into A (with the running
//     average and the bias border, whose sums come from the GEMM_BORDER row sums).
#include "kfac_internal.h"

namespace kfac {

typedef float corr_floatx4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void pad_kernel(const PadJob *__restrict__ jobs, int n_jobs)
{
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const PadJob &J = jobs[lo];
    const long long idx = (long long)(wg - J.wg_start) * 256 + threadIdx.x;
    const int H = J.H, W = J.W, Wp = J.Wp, PP = J.Hp * Wp, y0 = J.Hp - H, x0 = Wp - W;
    const long long planes = (long long)J.N * J.C;
    // Part 1: the padded tensor including its zero slack in front and behind, 4 elements per thread.  Instructions bound it, not
    // memory (4 bytes read and written per position).  The coordinates come from multiplications by precomputed reciprocals, and
    // the group's source is one run of 4 elements with the columns left of the image zeroed by value: one 16-byte load instead
    // of four.  Where the group runs into the next row, the elements there are zero columns again, but for the last one of a
    // group that starts in the last column where there are only two of them.  ResNet-50, batch 128 (32): 452 us (105), 528 (127)
    // with divisions and single loads here and in part 2.
    const long long n4 = J.padded_floats / 4;
    const Global<const float> src = global(J.src);
    if (idx < n4) {
        typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
        // (total and the front slack are multiples of 4: a group lies inside the planes or outside as a whole)
        const long long g0 = idx * 4 - J.front_slack, total = planes * PP;
        corr_floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (g0 >= 0 && g0 < total) {
            long long plane;
            int r, yp;
            if (J.magic_pp) {
                const unsigned q = (unsigned)__umul64hi((unsigned)g0, J.magic_pp);
                plane = q;
                r = (int)((unsigned)g0 - q * (unsigned)PP);
                yp = (int)__umulhi((unsigned)r, J.magic_w);
            } else {
                plane = g0 / PP;
                r = (int)(g0 - plane * PP);
                yp = r / Wp;
            }
            const int xp = r - yp * Wp;
            const Global<const float> sp = src + plane * H * W;
            if (yp >= y0) {
                const int c0 = xp - x0;                                     // source column of the first element
                const int o = (yp - y0) * W + c0;
                if ((plane > 0 || o >= 0) && (plane + 1 < planes || o + 4 <= H * W)) {
                    const floatx4_u x = *(Global<const floatx4_u>)(sp + o);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = c0 + e >= 0 && c0 + e < W ? x[e] : 0.f;
                } else {                                                    // first and last groups of the tensor
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c0 + e >= 0 && c0 + e < W) v[e] = sp[o + e];
                }
            }
            if (xp == Wp - 1 && x0 == 2 && yp + 1 >= y0 && yp + 1 < J.Hp) v[3] = sp[(yp + 1 - y0) * W];
        }
        *(Global<corr_floatx4>)(global(J.padded) + idx * 4) = v;
        return;
    }
    // Part 2: border rows (top, bottom) [2][C][N][Lw], border columns (left, right) [2][C][N][Lh], 4 elements of a line per thread
    // (every line ends in at least two zeros, four more follow the last one), then the corners [4][C][N].  Half the threads of a
    // 14 x 14 layer: with an element per thread and 64-bit divisions they took longer than part 1.
    const unsigned k0 = (unsigned)(idx - n4), CN = (unsigned)(J.C * J.N);
    auto line = [&](unsigned k, unsigned per, float *out, int len, auto source) {   // k: group of 4; per: groups of a line
        const unsigned l = k / per, q0 = 4 * (k - l * per);
        corr_floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (l < 2 * CN) {
            const unsigned which = l >= CN ? 1 : 0, cn = l - which * CN, c = cn / (unsigned)J.N, n = cn - c * (unsigned)J.N;
            const Global<const float> sp = src + ((long long)n * J.C + c) * H * W;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((int)q0 + e < len) v[e] = source(sp, which, (int)q0 + e);
        }
        *(Global<corr_floatx4>)(global(out) + 4LL * k) = v;
    };
    const unsigned rows4 = 2 * CN * (J.Lw / 4) + 1, cols4 = 2 * CN * (J.Lh / 4) + 1;
    if (k0 < rows4) {
        line(k0, J.Lw / 4, J.rows, W, [&](Global<const float> sp, unsigned which, int q) { return sp[(which ? H - 1 : 0) * W + q]; });
    } else if (k0 - rows4 < cols4) {
        line(k0 - rows4, J.Lh / 4, J.cols, H, [&](Global<const float> sp, unsigned which, int q) { return sp[q * W + (which ? W - 1 : 0)]; });
    } else if (k0 - rows4 - cols4 < 4 * CN) {
        const unsigned k = k0 - rows4 - cols4, which = k / CN, cn = k - which * CN, c = cn / (unsigned)J.N, n = cn - c * (unsigned)J.N;
        global(J.corners)[k] = src[((long long)n * J.C + c) * H * W + (which & 2 ? H - 1 : 0) * W + (which & 1 ? W - 1 : 0)];
    }
}

hipError_t launch_pad(const PadJob *jobs_dev, int n_jobs, int total_wgs, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    pad_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs);
    return hipGetLastError();
}

// bf16 activations: see PadJobBF16.  8 elements (16 bytes) per thread.
typedef unsigned short corr_ushortx8 __attribute__((ext_vector_type(8)));
typedef unsigned short corr_ushortx8_u __attribute__((ext_vector_type(8), aligned(2)));
typedef unsigned short corr_ushortx4_u __attribute__((ext_vector_type(4), aligned(2)));

__global__ __launch_bounds__(256) void pad_bf16_kernel(const PadJobBF16 *__restrict__ jobs, int n_jobs)
{
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const PadJobBF16 &J = jobs[lo];
    long long idx = (long long)(wg - J.wg_start) * 256 + threadIdx.x;
    const int H = J.H, W = J.W, Wp = J.Wp, PP = J.Hp * Wp, y0 = J.Hp - H, x0 = Wp - W;
    const long long planes = (long long)J.N * J.C;
    // part 1: the five shifted copies of the padded tensor.  One thread per aligned group of 8 positions: it takes the 12
    // values P(g - 2 .. g + 9) once and writes the group of every copy from that window.  HBM bound (2 bytes read and 10
    // written per position).  Wp is a multiple of 8, so a group lies in one row, and the positions around it that lie in
    // another row are zeros but for the last two columns of the row before the first group (which precede that group's row
    // in the source, too): the window is a run of 12 source elements with the columns outside the image zeroed by value,
    // two loads instead of twelve (ResNet-50, batch 32: 173 us, 200 with twelve).  Element-aligned 16-byte accesses.
    const long long per_copy = J.copy_elems / 8;
    const Global<const unsigned short> src = global(J.src);
    if (idx < per_copy) {
        const long long g = idx * 8 - J.front_slack, total = planes * PP;
        unsigned short win[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) win[e] = 0;
        if (g >= 0 && g <= total) {
            long long plane;
            int r;
            if (total < (1LL << 31)) {
                const unsigned q = (unsigned)g / (unsigned)PP;
                plane = q;
                r = (int)((unsigned)g - q * (unsigned)PP);
            } else {
                plane = g / PP;
                r = (int)(g - plane * PP);
            }
            const int yp = (int)((unsigned)r / (unsigned)Wp), xp = r - yp * Wp;
            const long long row = plane * H * W + (long long)max(0, yp - y0) * W;   // source row of the group
            if (g < total && yp >= y0) {
                const int c0 = xp - x0 - 2;                                      // source column of win[0]
                const long long o = row + c0;
                if (o >= 0 && o + 12 <= planes * H * W) {
                    const corr_ushortx8_u lo8 = *(Global<const corr_ushortx8_u>)(src + o);
                    const corr_ushortx4_u hi4 = *(Global<const corr_ushortx4_u>)(src + o + 8);
#pragma unroll
                    for (int e = 0; e < 12; ++e) {
                        const unsigned short x = e < 8 ? lo8[e & 7] : hi4[e & 3];
                        win[e] = c0 + e >= 0 && c0 + e < W ? x : (unsigned short)0;
                    }
                } else {                                                         // first and last groups of the tensor
#pragma unroll
                    for (int e = 0; e < 12; ++e)
                        if (c0 + e >= 0 && c0 + e < W) win[e] = src[o + e];
                }
            }
            // (yp == 0: the row before is the last one of the plane before; rows 1 .. y0 follow zero rows)
            if (xp == 0 && (yp > y0 || (yp == 0 && plane > 0))) {
                win[0] = src[row - 2];
                win[1] = src[row - 1];
            }
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            corr_ushortx8 v;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = win[q + e];
            *(Global<corr_ushortx8>)(global(J.padded) + (long long)q * J.copy_elems + idx * 8) = v;
        }
        return;
    }
    idx -= per_copy;
    // part 2: border rows, three copies shifted by 0, 1, 2 (one element per thread from here on)
    if (idx < 3 * J.rows_elems) {
        const int d = (int)(idx / J.rows_elems);
        const long long k = idx - d * J.rows_elems + d;      // copy d at position p holds the line buffer at p + d
        const long long row_elems = (long long)J.C * J.N * J.Lw;
        unsigned short x = 0;
        if (k < 2 * row_elems) {
            const int which = (int)(k / row_elems);
            const long long r = k - which * row_elems;
            const int qx = (int)(r % J.Lw);
            const long long cn = r / J.Lw;
            const int n = (int)(cn % J.N), c = (int)(cn / J.N);
            if (qx < W) x = src[((long long)n * J.C + c) * H * W + (long long)(which ? H - 1 : 0) * W + qx];
        }
        global(J.rows)[idx] = x;
        return;
    }
    idx -= 3 * J.rows_elems;
    if (idx < 3 * J.cols_elems) {
        const int d = (int)(idx / J.cols_elems);
        const long long k = idx - d * J.cols_elems + d;
        const long long col_elems = (long long)J.C * J.N * J.Lh;
        unsigned short x = 0;
        if (k < 2 * col_elems) {
            const int which = (int)(k / col_elems);
            const long long r = k - which * col_elems;
            const int py = (int)(r % J.Lh);
            const long long cn = r / J.Lh;
            const int n = (int)(cn % J.N), c = (int)(cn / J.N);
            if (py < H) x = src[((long long)n * J.C + c) * H * W + (long long)py * W + (which ? W - 1 : 0)];
        }
        global(J.cols)[idx] = x;
        return;
    }
    idx -= 3 * J.cols_elems;
    if (idx < 4LL * J.C * J.Ln) {
        const int which = (int)(idx / ((long long)J.C * J.Ln));
        const long long r = idx - (long long)which * J.C * J.Ln;
        const int n = (int)(r % J.Ln), c = (int)(r / J.Ln);
        const int py = (which & 2) ? H - 1 : 0, qx = (which & 1) ? W - 1 : 0;
        global(J.corners)[idx] = n < J.N ? src[((long long)n * J.C + c) * H * W + (long long)py * W + qx] : (unsigned short)0;
    }
}

hipError_t launch_pad_bf16(const PadJobBF16 *jobs_dev, int n_jobs, int total_wgs, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    pad_bf16_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs);
    return hipGetLastError();
}

// One workgroup per row i = (c, ky, kx) of A (plus one for the bias row), threads along the row.
// Which Gram matrices entry (c', ky', kx') comes from depends only on (ky, kx, ky', kx'): the
// workgroup first builds that table of 9 entries.  A displacement that is stored the other way
// round is read from the transposed copy the GEMM wrote alongside, so every read is along a
// row of a Gram matrix and every write along the row of A (the interleaving of the nine k'
// goes through LDS).
//
// What bounds it is the time of a workgroup, a chain of memory latencies (eight of them share a compute unit: 512 channels are 2.2
// rounds).  So a thread issues all loads of a channel, nine products, up to seven corrections and the old elements of A, before it
// waits for one, and the rows of a channel share an XCD.  512 channels in fp32 88 -> 73 us (222 MB, 3.0 TB/s), ResNet-50's 3x3
// layers 130 -> 93 (with a branch and a wait per correction, and rows dealt out in order).  Sources from scalar registers instead of the
// table are four levels of dependent loads: 110, and 64 channels 1 us more.
struct CorrSource {
    Global<const float> full, row, col, corner;   // row / col / corner: null if no such correction
    int ld_full, ld_row, ld_col;
};

__device__ __forceinline__ CorrSource corr_source(const AssembleJob &J, int ky, int kx, int kyp, int kxp)
{
    CorrSource S{};
    const int dy = kyp - ky, dx = kxp - kx;
    const bool fwd = dy > 0 || (dy == 0 && dx >= 0);
    const int ey = fwd ? dy : -dy, ex = fwd ? dx : -dx;
    const int slot = ey == 0 ? ex : 3 + (ey - 1) * 5 + (ex + 2);
    S.full = global(fwd ? J.full[slot] : J.full_t[slot]);
    S.ld_full = J.ld_full[slot];
    const int row_out = (ky == kyp) ? (ky == 2 ? 0 : (ky == 0 ? 1 : -1)) : -1;   // 0: top row left out, 1: bottom
    const int col_out = (kx == kxp) ? (kx == 2 ? 0 : (kx == 0 ? 1 : -1)) : -1;   // 0: left column, 1: right
    if (row_out >= 0) {
        const int d = dx >= 0 ? dx : -dx;
        S.row = global(dx >= 0 ? J.rows[row_out][d] : J.rows_t[row_out][d]);
        S.ld_row = J.ld_rows[row_out][d];
    }
    if (col_out >= 0) {
        const int d = dy >= 0 ? dy : -dy;
        S.col = global(dy >= 0 ? J.cols[col_out][d] : J.cols_t[col_out][d]);
        S.ld_col = J.ld_cols[col_out][d];
    }
    if (row_out >= 0 && col_out >= 0) S.corner = global(J.corners[2 * row_out + col_out]);
    return S;
}

// sum of the patch row (c, ky, kx) over all positions: the bias border
__device__ __forceinline__ float corr_row_sum(const AssembleJob &J, int c, int ky, int kx)
{
    const int row_out = ky == 2 ? 0 : (ky == 0 ? 1 : -1), col_out = kx == 2 ? 0 : (kx == 0 ? 1 : -1);
    float v = global(J.full[0])[(long long)c * J.ld_full[0] + J.C];
    if (row_out >= 0) v -= global(J.rows[row_out][0])[(long long)c * J.ld_rows[row_out][0] + J.C];
    if (col_out >= 0) v -= global(J.cols[col_out][0])[(long long)c * J.ld_cols[col_out][0] + J.C];
    if (row_out >= 0 && col_out >= 0) v += global(J.corners[2 * row_out + col_out])[(long long)c * J.ld_corner + J.C];
    return v;
}

__device__ __forceinline__ void corr_store(const AssembleJob &J, Global<float> out, float v)
{
    float r = J.alpha * v;
    if (J.beta != 0.f) r = fmaf(J.beta, *out, r);
    *out = r;
}

__global__ __launch_bounds__(256) void assemble_kernel(const AssembleJob *__restrict__ jobs, int n_jobs)
{
    const int wg = blockIdx.x;
    int lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (jobs[mid].wg_start <= wg) lo = mid; else hi = mid;
    }
    const AssembleJob &J = jobs[lo];
    const int d0 = 9 * J.C;
    int i = wg - J.wg_start;                // row of A
    // the nine rows of a channel, which read the same rows of the products, go to one XCD (as far as 8 divides the channels); not
    // where the products fit an L2 and the launch is one round of latencies (64 channels: 10.2 us without, 11.1 with)
    if (J.C >= 256 && i < J.C / 8 * 72) i = 9 * (i / 72 * 8 + (i & 7)) + (i / 8) % 9;
    const Global<float> out_row = global(J.A) + (long long)i * J.ldA;
    if (i < d0) {
        const int c = i / 9, k = i - 9 * c, ky = k / 3, kx = k - 3 * ky;
        typedef float v4 __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte access, element alignment
        __shared__ CorrSource src[9];
        __shared__ float vals[9][257];   // 256 channels c' at a time: [k'][c']
        if (threadIdx.x < 9) src[threadIdx.x] = corr_source(J, ky, kx, threadIdx.x / 3, threadIdx.x % 3);
        __syncthreads();
        for (int cp0 = 0; cp0 < J.C; cp0 += 256) {
            const int cp = cp0 + threadIdx.x, nout = 9 * min(256, J.C - cp0);
            const Global<float> dst = out_row + 9 * cp0;
            float full[9], row[3], col[3], corner = 0.f;
            v4 old[3];
            if (cp < J.C) {
#pragma unroll
                for (int kp = 0; kp < 9; ++kp) full[kp] = src[kp].full[(long long)c * src[kp].ld_full + cp];
                if (ky != 1)
#pragma unroll
                    for (int q = 0; q < 3; ++q) row[q] = src[3 * ky + q].row[(long long)c * src[3 * ky + q].ld_row + cp];
                if (kx != 1)
#pragma unroll
                    for (int q = 0; q < 3; ++q) col[q] = src[3 * q + kx].col[(long long)c * src[3 * q + kx].ld_col + cp];
                if (ky != 1 && kx != 1) corner = src[k].corner[(long long)c * J.ld_corner + cp];
            }
            if (J.beta != 0.f)
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    const int e = 4 * threadIdx.x + 1024 * m;
                    if (e + 3 < nout) old[m] = *(Global<const v4>)(dst + e);
                }
            if (cp < J.C) {
#pragma unroll
                for (int kp = 0; kp < 9; ++kp) {
                    float v = full[kp];
                    if (ky != 1 && kp / 3 == ky) v -= row[kp % 3];
                    if (kx != 1 && kp % 3 == kx) v -= col[kp / 3];
                    if (ky != 1 && kx != 1 && kp == k) v += corner;
                    vals[kp][threadIdx.x] = v;
                }
            }
            __syncthreads();
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const int e = 4 * threadIdx.x + 1024 * m;
                if (e + 3 < nout) {
                    v4 r;
#pragma unroll
                    for (int q = 0; q < 4; ++q) r[q] = J.alpha * vals[(e + q) % 9][(e + q) / 9];
                    if (J.beta != 0.f)
#pragma unroll
                        for (int q = 0; q < 4; ++q) r[q] = fmaf(J.beta, old[m][q], r[q]);
                    *(Global<v4>)(dst + e) = r;
                } else {
                    for (int q = 0; e + q < nout; ++q) corr_store(J, dst + e + q, vals[(e + q) % 9][(e + q) / 9]);
                }
            }
            __syncthreads();
        }
        if (J.bias && threadIdx.x == 0) corr_store(J, out_row + d0, corr_row_sum(J, c, ky, kx));
    } else {
        // the bias row
        for (int j = threadIdx.x; j <= d0; j += 256) {
            const int c = j / 9, k = j - 9 * c;
            corr_store(J, out_row + j, j < d0 ? corr_row_sum(J, c, k / 3, k % 3) : J.count);
        }
    }
}

hipError_t launch_assemble(const AssembleJob *jobs_dev, int n_jobs, int total_wgs, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    assemble_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(jobs_dev, n_jobs);
    return hipGetLastError();
}

}  // namespace kfac
