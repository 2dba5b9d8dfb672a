// Grouped "NT" GEMM on the gfx950 matrix cores: for every problem in a device table,
//     C[i][j] = alpha * sum_m a(i, m) * b(j, m) + beta * C[i][j]
// where both operands have their rows along the contraction index (see Operand).
// This one kernel carries every dense contraction of the K-FAC step:
//   - the Kronecker factors A = E[M_A M_A^T], G = E[D D^T] (Sec. 3.3, Eq. 9 and 11):
//     a == b, only lower-triangle tiles are computed and mirrored, the running average
//     is the alpha/beta epilogue, long contractions are split along K into partial tiles
//     that a second kernel sums in a fixed order (bitwise reproducible);
//   - the Schur-complement products of the blocked inverse (Eq. 12);
//   - the two products of the preconditioned gradient G^-1 dW A^-1 (Eq. 6).
//
// Tiling: a 256-thread workgroup (2x2 wavefronts of 64) owns a BM x BN tile; each wavefront owns TM x TN blocks of 32x32.  The
// contraction runs in tiles staged through LDS.  The matrix instructions of a block product:
//   - bf16 operands: v_mfma_f32_32x32x16_bf16;
//   - fp32 operands by default: v_mfma_f32_32x32x16_f16 on two fp16 planes of each (three per 16 k), or the bf16 one on three bf16
//     planes (six) where those do not serve and for operands stored transposed;
//   - fp32 operands on request: v_mfma_f32_32x32x2_f32.
#include "gemm_tiles.h"
#include <type_traits>

namespace kfac {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short ushortx8 __attribute__((ext_vector_type(8)));
typedef unsigned short ushortx4 __attribute__((ext_vector_type(4)));

constexpr int KT = 32;      // contraction tile
constexpr int LDF = 36;     // LDS row length in floats (32 + 4 pad: conflict-free 16-byte reads)

// operand stages, then the output tile
template <int TM, int TN>
constexpr size_t gemm_lds_bytes()
{
    const size_t stages = 2 * (64 * TM + 64 * TN) * LDF * sizeof(float);   // same size for LDH bf16 rows
    const size_t tile = (size_t)(64 * TM) * (64 * TN + 1) * sizeof(float);
    return stages > tile ? stages : tile;
}

// the same for the kernel of the products through planes: two stages of two fp16 planes or one of three bf16 planes; the scales
// and floors of the rows, two flags and the list of sums in doubt lie behind
constexpr int kMaxDoubts = 128;      // sums of a tile formed again one by one (see the two fp16 planes)
template <int TM, int TN>
constexpr size_t split_lds_bytes()
{
    constexpr size_t rows = 64 * TM + 64 * TN;
    const size_t two = 2 * 2 * rows * 32 * 2, three = 3 * rows * 40 * 2, tile = 64 * TM * (64 * TN + 1) * sizeof(float);
    const size_t most = two > three ? (two > tile ? two : tile) : (three > tile ? three : tile);
    return (most + 15) / 16 * 16 + (2 * rows + 2 + 1 + kMaxDoubts) * sizeof(float);
}

// Final write of a ROWS x COLS slab of accumulated sums held in LDS (T[r][c] at
// T[r * (COLS + 1) + c], global position (gi0 + r, gj0 + c)):
//     C[i][j] = alpha * T + beta * C[i][j]
// plus, for symmetric problems, the mirror image C[j][i] (for a tile on the diagonal only
// j <= i is written directly and j < i mirrored, which makes the result exactly symmetric),
// plus the optional transposed copy Ct[j][i].  Both passes write whole row segments with
// adjacent lanes on adjacent addresses; the transposition happens in the LDS reads.
// Of the old C (beta != 0) only the lower triangle is read.  Ct requires beta == 0.
typedef float floatx4_st __attribute__((ext_vector_type(4), aligned(4)));

template <int ROWS, int COLS>
__device__ __forceinline__ void store_slab(const GemmProblem &P, float *T, int gi0, int gj0, bool diag_tile, int tid)
{
    constexpr int LDT = COLS + 1;
    const bool sym = (P.flags & GEMM_SYM) != 0;
    const float alpha = P.alpha, beta = P.beta;
    const Global<float> C = global(P.C), mbase = global(!sym ? P.Ct : gi0 - gj0 - (COLS - 1) < P.mirror_band ? P.C : nullptr);
    // direct pass: a thread owns 4 adjacent columns of one row.  The old values (beta != 0) of all its rows are requested
    // before the first store: a load issued behind a store to the same matrix waits for it, and load - store pairs then
    // cost one memory round trip per row.
    {
        constexpr int TPR = COLS / 4, RPP = 256 / TPR, NIT = (ROWS + RPP - 1) / RPP;
        const int c = (tid % TPR) * 4, rr = tid / TPR;
        const int j = gj0 + c;
        floatx4 old[NIT];
        if (beta != 0.0f) {
#pragma unroll
            for (int q = 0; q < NIT; ++q) {
                const int r = rr + q * RPP, i = gi0 + r;
                const int jmax = min(diag_tile ? i : P.N - 1, P.N - 1);
                old[q] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (r < ROWS && i < P.M && j + 3 <= jmax) old[q] = *(Global<const floatx4_st>)(C + (long long)i * P.ldc + j);
            }
        }
#pragma unroll
        for (int q = 0; q < NIT; ++q) {
            const int r = rr + q * RPP, i = gi0 + r;
            if (r >= ROWS || i >= P.M || j >= P.N) continue;
            const int jmax = min(diag_tile ? i : P.N - 1, P.N - 1);   // last column this row may write
            if (j > jmax) continue;
            const Global<float> dst = C + (long long)i * P.ldc + j;
            float *t = T + r * LDT + c;
            if (j + 3 <= jmax) {
                floatx4 v = {alpha * t[0], alpha * t[1], alpha * t[2], alpha * t[3]};
                if (beta != 0.0f)
                    for (int e = 0; e < 4; ++e) v[e] = fmaf(beta, old[q][e], v[e]);   // same rounding in every path
                *(Global<floatx4_st>)dst = v;
                if (mbase)
                    for (int e = 0; e < 4; ++e) t[e] = v[e];
            } else {
                for (int e = 0; e < 4 && j + e <= jmax; ++e) {
                    float v = alpha * t[e];
                    if (beta != 0.0f) v = fmaf(beta, dst[e], v);
                    dst[e] = v;
                    t[e] = v;
                }
            }
        }
    }
    // mirrored / transposed pass over the values of the direct pass, left in T: a thread owns 4 adjacent rows i of one
    // column j, which are 4 adjacent addresses of row j of the mirror image
    if (mbase) {
        __syncthreads();
        const long long ldm = sym ? P.ldc : P.ldct;
        constexpr int TPR = ROWS / 4, RPP = 256 / TPR, NIT = (COLS + RPP - 1) / RPP;
        const int r = (tid % TPR) * 4, cc = tid / TPR;
        const int i = gi0 + r;
#pragma unroll
        for (int q = 0; q < NIT; ++q) {
            const int c = cc + q * RPP, j = gj0 + c;
            if (c >= COLS || i >= P.M || j >= P.N) continue;
            // rows i..i+3 that may be mirrored: i + e < M and, on a diagonal tile, j < i + e
            const int e0 = (sym && diag_tile) ? max(0, j + 1 - i) : 0;
            const int e1 = min(4, P.M - i);
            if (e0 >= e1) continue;
            const Global<float> dst = mbase + (long long)j * ldm + i;
            const float *t = T + r * LDT + c;
            if (e0 == 0 && e1 == 4) *(Global<floatx4_st>)dst = floatx4{t[0], t[LDT], t[2 * LDT], t[3 * LDT]};
            else
                for (int e = e0; e < e1; ++e) dst[e] = t[e * LDT];
        }
    }
}

// Border of a GEMM_BORDER problem: entry `row` of the extra row / column from the row sum
// of the operand, and the corner from the contraction length.
__device__ __forceinline__ void store_border(const GemmProblem &P, int row, float sum)
{
    const Global<float> C = global(P.C), pr = C + (long long)P.M * P.ldc + row;
    float v = P.alpha * sum;
    if (P.beta != 0.0f) v = fmaf(P.beta, *pr, v);
    *pr = v;
    C[(long long)row * P.ldc + P.M] = v;
}
__device__ __forceinline__ void store_corner(const GemmProblem &P)
{
    const Global<float> pc = global(P.C) + (long long)P.M * P.ldc + P.M;
    float v = P.alpha * (float)P.ones;
    if (P.beta != 0.0f) v = fmaf(P.beta, *pc, v);
    *pc = v;
}

// ------------------------------------------------------------------ operand loader (fp32)
// A thread owns one 4-wide k chunk (kq = 4 * (tid % 8)) of the rows r0 + 32*s (r0 = tid / 8)
// of the operand tile.  A chunk is one 16-byte load that only needs 4-byte alignment (any
// leading dimension works); the host guarantees that the 4 elements of a chunk are adjacent
// in memory (hw % 4 == 0 for NCHW operands).  Every load of the main loop has an
// unconditionally valid address and is masked by value afterwards, so the loads of a whole
// tile are issued back to back:
//   - rows outside the operand are clamped to its last row and replaced by 0;
//   - the contraction range of a workgroup is cut into full 32-wide tiles; a remaining
//     multiple of 4 is covered by one more full tile shifted back to end at the range end,
//     whose already-counted k positions are zeroed in ONE operand;
//   - a remaining K % 4 (only plain matrices have one) is added in the epilogue.
// Ranges shorter than 32 take a slow, careful tile instead.
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef const float __attribute__((address_space(1))) *gfloat_ptr;
typedef const floatx4_u __attribute__((address_space(1))) *gfloat4_ptr;

template <int BR>
struct LoaderF32 {
    static constexpr int SLOTS = BR / 32;
    gfloat_ptr base;
    long long rowoff[SLOTS];   // clamped row * row_stride (loop invariant)
    unsigned dead;             // bit s: slot row is outside the operand
    long long batch_stride;
    long long col;             // offset of the thread's chunk within a row: n * batch_stride + t
    int hw, kq, r0, t;
    int m;                     // first k of the chunk, as of the last seek
    bool zero_all;             // the tile held in registers is to be stored as zeros

    __device__ __forceinline__ void init(const Operand &op, int tile_row0, int tid)
    {
        base = (gfloat_ptr)op.base;
        batch_stride = op.batch_stride;
        hw = op.hw;
        kq = (tid & 7) * 4; r0 = tid >> 3;
        dead = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int row = tile_row0 + r0 + 32 * s;
            if (row >= op.rows) dead |= 1u << s;
            rowoff[s] = (long long)min(row, op.rows - 1) * op.row_stride;
        }
        m = t = 0;
        col = 0;
        zero_all = false;
    }
    __device__ __forceinline__ void seek(int tile_k0)   // position on the tile starting at tile_k0
    {
        m = tile_k0 + kq;
        const int n = m < hw ? 0 : m / hw;   // (plain matrices: one run)
        t = m - n * hw;
        col = (long long)n * batch_stride + t;
    }
    __device__ __forceinline__ void advance()
    {
        t += KT; col += KT;
        while (t >= hw) { t -= hw; col += batch_stride - hw; }
    }
    // the same for runs of at least one tile (hw >= KT): at most one wrap, no branch
    __device__ __forceinline__ void advance_once()
    {
        t += KT; col += KT;
        const bool wrap = t >= hw;
        t -= wrap ? hw : 0;
        col += wrap ? batch_stride - hw : 0;
    }
    // Raw loads only: the masks are applied in store_lds, one iteration later, so nothing
    // waits for the data before the matrix instructions of the current tile are issued.
    __device__ __forceinline__ void load_full(floatx4 (&reg)[SLOTS])
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) reg[s] = *(gfloat4_ptr)(base + rowoff[s] + col);
        zero_all = false;
    }
    // the shifted tile: k positions below mlo were already covered by the full tiles
    __device__ __forceinline__ void zero_below(int mlo) { zero_all = m < mlo; }
    // careful tile for short ranges: chunks at or beyond kend4 are not read
    __device__ __forceinline__ void load_careful(floatx4 (&reg)[SLOTS], int kend4)
    {
        const bool in = m < kend4;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (in) v = *(gfloat4_ptr)(base + rowoff[s] + col);
            reg[s] = v;
        }
        zero_all = !in;
    }
    // RS: also add what is stored to the running row sums rs[s] of the rows r0 + 32*s
    template <bool RS>
    __device__ __forceinline__ void store_lds(const floatx4 (&reg)[SLOTS], float *lds, float (&rs)[SLOTS]) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            floatx4 v = reg[s];
            if (((dead >> s) & 1) || zero_all) { v[0] = 0.f; v[1] = 0.f; v[2] = 0.f; v[3] = 0.f; }
            if constexpr (RS) rs[s] += (v[0] + v[1]) + (v[2] + v[3]);
            *(floatx4 *)(lds + (r0 + 32 * s) * LDF + kq) = v;
        }
    }
    // one slot of a tile without masked rows (dead == 0, not zero_all)
    template <bool RS>
    __device__ __forceinline__ void store_slot(const floatx4 (&reg)[SLOTS], float *lds, float (&rs)[SLOTS], int s) const
    {
        const floatx4 v = reg[s];
        if constexpr (RS) rs[s] += (v[0] + v[1]) + (v[2] + v[3]);
        *(floatx4 *)(lds + (r0 + 32 * s) * LDF + kq) = v;
    }
    __device__ __forceinline__ void load_slot(floatx4 (&reg)[SLOTS], int s)
    {
        reg[s] = *(gfloat4_ptr)(base + rowoff[s] + col);
    }
    // K % 4 remainder tile (plain matrices only: hw > K): thread tid < BR fills LDS row tid
    // with the elements k4 .. kend-1 of its operand row followed by zeros; returns their sum
    __device__ __forceinline__ static float fill_remainder(const Operand &op, int tile_row0, int k4, int kend,
                                                           int tid, float *lds)
    {
        if (tid >= BR) return 0.f;
        const int row = tile_row0 + tid;
        floatx4 x = {0.f, 0.f, 0.f, 0.f};
        if (row < op.rows) {
            gfloat_ptr p = (gfloat_ptr)op.base + (long long)row * op.row_stride + k4;
            for (int e = 0; e < 3; ++e)
                if (k4 + e < kend) x[e] = p[e];
        }
        float *dst = lds + tid * LDF;
        *(floatx4 *)dst = x;
#pragma unroll
        for (int q = 1; q < 8; ++q) *(floatx4 *)(dst + 4 * q) = floatx4{0.f, 0.f, 0.f, 0.f};
        return x[0] + x[1] + x[2];
    }
};

// Finishes the border row sums of a diagonal tile: adds up the 8 lanes that share a row,
// then either stores the border entries (splits == 1) or this split's partial sums.
// Uses the first BM floats of LDS; all 256 threads call it, between barriers of its own.
template <int BM>
__device__ __forceinline__ void finish_row_sums(const GemmProblem &P, float *lds, int tm, int tile, int split,
                                                int tid, float (&rs)[BM / 32], float rs_rem)
{
#pragma unroll
    for (int s = 0; s < BM / 32; ++s) {
        float v = rs[s];
        v += __shfl_xor(v, 1);
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 4);
        rs[s] = v;
    }
    __syncthreads();   // the operand stages are dead
    if ((tid & 7) == 0) {
#pragma unroll
        for (int s = 0; s < BM / 32; ++s) lds[(tid >> 3) + 32 * s] = rs[s];
    }
    __syncthreads();
    if (tid < BM) {
        const float total = lds[tid] + rs_rem;
        const int row = tm * BM + tid;
        if (P.splits > 1) global(P.partial_rs)[((long long)tm * P.splits + split) * BM + tid] = total;
        else if (row < P.M) store_border(P, row, total);
    }
    if (tile == 0 && tid == 0 && P.splits == 1) store_corner(P);
    __syncthreads();
}

// ------------------------------------------------------------------ fp32 kernel
// Software pipeline over the K tiles, two LDS stages, one barrier per tile.  While the matrix
// instructions of tile `it` run out of stage it & 1, the same wavefront
//   - stores tile it + 1 (held in registers since the previous iteration) into the other stage,
//   - issues the global loads of tile it + 2 into those registers,
//   - reads its operand fragments a quarter tile ahead of the matrix instructions,
// so that no wavefront depends on another one sharing its SIMD to keep the matrix pipe busy.
// The barrier sits before the last quarter: after it every wavefront has finished reading
// stage it & 1 up to the fragments it already holds, and has stored its part of tile it + 1,
// whose first fragments are read during the last quarter.
// RS: the row sums of the a-operand tile are accumulated on the side (rs: rows r0 + 32*s of
// the vector-loaded part, rs_rem: row tid of the K % 4 remainder).
template <int TM, int TN>
struct FragF32 {
    floatx4 a[TM], b[TN];
};

template <int TM, int TN>
__device__ __forceinline__ void read_frag(FragF32<TM, TN> &f, const float *pa, const float *pb, int q)
{
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = *(const floatx4 *)(pa + i * 32 * LDF + 4 * q);
#pragma unroll
    for (int j = 0; j < TN; ++j) f.b[j] = *(const floatx4 *)(pb + j * 32 * LDF + 4 * q);
}

template <int TM, int TN>
__device__ __forceinline__ void mma_frag(const FragF32<TM, TN> &f, floatx16 (&acc)[TM][TN])
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[i][e], f.b[j][e], acc[i][j], 0, 0, 0);
}

template <int TM, int TN, bool LIVE, bool RS>
__device__ __forceinline__ void gemm_f32_mainloop(const GemmProblem &P, int tm, int tn, int tid,
                                                  LoaderF32<64 * TM> &la, LoaderF32<64 * TN> &lb, float *lds,
                                                  int k0, int k1, int wave_m, int wave_n, int l32, int half,
                                                  floatx16 (&acc)[TM][TN], float (&rs)[2 * TM], float &rs_rem)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int STAGE = (BM + BN) * LDF;
    // [k0, k0 + klen4) is covered by vector-loaded tiles; a K % 4 remainder [k0 + klen4, k1)
    // exists only in the last split of a plain-matrix problem and gets a tile of its own
    const int klen = max(k1 - k0, 0);
    const int klen4 = klen & ~3;
    const int nfull = klen4 / KT;
    const bool shifted = nfull > 0 && klen4 > nfull * KT;   // one more full tile ending at k0 + klen4
    const bool careful = nfull == 0 && klen4 > 0;
    const int nvec = nfull + ((shifted || careful) ? 1 : 0);
    const int nk = nvec + (klen4 < klen ? 1 : 0);
    if (nk == 0) return;
    floatx4 ra[BM / 32], rb[BN / 32];

    // global loads of tile `it` into the staging registers (nothing beyond the vector tiles)
    auto load_tile = [&](int it) {
        if (it < nfull) {
            if (it > 0) { la.advance(); lb.advance(); }
            la.load_full(ra); lb.load_full(rb);
        } else if (it < nvec) {
            if (careful) {
                la.load_careful(ra, k0 + klen4); lb.load_careful(rb, k0 + klen4);
            } else {
                la.seek(k0 + klen4 - KT); lb.seek(k0 + klen4 - KT);
                la.load_full(ra); lb.load_full(rb);
                la.zero_below(k0 + nfull * KT);
            }
        }
    };
    // tile `it` (< nk) into its LDS stage: from the staging registers, or the K % 4 remainder
    auto store_tile = [&](int it) {
        float *sa = lds + (it & 1) * STAGE, *sb = sa + BM * LDF;
        if (it < nvec) {
            float unused[BN / 32];
            la.template store_lds<RS>(ra, sa, rs);
            lb.template store_lds<false>(rb, sb, unused);
        } else {
            rs_rem = LoaderF32<BM>::fill_remainder(P.a, tm * BM, k0 + klen4, k1, tid, sa);
            LoaderF32<BN>::fill_remainder(P.b, tn * BN, k0 + klen4, k1, tid, sb);
        }
    };
    // each half-wave takes 16 consecutive k of the tile (the same 16 for both operands)
    const int off_a = (wave_m * 32 * TM + l32) * LDF + half * 16;
    const int off_b = BM * LDF + (wave_n * 32 * TN + l32) * LDF + half * 16;

    la.seek(k0); lb.seek(k0);
    load_tile(0);
    store_tile(0);
    load_tile(1);
    __syncthreads();
    FragF32<TM, TN> f0, f1;
    if constexpr (LIVE) read_frag<TM, TN>(f0, lds + off_a, lds + off_b, 0);

    // One iteration of the general form: any kind of tile, stores and loads as blocks.
    auto step = [&](int it) {
        const float *cur = lds + (it & 1) * STAGE;
        const float *nxt = lds + ((it + 1) & 1) * STAGE;
        if constexpr (LIVE) read_frag<TM, TN>(f1, cur + off_a, cur + off_b, 1);
        if (it + 1 < nk) store_tile(it + 1);
        if constexpr (LIVE) mma_frag<TM, TN>(f0, acc);
        if constexpr (LIVE) read_frag<TM, TN>(f0, cur + off_a, cur + off_b, 2);
        load_tile(it + 2);
        if constexpr (LIVE) mma_frag<TM, TN>(f1, acc);
        if constexpr (LIVE) read_frag<TM, TN>(f1, cur + off_a, cur + off_b, 3);
        if constexpr (LIVE) mma_frag<TM, TN>(f0, acc);
        __syncthreads();
        if constexpr (LIVE) {
            if (it + 1 < nk) read_frag<TM, TN>(f0, nxt + off_a, nxt + off_b, 0);
            mma_frag<TM, TN>(f1, acc);
        }
    };
    // The steady state: tile it + 1 is a vector tile without masked rows and tile it + 2 a full
    // one reached by a single wrap of the position.  Straight-line code in a fixed order (the
    // scheduling barriers keep the compiler from regrouping it): the stores of tile it + 1 and
    // the loads of tile it + 2 are dealt out one by one behind the matrix instructions of the
    // first quarter, in whose shadow they issue; the loads then have the rest of the tile to
    // arrive, and every fragment read has a quarter.
    auto fast_step = [&](int it) {
        const float *cur = lds + (it & 1) * STAGE;
        float *nxt = lds + ((it + 1) & 1) * STAGE;
        constexpr int SA = BM / 32, SB = BN / 32, NOPS = 2 * (SA + SB);
        constexpr int NMMA = LIVE ? 4 * TM * TN : 1;
        constexpr int PER = (NOPS + NMMA - 1) / NMMA;
        auto side_op = [&](int k) {   // k-th of: stores of a, stores of b, loads of a, loads of b
            if (k < SA) {
                la.template store_slot<RS>(ra, nxt, rs, k);
            } else if (k < SA + SB) {
                float unused[SB];
                lb.template store_slot<false>(rb, nxt + BM * LDF, unused, k - SA);
            } else if (k < 2 * SA + SB) {
                if (k == SA + SB) { la.advance_once(); lb.advance_once(); }
                la.load_slot(ra, k - SA - SB);
            } else if (k < NOPS) {
                lb.load_slot(rb, k - 2 * SA - SB);
            }
        };
        if constexpr (LIVE) {
            read_frag<TM, TN>(f1, cur + off_a, cur + off_b, 1);
            __builtin_amdgcn_sched_barrier(0);
            int n = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f0.a[i][e], f0.b[j][e], acc[i][j], 0, 0, 0);
#pragma unroll
                        for (int u = 0; u < PER; ++u) side_op(n * PER + u);
                        ++n;
                        __builtin_amdgcn_sched_barrier(0);
                    }
            read_frag<TM, TN>(f0, cur + off_a, cur + off_b, 2);
            __builtin_amdgcn_sched_barrier(0);
            mma_frag<TM, TN>(f1, acc);
            __builtin_amdgcn_sched_barrier(0);
            read_frag<TM, TN>(f1, cur + off_a, cur + off_b, 3);
            __builtin_amdgcn_sched_barrier(0);
            mma_frag<TM, TN>(f0, acc);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            read_frag<TM, TN>(f0, nxt + off_a, nxt + off_b, 0);
            __builtin_amdgcn_sched_barrier(0);
            mma_frag<TM, TN>(f1, acc);
        } else {
#pragma unroll
            for (int k = 0; k < NOPS; ++k) side_op(k);
            __syncthreads();
        }
    };
    int it = 0;
    // (a condition the whole workgroup agrees on: every row of both operand tiles exists)
    if (la.hw >= KT && lb.hw >= KT && (tm + 1) * BM <= P.a.rows && (tn + 1) * BN <= P.b.rows)
        for (; it + 2 < nfull; ++it) fast_step(it);
    for (; it < nk; ++it) step(it);
}

// ------------------------------------------------------------------ fp32 through three bf16 planes
// The bf16 matrix instruction runs at 16 times the rate of the fp32 one.  An fp32 value is the
// exact sum of three bf16 values (8 + 8 + 8 significant bits: x = h + m + l by two truncations
// and two exact subtractions), and a product of two bf16 values is exact in fp32, so
//     x y  =  h h' + (h m' + m h') + (h l' + m m' + l h')  +  terms below 2^-23 |x y|
// with fp32 accumulation inside the matrix unit: six bf16 instructions give the product to
// fp32 accuracy in 6 x 32 cycles per 32x32x16 block instead of 8 x 64.  The operands stay fp32 in
// HBM; the loader of the fp32 kernel brings a K tile of 32 into registers and the split happens
// on the way into LDS, which holds one stage of three planes.  What the loop of two fp16 planes below
// leaves (and operands stored transposed).
constexpr int LDQ = 40;     // LDS row length in bf16 (32 + 8 pad: 80-byte rows, conflict-free 16-byte reads)
// Rows of a group of 8 are stored in the order 0 4 1 5 2 6 3 7: the 8-byte stores of 16 lanes cover two
// rows, and rows 80 bytes apart share 4 of their 16 banks while rows 4 apart (320 bytes) share none.  The
// fragment reads take the same 8 rows per group of lanes as before.
__device__ __forceinline__ int lds_row(int r) { return (r & ~7) | ((r & 1) << 2) | ((r >> 1) & 3); }

// the staged tile of one operand into its rows of the three planes (plane stride in bf16 units)
template <int BR, bool RS>
__device__ __forceinline__ void store_split(const LoaderF32<BR> &ld, const floatx4 (&reg)[BR / 32], unsigned short *rows,
                                            int plane, float (&rs)[BR / 32])
{
#pragma unroll
    for (int s = 0; s < BR / 32; ++s) {
        floatx4 v = reg[s];
        if (((ld.dead >> s) & 1) || ld.zero_all) { v[0] = 0.f; v[1] = 0.f; v[2] = 0.f; v[3] = 0.f; }
        if constexpr (RS) rs[s] += (v[0] + v[1]) + (v[2] + v[3]);
        uint2 h, m, l;
        split_pair(v[0], v[1], h.x, m.x, l.x);
        split_pair(v[2], v[3], h.y, m.y, l.y);
        unsigned short *dst = rows + (lds_row(ld.r0) + 32 * s) * LDQ + ld.kq;
        *(uint2 *)dst = h;
        *(uint2 *)(dst + plane) = m;
        *(uint2 *)(dst + 2 * plane) = l;
    }
}

// K % 4 remainder tile: thread tid < BR fills row tid of the three planes with the elements
// k4 .. kend-1 of its operand row followed by zeros; returns their sum
template <int BR>
__device__ __forceinline__ float fill_remainder_split(const Operand &op, int tile_row0, int k4, int kend, int tid,
                                                      unsigned short *rows, int plane)
{
    if (tid >= BR) return 0.f;
    const int row = tile_row0 + tid;
    float x[4] = {0.f, 0.f, 0.f, 0.f};
    if (row < op.rows) {
        gfloat_ptr p = (gfloat_ptr)op.base + (long long)row * op.row_stride + k4;
        for (int e = 0; e < 3; ++e)
            if (k4 + e < kend) x[e] = p[e];
    }
    uint2 v[3];
    split_pair(x[0], x[1], v[0].x, v[1].x, v[2].x);
    split_pair(x[2], x[3], v[0].y, v[1].y, v[2].y);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        unsigned short *dst = rows + q * plane + lds_row(tid) * LDQ;
        *(uint4 *)dst = uint4{v[q].x, v[q].y, 0u, 0u};
#pragma unroll
        for (int w = 1; w < 4; ++w) *(uint4 *)(dst + 8 * w) = uint4{0u, 0u, 0u, 0u};
    }
    return x[0] + x[1] + x[2];
}

template <int TM, int TN, bool LIVE, bool RS>
__device__ __forceinline__ void gemm_split_mainloop(const GemmProblem &P, int tm, int tn, int tid,
                                                    LoaderF32<64 * TM> &la,
                                                    LoaderF32<64 * TN> &lb, unsigned short *lds, int k0,
                                                    int k1, int wave_m, int wave_n, int l32, int half,
                                                    floatx16 (&acc)[TM][TN], float (&rs)[2 * TM], float &rs_rem)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int PLANE = (BM + BN) * LDQ;
    const int klen = max(k1 - k0, 0);
    const int klen4 = klen & ~3;
    const int nfull = klen4 / KT;
    const bool shifted = nfull > 0 && klen4 > nfull * KT;
    const bool careful = nfull == 0 && klen4 > 0;
    const int nvec = nfull + ((shifted || careful) ? 1 : 0);
    const int nk = nvec + (klen4 < klen ? 1 : 0);
    if (nk == 0) return;
    floatx4 ra[BM / 32], rb[BN / 32];
    la.seek(k0); lb.seek(k0);
    auto load_tile = [&](int it) {   // into registers, a tile ahead
        if (it < nfull) {
            if (it > 0) { la.advance(); lb.advance(); }
            la.load_full(ra); lb.load_full(rb);
        } else if (it < nvec && careful) {
            la.load_careful(ra, k0 + klen4); lb.load_careful(rb, k0 + klen4);
        } else if (it < nvec) {
            la.seek(k0 + klen4 - KT); lb.seek(k0 + klen4 - KT);
            la.load_full(ra); lb.load_full(rb);
            la.zero_below(k0 + nfull * KT);
        }
    };
    auto store_tile = [&](int it) {
        if (it == nvec) {
            rs_rem = fill_remainder_split<BM>(P.a, tm * BM, k0 + klen4, k1, tid, lds, PLANE);
            fill_remainder_split<BN>(P.b, tn * BN, k0 + klen4, k1, tid, lds + BM * LDQ, PLANE);
            return;
        }
        float unused[BN / 32];
        store_split<BM, RS>(la, ra, lds, PLANE, rs);
        store_split<BN, false>(lb, rb, lds + BM * LDQ, PLANE, unused);
    };
    // v_mfma_f32_32x32x16_bf16: a lane supplies 8 consecutive k of row lane % 32, the half-waves
    // two different groups of 8; step u of a tile uses k = 16u + 8*half + 0..7 for both operands
    const int off_a = (wave_m * 32 * TM + lds_row(l32)) * LDQ + 8 * half;
    const int off_b = BM * LDQ + (wave_n * 32 * TN + lds_row(l32)) * LDQ + 8 * half;
    // One step: the fragments of the h and m planes and of l' are requested up front, the l
    // fragments of the a operand take over the registers of h once its products are issued (their
    // latency lies under the m products).  Fixed order (the scheduling barriers keep the compiler
    // from hoisting the next step's reads, which would cost the second workgroup of the compute
    // unit its registers).
    auto compute = [&]() {
        if constexpr (LIVE) {
            auto rd = [&](int q, int off, int u) {
                return __builtin_bit_cast(bf16x8, *(const ushortx8 *)(lds + q * PLANE + off + 16 * u));
            };
            auto mm = [&](const bf16x8 (&x)[TM], const bf16x8 (&y)[TN]) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], y[j], acc[i][j], 0, 0, 0);
            };
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 ah[TM], am[TM], bh[TN], bm[TN], bl[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) ah[i] = rd(0, off_a + i * 32 * LDQ, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) bh[j] = rd(0, off_b + j * 32 * LDQ, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) bm[j] = rd(1, off_b + j * 32 * LDQ, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) bl[j] = rd(2, off_b + j * 32 * LDQ, u);
#pragma unroll
                for (int i = 0; i < TM; ++i) am[i] = rd(1, off_a + i * 32 * LDQ, u);
                __builtin_amdgcn_sched_barrier(0);
                mm(ah, bh);
                mm(ah, bm);
                mm(ah, bl);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TM; ++i) ah[i] = rd(2, off_a + i * 32 * LDQ, u);   // the l plane of a
                __builtin_amdgcn_sched_barrier(0);
                mm(am, bh);
                mm(am, bm);
                mm(ah, bh);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    load_tile(0);
    for (int it = 0; it < nk; ++it) {
        if (it > 0) __syncthreads();   // every wavefront has read the tile before
        store_tile(it);
        load_tile(it + 1);
        __syncthreads();
        compute();
    }
}

// ------------------------------------------------------------------ fp32 through two fp16 planes
// The main loop of the product mode (the one above is its fallback).  x s = h + l with s a power of two per operand row, h the
// fp16 value nearest to x s and l the one nearest to x s - h: 11 + 11 significant bits and the sign of l, so h + l is x s
// itself for three values of four and one unit of the 24th bit off for the fourth; with
//     x y  =  (h h' + h l' + l h') / (s s')  +  terms below 2^-22 |x y| of random sign
// three fp16 instructions do what took six bf16 ones.  What bounds the product is power: at the clock the chip holds under it
// (1.75 GHz) the six-instruction loop kept the matrix unit busy 0.54 of the time and did no more work at a higher share.  Half
// the matrix work, 2.5 instead of 5.5 vector instructions and 4 instead of 6 bytes of LDS a staged element:
// see the figures at gemm_nt_f32_split_kernel.  It is also the more accurate one, because the accumulator is rounded three
// times per 16 k instead of six.
//
// The range of fp16 is what the scale is for.  A workgroup takes it from its own rows, before its main loop: the largest of up
// to 128 elements of the row, 16 at each of eight places spread over the workgroup's part of the contraction (products with an
// inverse: 32 at each of four), goes to [2^t, 2^(t+1)).  (Rows that sample as zero are read on until an element is not; rows of
// an inverse also sample their diagonal.)
//   - Above, there is room to 2^16.  A row that goes beyond it leaves infinities or NaN in the accumulator, which costs nothing to
//     provide for: the workgroup finds them after its loop and repeats it in the three-plane mode, which has the range of fp32.
//     t = 6 leaves statistics a factor of 512 to 1024 (images and pixels differ), t = 10 the products with an inverse 32 to 64
//     (their largest element is mostly the diagonal one, and the others lie far below it).
//   - Below, elements down to 2^-2 (scaled) are exact as above, smaller ones to an absolute 2^-25, 2^-(t+25) of the largest.  That
//     is lost in the sum unless the large elements of a row meet zeros or tiny ones of the other, or one operand falls along k as
//     the other grows.  The result shows it: K terms off by at most 2^-25 2^t are within 2^-23 K of a sum of 2^(t-2), the bound of
//     a sum in fp32, and if only one term in q is off, within that of a sum of 2^(t-2) / q.  That is the floor of a row, with q from
//     32 of the sampled elements (RowSample::floor_of), 128 at most.  Sums below the floors of their rows are formed again one by
//     one, in fp32 from the operands (statistics of independent rows of random sign have sums of about sqrt(K) 2^10 and floors of
//     1/4 together: one tile in a hundred has such a sum; of the products of an inversion one in six).  Where there are many of
//     them the rows are read: if no element is below 2^-2, or all these sums are zero and no element has become zero, they are
//     right as they are; otherwise the tile is repeated in the three-plane mode.
// Where an operand is an inverse (or is multiplied with one before), the scales of the contraction's variables are its diagonal
// (P.kdiag): where its square roots spread over more than 2^11, so that the sums come out below the floors, the three-plane mode is
// taken from the start.
// What the input costs: statistics of 64 to 1024 channels (56 x 56 to 7 x 7, 32 to 128 samples) take the same time, to 7 %, for
// normal values, images scaled by exp(2 N(0,1)) and fifth powers; 5 % of dead channels cost 14 to 19 %; half of them, or 95 % of
// zeros, lead to the three-plane mode, whose time that is (541 us against 405 for 512 channels at 7 x 7, 128 samples).
constexpr int kHalfTop = 6, kHalfTopInverse = 10;   // t
constexpr float kHalfFloor = 0x1p4f, kHalfFloorInverse = 0x1p8f;
constexpr float kHalfExact = 0x1p-2f, kHalfNonzero = 0x1p-24f;   // smaller elements are exact in part; become zero
constexpr int kHalfSpread = kHalfTopInverse + 1;    // spread of a well-scaled contraction, in exponents of the variables
constexpr int kHalfFew = 8;          // a row with fewer elements of 32 above kHalfExact is dominated by them
constexpr float kNoFloor = -0x1p100f;   // of rows of zeros, and of rows outside the operand
constexpr int LDP = 32;              // LDS row length in fp16; 16-byte chunks of a row are permuted instead of padded (half_swz)
__device__ __forceinline__ int half_swz(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }

__device__ __forceinline__ int half_exponent(float s) { return (int)(__float_as_uint(s) >> 23) - 127; }   // log2 of a scale
__device__ __forceinline__ float max_abs(float m, const floatx4 &v)
{
    return fmaxf(fmaxf(m, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
}

// The floor that the counts of 32 sampled elements give, see RowSample::floor_of.
__device__ __forceinline__ float half_floor(float f, float most)
{
    const float n_small = floorf(f * 0x1p-16f);
    f -= n_small * 0x1p16f;
    const float n_larger = floorf(f * 0x1p-10f);
    f -= n_larger * 0x1p10f;
    return most * (n_larger <= 1.f ? 2.f : n_larger < kHalfFew ? 1.f : fminf(fmaxf(1.f / 128, n_small / (4.f * f)), 1.f));
}

// Largest sampled magnitudes of the thread's rows over [k0, k0 + klen): request() issues the loads of four chunks per row and lane,
// finish() waits for them, so that both operands' loads are in flight together.
template <int BR>
struct RowSample {
    static constexpr int SLOTS = BR / 32;
    floatx4 v[4][SLOTS];

    // four places of 32 elements instead of eight of 16: fewer lines of memory, where the rows are not made of many images
    __device__ __forceinline__ void request(LoaderF32<BR> &ld, int k0, int klen, bool four)
    {
        const int span = (klen & ~3) - (four ? 32 : 16), last = four ? 3 : 7;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = four ? q : 2 * q + ld.kq / 16;
            ld.seek(k0 - (four ? 0 : ld.kq & 16) + (c == last ? span : (span / last * c) & ~3));
            ld.load_full(v[q]);
        }
    }
    __device__ __forceinline__ void finish(const LoaderF32<BR> &ld, const Operand &op, int tile_row0, int k0, int klen, float (&mx)[SLOTS]) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            mx[s] = max_abs(max_abs(0.f, v[0][s]), v[1][s]);
            mx[s] = max_abs(max_abs(mx[s], v[2][s]), v[3][s]);
            const int row = tile_row0 + ld.r0 + 32 * s;
            if (op.diag && row >= k0 && row < k0 + klen && row < op.rows) mx[s] = fmaxf(mx[s], fabsf(ld.base[ld.rowoff[s] + row]));
            for (int k = klen & ~3; k < klen; ++k) mx[s] = fmaxf(mx[s], fabsf(ld.base[ld.rowoff[s] + k0 + k]));   // (plain matrices only)
        }
    }
    // The floor of the thread's row of slot s under its scale, from one element of each chunk: `most` for a row that a few elements
    // dominate (whether a small element of the other row meets one of these, no share tells; twice that where hardly any is left),
    // otherwise by the share of small ones and the mean (of what is above 16, 16), which their errors are measured against.
    __device__ __forceinline__ float floor_of(float scale, int s, float most) const
    {
        float f = 0.f;   // sum of up to 512 + 2^10 times the larger elements + 2^16 times the small ones, to 2^-2
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float y = fabsf(v[e][s][0]) * scale;
            f += fminf(y, 16.f) + (y >= kHalfExact ? 0x1p10f : y != 0.f ? 0x1p16f : 0.f);
        }
        f += __shfl_xor(f, 1);
        f += __shfl_xor(f, 2);
        f += __shfl_xor(f, 4);
        return half_floor(f, most);
    }
};
// over the 8 lanes of a row
__device__ __forceinline__ float row_max(float x)
{
    x = fmaxf(x, __shfl_xor(x, 1));
    x = fmaxf(x, __shfl_xor(x, 2));
    return fmaxf(x, __shfl_xor(x, 4));
}

// A row [k0, k0 + klen) for a wavefront, 2048 elements at a time, until f(thread's part) says that it is enough.
template <typename F>
__device__ __forceinline__ void walk_row(const Operand &op, int row, int k0, int klen, int lane, F f)
{
    constexpr int U = 8;
    gfloat_ptr p = (gfloat_ptr)op.base + (long long)min(row, op.rows - 1) * op.row_stride;
    const int last = (klen & ~3) - 4;
    bool enough = false;
    for (int k = 0; k <= last && !enough; k += 256 * U) {
        floatx4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {   // (beyond the end: the last four again)
            const int m = k0 + min(k + 256 * u + 4 * lane, last), n = m < op.hw ? 0 : m / op.hw;
            v[u] = *(gfloat4_ptr)(p + n * op.batch_stride + (m - n * op.hw));
        }
        enough = f(v);
    }
    if (!enough && (klen & 3)) {        // (plain matrices only)
        floatx4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (lane < (klen & 3)) v[0][0] = p[k0 + (klen & ~3) + lane];
        f(v);
    }
}

// Scales of the rows of both operand tiles into registers and into sc[0 .. BM) and sc[BM .. BM + BN), their floors into the BM + BN
// places behind; false: the two planes do not serve (see above).
template <int BM, int BN, bool SAME>
__device__ __forceinline__ bool half_scales(const GemmProblem &P, int tm, int tn, LoaderF32<BM> &la, LoaderF32<BN> &lb,
                                            int k0, int klen, float *sc, int tid, float (&sa)[BM / 32],
                                            float (&sb)[BN / 32])
{
    int *range = (int *)(sc + 2 * (BM + BN));   // largest exponent of kdiag, and 255 minus the smallest
    if (P.kdiag) {
        if (tid < 2) range[tid] = 0;
        __syncthreads();
    }
    RowSample<BM> va;
    RowSample<BN> vb;
    va.request(la, k0, klen, P.kdiag != nullptr);
    if constexpr (!SAME) vb.request(lb, k0, klen, P.kdiag != nullptr);
    if (P.kdiag) {
        int hi = 0, lo = 0;
        for (int k = k0 + tid; k < k0 + klen; k += 256) {
            const int e = (int)((__float_as_uint(global(P.kdiag)[(long long)k * P.kdiag_step]) >> 23) & 255);
            hi = max(hi, e);
            lo = max(lo, 255 - e);
        }
        for (int d = 32; d > 4; d >>= 1) { hi = max(hi, __shfl_xor(hi, d)); lo = max(lo, __shfl_xor(lo, d)); }
        if ((tid & 63) < 8) { atomicMax(range, hi); atomicMax(range + 1, lo); }
    }
    const bool first = (tid & 7) == 0;
    const int top = P.kdiag ? kHalfTopInverse : kHalfTop;
    const float most_floor = P.kdiag ? kHalfFloorInverse : kHalfFloor;
    bool odd = false;   // a row of the thread sampled as zero or nearly so
    auto scales = [&](auto &ld, const auto &v, const Operand &op, int row0, float *out, auto &scale) {
        constexpr int SLOTS = std::remove_reference_t<decltype(ld)>::SLOTS;
        v.finish(ld, op, row0, k0, klen, scale);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const float most = row_max(scale[s]);
            scale[s] = half_scale(most, top);
            const float floor = v.floor_of(scale[s], s, most_floor);
            if (most == 0.f) scale[s] = 0.f;
            odd |= floor > most_floor;
            if (first) {
                out[ld.r0 + 32 * s] = scale[s];
                out[BM + BN + ld.r0 + 32 * s] = (ld.dead >> s) & 1 ? kNoFloor : floor;
            }
        }
    };
    scales(la, va, P.a, tm * BM, sc, sa);
    if constexpr (!SAME) scales(lb, vb, P.b, tn * BN, sc + BM, sb);
    if (__syncthreads_or(odd)) {
        // Where a quarter of the rows on both sides has hardly any elements, too many sums would come out in doubt; and where they have
        // none that were sampled, reading on costs more than the two planes give.
        const bool few = tid < (SAME ? BM : BM + BN) && sc[BM + BN + tid] > most_floor;
        const int n_a = __syncthreads_count(few && tid < BM), n_b = SAME ? n_a : __syncthreads_count(few && tid >= BM);
        if (4 * n_a > BM && 4 * n_b > BN) return false;
        // rows that sampled as zero are dealt to the wavefronts, which read on until an element is not
        for (int r = tid >> 6; r < (SAME ? BM : BM + BN); r += 4) {
            if (sc[r] != 0.f) continue;
            float mx = 0.f;
            walk_row(r < BM ? P.a : P.b, r < BM ? tm * BM + r : tn * BN + r - BM, k0, klen, tid & 63, [&](const auto &v) {
#pragma unroll
                for (const floatx4 &x : v) mx = max_abs(mx, x);
                for (int d = 32; d > 0; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
                return mx != 0.f;
            });
            if ((tid & 63) == 0) {
                sc[r] = half_scale(mx, top);
                if (mx == 0.f) sc[BM + BN + r] = kNoFloor;
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < BM / 32; ++s) sa[s] = sc[la.r0 + 32 * s];
        if constexpr (!SAME)
#pragma unroll
            for (int s = 0; s < BN / 32; ++s) sb[s] = sc[BM + lb.r0 + 32 * s];
    }
    if constexpr (SAME) {
#pragma unroll
        for (int s = 0; s < BM / 32; ++s) {
            sb[s] = sa[s];
            if (first) {
                sc[BM + la.r0 + 32 * s] = sa[s];
                sc[BM + BN + BM + la.r0 + 32 * s] = sc[BM + BN + la.r0 + 32 * s];
            }
        }
    }
    return !(P.kdiag && range[0] + range[1] - 255 > 2 * kHalfSpread);
}

// Whether an element of the rows of a tile, scaled, is below `least` and not zero (the rows are dealt to the wavefronts).
template <int BR>
__device__ __forceinline__ bool any_below(const Operand &op, int tile_row0, int k0, int klen, const float *scales, float least, int tid)
{
    bool found = false;
    for (int r = tid >> 6; r < BR && tile_row0 + r < op.rows && !found; r += 4) {
        const float limit = __builtin_amdgcn_ldexpf(least, -half_exponent(scales[r]));
        walk_row(op, tile_row0 + r, k0, klen, tid & 63, [&](const auto &v) {
#pragma unroll
            for (const floatx4 &x : v)
#pragma unroll
                for (int e = 0; e < 4; ++e) found |= x[e] != 0.f && fabsf(x[e]) < limit;
            found = __any(found);
            return found;
        });
    }
    return found;
}

// One slot of a staged tile into its rows of the two planes (plane stride in fp16 units).  Rows outside the operand repeat its
// last row: what they contribute to is not stored.  MASK: the tile may hold k positions that count as zero.
template <int BR, bool RS, bool MASK>
__device__ __forceinline__ void store_half_slot(const LoaderF32<BR> &ld, const floatx4 &x, unsigned short *rows, int plane, float scale,
                                                float &rs, int s)
{
    floatx4 v = x;
    if constexpr (MASK) {
        if (ld.zero_all) { v[0] = 0.f; v[1] = 0.f; v[2] = 0.f; v[3] = 0.f; }
    }
    if constexpr (RS) rs += (v[0] + v[1]) + (v[2] + v[3]);
    uint2 h, l;
    split_half_pair(v[0], v[1], scale, h.x, l.x);
    split_half_pair(v[2], v[3], scale, h.y, l.y);
    unsigned short *dst = rows + (ld.r0 + 32 * s) * LDP + (((ld.kq >> 3) ^ half_swz(ld.r0)) << 3) + (ld.kq & 4);
    *(uint2 *)dst = h;
    *(uint2 *)(dst + plane) = l;
}

// K % 4 remainder tile: thread tid < BR fills row tid of the planes with the elements k4 .. kend-1 of its operand row followed
// by zeros; returns their sum
template <int BR>
__device__ __forceinline__ float fill_remainder_half(const Operand &op, int tile_row0, int k4, int kend, int tid,
                                                     unsigned short *rows, int plane, const float *sc)
{
    if (tid >= BR) return 0.f;
    const int row = tile_row0 + tid;
    float x[4] = {0.f, 0.f, 0.f, 0.f};
    if (row < op.rows) {
        gfloat_ptr p = (gfloat_ptr)op.base + (long long)row * op.row_stride + k4;
        for (int e = 0; e < 3; ++e)
            if (k4 + e < kend) x[e] = p[e];
    }
    uint2 v[2];
    const float scale = sc[tid];
    split_half_pair(x[0], x[1], scale, v[0].x, v[1].x);
    split_half_pair(x[2], x[3], scale, v[0].y, v[1].y);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            *(uint4 *)(rows + q * plane + tid * LDP + ((c ^ half_swz(tid)) << 3)) = c == 0 ? uint4{v[q].x, v[q].y, 0u, 0u} : uint4{0u, 0u, 0u, 0u};
    return x[0] + x[1] + x[2];
}

template <int TM, int TN>
__device__ __forceinline__ void zero_acc(floatx16 (&acc)[TM][TN])
{
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

// Software pipeline over K tiles of 32 with two stages in LDS and one barrier per tile.  While the matrix instructions of tile
// `it` run, the wavefront converts tile it + 1, which its registers hold, stores it into the other stage and issues the loads
// of tile it + 2.  The six phases of a tile (h h', h l', l h' of its first and of its second 16 k) need 2 TM + 2 TN fragments
// between them: each is requested one phase ahead, into the registers of one whose last product has been issued (the two sets
// of b fragments change roles at the second half).
// SAME: a and b are the same operand tile (a diagonal tile of a Gram matrix): staged once.
template <int TM, int TN, bool LIVE, bool RS, bool SAME>
__device__ __forceinline__ bool gemm_half_mainloop(const GemmProblem &P, int tm, int tn, int tid,
                                                   LoaderF32<64 * TM> &la,
                                                   LoaderF32<64 * TN> &lb, unsigned short *lds, float *sc,
                                                   int k0, int k1, int wave_m, int wave_n, int l32, int half,
                                                   floatx16 (&acc)[TM][TN], float (&rs)[2 * TM], float &rs_rem)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int PLANE = (BM + BN) * LDP, STAGE = 2 * PLANE;
    constexpr int SA = BM / 32, SB = SAME ? 0 : BN / 32;
    const int klen = k1 - k0;                            // more than one K tile
    const int klen4 = klen & ~3;
    const int nfull = klen4 / KT;
    const int nvec = nfull + (klen4 > nfull * KT ? 1 : 0);   // one more full tile ending at k0 + klen4
    const int nk = nvec + (klen4 < klen ? 1 : 0);
    float sa[BM / 32], sb[BN / 32];
    floatx4 ra[BM / 32], rb[BN / 32];

    auto load_tile = [&](int it) {
        if (it < nfull) {
            if (it > 0) {
                la.advance();
                if constexpr (!SAME) lb.advance();
            }
            la.load_full(ra);
            if constexpr (!SAME) lb.load_full(rb);
        } else if (it < nvec) {
            la.seek(k0 + klen4 - KT);
            la.load_full(ra);
            if constexpr (!SAME) {
                lb.seek(k0 + klen4 - KT);
                lb.load_full(rb);
            }
            la.zero_below(k0 + nfull * KT);
        }
    };
    auto store_tile = [&](int it) {
        unsigned short *st = lds + (it & 1) * STAGE;
        if (it < nvec) {
            float unused = 0.f;
#pragma unroll
            for (int s = 0; s < SA; ++s) store_half_slot<BM, RS, true>(la, ra[s], st, PLANE, sa[s], rs[s], s);
#pragma unroll
            for (int s = 0; s < SB; ++s) store_half_slot<BN, false, true>(lb, rb[s], st + BM * LDP, PLANE, sb[s], unused, s);
        } else {
            rs_rem = fill_remainder_half<BM>(P.a, tm * BM, k0 + klen4, k1, tid, st, PLANE, sc);
            if constexpr (!SAME) fill_remainder_half<BN>(P.b, tn * BN, k0 + klen4, k1, tid, st + BM * LDP, PLANE, sc + BM);
        }
    };
    // v_mfma_f32_32x32x16_f16: a lane supplies 8 consecutive k of row lane % 32, the half-waves two different groups of 8;
    // half u of a tile uses k = 16u + 8*half + 0..7 (chunk 2u + half of the row) for both operands
    const int off_a = (wave_m * 32 * TM + l32) * LDP + ((half ^ half_swz(l32)) << 3);
    const int off_b = ((SAME ? 0 : BM) + wave_n * 32 * TN + l32) * LDP + ((half ^ half_swz(l32)) << 3);
    halfx8 ah[TM], al[TM], b0[TN], b1[TN];
    auto read_a = [&](halfx8 (&f)[TM], const unsigned short *st, int plane, int u) {
#pragma unroll
        for (int i = 0; i < TM; ++i) f[i] = __builtin_bit_cast(halfx8, *(const ushortx8 *)(st + (off_a ^ (u << 4)) + i * 32 * LDP + plane * PLANE));
    };
    auto read_b = [&](halfx8 (&f)[TN], const unsigned short *st, int plane, int u) {
#pragma unroll
        for (int j = 0; j < TN; ++j) f[j] = __builtin_bit_cast(halfx8, *(const ushortx8 *)(st + (off_b ^ (u << 4)) + j * 32 * LDP + plane * PLANE));
    };
    // one phase; side(0) behind its first matrix instruction, side(1) behind the middle one.  Fixed order: the scheduling
    // barriers keep the compiler from drawing loads and conversions together, for which there are no registers.
    auto mma = [&](const halfx8 (&x)[TM], const halfx8 (&y)[TN], auto side) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < TM * TN; ++n) {
            const int i = n / TN, j = n % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[i], y[j], acc[i][j], 0, 0, 0);
            if (n == 0 || 2 * n == TM * TN) {
                __builtin_amdgcn_sched_barrier(0);
                side(n != 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto nothing = [](int) {};
    // the phases of one tile; side(q), q = 0 .. 7, is dealt out over the first four, which lie before the barrier
    auto phases = [&](const unsigned short *cur, const unsigned short *nxt, bool more, auto side) {
        if constexpr (LIVE) {
            read_b(b1, cur, 1, 0);
            read_a(al, cur, 1, 0);
            mma(ah, b0, [&](int q) { side(q); });
            mma(ah, b1, [&](int q) { side(2 + q); });
            read_b(b1, cur, 0, 1);
            read_a(ah, cur, 0, 1);
            mma(al, b0, [&](int q) { side(4 + q); });
            read_b(b0, cur, 1, 1);
            read_a(al, cur, 1, 1);
            mma(ah, b1, [&](int q) { side(6 + q); });
            __syncthreads();
            mma(ah, b0, nothing);
            if (more) {
                read_b(b0, nxt, 0, 0);
                read_a(ah, nxt, 0, 0);
            }
            mma(al, b1, nothing);
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) side(q);
            __syncthreads();
        }
    };

    // the loads of the first tile are on their way while the rows are sampled
    la.seek(k0);
    if constexpr (!SAME) lb.seek(k0);
    load_tile(0);
    if (!half_scales<BM, BN, SAME>(P, tm, tn, la, lb, k0, klen, sc, tid, sa, sb)) return false;
    la.seek(k0);
    if constexpr (!SAME) lb.seek(k0);
    zero_acc(acc);
    store_tile(0);
    load_tile(1);
    __syncthreads();
    if constexpr (LIVE) {
        read_b(b0, lds, 0, 0);
        read_a(ah, lds, 0, 0);
    }
    int it = 0;
    // The steady state: tile it + 2 is a full one reached by a single wrap of the position.
    if (la.hw >= KT && lb.hw >= KT)
        for (; it + 2 < nfull; ++it) {
            const unsigned short *cur = lds + (it & 1) * STAGE;
            unsigned short *nxt = lds + ((it + 1) & 1) * STAGE;
            la.advance_once();
            if constexpr (!SAME) lb.advance_once();
            phases(cur, nxt, true, [&](int q) {
                constexpr int EVERY = 8 / (SA + SB);   // 8, 4 or (one operand) 2 slots
                if (q % EVERY == 0) {
                    const int k = q / EVERY;
                    float unused = 0.f;
                    if (k < SA) {
                        store_half_slot<BM, RS, false>(la, ra[k], nxt, PLANE, sa[k], rs[k], k);
                        la.load_slot(ra, k);
                    } else if (k < SA + SB) {
                        store_half_slot<BN, false, false>(lb, rb[k - SA], nxt + BM * LDP, PLANE, sb[k - SA], unused, k - SA);
                        lb.load_slot(rb, k - SA);
                    }
                }
            });
        }
    for (; it < nk; ++it)
        phases(lds + (it & 1) * STAGE, lds + ((it + 1) & 1) * STAGE, it + 1 < nk, [&](int q) {
            if (q != 0) return;
            if (it + 1 < nk) store_tile(it + 1);
            load_tile(it + 2);
        });
    return true;
}

// acc[i][j][v] is element (row, column) = (8 (v / 4) + 4 half + v % 4, l32) of block (i, j).  Returns bit 0 if a sum is below
// the floors of its rows, bit 1 if one is not finite, bit 2 if one of the former is not zero either.  The
// former are counted in doubts[0] and the first kMaxDoubts listed behind it (row * 256 + column).
template <int TM, int TN>
__device__ __forceinline__ int half_doubts(const floatx16 (&acc)[TM][TN], const float *sc, int *doubts, int wave_m, int wave_n, int l32, int half)
{
    const float *floors = sc + 64 * TM + 64 * TN;
    float fb[TN], z = 0.f, least = 0.f;   // z: (0 * inf and 0 * NaN are NaN, which differs from 0)
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = floors[64 * TM + wave_n * 32 * TN + j * 32 + l32];
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int row = wave_m * 32 * TM + i * 32 + 8 * g + 4 * half;
                const floatx4 fa = *(const floatx4 *)(floors + row);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < TN; ++j) f(fabsf(acc[i][j][4 * g + e]), fa[e] + fb[j], row + e, wave_n * 32 * TN + j * 32 + l32);
            }
    };
    each([&](float v, float floor, int, int) {
        z = fmaf(v, 0.f, z);
        least = fminf(least, v - floor);
    });
    int bits = z != 0.f ? 2 : 0;
    if (least < 0.f)
        each([&](float v, float floor, int row, int column) {
            if (v < floor) {
                bits |= v == 0.f ? 1 : 5;
                const int n = atomicAdd(doubts, 1);
                if (n < kMaxDoubts) doubts[1 + n] = row * 256 + column;
            }
        });
    return bits;
}

// The listed sums in fp32, four per wavefront at a time, into their places in `out` (rows of ld elements).
template <int BM, int BN, typename Out>
__device__ __forceinline__ void half_settle(const GemmProblem &P, const int *doubts, int n, int tm, int tn, int k0, int k1, int tid, Out out, int ld)
{
    constexpr int U = 4;
    const int lane = tid & 63, end4 = k0 + ((k1 - k0) & ~3);
    for (int q = U * (tid >> 6); q < n; q += 4 * U) {
        gfloat_ptr a[U], b[U];
        float sum[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int d = doubts[1 + min(q + u, n - 1)];
            a[u] = (gfloat_ptr)P.a.base + (long long)(tm * BM + (d >> 8)) * P.a.row_stride;
            b[u] = (gfloat_ptr)P.b.base + (long long)(tn * BN + (d & 255)) * P.b.row_stride;
            sum[u] = 0.f;
        }
        for (int k = k0 + 4 * lane; k < end4; k += 256) {
            const int na = k / P.a.hw, nb = k / P.b.hw;
            const long long ka = na * P.a.batch_stride + (k - na * P.a.hw), kb = nb * P.b.batch_stride + (k - nb * P.b.hw);
            floatx4 x[U], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) { x[u] = *(gfloat4_ptr)(a[u] + ka); y[u] = *(gfloat4_ptr)(b[u] + kb); }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[u] = fmaf(x[u][e], y[u][e], sum[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (end4 + lane < k1) sum[u] = fmaf(a[u][end4 + lane], b[u][end4 + lane], sum[u]);   // (plain matrices only)
            for (int d = 32; d > 0; d >>= 1) sum[u] += __shfl_xor(sum[u], d);
            if (lane == 0 && q + u < n) out[(doubts[1 + q + u] >> 8) * ld + (doubts[1 + q + u] & 255)] = sum[u];
        }
    }
}

// Undoes the scales of the rows.  Both exponents at once: one after the other, a row near 2^110 against one near 2^-100 leaves the
// range in between.
template <int TM, int TN>
__device__ __forceinline__ void half_unscale_tile(floatx16 (&acc)[TM][TN], const float *sc, int wave_m, int wave_n, int l32, int half)
{
    int eb[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) eb[j] = half_exponent(sc[64 * TM + wave_n * 32 * TN + j * 32 + l32]);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const floatx4 s = *(const floatx4 *)(sc + wave_m * 32 * TM + i * 32 + 8 * g + 4 * half);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ea = half_exponent(s[e]);
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j][4 * g + e] = __builtin_amdgcn_ldexpf(acc[i][j][4 * g + e], -(ea + eb[j]));
            }
        }
}

// ------------------------------------------------------------------ transposed operands (NHWC in place)
// Element (r, m) of the operand lives at base + m * ld + r: the rows are the contiguous direction.  A thread
// loads 16 bytes = four adjacent rows at one m (lanes along the rows: 512 contiguous bytes per 32 lanes), splits
// them and stores 8 bytes per plane into an LDS tile that keeps this order, [m][row]; the fragments of the
// matrix instruction (8 consecutive m of one row per lane) come out of that tile through the transposing LDS
// read of gfx950 (ds_read_b64_tr_b16: within 16 lanes, lane i receives element i % 4 of the four 8-byte groups
// addressed by lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12).  Every m of the range is read where it is: no
// shifted tile, no remainder tile; loads beyond the range are clamped and zeroed by value.
template <int BR>
struct LoaderF32T {
    static constexpr int SLOTS = BR / 32;
    static constexpr int CG = BR / 4;          // row chunks of the tile
    static constexpr int MSTEP = 256 / CG;     // m positions covered by one slot of all threads
    static constexpr int RS = BR + 16;         // LDS row (one m) in bf16: four rows of a read 32 bytes apart in banks
    gfloat_ptr base;
    long long ld;
    int c_local, c_load, mk, K;
    bool dead;

    __device__ __forceinline__ void init(const Operand &op, int tile_row0, int tid, int K_)
    {
        base = (gfloat_ptr)op.base;
        ld = op.row_stride;
        c_local = 4 * (tid % CG);
        mk = tid / CG;
        const int c = tile_row0 + c_local;
        dead = c >= op.rows;                         // rows % 4 == 0: a chunk is inside or outside as a whole
        c_load = min(c, op.rows - 4);
        K = K_;
    }
    __device__ __forceinline__ void load(floatx4 (&reg)[SLOTS], int tile_m0) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int m = min(tile_m0 + mk + MSTEP * s, K - 1);
            reg[s] = *(gfloat4_ptr)(base + (long long)m * ld + c_load);
        }
    }
    // mend: end of the workgroup's range; rs: running sums of the thread's four rows
    template <bool RSUM>
    __device__ __forceinline__ void store(const floatx4 (&reg)[SLOTS], unsigned short *rows, int plane, int tile_m0,
                                          int mend, float (&rs)[4]) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            floatx4 v = reg[s];
            const int ml = mk + MSTEP * s;
            if (dead || tile_m0 + ml >= mend) { v[0] = 0.f; v[1] = 0.f; v[2] = 0.f; v[3] = 0.f; }
            if constexpr (RSUM) { rs[0] += v[0]; rs[1] += v[1]; rs[2] += v[2]; rs[3] += v[3]; }
            uint2 h, m, l;
            split_pair(v[0], v[1], h.x, m.x, l.x);
            split_pair(v[2], v[3], h.y, m.y, l.y);
            unsigned short *dst = rows + ml * RS + c_local;
            *(uint2 *)dst = h;
            *(uint2 *)(dst + plane) = m;
            *(uint2 *)(dst + 2 * plane) = l;
        }
    }
};

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4 *lds_shortx4_ptr;

template <int TM, int TN, bool LIVE, bool RSUM>
__device__ __forceinline__ void gemm_split_mainloop_trans(const GemmProblem &P, int tm, int tn, int tid,
                                                          unsigned short *lds, int k0, int k1, int wave_m, int wave_n,
                                                          int lane, floatx16 (&acc)[TM][TN], float (&rs)[4])
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int RSA = LoaderF32T<BM>::RS, RSB = LoaderF32T<BN>::RS;
    constexpr int PLANE_A = KT * RSA, PLANE_B = KT * RSB;
    unsigned short *lds_b = lds + 3 * PLANE_A;
    LoaderF32T<BM> la;
    LoaderF32T<BN> lb;
    la.init(P.a, tm * BM, tid, P.K);
    lb.init(P.b, tn * BN, tid, P.K);
    const int nk = (max(k1 - k0, 0) + KT - 1) / KT;
    if (nk == 0) return;
    floatx4 ra0[BM / 32], rb0[BN / 32], ra1[BM / 32], rb1[BN / 32];
    // fragment addressing of the transposing read: lane -> (m within the 16-wide step, first of four rows)
    const int frag_m = 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int frag_r = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const int off_a = frag_m * RSA + wave_m * 32 * TM + frag_r;
    const int off_b = frag_m * RSB + wave_n * 32 * TN + frag_r;
    auto compute = [&]() {
        if constexpr (LIVE) {
            auto rd = [&](const unsigned short *plane, int rs_, int off, int u) {
                const unsigned short *p = plane + off + 16 * u * rs_;
                const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_ptr)p);
                const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_ptr)(p + 4 * rs_));
                typedef short shortx8 __attribute__((ext_vector_type(8)));
                return __builtin_bit_cast(bf16x8, shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            };
            auto mm = [&](const bf16x8 (&x)[TM], const bf16x8 (&y)[TN]) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], y[j], acc[i][j], 0, 0, 0);
            };
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 ah[TM], am[TM], bh[TN], bm[TN], bl[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) ah[i] = rd(lds, RSA, off_a + i * 32, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) bh[j] = rd(lds_b, RSB, off_b + j * 32, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) bm[j] = rd(lds_b + PLANE_B, RSB, off_b + j * 32, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) bl[j] = rd(lds_b + 2 * PLANE_B, RSB, off_b + j * 32, u);
#pragma unroll
                for (int i = 0; i < TM; ++i) am[i] = rd(lds + PLANE_A, RSA, off_a + i * 32, u);
                __builtin_amdgcn_sched_barrier(0);
                mm(ah, bh);
                mm(ah, bm);
                mm(ah, bl);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TM; ++i) ah[i] = rd(lds + 2 * PLANE_A, RSA, off_a + i * 32, u);   // the l plane of a
                __builtin_amdgcn_sched_barrier(0);
                mm(am, bh);
                mm(am, bm);
                mm(ah, bh);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    float unused[4] = {0.f, 0.f, 0.f, 0.f};
    la.load(ra0, k0); lb.load(rb0, k0);
    la.load(ra1, k0 + KT); lb.load(rb1, k0 + KT);
    for (int it = 0; it < nk; it += 2) {
        if (it > 0) __syncthreads();   // every wavefront has read the tile before
        la.template store<RSUM>(ra0, lds, PLANE_A, k0 + it * KT, k1, rs);
        lb.template store<false>(rb0, lds_b, PLANE_B, k0 + it * KT, k1, unused);
        la.load(ra0, k0 + (it + 2) * KT); lb.load(rb0, k0 + (it + 2) * KT);
        __syncthreads();
        compute();
        if (it + 1 < nk) {
            __syncthreads();
            la.template store<RSUM>(ra1, lds, PLANE_A, k0 + (it + 1) * KT, k1, rs);
            lb.template store<false>(rb1, lds_b, PLANE_B, k0 + (it + 1) * KT, k1, unused);
            la.load(ra1, k0 + (it + 3) * KT); lb.load(rb1, k0 + (it + 3) * KT);
            __syncthreads();
            compute();
        }
    }
}

// Row sums of a diagonal tile whose operand is stored transposed: a thread holds the sums of its four rows over
// the m positions it loaded; the 256 / (BM / 4) threads that share a row chunk are added up through LDS.
template <int BM, int E>
__device__ __forceinline__ void finish_row_sums_trans(const GemmProblem &P, float *lds, int tm, int tile, int split,
                                                      int tid, const float (&rs)[E])
{
    constexpr int CG = BM / E, PARTS = 256 / CG;
    __syncthreads();   // the operand stages are dead
#pragma unroll
    for (int e = 0; e < E; ++e) lds[(tid / CG) * BM + E * (tid % CG) + e] = rs[e];
    __syncthreads();
    if (tid < BM) {
        float total = 0.f;
#pragma unroll
        for (int q = 0; q < PARTS; ++q) total += lds[q * BM + tid];
        const int row = tm * BM + tid;
        if (P.splits > 1) global(P.partial_rs)[((long long)tm * P.splits + split) * BM + tid] = total;
        else if (row < P.M) store_border(P, row, total);
    }
    if (tile == 0 && tid == 0 && P.splits == 1) store_corner(P);
    __syncthreads();
}

// TRANS: the product mode of three bf16 planes on operands stored with the rows contiguous; otherwise the fp32 instruction.
template <int TM, int TN, bool TRANS>
__device__ __forceinline__ void gemm_nt_f32_body(const GemmProblem *__restrict__ probs,
                                                 const int *__restrict__ tile_start, int n_probs)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    extern __shared__ __attribute__((aligned(16))) float lds[];   // 2 stages of (BM + BN) * LDF floats

    const int wg = blockIdx.x;
    const int pi = find_problem(tile_start, n_probs, wg);
    const GemmProblem &P = probs[pi];
    const int local = wg - tile_start[pi];
    if (local >= n_workgroups(P)) return;   // padding up to the next problem
    int tile, split, tm, tn;
    const bool part_of_k = locate_tile(P, local, tile, split);   // neighbours: neighbouring tiles of the same K range
    decode_tile(P, tile, tm, tn);
    const int k0 = split * P.k_per_split;
    const int k1 = part_of_k ? min(P.K, k0 + P.k_per_split) : P.K;
    const int tid = threadIdx.x;

    LoaderF32<BM> la;
    LoaderF32<BN> lb;
    la.init(P.a, tm * BM, tid);
    lb.init(P.b, tn * BN, tid);

    floatx16 acc[TM][TN];
    zero_acc(acc);

    const int lane = tid & 63, wid = tid >> 6;
    const int wave_m = wid >> 1, wave_n = wid & 1;
    const int l32 = lane & 31, half = lane >> 5;

    // A wavefront whose whole sub-tile lies outside the matrix, or above the diagonal of a
    // symmetric product, stores nothing: it only helps with the loads and skips the math.
    const bool diag_tile = (P.flags & GEMM_SYM) && tm == tn;
    const int wave_r0 = tm * BM + wave_m * 32 * TM, wave_c0 = tn * BN + wave_n * 32 * TN;
    const bool live = wave_r0 < P.M && wave_c0 < P.N && !(diag_tile && wave_c0 >= wave_r0 + 32 * TM);

    // The diagonal tiles of a bordered problem also take the row sums of their operand rows.
    const bool border = diag_tile && (P.flags & GEMM_BORDER);
    float rs[BM / 32], rs_rem = 0.f;
#pragma unroll
    for (int s = 0; s < BM / 32; ++s) rs[s] = 0.f;
    auto mainloop = [&](auto live_c, auto rs_c) {
        gemm_f32_mainloop<TM, TN, decltype(live_c)::value, decltype(rs_c)::value>(P, tm, tn, tid, la, lb, lds, k0, k1, wave_m,
                                                                                 wave_n, l32, half, acc, rs, rs_rem);
    };
    if constexpr (TRANS) {   // both operands stored with the rows contiguous (a launch of its own)
        float rst[4] = {0.f, 0.f, 0.f, 0.f};
        unsigned short *l16 = (unsigned short *)lds;
        if (border) {
            if (live) gemm_split_mainloop_trans<TM, TN, true, true>(P, tm, tn, tid, l16, k0, k1, wave_m, wave_n, lane, acc, rst);
            else      gemm_split_mainloop_trans<TM, TN, false, true>(P, tm, tn, tid, l16, k0, k1, wave_m, wave_n, lane, acc, rst);
            finish_row_sums_trans<BM, 4>(P, lds, tm, tile, split, tid, rst);
        } else {
            if (live) gemm_split_mainloop_trans<TM, TN, true, false>(P, tm, tn, tid, l16, k0, k1, wave_m, wave_n, lane, acc, rst);
            else      gemm_split_mainloop_trans<TM, TN, false, false>(P, tm, tn, tid, l16, k0, k1, wave_m, wave_n, lane, acc, rst);
        }
    } else if (border) {
        if (live) mainloop(std::true_type{}, std::true_type{});
        else      mainloop(std::false_type{}, std::true_type{});
        finish_row_sums<BM>(P, lds, tm, tile, split, tid, rs, rs_rem);
    } else {
        if (live) mainloop(std::true_type{}, std::false_type{});
        else      mainloop(std::false_type{}, std::false_type{});
    }

    // accumulator layout of the 32x32 block: column = lane % 32,
    // row = 8 * (v / 4) + 4 * (lane / 32) + v % 4 for register v = 0..15
    if (part_of_k) {
        const Global<float> part = global(P.partial) + ((long long)(tile - P.split_from) * P.splits + split) * (BM * BN);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = wave_m * 32 * TM + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                    const int c = wave_n * 32 * TN + j * 32 + l32;
                    part[r * BN + c] = acc[i][j][v];
                }
    } else {
        // stage the tile in LDS (the operand stages are dead by now), then store whole rows
        __syncthreads();
        if (live) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int r = wave_m * 32 * TM + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                        const int c = wave_n * 32 * TN + j * 32 + l32;
                        lds[r * (BN + 1) + c] = acc[i][j][v];
                    }
        }
        __syncthreads();
        store_slab<BM, BN>(P, lds, tm * BM, tn * BN, diag_tile, tid);
    }
}

template <int TM, int TN>
__global__ __launch_bounds__(256) void gemm_nt_f32_kernel(const GemmProblem *__restrict__ probs,
                                                          const int *__restrict__ tile_start, int n_probs)
{
    gemm_nt_f32_body<TM, TN, false>(probs, tile_start, n_probs);
}

// the same for problems whose operands are stored transposed (GEMM_TRANS)
template <int TM, int TN>
__global__ __launch_bounds__(256, 2) void gemm_nt_f32_split_trans_kernel(const GemmProblem *__restrict__ probs,
                                                                         const int *__restrict__ tile_start, int n_probs)
{
    gemm_nt_f32_body<TM, TN, true>(probs, tile_start, n_probs);
}

// fp32 products through planes: two of fp16, or three of bf16 where the scales do not serve.
// What bounds it: of its energy, which the clock pays for (1.65 GHz under it), the matrix instructions and fragment reads take
// about half, the conversion on the way into LDS a third and the loads the rest; without the staging it would run at 540
// TFLOP/s, without the matrix instructions at 490.  Random operands, 128-tile (64-tile): 4096^3 260 (200) TFLOP/s against 167
// to 185 with three planes, ResNet-50's statistics at batch 128 268 (123) against 169 (107), 512 channels at 7x7 301 (200; with
// three planes 143).  Eight places of a row and the floors of the rows take 2 to 5 % (without them 268, 274 and 318).  Tiles of 256 x 128 by eight wavefronts were 5 % faster on 4096^3 and too coarse for the rest; 256 x 256 spills.
// (Two wavefronts per SIMD, four of the small tile: the register allocation is held to 256 and 128.)
template <int TM, int TN>
__device__ __forceinline__ void gemm_nt_f32_split_tile(const GemmProblem &P, int tile, int split, bool part_of_k, float *lds)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    float *sc = lds + split_lds_bytes<TM, TN>() / sizeof(float) - (2 * (BM + BN) + 2 + 1 + kMaxDoubts);
    int *doubts = (int *)(sc + 2 * (BM + BN) + 2);
    unsigned short *l16 = (unsigned short *)lds;
    int tm, tn;
    decode_tile(P, tile, tm, tn);
    const int k0 = split * P.k_per_split;
    const int k1 = part_of_k ? min(P.K, k0 + P.k_per_split) : P.K;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wid = tid >> 6;
    const int wave_m = wid >> 1, wave_n = wid & 1;
    const int l32 = lane & 31, half = lane >> 5;

    // A wavefront whose whole sub-tile lies outside the matrix, or above the diagonal of a
    // symmetric product, stores nothing: it only helps with the loads and skips the math.
    const bool diag_tile = (P.flags & GEMM_SYM) && tm == tn;
    const int wave_r0 = tm * BM + wave_m * 32 * TM, wave_c0 = tn * BN + wave_n * 32 * TN;
    const bool live = wave_r0 < P.M && wave_c0 < P.N && !(diag_tile && wave_c0 >= wave_r0 + 32 * TM);

    // The diagonal tiles of a bordered problem also take the row sums of their operand rows.
    const bool border = diag_tile && (P.flags & GEMM_BORDER);
    floatx16 acc[TM][TN];
    float rs[BM / 32], rs_rem = 0.f;
    // a diagonal tile of a Gram matrix (a and b the same operand) stages its operand tile once (64 x 64 tiles only: the others
    // have no registers to spare for one more copy of the main loop)
    constexpr bool CAN_SHARE = TM == 1 && TN == 1;
    const bool same = CAN_SHARE && tm == tn && P.a.base == P.b.base && P.a.row_stride == P.b.row_stride &&
                      P.a.batch_stride == P.b.batch_stride && P.a.hw == P.b.hw && P.a.rows == P.b.rows;
    auto dispatch = [&](auto f) {
        if (border) {
            if (live) f(std::true_type{}, std::true_type{});
            else      f(std::false_type{}, std::true_type{});
        } else {
            if (live) f(std::true_type{}, std::false_type{});
            else      f(std::false_type{}, std::false_type{});
        }
    };
    auto no_sums = [&]() {
#pragma unroll
        for (int s = 0; s < BM / 32; ++s) rs[s] = 0.f;
    };
    // (a single K tile is not worth the scales, which take a memory latency: 64 -> 32 units, 32 samples, as a step 52 us against 51)
    bool wide = k1 - k0 <= KT;
    int n_doubts = 0;
    if (!wide) {
        if (tid == 0) doubts[0] = 0;
        no_sums();
        dispatch([&](auto live_c, auto rs_c) {
            constexpr bool LV = decltype(live_c)::value, RSUM = decltype(rs_c)::value;
            LoaderF32<BM> la;
            LoaderF32<BN> lb;
            la.init(P.a, tm * BM, tid);
            lb.init(P.b, tn * BN, tid);
            if (CAN_SHARE && same)
                wide = !gemm_half_mainloop<TM, TN, LV, RSUM, CAN_SHARE>(P, tm, tn, tid, la, lb, l16, sc, k0, k1, wave_m, wave_n, l32, half, acc,
                                                                        rs, rs_rem);
            else
                wide = !gemm_half_mainloop<TM, TN, LV, RSUM, false>(P, tm, tn, tid, la, lb, l16, sc, k0, k1, wave_m, wave_n, l32, half, acc,
                                                                    rs, rs_rem);
        });
    }
    if (!wide) {
        const int bits = live ? half_doubts(acc, sc, doubts, wave_m, wave_n, l32, half) : 0;
        if (__syncthreads_or(bits)) {
            wide = __syncthreads_or(bits & 2);
            n_doubts = doubts[0];
            // (sixteen sums at a time take about 2 us, most of it latency: no more of them than take a part of the tile's time)
            if (wide || n_doubts > min(kMaxDoubts, 24 + (k1 - k0) / 32)) {
                n_doubts = 0;
                if (!wide) {
                    const float least = __syncthreads_or(bits & 4) ? kHalfExact : kHalfNonzero;
                    wide = __syncthreads_or(any_below<BM>(P.a, tm * BM, k0, k1 - k0, sc, least, tid) ||
                                            any_below<BN>(P.b, tn * BN, k0, k1 - k0, sc + BM, least, tid));
                }
            }
        }
    }
    if (!wide) {
        if (live) half_unscale_tile(acc, sc, wave_m, wave_n, l32, half);
    } else {
        zero_acc(acc);
        no_sums();
        LoaderF32<BM> la;
        LoaderF32<BN> lb;
        la.init(P.a, tm * BM, tid);
        lb.init(P.b, tn * BN, tid);
        dispatch([&](auto live_c, auto rs_c) {
            gemm_split_mainloop<TM, TN, decltype(live_c)::value, decltype(rs_c)::value>(P, tm, tn, tid, la, lb, l16, k0, k1, wave_m, wave_n,
                                                                                        l32, half, acc, rs, rs_rem);
        });
    }
    if (border) finish_row_sums<BM>(P, lds, tm, tile, split, tid, rs, rs_rem);

    // accumulator layout of the 32x32 block: column = lane % 32,
    // row = 8 * (v / 4) + 4 * (lane / 32) + v % 4 for register v = 0..15
    if (part_of_k) {
        const Global<float> part = global(P.partial) + ((long long)(tile - P.split_from) * P.splits + split) * (BM * BN);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = wave_m * 32 * TM + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                    const int c = wave_n * 32 * TN + j * 32 + l32;
                    part[r * BN + c] = acc[i][j][v];
                }
        if (n_doubts) {
            __syncthreads();
            half_settle<BM, BN>(P, doubts, n_doubts, tm, tn, k0, k1, tid, part, BN);
        }
    } else {
        // stage the tile in LDS (the operand stages are dead by now), then store whole rows
        __syncthreads();
        if (live) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int r = wave_m * 32 * TM + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                        const int c = wave_n * 32 * TN + j * 32 + l32;
                        lds[r * (BN + 1) + c] = acc[i][j][v];
                    }
        }
        __syncthreads();
        if (n_doubts) {
            half_settle<BM, BN>(P, doubts, n_doubts, tm, tn, k0, k1, tid, lds, BN + 1);
            __syncthreads();
        }
        store_slab<BM, BN>(P, lds, tm * BM, tn * BN, diag_tile, tid);
    }
}

template <int TM, int TN>
__global__ __launch_bounds__(256, TM * TN == 1 ? 4 : 2) void gemm_nt_f32_split_kernel(const GemmProblem *__restrict__ probs,
                                                                            const int *__restrict__ tile_start, int n_probs)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // operand stages, then the output tile; scales behind
    const int wg = blockIdx.x;
    const int pi = find_problem(tile_start, n_probs, wg);
    const GemmProblem &P = probs[pi];
    const int local = wg - tile_start[pi];
    if (local >= n_workgroups(P)) return;   // padding up to the next problem
    int tile, split;
    const bool part_of_k = locate_tile(P, local, tile, split);   // neighbours: neighbouring tiles of the same K range
    gemm_nt_f32_split_tile<TM, TN>(P, tile, split, part_of_k, lds);
}

// ------------------------------------------------------------------ bf16 operand loader
// Same scheme as the fp32 loader with 64-wide K tiles: a thread owns one chunk of 8 bf16
// (16 bytes, 16-byte aligned: the host only contracts NCHW tensors in place when
// hw % 8 == 0 and the base is aligned; everything else goes through the repack kernel,
// whose rows are padded) of the rows r0 + 32*s.
constexpr int KTH = 64;     // contraction tile of the bf16 kernel
constexpr int LDH = 72;     // LDS row length in bf16 (64 + 8 pad: 144-byte rows, conflict-free 16-byte reads)
typedef const unsigned short __attribute__((address_space(1))) *gushort_ptr;
typedef const ushortx8 __attribute__((address_space(1))) *gushort8_ptr;

template <int BR, bool TAIL = false>
struct LoaderBF16 {
    static constexpr int SLOTS = BR / 32;
    gushort_ptr base;
    long long rowoff[SLOTS];
    unsigned dead;
    long long batch_stride;
    long long col;             // offset of the thread's chunk within a row: n * batch_stride + t
    int hw, kq, r0, m, n, t;
    int tail;                  // see Operand
    int n_last;                // TAIL: index of the last run of a row
    unsigned lastrow;          // TAIL: bit s set if slot s reads the last row of the operand
    bool zero_all;

    __device__ __forceinline__ void init(const Operand &op, int tile_row0, int tid, int K = 0)
    {
        base = (gushort_ptr)op.base;
        batch_stride = op.batch_stride;
        hw = op.hw;
        tail = op.tail;
        kq = (tid & 7) * 8; r0 = tid >> 3;
        dead = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int row = tile_row0 + r0 + 32 * s;
            if (row >= op.rows) dead |= 1u << s;
            rowoff[s] = (long long)min(row, op.rows - 1) * op.row_stride;
        }
        m = n = t = 0;
        col = 0;
        zero_all = false;
        n_last = 0;
        lastrow = 0;
        if constexpr (TAIL) {
            n_last = K / hw - 1;
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (tile_row0 + r0 + 32 * s >= op.rows - 1) lastrow |= 1u << s;
        }
    }
    __device__ __forceinline__ void seek(int tile_k0)
    {
        m = tile_k0 + kq;
        n = m / hw;
        t = m - n * hw;
        col = (long long)n * batch_stride + t;
    }
    __device__ __forceinline__ void advance()
    {
        m += KTH; t += KTH; col += KTH;
        while (t >= hw) {
            t -= hw; col += batch_stride - hw;
            if constexpr (TAIL) ++n;
        }
    }
    // the same for runs of at least one tile (hw >= KTH): at most one wrap, no branch
    __device__ __forceinline__ void advance_once()
    {
        m += KTH; t += KTH; col += KTH;
        const bool wrap = t >= hw;
        t -= wrap ? hw : 0;
        col += wrap ? batch_stride - hw : 0;
        if constexpr (TAIL) n += wrap ? 1 : 0;
    }
    // The thread's chunk of row slot s.  Runs with a tail: the last chunk of a run is loaded whole as well (its
    // upper half lies in the next row of the tensor) and the upper half set to zero; only behind the last run
    // of the last row there is no next row, so that one chunk is loaded four elements lower and moved up.
    __device__ __forceinline__ ushortx8 fetch(int s) const
    {
        const long long off = rowoff[s] + col;
        if constexpr (!TAIL) return *(gushort8_ptr)(base + off);
        typedef unsigned short ushortx8_a8 __attribute__((ext_vector_type(8), aligned(8)));
        typedef const ushortx8_a8 __attribute__((address_space(1))) *gushort8a8_ptr;
        const bool last = tail != 0 && t + 8 == hw;
        const bool edge = last && n == n_last && ((lastrow >> s) & 1);
        const ushortx8_a8 v = *(gushort8a8_ptr)(base + off - (edge ? 4 : 0));
        ushortx8 r = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
        if (edge) { r[0] = v[4]; r[1] = v[5]; r[2] = v[6]; r[3] = v[7]; }
        if (last) { r[4] = 0; r[5] = 0; r[6] = 0; r[7] = 0; }
        return r;
    }
    __device__ __forceinline__ void load_full(ushortx8 (&reg)[SLOTS])
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) reg[s] = fetch(s);
        zero_all = false;
    }
    __device__ __forceinline__ void zero_below(int mlo) { zero_all = m < mlo; }
    __device__ __forceinline__ void load_careful(ushortx8 (&reg)[SLOTS], int kend8)
    {
        const bool in = m < kend8;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            ushortx8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (in) v = fetch(s);
            reg[s] = v;
        }
        zero_all = !in;
    }
    static __device__ __forceinline__ float widen(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
    template <bool RS>
    __device__ __forceinline__ void store_lds(const ushortx8 (&reg)[SLOTS], unsigned short *lds, float (&rs)[SLOTS]) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            ushortx8 v = reg[s];
            if (((dead >> s) & 1) || zero_all) v = ushortx8{0, 0, 0, 0, 0, 0, 0, 0};
            if constexpr (RS)
                rs[s] += ((widen(v[0]) + widen(v[1])) + (widen(v[2]) + widen(v[3]))) +
                         ((widen(v[4]) + widen(v[5])) + (widen(v[6]) + widen(v[7])));
            *(ushortx8 *)(lds + (r0 + 32 * s) * LDH + kq) = v;
        }
    }
    // one slot of a tile without masked rows (dead == 0, not zero_all)
    template <bool RS>
    __device__ __forceinline__ void store_slot(const ushortx8 (&reg)[SLOTS], unsigned short *lds, float (&rs)[SLOTS], int s) const
    {
        const ushortx8 v = reg[s];
        if constexpr (RS)
            rs[s] += ((widen(v[0]) + widen(v[1])) + (widen(v[2]) + widen(v[3]))) +
                     ((widen(v[4]) + widen(v[5])) + (widen(v[6]) + widen(v[7])));
        *(ushortx8 *)(lds + (r0 + 32 * s) * LDH + kq) = v;
    }
    __device__ __forceinline__ void load_slot(ushortx8 (&reg)[SLOTS], int s)
    {
        reg[s] = fetch(s);
    }
    // K % 8 remainder tile (repacked operands only): thread tid < BR fills LDS row tid
    __device__ __forceinline__ static float fill_remainder(const Operand &op, int tile_row0, int k8, int kend,
                                                           int tid, unsigned short *lds)
    {
        if (tid >= BR) return 0.f;
        const int row = tile_row0 + tid;
        ushortx8 x = {0, 0, 0, 0, 0, 0, 0, 0};
        if (row < op.rows) {
            gushort_ptr p = (gushort_ptr)op.base + (long long)row * op.row_stride + k8;
            for (int e = 0; e < 7; ++e)
                if (k8 + e < kend) x[e] = p[e];
        }
        unsigned short *dst = lds + tid * LDH;
        *(ushortx8 *)dst = x;
#pragma unroll
        for (int q = 1; q < 8; ++q) *(ushortx8 *)(dst + 8 * q) = ushortx8{0, 0, 0, 0, 0, 0, 0, 0};
        float sum = 0.f;
        for (int e = 0; e < 7; ++e) sum += widen(x[e]);
        return sum;
    }
};

// ------------------------------------------------------------------ bf16 kernel
// The software pipeline of the fp32 kernel with 64-wide K tiles.  v_mfma_f32_32x32x16_bf16: a
// lane supplies 8 consecutive k of row lane % 32, the two half-waves supply two different k
// groups; step u (0..3) of a tile uses k = 16u + 8*half + 0..7, identically for both operands.
// A matrix instruction takes a quarter of the time of the fp32 one while a tile moves the same
// number of bytes, so the stores and loads are dealt out over the first three steps.
template <int TM, int TN>
struct FragBF16 {
    ushortx8 a[TM], b[TN];
};

template <int TM, int TN>
__device__ __forceinline__ void read_frag16(FragBF16<TM, TN> &f, const unsigned short *pa, const unsigned short *pb, int u)
{
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = *(const ushortx8 *)(pa + i * 32 * LDH + 16 * u);
#pragma unroll
    for (int j = 0; j < TN; ++j) f.b[j] = *(const ushortx8 *)(pb + j * 32 * LDH + 16 * u);
}

template <int TM, int TN>
__device__ __forceinline__ void mma_frag16(const FragBF16<TM, TN> &f, floatx16 (&acc)[TM][TN])
{
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.a[i]),
                                                                __builtin_bit_cast(bf16x8, f.b[j]), acc[i][j], 0, 0, 0);
}

// SAME: as in gemm_split_mainloop (a diagonal tile of a Gram matrix stages its operand tile once).
template <int TM, int TN, bool LIVE, bool RS, bool TAIL, bool SAME>
__device__ __forceinline__ void gemm_bf16_mainloop(const GemmProblem &P, int tm, int tn, int tid,
                                                   LoaderBF16<64 * TM, TAIL> &la, LoaderBF16<64 * TN, TAIL> &lb,
                                                   unsigned short *lds, int k0, int k1, int wave_m, int wave_n,
                                                   int l32, int half, floatx16 (&acc)[TM][TN], float (&rs)[2 * TM],
                                                   float &rs_rem)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int STAGE = (BM + BN) * LDH;
    const int klen = max(k1 - k0, 0);
    const int klen8 = klen & ~7;
    const int nfull = klen8 / KTH;
    const bool shifted = nfull > 0 && klen8 > nfull * KTH;
    const bool careful = nfull == 0 && klen8 > 0;
    const int nvec = nfull + ((shifted || careful) ? 1 : 0);
    const int nk = nvec + (klen8 < klen ? 1 : 0);
    if (nk == 0) return;
    ushortx8 ra[BM / 32], rb[BN / 32];

    auto load_tile = [&](int it) {
        if (it < nfull) {
            if constexpr (SAME) {
                if (it > 0) la.advance();
                la.load_full(ra);
            } else {
                if (it > 0) { la.advance(); lb.advance(); }
                la.load_full(ra); lb.load_full(rb);
            }
        } else if (it < nvec) {
            if (careful) {
                la.load_careful(ra, k0 + klen8);
                if constexpr (!SAME) lb.load_careful(rb, k0 + klen8);
            } else if constexpr (SAME) {
                la.seek(k0 + klen8 - KTH);
                la.load_full(ra);
                la.zero_below(k0 + nfull * KTH);
            } else {
                la.seek(k0 + klen8 - KTH); lb.seek(k0 + klen8 - KTH);
                la.load_full(ra); lb.load_full(rb);
                la.zero_below(k0 + nfull * KTH);
            }
        }
    };
    auto store_tile = [&](int it) {
        unsigned short *sa = lds + (it & 1) * STAGE, *sb = sa + BM * LDH;
        if (it < nvec) {
            float unused[BN / 32];
            la.template store_lds<RS>(ra, sa, rs);
            if constexpr (!SAME) lb.template store_lds<false>(rb, sb, unused);
        } else {
            rs_rem = LoaderBF16<BM>::fill_remainder(P.a, tm * BM, k0 + klen8, k1, tid, sa);
            if constexpr (!SAME) LoaderBF16<BN>::fill_remainder(P.b, tn * BN, k0 + klen8, k1, tid, sb);
        }
    };
    const int off_a = (wave_m * 32 * TM + l32) * LDH + 8 * half;
    const int off_b = (SAME ? 0 : BM * LDH) + (wave_n * 32 * TN + l32) * LDH + 8 * half;

    if constexpr (SAME) la.seek(k0);
    else { la.seek(k0); lb.seek(k0); }
    load_tile(0);
    store_tile(0);
    load_tile(1);
    __syncthreads();
    FragBF16<TM, TN> f0, f1;
    if constexpr (LIVE) read_frag16<TM, TN>(f0, lds + off_a, lds + off_b, 0);

    auto step = [&](int it) {
        const unsigned short *cur = lds + (it & 1) * STAGE;
        const unsigned short *nxt = lds + ((it + 1) & 1) * STAGE;
        if constexpr (LIVE) read_frag16<TM, TN>(f1, cur + off_a, cur + off_b, 1);
        if (it + 1 < nk) store_tile(it + 1);
        if constexpr (LIVE) mma_frag16<TM, TN>(f0, acc);
        if constexpr (LIVE) read_frag16<TM, TN>(f0, cur + off_a, cur + off_b, 2);
        load_tile(it + 2);
        if constexpr (LIVE) mma_frag16<TM, TN>(f1, acc);
        if constexpr (LIVE) read_frag16<TM, TN>(f1, cur + off_a, cur + off_b, 3);
        if constexpr (LIVE) mma_frag16<TM, TN>(f0, acc);
        __syncthreads();
        if constexpr (LIVE) {
            if (it + 1 < nk) read_frag16<TM, TN>(f0, nxt + off_a, nxt + off_b, 0);
            mma_frag16<TM, TN>(f1, acc);
        }
    };
    auto fast_step = [&](int it) {
        const unsigned short *cur = lds + (it & 1) * STAGE;
        unsigned short *nxt = lds + ((it + 1) & 1) * STAGE;
        constexpr int SA = BM / 32, SB = SAME ? 0 : BN / 32, NOPS = 2 * (SA + SB);
        constexpr int NMMA = LIVE ? 3 * TM * TN : 1;   // matrix instructions ahead of the barrier
        constexpr int PER = (NOPS + NMMA - 1) / NMMA;
        auto side_op = [&](int k) {   // k-th of: stores of a, stores of b, loads of a, loads of b
            if (k < SA) {
                la.template store_slot<RS>(ra, nxt, rs, k);
            } else if (k < SA + SB) {
                if constexpr (!SAME) {
                    float unused[BN / 32];
                    lb.template store_slot<false>(rb, nxt + BM * LDH, unused, k - SA);
                }
            } else if (k < 2 * SA + SB) {
                if (k == SA + SB) {
                    if constexpr (SAME) la.advance_once();
                    else { la.advance_once(); lb.advance_once(); }
                }
                la.load_slot(ra, k - SA - SB);
            } else if (k < NOPS) {
                if constexpr (!SAME) lb.load_slot(rb, k - 2 * SA - SB);
            }
        };
        if constexpr (LIVE) {
            int n = 0;
            // step u multiplies the fragments read during step u - 1 and reads those of step u + 1
            auto group = [&](FragBF16<TM, TN> &use, FragBF16<TM, TN> &fill, int u_fill) {
                read_frag16<TM, TN>(fill, cur + off_a, cur + off_b, u_fill);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, use.a[i]),
                                                                            __builtin_bit_cast(bf16x8, use.b[j]),
                                                                            acc[i][j], 0, 0, 0);
#pragma unroll
                        for (int q = 0; q < PER; ++q) side_op(n * PER + q);
                        ++n;
                        __builtin_amdgcn_sched_barrier(0);
                    }
            };
            group(f0, f1, 1);
            group(f1, f0, 2);
            group(f0, f1, 3);
            __syncthreads();
            read_frag16<TM, TN>(f0, nxt + off_a, nxt + off_b, 0);
            __builtin_amdgcn_sched_barrier(0);
            mma_frag16<TM, TN>(f1, acc);
        } else {
#pragma unroll
            for (int k = 0; k < NOPS; ++k) side_op(k);
            __syncthreads();
        }
    };
    int it = 0;
    // (a condition the whole workgroup agrees on: every row of both operand tiles exists)
    if (la.hw >= KTH && lb.hw >= KTH && (tm + 1) * BM <= P.a.rows && (tn + 1) * BN <= P.b.rows)
        for (; it + 2 < nfull; ++it) fast_step(it);
    for (; it < nk; ++it) step(it);
}

// ------------------------------------------------------------------ bf16 operands stored transposed
// As LoaderF32T / gemm_split_mainloop_trans with one plane and no conversion: a thread loads 16 bytes = eight
// adjacent rows at one m and stores them as they are into the [m][row] tile; rows % 8 == 0, 16-byte aligned base.
template <int BR>
struct LoaderBF16T {
    static constexpr int CG = BR / 8;
    static constexpr int MSTEP = 256 / CG;
    static constexpr int SLOTS = KT / MSTEP;   // K tiles of 32 here
    static constexpr int RS = BR + 16;
    gushort_ptr base;
    long long ld;
    int c_local, c_load, mk, K;
    bool dead;

    __device__ __forceinline__ void init(const Operand &op, int tile_row0, int tid, int K_)
    {
        base = (gushort_ptr)op.base;
        ld = op.row_stride;
        c_local = 8 * (tid % CG);
        mk = tid / CG;
        const int c = tile_row0 + c_local;
        dead = c >= op.rows;
        c_load = min(c, op.rows - 8);
        K = K_;
    }
    __device__ __forceinline__ void load(ushortx8 (&reg)[SLOTS], int tile_m0) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int m = min(tile_m0 + mk + MSTEP * s, K - 1);
            reg[s] = *(gushort8_ptr)(base + (long long)m * ld + c_load);
        }
    }
    template <bool RSUM>
    __device__ __forceinline__ void store(const ushortx8 (&reg)[SLOTS], unsigned short *rows, int tile_m0, int mend,
                                          float (&rs)[8]) const
    {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            ushortx8 v = reg[s];
            const int ml = mk + MSTEP * s;
            if (dead || tile_m0 + ml >= mend) v = ushortx8{0, 0, 0, 0, 0, 0, 0, 0};
            if constexpr (RSUM) {
#pragma unroll
                for (int e = 0; e < 8; ++e) rs[e] += __uint_as_float((unsigned)v[e] << 16);
            }
            *(ushortx8 *)(rows + ml * RS + c_local) = v;
        }
    }
};

template <int TM, int TN, bool LIVE, bool RSUM>
__device__ __forceinline__ void gemm_bf16_mainloop_trans(const GemmProblem &P, int tm, int tn, int tid,
                                                         unsigned short *lds, int k0, int k1, int wave_m, int wave_n,
                                                         int lane, floatx16 (&acc)[TM][TN], float (&rs)[8])
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int RSA = LoaderBF16T<BM>::RS, RSB = LoaderBF16T<BN>::RS;
    unsigned short *lds_b = lds + KT * RSA;
    LoaderBF16T<BM> la;
    LoaderBF16T<BN> lb;
    la.init(P.a, tm * BM, tid, P.K);
    lb.init(P.b, tn * BN, tid, P.K);
    const int nk = (max(k1 - k0, 0) + KT - 1) / KT;
    if (nk == 0) return;
    ushortx8 ra0[LoaderBF16T<BM>::SLOTS], rb0[LoaderBF16T<BN>::SLOTS], ra1[LoaderBF16T<BM>::SLOTS], rb1[LoaderBF16T<BN>::SLOTS];
    const int frag_m = 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int frag_r = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const int off_a = frag_m * RSA + wave_m * 32 * TM + frag_r;
    const int off_b = frag_m * RSB + wave_n * 32 * TN + frag_r;
    auto compute = [&]() {
        if constexpr (LIVE) {
            auto rd = [&](const unsigned short *tile, int rs_, int off, int u) {
                const unsigned short *p = tile + off + 16 * u * rs_;
                const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_ptr)p);
                const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_ptr)(p + 4 * rs_));
                typedef short shortx8 __attribute__((ext_vector_type(8)));
                return __builtin_bit_cast(bf16x8, shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            };
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 a[TM], b[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i] = rd(lds, RSA, off_a + i * 32, u);
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j] = rd(lds_b, RSB, off_b + j * 32, u);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    };
    float unused[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    la.load(ra0, k0); lb.load(rb0, k0);
    la.load(ra1, k0 + KT); lb.load(rb1, k0 + KT);
    for (int it = 0; it < nk; it += 2) {
        if (it > 0) __syncthreads();
        la.template store<RSUM>(ra0, lds, k0 + it * KT, k1, rs);
        lb.template store<false>(rb0, lds_b, k0 + it * KT, k1, unused);
        la.load(ra0, k0 + (it + 2) * KT); lb.load(rb0, k0 + (it + 2) * KT);
        __syncthreads();
        compute();
        if (it + 1 < nk) {
            __syncthreads();
            la.template store<RSUM>(ra1, lds, k0 + (it + 1) * KT, k1, rs);
            lb.template store<false>(rb1, lds_b, k0 + (it + 1) * KT, k1, unused);
            la.load(ra1, k0 + (it + 3) * KT); lb.load(rb1, k0 + (it + 3) * KT);
            __syncthreads();
            compute();
        }
    }
}

// TAIL: an operand of the problem has runs with a four-element tail (Operand::tail); a variant of its
// own, so that the loads of all other problems stay single 16-byte loads without a branch.
template <int TM, int TN, bool TAIL, bool TRANS = false>
__device__ __forceinline__ void gemm_nt_bf16_body(const GemmProblem &P, int local, float *lds)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    int tile, split, tm, tn;
    const bool part_of_k = locate_tile(P, local, tile, split);
    decode_tile(P, tile, tm, tn);
    const int k0 = split * P.k_per_split;
    const int k1 = part_of_k ? min(P.K, k0 + P.k_per_split) : P.K;
    const int tid = threadIdx.x;

    LoaderBF16<BM, TAIL> la;
    LoaderBF16<BN, TAIL> lb;
    la.init(P.a, tm * BM, tid, P.K);
    lb.init(P.b, tn * BN, tid, P.K);

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int lane = tid & 63, wid = tid >> 6;
    const int wave_m = wid >> 1, wave_n = wid & 1;
    const int l32 = lane & 31, half = lane >> 5;
    const bool diag_tile = (P.flags & GEMM_SYM) && tm == tn;
    const int wave_r0 = tm * BM + wave_m * 32 * TM, wave_c0 = tn * BN + wave_n * 32 * TN;
    const bool live = wave_r0 < P.M && wave_c0 < P.N && !(diag_tile && wave_c0 >= wave_r0 + 32 * TM);

    unsigned short *lds16 = (unsigned short *)lds;
    const bool border = diag_tile && (P.flags & GEMM_BORDER);
    float rs[BM / 32], rs_rem = 0.f;
#pragma unroll
    for (int s = 0; s < BM / 32; ++s) rs[s] = 0.f;
    if constexpr (TRANS) {
        float rst[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (border) {
            if (live) gemm_bf16_mainloop_trans<TM, TN, true, true>(P, tm, tn, tid, lds16, k0, k1, wave_m, wave_n, lane, acc, rst);
            else      gemm_bf16_mainloop_trans<TM, TN, false, true>(P, tm, tn, tid, lds16, k0, k1, wave_m, wave_n, lane, acc, rst);
            finish_row_sums_trans<BM, 8>(P, lds, tm, tile, split, tid, rst);
        } else {
            if (live) gemm_bf16_mainloop_trans<TM, TN, true, false>(P, tm, tn, tid, lds16, k0, k1, wave_m, wave_n, lane, acc, rst);
            else      gemm_bf16_mainloop_trans<TM, TN, false, false>(P, tm, tn, tid, lds16, k0, k1, wave_m, wave_n, lane, acc, rst);
        }
    } else {
        // a diagonal tile of a Gram matrix (a and b the same operand) stages its operand tile once (64 x 64 tiles
        // only: the large tile has no registers to spare for one more copy of the main loop)
        constexpr bool CAN_SHARE = TM == 1 && TN == 1;
        const bool same = CAN_SHARE && tm == tn && P.a.base == P.b.base && P.a.row_stride == P.b.row_stride &&
                          P.a.batch_stride == P.b.batch_stride && P.a.hw == P.b.hw && P.a.rows == P.b.rows;
        auto mainloop = [&](auto live_c, auto rs_c) {
            constexpr bool LV = decltype(live_c)::value, RSUM = decltype(rs_c)::value;
            if (CAN_SHARE && same)
                gemm_bf16_mainloop<TM, TN, LV, RSUM, TAIL, CAN_SHARE>(P, tm, tn, tid, la, lb, lds16, k0, k1, wave_m, wave_n, l32, half, acc, rs, rs_rem);
            else
                gemm_bf16_mainloop<TM, TN, LV, RSUM, TAIL, false>(P, tm, tn, tid, la, lb, lds16, k0, k1, wave_m, wave_n, l32, half, acc, rs, rs_rem);
        };
        if (border) {
            if (live) mainloop(std::true_type{}, std::true_type{});
            else      mainloop(std::false_type{}, std::true_type{});
            finish_row_sums<BM>(P, lds, tm, tile, split, tid, rs, rs_rem);
        } else {
            if (live) mainloop(std::true_type{}, std::false_type{});
            else      mainloop(std::false_type{}, std::false_type{});
        }
    }

    if (part_of_k) {
        const Global<float> part = global(P.partial) + ((long long)(tile - P.split_from) * P.splits + split) * (BM * BN);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = wave_m * 32 * TM + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                    const int c = wave_n * 32 * TN + j * 32 + l32;
                    part[r * BN + c] = acc[i][j][v];
                }
    } else {
        __syncthreads();
        if (live) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int r = wave_m * 32 * TM + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                        const int c = wave_n * 32 * TN + j * 32 + l32;
                        lds[r * (BN + 1) + c] = acc[i][j][v];
                    }
        }
        __syncthreads();
        store_slab<BM, BN>(P, lds, tm * BM, tn * BN, diag_tile, tid);
    }
}

// ------------------------------------------------------------------ split-K reduction + epilogue
// One workgroup per slab of rows of a partial tile: sums the partial tiles in a fixed order (reproducible bit for bit) into
// LDS and applies the same row-wise epilogue.  red_start counts slabs.  A chain of load latencies where the splits are many
// and the tiles few (13 tiles of 147 parts for the 64-channel correlations): slabs of 8 rows then (red_rows), the splits dealt
// to the thread groups a slab leaves, 8 loads in flight a thread, the border's row sums likewise: those 13 tiles 13 us,
// ResNet-50's 64-row tiles (bf16) 17 us.
// Few splits stream at the memory's rate and keep slabs of 32 rows, whose mirror image is written in 128-byte pieces.
template <int B, int ROWS>
__device__ __forceinline__ void reduce_slab(const GemmProblem &P, int tile, int slab, int tm, int tn, float *T, floatx4 *sums)
{
    static_assert(B % ROWS == 0 && ROWS % 4 == 0 && ROWS <= kRedRows && B <= 128, "slabs of a tile, in T");
    static_assert((ROWS * B / 4) % 256 == 0 || 256 % (ROWS * B / 4) == 0, "whole passes, or whole groups of threads");
    const bool diag_tile = (P.flags & GEMM_SYM) && tm == tn;
    const Global<const float> part = global((const float *)P.partial) + (long long)(tile - P.split_from) * P.splits * (B * B) + slab * ROWS * B;
    // ROWS * B elements, 4 per thread per pass; where they are fewer than 4 per thread, `groups` groups of threads take every
    // groups-th split.  A thread's U splits in flight go into U partial sums.
    constexpr int VECS = ROWS * B / 4, PASSES = VECS >= 256 ? VECS / 256 : 1, GROUPS = VECS >= 256 ? 1 : 256 / VECS;
    constexpr int U = PASSES > 1 ? 4 : 8;
    const int group = GROUPS > 1 ? (int)threadIdx.x / VECS : 0, vec = GROUPS > 1 ? (int)threadIdx.x % VECS : (int)threadIdx.x;
    floatx4 acc[PASSES][U];
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
#pragma unroll
        for (int k = 0; k < U; ++k) acc[p][k] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int q = group; q < P.splits; q += U * GROUPS) {
        floatx4 v[PASSES][U];
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int p = 0; p < PASSES; ++p) {
                v[p][k] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (q + k * GROUPS < P.splits)
                    v[p][k] = __builtin_nontemporal_load((Global<const floatx4>)(part + (long long)(q + k * GROUPS) * (B * B) + vec * 4 + p * 1024));
            }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int p = 0; p < PASSES; ++p) acc[p][k] += v[p][k];
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
#pragma unroll
        for (int d = U / 2; d > 0; d /= 2)
#pragma unroll
            for (int k = 0; k < d; ++k) acc[p][k] += acc[p][k + d];
        floatx4 s = acc[p][0];
        if constexpr (GROUPS > 1) {
            sums[threadIdx.x] = s;
            __syncthreads();
            if (group == 0)
#pragma unroll
                for (int g = 1; g < GROUPS; ++g) s += sums[g * VECS + vec];
        }
        const int e = vec * 4 + p * 1024;
        const int r = e / B, c = e - r * B;
        float *t = T + r * (B + 1) + c;
        if (group == 0) { t[0] = s[0]; t[1] = s[1]; t[2] = s[2]; t[3] = s[3]; }
    }
    __syncthreads();
    store_slab<ROWS, B>(P, T, tm * B + slab * ROWS, tn * B, diag_tile, threadIdx.x);
    if (diag_tile && (P.flags & GEMM_BORDER)) {
        // the row sums: the splits dealt to groups of ROWS threads, whose sums are added in order (one thread after all the
        // splits of its row is a chain of memory latencies: 79 of them cost 15 us)
        constexpr int RG = 256 / ROWS;
        const int r = threadIdx.x % ROWS, g = threadIdx.x / ROWS;
        const Global<const float> prs = global((const float *)P.partial_rs) + (long long)tm * P.splits * B + slab * ROWS + r;
        float sum = 0.f;
        for (int q = g; q < P.splits; q += RG) sum += prs[(long long)q * B];
        float *part_sums = (float *)sums;
        __syncthreads();
        part_sums[threadIdx.x] = sum;
        __syncthreads();
        const int row = tm * B + slab * ROWS + threadIdx.x;
        if (threadIdx.x < ROWS && row < P.M) {
            float total = 0.f;
            for (int q = 0; q < RG; ++q) total += part_sums[q * ROWS + threadIdx.x];
            store_border(P, row, total);
        }
        if (tile == 0 && slab == 0 && threadIdx.x == 0) store_corner(P);
    }
}

__global__ __launch_bounds__(256) void gemm_reduce_kernel(const GemmProblem *__restrict__ probs,
                                                          const int *__restrict__ red_start, int n_probs)
{
    __shared__ float T[kRedRows * 129];
    __shared__ floatx4 sums[256];
    const int wg = blockIdx.x;
    const int pi = find_problem(red_start, n_probs, wg);
    const GemmProblem &P = probs[pi];
    if (P.splits <= 1) return;
    const int B = (P.tile_cfg == 0) ? 128 : 64;
    const int rows = red_rows(P.splits), slabs = B / rows;
    const int local = wg - red_start[pi];
    const int tile = P.split_from + local / slabs;
    const int slab = local % slabs;
    int tm, tn;
    decode_tile(P, tile, tm, tn);
    if (tm * B + slab * rows >= P.M) return;
    if (rows == kRedRows) {
        if (B == 128) reduce_slab<128, kRedRows>(P, tile, slab, tm, tn, T, sums);
        else               reduce_slab<64, kRedRows>(P, tile, slab, tm, tn, T, sums);
    } else {
        if (B == 128) reduce_slab<128, kRedRowsMany>(P, tile, slab, tm, tn, T, sums);
        else               reduce_slab<64, kRedRowsMany>(P, tile, slab, tm, tn, T, sums);
    }
}

// (the small tile held to 128 registers: four workgroups a compute unit, as many as its LDS allows, instead of three;
// ResNet-50's 64-row tiles 265 -> 247 us)
template <int TM, int TN>
__global__ __launch_bounds__(256, TM * TN == 1 ? 4 : 1) void gemm_nt_bf16_kernel(const GemmProblem *__restrict__ probs,
                                                           const int *__restrict__ tile_start, int n_probs)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // operand stages, then the output tile

    const int wg = blockIdx.x;
    const int pi = find_problem(tile_start, n_probs, wg);
    const GemmProblem &P = probs[pi];
    const int local = wg - tile_start[pi];
    if (local >= n_workgroups(P)) return;
    if (P.a.tail | P.b.tail) gemm_nt_bf16_body<TM, TN, true>(P, local, lds);
    else                     gemm_nt_bf16_body<TM, TN, false>(P, local, lds);
}
template <int TM, int TN>
__global__ __launch_bounds__(256) void gemm_nt_bf16_trans_kernel(const GemmProblem *__restrict__ probs,
                                                                 const int *__restrict__ tile_start, int n_probs)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int wg = blockIdx.x;
    const int pi = find_problem(tile_start, n_probs, wg);
    const GemmProblem &P = probs[pi];
    const int local = wg - tile_start[pi];
    if (local >= n_workgroups(P)) return;
    gemm_nt_bf16_body<TM, TN, false, true>(P, local, lds);
}

// ------------------------------------------------------------------ the displaced products of one image together
// The 13 products of a padded image of up to 64 channels with itself displaced by (dy, dx) (corr.hip), as parts of their
// contraction (the partial tiles of gemm_reduce_kernel).  One by one, as 64-row tiles, each of them read its two operands from
// memory: 26 times the tensor, which bound them (64 channels at 56 x 56, 32 samples, bf16: 1.36 GB and 165 us for three layers;
// fp32: 26 conversions of every element as well).  Here a workgroup stages the rows of the image and of six displaced ones in LDS
// and forms seven (or six) products out of them: two workgroups, on the same XCD, share a part.  7 x 16 accumulators leave
// two workgroups to a compute unit (all thirteen in one: 208, one workgroup, and half the parts).
// Three images of 64 channels at 56 x 56: fp32 187 -> 135 us with 32 samples (255 TFLOP/s), 959 -> 437 with 128 (315), 500 once the
// clock has gone down to 1.9 GHz; bf16 130 -> 127 with 32, 414 (365 TFLOP/s) with 128.  Bound: fp32 by power, at that clock with the matrix
// unit busy 0.39 to 0.47 of the time; bf16 (0.13 to 0.16, at 2.2 GHz, wavefronts waiting 0.7 of the time) by the loads of a step, which wait
// for its barrier (one stage: two would leave one workgroup to a compute unit).  Errors of the factors against 64 bits, over batches of 8 to 128, 17 to 64 channels and 28 to 112
// positions a side: fp32 0.88, bf16 0.96 of those of single products.
// A thread loads and stores 16 bytes of two rows of every staged tile: the tiles differ by a uniform base address only.  (The planes
// of a padded image have at least 28 positions in fp32 and 40 in bf16, so that a step wraps twice at most.)
constexpr int DISP_TILES = 7, DISP_TILE_BYTES = 8192, DISP_STAGE = DISP_TILES * DISP_TILE_BYTES;
constexpr int DISP_SCALES = DISP_STAGE / 4, DISP_DOUBTS = DISP_SCALES + 384, DISP_INFINITE = DISP_DOUBTS + DISP_TILES * (1 + kMaxDoubts);   // in LDS, words
constexpr size_t displaced_lds_bytes() { return (DISP_INFINITE + 1) * sizeof(float); }

// Position of a thread's chunk in the contraction.
struct DisplacedCursor {
    unsigned at;               // byte offset from a tile's base address
    int t, m;
    __device__ __forceinline__ void seek(const Operand &op, int row, int m_, int esize)
    {
        m = m_;
        const int n = m / op.hw;
        t = m - n * op.hw;
        at = (unsigned)((n * op.batch_stride + (long long)row * op.row_stride + t) * esize);
    }
    // by `step` < 2 hw positions; beyond kend: where it is (what is read there counts as zero)
    __device__ __forceinline__ void advance(const Operand &op, int step, int kend, int esize)
    {
        m += step;
        if (m >= kend) return;
        t += step;
        at += (unsigned)(step * esize);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool wrap = t >= op.hw;
            t -= wrap ? op.hw : 0;
            at += wrap ? (unsigned)((op.batch_stride - op.hw) * esize) : 0u;
        }
    }
};

// Scales and floors of the 64 rows, as half_scales makes them: 32 sampled elements of each for the floor.  Both sides of the products
// share them, so they are those of [k0, k0 + klen), klen > 16: the rows' own part, which ends at k1, and what the displaced images
// have behind it, up to 2 Wp + 2 positions (what is behind an image is zero there).  take_displaced keeps parts at least twice as long
// as that, so that the samples are those of every displaced image.  The eight places are unevenly spread and the element of a chunk that
// counts for the floor changes: even steps of nearly a plane's length met little but the zero lines above its image (seven images of 3 to 49
// channels, 57 samples, 14 x 14 planes among them: 311 us, 100 without).  sc[0 .. 256): scales of rows and columns and their floors;
// sc[256 .. 384): floors for the product of the image with itself.  False: the two planes do not serve, since more than 16 rows have
// hardly an element, and nearly all sums of theirs would come out in doubt.
__device__ __forceinline__ bool displaced_scales(const Operand &op, int k0, int k1, int klen, float *sc, int tid)
{
    const int row = tid >> 2, kq = 4 * (tid & 3);
    const Global<const char> base = global((const char *)op.base);
    floatx4 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        DisplacedCursor at;
        constexpr int place[8] = {0, 7, 19, 24, 34, 45, 53, 64};   // in 64ths
        at.seek(op, min(row, op.rows - 1), k0 + kq + (((klen - 16) * place[q] / 64) & ~3), 4);
        v[q] = *(Global<const floatx4_u>)(base + at.at);
    }
    float mx = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) mx = max_abs(mx, v[q]);
    mx = fmaxf(mx, __shfl_xor(mx, 1));
    mx = fmaxf(mx, __shfl_xor(mx, 2));
    float scale = half_scale(mx, kHalfTop), f = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float y = fabsf(v[q][q & 3]) * scale;
        f += fminf(y, 16.f) + (y >= kHalfExact ? 0x1p10f : y != 0.f ? 0x1p16f : 0.f);
    }
    f += __shfl_xor(f, 1);
    f += __shfl_xor(f, 2);
    const float floor = half_floor(f, kHalfFloor);
    const bool zero = mx == 0.f, dead = row >= op.rows;
    if ((tid & 3) == 0) {
        sc[row] = sc[64 + row] = zero && !dead ? 0.f : scale;
        sc[128 + row] = sc[192 + row] = sc[256 + row] = sc[320 + row] = dead ? kNoFloor : floor;
    }
    const bool odd = !dead && floor > kHalfFloor;
    if (!__syncthreads_or(odd)) return true;
    if (__syncthreads_count(odd && !zero && (tid & 3) == 0) > 16) return false;
    for (int r = tid >> 6; r < 64; r += 4) {              // rows that sampled as zero are read on until an element is not
        if (sc[r] != 0.f) continue;
        auto largest = [&](int to) {
            float most = 0.f;
            walk_row(op, r, k0, to - k0, tid & 63, [&](const auto &x) {
#pragma unroll
                for (const floatx4 &y : x) most = max_abs(most, y);
                for (int d = 32; d > 0; d >>= 1) most = fmaxf(most, __shfl_xor(most, d));
                return most != 0.f;
            });
            return most;
        };
        const float most = largest(k0 + klen);
        const bool none = most == 0.f || largest(k1) == 0.f;   // none of its own part
        if ((tid & 63) == 0) {
            sc[r] = sc[64 + r] = half_scale(most, kHalfTop);
            if (none) sc[128 + r] = sc[256 + r] = sc[320 + r] = kNoFloor;
            if (most == 0.f) sc[192 + r] = kNoFloor;
        }
    }
    __syncthreads();
    return __syncthreads_count(tid < 64 && sc[192 + (tid & 63)] > kHalfFloor) <= 16;
}

template <bool BF16>
__global__ __launch_bounds__(256, 2) void gemm_displaced_kernel(const GemmProblem *__restrict__ probs, const int *__restrict__ start, int n_groups,
                                                                int *__restrict__ left)
{
    constexpr int KS = BF16 ? 64 : 32, CHUNK = KS / 8, ESIZE = BF16 ? 2 : 4;   // positions a step, a thread's chunk
    extern __shared__ __attribute__((aligned(16))) float lds[];
    char *stage = (char *)lds;
    float *sc = lds + DISP_SCALES;
    int *doubts = (int *)lds + DISP_DOUBTS, *infinite = (int *)lds + DISP_INFINITE;   // doubts: a list for each product
    // the parts of all images in a row, start[]: each image's first (two workgroups of a part on the same XCD, as many parts on each)
    const int wg = blockIdx.x, second = (wg >> 3) & 1, part_of_all = (wg & 7) + 8 * (wg >> 4);
    if (part_of_all >= start[n_groups]) return;
    const int g = find_problem(start, n_groups, part_of_all), split = part_of_all - start[g];
    const GemmProblem *Q = probs + 13 * g;
    const Operand op = Q->a;
    const int k0 = split * Q->k_per_split, k1 = min(Q->K, k0 + Q->k_per_split);
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wave_m = wid >> 1, wave_n = wid & 1, l32 = lane & 31, half = lane >> 5;
    const bool live = 32 * wave_m < op.rows && 32 * wave_n < op.rows;
    const int row = tid >> 3, chunk = tid & 7;            // a thread: this chunk of rows `row` and row + 32

    // tile 0: the image; tile j: the image as displacement 6 * second + j displaces it
    Global<const char> base[DISP_TILES];
    base[0] = global((const char *)op.base);
#pragma unroll
    for (int j = 1; j < DISP_TILES; ++j) base[j] = global((const char *)Q[6 * second + j].b.base);

    float scale[2] = {1.f, 1.f};
    bool one_by_one = false;
    if constexpr (!BF16) {
        if (tid < DISP_TILES) doubts[tid * (1 + kMaxDoubts)] = 0;
        if (tid == 0) *infinite = 0;
        // (the samples of a last part of up to one step, of any four positions more, would reach beyond it; see gemm_nt_f32_split_tile)
        const int to = min(Q->K, (k1 + (int)((base[DISP_TILES - 1] - base[0]) / ESIZE) + 3) & ~3);
        one_by_one = k1 - k0 <= KT || !displaced_scales(op, k0, k1, to - k0, sc, tid);
        scale[0] = sc[row];
        scale[1] = sc[row + 32];
    }
    floatx16 acc[DISP_TILES];
    float rs[2] = {0.f, 0.f};
    if (!one_by_one) {
        typedef std::conditional_t<BF16, ushortx8, floatx4> chunk_t;
        typedef std::conditional_t<BF16, ushortx8, floatx4_u> chunk_mem_t;
        chunk_t reg[DISP_TILES][2];
        DisplacedCursor at;
        at.seek(op, min(row, op.rows - 1), min(k0 + CHUNK * chunk, k1 - CHUNK), ESIZE);
        at.m = k0 + CHUNK * chunk;
        const unsigned down = (unsigned)((min(row + 32, op.rows - 1) - min(row, op.rows - 1)) * op.row_stride * ESIZE);
        bool in = at.m < k1;                              // what the registers hold counts
        auto load = [&]() {
#pragma unroll
            for (int j = 0; j < DISP_TILES; ++j) {
                reg[j][0] = *(Global<const chunk_mem_t>)(base[j] + at.at);
                reg[j][1] = *(Global<const chunk_mem_t>)(base[j] + (at.at + down));
            }
        };
        // 16-byte chunks of a row are permuted so that fragment reads spread over the banks (32 rows further down alike)
        const int to = BF16 ? row * 128 + ((chunk ^ (row & 7)) << 4) : row * 64 + (((chunk >> 1) ^ half_swz(row)) << 4) + 8 * (chunk & 1);
        auto store = [&](int j, int s) {
            char *dst = stage + j * DISP_TILE_BYTES + to + s * (BF16 ? 4096 : 2048);
            chunk_t x = reg[j][s];
            if (j == 0 && !in)
#pragma unroll
                for (int e = 0; e < CHUNK; ++e) x[e] = 0;
            if constexpr (BF16) {
                if (j == 0)
#pragma unroll
                    for (int e = 0; e < 8; e += 2) rs[s] += __uint_as_float((unsigned)x[e] << 16) + __uint_as_float((unsigned)x[e + 1] << 16);
                *(ushortx8 *)dst = x;
            } else {
                if (j == 0) rs[s] += (x[0] + x[1]) + (x[2] + x[3]);
                uint2 h, l;
                split_half_pair(x[0], x[1], scale[s], h.x, l.x);
                split_half_pair(x[2], x[3], scale[s], h.y, l.y);
                *(uint2 *)dst = h;
                *(uint2 *)(dst + 4096) = l;
            }
        };
        // fragments of 32 rows of a tile: bf16 the four 16-wide parts of the step; fp32 its two, of both planes
        struct Frag { ushortx8 v[4]; };
        auto read = [&](int j, int r0) {
            const int r = r0 + l32;
            Frag f;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                f.v[u] = *(const ushortx8 *)(stage + j * DISP_TILE_BYTES +
                                             (BF16 ? r * 128 + (((2 * u + half) ^ (r & 7)) << 4) : r * 64 + (((2 * (u & 1) + half) ^ half_swz(r)) << 4) + 4096 * (u >> 1)));
            return f;
        };
        auto multiply = [&](floatx16 &c, const Frag &a, const Frag &b) {
            if constexpr (BF16) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.v[u]), __builtin_bit_cast(bf16x8, b.v[u]), c, 0, 0, 0);
            } else {
                auto h = [](const ushortx8 &v) { return __builtin_bit_cast(halfx8, v); };
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(h(a.v[u]), h(b.v[u]), c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(h(a.v[u]), h(b.v[u + 2]), c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(h(a.v[u + 2]), h(b.v[u]), c, 0, 0, 0);
                }
            }
        };
        auto partial = [&](int j) { return global(Q[j == 0 ? 0 : 6 * second + j].partial) + (long long)split * 4096 + (32 * wave_m + 4 * half) * 64 + 32 * wave_n + l32; };
        auto at_row = [](int v) { return (8 * (v >> 2) + (v & 3)) * 64; };
        // No chain of sums over more positions than the split rule gives a part (128 parts, 512 to 4096 positions): such lengths are added up in the partial tile
        // (9 to 20 us more where there are two; without it the errors against 64 bits grew by a tenth).
        const int steps = (k1 - k0 + KS - 1) / KS, longest = (min(4096, max(512, (Q->K + 127) / 128)) + KS - 1) / KS;
        const int chains = (steps + longest - 1) / longest, chain = (steps + chains - 1) / chains;
        int left = chain;
        bool first = true;                                // nothing in the partial tiles yet
        load();
#pragma unroll
        for (int j = 0; j < DISP_TILES; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
        for (int k = k0; k < k1; k += KS) {
            __syncthreads();                              // the step before has been read
#pragma unroll
            for (int j = 0; j < DISP_TILES; ++j) {
                store(j, 0);
                store(j, 1);
            }
            at.advance(op, KS, k1, ESIZE);
            in = at.m < k1;
            load();                                       // (behind the last step: the same again)
            __syncthreads();
            if (!live) continue;
            const Frag a = read(0, 32 * wave_m);
            Frag b = read(0, 32 * wave_n);
#pragma unroll
            for (int j = 0; j < DISP_TILES; ++j) {
                Frag next = b;
                if (j + 1 < DISP_TILES) next = read(j + 1, 32 * wave_n);
                __builtin_amdgcn_sched_barrier(0);
                if (j > 0 || !second) multiply(acc[j], a, b);
                __builtin_amdgcn_sched_barrier(0);
                b = next;
            }
            if (--left > 0 || k + KS >= k1) continue;
            left = chain;
#pragma unroll
            for (int j = 0; j < DISP_TILES; ++j) {
                if (j == 0 && second) continue;
                const Global<float> part = partial(j);
                if (!first)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[j][v] += part[at_row(v)];
#pragma unroll
                for (int v = 0; v < 16; ++v) part[at_row(v)] = acc[j][v];
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
            }
            first = false;
        }
        if (!second) {                                     // the border: sums of the rows
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                rs[s] += __shfl_xor(rs[s], 1);
                rs[s] += __shfl_xor(rs[s], 2);
                rs[s] += __shfl_xor(rs[s], 4);
                if (chunk == 0 && (Q->flags & GEMM_BORDER)) global(Q->partial_rs)[(long long)split * 64 + row + 32 * s] = rs[s];
            }
        }
        unsigned mine = 0;
#pragma unroll
        for (int j = 0; j < DISP_TILES; ++j) {
            if (!live || (j == 0 && second)) continue;
            const Global<float> part = partial(j);
            if (!first)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][v] += part[at_row(v)];
            floatx16 one[1][1] = {{acc[j]}};
            if constexpr (!BF16) {
                if (half_doubts<1, 1>(one, j == 0 ? sc + 128 : sc, doubts + j * (1 + kMaxDoubts), wave_m, wave_n, l32, half) & 2) mine |= 1u << j;
                half_unscale_tile<1, 1>(one, sc, wave_m, wave_n, l32, half);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) part[at_row(v)] = one[0][0][v];
        }
        if constexpr (!BF16) {
            if (mine) atomicOr(infinite, (int)mine);
        }
    }
    if constexpr (!BF16) {
        // A few sums in doubt (of rows of random sign, one product in fourteen has some) are formed again here.  Products with more than a
        // single tile settles, or with sums that are not finite, and all of them where the two planes do not serve, are left to the
        // next launch: one after the other here, the few of a launch took up to 100 us, all of them 230.
        __syncthreads();
        int alone = (1 << DISP_TILES) - 1;
        if (!one_by_one) {
            alone = *infinite;
            for (int j = second; j < DISP_TILES; ++j) {
                const int *list = doubts + j * (1 + kMaxDoubts), n = list[0];
                if ((alone >> j) & 1) continue;
                const GemmProblem &P = Q[j == 0 ? 0 : 6 * second + j];
                if (n > min(kMaxDoubts, 24 + (k1 - k0) / 32)) alone |= 1 << j;
                else if (n) half_settle<64, 64>(P, list, n, 0, 0, k0, k1, tid, global(P.partial) + (long long)split * 4096, 64);
            }
        }
        if (tid == 0) global(left)[2 * part_of_all + second] = alone;
    }
}

// The products of a launch on 64-row tiles, and behind them a workgroup for each part of each displaced product, which ends at once
// where gemm_displaced_kernel has not left it: the thirteen of a part one after the other on one XCD.  (Workgroups that take what is left
// in turn would be fewer, but the loop around a tile spills 175 registers; those that end at once cost nothing that can be measured.)
__global__ __launch_bounds__(256, 4) void gemm_nt_f32_split_rest_kernel(const GemmProblem *__restrict__ probs, const int *__restrict__ tile_start,
                                                                        int n_probs, Displaced d)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int own = tile_start[n_probs], wg = blockIdx.x;
    const GemmProblem *P;
    int tile = 0, split;
    bool part_of_k = true;
    if (wg < own) {
        const int pi = find_problem(tile_start, n_probs, wg), local = wg - tile_start[pi];
        P = probs + pi;
        if (local >= n_workgroups(*P)) return;   // padding up to the next problem
        part_of_k = locate_tile(*P, local, tile, split);
    } else {
        const int at = (wg >> 3) - ((own + 7) >> 3);
        if (at < 0) return;
        const int q = 8 * (at / 13) + (wg & 7), r = at % 13;
        if (q >= d.start[d.n_groups] || !((d.left[2 * q + (r > 6)] >> (r > 6 ? r - 6 : r)) & 1)) return;
        const int g = find_problem(d.start, d.n_groups, q);
        P = d.probs + 13 * g + r;
        split = q - d.start[g];
    }
    gemm_nt_f32_split_tile<1, 1>(*P, tile, split, part_of_k, lds);
}

template <typename Kernel, typename... Args>
static hipError_t launch_one(Kernel kernel, bool &configured, size_t lds_bytes, int total_wgs, hipStream_t s, Args... args)
{
    if (!configured) {   // the attribute is per function, set once per process
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kernel<<<dim3(total_wgs), dim3(256), lds_bytes, s>>>(args...);
    return hipGetLastError();
}

// dtype 0: fp32 instruction, 1: bf16, 2: fp32 through planes, 3 / 4: 2 / 1 on operands stored transposed
hipError_t launch_gemm(const GemmProblem *probs_dev, const int *tile_start_dev, int n_probs,
                       int total_wgs, int tile_cfg, int dtype, hipStream_t s)
{
    static_assert(2 * LDH == 4 * LDF, "bf16 and fp32 stages have the same size");
    static_assert(3 * KT * (128 + 16 + 128 + 16) * sizeof(unsigned short) <= gemm_lds_bytes<2, 2>() &&
                  3 * KT * (64 + 16 + 64 + 16) * sizeof(unsigned short) <= gemm_lds_bytes<1, 1>(), "three transposed planes fit");
    if (total_wgs <= 0) return hipSuccess;
    static bool configured[5][2];
    auto go = [&](auto kernel, size_t lds_bytes) {
        return launch_one(kernel, configured[dtype][tile_cfg == 0], lds_bytes, total_wgs, s, probs_dev, tile_start_dev, n_probs);
    };
    constexpr size_t big = gemm_lds_bytes<2, 2>(), small = gemm_lds_bytes<1, 1>();
    switch (dtype) {
        case 0: return tile_cfg == 0 ? go(gemm_nt_f32_kernel<2, 2>, big) : go(gemm_nt_f32_kernel<1, 1>, small);
        case 1: return tile_cfg == 0 ? go(gemm_nt_bf16_kernel<2, 2>, big) : go(gemm_nt_bf16_kernel<1, 1>, small);
        case 3: return tile_cfg == 0 ? go(gemm_nt_f32_split_trans_kernel<2, 2>, big) : go(gemm_nt_f32_split_trans_kernel<1, 1>, small);
        case 4: return tile_cfg == 0 ? go(gemm_nt_bf16_trans_kernel<2, 2>, big) : go(gemm_nt_bf16_trans_kernel<1, 1>, small);
    }
    if (tile_cfg == 0) return go(gemm_nt_f32_split_kernel<2, 2>, split_lds_bytes<2, 2>());
    return go(gemm_nt_f32_split_kernel<1, 1>, split_lds_bytes<1, 1>());
}

hipError_t launch_gemm_displaced(const Displaced &d, int total_wgs, int bf16, hipStream_t s)
{
    static bool configured[2];
    return launch_one(bf16 ? gemm_displaced_kernel<true> : gemm_displaced_kernel<false>, configured[bf16 != 0], displaced_lds_bytes(), total_wgs, s,
                      d.probs, d.start, d.n_groups, d.left);
}

hipError_t launch_gemm_rest(const GemmProblem *probs_dev, const int *tile_start_dev, int n_probs, const Displaced &d, int total_wgs, hipStream_t s)
{
    static bool configured;
    return launch_one(gemm_nt_f32_split_rest_kernel, configured, split_lds_bytes<1, 1>(), total_wgs, s, probs_dev, tile_start_dev, n_probs, d);
}

hipError_t launch_gemm_reduce(const GemmProblem *probs_dev, const int *red_start_dev, int n_probs,
                              int total_wgs, hipStream_t s)
{
    if (total_wgs <= 0) return hipSuccess;
    gemm_reduce_kernel<<<dim3(total_wgs), dim3(256), 0, s>>>(probs_dev, red_start_dev, n_probs);
    return hipGetLastError();
}

}  // namespace kfac
