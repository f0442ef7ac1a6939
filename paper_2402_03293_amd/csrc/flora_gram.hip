// The reduction passes of the factored Adafactor rule (the base optimizer of the paper's
// experiments, Section 3.1) without the n x m product.  With Gt = alpha S A^T (S the n x r
// state, A the m x r projection) the row sums, column sums and the clipping sum of the rule are
// quadratic forms in r x r Gram matrices:
//     sum_j Gt_ij^2              = alpha^2 S_i P S_i^T,   P  = A^T A          (r x r, sum over m)
//     sum_i Gt_ij^2              = alpha^2 A_j Q A_j^T,   Q  = S^T S          (r x r, sum over n)
//     sum_ij Gt_ij^2 / (R_i K_j) = alpha^2 sum_i (S_i P' S_i^T) / R_i,   P' = A^T diag(1 / K) A
// which costs 6 (m + n) r^2 flops per matrix instead of the 4 n m r of two passes over the
// decompressed gradient.  Everything runs on the bf16 matrix cores with fp32 accumulation, the
// precision of the decompression itself: A and S are rounded to bf16 exactly as the update pass
// rounds them, the Gram matrices are accumulated in fp32 and rounded to bf16 once.
//
// What the kernels cost is regenerating A (the vector ALU), so the sums are ordered to sweep A
// twice, not three times: Q from one read of S and the column statistics K from a sweep over
// generated rows of A; then ONE further sweep over A yields both P and P'; then the row statistics
// R and the clipping sum from one read of S.
//
// gram_sym_kernel (ranks >= 128) / gram_block_kernel (P and P' of few chunks, and at rank 64) / gram_kernel (Q at rank
//   64): one workgroup sums X_t X_t^T over a chunk
//   of the long index t (X_t = row t of A, regenerated, plain and scaled with 1 / K_t; or row t of
//   S, loaded) into partial r x r matrices; tiles of 64 t are staged in LDS transposed ([k][t],
//   bf16), both MFMA operands come from there.  combine_gram_kernel adds the chunks' partials in
//   chunk order and stores the result as bf16 in the arrangement the quadratic-form kernel that
//   reads it copies into LDS.
// quadform_rows_kernel: q_i = Z_i B Z_i^T for a block of rows of Z = S, B a Gram matrix that passes through
//   LDS.  The product is taken transposed,
//   D[k2][i] = sum_k1 B[k2][k1] Z[i][k1], so that lane (i, g) ends up with D[16 c + 4 g + v][i]; the
//   contraction order over k1 is free, and it is chosen so that the same lane's operand
//   registers hold exactly Z[i][16 c + 4 g + v]: q_i is then a dot product of registers the lane
//   already has, summed over the four lanes that share a row.  quadform_cols_small_kernel (rank 64) and
//   quadform_cols_kernel (ranks >= 128, on 32 x 32 x 16 tiles) are the same scheme for rows of A generated
//   into the operand registers.
//   The kernels finish the statistics themselves (R_i, K_j, one partial sum of R per row block).
#include <type_traits>

#include "flora_gen.hip.h"
#include "flora_internal.h"

namespace flora {

namespace {

constexpr int kGT = 64;          // long-index entries per tile
constexpr int kGLd = kGT + 8;    // padded LDS row (bf16 elements): 144 bytes

// Position within a 32-block of the contraction index k1 = 32 s + x, x = 16 h + 4 g + v (h < 2, g < 4,
// v < 4): lane group g holds, for step s, the eight values x = 4 g + v and x = 16 + 4 g + v.
__device__ __forceinline__ int perm32(int x) { return 8 * ((x >> 2) & 3) + 4 * (x >> 4) + (x & 3); }
// The same for quadform_cols_kernel (32 x 32 x 16 tiles): x = 8 a + 4 g + v (a < 4, g < 2, v < 4); lane half
// g holds, for step 2 s + (a >> 1) of the contraction, the values x = 8 a + 4 g + v in elements 4 (a & 1) + v.
__device__ __forceinline__ int perm32w(int x) { return 16 * (x >> 4) + 8 * ((x >> 2) & 1) + 4 * ((x >> 3) & 1) + (x & 3); }

// Q = S^T S at rank 64: a wave makes two of the sixteen 16 x 16 tiles
__global__ __launch_bounds__(512) void gram_kernel(const MatDev* __restrict__ mats, const WorkItem* __restrict__ items)
{
    constexpr int R = 64;
    constexpr int CT = 2;                             // column tiles per wave
    __shared__ __attribute__((aligned(16))) uint16_t ldsX[2][R][kGLd];

    const WorkItem it = items[blockIdx.x];
    const MatDev& M = mats[it.mat];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const long long t0 = it.col0, t1 = it.col1;       // this chunk of the long index
    const int ntiles = (int)((t1 - t0 + kGT - 1) / kGT);
    const int row_tile = wave % 4, col_tile0 = (wave / 4) * CT;

    // ---- a 64 x R tile of S, transposed, bf16
    // unit = (pair of rows 2 p, 2 p + 1; four columns 4 k4 ..), one per thread; eight consecutive lanes take
    // eight row pairs (consecutive words of an LDS row), the lanes 8 apart the next columns (a whole 128-byte line
    // per row).  Fetched one tile ahead of being stashed, so that the loads are in flight while the
    // current tile multiplies; rows past the chunk read through a resource that ends there.
    const long long chunk_rows = t1 - t0;
    const rsrc_t srs = make_rsrc(M.state + t0 * R, chunk_rows * R * 4);
    const int k4 = (tid >> 3) % (R / 4), p = ((tid >> 3) / (R / 4)) * 8 + (tid & 7);
    auto fetch = [&](v4f (&st)[2], int tile) {
        const long long ra = (long long)tile * kGT + 2 * p;           // relative to the chunk
        const uint32_t off = (uint32_t)((ra * R + 4 * k4) * 4);
        st[0] = (ra < chunk_rows) ? buf_load_f4(srs, off) : v4f{0.f, 0.f, 0.f, 0.f};
        st[1] = (ra + 1 < chunk_rows) ? buf_load_f4(srs, off + (uint32_t)(R * 4)) : v4f{0.f, 0.f, 0.f, 0.f};
    };
    auto stash = [&](const v4f (&st)[2], int buf) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            *reinterpret_cast<uint32_t*>(&ldsX[buf][4 * k4 + e][2 * p]) = pack_bf16x2(st[0][e], st[1][e]);
    };

    f32x4 acc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};

    v4f stage[2];
    fetch(stage, 0);
    stash(stage, 0);
    if (ntiles > 1) fetch(stage, 1);
    __syncthreads();
    for (int tile = 0; tile < ntiles; ++tile) {
        const int buf = tile & 1;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const bf16x8 av = *reinterpret_cast<const bf16x8*>(&ldsX[buf][16 * row_tile + li][32 * s + 8 * g]);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8*>(&ldsX[buf][16 * (col_tile0 + ct) + li][32 * s + 8 * g]);
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[ct], 0, 0, 0);
            }
        }
        if (tile + 1 < ntiles) {
            stash(stage, buf ^ 1);                               // tile + 1, fetched a round ago
            if (tile + 2 < ntiles) fetch(stage, tile + 2);
        }
        __syncthreads();
    }

    // partial of this chunk: D layout, lane holds column 16 ct + li and rows 4 g + v of each tile; kept are the 32 x 32
    // tiles on and above the diagonal
    float* part = M.grampart + (size_t)it.part * gram_piece_floats(R);
    const int ti = row_tile / 2, tj = col_tile0 / 2;
    if (ti > tj) return;
    float* tile = part + (ti * (R / 32) - ti * (ti - 1) / 2 + tj - ti) * 1024;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) stg(tile + (16 * (row_tile & 1) + 4 * g + v) * 32 + 16 * ct + li, acc[ct][v]);
}

// P = A^T A and P' = A^T diag(1 / K) A from ONE regeneration of A, at ranks >= 128.  The vector
// ALU work of the generator is what these sums cost, so both are taken from the same tile: the
// tile goes to LDS twice, plain and with its long-index entries scaled by 1 / K, and
// P'[k1][k2] = sum_t X[t][k1] (X[t][k2] / K_t) takes one operand from each copy.
// 16 waves (12 for both sums at r = 256: 36 tiles, three a wave, in 168 registers; with eight waves of up to five 24 matrices of
// 768 x 3072 285 us instead of 279, GPT-2 base 341 and 337), so that four share a SIMD and one wave's generator chains run in the shadow of the
// others'; v_mfma_f32_32x32x16_bf16 tiles; only the tiles on or above the diagonal of the
// symmetric results are computed (36 of 64 at r = 256), consecutive ones to a wave (they mostly
// share an operand), every SIMD multiplying the same number of them, and only they are stored.
// MODE 0: P alone (no clipping asked for); 1: P and P'; 2: Q = S^T S, the tiles being rows of the
// state, fetched one tile ahead and rounded to bf16 on their way into LDS.
template <int R>
struct UpperTiles {
    static constexpr int NT = R / 32;                      // 32-wide tiles per dimension
    static constexpr int COUNT = NT * (NT + 1) / 2;
    // the idx-th tile (ti <= tj) in row-major order of the upper triangle
    __device__ static void at(int idx, int& ti, int& tj)
    {
        int c = idx, row = 0;
        while (c >= NT - row) { c -= NT - row; ++row; }
        ti = row; tj = row + c;
    }
};

template <int R, int MODE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void gram_sym_kernel(const MatDev* __restrict__ mats, const WorkItem* __restrict__ items,
                                                         const SeedArgs seeds)
{
    static_assert(R >= 128, "ranks 128 and 256");
    typedef UpperTiles<R> UT;
    constexpr int TW = (UT::COUNT + WAVES - 1) / WAVES;   // tiles per wave
    constexpr bool PAIR = MODE == 1;
    constexpr int NC = PAIR ? 2 : 1;                       // copies of a tile: plain, scaled
    __shared__ __attribute__((aligned(16))) uint16_t ldsX[2][NC][R][kGLd];                 // [buffer][copy][k][t]

    const WorkItem it = items[blockIdx.x];
    const MatDev& M = mats[it.mat];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, g = lane >> 5;
    const long long t0 = it.col0, t1 = it.col1;
    const int ntiles = (int)((t1 - t0 + kGT - 1) / kGT);

    // this wave's tiles of the results: numbers wave, wave + WAVES, ... of the upper triangle, which
    // gives every SIMD (waves w, w + 4, ...) the same number of them
    int ti[TW], tj[TW];
    bool own[TW];
#pragma unroll
    for (int w = 0; w < TW; ++w) {
        const int idx = wave + WAVES * w;
        own[w] = idx < UT::COUNT;
        ti[w] = tj[w] = 0;
        if (own[w]) UT::at(idx, ti[w], tj[w]);
        ti[w] = __builtin_amdgcn_readfirstlane(ti[w]);
        tj[w] = __builtin_amdgcn_readfirstlane(tj[w]);
    }

    const uint32_t seed_lo = seeds.s[it.mat].x, seed_hi = seeds.s[it.mat].y;
    const float cgen = neg2_ln2_over(R);
    constexpr bool kEven = R % (4 * WAVES) == 0;
    constexpr int NQ = kEven ? R / (4 * WAVES) : 2;   // quads per thread and tile (12 waves: and round)
    constexpr int JG = kGT / NQ, UNITS = JG * (R / 4);
    auto produce_unit = [&](int buf, int tile, int unit) {
        const int gen_j = NQ * (unit % JG);
        const uint32_t gen_q = (uint32_t)(unit / JG);
        const long long j = t0 + (long long)tile * kGT + gen_j;
        float wt[NQ];
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
            wt[e] = 1.f;
            if (PAIR) wt[e] = ldg(M.col_stat + ((j + e < t1) ? j + e : t1 - 1));
        }
        uint32_t pk[NC][NQ / 2][4];
#pragma unroll
        for (int e = 0; e < NQ; e += 2) {
            const Quad z0 = normal_quad(seed_lo, seed_hi, (uint32_t)(j + e), gen_q, cgen);
            const Quad z1 = normal_quad(seed_lo, seed_hi, (uint32_t)(j + e + 1), gen_q, cgen);
            const float m0 = (j + e < t1) ? 1.f : 0.f, m1 = (j + e + 1 < t1) ? 1.f : 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) pk[0][e / 2][i] = pack_bf16x2(m0 * z0.z[i], m1 * z1.z[i]);
            if (PAIR) {
                const float w0 = m0 * __builtin_amdgcn_rcpf(wt[e]), w1 = m1 * __builtin_amdgcn_rcpf(wt[e + 1]);
#pragma unroll
                for (int i = 0; i < 4; ++i) pk[NC - 1][e / 2][i] = pack_bf16x2(w0 * z0.z[i], w1 * z1.z[i]);
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint16_t* dst = &ldsX[buf][c][4 * gen_q + i][gen_j];
                if (NQ == 8) *reinterpret_cast<uint4*>(dst) = make_uint4(pk[c][0][i], pk[c][NQ / 8][i], pk[c][NQ / 4][i], pk[c][NQ / 2 - 1][i]);
                else if (NQ == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(pk[c][0][i], pk[c][NQ / 2 - 1][i]);
                else *reinterpret_cast<uint32_t*>(dst) = pk[c][0][i];
            }
    };
    auto produce = [&](int buf, int tile) {
        if constexpr (kEven) {
            produce_unit(buf, tile, tid);
        } else {
#pragma unroll 1
            for (int u = tid; u < UNITS; u += 64 * WAVES) produce_unit(buf, tile, u);
        }
    };

    // loaded X (MODE 2): unit = (pair of rows 2 p, 2 p + 1; four columns 4 k4 ..); eight consecutive
    // lanes take eight row pairs (consecutive words of an LDS row), the lanes 8 apart the next
    // columns (a whole 128-byte line per row); rows past the chunk read through a resource that
    // ends there
    constexpr int NU = (8 * R) / (64 * WAVES) > 0 ? (8 * R) / (64 * WAVES) : 1;
    const long long chunk_rows = t1 - t0;
    const rsrc_t srs = make_rsrc(M.state + (MODE == 2 ? t0 * R : 0),
                                 chunk_rows * (long long)R * 4 < 0x7fffffffLL ? chunk_rows * R * 4 : 0x7fffffffLL);
    auto fetch_loaded = [&](v4f (&st)[NU][2], int tile) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int flat = tid + 64 * WAVES * u;
            const int rest = flat >> 3;
            const int k4 = rest % (R / 4);
            const int p = (rest / (R / 4)) * 8 + (flat & 7);
            const long long ra = (long long)tile * kGT + 2 * p;       // relative to the chunk
            const uint32_t off = (uint32_t)((ra * R + 4 * k4) * 4);
            st[u][0] = (ra < chunk_rows) ? buf_load_f4(srs, off) : v4f{0.f, 0.f, 0.f, 0.f};
            st[u][1] = (ra + 1 < chunk_rows) ? buf_load_f4(srs, off + (uint32_t)(R * 4)) : v4f{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto stash_loaded = [&](const v4f (&st)[NU][2], int buf) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int flat = tid + 64 * WAVES * u;
            const int rest = flat >> 3;
            const int k4 = rest % (R / 4);
            const int p = (rest / (R / 4)) * 8 + (flat & 7);
            const v4f a = st[u][0], b = st[u][1];
            *reinterpret_cast<uint32_t*>(&ldsX[buf][0][4 * k4 + 0][2 * p]) = pack_bf16x2(a.x, b.x);
            *reinterpret_cast<uint32_t*>(&ldsX[buf][0][4 * k4 + 1][2 * p]) = pack_bf16x2(a.y, b.y);
            *reinterpret_cast<uint32_t*>(&ldsX[buf][0][4 * k4 + 2][2 * p]) = pack_bf16x2(a.z, b.z);
            *reinterpret_cast<uint32_t*>(&ldsX[buf][0][4 * k4 + 3][2 * p]) = pack_bf16x2(a.w, b.w);
        }
    };

    f32x16 acc[NC][TW];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int w = 0; w < TW; ++w)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][w][v] = 0.f;

    // the waves of a SIMD (w, w + 4, ...) take producing the next tile and multiplying the current
    // one in alternating orders
    const bool produce_first = ((wave >> 2) & 1) == 0;
    v4f stage[NU][2];
    if (MODE == 2) {
        fetch_loaded(stage, 0);
        stash_loaded(stage, 0);
        if (ntiles > 1) fetch_loaded(stage, 1);
    } else {
        produce(0, 0);
    }
    __syncthreads();
    for (int tile = 0; tile < ntiles; ++tile) {
        const int buf = tile & 1;
        if (MODE != 2 && produce_first && tile + 1 < ntiles) produce(buf ^ 1, tile + 1);
        // Straight-line code over all TW slots (a wave that owns TW - 1 tiles multiplies tile (0, 0)
        // again in its last slot and drops the result), so that the LDS reads of several
        // matrix-core instructions are in flight together.
#pragma unroll
        for (int s = 0; s < kGT / 16; ++s) {
#pragma unroll
            for (int w = 0; w < TW; ++w) {
                const bf16x8 av = *reinterpret_cast<const bf16x8*>(&ldsX[buf][0][32 * ti[w] + ln][16 * s + 8 * g]);
                const bf16x8 bv = *reinterpret_cast<const bf16x8*>(&ldsX[buf][0][32 * tj[w] + ln][16 * s + 8 * g]);
                acc[0][w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[0][w], 0, 0, 0);
                if (PAIR) {
                    const bf16x8 bs = *reinterpret_cast<const bf16x8*>(&ldsX[buf][NC - 1][32 * tj[w] + ln][16 * s + 8 * g]);
                    acc[NC - 1][w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bs, acc[NC - 1][w], 0, 0, 0);
                }
            }
        }
        if (MODE != 2 && !produce_first && tile + 1 < ntiles) produce(buf ^ 1, tile + 1);
        if (MODE == 2 && tile + 1 < ntiles) {
            stash_loaded(stage, buf ^ 1);                        // tile + 1, fetched a round ago
            if (tile + 2 < ntiles) fetch_loaded(stage, tile + 2);
        }
        __syncthreads();
    }

    // D layout of a 32 x 32 tile: lane holds column ln and rows 8 (v / 4) + 4 g + v % 4.  A partial is the tiles of
    // the upper triangle one after another, 4 KB each.
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        // (partials: those of P over chunks of m, then those of P'; or those of Q over chunks of n, combined before)
        const int part0 = c ? M.gchunks_m : 0;
        float* part = M.grampart + (size_t)(part0 + it.part) * gram_piece_floats(R);
#pragma unroll
        for (int w = 0; w < TW; ++w)
            if (own[w]) {
#pragma unroll
                for (int v = 0; v < 16; ++v) stg(part + (wave + WAVES * w) * 1024 + (8 * (v / 4) + 4 * g + (v % 4)) * 32 + ln, acc[c][w][v]);
            }
    }
}

// P (and P') of a launch with few chunks, and of every launch at rank 64, where the one block is the whole matrix (P and P' used to
// take a sweep over A each: factored update, us before / after, one 768 x 3072 matrix 55 / 45, one 1600 x 6400 65 / 57, GPT-2
// base 175 / 172, 24 of 768 x 3072 127 / 119; with blocks of 32 48, 58, 205, 133): a workgroup makes the tiles of one pair of blocks of SB ranks, regenerating those
// ranks only, where gram_sym_kernel would leave most compute units idle beside a chain of up to 48 whole tiles of A.
// (Blocks take no memory; shorter chunks would.)  16 waves in groups of SB / 16 that take every KG-th tile of
// the chunk each and whose sums are added in the groups' order.  A block pair generates SB or 2 SB ranks: with SB =
// 32 / 64 the entries of A are made 9 / 4.8 times at r = 256, 4.8 times with 32 at r = 128.  Blocks of 32 pay while every
// pair has a compute unit of its own, those of 64 at r = 256 up to two rounds of them.  Factored update, us with whole matrices / blocks of
// 64 / of 32, by chunks: r = 256 2 chunks 176 / 126 / 109, 5 173 / 132 / 120, 8 187 / 138 / 139, 16 201 / 153 / 170, 24
// 220 / 171 / 208, 36 207 / 198 / 235, 48 300 / 287 / 345, 88 362 / 393 / 469; r = 128 4 chunks 68 / 67 / 61, 16 78 / 76 / 71, 18 69 /
// 70 / 64, 32 101 / 99 / 106, 64 123 / 121 / 139, 96 150 / 163 / 175.
template <int R, int SB, bool PAIR>
__global__ __launch_bounds__(1024) void gram_block_kernel(const MatDev* __restrict__ mats, const WorkItem* __restrict__ items,
                                                          const SeedArgs seeds)
{
    typedef UpperTiles<R> UT;
    constexpr int GW = SB / 16, KG = 16 / GW, GT = 64 * GW;      // waves of a group, groups, threads of a group
    constexpr int NB = R / SB, PAIRS = NB * (NB + 1) / 2;        // consecutive workgroups of a chunk
    constexpr int SBT = SB / 32;                                 // 32-wide tiles of a block each way
    constexpr bool SPLIT = SB == 32;                             // one tile: wave 0 makes P's, wave 1 P''s
    constexpr int TW = SPLIT ? 1 : SBT * SBT / GW;               // tiles per wave
    constexpr int NC = PAIR ? 2 : 1;                             // results
    constexpr int NA = SPLIT ? 1 : NC;                           // of them in a wave
    constexpr int SCALED = SB == R ? SB : 2 * SB;                // first row of the second block's scaled copy (SB == R: of the only one's)
    constexpr int ROWS = (SB == R || !PAIR ? 2 : 3) * SB;        // first block, second block, second block scaled
    constexpr int NQ = SB == R ? 4 : 8;                          // quads per thread and tile
    static_assert(kGT / NQ * ((SB == R ? 1 : 2) * SB / 4) == GT, "a quad of ranks and NQ entries per thread");
    static_assert((KG - 1) * SB * SB * 4 * (SPLIT ? NC : 1) <= KG * ROWS * kGLd * 2, "a result's sums take the place of the tiles");
    __shared__ __attribute__((aligned(16))) uint16_t lds[KG][ROWS][kGLd];

    const WorkItem it = items[blockIdx.x / PAIRS];
    const MatDev& M = mats[it.mat];
    int bi = 0, c = (int)(blockIdx.x % PAIRS);
    while (c >= NB - bi) { c -= NB - bi; ++bi; }
    const int bj = bi + c;
    const bool diag = bi == bj;
    const int kg = __builtin_amdgcn_readfirstlane((int)threadIdx.x / GT);
    const int tid = (int)threadIdx.x % GT;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, g = lane >> 5;
    const long long t0 = it.col0, t1 = it.col1;
    const int ntiles = (int)((t1 - t0 + KG * kGT - 1) / (KG * kGT));         // of each group (zeros beyond the chunk)

    const uint32_t seed_lo = seeds.s[it.mat].x, seed_hi = seeds.s[it.mat].y;
    const float cgen = neg2_ln2_over(R);
    const int gen_j = NQ * (tid % (kGT / NQ)), q = tid / (kGT / NQ);         // LDS rows 4 q .. 4 q + 3
    const bool second = q >= SB / 4;                                         // (a pair on the diagonal needs one block)
    const bool gen = !(diag && second);
    const uint32_t gen_q = (uint32_t)(second ? bj * (SB / 4) + q - SB / 4 : bi * (SB / 4) + q);
    const bool scaled = PAIR && (second || diag);
    uint32_t pk[NC][NQ / 2][4];
    auto produce = [&](int tile) {
        const long long j = t0 + (long long)(tile * KG + kg) * kGT + gen_j;
        float wt[NQ];
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
            wt[e] = 1.f;
            if (PAIR) wt[e] = ldg(M.col_stat + ((j + e < t1) ? j + e : t1 - 1));
        }
#pragma unroll
        for (int e = 0; e < NQ; e += 2) {
            const Quad z0 = normal_quad(seed_lo, seed_hi, (uint32_t)(j + e), gen_q, cgen);
            const Quad z1 = normal_quad(seed_lo, seed_hi, (uint32_t)(j + e + 1), gen_q, cgen);
            const float m0 = (j + e < t1) ? 1.f : 0.f, m1 = (j + e + 1 < t1) ? 1.f : 0.f;
            const float w0 = m0 * __builtin_amdgcn_rcpf(wt[e]), w1 = m1 * __builtin_amdgcn_rcpf(wt[e + 1]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pk[0][e / 2][i] = pack_bf16x2(m0 * z0.z[i], m1 * z1.z[i]);
                if (PAIR) pk[NC - 1][e / 2][i] = pack_bf16x2(w0 * z0.z[i], w1 * z1.z[i]);
            }
        }
    };
    auto stash = [&]() {
        if (!gen) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            auto put = [&](int row, const uint32_t (&x)[NQ / 2][4]) {
                uint16_t* at = &lds[kg][row][gen_j];
                if constexpr (NQ == 8) *reinterpret_cast<v4u*>(at) = v4u{x[0][i], x[1][i], x[2][i], x[3][i]};
                else *reinterpret_cast<v2u*>(at) = v2u{x[0][i], x[1][i]};
            };
            put(4 * q + i, pk[0]);
            if (scaled) put(PAIR ? (diag ? SCALED : SCALED - SB) + 4 * q + i : 0, pk[NC - 1]);
        }
    };

    f32x16 acc[NA][TW];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int w = 0; w < TW; ++w)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][w][v] = 0.f;
    const int brow = diag ? 0 : SB;                // second operand, plain

    if (gen) produce(0);
    stash();
    __syncthreads();
    for (int tile = 0; tile < ntiles; ++tile) {
#pragma unroll
        for (int s = 0; s < kGT / 16; ++s)
#pragma unroll
            for (int w = 0; w < TW; ++w) {
                const int ra = SPLIT ? 0 : (wave * TW + w) / SBT, cb = SPLIT ? 0 : (wave * TW + w) % SBT;
                const int k = 16 * s + 8 * g;
                const bf16x8 av = *reinterpret_cast<const bf16x8*>(&lds[kg][32 * ra + ln][k]);
                const int b0 = SPLIT && PAIR && wave == 1 ? SCALED : brow;
                const bf16x8 bv = *reinterpret_cast<const bf16x8*>(&lds[kg][b0 + 32 * cb + ln][k]);
                acc[0][w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[0][w], 0, 0, 0);
                if (NA == 2) {
                    const bf16x8 bs = *reinterpret_cast<const bf16x8*>(&lds[kg][(PAIR ? SCALED : 0) + 32 * cb + ln][k]);
                    acc[NA - 1][w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bs, acc[NA - 1][w], 0, 0, 0);
                }
            }
        const bool more = tile + 1 < ntiles;
        if (more && gen) produce(tile + 1);
        __syncthreads();
        if (more) {
            stash();
            __syncthreads();
        }
    }

    // the groups' sums, one result after the other, then the tiles on and above the diagonal
    float* const sums = reinterpret_cast<float*>(lds);
    constexpr int kWave = TW * 1024;               // floats of a wave and result
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        if (a > 0) __syncthreads();
        if (kg > 0 && wave * kWave < (SPLIT ? NC : 1) * SB * SB) {
#pragma unroll
            for (int w = 0; w < TW; ++w)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    sums[((kg - 1) * (SPLIT ? NC : GW) + wave) * kWave + (w * 16 + v) * 64 + lane] = acc[a][w][v];
        }
        __syncthreads();
        if (kg == 0 && !(SPLIT && wave >= NC)) {
            const int which = SPLIT ? wave : a;
            float* part = M.grampart + (size_t)((which ? M.gchunks_m : 0) + it.part) * gram_piece_floats(R);
#pragma unroll
            for (int w = 0; w < TW; ++w) {
#pragma unroll
                for (int k = 1; k < KG; ++k)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[a][w][v] += sums[((k - 1) * (SPLIT ? NC : GW) + wave) * kWave + (w * 16 + v) * 64 + lane];
                const int ti = bi * SBT + (SPLIT ? 0 : (wave * TW + w) / SBT), tj = bj * SBT + (SPLIT ? 0 : (wave * TW + w) % SBT);
                if (ti > tj) continue;
                const int idx = ti * UT::NT - ti * (ti - 1) / 2 + tj - ti;
#pragma unroll
                for (int v = 0; v < 16; ++v) stg(part + idx * 1024 + (8 * (v / 4) + 4 * g + (v % 4)) * 32 + ln, acc[a][w][v]);
            }
        }
    }
}

// B <- sum over the chunks of their partials, in chunk order; stored as bf16 with the columns of
// every 32-block in the order the quadratic-form kernels contract them.  which 0: P (chunks of m), 1: Q
// (chunks of n), 2: P' (chunks of m; it is kept right behind Q); 0 and 2 together as blockIdx.z = 0, 1.
// Partials hold the tiles of the upper triangle (0.56 of the matrix at r = 256, 0.63 at r = 128, 0.75 at r = 64: less
// traffic, 384 T5-3B matrices' factored update 6139 -> 6045 us, and more pieces in the same memory, the pair kernel on
// one 1600 x 6400 matrix at r = 256 124 -> 72, on 16 GPT-2 base matrices at r = 128 23 -> 14): a tile per workgroup,
// written to both of its places.
template <int R>
__global__ __launch_bounds__(256) void combine_gram_kernel(const MatDev* __restrict__ mats, int first)
{
    __shared__ float turn[32][33];
    const MatDev& M = mats[blockIdx.y];
    const int which = first + 2 * (int)blockIdx.z;
    const int nch = which == 1 ? M.gchunks_n : M.gchunks_m;
    const int part0 = which == 2 ? M.gchunks_m : 0;
    constexpr size_t kPiece = gram_piece_floats(R);
    const int row = threadIdx.x / 8, col = 4 * (threadIdx.x % 8);
    const float* src = M.grampart + (size_t)part0 * kPiece + (size_t)blockIdx.x * 1024 + row * 32 + col;
    v4f s = {0.f, 0.f, 0.f, 0.f};
    int c = 0;
    for (; c + 8 <= nch; c += 8) {                              // eight loads in flight
        v4f p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = ldg4(src + (size_t)(c + e) * kPiece);
#pragma unroll
        for (int e = 0; e < 8; ++e) s += p[e];
    }
    for (; c < nch; ++c) s += ldg4(src + (size_t)c * kPiece);
    uint16_t* B = which == 0 ? M.gramP : (which == 1 ? M.gramQ : M.gramQ + R * R);
    int ti, tj;
    UpperTiles<R>::at(blockIdx.x, ti, tj);
    // (Q at ranks >= 128 is read by quadform_cols_kernel, all else in the other order; four consecutive entries stay together)
    auto put = [&](int k2, int k1, v4f x) {
        const int pos = (k1 & ~31) + (which == 1 && R >= 128 ? perm32w(k1 & 31) : perm32(k1 & 31));
        *reinterpret_cast<FLORA_GLOBAL v2u*>((FLORA_GLOBAL uint16_t*)(B + k2 * R + pos)) =
            v2u{pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w)};
    };
    put(32 * ti + row, 32 * tj + col, s);
    if (ti == tj) return;
    turn[row][col] = s.x;
    turn[row][col + 1] = s.y;
    turn[row][col + 2] = s.z;
    turn[row][col + 3] = s.w;
    __syncthreads();
    put(32 * tj + row, 32 * ti + col, v4f{turn[col][row], turn[col + 1][row], turn[col + 2][row], turn[col + 3][row]});
}

// q_i = Z_i B Z_i^T for 16 ZT rows of Z held in operand registers, rows [16 CT0, 16 (CT0 + NCT)) of B in LDS:
// D[16 ct + 4 g + v][i], then its dot product with Z[i][16 ct + 4 g + v], which is elements 4 (ct % 2) + v
// of step ct / 2 of this lane's own operand registers.
template <int S, int ZT, int CT0, int NCT, int LDB>
__device__ __forceinline__ void quadform_tiles(float (&q)[ZT], const bf16x8 (&zreg)[ZT][S], const uint16_t (*ldsB)[LDB], int li, int g)
{
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
        const int ct = CT0 + c;
        f32x4 acc[ZT];
#pragma unroll
        for (int z = 0; z < ZT; ++z) acc[z] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const bf16x8 bv = *reinterpret_cast<const bf16x8*>(&ldsB[16 * c + li][32 * s + 8 * g]);
#pragma unroll
            for (int z = 0; z < ZT; ++z)
                acc[z] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, zreg[z][s], acc[z], 0, 0, 0);
        }
#pragma unroll
        for (int z = 0; z < ZT; ++z) {
            const v4u zz = __builtin_bit_cast(v4u, zreg[z][ct / 2]);
            const uint32_t w0 = (ct & 1) ? zz.z : zz.x, w1 = (ct & 1) ? zz.w : zz.y;
            q[z] = __builtin_fmaf(acc[z][0], __uint_as_float(w0 << 16), q[z]);
            q[z] = __builtin_fmaf(acc[z][1], __uint_as_float(w0 & 0xffff0000u), q[z]);
            q[z] = __builtin_fmaf(acc[z][2], __uint_as_float(w1 << 16), q[z]);
            q[z] = __builtin_fmaf(acc[z][3], __uint_as_float(w1 & 0xffff0000u), q[z]);
        }
        // (keeps the compiler from hoisting every column tile's LDS reads to the top: the
        // registers are the operand tiles' and must not spill)
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The row statistics and the clipping sum from ONE read of S (a pass each
// took 0.61 ms on 384 T5-3B matrices at r = 256, together they take 0.55; on 16 GPT-2 base matrices at
// r = 128, 22 + 20 us against 11):
//   R_i <- beta2 R_i + (1 - beta2) (alpha^2 S_i P S_i^T / m + eps1), rowpart[block] <- the block's sum of the
//          new R_i (for mean(R));
//   CLIP: itempart[block] <- alpha^2 sum_i (S_i P' S_i^T) / R_i (the clipping sum of this row block, but for
//         the factor mean(R), which rms_finalize_kernel supplies).
// A workgroup's 256 rows of S stay in operand registers (32 to a wave) while P and then P' pass through LDS, at
// r = 256 by halves: 68 KB instead of 135, so that two workgroups share a compute unit and one loads while
// the other multiplies.
// 128 rows in four waves where that leaves no workgroup without a compute unit: less to do beside the passage of P and P'.
template <int R, bool CLIP, int WAVES>
__global__ __launch_bounds__(64 * WAVES, R >= 256 && WAVES == 8 ? 4 : 2) void quadform_rows_kernel(const MatDev* __restrict__ mats, const WorkItem* __restrict__ items,
                                                            float alpha, float beta2, float eps1)
{
    constexpr int S = R / 32;                      // contraction steps
    constexpr int ZT = 2;                          // 16-row tiles of S per wave
    constexpr int KB = R < 128 ? R : 128;          // rows of B in LDS at a time
    constexpr int LDB = R + 8;                     // padded LDS row (bf16 elements)
    __shared__ __attribute__((aligned(16))) uint16_t ldsB[KB][LDB];
    __shared__ float lds_fin[2][WAVES];

    const WorkItem it = items[blockIdx.x];
    const MatDev& M = mats[it.mat];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const long long row_end = ((long long)it.row0 + it.rows < M.n) ? (long long)it.row0 + it.rows : M.n;

    // this wave's rows: row0 + wave * 16 ZT + 16 z + li
    const long long wrow = (long long)it.row0 + wave * (16 * ZT);
    long long valid = row_end - wrow;
    valid = valid < 0 ? 0 : (valid > 16 * ZT ? 16 * ZT : valid);
    const rsrc_t srs = make_rsrc(M.state + (wrow < M.n ? wrow : 0) * R, valid * R * 4);      // rows past the end read as zero
    bf16x8 zreg[ZT][S];
#pragma unroll
    for (int z = 0; z < ZT; ++z)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t off = (uint32_t)((16 * z + li) * R + 32 * s + 4 * g) * 4u;
            const v4f lo = buf_load_f4(srs, off), hi = buf_load_f4(srs, off + 64u);
            const v4u pk = {pack_bf16x2(lo.x, lo.y), pack_bf16x2(lo.z, lo.w), pack_bf16x2(hi.x, hi.y), pack_bf16x2(hi.z, hi.w)};
            zreg[z][s] = __builtin_bit_cast(bf16x8, pk);
        }

    auto stage_B = [&](const uint16_t* B) {
#pragma unroll
        for (int f0 = 0; f0 < KB * (R / 8); f0 += 64 * WAVES) {
            const int f = f0 + tid;
            *reinterpret_cast<v4u*>(&ldsB[f / (R / 8)][8 * (f % (R / 8))]) = ldg4(B + (f / (R / 8)) * R + 8 * (f % (R / 8)));
        }
    };
    auto form = [&](float (&q)[ZT], const uint16_t* B) {
#pragma unroll
        for (int z = 0; z < ZT; ++z) q[z] = 0.f;
        __syncthreads();                           // the readers of what LDS held before are done
        stage_B(B);
        __syncthreads();
        quadform_tiles<S, ZT, 0, KB / 16, LDB>(q, zreg, ldsB, li, g);
        if constexpr (R > KB) {
            static_assert(R <= 2 * KB, "two halves");
            __syncthreads();
            stage_B(B + KB * R);
            __syncthreads();
            quadform_tiles<S, ZT, KB / 16, KB / 16, LDB>(q, zreg, ldsB, li, g);
        }
#pragma unroll
        for (int z = 0; z < ZT; ++z) {             // all four lanes of row li then hold q_i
            q[z] += __shfl_xor(q[z], 16);
            q[z] += __shfl_xor(q[z], 32);
        }
    };

    float q[ZT], rn[ZT], total_r = 0.f, total_u = 0.f;
    form(q, M.gramP);
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const long long row = wrow + 16 * z + li;
        rn[z] = 1.f;
        if (row < row_end) {
            rn[z] = beta2 * ldg(M.row_stat + row) + (1.f - beta2) * (alpha * alpha * q[z] / (float)M.m + eps1);
            if (g == 0) {
                stg(M.row_stat + row, rn[z]);
                total_r += rn[z];
            }
        }
    }
    if (CLIP) {
        form(q, M.gramQ + R * R);
#pragma unroll
        for (int z = 0; z < ZT; ++z)
            if (wrow + 16 * z + li < row_end && g == 0) total_u += q[z] / rn[z];
    }
    auto wave_sum = [](float t) {                  // (only the lanes g == 0 hold anything)
        t += __shfl_xor(t, 8);
        t += __shfl_xor(t, 4);
        t += __shfl_xor(t, 2);
        t += __shfl_xor(t, 1);
        return t;
    };
    total_r = wave_sum(total_r);
    if (CLIP) total_u = wave_sum(total_u);
    if (lane == 0) { lds_fin[0][wave] = total_r; lds_fin[1][wave] = total_u; }
    __syncthreads();
    if (tid == 0) {
        float fr = 0.f, fu = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { fr += lds_fin[0][w]; fu += lds_fin[1][w]; }
        M.rowpart[it.part] = fr;
        if (CLIP) M.itempart[it.part] = alpha * alpha * fu;
    }
}

// The column statistics at rank 64: K_j <- beta2 K_j + (1 - beta2) (alpha^2 A_j Q A_j^T / n + eps1), rows A_j
// regenerated straight into the operand registers.
template <int R, int ZT>
__global__ __launch_bounds__(512) void quadform_cols_small_kernel(const MatDev* __restrict__ mats, const WorkItem* __restrict__ items,
                                                                  const SeedArgs seeds, float alpha, float beta2, float eps1)
{
    constexpr int S = R / 32;            // contraction steps
    constexpr int LDB = R + 8;           // padded LDS row (bf16 elements)
    __shared__ __attribute__((aligned(16))) uint16_t ldsB[R][LDB];

    const WorkItem it = items[blockIdx.x];
    const MatDev& M = mats[it.mat];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const long long zn = M.m;
    const long long row_end = ((long long)it.row0 + it.rows < zn) ? (long long)it.row0 + it.rows : zn;
    const uint32_t seed_lo = seeds.s[it.mat].x, seed_hi = seeds.s[it.mat].y;
    const float cgen = neg2_ln2_over(R);

    for (int f = tid; f < R * (R / 8); f += 512) {
        const int k2 = f / (R / 8), c8 = f % (R / 8);
        *reinterpret_cast<v4u*>(&ldsB[k2][8 * c8]) = ldg4(M.gramQ + k2 * R + 8 * c8);
    }
    __syncthreads();

    for (long long rb = it.row0; rb < row_end; rb += 8 * 16 * ZT) {
        // this wave's rows: rb + wave * 16 ZT + 16 z + li
        bf16x8 zreg[ZT][S];
#pragma unroll
        for (int z = 0; z < ZT; ++z) {
            const long long row = rb + (wave * ZT + z) * 16 + li;
            // (all lanes generate: rows past the end take the last row's values and are not stored)
            const uint32_t jr = (uint32_t)(row < row_end ? row : zn - 1);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const Quad q0 = normal_quad(seed_lo, seed_hi, jr, (uint32_t)(8 * s + g), cgen);
                const Quad q1 = normal_quad(seed_lo, seed_hi, jr, (uint32_t)(8 * s + 4 + g), cgen);
                const v4u pk = {pack_bf16x2(q0.z[0], q0.z[1]), pack_bf16x2(q0.z[2], q0.z[3]),
                                pack_bf16x2(q1.z[0], q1.z[1]), pack_bf16x2(q1.z[2], q1.z[3])};
                zreg[z][s] = __builtin_bit_cast(bf16x8, pk);
            }
        }
        float q[ZT];
#pragma unroll
        for (int z = 0; z < ZT; ++z) q[z] = 0.f;
        quadform_tiles<S, ZT, 0, R / 16, LDB>(q, zreg, ldsB, li, g);
#pragma unroll
        for (int z = 0; z < ZT; ++z) {
            float v = q[z];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);             // all four lanes of row li now hold q_i
            const long long row = rb + (wave * ZT + z) * 16 + li;
            if (row < row_end && g == 0)
                stg(M.col_stat + row, beta2 * ldg(M.col_stat + row) + (1.f - beta2) * (alpha * alpha * v / (float)M.n + eps1));
        }
    }
}

// The column statistics at ranks >= 128: K_j <- beta2 K_j + (1 - beta2) (alpha^2 A_j Q A_j^T / n + eps1),
// rows A_j regenerated straight into matrix-core operand registers, Q in LDS.  The scheme of
// quadform_rows_kernel on v_mfma_f32_32x32x16_bf16: a wave owns 32 rows per round, D[k2][j] =
// sum_k1 Q[k2][k1] A[j][k1] comes out with lane (j, g) holding k2 = 32 c + 8 a + 4 g + v, and the
// contraction order is chosen (perm32w) so that the lane's own operand registers hold exactly
// A[j][32 c + 8 a + 4 g + v].  Twice the rows per LDS read of Q and the faster tile shape.
template <int R, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void quadform_cols_kernel(const MatDev* __restrict__ mats,
                                                                   const WorkItem* __restrict__ items, const SeedArgs seeds,
                                                                   float alpha, float beta2, float eps1)
{
    constexpr int S = R / 16;            // contraction steps
    constexpr int CT = R / 32;           // 32-row tiles of Q
    constexpr int LDB = R + 8;           // padded LDS row (bf16 elements)
    __shared__ __attribute__((aligned(16))) uint16_t ldsB[R][LDB];

    const WorkItem it = items[blockIdx.x];
    const MatDev& M = mats[it.mat];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, g = lane >> 5;
    const long long zn = M.m;
    const long long row_end = ((long long)it.row0 + it.rows < zn) ? (long long)it.row0 + it.rows : zn;
    const uint32_t seed_lo = seeds.s[it.mat].x, seed_hi = seeds.s[it.mat].y;
    const float cgen = neg2_ln2_over(R);

    for (int f = tid; f < R * (R / 8); f += 64 * WAVES) {
        const int k2 = f / (R / 8), c8 = f % (R / 8);
        *reinterpret_cast<v4u*>(&ldsB[k2][8 * c8]) = ldg4(M.gramQ + k2 * R + 8 * c8);
    }
    __syncthreads();

    for (long long rb = it.row0; rb < row_end; rb += WAVES * 32) {
        const long long row = rb + wave * 32 + ln;
        const bool ok = row < row_end;
        // (all lanes generate: rows past the end take the last row's values and are masked below)
        const long long jr = ok ? row : zn - 1;
        const float w = ok ? 1.f : 0.f;
        bf16x8 zreg[S];
        // (opaque, or the parts of every quad that depend on its number alone are kept over the loop, and spill)
        uint32_t gq = (uint32_t)g;
        asm volatile("" : "+v"(gq));
#pragma unroll
        for (int s = 0; s < S; ++s) {
            // step s = 2 beta + sl holds k1 = 32 beta + 16 sl + 4 g + (0..3) and the same + 8: quads 8 beta + 4 sl + g and + 2
            const uint32_t q0 = (uint32_t)(8 * (s >> 1) + 4 * (s & 1)) + gq;
            const Quad a = normal_quad(seed_lo, seed_hi, (uint32_t)jr, q0, cgen);
            const Quad b = normal_quad(seed_lo, seed_hi, (uint32_t)jr, q0 + 2u, cgen);
            const v4u pk = {pack_bf16x2(w * a.z[0], w * a.z[1]), pack_bf16x2(w * a.z[2], w * a.z[3]),
                            pack_bf16x2(w * b.z[0], w * b.z[1]), pack_bf16x2(w * b.z[2], w * b.z[3])};
            zreg[s] = __builtin_bit_cast(bf16x8, pk);
        }
        float q = 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            f32x16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8*>(&ldsB[32 * c + ln][16 * s + 8 * g]);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv, zreg[s], acc, 0, 0, 0);
            }
            // acc[4 a + v] = D[32 c + 8 a + 4 g + v][j]; A[j][that k2] is element 4 (a & 1) + v of step 2 c + (a >> 1)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const v4u zz = __builtin_bit_cast(v4u, zreg[2 * c + (a >> 1)]);
                const uint32_t w0 = (a & 1) ? zz.z : zz.x, w1 = (a & 1) ? zz.w : zz.y;
                q = __builtin_fmaf(acc[4 * a + 0], __uint_as_float(w0 << 16), q);
                q = __builtin_fmaf(acc[4 * a + 1], __uint_as_float(w0 & 0xffff0000u), q);
                q = __builtin_fmaf(acc[4 * a + 2], __uint_as_float(w1 << 16), q);
                q = __builtin_fmaf(acc[4 * a + 3], __uint_as_float(w1 & 0xffff0000u), q);
            }
            // (keeps the compiler from hoisting every tile's LDS reads to the top)
            __builtin_amdgcn_sched_barrier(0);
        }
        q += __shfl_xor(q, 32);                 // both lanes of row j now hold A_j Q A_j^T
        if (ok && g == 0)
            stg(M.col_stat + row, beta2 * ldg(M.col_stat + row) + (1.f - beta2) * (alpha * alpha * q / (float)M.n + eps1));
    }
}

template <int R>
hipError_t launch_gram_r(const MatDev* mats, const WorkItem* items, int nitems, int count, const SeedArgs& seeds, int src,
                         hipStream_t s)
{
    const dim3 grid((unsigned)nitems);
    bool p = false, q = false, p2 = false;               // which sums this launch produces
#define FLORA_GRAM_BLOCKS(SB)                                                                                                     \
    do {                                                                                                                          \
        const dim3 bgrid((unsigned)(nitems * (R / SB) * (R / SB + 1) / 2));                                                       \
        if (src == 0) hipLaunchKernelGGL((gram_block_kernel<R, SB, false>), bgrid, dim3(1024), 0, s, mats, items, seeds);         \
        else hipLaunchKernelGGL((gram_block_kernel<R, SB, true>), bgrid, dim3(1024), 0, s, mats, items, seeds);                   \
    } while (0)
    if constexpr (R >= 128) {
        constexpr int PW = R >= 256 ? 12 : 16;          // waves that can hold both sets of accumulators
        if (src == 0 || src == 3) {
            p = true;
            p2 = src == 3;
            if (nitems <= (R == 256 ? 7 : 25)) FLORA_GRAM_BLOCKS(32);
            else if (R == 256 && nitems <= 48) FLORA_GRAM_BLOCKS((R == 256 ? 64 : 32));
            else if (src == 0) hipLaunchKernelGGL((gram_sym_kernel<R, 0, 16>), grid, dim3(1024), 0, s, mats, items, seeds);
            else hipLaunchKernelGGL((gram_sym_kernel<R, 1, PW>), grid, dim3(64 * PW), 0, s, mats, items, seeds);
        }
        if (src == 2) { hipLaunchKernelGGL((gram_sym_kernel<R, 2, 16>), grid, dim3(1024), 0, s, mats, items, seeds); q = true; }
    } else {
        if (src == 0 || src == 3) {
            p = true;
            p2 = src == 3;
            FLORA_GRAM_BLOCKS(64);
        }
        if (src == 2) { hipLaunchKernelGGL(gram_kernel, grid, dim3(512), 0, s, mats, items); q = true; }
    }
#undef FLORA_GRAM_BLOCKS
    if (!p && !q && !p2) return hipErrorInvalidValue;
    hipLaunchKernelGGL((combine_gram_kernel<R>), dim3((unsigned)UpperTiles<R>::COUNT, (unsigned)count, p2 ? 2 : 1), dim3(256), 0, s, mats,
                       q ? 1 : 0);
    return hipGetLastError();
}

template <int R>
hipError_t launch_quadform_r(const MatDev* mats, const WorkItem* items, int nitems, int rows, const SeedArgs& seeds, int out,
                             float alpha, float beta2, float eps1, hipStream_t s)
{
    const dim3 grid((unsigned)nitems);
    const bool few = R >= 128 && rows <= 128;            // (rank 64 always takes 256 rows)
    switch (out) {
#define FLORA_ROWS(CLIP, W) hipLaunchKernelGGL((quadform_rows_kernel<R, CLIP, W>), grid, dim3(64 * W), 0, s, mats, items, alpha, beta2, eps1)
#define FLORA_COLS(W) hipLaunchKernelGGL((quadform_cols_kernel<R, W>), grid, dim3(64 * W), 0, s, mats, items, seeds, alpha, beta2, eps1)
    case 0:
    case 2:
        if constexpr (R >= 128) {
            if (few && out == 0) FLORA_ROWS(false, 4);
            if (few && out == 2) FLORA_ROWS(true, 4);
        }
        if (!few && out == 0) FLORA_ROWS(false, 8);
        if (!few && out == 2) FLORA_ROWS(true, 8);
        break;
    case 1:
        if constexpr (R >= 128) {
            if (rows <= 128) FLORA_COLS(4);
            else if (rows <= 256) FLORA_COLS(8);
            else FLORA_COLS(16);
        } else
            hipLaunchKernelGGL((quadform_cols_small_kernel<R, 2>), grid, dim3(512), 0, s, mats, items, seeds, alpha, beta2, eps1);
        break;
#undef FLORA_ROWS
#undef FLORA_COLS
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// src 0: P = A^T A; 3: P and P' = A^T diag(1 / K) A from one regeneration of A (over chunks of m);
// 2: Q = S^T S (chunks of n).  Partial sums per work item, then the chunks are added in order and
// stored as bf16.
hipError_t launch_gram(const MatDev* mats, const WorkItem* items, int nitems, int count, const SeedArgs& seeds, int r,
                       int src, hipStream_t s)
{
    if (nitems == 0 || count == 0) return hipSuccess;
    switch (r) {
    case 64: return launch_gram_r<64>(mats, items, nitems, count, seeds, src, s);
    case 128: return launch_gram_r<128>(mats, items, nitems, count, seeds, src, s);
    case 256: return launch_gram_r<256>(mats, items, nitems, count, seeds, src, s);
    default: return hipErrorInvalidValue;
    }
}

// out 0: row sums of Gt^2 (Z = S, B = P) into the row statistics, 2: the same and the clipping sum (B = P'),
// 1: column sums (Z = A, B = Q) into the column statistics; rows: of Z per workgroup, at most
hipError_t launch_quadform(const MatDev* mats, const WorkItem* items, int nitems, int rows, const SeedArgs& seeds, int r, int out,
                           float alpha, float beta2, float eps1, hipStream_t s)
{
    if (nitems == 0) return hipSuccess;
    switch (r) {
    case 64: return launch_quadform_r<64>(mats, items, nitems, rows, seeds, out, alpha, beta2, eps1, s);
    case 128: return launch_quadform_r<128>(mats, items, nitems, rows, seeds, out, alpha, beta2, eps1, s);
    case 256: return launch_quadform_r<256>(mats, items, nitems, rows, seeds, out, alpha, beta2, eps1, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace flora
