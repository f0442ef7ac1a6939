// What happens to a 32 x 32 tile of the decompressed gradient
// Gt = alpha * state A^T while it is still in the accumulator registers of a
// 32x32 MFMA (lane holds column lane % 32; register v holds row
// 8 * (v / 4) + 4 * (lane / 32) + v % 4).  Shared by the fp32 and bf16
// decompression kernels; Gt is never written to memory except by kModeOut.
#pragma once
#include "flora_internal.h"

namespace flora {

__device__ __forceinline__ float half_wave_sum(float v)
{
    // sum over the 32 lanes that share lane / 32
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 8);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 1);
    return v;
}

// Per-lane state that lives across the row loop of one workgroup.
struct EpilogueLane {
    float colsum;   // kModeStats: sum of Gt^2 down this lane's column; otherwise this lane's running total
                    // (kModeRms / kModeFull1: of U^2; kModeFactored / kModeFull2: of the new W^2)
    float kfac;     // per-column factor of kModeFactored / kModeRms; step factor of kModeFull2
};

template <int MODE>
__device__ __forceinline__ EpilogueLane epilogue_begin(const MatDev& M, const DecompressParams& p,
                                                       long long j, bool jok)
{
    EpilogueLane e;
    e.colsum = 0.f;
    e.kfac = 0.f;
    if (MODE == kModeFactored) {
        // U = Gt / sqrt(R_i K_j / mean R), scaled by lr and the RMS clip factor
        // (scal[2]: the parameter scale max(eps2, RMS(W)), or 1)
        const float meanR = ldg(M.scal), clip = ldg(M.scal + 1), ps = ldg(M.scal + 2);
        e.kfac = jok ? p.coef * p.alpha * clip * ps * sqrtf(meanR) * rsqrtf(ldg(M.col_stat + j)) : 0.f;
    }
    if (MODE == kModeFull2) {
        // U = Gt / sqrt(V_ij), scaled the same way
        const float clip = ldg(M.scal + 1), ps = ldg(M.scal + 2);
        e.kfac = jok ? p.coef * p.alpha * clip * ps : 0.f;
    }
    if (MODE == kModeRms) {
        const float meanR = ldg(M.scal);
        e.kfac = jok ? p.alpha * p.alpha * meanR / ldg(M.col_stat + j) : 0.f;
    }
    return e;
}

// Row of register v of this lane, relative to the tile's first row.
__device__ __forceinline__ int tile_row(int v, int g) { return 8 * (v / 4) + 4 * g + (v % 4); }

// Which of its tile's arrays a pass moves.
template <int MODE>
struct Moves {
    static constexpr bool w = MODE == kModeSgd || MODE == kModeFactored || MODE == kModeFull2;
    static constexpr bool v = MODE == kModeFull1 || MODE == kModeFull2;
    static constexpr bool rs = MODE == kModeRms || MODE == kModeFactored;
};

// Values of a tile that the epilogue reads from memory (old weights as their bits, row statistics, second moment),
// fetched one tile ahead so that their latency overlaps the previous tile's work.
template <int MODE>
struct TilePre {
    uint32_t w[Moves<MODE>::w ? 16 : 1];
    float rs[Moves<MODE>::rs ? 16 : 1];
    float v[Moves<MODE>::v ? 16 : 1];
};

// Addresses.  A buffer resource covers a tile's valid rows of an array (32 rows of at most 2^24 columns of 4
// bytes), so loads past them return zero and stores past them are dropped; a lane whose column is past m
// points at kOob, which stays out of range whatever row is added.  No access sits behind a branch: the
// compiler can then count what is in flight and waits for the tile's own loads.  With a branch round each store
// every tile waited for the stores of the one before.  us with branches / without: GPT-2 base at r = 16, SGD 137 / 127,
// unfactored 348 / 314; at r = 32, factored 425 / 359; T5-small at r = 32, bf16 weights, SGD 76 / 56, unfactored step 253 /
// 218; 12 matrices of 1100 x 1003 and 257 x 2051 at r = 256, bf16 weights 31 / 22.
template <typename T>
__device__ __forceinline__ rsrc_t tile_rsrc(const T* base, long long m, long long rb, long long row_end)
{
    long long rows = row_end - rb;
    rows = rows < 0 ? 0 : (rows > 32 ? 32 : rows);
    return make_rsrc(base + (rows > 0 ? rb : 0) * m, rows * m * (long long)sizeof(T));
}
template <typename T>
__device__ __forceinline__ uint32_t tile_lane(uint32_t m, uint32_t j, bool jok)
{
    return jok ? (4u * ((threadIdx.x & 63) >> 5) * m + j) * (uint32_t)sizeof(T) : kOob;
}
// ... and what register v adds to it (uniform)
template <typename T>
__device__ __forceinline__ uint32_t tile_step(uint32_t m, int v) { return (uint32_t)(8 * (v / 4) + v % 4) * m * (uint32_t)sizeof(T); }

// WP: cache policy of the n x m arrays (DecompressParams::wpolicy).  rb may lie past the last tile: nothing is fetched.
template <int MODE, typename OT, int WP>
__device__ __forceinline__ void epilogue_fetch(TilePre<MODE>& pre, const MatDev& M, long long rb, long long row_end, long long j, bool jok)
{
    const uint32_t m32 = (uint32_t)M.m;
    if constexpr (Moves<MODE>::w) {
        const rsrc_t r = tile_rsrc(reinterpret_cast<const OT*>(M.weight), M.m, rb, row_end);
        const uint32_t at = tile_lane<OT>(m32, (uint32_t)j, jok);
#pragma unroll
        for (int v = 0; v < 16; ++v) pre.w[v] = buf_load_bits<OT, (WP & 1) != 0>(r, at + tile_step<OT>(m32, v));
    }
    if constexpr (Moves<MODE>::v) {
        const rsrc_t r = tile_rsrc(M.vfull, M.m, rb, row_end);
        const uint32_t at = tile_lane<float>(m32, (uint32_t)j, jok);
#pragma unroll
        for (int v = 0; v < 16; ++v) pre.v[v] = __uint_as_float(buf_load_bits<float, (WP & 1) != 0>(r, at + tile_step<float>(m32, v)));
    }
    if constexpr (Moves<MODE>::rs) {
        const rsrc_t r = tile_rsrc(M.row_stat, 1, rb, row_end);
#pragma unroll
        for (int v = 0; v < 16; ++v) pre.rs[v] = buf_load_f(r, tile_lane<float>(1u, 0u, true) + tile_step<float>(1u, v));
    }
}

// lds_red: float[4][32] scratch of the workgroup (kModeStats / kModeRms only).
template <int MODE, typename OT, int WP>
__device__ __forceinline__ void epilogue_tile(const f32x16& acc, const TilePre<MODE>& pre, const MatDev& M,
                                              const WorkItem& it, const DecompressParams& p, long long rb,
                                              long long row_end, long long j, bool jok,
                                              EpilogueLane& e, float (*lds_red)[32])
{
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int ln = lane & 31, g = lane >> 5;
    const long long n = M.n;
    const int rows_here = (int)((row_end - rb < 32) ? row_end - rb : 32);
    const uint32_t m32 = (uint32_t)M.m, j32 = (uint32_t)j;
    constexpr bool kStream = (WP & 2) != 0;
    // Sums over rows leave out those past the end (their operands read as zero, which divides); columns past m are left
    // out by epilogue_end, a lane being one column.  Only a matrix's last tile has such rows.
    auto over_rows = [&](auto&& term) {
        if (rows_here == 32) {
#pragma unroll
            for (int v = 0; v < 16; ++v) e.colsum = term(v, e.colsum);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float s = term(v, e.colsum);
                e.colsum = tile_row(v, g) < rows_here ? s : e.colsum;
            }
        }
    };
    if constexpr (MODE == kModeOut) {
        const rsrc_t r = tile_rsrc(reinterpret_cast<OT*>(M.out), M.m, rb, row_end);
        const uint32_t at = tile_lane<OT>(m32, j32, jok);
#pragma unroll
        for (int v = 0; v < 16; ++v) buf_store_bits<OT, (WP & 2) != 0>(r, at + tile_step<OT>(m32, v), to_bits<OT>(p.alpha * acc[v]));
    } else if constexpr (Moves<MODE>::w) {
        const rsrc_t r = tile_rsrc(reinterpret_cast<OT*>(M.weight), M.m, rb, row_end);
        const uint32_t at = tile_lane<OT>(m32, j32, jok);
        float wn[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float w = from_bits<OT>(pre.w[v]);
            float x;
            if constexpr (MODE == kModeSgd) x = w - p.coef * acc[v];
            else if constexpr (MODE == kModeFactored) x = w - e.kfac * rsqrtf(pre.rs[v]) * acc[v];
            else x = w - e.kfac * rsqrtf(pre.v[v]) * acc[v];
            const uint32_t b = to_bits<OT>(x);
            buf_store_bits<OT, kStream>(r, at + tile_step<OT>(m32, v), b);
            wn[v] = from_bits<OT>(b);
        }
        // sum of the new W^2, of the values as stored
        if constexpr (MODE != kModeSgd) over_rows([&](int v, float s) { return __builtin_fmaf(wn[v], wn[v], s); });
    } else if constexpr (MODE == kModeStats) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float gt = p.alpha * acc[v];
            const float q = (jok && tile_row(v, g) < rows_here) ? gt * gt : 0.f;
            e.colsum += q;
            const float s = half_wave_sum(q);      // row sums over this wave's 32 columns ...
            if (ln == 0) lds_red[wave][tile_row(v, g)] = s;
        }
        __syncthreads();                           // ... then over the 4 waves in a fixed order
        if (tid < 32) {
            const long long row = rb + tid;
            if (row < row_end) {
                const float s = ((lds_red[0][tid] + lds_red[1][tid]) + lds_red[2][tid]) + lds_red[3][tid];
                stg(M.rowpart + (long long)it.slice * n + row, s);
            }
        }
        __syncthreads();
    } else if constexpr (MODE == kModeRms) {
        over_rows([&](int v, float s) { return s + acc[v] * acc[v] * e.kfac / pre.rs[v]; });
    } else if constexpr (MODE == kModeFull1) {
        const rsrc_t r = tile_rsrc(M.vfull, M.m, rb, row_end);
        const uint32_t at = tile_lane<float>(m32, j32, jok);
        float u[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float gt = p.alpha * acc[v];
            const float vn = p.beta2 * pre.v[v] + (1.f - p.beta2) * (gt * gt + p.eps1);
            buf_store_bits<float, kStream>(r, at + tile_step<float>(m32, v), __float_as_uint(vn));
            u[v] = gt * gt / vn;
        }
        over_rows([&](int v, float s) { return s + u[v]; });
    }
}

template <int MODE>
__device__ __forceinline__ void epilogue_end(const MatDev& M, const WorkItem& it, long long j,
                                             bool jok, EpilogueLane& e, float (*lds_red)[32])
{
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 5;
    if (MODE == kModeStats) {
        e.colsum += __shfl_xor(e.colsum, 32);
        if (g == 0 && jok) stg(M.colpart + (long long)it.rblock * M.m + j, e.colsum);
    }
    if (MODE == kModeRms || MODE == kModeFactored || MODE == kModeFull1 || MODE == kModeFull2) {
        float s = half_wave_sum(jok ? e.colsum : 0.f);
        s += __shfl_xor(s, 32);
        if (lane == 0) lds_red[wave][0] = s;
        __syncthreads();
        if (tid == 0)
            M.itempart[it.part] =
                ((lds_red[0][0] + lds_red[1][0]) + lds_red[2][0]) + lds_red[3][0];
    }
}

}  // namespace flora
