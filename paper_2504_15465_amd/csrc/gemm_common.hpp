// Shared device helpers of the atom-aware bf16 GEMM kernels for gfx950:
// argument block, epilogue (bias, GELU, residual, bf16 rounding; element-wise or
// through LDS), LDS tile layout, logical-block -> tile order.
#pragma once
#include "common.hpp"
#include <math.h>

namespace lithos {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
typedef short s16x4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
    const uint16_t* A;
    const uint16_t* B;
    void* C;
    const float* bias;
    const float* resid;
    int M, N, K;
    int64_t lda, ldb, ldc, ldr;
    uint32_t flags;
    uint32_t tiles_m, tiles_n;
    int64_t a_plane;     // SPLIT_A: elements between the hi and the lo plane of A
    int64_t c_plane;     // OUT_SPLIT: elements between the hi and the lo plane of C
    int k_slices;        // > 1: logical block z computes k-tiles [z*KT/S, (z+1)*KT/S) into fp32 plane z of C
    int64_t c_slice;     // elements between the planes of consecutive K slices
    const float* gamma;  // NORM_LN / NORM_RMS: per-k scale of the normalised rows of A
    const float* colsum; // NORM_LN: [2, ldcs] = the rows gamma and beta multiplied with op(B)
    int64_t ldcs;
    float eps;
    int wide;            // whole 16-byte pieces of C can be stored (see staged_epilogue)
};

// K slices (the logical grid's z axis): slice z of S owns the k-tiles [z*KT/S, (z+1)*KT/S),
// a balanced cut that depends on nothing but z, so a slice's sum is the same in every launch.
__device__ __forceinline__ void slice_ktiles(const GemmArgs& g, uint32_t z, int KT, int& kt0, int& kt1)
{
    if (g.k_slices <= 1) { kt0 = 0; kt1 = KT; return; }
    kt0 = (int)(((int64_t)z * KT) / g.k_slices);
    kt1 = (int)(((int64_t)(z + 1) * KT) / g.k_slices);
}

// Compile-time loop: the body sees its index as a constant, so register
// arrays indexed with it never become memory.
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ void epilogue_store(const GemmArgs& g, int m, int n, float v)
{
    if (m >= g.M || n >= g.N) return;
    if (g.flags & LITHOS_F_BIAS) v += g.bias[n];
    if (g.flags & LITHOS_F_GELU) v = gelu_erf(v);
    if (g.flags & LITHOS_F_RESIDUAL) v += g.resid[(int64_t)m * g.ldr + n];
    if (g.flags & LITHOS_F_OUT_F32) {
        reinterpret_cast<float*>(g.C)[(int64_t)m * g.ldc + n] = v;
    } else {
        uint16_t hi = f32_to_bf16(v);
        reinterpret_cast<uint16_t*>(g.C)[(int64_t)m * g.ldc + n] = hi;
        if (g.flags & LITHOS_F_OUT_SPLIT)       // second bf16 carries what the first one dropped
            reinterpret_cast<uint16_t*>(g.C)[g.c_plane + (int64_t)m * g.ldc + n] =
                f32_to_bf16(v - __uint_as_float((uint32_t)hi << 16));
    }
}

// One finished value of C.
__device__ __forceinline__ void store_value(const GemmArgs& g, int64_t i, float v)
{
    if (g.flags & LITHOS_F_OUT_F32) {
        reinterpret_cast<float*>(g.C)[i] = v;
    } else {
        uint16_t hi = f32_to_bf16(v);
        reinterpret_cast<uint16_t*>(g.C)[i] = hi;
        if (g.flags & LITHOS_F_OUT_SPLIT)       // second bf16 carries what the first one dropped
            reinterpret_cast<uint16_t*>(g.C)[g.c_plane + i] = f32_to_bf16(v - bf16_to_f32(hi));
    }
}

// An accumulator block whose elements leave one by one: element e of the lane is (m, n) moved by 8*(e/4) + e%4 rows, or
// columns with exchanged operands.  The bits of epilogue_store, but all loads of bias and residual come before the first
// store (the compiler may not move a load of the residual above a store of C, and a round trip for each element is what a
// ragged tile's time consisted of), and a block inside the matrix is stored without a test per element.  Elements beyond
// the matrix compute on its last row and column and are not stored.
template <bool SWAPPED>
__device__ __forceinline__ void epilogue_store_block(const GemmArgs& g, int m, int n, f32x16 v, bool inside)
{
    const auto row = [&](int e) { return SWAPPED ? m : m + 8 * (e >> 2) + (e & 3); };
    const auto col = [&](int e) { return SWAPPED ? n + 8 * (e >> 2) + (e & 3) : n; };
    const bool with_bias = g.flags & LITHOS_F_BIAS, with_resid = g.flags & LITHOS_F_RESIDUAL;      // uniform
    float bv[16], rv[16];
    if (with_bias) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; bv[e] = g.bias[min(col(e), g.N - 1)]; });
    if (with_resid)
        static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; rv[e] = g.resid[min(row(e), g.M - 1) * g.ldr + min(col(e), g.N - 1)]; });
    if (with_bias) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; v[e] += bv[e]; });
    if (g.flags & LITHOS_F_GELU) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; v[e] = gelu_erf(v[e]); });
    if (with_resid) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; v[e] += rv[e]; });
    const int64_t first = m * g.ldc + n, step = SWAPPED ? 1 : g.ldc;
    if (inside) {
        static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; store_value(g, first + (8 * (e >> 2) + (e & 3)) * step, v[e]); });
    } else {
        static_for<16>([&](auto ee) {
            constexpr int e = decltype(ee)::value;
            if (row(e) < g.M && col(e) < g.N) store_value(g, first + (8 * (e >> 2) + (e & 3)) * step, v[e]);
        });
    }
}

// ---- epilogue of a full bf16 tile through LDS ---------------------------------
// Storing accumulators one element at a time costs a 2-byte global store per
// element (1024 wavefront-wide stores for a 256x256 tile, ~25 us: as long as 14
// k-tiles of the main loop).  Kernels built with ST = true therefore feed the
// MFMA with the operands exchanged, so that a lane holds four CONSECUTIVE
// columns of one output row per accumulator quad, write those 8 bytes into the
// (now idle) operand buffers as a row-major bf16 tile, and then store whole
// 512-byte rows with 16 bytes per lane.  Row r keeps its 16-byte piece p at
// piece p ^ (r mod pieces-per-row): the 32 lanes that write one piece of 32
// different rows then fall into different banks, and a row read back is a
// permutation of its pieces.  The values (and their rounding) are those of
// epilogue_store, so which path a tile takes never changes a bit of C.
template <int BN>
__device__ __forceinline__ int stage_index(int r, int p)
{
    constexpr int PPR = BN / 8;
    return r * BN + ((p ^ (r & (PPR - 1))) << 3);
}

// accumulator block with exchanged operands: lane holds output row (lane & 31) of the
// block and columns 8*q + 4*(lane >> 5) + t, q = 0..3, t = 0..3

// four consecutive floats, 4-byte aligned (one 16-byte load; bias and residual need no alignment)
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

// bias, GELU and residual applied in place (a no-op without those flags); a lane's columns 8*q + 4*(lane >> 5) .. +3
// are one 16-byte load of each operand.  Rows and column quads beyond the matrix (N % 4 == 0 then) compute on
// its last ones and are not stored.
__device__ __forceinline__ void epilogue_block_swapped(const GemmArgs& g, int m, int n_glob, f32x16& acc, int lane)
{
    if (!(g.flags & (LITHOS_F_BIAS | LITHOS_F_GELU | LITHOS_F_RESIDUAL))) return;   // uniform
    const float* const rrow = g.resid + (int64_t)min(m, g.M - 1) * g.ldr;
    f32x4_u bv[4], rv[4];
    const auto col = [&](int q) { return min(n_glob + 8 * q + 4 * (lane >> 5), g.N - 4); };
    if (g.flags & LITHOS_F_BIAS) {
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[q] = *reinterpret_cast<const f32x4_u*>(g.bias + col(q));
    }
    if (g.flags & LITHOS_F_RESIDUAL) {
#pragma unroll
        for (int q = 0; q < 4; ++q) rv[q] = *reinterpret_cast<const f32x4_u*>(rrow + col(q));
    }
    if (g.flags & LITHOS_F_BIAS) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; acc[e] += bv[e >> 2][e & 3]; });
    if (g.flags & LITHOS_F_GELU) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; acc[e] = gelu_erf(acc[e]); });
    if (g.flags & LITHOS_F_RESIDUAL) static_for<16>([&](auto ee) { constexpr int e = decltype(ee)::value; acc[e] += rv[e >> 2][e & 3]; });
}

// the block's values rounded to bf16 into the staged tile; LO: what the first rounding dropped,
// bf16(v - bf16(v)), the second plane of a split-bf16 output
template <int BN, bool LO>
__device__ __forceinline__ void stage_block_values(uint16_t* st, int r, int n_tile, const f32x16& acc, int lane)
{
    static_for<4>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        const int nl = n_tile + 8 * q + 4 * (lane >> 5);
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            v[t] = acc[4 * q + t];
            if constexpr (LO) v[t] -= bf16_to_f32(f32_to_bf16(v[t]));
        }
        *reinterpret_cast<uint2*>(st + stage_index<BN>(r, nl >> 3) + (nl & 4)) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    });
}

template <int BN>
__device__ __forceinline__ void stage_block(const GemmArgs& g, uint16_t* st, int r, int m, int n_tile, int n_glob,
                                            const f32x16& acc, int lane)
{
    f32x16 v = acc;
    epilogue_block_swapped(g, m, n_glob, v, lane);
    stage_block_values<BN, false>(st, r, n_tile, v, lane);
}

// the same block of an fp32 tile: 16 bytes (four columns) per lane and store, what lies beyond the matrix left out
__device__ __forceinline__ void store_block_swapped_f32(const GemmArgs& g, float* C, int m, int n_glob, const f32x16& acc, int lane)
{
    f32x16 v = acc;
    epilogue_block_swapped(g, m, n_glob, v, lane);
    static_for<4>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        const int n = n_glob + 8 * q + 4 * (lane >> 5);
        if (m < g.M && n < g.N)
            *reinterpret_cast<float4*>(C + (int64_t)m * g.ldc + n) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    });
}

// the same block stored element by element (edge tiles)
__device__ __forceinline__ void store_block_swapped(const GemmArgs& g, int m, int n_glob, const f32x16& acc, int lane)
{
    static_for<16>([&](auto ee) {
        constexpr int e = decltype(ee)::value;
        epilogue_store(g, m, n_glob + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3), acc[e]);
    });
}

// LDS tiles are [rows][64] bf16 (128-byte rows of eight 16-byte chunks).
// Chunk kc of row r lives in slot kc ^ swz(r); both the row-wise MFMA operand
// reads (32 consecutive rows, one chunk) and the transposing stores (rows 8
// apart, one chunk) then touch distinct banks within every 8-lane group.
__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }
__device__ __forceinline__ int lds_index(int row, int kc) { return row * 64 + ((kc ^ swz(row)) << 3); }

// Tile order inside the logical grid: groups of GM tile-rows are walked
// column-major, so 32 neighbouring logical blocks form a GM x (32/GM) patch
// that shares A and B panels in one die's L2.
__device__ __forceinline__ void tile_of_block(uint32_t lin, uint32_t tiles_m, uint32_t tiles_n,
                                              uint32_t& tm, uint32_t& tn)
{
    constexpr uint32_t GM = 4;
    uint32_t per_group = GM * tiles_n;
    uint32_t grp = lin / per_group, rem = lin % per_group;
    uint32_t first = grp * GM;
    uint32_t gm = min(tiles_m - first, GM);
    tm = first + rem % gm;
    tn = rem / gm;
}

typedef void (*gemm_fn)(GemmArgs, AtomArgs);

// kernel tables, one translation unit per family
gemm_fn gemm_tile64_fn(bool ta, bool tb, bool split, bool st, bool two_groups);
gemm_fn gemm_tile128_fn(bool ta, bool tb, bool split, bool st);
gemm_fn gemm_mid128_fn(bool ta, bool tb, bool split);
gemm_fn gemm_mid128_pair_fn(bool ta, bool tb);
gemm_fn gemm_mid192_fn(bool tb);
gemm_fn gemm_thin_fn(bool tb);
gemm_fn gemm_tile256_wide_fn(bool ta, bool tb);
gemm_fn gemm_tile256_elem_fn(bool ta, bool tb);
gemm_fn gemm_lds256_fn(bool tb);
gemm_fn gemm_lds256_ta_fn(bool tb);
gemm_fn gemm_lds256w8_wide_fn(bool ta, bool tb);
gemm_fn gemm_lds256w8_elem_fn(bool ta, bool tb);
gemm_fn gemm_skinny_fn(int variant, bool a32, int norm);

constexpr int SKINNY_WAVES = 8;     // wavefronts per workgroup of the skinny kernels, each owning one slice of K
constexpr int SKINNY_NB = 2;        // 16-column blocks per workgroup of the skinny kernels

enum { V_SKINNY32 = 3, V_TILE64 = 10, V_TILE64_2K = 11, V_TILE128 = 20, V_MID128 = 21, V_MID128_PAIR = 22, V_MID192 = 23, V_THIN = 24, V_TILE256 = 30, V_LDS256 = 31, V_LDS256W8 = 32,
       V_SKL4 = 40, V_SKL8 = 41, V_SKL16 = 42 };   // 2K: two groups of wavefronts split K; SKL: LDS-staged activations of at most 4 / 8 / 16 rows

} // namespace lithos
