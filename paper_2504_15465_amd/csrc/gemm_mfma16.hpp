// What the GEMM kernels on v_mfma_f32_16x16x32_bf16 share: accumulators and the epilogue.  The MFMA operands are
// exchanged, so a lane holds row lane % 16 of a 16x16 block of C and its columns 4 (lane / 16) .. +3.
#pragma once
#include "gemm_common.hpp"

namespace lithos {

typedef float f32x4a __attribute__((ext_vector_type(4)));

// four floats of a row from column n on, or the last four
__device__ __forceinline__ f32x4a load_quad(const float* row, int n, int N) { return *reinterpret_cast<const f32x4_u*>(row + min(n, N - 4)); }

// A block of accumulators that lives in an AGPR, in vector registers from here on (copies of all blocks ahead of the
// epilogue's first branch would go to memory).
__device__ __forceinline__ f32x4a agpr_read(f32x4a& c)
{
    asm volatile("" : "+a"(c));
    return c;
}
// The value of accumulator block (i, j); AGPR: where the accumulators live.
template <bool AGPR, int MI, int NI>
__device__ __forceinline__ f32x4a acc_block(f32x4a (&acc)[MI][NI], int i, int j)
{
    if constexpr (AGPR) return agpr_read(acc[i][j]);
    else return acc[i][j];
}

// Bias, GELU and residual of a wavefront's blocks in registers, before anything is stored (a wait for a load would wait for
// the stores before it too).  The bias is loaded once, the residual a strip of 16 rows ahead.  Rows and columns beyond the
// matrix compute on its last ones and are not stored.
template <int MI, int NI>
__device__ __forceinline__ void epilogue_apply16(const GemmArgs& g, f32x4a (&acc)[MI][NI], int mw, int nw, int lane)
{
    const bool with_bias = g.flags & LITHOS_F_BIAS, with_gelu = g.flags & LITHOS_F_GELU, with_resid = g.flags & LITHOS_F_RESIDUAL;
    const int l16 = lane & 15, col = nw + (lane >> 4) * 4;
    f32x4a bias[NI], resid[2][NI];
    const auto load_resid = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        const float* const row = g.resid + (int64_t)min(mw + i * 16 + l16, g.M - 1) * g.ldr;
        if (with_resid) static_for<NI>([&](auto j) __attribute__((always_inline)) { resid[i & 1][j] = load_quad(row, col + j * 16, g.N); });
    };
    if (with_bias) static_for<NI>([&](auto j) __attribute__((always_inline)) { bias[j] = load_quad(g.bias, col + j * 16, g.N); });
    load_resid(std::integral_constant<int, 0>{});
    static_for<MI>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i + 1 < MI) load_resid(std::integral_constant<int, i + 1>{});
        if (with_bias) static_for<NI>([&](auto j) __attribute__((always_inline)) { acc[i][j] += bias[j]; });
        if (with_gelu) static_for<NI * 4>([&](auto je) __attribute__((always_inline)) {
            constexpr int j = decltype(je)::value / 4, e = decltype(je)::value % 4;
            acc[i][j][e] = gelu_erf(acc[i][j][e]);
        });
        if (with_resid) static_for<NI>([&](auto j) __attribute__((always_inline)) { acc[i][j] += resid[i & 1][j]; });
    });
}

// D strips of 16 rows of a wavefront's blocks into `scratch` (LDS of its own, D * 16 rows of NI * 16 floats): chunk c of four
// columns of row r lies at c ^ (r % 8).
template <int D, int DUMP, int MI, int NI>
__device__ __forceinline__ void dump_strips16(f32x4a (&acc)[MI][NI], int lane, float* scratch)
{
    wave_lds_sync();
    static_for<D * NI>([&](auto hj) __attribute__((always_inline)) {
        constexpr int h = decltype(hj)::value / NI, j = decltype(hj)::value % NI;
        const int r = h * 16 + (lane & 15);
        *reinterpret_cast<f32x4a*>(scratch + (r * NI * 4 + ((j * 4 + (lane >> 4)) ^ (r & 7))) * 4) = acc[DUMP * D + h][j];
    });
    wave_lds_sync();
}

// Element by element, where C does not divide into 16-byte pieces: the blocks go through LDS too, so that a lane has one
// column (or two) and a row leaves in one or two stores of neighbouring lanes, from a base in scalar registers.  A strip of 16
// rows at a time; its residual is loaded before the stores of the strip above.  Rows and columns beyond the matrix compute
// on its last ones and are not stored.  In turns of four elements per lane, each waiting for its LDS reads and computing 64-bit
// addresses (us, turns / strips): 6000 x 2000 x 136 NN fp32 on 64 CUs 84 / 51, 2000 x 1000 x 520 split in 64x192 tiles 34 / 22,
// 1000^3 TN with epilogue 23.4 / 17.4.
template <int D, int MI, int NI>
__device__ __forceinline__ void epilogue_elements16(const GemmArgs& g, f32x4a (&acc)[MI][NI], int mw, int nw, int lane, float* scratch)
{
    constexpr int WN = NI * 16, H = (WN + 63) / 64, R = 16;      // columns; of which a lane has H; rows of a strip
    const bool with_bias = g.flags & LITHOS_F_BIAS, with_gelu = g.flags & LITHOS_F_GELU, with_resid = g.flags & LITHOS_F_RESIDUAL;
    int col[H], n[H];
    float bias[H], resid[H][R];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        col[h] = min(h * 64 + lane, WN - 1);
        n[h] = min(nw + col[h], g.N - 1);
        if (with_bias) bias[h] = g.bias[n[h]];
    }
    const auto fetch = [&](int strip) __attribute__((always_inline)) {
        if (with_resid)
            static_for<H * R>([&](auto hr) __attribute__((always_inline)) {
                constexpr int h = decltype(hr)::value / R, r = decltype(hr)::value % R;
                resid[h][r] = (g.resid + (int64_t)min(mw + strip * R + r, g.M - 1) * g.ldr)[n[h]];
            });
    };
    fetch(0);
    static_for<MI / D>([&](auto dc) __attribute__((always_inline)) {
        constexpr int d = decltype(dc)::value;
        dump_strips16<D, d>(acc, lane, scratch);
#pragma unroll 1
        for (int s = 0; s < D; ++s) {
            const int strip = d * D + s, m = mw + strip * R, rows = g.M - m;
            float v[H][R];
            static_for<H * R>([&](auto hr) __attribute__((always_inline)) {
                constexpr int h = decltype(hr)::value / R, r = decltype(hr)::value % R;
                v[h][r] = scratch[(s * R + r) * WN + (((col[h] >> 2) ^ (r & 7)) << 2) + (col[h] & 3)];
            });
            if (with_bias) static_for<H * R>([&](auto hr) __attribute__((always_inline)) { v[decltype(hr)::value / R][decltype(hr)::value % R] += bias[decltype(hr)::value / R]; });
            if (with_gelu) static_for<H * R>([&](auto hr) __attribute__((always_inline)) { float& x = v[decltype(hr)::value / R][decltype(hr)::value % R]; x = gelu_erf(x); });
            if (with_resid) static_for<H * R>([&](auto hr) __attribute__((always_inline)) { v[decltype(hr)::value / R][decltype(hr)::value % R] += resid[decltype(hr)::value / R][decltype(hr)::value % R]; });
            fetch(min(strip + 1, MI - 1));
            const auto store = [&](auto* C, auto value) __attribute__((always_inline)) {
                static_for<H>([&](auto hc) __attribute__((always_inline)) {
                    constexpr int h = decltype(hc)::value;
                    if (h * 64 + lane < WN && nw + col[h] < g.N)
                        static_for<R>([&](auto rc) __attribute__((always_inline)) {
                            constexpr int r = decltype(rc)::value;
                            if (r < rows) (C + (int64_t)(m + r) * g.ldc)[n[h]] = value(v[h][r]);
                        });
                });
            };
            if (g.flags & LITHOS_F_OUT_F32) {
                store(reinterpret_cast<float*>(g.C), [](float x) __attribute__((always_inline)) { return x; });
                continue;
            }
            store(reinterpret_cast<uint16_t*>(g.C), [](float x) __attribute__((always_inline)) { return f32_to_bf16(x); });
            if (g.flags & LITHOS_F_OUT_SPLIT)       // second plane: what the first rounding dropped
                store(reinterpret_cast<uint16_t*>(g.C) + g.c_plane, [](float x) __attribute__((always_inline)) { return f32_to_bf16(x - bf16_to_f32(f32_to_bf16(x))); });
        }
    });
}

// Stores a wavefront's blocks as they are, 16 bytes at a time; bf16 values go a strip of 16 rows at a time through `scratch`
// (LDS of the wavefront's own), so that whole rows leave.
template <bool AGPR, int MI, int NI>
__device__ __forceinline__ void epilogue_plain16(const GemmArgs& g, f32x4a (&acc)[MI][NI], int mw, int nw, int lane, uint16_t* scratch)
{
    constexpr int WN = NI * 16, PW = WN / 8;        // 16-byte pieces of a row
    static_assert(16 * PW % 64 == 0, "whole wavefronts of pieces");
    const int l16 = lane & 15, quad = lane >> 4;
    if (g.flags & LITHOS_F_OUT_F32) {
        static_for<MI * NI>([&](auto ij) __attribute__((always_inline)) {
            constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
            const int m = mw + i * 16 + l16, n = nw + j * 16 + quad * 4;
            const f32x4a v = acc_block<AGPR>(acc, i, j);
            if (m < g.M && n < g.N) *reinterpret_cast<f32x4a*>(reinterpret_cast<float*>(g.C) + (int64_t)m * g.ldc + n) = v;
        });
        return;
    }
    // row r keeps its piece p at p ^ r, or as much of r as a row's pieces allow
    const auto at = [&](int r, int p) __attribute__((always_inline)) { return scratch + r * WN + ((p ^ ((PW & (PW - 1)) ? (r >> 2) & 3 : r & (PW - 1))) << 3); };
    const auto store = [&](auto lo, uint16_t* C) __attribute__((always_inline)) {     // lo: what the first rounding dropped
        static_for<MI>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            static_for<NI>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                const f32x4a v = acc_block<AGPR>(acc, i, j);
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { x[e] = v[e]; if constexpr (decltype(lo)::value) x[e] -= bf16_to_f32(f32_to_bf16(x[e])); }
                *reinterpret_cast<uint2*>(at(l16, j * 2 + (quad >> 1)) + 4 * (quad & 1)) = make_uint2(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]));
            });
            wave_lds_sync();
            uint4 w[PW / 4];
#pragma unroll
            for (int t = 0; t < PW / 4; ++t) w[t] = *reinterpret_cast<const uint4*>(at((t * 64 + lane) / PW, (t * 64 + lane) % PW));
#pragma unroll
            for (int t = 0; t < PW / 4; ++t) {
                const int m = mw + i * 16 + (t * 64 + lane) / PW, n = nw + (t * 64 + lane) % PW * 8;
                if (m < g.M && n < g.N) *reinterpret_cast<uint4*>(C + (int64_t)m * g.ldc + n) = w[t];
            }
            wave_lds_sync();
        });
    };
    store(std::false_type{}, reinterpret_cast<uint16_t*>(g.C));
    if (g.flags & LITHOS_F_OUT_SPLIT) store(std::true_type{}, reinterpret_cast<uint16_t*>(g.C) + g.c_plane);
}

// A wavefront's blocks, the first of which begins at (mw, nw).  whole: 16-byte pieces of C can be stored.
template <int D, int MI, int NI>
__device__ __forceinline__ void epilogue16(const GemmArgs& g, f32x4a (&acc)[MI][NI], int mw, int nw, int lane, bool whole, uint16_t* scratch)
{
    if (!whole) {
        epilogue_elements16<D>(g, acc, mw, nw, lane, reinterpret_cast<float*>(scratch));
        return;
    }
    if (g.flags & (LITHOS_F_BIAS | LITHOS_F_GELU | LITHOS_F_RESIDUAL)) epilogue_apply16(g, acc, mw, nw, lane);
    epilogue_plain16<false>(g, acc, mw, nw, lane, scratch);
}

} // namespace lithos
