// 32x64 tiles for the GEMMs of few rows with a split A (a request of one sequence): grids of at most 64 tiles.
//
// Such a grid leaves each CU one tile and nothing to hide its latencies with; every launch finds the L2 of a die cold, so the chain
// of k-tiles waits for what lies behind it, about 0.8 us each time.  So the four wavefronts split K between them, chunk c of 64
// going to wavefront c % 4, and each fetches two chunks at a time into its own LDS (128 KB in flight per CU),
// without a barrier until their sums are added, in wavefront order.  128 x 768 x 3072 with bias and residual 12.2 us against
// 16.8 with 64x64 tiles (24 tiles, two groups of wavefronts), 128 x 1024 x 1024 7.1 against 8.5, 128 x 768 x 768 6.3 against 7.4.
// Made for partitions of a quarter of the chip or more: where CUs are fewer than about 1.3 times the tiles some get two, one after
// the other, and 64x64 tiles are faster (128 x 768 x 768 10.9 / 7.5 on 24 to 48 CUs, 15.6 / 10.9 on 16, 29 / 15.5 on 8); a grid cannot
// depend on the partition.  Two workgroups per CU (64 KB of LDS, the fragments of A loaded into registers) help neither: K = 3072 takes
// 30 us against 22 on 48 CUs and 17.0 against 12.4 on 64.
// The same for plain operands in 64x64 tiles is slower up to K = 4096 (512^3 6.6 / 5.3, 512 x 512 x 4096 17.0 / 16.0).
#include "gemm_mfma16.hpp"

namespace lithos {

template <bool KSB>
__global__ __launch_bounds__(256, 1)
void gemm_thin_kernel(GemmArgs g, AtomArgs atom)
{
#ifdef __HIP_DEVICE_COMPILE__       // the buffer types exist on the device only
    constexpr int BM = 32, BN = 64, BK = 64, MI = BM / 16, NI = BN / 16, AE = BM * BK, BE = BN * BK;
    constexpr int NA = AE / 512, NB = BE / 512, NL = 2 * NA + NB;        // loads of 1 KB: of a plane, of B, of a chunk
    // two chunks per wavefront, each the two planes of A [32][64 k], and B
    __shared__ __attribute__((aligned(1024))) uint16_t A0[4 * 2 * AE];
    __shared__ __attribute__((aligned(1024))) uint16_t A1[4 * 2 * AE];
    __shared__ __attribute__((aligned(1024))) uint16_t B0[4 * BE];
    __shared__ __attribute__((aligned(1024))) uint16_t B1[4 * BE];

    const uint32_t L = atom_logical_block(atom);
    uint32_t tm, tn;
    tile_of_block(L, g.tiles_m, g.tiles_n, tm, tn);
    const int m0 = __builtin_amdgcn_readfirstlane(tm) * BM, n0 = __builtin_amdgcn_readfirstlane(tn) * BN;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // this thread's quads of C: columns 4 (tid % 16) .. +3 of rows tid / 16 and 16 more
    const bool whole = g.wide && ((g.N & 7) == 0 || n0 + BN <= g.N);
    const bool with_bias = g.flags & LITHOS_F_BIAS, with_gelu = g.flags & LITHOS_F_GELU, with_resid = g.flags & LITHOS_F_RESIDUAL;
    const int cn = n0 + (tid & 15) * 4;
    float bias[4], resid[2][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int n = min(cn + e, g.N - 1);
        if (with_bias) bias[e] = g.bias[n];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (with_resid) resid[h][e] = g.resid[(int64_t)min(m0 + h * 16 + (tid >> 4), g.M - 1) * g.ldr + n];
    }

    // Loads: lane l fills 16-byte piece l of a 1 KB block.  k-contiguous: a block is 8 rows of 64 k, piece p of row r holds
    // chunk p ^ (r % 8).  k-strided: 8 k-rows of 64 columns, piece p of k-row k holds chunk p ^ ks_rot(k).  Rows and columns beyond
    // the matrix re-read its last ones; k beyond it arrives as zeros (an offset that no buffer holds; the buffer's end).
    const auto ks_rot = [](int k) __attribute__((always_inline)) { return ((k >> 1) & 1) << 2; };
    const int lk = ((lane & 7) ^ (lane >> 3)) * 8;
    uint32_t oa[NA], ob[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) oa[i] = (uint32_t)(min(i * 8 + (lane >> 3), g.M - 1 - m0) * (int)g.lda + lk) * 2;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int r = i * 8 + (lane >> 3);
        if constexpr (KSB) ob[i] = (uint32_t)(r * (int)g.ldb + min(((lane & 7) ^ ks_rot(r)) * 8, g.N - 8 - n0)) * 2;
        else ob[i] = (uint32_t)(min(r, g.N - 1 - n0) * (int)g.ldb + lk) * 2;
    }
    int left = g.K - wave * BK;                     // k from this wavefront's next chunk on
    const uint16_t* pa = g.A + (int64_t)m0 * g.lda + wave * BK;
    const uint16_t* pb = g.B + (KSB ? n0 + (int64_t)wave * BK * g.ldb : (int64_t)n0 * g.ldb + wave * BK);
    const int64_t b_step = KSB ? 4 * BK * g.ldb : 4 * BK;
    const auto fetch = [&](uint16_t* At, uint16_t* Bt) __attribute__((always_inline)) {
        const uint32_t beyond = lk < left ? 0u : ~0u;
        const int b_range = KSB ? min(__builtin_amdgcn_readfirstlane(max(left, 0)), BK) * (int)g.ldb * 2 : -1;
#pragma unroll
        for (int i = 0; i < NB; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)pb, 0, b_range, 0x00020000), (lptr_t)(Bt + wave * BE + i * 512), 16, KSB ? ob[i] : ob[i] | beyond, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 2 * NA; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)(pa + (i / NA) * g.a_plane), 0, -1, 0x00020000), (lptr_t)(At + wave * (2 * AE) + i * 512), 16, oa[i % NA] | beyond, 0, 0, 0);
        left -= 4 * BK;
        pa += 4 * BK;
        pb += b_step;
    };

    f32x4a acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4a{0.f, 0.f, 0.f, 0.f};
    bf16x8 af[2][2][2][MI], bf[2][2][NI];            // fragments: chunk, k-half, (plane,) block
    const auto read = [&](int x, const uint16_t* At, const uint16_t* Bt) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    af[x][kk][p][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(At + wave * (2 * AE) + p * AE + (i * 16 + l16) * 64 + (((kk * 4 + quad) ^ (l16 & 7)) << 3)));
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                if constexpr (KSB) {
                    // k-row 8 quad + l16/4 (and 4 more), columns 4 (l16 % 4) .. +3 of the fragment's 16
                    typedef __attribute__((address_space(3))) s16x4* tr_t;
                    const int k = kk * 32 + 8 * quad + (l16 >> 2);
                    const uint16_t* const at = Bt + wave * BE + k * 64 + (((j * 2 + ((l16 & 3) >> 1)) ^ ks_rot(k)) << 3) + (l16 & 1) * 4;
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_t)at), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_t)(at + 4 * 64));
                    bf[x][kk][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                } else {
                    bf[x][kk][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(Bt + wave * BE + (j * 16 + l16) * 64 + (((kk * 4 + quad) ^ (l16 & 7)) << 3)));
                }
            }
        }
    };
    const auto multiply = [&](int x) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int p = 1; p >= 0; --p)             // the small plane first
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)     // operands exchanged: a lane holds four consecutive columns of one row of C
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[x][kk][j], af[x][kk][p][i], acc[i][j], 0, 0, 0);
    };
    // Chunks that do not exist are neither fetched nor multiplied: loads without a lane inside their buffer take time too
    // (128 x 768 x 768 7.0 us with them, 6.3 without).
    int chunks = ((g.K + BK - 1) / BK - wave + 3) / 4;       // this wavefront's
    if (chunks > 0) fetch(A0, B0);
    if (chunks > 1) fetch(A1, B1);
    for (; chunks > 0; chunks -= 2) {                // two a turn
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0): both have landed
        asm volatile("" ::: "memory");
        read(0, A0, B0);
        if (chunks > 1) read(1, A1, B1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0): both have been read and can be filled again
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (chunks > 2) fetch(A0, B0);
        if (chunks > 3) fetch(A1, B1);
        multiply(0);
        if (chunks > 1) multiply(1);
    }
    __syncthreads();

    // the wavefronts' sums, [32][64] each, 16-byte chunk c of row r at c ^ (r % 8)
    float* const red = reinterpret_cast<float*>(A0);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int r = i * 16 + l16;
            *reinterpret_cast<f32x4a*>(red + wave * (BM * BN) + r * BN + (((j * 4 + quad) ^ (r & 7)) << 2)) = acc[i][j];
        }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = h * 16 + (tid >> 4), m = m0 + r;
        f32x4a v = f32x4a{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const f32x4a*>(red + w * (BM * BN) + r * BN + (((tid & 15) ^ (r & 7)) << 2));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (with_bias) v[e] += bias[e];
            if (with_gelu) v[e] = gelu_erf(v[e]);
            if (with_resid) v[e] += resid[h][e];
        }
        if (m >= g.M) continue;
        const int64_t at = (int64_t)m * g.ldc + cn;
        if (!whole) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (cn + e < g.N) store_value(g, at + e, v[e]);
        } else if (cn < g.N) {
            if (g.flags & LITHOS_F_OUT_F32) {
                *reinterpret_cast<f32x4a*>(reinterpret_cast<float*>(g.C) + at) = v;
                continue;
            }
            uint16_t* const C = reinterpret_cast<uint16_t*>(g.C) + at;
            *reinterpret_cast<uint2*>(C) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            if (g.flags & LITHOS_F_OUT_SPLIT) {      // second plane: what the first rounding dropped
                float lo[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) lo[e] = v[e] - bf16_to_f32(f32_to_bf16(v[e]));
                *reinterpret_cast<uint2*>(C + g.c_plane) = make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]));
            }
        }
    }
#endif
}

gemm_fn gemm_thin_fn(bool tb) { return tb ? (gemm_fn)gemm_thin_kernel<false> : (gemm_fn)gemm_thin_kernel<true>; }

} // namespace lithos
