// Register-staged MFMA tile GEMM (v_mfma_f32_32x32x16_bf16) for any operand layout: 256x256 output tiles, BK = 64,
// the K that gemm_lds256_kernel does not take (K % 64 != 0).  Every workgroup computes the tile named by its
// LOGICAL block index (LithOS Section 4.4).
#pragma once
#include "gemm_common.hpp"

namespace lithos {

// ---- global -> register -> LDS staging of one [256 x 64] operand tile ------
// KSTRIDED = false: the operand is k-contiguous in memory (A[m][k], or B given
// as [N,K]); a thread moves 16-byte chunks.
// KSTRIDED = true: the operand is stored [k][row] (row-contiguous: A given as
// [K,M], or B as [K,N]); a thread loads a KB x 8 block and writes it
// transposed, so LDS always holds k-contiguous rows.
constexpr int TILE = 256, TILE_T = 512;                         // output tile, threads (8 wavefronts, 2x4)

template <bool KSTRIDED>
struct TileStage {
    static constexpr int NCH = TILE * 8 / TILE_T;               // 16-byte registers per thread
    static constexpr int KB = 4;                                // k-rows of a thread's block of a k-strided operand
    uint4 r[NCH];

    __device__ __forceinline__ void load(const uint16_t* base, int64_t ld, int row0, int rows_total,
                                         int k0, int K, int tid)
    {
        if constexpr (!KSTRIDED) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                int c = tid + i * TILE_T;
                int row = c >> 3, kc = c & 7;
                int gr = min(row0 + row, rows_total - 1);
                int k = k0 + kc * 8;
                uint4 v = make_uint4(0, 0, 0, 0);
                if (k < K) v = *reinterpret_cast<const uint4*>(base + (int64_t)gr * ld + k);
                r[i] = v;
            }
        } else {
            int nb = tid % (TILE / 8), kb = tid / (TILE / 8);
            int gr = min(row0 + nb * 8, rows_total - 8);
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                int k = k0 + kb * KB + q;
                uint4 v = make_uint4(0, 0, 0, 0);
                if (k < K) v = *reinterpret_cast<const uint4*>(base + (int64_t)k * ld + gr);
                r[q] = v;
            }
        }
    }

    __device__ __forceinline__ void store(uint16_t* lds, int tid) const
    {
        if constexpr (!KSTRIDED) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                int c = tid + i * TILE_T;
                int row = c >> 3, kc = c & 7;
                *reinterpret_cast<uint4*>(lds + lds_index(row, kc)) = r[i];
            }
        } else {
            int nb = tid % (TILE / 8), kb = tid / (TILE / 8);
            int kbase = kb * KB;
#pragma unroll
            for (int j = 0; j < 8; ++j) {               // j-th row of the 8-row block
                int row = nb * 8 + j;
                uint32_t w[KB / 2];
#pragma unroll
                for (int p = 0; p < KB / 2; ++p) {      // pack k = 2p, 2p+1 of row j
                    const uint4& lo4 = r[2 * p];
                    const uint4& hi4 = r[2 * p + 1];
                    uint32_t lo = (j < 2) ? lo4.x : (j < 4) ? lo4.y : (j < 6) ? lo4.z : lo4.w;
                    uint32_t hi = (j < 2) ? hi4.x : (j < 4) ? hi4.y : (j < 6) ? hi4.z : hi4.w;
                    if (j & 1) w[p] = (lo >> 16) | (hi & 0xffff0000u);
                    else       w[p] = (lo & 0xffffu) | (hi << 16);
                }
                *reinterpret_cast<uint2*>(lds + lds_index(row, kbase >> 3) + (kbase & 7)) = make_uint2(w[0], w[1]);
            }
        }
    }
};

// ST: full bf16 tiles leave through LDS (operands exchanged in the MFMA, see stage_block).
// Registers are capped so that a 256x256 tile keeps two wavefronts per SIMD (one 8-wave workgroup
// per CU): left alone, the compiler spends the whole register file on hoisted epilogue addresses and halves the
// occupancy.
template <bool TA, bool TB, bool ST>
__global__ __launch_bounds__(TILE_T, 2)
void gemm_tile_kernel(GemmArgs g, AtomArgs atom)
{
    constexpr int BM = TILE, BN = TILE, WGM = 2, WGN = 4, T = TILE_T, BK = 64;
    constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32;
    // operand buffers; a staged epilogue needs room for the whole bf16 output tile
    constexpr int OPERAND_ELEMS = (BM + BN) * BK;
    __shared__ __attribute__((aligned(16))) uint16_t smem[ST && BM * BN > OPERAND_ELEMS ? BM * BN : OPERAND_ELEMS];
    uint16_t* const As = smem;
    uint16_t* const Bs = smem + BM * BK;

    const uint32_t L = atom_logical_block(atom);
    const Block3 blk = atom_delinearize(L, atom);
    uint32_t tm, tn;
    tile_of_block(blk.y * atom.gx + blk.x, g.tiles_m, g.tiles_n, tm, tn);   // blk.z is the K slice
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    TileStage<TA> sa;        // A is k-strided in memory when transposed
    TileStage<!TB> sb;       // B is k-strided in memory when NOT transposed

    int kt0, kt1;
    slice_ktiles(g, blk.z, (g.K + BK - 1) / BK, kt0, kt1);
    const int KT = kt1;
    if (g.k_slices > 1) g.C = reinterpret_cast<float*>(g.C) + (int64_t)blk.z * g.c_slice;
    if (kt0 < kt1) {
        sa.load(g.A, g.lda, m0, g.M, kt0 * BK, g.K, tid);
        sb.load(g.B, g.ldb, n0, g.N, kt0 * BK, g.K, tid);
        sa.store(As, tid);
        sb.store(Bs, tid);
    }
    __syncthreads();

    for (int kt = kt0; kt < KT; ++kt) {
        if (kt + 1 < KT) {          // next tile's global loads fly during the MFMAs
            sa.load(g.A, g.lda, m0, g.M, (kt + 1) * BK, g.K, tid);
            sb.load(g.B, g.ldb, n0, g.N, (kt + 1) * BK, g.K, tid);
        }
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int kc = kk * 2 + (lane >> 5);
            bf16x8 af[MI], bfr[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                int row = wm * WM + i * 32 + (lane & 31);
                af[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(As + lds_index(row, kc)));
            }
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                int row = wn * WN + j * 32 + (lane & 31);
                bfr[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(Bs + lds_index(row, kc)));
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    if constexpr (ST)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
                }
        }
        __syncthreads();            // every wave is done reading this tile
        if (kt + 1 < KT) {
            sa.store(As, tid);
            sb.store(Bs, tid);
            __syncthreads();
        }
    }

    if constexpr (ST) {
        // the operand buffers are free after the loop's last barrier
        constexpr int PPR = BN / 8;
        if (m0 + BM <= g.M && n0 + BN <= g.N && (g.flags & LITHOS_F_OUT_F32)) {
            static_for<MI * NI>([&](auto ij) {
                constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                store_block_swapped_f32(g, reinterpret_cast<float*>(g.C), m0 + wm * WM + i * 32 + (lane & 31),
                                        n0 + wn * WN + j * 32, acc[i][j], lane);
            });
        } else if (m0 + BM <= g.M && n0 + BN <= g.N) {
            uint16_t* const C = reinterpret_cast<uint16_t*>(g.C);
            static_for<MI * NI>([&](auto ij) {
                constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                const int rb = wm * WM + i * 32;
                epilogue_block_swapped(g, m0 + rb + (lane & 31), n0 + wn * WN + j * 32, acc[i][j], lane);
                stage_block_values<BN, false>(smem, rb + (lane & 31), wn * WN + j * 32, acc[i][j], lane);
            });
            auto store_tile = [&](uint16_t* dst) {
                __syncthreads();
#pragma unroll 4
                for (int c = tid; c < BM * PPR; c += T) {
                    const int r = c / PPR, p = c % PPR;
                    const uint4 v = *reinterpret_cast<const uint4*>(smem + stage_index<BN>(r, p));
                    *reinterpret_cast<uint4*>(dst + (int64_t)(m0 + r) * g.ldc + n0 + p * 8) = v;
                }
            };
            store_tile(C);
            if (g.flags & LITHOS_F_OUT_SPLIT) {          // second plane: what the bf16 rounding dropped
                __syncthreads();
                static_for<MI * NI>([&](auto ij) {
                    constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                    stage_block_values<BN, true>(smem, wm * WM + i * 32 + (lane & 31), wn * WN + j * 32, acc[i][j], lane);
                });
                store_tile(C + g.c_plane);
            }
        } else {
            static_for<MI * NI>([&](auto ij) {
                constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                store_block_swapped(g, m0 + wm * WM + i * 32 + (lane & 31), n0 + wn * WN + j * 32, acc[i][j], lane);
            });
        }
        return;
    }

    // 32x32 accumulator block: lane holds column (lane & 31); element e is
    // row 8*(e/4) + 4*(lane/32) + e%4.
    static_for<MI * NI>([&](auto ij) {
        constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
        const int n = n0 + wn * WN + j * 32 + (lane & 31);
        const int mb = m0 + wm * WM + i * 32 + 4 * (lane >> 5);
        static_for<16>([&](auto ee) {
            constexpr int e = decltype(ee)::value;
            epilogue_store(g, mb + 8 * (e >> 2) + (e & 3), n, acc[i][j][e]);
        });
    });
}

#define LITHOS_TILE_PICK(ST)                                                                            \
    (ta ? (tb ? (gemm_fn)gemm_tile_kernel<true, true, ST> : (gemm_fn)gemm_tile_kernel<true, false, ST>)   \
        : (tb ? (gemm_fn)gemm_tile_kernel<false, true, ST> : (gemm_fn)gemm_tile_kernel<false, false, ST>))

} // namespace lithos
