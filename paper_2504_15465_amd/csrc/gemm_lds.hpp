// Direct-to-LDS MFMA tile GEMM (v_mfma_f32_32x32x16_bf16), 64x64 (and some 128x128) output tiles, any operand
// layout, any K % 8 == 0, split-bf16 A.  Every workgroup computes the tile named by its LOGICAL block
// index (LithOS Section 4.4).
#pragma once
#include "gemm_common.hpp"

namespace lithos {

// what a lane fetches where its k lies beyond the operand (or the K slice)
__device__ const uint4 gemm_zero_chunk = {0, 0, 0, 0};

// One k-tile of an operand in LDS.  k-contiguous operand: [rows][BK], in lines of 128 bytes (one row of 64 k or
// two rows of 32); 16-byte chunk p of line l is stored at p ^ swz(l), so 8 lanes that read one chunk column of
// consecutive rows touch 8 different slots.
template <int BK>
__device__ __forceinline__ int kc_index(int row, int kc)
{
    constexpr int CH = BK / 8, RPL = 8 / CH;
    const int line = row / RPL;
    return line * 64 + ((((row % RPL) * CH + kc) ^ swz(line)) << 3);
}

// k-strided operand: [BK][R rows] as in memory, read with the transposing LDS load, in which 16 lanes touch four
// k-rows: 16-byte chunks are rotated by 64 bytes so that the four land in different banks.
template <int R>
__device__ __forceinline__ int kr_shift(int k) { return R >= 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; }
template <int R>
__device__ __forceinline__ int kr_index(int k, int row) { return k * R + (((row >> 3) ^ kr_shift<R>(k)) << 3) + (row & 7); }

// s_waitcnt vmcnt(n) lgkmcnt(0)
constexpr int wait_imm(int n) { return (n & 15) | 0x70 | ((n >> 4) << 14); }

// KG groups of WGM x WGN wavefronts share the output tile: group g takes the k-tiles g, g + KG, .. and the
// groups' sums are added in group order.  With few output tiles the workgroup's chain of k-tiles, each a round
// trip to L2, is what its time consists of, and KG = 2 halves it.
//
// S stages of LDS: k-tiles go from global memory straight into LDS (global_load_lds_dwordx4, 1 KB per
// wavefront and instruction) S - 1 tiles ahead, with one barrier per tile; operand fragments of step kk + 1 are
// read before the MFMAs of step kk, across the barrier too.  A chunk beyond K is fetched from gemm_zero_chunk.
//
// Bound by the latency of the chain of k-tiles: what a k-tile brings is new to the die's L2, about 0.65 us a tile for grids of
// a few blocks whatever the number of stages.  Against the form that staged through registers into one buffer 512^3 in eight
// atoms on 32 CUs 55 -> 41 us.  Larger tiles, and a split A in grids of more or fewer tiles, are gemm_mid_kernel's and
// gemm_thin_kernel's; here stay 128 tiles of rows that need 64-bit addresses, and of two k-contiguous operands with a long K
// and many tiles, whose lines 64-deep k-tiles read whole (see gemm_plan).
template <int BM, int BN, int WGM, int WGN, int KG, int BK, int S, int MINW, bool TA, bool TB, bool SPLIT, bool ST>
__global__ __launch_bounds__(WGM * WGN * KG * 64, MINW)
void gemm_lds_kernel(GemmArgs g, AtomArgs atom)
{
    static_assert((S == 2 || S == 3) && (KG == 1 || KG == 2) && (BK == 32 || BK == 64), "built forms");
    constexpr bool KSA = TA, KSB = !TB;              // k-strided in memory
    constexpr int GW = WGM * WGN, T = GW * KG * 64, WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32;
    constexpr int AP = SPLIT ? 2 : 1;                // planes of A
    constexpr int AE = BM * BK, BE = BN * BK;        // elements of a plane's k-tile
    constexpr int NA = AE / 512 / GW, NB = BE / 512 / GW;    // 1 KB blocks per wavefront, plane and k-tile
    static_assert(NA * GW * 512 == AE && NB * GW * 512 == BE, "whole 1 KB blocks per wavefront");
    constexpr int NL = AP * NA + NB;                 // loads in flight per wavefront and k-tile
    constexpr int KK = BK / 16;
    // separate arrays, each addressed statically: the compiler can then tell that the LDS reads of one stage do
    // not depend on the loads in flight into another
    __shared__ __attribute__((aligned(1024))) uint16_t A0[KG * AP * AE];
    __shared__ __attribute__((aligned(1024))) uint16_t A1[KG * AP * AE];
    __shared__ __attribute__((aligned(1024))) uint16_t A2[S == 3 ? KG * AP * AE : 8];
    __shared__ __attribute__((aligned(1024))) uint16_t B0[KG * BE];
    __shared__ __attribute__((aligned(1024))) uint16_t B1[KG * BE];
    __shared__ __attribute__((aligned(1024))) uint16_t B2[S == 3 ? KG * BE : 8];

    const uint32_t L = atom_logical_block(atom);
    const Block3 blk = atom_delinearize(L, atom);
    uint32_t tm, tn;
    tile_of_block(blk.y * atom.gx + blk.x, g.tiles_m, g.tiles_n, tm, tn);   // blk.z is the K slice
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = KG == 1 ? 0 : wave_all / GW, wave = KG == 1 ? wave_all : wave_all % GW;
    const int wm = wave / WGN, wn = wave % WGN;

    int ks0, ks1;                                    // this block's k range is [klo, khi)
    slice_ktiles(g, blk.z, (g.K + 63) / 64, ks0, ks1);
    const int klo = ks0 * 64, khi = min(g.K, ks1 * 64);
    const int n_it = (khi - klo + BK * KG - 1) / (BK * KG);
    if (g.k_slices > 1) g.C = reinterpret_cast<float*>(g.C) + (int64_t)blk.z * g.c_slice;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // Block b of an operand's k-tile is the 1 KB of LDS that one load instruction fills, lane l its 16-byte piece l:
    // which k and row of the operand that piece holds.  Rows beyond the matrix re-read its last row (or last 8).
    auto lane_k = [&](auto ks, auto rows_c, int b) -> int {
        constexpr int R = decltype(rows_c)::value;
        if constexpr (decltype(ks)::value) return b * (512 / R) + lane / (R / 8);
        else { const int line = b * 8 + (lane >> 3); return (((lane & 7) ^ swz(line)) % (BK / 8)) * 8; }
    };
    auto lane_ptr = [&](auto ks, auto rows_c, const uint16_t* base, int64_t ld, int r0, int rows, int b) {
        constexpr int R = decltype(rows_c)::value;
        const int k = lane_k(ks, rows_c, b);
        if constexpr (decltype(ks)::value) {
            const int c = (lane % (R / 8)) ^ kr_shift<R>(k);
            return base + (int64_t)k * ld + min(r0 + c * 8, rows - 8);
        } else {
            const int line = b * 8 + (lane >> 3);
            const int row = line * (64 / BK) + ((lane & 7) ^ swz(line)) / (BK / 8);
            return base + (int64_t)min(r0 + row, rows - 1) * ld + k;
        }
    };
    constexpr std::integral_constant<int, BM> rows_a{};
    constexpr std::integral_constant<int, BN> rows_b{};
    constexpr std::bool_constant<KSA> ksa{};
    constexpr std::bool_constant<KSB> ksb{};
    const uint16_t* ga[NA];
    const uint16_t* gb[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) ga[i] = lane_ptr(ksa, rows_a, g.A, g.lda, m0, g.M, wave * NA + i);
#pragma unroll
    for (int i = 0; i < NB; ++i) gb[i] = lane_ptr(ksb, rows_b, g.B, g.ldb, n0, g.N, wave * NB + i);
    const int64_t a_kstep = KSA ? g.lda : 1, b_kstep = KSB ? g.ldb : 1;    // elements per unit of k
    const int64_t a_plane = SPLIT ? g.a_plane : 0;

    // Always the same number of loads: a chunk beyond the k range (the ragged end, a group's missing last tile, the
    // tiles behind the last) comes from gemm_zero_chunk, by a select and not a branch, so that the counted wait in
    // tile_barrier holds on every path and the compiler adds none of its own.
    const uint64_t zero = reinterpret_cast<uint64_t>(&gemm_zero_chunk);
    auto load = [&](const uint16_t* src, bool in, uint16_t* dst) {
        const uint64_t p = reinterpret_cast<uint64_t>(src);
        __builtin_amdgcn_global_load_lds((gptr_t)(in ? p : zero), (lptr_t)dst, 16, 0, 0);
    };
    auto fetch = [&](uint16_t* Ad, uint16_t* Bd, int it) {
        const int k0 = klo + (it * KG + grp) * BK;
        const int64_t ka = k0 * a_kstep, kb = k0 * b_kstep;
        uint16_t* const a_dst = Ad + grp * (AP * AE) + wave * (NA * 512);
        uint16_t* const b_dst = Bd + grp * BE + wave * (NB * 512);
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const bool in = lane_k(ksa, rows_a, wave * NA + i) < khi - k0;
#pragma unroll
            for (int p = 0; p < AP; ++p) load(ga[i] + ka + p * a_plane, in, a_dst + p * AE + i * 512);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) load(gb[i] + kb, lane_k(ksb, rows_b, wave * NB + i) < khi - k0, b_dst + i * 512);
    };

    bf16x8 af[2][AP][MI], bfr[2][NI];                // operand fragments: two sets alternate between the steps
    // one 32-row fragment of k-step kk: rows r0 .. r0+31 of the tile, this lane's 8 k
    auto read_frag = [&](auto ks, auto rows_c, const uint16_t* tile, int r0, int kk) -> bf16x8 {
        constexpr int R = decltype(rows_c)::value;
        if constexpr (decltype(ks)::value) {
            // source lane s of a 16-lane group addresses k-row s/4, rows 4*(s%4)..+3 of the group's 16
            const int q = lane >> 4, s = lane & 15;
            const int k = kk * 16 + 8 * (q >> 1) + (s >> 2), row = r0 + 16 * (q & 1) + 4 * (s & 3);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(tile + kr_index<R>(k, row)));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(tile + kr_index<R>(k + 4, row)));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tile + kc_index<BK>(r0 + (lane & 31), kk * 2 + (lane >> 5))));
        }
    };
    auto read_frags = [&](const uint16_t* Ac, const uint16_t* Bc, int kk, int set) {
#pragma unroll
        for (int p = 0; p < AP; ++p)
#pragma unroll
            for (int i = 0; i < MI; ++i) af[set][p][i] = read_frag(ksa, rows_a, Ac + (grp * AP + p) * AE, wm * WM + i * 32, kk);
#pragma unroll
        for (int j = 0; j < NI; ++j) bfr[set][j] = read_frag(ksb, rows_b, Bc + grp * BE, wn * WN + j * 32, kk);
    };
    auto mfmas = [&](int set, int i0, int i1) {
#pragma unroll
        for (int p = AP - 1; p >= 0; --p)            // the small plane of a split A first
#pragma unroll
            for (int i = i0; i < i1; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    if constexpr (ST) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][p][i], acc[i][j], 0, 0, 0);
                    else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[set][p][i], bfr[set][j], acc[i][j], 0, 0, 0);
                }
    };
    // this wavefront's share of the tile that is read next has landed, its own LDS reads are done; then everybody's
    auto tile_barrier = [&](auto in_flight) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(wait_imm(decltype(in_flight)::value));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, (S - 2) * NL> tiles_behind{};
    // One k-tile: on entry set 0 holds its step 0; tile it + S - 1 is fetched into the stage that was last read before
    // the previous barrier.
    auto tile_step = [&](const uint16_t* Ac, const uint16_t* Bc, const uint16_t* An, const uint16_t* Bn, uint16_t* Af, uint16_t* Bf, int it) {
        fetch(Af, Bf, it + S - 1);
        __builtin_amdgcn_sched_barrier(0);
        static_for<KK - 1>([&](auto kc) {
            constexpr int kk = decltype(kc)::value;
            mfmas(kk & 1, 0, MI > 1 ? 1 : 0);
            __builtin_amdgcn_sched_barrier(0);
            read_frags(Ac, Bc, kk + 1, (kk + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(kk & 1, MI > 1 ? 1 : 0, MI);
            __builtin_amdgcn_sched_barrier(0);
        });
        tile_barrier(tiles_behind);
        read_frags(An, Bn, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        mfmas((KK - 1) & 1, 0, MI);
        __builtin_amdgcn_sched_barrier(0);
    };

    fetch(A0, B0, 0);
    if constexpr (S == 3) fetch(A1, B1, 1);
    tile_barrier(tiles_behind);
    read_frags(A0, B0, 0, 0);
    // Whole rounds of the stages, then the rest: steps that could leave the loop would share its back edge in the
    // compiler's eyes, which then waits for all loads once a round.
    int it = 0;
    if constexpr (S == 2) {
        for (; it + 2 <= n_it; it += 2) {
            tile_step(A0, B0, A1, B1, A1, B1, it);
            tile_step(A1, B1, A0, B0, A0, B0, it + 1);
        }
        if (it < n_it) tile_step(A0, B0, A1, B1, A1, B1, it);
    } else {
        for (; it + 3 <= n_it; it += 3) {
            tile_step(A0, B0, A1, B1, A2, B2, it);
            tile_step(A1, B1, A2, B2, A0, B0, it + 1);
            tile_step(A2, B2, A0, B0, A1, B1, it + 2);
        }
        if (it < n_it) tile_step(A0, B0, A1, B1, A2, B2, it);
        if (it + 1 < n_it) tile_step(A1, B1, A2, B2, A0, B0, it + 1);
    }
    tile_barrier(std::integral_constant<int, 0>{});  // the zero tiles behind the last have landed too: the stages are free

    if constexpr (KG == 2) {
        static_assert(KG * AP * AE * 2 >= GW * MI * NI * 4096, "group 1's accumulators fit one stage of A");
        float4* const red = reinterpret_cast<float4*>(A1);
        static_for<MI * NI * 4>([&](auto qq) {
            constexpr int q = decltype(qq)::value, b = q >> 2, e = (q & 3) * 4;
            if (grp == 1) red[(wave * (MI * NI * 4) + q) * 64 + lane] = make_float4(acc[b / NI][b % NI][e], acc[b / NI][b % NI][e + 1], acc[b / NI][b % NI][e + 2], acc[b / NI][b % NI][e + 3]);
        });
        __syncthreads();
        static_for<MI * NI * 4>([&](auto qq) {
            constexpr int q = decltype(qq)::value, b = q >> 2, e = (q & 3) * 4;
            if (grp == 0) {
                const float4 v = red[(wave * (MI * NI * 4) + q) * 64 + lane];
                acc[b / NI][b % NI][e] += v.x; acc[b / NI][b % NI][e + 1] += v.y;
                acc[b / NI][b % NI][e + 2] += v.z; acc[b / NI][b % NI][e + 3] += v.w;
            }
        });
    }

    if constexpr (ST) {
        // whole 16-byte pieces of C: every tile when N divides into them, else the full ones
        const bool wide = (g.N & 7) == 0 || n0 + BN <= g.N;
        if (wide && (g.flags & LITHOS_F_OUT_F32)) {
            if (grp != 0) return;
            static_for<MI * NI>([&](auto ij) {
                constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                store_block_swapped_f32(g, reinterpret_cast<float*>(g.C), m0 + wm * WM + i * 32 + (lane & 31),
                                        n0 + wn * WN + j * 32, acc[i][j], lane);
            });
        } else if (wide) {
            // rows 0 .. HALF-1 of the bf16 tile are staged in A0, the others in hi_half
            constexpr int PPR = BN / 8, HALF = BM == 64 ? 64 : BM / 2;
            static_assert(KG * AP * AE >= HALF * BN && (BM == 64 || (S == 3 ? KG * AP * AE : KG * BE) >= HALF * BN), "staged output");
            uint16_t* const C = reinterpret_cast<uint16_t*>(g.C);
            uint16_t* const hi_half = S == 3 ? A2 : B0;
            if (grp == 0)
                static_for<MI * NI>([&](auto ij) {
                    constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                    epilogue_block_swapped(g, m0 + wm * WM + i * 32 + (lane & 31), n0 + wn * WN + j * 32, acc[i][j], lane);
                });
            auto store_tile = [&](auto lo, uint16_t* dst) {
                if (grp == 0)
                    static_for<MI * NI>([&](auto ij) {
                        constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                        const int rb = wm * WM + i * 32;
                        stage_block_values<BN, decltype(lo)::value>(rb < HALF ? A0 : hi_half, rb % HALF + (lane & 31), wn * WN + j * 32, acc[i][j], lane);
                    });
                __syncthreads();
#pragma unroll 4
                for (int c = tid; c < BM * PPR; c += T) {
                    const int r = c / PPR, p = c % PPR;
                    const uint4 v = *reinterpret_cast<const uint4*>((r < HALF ? A0 : hi_half) + stage_index<BN>(r % HALF, p));
                    if (m0 + r < g.M && n0 + p * 8 < g.N) *reinterpret_cast<uint4*>(dst + (int64_t)(m0 + r) * g.ldc + n0 + p * 8) = v;
                }
            };
            store_tile(std::false_type{}, C);
            if (g.flags & LITHOS_F_OUT_SPLIT) {          // second plane: what the bf16 rounding dropped
                __syncthreads();
                store_tile(std::true_type{}, C + g.c_plane);
            }
        } else if (grp == 0) {
            static_for<MI * NI>([&](auto ij) {
                constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
                epilogue_store_block<true>(g, m0 + wm * WM + i * 32 + (lane & 31), n0 + wn * WN + j * 32 + 4 * (lane >> 5), acc[i][j], false);
            });
        }
        return;
    }

    if (grp != 0) return;
    // 32x32 accumulator block: lane holds column (lane & 31); element e is
    // row 8*(e/4) + 4*(lane/32) + e%4.
    const bool inside = m0 + BM <= g.M && n0 + BN <= g.N;
    static_for<MI * NI>([&](auto ij) {
        constexpr int i = decltype(ij)::value / NI, j = decltype(ij)::value % NI;
        epilogue_store_block<false>(g, m0 + wm * WM + i * 32 + 4 * (lane >> 5), n0 + wn * WN + j * 32 + (lane & 31), acc[i][j], inside);
    });
}

} // namespace lithos
