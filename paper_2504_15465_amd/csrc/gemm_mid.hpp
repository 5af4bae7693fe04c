#pragma once
#include "gemm_mfma16.hpp"

namespace lithos {

// ---- 128x128 and 64x192 tiles, four wavefronts, any K % 8 == 0, any operand layout, split-bf16 A ----
// The loop of gemm_lds256_kernel (v_mfma_f32_16x16x32_bf16, 32-deep k-tiles by buffer loads into S LDS stages, fragments read a
// tile ahead, one LDS read or load behind each MFMA, one barrier per k-tile) in tiles of which two workgroups share a CU,
// so that one's prologue and epilogue run beside the other's MFMAs.  The power that the MFMAs take bounds the larger
// grids here too (4096 x 2304 x 768 split: MFMA pipes 80 % busy at 1.73 GHz), the number of tiles that the busiest CU gets
// the smaller ones: a split A, whose N are multiples of 192 in the encoder, takes 64x192 (768 tiles for 4096 x 2304, three to a CU).
//
// S = 5: two k-tiles at a time, every second turn, so that both halves of a line of a k-contiguous operand are fetched one after the
// other and the second comes from the L1.  A k-tile late: with two workgroups per CU the line is gone by then (K <= 2048, NT,
// rows that do not begin on lines, more than two tiles per CU: 0.80 to 0.97 of the time of S = 4; see gemm_plan).
//
// Against 32x32x16 MFMAs whose loads took five vector instructions each (us): 2048^3 NN 30 -> 21, 1536 x 1536 x 8192 TN 88 ->
// 51, 1003 x 3000 x 1160 NT with epilogue 26.5 -> 23, split 4096 x 2304 x 768 41 -> 31, 4096 x 768 x 3072 55 -> 39.
template <int BM, int BN, int S, bool KSA, bool KSB, bool SPLIT>
__global__ __launch_bounds__(256, 2)
void gemm_mid_kernel(GemmArgs g, AtomArgs atom)
{
#ifdef __HIP_DEVICE_COMPILE__       // the buffer types exist on the device only
    static_assert(S >= 3 && S <= 5, "built forms");
    constexpr bool PAIR = S == 5;                                        // k-tiles are fetched two at a time
    constexpr int BK = 32, WM = BM / 2, WN = BN / 2, MI = WM / 16, NI = WN / 16, AP = SPLIT ? 2 : 1;
    constexpr int NF = AP * MI + NI, NM = AP * MI * NI;                  // fragments and MFMAs of a k-tile
    constexpr int TA = BM / 16, TB = BN / 16;                            // 1 KB blocks of an operand's k-tile
    constexpr int NA = TA / 4, NB = TB / 4, NL = AP * NA + NB;     // .. that a wavefront fetches
    static_assert(TA % 4 == 0 && TB % 4 == 0 && (S - 1) * NL < 64, "loads");
    // separate arrays, each addressed statically: the compiler can then tell that the LDS reads of one stage do
    // not depend on the loads in flight into another
    __shared__ __attribute__((aligned(1024))) uint16_t A0[AP * BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t A1[AP * BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t A2[AP * BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t A3[S > 3 ? AP * BM * BK : 8];
    __shared__ __attribute__((aligned(1024))) uint16_t A4[S > 4 ? AP * BM * BK : 8];
    __shared__ __attribute__((aligned(1024))) uint16_t B0[BN * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B1[BN * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B2[BN * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B3[S > 3 ? BN * BK : 8];
    __shared__ __attribute__((aligned(1024))) uint16_t B4[S > 4 ? BN * BK : 8];
    const auto stage_a = [&](auto s) __attribute__((always_inline)) -> uint16_t* {
        constexpr int v = decltype(s)::value % S;
        if constexpr (v == 0) return A0; else if constexpr (v == 1) return A1; else if constexpr (v == 2) return A2; else if constexpr (v == 3) return A3; else return A4;
    };
    const auto stage_b = [&](auto s) __attribute__((always_inline)) -> uint16_t* {
        constexpr int v = decltype(s)::value % S;
        if constexpr (v == 0) return B0; else if constexpr (v == 1) return B1; else if constexpr (v == 2) return B2; else if constexpr (v == 3) return B3; else return B4;
    };

    const uint32_t L = atom_logical_block(atom);
    const Block3 blk = atom_delinearize(L, atom);
    uint32_t tm, tn;
    tile_of_block(blk.y * atom.gx + blk.x, g.tiles_m, g.tiles_n, tm, tn);   // blk.z is the K slice
    const int m0 = __builtin_amdgcn_readfirstlane(tm) * BM, n0 = __builtin_amdgcn_readfirstlane(tn) * BN;
    const uint32_t z = __builtin_amdgcn_readfirstlane(blk.z);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    int ks0, ks1;                                   // this block's k range is [klo, klo + to_fetch)
    slice_ktiles(g, z, (g.K + 63) / 64, ks0, ks1);
    const int64_t klo = __builtin_amdgcn_readfirstlane(ks0) * 64;
    int to_fetch = min(g.K, __builtin_amdgcn_readfirstlane(ks1) * 64) - (int)klo;
    const int n_it = (to_fetch + BK - 1) / BK;
    if (g.k_slices > 1) g.C = reinterpret_cast<float*>(g.C) + (int64_t)z * g.c_slice;

    const int mw = m0 + wm * WM, nw = n0 + wn * WN;
    const bool whole = g.wide && ((g.N & 7) == 0 || n0 + BN <= g.N);     // whole 16-byte pieces of C

    // Block b of an operand's k-tile is 1 KB of LDS, filled by one load instruction, lane l its 16-byte piece l.
    // k-contiguous: 8 lines of two rows, piece p of line n holds chunk c of row 2n + r where 4r + c = p ^ (n & 7); rows
    // beyond the matrix re-read its last row.  k-strided: rows of R / 8 chunks, piece p of k-row k holds chunk p ^ ks_rot(k);
    // chunks beyond the matrix re-read its last one.  Byte offsets from the tile's first row (gemm_plan bounds them).
    const auto ks_rot = [](auto rows, int k) __attribute__((always_inline)) { return decltype(rows)::value % 128 == 0 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; };
    const auto lane_off = [&](auto ks, auto rows_c, int ld, int r0, int rows, int b) __attribute__((always_inline)) -> uint32_t {
        constexpr int CPR = decltype(rows_c)::value / 8;
        if constexpr (decltype(ks)::value) {
            const int k = (b * 64 + lane) / CPR, c = ((b * 64 + lane) % CPR) ^ ks_rot(rows_c, k);
            return (uint32_t)(k * ld + min(c * 8, rows - 8 - r0)) * 2;
        } else {
            const int line = b * 8 + (lane >> 3), p = (lane & 7) ^ (line & 7);
            return (uint32_t)(min(line * 2 + (p >> 2), rows - 1 - r0) * ld + (p & 3) * 8) * 2;
        }
    };
    constexpr std::bool_constant<KSA> ksa{};
    constexpr std::bool_constant<KSB> ksb{};
    constexpr std::integral_constant<int, BM> rows_a{};
    constexpr std::integral_constant<int, BN> rows_b{};
    // The bound is never reached: without it the compiler keeps more addresses in registers (181 against 158 with B k-strided) and
    // 2048 x 2048 x 256 NN on 192 CUs takes 8.9 us instead of 8.5.
    const auto b_block = [&](int i) __attribute__((always_inline)) { return min(wave * NB + i, TB - 1); };
    uint32_t oa[NA], ob[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) oa[i] = lane_off(ksa, rows_a, (int)g.lda, m0, g.M, wave * NA + i);
#pragma unroll
    for (int i = 0; i < NB; ++i) ob[i] = lane_off(ksb, rows_b, (int)g.ldb, n0, g.N, b_block(i));
    const int64_t a_step = KSA ? g.lda * BK : BK, b_step = KSB ? g.ldb * BK : BK;
    const uint16_t* pa = g.A + (KSA ? m0 + klo * g.lda : m0 * g.lda + klo);
    const uint16_t* pb = g.B + (KSB ? n0 + klo * g.ldb : n0 * g.ldb + klo);
    // k beyond the block's range must arrive as zeros.  k-strided: the buffer ends behind the last k-row.  k-contiguous:
    // the lanes whose chunk lies beyond get an offset that no buffer holds (all of them behind the last tile).
    const int lane_k = ((lane & 7) ^ (lane >> 3)) % 4 * 8;
    // Load q of the d-th of the k-tiles that are not yet fetched, and then to the tiles behind them.
    const auto load = [&](auto qc, auto dc, uint16_t* At, uint16_t* Bt) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, d = decltype(dc)::value;
        const int left = __builtin_amdgcn_readfirstlane(max(to_fetch - d * BK, 0));
        const uint32_t beyond = lane_k < to_fetch - d * BK ? 0u : ~0u;
        const auto rsrc = [&](auto ks, const uint16_t* p, int64_t ld) __attribute__((always_inline)) {
            return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, decltype(ks)::value ? min(left, BK) * (int)ld * 2 : -1, 0x00020000);
        };
        if constexpr (q < NB) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc(ksb, pb + d * b_step, g.ldb), (lptr_t)(Bt + b_block(q) * 512), 16, KSB ? ob[q] : ob[q] | beyond, 0, 0, 0);
        } else {
            constexpr int i = (q - NB) / AP, p = (q - NB) % AP;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc(ksa, (SPLIT ? pa + p * g.a_plane : pa) + d * a_step, g.lda), (lptr_t)(At + p * (BM * BK) + (wave * NA + i) * 512), 16,
                                                     KSA ? oa[i] : oa[i] | beyond, 0, 0, 0);
        }
    };
    const auto fetched = [&](int tiles) __attribute__((always_inline)) { to_fetch -= tiles * BK; pa += tiles * a_step; pb += tiles * b_step; };
    // Loads i0 .. i1 - 1 of k-tile t, or of the pair t, t + 1, the same block of both one after the other.
    const auto load_range = [&](auto tc, auto i0c, auto i1c) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value, i0 = decltype(i0c)::value, i1 = decltype(i1c)::value, N = PAIR ? 2 : 1;
        static_for<i1 - i0>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = i0 + decltype(ic)::value;
            constexpr std::integral_constant<int, t + i % N> tile{};
            load(std::integral_constant<int, i / N>{}, std::integral_constant<int, i % N>{}, stage_a(tile), stage_b(tile));
        });
        if constexpr (i1 > i0 && i1 == N * NL) fetched(N);
    };

    // Where this lane reads in a stage: a fragment is 16 rows, this lane row l16, the 8 k of chunk `quad`.  k-strided:
    // k-row 8 quad + l16/4, rows 4 (l16 % 4) .. +3 of the fragment's 16; the rotation mixes into the chunk's bits from 2 on,
    // so every second fragment needs an offset of its own.
    int ra[KSA ? (MI + 1) / 2 : 1], rb[KSB ? (NI + 1) / 2 : 1];
    const auto read_base = [&](auto ks, auto rows_c, int row0, auto& r) __attribute__((always_inline)) {
        constexpr int R = decltype(rows_c)::value;
        if constexpr (decltype(ks)::value) {
#pragma unroll
            for (int v = 0; v < (int)(sizeof(r) / sizeof(int)); ++v) {
                const int k = 8 * quad + (l16 >> 2);
                r[v] = k * R + (((row0 / 8 + 4 * v + ((l16 & 3) >> 1)) ^ ks_rot(rows_c, k)) << 3) + (l16 & 1) * 4;
            }
        } else {
            r[0] = row0 * 32 + (l16 >> 1) * 64 + ((((l16 & 1) * 4 + quad) ^ (l16 >> 1)) << 3);
        }
    };
    read_base(ksa, rows_a, wm * WM, ra);
    read_base(ksb, rows_b, wn * WN, rb);
    const auto frag = [&](auto ks, auto rows_c, auto fc, const uint16_t* T, const auto& r) __attribute__((always_inline)) -> bf16x8 {
        constexpr int f = decltype(fc)::value;
        if constexpr (decltype(ks)::value) {
            typedef __attribute__((address_space(3))) s16x4* tr_t;
            const uint16_t* const p = T + r[f >> 1] + (f & 1) * 16;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_t)p), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_t)(p + 4 * decltype(rows_c)::value));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(T + r[0] + f * 512));
        }
    };

    f32x4a acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4a{0.f, 0.f, 0.f, 0.f};
    bf16x8 fr[2][NF];                               // two sets of fragments, A's (plane by plane), then B's, alternating between the tiles
    // in the order of their first use: the first of A's small plane, all of B's, the rest of A's
    const auto read = [&](auto qc, const uint16_t* At, const uint16_t* Bt, auto set) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        if constexpr (q >= 1 && q <= NI) {
            fr[decltype(set)::value][AP * MI + q - 1] = frag(ksb, rows_b, std::integral_constant<int, q - 1>{}, Bt, rb);
        } else {
            constexpr int a = q == 0 ? 0 : q - NI, p = AP - 1 - a / MI, i = a % MI;
            fr[decltype(set)::value][p * MI + i] = frag(ksa, rows_a, std::integral_constant<int, i>{}, At + p * (BM * BK), ra);
        }
    };
    const auto turn = [&](auto in_flight) __attribute__((always_inline)) {
        // this wavefront's share of the tile that is read next has landed, its own LDS reads are done; then everybody's
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt((decltype(in_flight)::value & 15) | 0x70 | ((decltype(in_flight)::value >> 4) << 14));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int RS = NM * 3 / 4;                  // MFMAs that are followed by the reads of the next tile
    const auto tile_step = [&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        constexpr std::integral_constant<int, t + 1> next{};
        constexpr int F = !PAIR ? NL : t % 2 == 0 ? 2 * NL : 0;     // loads to issue: tile t + S, or the pair t + 4, t + 5
        // May still be in flight, tile t + 1 having landed: the S - 2 tiles behind it; the pair behind its own and, where it is the
        // first of its own, that pair's last load.
        turn(std::integral_constant<int, !PAIR ? (S - 2) * NL : 2 * NL + t % 2>{});
        static_for<NM>([&](auto mc) __attribute__((always_inline)) {
            // the small plane of a split A first; operands exchanged: a lane then holds four consecutive columns of one row of C
            constexpr int m = decltype(mc)::value, p = AP - 1 - m / (MI * NI), i = m % (MI * NI) / NI, j = m % NI;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[t & 1][AP * MI + j], fr[t & 1][p * MI + i], acc[i][j], 0, 0, 0);
            if constexpr (m < RS) {
                constexpr int r0 = m * NF / RS, r1 = (m + 1) * NF / RS;
                static_for<r1 - r0>([&](auto r) __attribute__((always_inline)) {
                    read(std::integral_constant<int, r0 + decltype(r)::value>{}, stage_a(next), stage_b(next), std::integral_constant<int, (t + 1) & 1>{});
                });
            }
            load_range(std::integral_constant<int, PAIR ? t + 4 : t + S>{}, std::integral_constant<int, m * F / NM>{}, std::integral_constant<int, (m + 1) * F / NM>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    constexpr int G = PAIR ? 2 : 1;                 // tiles that are fetched together
    static_for<PAIR ? 2 : S>([&](auto f) __attribute__((always_inline)) {
        load_range(std::integral_constant<int, decltype(f)::value * G>{}, std::integral_constant<int, 0>{}, std::integral_constant<int, G * NL>{});
    });
    turn(std::integral_constant<int, PAIR ? 2 * NL + 1 : (S - 1) * NL>{});      // tile 0 has landed
    static_for<NF>([&](auto q) __attribute__((always_inline)) { read(q, A0, B0, std::integral_constant<int, 0>{}); });
    // whole rounds of the stages and fragment sets, then the rest
    constexpr int U = S % 2 ? 2 * S : S;
    int it = 0;
    for (; it + U <= n_it; it += U) static_for<U>([&](auto t) __attribute__((always_inline)) { tile_step(t); });
    static_for<U - 1>([&](auto t) __attribute__((always_inline)) { if (it + decltype(t)::value < n_it) tile_step(t); });
    turn(std::integral_constant<int, 0>{});         // the stages are free

    // Strips, 32 WN elements of LDS each as floats: a stage of B for each wavefront, of three stages two of either operand.
    constexpr int ROOM = (S > 3 || BN < AP * BM ? BN : AP * BM) * BK / (32 * WN), D = ROOM >= MI ? MI : ROOM >= 2 ? 2 : 1;
    static_assert(ROOM >= 1 && MI % D == 0, "a strip in one stage of an operand");
    uint16_t* scratch;
    if constexpr (S > 3) scratch = wave == 0 ? B0 : wave == 1 ? B1 : wave == 2 ? B2 : B3;
    else scratch = wave == 0 ? A0 : wave == 1 ? A1 : wave == 2 ? B0 : B1;
    epilogue16<D>(g, acc, mw, nw, lane, whole, scratch);
#endif
}

} // namespace lithos
