#pragma once
#include "gemm_mfma16.hpp"

namespace lithos {

// ---- 256x256 tile, K a multiple of 64, any operand layout, plain stores of 16-byte pieces ----------
// Four wavefronts of 128x128, one per SIMD: 256 accumulator registers and 256 for the rest.
//
// What bounds it: on random data the chip lowers its clock with the power that the MFMAs and everything around them
// take (8192^3: 2.39 GHz on zeros; on random data 1.8 for a loop with the MFMA pipes 62 % busy, 1.55 for one of the same
// MFMAs and 81 %, 1.84 for this one and 79 %), so a kernel that only fills the pipes better gains little, and one that does
// less beside the MFMAs gains twice.  Hence
//  * 128x128 per wavefront: 8 + 8 KB of LDS reads for 64 MFMAs; 128x64 reads half as much again;
//  * v_mfma_f32_16x16x32_bf16: per multiplication it moves half the accumulators of the 32x32x16 form, and twice the
//    operands, 0.5 bytes against 0.625: 8192^3 NN 735 us against 773;
//  * no vector instruction in the loop but MFMAs and LDS reads: the k-tiles come by buffer_load ... lds, whose base
//    advances in scalar registers and whose range is set to nothing behind the last tile (zeros arrive, no memory
//    is read); addresses in vector registers and a select per load made 820 of the 773;
//  * each MFMA is followed by at most one LDS read or load, in this order, so that the pipe never waits for the issue.
// The accumulators are named as AGPRs in inline assembly: left to itself the register allocator moves them
// between the two halves of the register file in every k-tile (8192^3: 5644 us).
//
// k-tiles are 32 deep in four LDS stages of 32 KB: during tile t the fragments of tile t + 1 are read into the second
// register set and tile t + 4 is fetched into the stage of tile t, whose fragments were read a tile before; one barrier
// per tile.  64-deep tiles in two stages (one tile ahead) take 929 us: the first touch of a k range comes from beyond L2.
//
// An operand that is k-contiguous in memory (A [M,K]; B given as [N,K]) lies in LDS as lines of 128 bytes, two rows
// of 32 k each, and a lane reads its 8 consecutive k with one 16-byte load.  An operand that is k-strided in
// memory (KSA: A given as [K,M]; KSB: B given as [K,N]) lies in LDS as it lies in memory, [32 k][256 rows],
// and is read with the transposing LDS load (ds_read_b64_tr_b16): within 16 lanes, source lane s supplies 4
// consecutive rows of k-row s/4, and lane l receives row l of the four k-rows: 4 consecutive k of one row, which is
// the MFMA operand layout.  Two such loads make a fragment; nothing is transposed in registers.
//
// 8192^3 NN 864 -> 735 us (1495 TFLOP/s; eight wavefronts of 128x64, 64-deep tiles, before), 4096^3 111 -> 96,
// 16384 x 1024 x 4096 NT 121 -> 104, 16384 x 4096 x 1024 NN 131 -> 116.

// The compiler does not see the latency of an MFMA written here: the accumulators are first read by other
// instructions behind the loop's last barrier and mfma16_settle.
__device__ __forceinline__ void mfma16_agpr(f32x4a& c, bf16x8 x, bf16x8 y)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
}
__device__ __forceinline__ void mfma16_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

template <bool KSA, bool KSB>
__global__ __launch_bounds__(256, 1)
void gemm_lds256_kernel(GemmArgs g, AtomArgs atom)
{
#ifdef __HIP_DEVICE_COMPILE__       // the buffer types exist on the device only
    constexpr int BM = 256, BN = 256, BK = 32, S = 4, MI = 8, NI = 8, NF = MI + NI, NM = MI * NI;
    constexpr int NBLK = 4, NL = 2 * NBLK;          // 1 KB blocks of each operand that a wavefront fetches; loads per k-tile
    // separate arrays, each addressed statically: the compiler can then tell that the LDS reads of one stage do
    // not depend on the loads in flight into another
    __shared__ __attribute__((aligned(1024))) uint16_t A0[BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t A1[BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t A2[BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t A3[BM * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B0[BN * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B1[BN * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B2[BN * BK];
    __shared__ __attribute__((aligned(1024))) uint16_t B3[BN * BK];
    const auto stage_a = [&](auto s) __attribute__((always_inline)) -> uint16_t* {
        constexpr int v = decltype(s)::value % S;
        if constexpr (v == 0) return A0; else if constexpr (v == 1) return A1; else if constexpr (v == 2) return A2; else return A3;
    };
    const auto stage_b = [&](auto s) __attribute__((always_inline)) -> uint16_t* {
        constexpr int v = decltype(s)::value % S;
        if constexpr (v == 0) return B0; else if constexpr (v == 1) return B1; else if constexpr (v == 2) return B2; else return B3;
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
    int kt0, kt1;                                   // this block's k range in units of 64
    slice_ktiles(g, z, g.K / 64, kt0, kt1);
    const int n_it = __builtin_amdgcn_readfirstlane(kt1 - kt0) * 2;
    const int64_t klo = __builtin_amdgcn_readfirstlane(kt0) * 64;
    if (g.k_slices > 1) g.C = reinterpret_cast<float*>(g.C) + (int64_t)z * g.c_slice;

    // Wavefront w fills LDS blocks 4w .. 4w+3 of each operand's k-tile, lane l the 16-byte piece l of a block.
    // k-contiguous: a block is 8 lines of two rows, piece p of line n holds chunk c of row 2n + r where 4r + c = p ^ (n & 7);
    // rows beyond the matrix re-read its last row.  k-strided: a block is 2 k-rows of 32 chunks, piece p of k-row k holds
    // chunk p ^ ((k & 3) << 2), so the four k-rows that one transposing load touches fall into different banks; chunks
    // beyond the matrix re-read its last one.  Byte offsets from the tile's first row (gemm_plan bounds them).
    const auto lane_off = [&](auto ks, int ld, int r0, int rows, int b) __attribute__((always_inline)) -> uint32_t {
        if constexpr (decltype(ks)::value) {
            const int k = b * 2 + (lane >> 5), c = (lane & 31) ^ ((k & 3) << 2);
            return (uint32_t)(k * ld + min(c * 8, rows - 8 - r0)) * 2;
        } else {
            const int line = b * 8 + (lane >> 3), p = (lane & 7) ^ (line & 7);
            return (uint32_t)(min(line * 2 + (p >> 2), rows - 1 - r0) * ld + (p & 3) * 8) * 2;
        }
    };
    constexpr std::bool_constant<KSA> ksa{};
    constexpr std::bool_constant<KSB> ksb{};
    uint32_t oa[NBLK], ob[NBLK];
#pragma unroll
    for (int i = 0; i < NBLK; ++i) {
        oa[i] = lane_off(ksa, (int)g.lda, m0, g.M, wave * NBLK + i);
        ob[i] = lane_off(ksb, (int)g.ldb, n0, g.N, wave * NBLK + i);
    }
    const int64_t a_step = KSA ? g.lda * BK : BK, b_step = KSB ? g.ldb * BK : BK;
    const uint16_t* pa = g.A + (KSA ? m0 + klo * g.lda : m0 * g.lda + klo);
    const uint16_t* pb = g.B + (KSB ? n0 + klo * g.ldb : n0 * g.ldb + klo);
    int to_fetch = n_it;
    const auto load = [&](auto qc, uint16_t* At, uint16_t* Bt) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const int range = __builtin_amdgcn_readfirstlane(~((to_fetch - 1) >> 31));      // everything, or nothing behind the last tile
        if constexpr (q < NBLK)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)pb, 0, range, 0x00020000), (lptr_t)(Bt + (wave * NBLK + q) * 512), 16, ob[q], 0, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)pa, 0, range, 0x00020000), (lptr_t)(At + (wave * NBLK + q - NBLK) * 512), 16, oa[q - NBLK], 0, 0, 0);
        if constexpr (q == NL - 1) { --to_fetch; pa += a_step; pb += b_step; }
    };

    // Where this lane reads in a stage.  A fragment is 16 rows: row l16, the 8 k of chunk `quad`.  k-contiguous: one
    // offset for all of a wavefront's fragments.  k-strided: k-row 8 quad + l16/4, rows 4 (l16 % 4) .. +3 of the fragment's
    // 16; the rotation mixes into bits 2 and 3 of the chunk, so fragments two apart need offsets of their own.
    int ra[KSA ? 4 : 1], rb[KSB ? 4 : 1];
    const auto read_base = [&](auto ks, int half, auto& r) __attribute__((always_inline)) {
        if constexpr (decltype(ks)::value) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                r[v] = (8 * quad + (l16 >> 2)) * 256 + half * 128 + ((v ^ (l16 >> 2)) << 5) + ((l16 & 3) >> 1) * 8 + (l16 & 1) * 4;
        } else {
            r[0] = half * 4096 + (l16 >> 1) * 64 + ((((l16 & 1) * 4 + quad) ^ (l16 >> 1)) << 3);
        }
    };
    read_base(ksa, wm, ra);
    read_base(ksb, wn, rb);
    const auto frag = [&](auto ks, auto fc, const uint16_t* T, const auto& r) __attribute__((always_inline)) -> bf16x8 {
        constexpr int f = decltype(fc)::value;
        if constexpr (decltype(ks)::value) {
            typedef __attribute__((address_space(3))) s16x4* tr_t;
            const uint16_t* const p = T + r[f >> 1] + (f & 1) * 16;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_t)p), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_t)(p + 4 * 256));
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
    bf16x8 fr[2][NF];                               // two sets of fragments, A's then B's, alternating between the tiles
    // in the order of their first use: A's first, all of B's, the rest of A's
    const auto read = [&](auto qc, const uint16_t* At, const uint16_t* Bt, auto set) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        if constexpr (q >= 1 && q <= NI) fr[decltype(set)::value][MI + q - 1] = frag(ksb, std::integral_constant<int, q - 1>{}, Bt, rb);
        else { constexpr int a = q == 0 ? 0 : q - NI; fr[decltype(set)::value][a] = frag(ksa, std::integral_constant<int, a>{}, At, ra); }
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
        constexpr std::integral_constant<int, t> cur{};
        constexpr std::integral_constant<int, t + 1> next{};
        turn(std::integral_constant<int, (S - 2) * NL>{});
        static_for<NM>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            // operands exchanged: a lane then holds four consecutive columns of one row of C
            mfma16_agpr(acc[m / NI][m % NI], fr[t & 1][MI + m % NI], fr[t & 1][m / NI]);
            if constexpr (m < RS && (m + 1) * NF / RS > m * NF / RS)
                read(std::integral_constant<int, m * NF / RS>{}, stage_a(next), stage_b(next), std::integral_constant<int, (t + 1) & 1>{});
            if constexpr ((m + 1) * NL / NM > m * NL / NM)
                load(std::integral_constant<int, m * NL / NM>{}, stage_a(cur), stage_b(cur));
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    static_for<S>([&](auto s) __attribute__((always_inline)) { static_for<NL>([&](auto q) __attribute__((always_inline)) { load(q, stage_a(s), stage_b(s)); }); });
    turn(std::integral_constant<int, (S - 1) * NL>{});
    static_for<NF>([&](auto q) __attribute__((always_inline)) { read(q, A0, B0, std::integral_constant<int, 0>{}); });
    // whole rounds of the stages, then the rest
    int it = 0;
    for (; it + S <= n_it; it += S) static_for<S>([&](auto t) __attribute__((always_inline)) { tile_step(t); });
    if (it < n_it) {                                // n_it is even
        tile_step(std::integral_constant<int, 0>{});
        tile_step(std::integral_constant<int, 1>{});
    }
    turn(std::integral_constant<int, 0>{});         // the stages are free
    mfma16_settle();

    epilogue_plain16<true>(g, acc, m0 + wm * 128, n0 + wn * 128, lane, wave == 0 ? A0 : wave == 1 ? A1 : wave == 2 ? A2 : A3);
#endif
}

} // namespace lithos
