// Atom-aware bf16 GEMM for gfx950: C = op(A) op(B) [+bias][GELU][+residual].
// This file validates a GEMM descriptor, picks the kernel and launches one atom.
//
// Kernel families (one translation unit each):
//  * gemm_lds256_kernel (gemm_lds256.hpp, gemm_lds256{,_ta}.hip) - 256x256 tiles, K % 64 == 0, any operand
//    layout: global memory straight into LDS, k-strided operands read with the
//    transposing LDS load; the best-effort and training-shaped GEMMs;
//  * gemm_lds256w8_kernel (gemm_lds256w8.hpp) - the same tiles by eight wavefronts, for an epilogue and element-wise stores;
//  * gemm_mid_kernel (gemm_mid.hpp, gemm_mid{128,192}.hip) - 128x128 and 64x192 tiles, any K % 8 == 0,
//    split-bf16 A; global memory straight into LDS, three or four stages;
//  * gemm_lds_kernel (gemm_lds.hpp, gemm_tile{64,128}.hip) - 64 tiles, any K % 8 == 0, split-bf16 A, and the 128 tiles that
//    gemm_mid_kernel does not serve (see gemm_plan); global memory straight into LDS, two or three stages;
//  * gemm_tile_kernel (gemm_tile.hpp, gemm_tile256_{wide,elem}.hip) - 256 tiles with any other K, through registers;
//  * gemm_skinny_*_kernel (gemm_skinny.hip) - M <= 32 rows (bf16 or fp32
//    activations) against a [N,K] bf16 weight matrix: HBM-bound, the weights are
//    streamed exactly once.  The products still go through MFMA 16x16x32
//    (weights as the row operand): on a 64-CU partition the plain vector ALUs
//    would need longer for the 2*M*N*K flops than HBM needs for the weights.
//
// Every workgroup computes the output tile named by its LOGICAL block index
// (LithOS Section 4.4), so a launch of any sub-range of blocks writes exactly
// what the full launch writes for those tiles.  No atomics; a K that is cut
// into slices (dim[5]) puts the slice on the logical grid's z axis and writes
// one fp32 plane per slice, which SUM_SLICES adds in slice order: each block's
// arithmetic depends only on its logical index.
#include "gemm_common.hpp"

namespace lithos {

// ---- host side -------------------------------------------------------------

// gemm_lds256_kernel, gemm_mid_kernel and gemm_thin_kernel address their operands with 32-bit byte offsets from the tile's
// first row: 256 rows of this many elements are 2 GiB.  Longer rows take the same tiles, and choose among them, as the kernels
// with 64-bit addresses do.
constexpr int64_t MAX_OFFSET_LD = 1 << 22;

// Tile shapes that auto_tile alone chooses.
constexpr int TILE_64X192 = 64192, TILE_32X64 = 32064;

// The tile of a GEMM that names none.  lines: rows of its k-contiguous operands begin on 128-byte lines.
static int auto_tile(int64_t M, int64_t N, bool tb, bool split, bool sliced, bool long_rows, bool lines)
{
    const auto blocks = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const auto rounds = [](int64_t blocks) { return (blocks + 255) / 256; };       // tiles of the busiest CU of the whole chip
    const int64_t n128 = blocks(128, 128);
    if (split && !long_rows) {
        // At most one 32x64 tile per CU of a quarter of the chip: see gemm_thin.hip.
        if (!sliced && blocks(32, 64) <= 64) return TILE_32X64;
        // 64x192 tiles, if there is at least one for every second CU.  With few 128x128 tiles the choice is between them and 64x64
        // tiles, which win while every CU has one at most (us, 64x192 / 64x64: 4096 x 256 x 768 10.2 / 7.7, 8192 x 128 x 3072 32 / 23;
        // 4096 x 320 x 3072 on 128 CUs 38 / 53, 2048 x 768 x 768 NT on 64 18 / 27).
        const int64_t n64 = blocks(64, 64), n192 = blocks(64, 192);
        if (n128 < 128) return n192 >= 128 && n64 > 256 ? TILE_64X192 : 64;
        // Else against 128x128, by the area of the busiest CU's tiles and of all (us, 64x192 / 128x128: 4096 x 768 x 3072 36 / 43, 4096 x
        // 2304 x 768 31 / 37, 1500 x 2304 x 3072 62 / 47, 8192 x 256 x 768 on 64 CUs 35 / 27; as much area in 4096 x 3072 x 768 48.6 / 48.2, and
        // the encoder of 4096 tokens 0.6 % faster); not with half lines of two operands, of which the narrower tile fetches more
        // (2048 x 2048 x 2056 NT 66 / 50).
        return (lines || !tb) && rounds(n192) * 3 <= rounds(n128) * 4 && n192 * 3 <= n128 * 4 ? TILE_64X192 : 128;
    }
    if (n128 < 128) return 64;
    return !split && blocks(256, 256) >= 256 ? 256 : 128;
}

int gemm_square_tile(const lithos_op_t& op) { return ((op.dim[0] + 127) / 128) * ((op.dim[1] + 127) / 128) >= 128 ? 128 : 64; }

static int tile_threads(int variant) { return variant == V_TILE64 || variant == V_TILE128 || variant == V_MID128 || variant == V_MID128_PAIR || variant == V_MID192 || variant == V_THIN || variant == V_LDS256 ? 256 : 512; }

// full bf16 tiles can leave through LDS when whole 16-byte pieces of C rows are addressable
// (fp32 tiles of the same kernels are stored from registers, 16 bytes per lane)
static bool staged_epilogue(const lithos_op_t& op)
{
    if ((op.flags & LITHOS_F_OUT_SPLIT) && op.dim[4] % 8) return false;
    if (op.flags & LITHOS_F_OUT_F32) return op.ld[2] % 4 == 0 && op.dim[6] % 4 == 0 && aligned16(op.out[0]);
    return op.ld[2] % 8 == 0 && aligned16(op.out[0]);
}

static int norm_of(uint32_t flags) { return (flags & LITHOS_F_NORM_LN) ? 1 : (flags & LITHOS_F_NORM_RMS) ? 2 : 0; }

static gemm_fn variant_fn(int variant, bool ta, bool tb, bool a32, bool split, bool st, int norm)
{
    switch (variant) {
    case V_LDS256: return ta ? gemm_lds256_ta_fn(tb) : gemm_lds256_fn(tb);
    case V_LDS256W8: return st ? gemm_lds256w8_wide_fn(ta, tb) : gemm_lds256w8_elem_fn(ta, tb);
    case V_TILE64: return gemm_tile64_fn(ta, tb, split, st, false);
    case V_TILE64_2K: return gemm_tile64_fn(ta, tb, split, st, true);
    case V_TILE128: return gemm_tile128_fn(ta, tb, split, st);
    case V_MID128: return gemm_mid128_fn(ta, tb, split);
    case V_THIN: return gemm_thin_fn(tb);
    case V_MID128_PAIR: return gemm_mid128_pair_fn(ta, tb);
    case V_MID192: return gemm_mid192_fn(tb);
    case V_TILE256: return st ? gemm_tile256_wide_fn(ta, tb) : gemm_tile256_elem_fn(ta, tb);
    default: return gemm_skinny_fn(variant, a32, norm);
    }
}

int gemm_plan(const lithos_op_t& op, OpPlan* plan)
{
    const int64_t M = op.dim[0], N = op.dim[1], K = op.dim[2];
    const bool ta = op.flags & LITHOS_F_TRANS_A, tb = op.flags & LITHOS_F_TRANS_B, a32 = op.flags & LITHOS_F_IN_F32;
    const bool split = op.flags & LITHOS_F_SPLIT_A, out_split = op.flags & LITHOS_F_OUT_SPLIT;
    if (M <= 0 || N <= 0 || K <= 0 || M > (1 << 30) || N > (1 << 30) || K > (1 << 30))
        return fail(LITHOS_EINVAL, "gemm: M,N,K must be positive (got %lld,%lld,%lld)", (long long)M, (long long)N, (long long)K);
    if (K % 8) return fail(LITHOS_EINVAL, "gemm: K must be a multiple of 8 (got %lld)", (long long)K);
    const int64_t lda = op.ld[0], ldb = op.ld[1], ldc = op.ld[2], ldr = op.ld[3];
    if (lda % 8 || ldb % 8) return fail(LITHOS_EINVAL, "gemm: lda and ldb must be multiples of 8");
    if (lda < (ta ? M : K) || ldb < (tb ? K : N) || ldc < N)
        return fail(LITHOS_EINVAL, "gemm: leading dimension smaller than the row length");
    if (ta && (M % 8)) return fail(LITHOS_EINVAL, "gemm: a transposed A needs M %% 8 == 0");
    if (!tb && (N % 8)) return fail(LITHOS_EINVAL, "gemm: a non-transposed B needs N %% 8 == 0");
    if (!op.in[0] || !op.in[1] || !op.out[0]) return fail(LITHOS_EINVAL, "gemm: null operand");
    if (!aligned16(op.in[0]) || !aligned16(op.in[1])) return fail(LITHOS_EINVAL, "gemm: A and B must be 16-byte aligned");
    if ((op.flags & LITHOS_F_BIAS) && !op.in[2]) return fail(LITHOS_EINVAL, "gemm: BIAS set but in[2] is null");
    if (op.flags & LITHOS_F_RESIDUAL) {
        if (!op.in[3]) return fail(LITHOS_EINVAL, "gemm: RESIDUAL set but in[3] is null");
        if (ldr < N) return fail(LITHOS_EINVAL, "gemm: ldr smaller than N");
    }
    if (split && (ta || a32 || op.dim[3] <= 0 || op.dim[3] % 8))
        return fail(LITHOS_EINVAL, "gemm: SPLIT_A needs bf16 A, no TRANS_A and a plane stride (dim[3]) that is a positive multiple of 8");
    if (out_split && ((op.flags & LITHOS_F_OUT_F32) || op.dim[4] <= 0))
        return fail(LITHOS_EINVAL, "gemm: OUT_SPLIT needs a bf16 output and a positive plane stride (dim[4])");
    const int64_t slices = op.dim[5];
    if (slices < 0 || slices > LITHOS_GEMM_MAX_SLICES) return fail(LITHOS_EINVAL, "gemm: K slices (dim[5]) must be in [0, %d]", LITHOS_GEMM_MAX_SLICES);
    if (slices > 1) {
        if (!(op.flags & LITHOS_F_OUT_F32) || (op.flags & (LITHOS_F_BIAS | LITHOS_F_GELU | LITHOS_F_RESIDUAL | LITHOS_F_OUT_SPLIT | LITHOS_F_IN_F32)))
            return fail(LITHOS_EINVAL, "gemm: K slices write plain fp32 partial planes (OUT_F32, no epilogue flags); SUM_SLICES applies the epilogue");
        if (op.dim[6] < M * ldc) return fail(LITHOS_EINVAL, "gemm: slice plane stride (dim[6]) smaller than M*ldc");
        if (slices > (K + 63) / 64) return fail(LITHOS_EINVAL, "gemm: more K slices than 64-wide k-tiles");
    }
    const int norm = norm_of(op.flags);
    const bool glu = op.flags & LITHOS_F_GLU, fused = norm || glu;
    const bool long_rows = lda > MAX_OFFSET_LD || ldb > MAX_OFFSET_LD;
    const bool lines = (ta || lda % 64 == 0) && (!tb || ldb % 64 == 0);     // rows of the k-contiguous operands begin on 128-byte lines
    int tile = op.tile;
    // What a caller may name.  The shapes that auto_tile alone chooses are built for fewer descriptors and not checked for below.
    if (tile != 0 && tile != LITHOS_TILE_SKINNY && tile != 64 && tile != 128 && tile != 256)
        return fail(LITHOS_EINVAL, "gemm: unknown tile selector %d", tile);
    if (a32 && !(M <= 32 && tb && !ta && (tile == 0 || tile == LITHOS_TILE_SKINNY)))
        return fail(LITHOS_EINVAL, "gemm: fp32 activations (IN_F32) are only taken by the skinny kernel (M <= 32, TRANS_B)");
    if (tile == 0) {
        if (M <= 32 && tb && !ta && slices <= 1) tile = LITHOS_TILE_SKINNY;
        else tile = auto_tile(M, N, tb, split, slices > 1, long_rows, lines);
    }
    int variant;
    if (tile == LITHOS_TILE_SKINNY) {
        if (split) return fail(LITHOS_EINVAL, "gemm: the skinny kernel takes fp32 activations instead of SPLIT_A");
        if (slices > 1) return fail(LITHOS_EINVAL, "gemm: the skinny kernel splits K inside the workgroup; K slices need a tile kernel");
        if (M > 32 || !tb || ta) return fail(LITHOS_EINVAL, "gemm: the skinny kernel needs M <= 32, TRANS_B and no TRANS_A");
        if (N * ldb * 2 >= (1ll << 32)) return fail(LITHOS_EINVAL, "gemm: the skinny kernel addresses weight rows with 32-bit byte offsets (N*ldb*2 < 4 GiB)");
        if (a32 && (lda % 4)) return fail(LITHOS_EINVAL, "gemm: fp32 activations need lda %% 4 == 0");
        variant = V_SKINNY32;
        if (M <= 16) variant = M <= 4 ? V_SKL4 : M <= 8 ? V_SKL8 : V_SKL16;
        if (fused && M > 16) return fail(LITHOS_EINVAL, "gemm: NORM_LN, NORM_RMS and GLU need M <= 16");
        if (norm) {
            if ((op.flags & LITHOS_F_NORM_LN) && (op.flags & LITHOS_F_NORM_RMS)) return fail(LITHOS_EINVAL, "gemm: NORM_LN and NORM_RMS exclude each other");
            if (!a32) return fail(LITHOS_EINVAL, "gemm: NORM_LN / NORM_RMS need fp32 activations (IN_F32)");
            if (!op.in[4] || ((op.flags & LITHOS_F_NORM_LN) && !op.in[5])) return fail(LITHOS_EINVAL, "gemm: NORM_* set but gamma (in[4]) or the column sums (in[5]) are null");
            if ((op.flags & LITHOS_F_NORM_LN) && op.dim[7] < (glu ? 2 * N : N)) return fail(LITHOS_EINVAL, "gemm: NORM_LN needs the row stride of the column sums (dim[7]) >= the rows of B");
            if (!(op.fparam[0] >= 0.0f)) return fail(LITHOS_EINVAL, "gemm: NORM_* needs eps (fparam0) >= 0");
        }
        if (glu) {
            if (op.flags & (LITHOS_F_BIAS | LITHOS_F_GELU | LITHOS_F_RESIDUAL | LITHOS_F_OUT_SPLIT)) return fail(LITHOS_EINVAL, "gemm: GLU takes no BIAS, GELU, RESIDUAL or OUT_SPLIT");
            if (2 * N * ldb * 2 >= (1ll << 32)) return fail(LITHOS_EINVAL, "gemm: the skinny kernel addresses weight rows with 32-bit byte offsets (2N*ldb*2 < 4 GiB with GLU)");
        }
        plan->grid = {(uint32_t)(glu ? (N + 15) / 16 : (N + 16 * SKINNY_NB - 1) / (16 * SKINNY_NB)), 1, 1};
    } else {
        if (fused) return fail(LITHOS_EINVAL, "gemm: NORM_LN, NORM_RMS and GLU are built into the weight-streaming kernel only (TRANS_B, M <= 16)");
        if (split && tile == 256) return fail(LITHOS_EINVAL, "gemm: SPLIT_A is built for the 64 and 128 tiles only");
        variant = tile == 64 ? V_TILE64 : tile == 256 ? V_TILE256 : tile == TILE_32X64 ? V_THIN : V_MID192;     // 128: below
        const bool pieces = staged_epilogue(op) && N % 8 == 0;      // every row of C leaves in 16-byte pieces
        // Four wavefronts gain 15 % in the loop and lose in an epilogue, 5 us a tile with bias and residual and 13 with GELU (us, four /
        // eight wavefronts: 2048 x 2048 x 512 with bias 24 / 18, with residual too 36 / 25, with GELU too 47 / 31; 4096 x 4096 x 1024 with
        // bias and residual 55 / 44; with all three 4096 x 8192 x 4096 284 / 265, 256 x 256 x 8192 167 / 165).
        // Whole bf16 tiles of a short K, too: four wavefronts take 1.3 us longer in prologue and stores (1024 x 1024 x 64 8.2 / 6.9, x 256
        // 11.2 / 10.3, x 512 15.1 / 15.0).  Tiles that reach beyond the matrix leave element by element from eight (1000 x 1000 x 64
        // fp32 10.4 / 35), and more than a tile per CU of the chip hide more of it (8192 x 8192 x 256 TN 50 / 56, 8192 x 4096 x 128 NN on
        // 64 CUs 68 / 58).
        const bool short_whole = K <= ((M / 256) * (N / 256) < 256 ? 384 : 192) && M % 256 == 0 && N % 256 == 0 && !(op.flags & LITHOS_F_OUT_F32);
        if (tile == 256 && K % 64 == 0)
            variant = long_rows || !pieces || short_whole || (op.flags & (LITHOS_F_BIAS | LITHOS_F_GELU | LITHOS_F_RESIDUAL)) ? V_LDS256W8 : V_LDS256;
        if (tile == 128) {
            // V_MID128's k-tiles are 32 deep: 64 bytes, half a line, of a row of a k-contiguous operand.  With several workgroups on a CU
            // the line has left the L1 when its other half is fetched, a k-tile later.  V_MID128_PAIR fetches both halves in one turn,
            // which costs 0.3 us and pays from 512 of K on, where rows do not begin on lines (a half then touches two) from 256 (us,
            // single / in pairs: 1024 x 1024 x 256 NT on 64 CUs 5.4 / 5.7, 2048 x 2048 x 1544 on 256 24.0 / 21.2, x 2040 on 192 48 / 41).
            // V_TILE128's are 64 deep and touch half the lines per load: better for two such operands with more than a tile per CU and
            // a long K (in pairs / 64 deep: 3000 x 2048 x 1544 on 192 CUs 35.3 / 32.0, 8192 x 512 x 5000 on 64 194 / 165, but
            // 2048 x 2048 x 1544 on 256 21.2 / 27.3, 512 x 1024 x 4096 on 64 28 / 45).
            const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
            const bool nt = !ta && tb;
            const bool pair = !split && (!ta || tb) && K > (lines ? 512 : 256);
            const bool deep = !split && nt && (K > 2048 ? tiles > 64 : !lines && K > 1280 && tiles > 256);
            variant = long_rows || deep ? V_TILE128 : pair ? V_MID128_PAIR : V_MID128;
        }
        const int64_t bm = tile == TILE_64X192 ? 64 : tile == TILE_32X64 ? 32 : tile, bn = tile == TILE_64X192 ? 192 : tile == TILE_32X64 ? 64 : tile;
        plan->grid = {(uint32_t)((N + bn - 1) / bn), (uint32_t)((M + bm - 1) / bm), (uint32_t)(slices > 1 ? slices : 1)};
        // The 64 tile splits K between two groups of wavefronts while all blocks of the whole grid (never of an atom: the
        // sums must not depend on the cut) find room at two per CU of the whole chip: then the chain of k-tiles is the
        // time (us, two groups / one: 1024 x 1024 x 8192 NN 47 / 65, split 128 x 768 x 3072 19 / 22).  More blocks hide it,
        // and the second group only waits in the prologue and epilogue (8192 x 1024 x 512 NT 25 / 21, 4096 x 4096 x 64
        // 29 / 17, 4096^3 NN 240 / 211, split 4096 x 768 x 3072 59 / 52), up to chains so long that more blocks in
        // flight cost more in L2 than they hide (8192^3 TN 1661 / 2204, NN 1711 / 1708).  Such a grid cut into atoms far
        // smaller than what the chip holds would still run faster with two groups (2048^3 in atoms of 64 blocks 183 / 234,
        // of 512 36 / 41); atoms are whole waves of resident workgroups.
        const uint64_t blocks = (uint64_t)plan->grid.x * plan->grid.y * plan->grid.z;
        if (tile == 64 && (blocks <= 512 || (!split && K / plan->grid.z > 4096))) variant = V_TILE64_2K;
    }
    plan->total = plan->grid.x * plan->grid.y * plan->grid.z;
    plan->threads = tile_threads(variant);
    plan->variant = variant;
    plan->wg_per_cu = cached_occupancy((const void*)variant_fn(variant, ta, tb, a32, split, staged_epilogue(op), norm), tile_threads(variant), 1);
    return LITHOS_OK;
}

int gemm_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s)
{
    GemmArgs g;
    g.A = (const uint16_t*)op.in[0];
    g.B = (const uint16_t*)op.in[1];
    g.C = op.out[0];
    g.bias = (const float*)op.in[2];
    g.resid = (const float*)op.in[3];
    g.M = (int)op.dim[0]; g.N = (int)op.dim[1]; g.K = (int)op.dim[2];
    g.lda = op.ld[0]; g.ldb = op.ld[1]; g.ldc = op.ld[2]; g.ldr = op.ld[3];
    g.flags = op.flags;
    g.tiles_m = plan.grid.y; g.tiles_n = plan.grid.x;
    g.a_plane = op.dim[3]; g.c_plane = op.dim[4];
    g.k_slices = (int)op.dim[5]; g.c_slice = op.dim[6];
    g.gamma = (const float*)op.in[4]; g.colsum = (const float*)op.in[5]; g.ldcs = op.dim[7]; g.eps = op.fparam[0];
    g.wide = staged_epilogue(op);
    gemm_fn fn = variant_fn(plan.variant, op.flags & LITHOS_F_TRANS_A, op.flags & LITHOS_F_TRANS_B, op.flags & LITHOS_F_IN_F32,
                            op.flags & LITHOS_F_SPLIT_A, staged_epilogue(op), norm_of(op.flags));
    LITHOS_HIP(launch_kernel(fn, dim3(LITHOS_ATOM_LAUNCH_BLOCKS(atom)), dim3(plan.threads), s, g, atom));
    return LITHOS_OK;
}

} // namespace lithos
