// Atom-aware row and elementwise kernels for gfx950: bias+activation,
// LayerNorm, RMSNorm, softmax, SiLU-gate, rotary embedding + cache append,
// and a fixed-duration spin kernel for scheduler tests.
//
// All are HBM-bound (a few flops per byte): the design rule is coalesced
// access and wavefront reductions, fp32 arithmetic on bf16 or fp32 data.
// Each workgroup handles the rows / elements named by its LOGICAL block index
// (LithOS Section 4.4), so any sub-range of blocks is a valid atom.
#include "common.hpp"
#include <math.h>

namespace lithos {

struct RowArgs {
    const void* x;
    const float* p0;     // bias / gamma / weight
    const float* p1;     // beta
    void* y;
    void* y2;            // optional bf16 copy
    int64_t rows, cols;
    float f0;            // eps / scale / theta
    uint32_t flags;
    int64_t aux[5];
};

template <bool F32>
__device__ __forceinline__ float load_elem(const void* p, int64_t i)
{
    if constexpr (F32) return reinterpret_cast<const float*>(p)[i];
    else return bf16_to_f32(reinterpret_cast<const uint16_t*>(p)[i]);
}

template <bool F32>
__device__ __forceinline__ void store_elem(void* p, int64_t i, float v)
{
    if constexpr (F32) reinterpret_cast<float*>(p)[i] = v;
    else reinterpret_cast<uint16_t*>(p)[i] = f32_to_bf16(v);
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

// Sum over the TPR threads that share a row (TPR = 64: one wavefront;
// TPR = 256: the whole workgroup through LDS).  Fixed order: deterministic.
template <int TPR>
__device__ __forceinline__ float row_sum(float v, float* red)
{
    v = wave_sum(v);
    if constexpr (TPR == 256) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        v = red[0] + red[1] + red[2] + red[3];
    }
    return v;
}

template <int TPR>
__device__ __forceinline__ float row_max(float v, float* red)
{
    v = wave_max(v);
    if constexpr (TPR == 256) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        v = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    }
    return v;
}

// W consecutive elements of a row or of a flat tensor, 16 bytes (or as close as W comes) at a time
template <bool F32, int W>
__device__ __forceinline__ void load_run(const void* p, int64_t i, float (&v)[W])
{
    if constexpr (W == 1) {
        v[0] = load_elem<F32>(p, i);
    } else if constexpr (F32) {
#pragma unroll
        for (int q = 0; q < W / 4; ++q) {
            const float4 f = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + i)[q];
            v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
        }
    } else {
        const uint16_t* h = reinterpret_cast<const uint16_t*>(p) + i;
        uint32_t u[W / 2];
        if constexpr (W == 8) { const uint4 t = *reinterpret_cast<const uint4*>(h); u[0] = t.x; u[1] = t.y; u[2] = t.z; u[3] = t.w; }
        else { const uint2 t = *reinterpret_cast<const uint2*>(h); u[0] = t.x; u[1] = t.y; }
#pragma unroll
        for (int q = 0; q < W / 2; ++q) { v[2 * q] = __uint_as_float(u[q] << 16); v[2 * q + 1] = __uint_as_float(u[q] & 0xffff0000u); }
    }
}

template <bool F32, int W>
__device__ __forceinline__ void store_run(void* p, int64_t i, const float (&v)[W])
{
    if constexpr (W == 1) {
        store_elem<F32>(p, i, v[0]);
    } else if constexpr (F32) {
#pragma unroll
        for (int q = 0; q < W / 4; ++q)
            reinterpret_cast<float4*>(reinterpret_cast<float*>(p) + i)[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
        uint32_t u[W / 2];
#pragma unroll
        for (int q = 0; q < W / 2; ++q) u[q] = pack_bf16(v[2 * q], v[2 * q + 1]);
        uint16_t* h = reinterpret_cast<uint16_t*>(p) + i;
        if constexpr (W == 8) *reinterpret_cast<uint4*>(h) = make_uint4(u[0], u[1], u[2], u[3]);
        else *reinterpret_cast<uint2*>(h) = make_uint2(u[0], u[1]);
    }
}

// the elements' bf16 rounding, and what it dropped (the second plane of a split-bf16 tensor)
template <int W>
__device__ __forceinline__ void drop_rounded(float (&v)[W])
{
#pragma unroll
    for (int e = 0; e < W; ++e) v[e] -= bf16_to_f32(f32_to_bf16(v[e]));
}

// ---- y = act(x + bias): 2048 consecutive elements per block ---------------
// W = 8: a thread owns eight consecutive elements of one row (cols % 8 == 0, aligned operands): 16-byte
// accesses, one column index per thread.  W = 1: any sizes; a thread's elements are 256 apart and its column
// index is stepped, not divided for.  All loads of x come first and unconditionally (beyond the tensor: its last elements,
// which nobody stores): the compiler waits for a conditional load where it is issued.  Bound by HBM once neither a
// 64-bit remainder per element nor erff is in the way: 16384 x 1024 bf16 13.8 us without and 20.0 with GELU (33 and 38.7),
// 16384 x 1023 18.0 and 25 (33 and 38; 25 and 31 with conditional loads), fp32 without GELU 26.4 (27.1; 28.0).
template <bool IN32, bool OUT32, int W>
__global__ __launch_bounds__(256) void bias_act_kernel(RowArgs a, AtomArgs atom)
{
    const uint32_t L = atom_logical_block(atom);
    const int64_t total = a.rows * a.cols;
    const int64_t base = (int64_t)L * 2048 + threadIdx.x * W;
    const uint32_t cols = (uint32_t)a.cols;
    uint32_t c = total >> 32 ? (uint32_t)(base % a.cols) : (uint32_t)base % cols;
    const uint32_t step = (256 * W) % cols;
    float v[8 / W][W];
#pragma unroll
    for (int i = 0; i < 8 / W; ++i)
        load_run<IN32>(a.x, min(base + i * 256 * W, total - W), v[i]);
#pragma unroll
    for (int i = 0; i < 8 / W; ++i) {
        const int64_t idx = base + i * 256 * W;
        if (idx >= total) break;
        if (a.flags & LITHOS_F_BIAS) {
            float b[W];
            load_run<true>(a.p0, c, b);
#pragma unroll
            for (int e = 0; e < W; ++e) v[i][e] += b[e];
        }
        if (a.flags & LITHOS_F_GELU)
#pragma unroll
            for (int e = 0; e < W; ++e) v[i][e] = gelu_erf<true>(v[i][e]);
        store_run<OUT32>(a.y, idx, v[i]);
        if (!OUT32 && (a.flags & LITHOS_F_OUT_SPLIT)) {      // lo plane follows the hi plane
            drop_rounded(v[i]);
            store_run<false>(a.y, total + idx, v[i]);
        }
        c += step;
        if (c >= cols) c -= cols;
    }
}

// ---- y = act(sum_z plane_z + bias) + residual: 2048 consecutive elements per block ----
// The planes are the fp32 partial products of a K-sliced GEMM; they are added in
// slice order, starting from plane 0, so the sum is the same for every launch shape.
// VEC: four elements per thread and step (cols, strides and pointers permit 16-byte access).
template <bool OUT32, bool VEC>
__global__ __launch_bounds__(256) void sum_slices_kernel(RowArgs a, AtomArgs atom)
{
    const uint32_t L = atom_logical_block(atom);
    const int64_t total = a.rows * a.cols;
    const int64_t base = (int64_t)L * 2048;
    const float* planes = reinterpret_cast<const float*>(a.x);
    const int64_t S = a.aux[0], plane = a.aux[1], ldx = a.aux[2], ldy = a.aux[3];
    const int64_t ldr = a.aux[4];
    constexpr int W = VEC ? 4 : 1;
#pragma unroll
    for (int i = 0; i < 8 / W; ++i) {
        const int64_t idx = base + ((int64_t)threadIdx.x + i * 256) * W;
        if (idx >= total) continue;
        const int64_t r = idx / a.cols, c = idx % a.cols;
        float v[W];
        if constexpr (VEC) {
            float4 s = *reinterpret_cast<const float4*>(planes + r * ldx + c);
            for (int64_t z = 1; z < S; ++z) {
                const float4 t = *reinterpret_cast<const float4*>(planes + z * plane + r * ldx + c);
                s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
            }
            v[0] = s.x; v[1] = s.y; v[2] = s.z; v[3] = s.w;
        } else {
            float s = planes[r * ldx + c];
            for (int64_t z = 1; z < S; ++z) s += planes[z * plane + r * ldx + c];
            v[0] = s;
        }
#pragma unroll
        for (int t = 0; t < W; ++t) {
            if (a.flags & LITHOS_F_BIAS) v[t] += a.p0[c + t];
            if (a.flags & LITHOS_F_GELU) v[t] = gelu_erf(v[t]);
            if (a.flags & LITHOS_F_RESIDUAL) v[t] += a.p1[r * ldr + c + t];
        }
        if constexpr (VEC && OUT32) {
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.y) + r * ldy + c) = make_float4(v[0], v[1], v[2], v[3]);
        } else if constexpr (VEC) {
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.y) + r * ldy + c) =
                make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        } else {
            store_elem<OUT32>(a.y, r * ldy + c, v[0]);
        }
    }
}

// ---- y[r, :F] = silu(gu[r, :F]) * gu[r, F:2F] ------------------------------
template <bool IN32, bool OUT32>
__global__ __launch_bounds__(256) void silu_mul_kernel(RowArgs a, AtomArgs atom)
{
    const uint32_t L = atom_logical_block(atom);
    const int64_t F = a.cols, total = a.rows * F;
    const int64_t base = (int64_t)L * 2048;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        int64_t idx = base + threadIdx.x + i * 256;
        if (idx < total) {
            int64_t r = idx / F, c = idx % F;
            float g = load_elem<IN32>(a.x, r * 2 * F + c);
            float u = load_elem<IN32>(a.x, r * 2 * F + F + c);
            float v = g / (1.0f + expf(-g)) * u;
            store_elem<OUT32>(a.y, idx, v);
        }
    }
}

// ---- LayerNorm: two passes over the row (mean, then centred variance) ------
template <bool IN32, bool OUT32, int TPR>
__global__ __launch_bounds__(256) void layernorm_kernel(RowArgs a, AtomArgs atom)
{
    __shared__ float red[4];
    const uint32_t L = atom_logical_block(atom);
    constexpr int RPB = 256 / TPR;
    const int64_t row = (int64_t)L * RPB + threadIdx.x / TPR;
    const int t = threadIdx.x % TPR;
    const bool live = row < a.rows;
    const int64_t H = a.cols, off = row * H;
    float s = 0.0f;
    if (live) for (int64_t c = t; c < H; c += TPR) s += load_elem<IN32>(a.x, off + c);
    const float mean = row_sum<TPR>(s, red) / (float)H;
    float q = 0.0f;
    if (live) for (int64_t c = t; c < H; c += TPR) { float d = load_elem<IN32>(a.x, off + c) - mean; q += d * d; }
    const float var = row_sum<TPR>(q, red) / (float)H;
    const float rstd = 1.0f / sqrtf(var + a.f0);
    if (live) for (int64_t c = t; c < H; c += TPR) {
        float v = (load_elem<IN32>(a.x, off + c) - mean) * rstd * a.p0[c] + a.p1[c];
        store_elem<OUT32>(a.y, off + c, v);
        if (OUT32 && a.y2) {
            uint16_t hi = f32_to_bf16(v);
            reinterpret_cast<uint16_t*>(a.y2)[off + c] = hi;
            if (a.flags & LITHOS_F_OUT_SPLIT)
                reinterpret_cast<uint16_t*>(a.y2)[a.rows * H + off + c] = f32_to_bf16(v - bf16_to_f32(hi));
        }
    }
}

// Register-resident variant: the row is read ONCE and stays in registers (16 elements per thread) for the
// mean, the centred variance and the output; needs H <= 16 * TPR and rows that 16-byte accesses fit: a thread holds
// 16 / W runs of W = 4 (fp32) or 8 (bf16) consecutive elements.  Bound by HBM on many rows (16384 x 1024 bf16: 16.3 us
// by events = 4.1 TB/s, 14.0 in a kernel trace), by launch and latency on few.  Other rows take the general kernel above: with single elements this form
// has 16 conditional loads of x, gamma and beta each in a row, and the compiler waits for every one where it is issued
// (16384 x 1025 bf16: 151 us against 46, 16384 x 127: 25 against 10).
template <bool IN32, bool OUT32, int TPR, int W>
__global__ __launch_bounds__(256) void layernorm_vec_kernel(RowArgs a, AtomArgs atom)
{
    __shared__ float red[4];
    constexpr int NV = 16 / W;
    const uint32_t L = atom_logical_block(atom);
    constexpr int RPB = 256 / TPR;
    const int64_t row = (int64_t)L * RPB + threadIdx.x / TPR;
    const int t = threadIdx.x % TPR;
    const bool live = row < a.rows;
    const int H = (int)a.cols;
    const int64_t off = row * H;
    float v[NV][W];
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = W * (t + j * TPR);
#pragma unroll
        for (int e = 0; e < W; ++e) v[j][e] = 0.0f;
        if (live && c < H) load_run<IN32>(a.x, off + c, v[j]);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int e = 0; e < W; ++e) s += v[j][e];
    const float mean = row_sum<TPR>(s, red) / (float)H;
    float q = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j)
        if (live && W * (t + j * TPR) < H)
#pragma unroll
            for (int e = 0; e < W; ++e) { const float d = v[j][e] - mean; q += d * d; }
    const float var = row_sum<TPR>(q, red) / (float)H;
    const float rstd = 1.0f / sqrtf(var + a.f0);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = W * (t + j * TPR);
        if (!live || c >= H) continue;
        float gm[W], bt[W];
        load_run<true>(a.p0, c, gm);
        load_run<true>(a.p1, c, bt);
#pragma unroll
        for (int e = 0; e < W; ++e) v[j][e] = (v[j][e] - mean) * rstd * gm[e] + bt[e];
        store_run<OUT32>(a.y, off + c, v[j]);
        if (OUT32 && a.y2) {
            store_run<false>(a.y2, off + c, v[j]);
            if (a.flags & LITHOS_F_OUT_SPLIT) {
                drop_rounded(v[j]);
                store_run<false>(a.y2, a.rows * H + off + c, v[j]);
            }
        }
    }
}

// ---- RMSNorm ----------------------------------------------------------------
template <bool IN32, bool OUT32, int TPR>
__global__ __launch_bounds__(256) void rmsnorm_kernel(RowArgs a, AtomArgs atom)
{
    __shared__ float red[4];
    const uint32_t L = atom_logical_block(atom);
    constexpr int RPB = 256 / TPR;
    const int64_t row = (int64_t)L * RPB + threadIdx.x / TPR;
    const int t = threadIdx.x % TPR;
    const bool live = row < a.rows;
    const int64_t H = a.cols, off = row * H;
    float s = 0.0f;
    if (live) for (int64_t c = t; c < H; c += TPR) { float v = load_elem<IN32>(a.x, off + c); s += v * v; }
    const float ms = row_sum<TPR>(s, red) / (float)H;
    const float rinv = 1.0f / sqrtf(ms + a.f0);
    if (live) for (int64_t c = t; c < H; c += TPR)
        store_elem<OUT32>(a.y, off + c, load_elem<IN32>(a.x, off + c) * rinv * a.p0[c]);
}

// Register-resident variant (H % 4 == 0, H <= 16 * TPR): the row is read once with
// 16-byte (fp32) or 8-byte (bf16) loads that are all in flight together.
template <bool IN32, bool OUT32, int TPR>
__global__ __launch_bounds__(256) void rmsnorm_vec_kernel(RowArgs a, AtomArgs atom)
{
    __shared__ float red[4];
    constexpr int NV = 4;
    const uint32_t L = atom_logical_block(atom);
    constexpr int RPB = 256 / TPR;
    const int64_t row = (int64_t)L * RPB + threadIdx.x / TPR;
    const int t = threadIdx.x % TPR;
    const bool live = row < a.rows;
    const int64_t H = a.cols, off = row * H;
    float v[NV][4];
    float4 w[NV];
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int64_t c = 4 * (t + (int64_t)j * TPR);
        v[j][0] = v[j][1] = v[j][2] = v[j][3] = 0.0f;
        w[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live && c < H) {
            if constexpr (IN32) {
                const float4 f = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.x) + off + c);
                v[j][0] = f.x; v[j][1] = f.y; v[j][2] = f.z; v[j][3] = f.w;
            } else {
                const uint2 u = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(a.x) + off + c);
                v[j][0] = __uint_as_float(u.x << 16); v[j][1] = __uint_as_float(u.x & 0xffff0000u);
                v[j][2] = __uint_as_float(u.y << 16); v[j][3] = __uint_as_float(u.y & 0xffff0000u);
            }
            w[j] = *reinterpret_cast<const float4*>(a.p0 + c);
        }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) s += v[j][e] * v[j][e];
    const float ms = row_sum<TPR>(s, red) / (float)H;
    const float rinv = 1.0f / sqrtf(ms + a.f0);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int64_t c = 4 * (t + (int64_t)j * TPR);
        if (live && c < H) {
            const float y[4] = {v[j][0] * rinv * w[j].x, v[j][1] * rinv * w[j].y, v[j][2] * rinv * w[j].z, v[j][3] * rinv * w[j].w};
            if constexpr (OUT32) {
                *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.y) + off + c) = make_float4(y[0], y[1], y[2], y[3]);
            } else {
                *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.y) + off + c) = make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
            }
        }
    }
}

// ---- softmax(scale * s) -----------------------------------------------------
// e^x for x <= 0 (NaN stays NaN) as 2^n 2^a: n is x log2 e rounded (by adding 1.5 * 2^23), the remainder a lies within
// half a unit and is exact but for its last two roundings (log2 e in two floats), so the error is that of the hardware's
// 2^a and a little more: worst 8.4e-8, mean 2.2e-8 relative on 524 288 points in [-87, -30], as expf.  One scaling by 2^n,
// which rounds a subnormal result once.  Below -150, where e^x is zero, the argument is clamped, by the maximum that
// keeps NaN.
__device__ __forceinline__ float exp_nonpositive(float x)
{
    x = __builtin_elementwise_maximum(x, -150.0f);
    const float t = fmaf(x, 1.44269502162933349609f, 12582912.0f), n = t - 12582912.0f;
    const float a = fmaf(x, 1.92596299112661746887e-8f, fmaf(x, 1.44269502162933349609f, -n));
    return ldexpf(__builtin_amdgcn_exp2f(a), __float_as_int(t) - 0x4b400000);
}

// Register-resident rows (n <= 16 * TPR), as in layernorm_vec_kernel: one read of the row and one exponential
// per element, where the general kernel below reads the row three times and takes the exponential twice.
// 16384 x 1024 bf16: 18.0 us (17.7 with half of the scores masked) against 41; 20 with expf and a division per element,
// which bound this form; 8192 x 4096: 29 us against 75.
template <bool IN32, bool OUT32, int TPR, int W>
__global__ __launch_bounds__(256) void softmax_vec_kernel(RowArgs a, AtomArgs atom)
{
    __shared__ float red[4];
    constexpr int NV = 16 / W;
    const uint32_t L = atom_logical_block(atom);
    constexpr int RPB = 256 / TPR;
    const int64_t row = (int64_t)L * RPB + threadIdx.x / TPR;
    const int t = threadIdx.x % TPR;
    const bool live = row < a.rows;
    const int n = (int)a.cols;
    const int64_t off = row * n;
    float v[NV][W];
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = W * (t + j * TPR);
#pragma unroll
        for (int e = 0; e < W; ++e) v[j][e] = 0.0f;
        if (live && c < n) load_run<IN32>(a.x, off + c, v[j]);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int e = 0; e < W; ++e) {
            v[j][e] = live && W * (t + j * TPR) < n ? v[j][e] * a.f0 : -INFINITY;
            mx = fmaxf(mx, v[j][e]);
        }
    mx = row_max<TPR>(mx, red);
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j)
        if (live && W * (t + j * TPR) < n)
#pragma unroll
            for (int e = 0; e < W; ++e) { v[j][e] = exp_nonpositive(v[j][e] - mx); s += v[j][e]; }
    const float den = row_sum<TPR>(s, red);
    const float inv = 1.0f / den;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = W * (t + j * TPR);
        if (!live || c >= n) continue;
#pragma unroll
        for (int e = 0; e < W; ++e) {               // v / den: the quotient by the reciprocal, then one Newton correction
            const float q = v[j][e] * inv;
            v[j][e] = fmaf(fmaf(-q, den, v[j][e]), inv, q);
        }
        store_run<OUT32>(a.y, off + c, v[j]);
    }
}

// rows longer than 16 * TPR
template <bool IN32, bool OUT32, int TPR>
__global__ __launch_bounds__(256) void softmax_kernel(RowArgs a, AtomArgs atom)
{
    __shared__ float red[4];
    const uint32_t L = atom_logical_block(atom);
    constexpr int RPB = 256 / TPR;
    const int64_t row = (int64_t)L * RPB + threadIdx.x / TPR;
    const int t = threadIdx.x % TPR;
    const bool live = row < a.rows;
    const int64_t n = a.cols, off = row * n;
    float mx = -INFINITY;
    if (live) for (int64_t c = t; c < n; c += TPR) mx = fmaxf(mx, load_elem<IN32>(a.x, off + c) * a.f0);
    mx = row_max<TPR>(mx, red);
    float s = 0.0f;
    if (live) for (int64_t c = t; c < n; c += TPR) s += expf(load_elem<IN32>(a.x, off + c) * a.f0 - mx);
    const float den = row_sum<TPR>(s, red);
    if (live) for (int64_t c = t; c < n; c += TPR)
        store_elem<OUT32>(a.y, off + c, expf(load_elem<IN32>(a.x, off + c) * a.f0 - mx) / den);
}

// ---- rotary embedding of q and k heads in place + k,v appended to the cache --
// One wavefront per (row, head slot); slots 0..n_q-1 are query heads,
// n_q..n_q+n_kv-1 key heads, the rest value heads (copied to the cache only).
// aux = {n_q, n_kv, pos, cap}; cols = d.
template <bool F32>
__global__ __launch_bounds__(256) void rope_kv_kernel(RowArgs a, AtomArgs atom)
{
    const uint32_t L = atom_logical_block(atom);
    const int64_t n_q = a.aux[0], n_kv = a.aux[1], pos = a.aux[2], cap = a.aux[3], d = a.cols;
    const int64_t slots = n_q + 2 * n_kv;
    const int64_t unit = (int64_t)L * 4 + (threadIdx.x >> 6);
    if (unit >= a.rows * slots) return;
    const int lane = threadIdx.x & 63;
    const int64_t row = unit / slots, slot = unit % slots;
    void* head = const_cast<void*>(a.x);
    const int64_t hoff = row * slots * d + slot * d;
    uint16_t* kc = reinterpret_cast<uint16_t*>(a.y);
    uint16_t* vc = reinterpret_cast<uint16_t*>(a.y2);
    const int64_t half = d / 2;
    if (slot < n_q + n_kv) {
        uint16_t* dst = nullptr;
        if (slot >= n_q) dst = kc + ((row * cap + pos) * n_kv + (slot - n_q)) * d;
        for (int64_t e = lane; e < half; e += 64) {
            float inv = powf(a.f0, -2.0f * (float)e / (float)d);
            float sn, cs;
            sincosf((float)pos * inv, &sn, &cs);
            float x0 = load_elem<F32>(head, hoff + e), x1 = load_elem<F32>(head, hoff + e + half);
            float r0 = x0 * cs - x1 * sn, r1 = x1 * cs + x0 * sn;
            store_elem<F32>(head, hoff + e, r0);
            store_elem<F32>(head, hoff + e + half, r1);
            if (dst) { dst[e] = f32_to_bf16(r0); dst[e + half] = f32_to_bf16(r1); }
        }
    } else {
        uint16_t* dst = vc + ((row * cap + pos) * n_kv + (slot - n_q - n_kv)) * d;
        for (int64_t e = lane; e < d; e += 64) dst[e] = f32_to_bf16(load_elem<F32>(head, hoff + e));
    }
}

// ---- spin: every block waits `ticks` of the constant 100 MHz counter -------
// 1024 threads and 64 KB of LDS per block: exactly two blocks fit on a CU, so
// the kernel's latency is ticks * ceil(blocks / (2 * CUs)) - a known scaling
// curve for scheduler and right-sizing tests.
__global__ __launch_bounds__(1024) void spin_kernel(uint64_t ticks, AtomArgs atom)
{
    __shared__ uint32_t pad[16384];
    const uint32_t L = atom_logical_block(atom);
    if (threadIdx.x == 0) reinterpret_cast<volatile uint32_t*>(pad)[L & 16383] = L;
    const uint64_t t0 = wall_clock64();
    while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(8);
}

// ---- host side ----------------------------------------------------------------

static RowArgs make_args(const lithos_op_t& op)
{
    RowArgs a{};
    a.x = op.in[0];
    a.p0 = (const float*)op.in[1];
    a.p1 = (const float*)op.in[2];
    a.y = op.out[0];
    a.y2 = op.out[1];
    a.rows = op.dim[0];
    a.cols = op.dim[1];
    a.f0 = op.fparam[0];
    a.flags = op.flags;
    return a;
}

static int tpr_for(int64_t cols) { return cols <= 1024 ? 64 : 256; }

// Variants of the row kernels: rows of any length read several times; register-resident rows (at most
// 16 * TPR elements) with runs of 1, or of 4 (fp32) / 8 (bf16 in and out) consecutive elements per access.
enum { RV_ANY = 0, RV_VEC4 = 1, RV_WIDE = 2, RV_SCALAR = 3 };

// Longest row of the register-resident kernels: 16 elements per thread of 64 or 256 threads per row.
static int row_variant(const lithos_op_t& op, bool aligned)
{
    const int64_t cols = op.dim[1];
    if (cols > 16 * tpr_for(cols)) return RV_ANY;
    if (!aligned || cols % 4) return RV_SCALAR;
    return cols % 8 == 0 && !(op.flags & (LITHOS_F_IN_F32 | LITHOS_F_OUT_F32)) ? RV_WIDE : RV_VEC4;
}

// The kernel that serves a descriptor (everything but SPIN, whose kernel has its own signature).
typedef void (*row_fn)(RowArgs, AtomArgs);
#define PICK2(K) (in32 ? (out32 ? (row_fn)K<true, true> : (row_fn)K<true, false>) : (out32 ? (row_fn)K<false, true> : (row_fn)K<false, false>))
#define PICK2W(K, W) (in32 ? (out32 ? (row_fn)K<true, true, W> : (row_fn)K<true, false, W>) : (out32 ? (row_fn)K<false, true, W> : (row_fn)K<false, false, W>))
#define PICK3(K, T) (in32 ? (out32 ? (row_fn)K<true, true, T> : (row_fn)K<true, false, T>) : (out32 ? (row_fn)K<false, true, T> : (row_fn)K<false, false, T>))
#define PICK3W(K, T, W) (in32 ? (out32 ? (row_fn)K<true, true, T, W> : (row_fn)K<true, false, T, W>) : (out32 ? (row_fn)K<false, true, T, W> : (row_fn)K<false, false, T, W>))
#define PICKROW(K)                                                                                                    \
    (variant == RV_WIDE ? (wide ? (row_fn)K<false, false, 256, 8> : (row_fn)K<false, false, 64, 8>)                   \
                        : (wide ? PICK3W(K, 256, 4) : PICK3W(K, 64, 4)))
static row_fn row_kernel(const lithos_op_t& op, int variant)
{
    const bool in32 = op.flags & LITHOS_F_IN_F32, out32 = op.flags & LITHOS_F_OUT_F32;
    const bool wide = tpr_for(op.dim[1]) == 256;
    switch (op.kind) {
    case LITHOS_OP_BIAS_ACT: return variant == RV_WIDE ? PICK2W(bias_act_kernel, 8) : PICK2W(bias_act_kernel, 1);
    case LITHOS_OP_SILU_MUL: return PICK2(silu_mul_kernel);
    case LITHOS_OP_SUM_SLICES:
        return variant == 1 ? (out32 ? (row_fn)sum_slices_kernel<true, true> : (row_fn)sum_slices_kernel<false, true>)
                            : (out32 ? (row_fn)sum_slices_kernel<true, false> : (row_fn)sum_slices_kernel<false, false>);
    case LITHOS_OP_LAYERNORM:
        if (variant) return PICKROW(layernorm_vec_kernel);
        return wide ? PICK3(layernorm_kernel, 256) : PICK3(layernorm_kernel, 64);
    case LITHOS_OP_RMSNORM:
        if (variant == 1) return wide ? PICK3(rmsnorm_vec_kernel, 256) : PICK3(rmsnorm_vec_kernel, 64);
        return wide ? PICK3(rmsnorm_kernel, 256) : PICK3(rmsnorm_kernel, 64);
    case LITHOS_OP_SOFTMAX:
        if (variant == RV_SCALAR) return wide ? PICK3W(softmax_vec_kernel, 256, 1) : PICK3W(softmax_vec_kernel, 64, 1);
        if (variant) return PICKROW(softmax_vec_kernel);
        return wide ? PICK3(softmax_kernel, 256) : PICK3(softmax_kernel, 64);
    case LITHOS_OP_ROPE_KV: return in32 ? (row_fn)rope_kv_kernel<true> : (row_fn)rope_kv_kernel<false>;
    default: return nullptr;
    }
}
#undef PICK2
#undef PICK2W
#undef PICK3
#undef PICK3W
#undef PICKROW

int rowops_plan(const lithos_op_t& op, OpPlan* plan)
{
    const int64_t rows = op.dim[0], cols = op.dim[1];
    if (rows <= 0 || cols <= 0 || rows > (1ll << 31) || cols > (1ll << 24))
        return fail(LITHOS_EINVAL, "row op %d: rows and cols must be positive (got %lld, %lld)", op.kind, (long long)rows, (long long)cols);
    if (!op.in[0] && op.kind != LITHOS_OP_SPIN) return fail(LITHOS_EINVAL, "row op %d: null input", op.kind);
    plan->threads = 256;
    plan->variant = 0;
    plan->wg_per_cu = 8;
    uint64_t blocks = 0;
    switch (op.kind) {
    case LITHOS_OP_BIAS_ACT:
        if (!op.out[0]) return fail(LITHOS_EINVAL, "bias_act: null output");
        if ((op.flags & LITHOS_F_BIAS) && !op.in[1]) return fail(LITHOS_EINVAL, "bias_act: BIAS set but in[1] is null");
        blocks = ((uint64_t)rows * cols + 2047) / 2048;
        plan->variant = cols % 8 == 0 && aligned16(op.in[0]) && aligned16(op.out[0]) && (!op.in[1] || aligned16(op.in[1])) ? RV_WIDE : RV_SCALAR;
        break;
    case LITHOS_OP_SILU_MUL:
        if (!op.out[0]) return fail(LITHOS_EINVAL, "silu_mul: null output");
        blocks = ((uint64_t)rows * cols + 2047) / 2048;
        break;
    case LITHOS_OP_SUM_SLICES: {
        // dim = rows, cols, slices, slice plane stride; ld = row strides of the planes, of y, of the residual
        const int64_t S = op.dim[2], plane = op.dim[3], ldx = op.ld[0], ldy = op.ld[1], ldr = op.ld[2];
        if (!op.out[0]) return fail(LITHOS_EINVAL, "sum_slices: null output");
        if (S < 1 || S > LITHOS_GEMM_MAX_SLICES) return fail(LITHOS_EINVAL, "sum_slices: slices must be in [1, %d]", LITHOS_GEMM_MAX_SLICES);
        if (ldx < cols || ldy < cols || plane < rows * ldx) return fail(LITHOS_EINVAL, "sum_slices: row or plane stride too small");
        if ((op.flags & LITHOS_F_BIAS) && !op.in[1]) return fail(LITHOS_EINVAL, "sum_slices: BIAS set but in[1] is null");
        if ((op.flags & LITHOS_F_RESIDUAL) && (!op.in[2] || ldr < cols)) return fail(LITHOS_EINVAL, "sum_slices: RESIDUAL needs in[2] and ld[2] >= cols");
        if (op.flags & (LITHOS_F_IN_F32 | LITHOS_F_OUT_SPLIT)) return fail(LITHOS_EINVAL, "sum_slices: the planes are always fp32; no split output");
        blocks = ((uint64_t)rows * cols + 2047) / 2048;
        if (cols % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 && plane % 4 == 0 && aligned16(op.in[0]) && aligned16(op.out[0]) &&
            (!(op.flags & LITHOS_F_RESIDUAL) || ldr % 4 == 0))
            plan->variant = 1;
        break;
    }
    case LITHOS_OP_LAYERNORM:
        if (!op.in[1] || !op.in[2] || !op.out[0]) return fail(LITHOS_EINVAL, "layernorm: null gamma, beta or output");
        if (!(op.flags & LITHOS_F_OUT_F32) && op.out[1]) return fail(LITHOS_EINVAL, "layernorm: a bf16 copy needs OUT_F32");
        blocks = (rows + (256 / tpr_for(cols)) - 1) / (256 / tpr_for(cols));
        plan->variant = row_variant(op, aligned16(op.in[0]) && aligned16(op.in[1]) && aligned16(op.in[2]) && aligned16(op.out[0]) &&
                                            (!op.out[1] || aligned16(op.out[1])));
        if (plan->variant == RV_SCALAR) plan->variant = RV_ANY;     // slower than several passes, see layernorm_vec_kernel
        break;
    case LITHOS_OP_RMSNORM:
        if (!op.in[1] || !op.out[0]) return fail(LITHOS_EINVAL, "rmsnorm: null weight or output");
        blocks = (rows + (256 / tpr_for(cols)) - 1) / (256 / tpr_for(cols));
        if (cols % 4 == 0 && cols <= 16 * tpr_for(cols) && aligned16(op.in[0]) && aligned16(op.in[1]) && aligned16(op.out[0]))
            plan->variant = 1;
        break;
    case LITHOS_OP_SOFTMAX:
        if (!op.out[0]) return fail(LITHOS_EINVAL, "softmax: null output");
        blocks = (rows + (256 / tpr_for(cols)) - 1) / (256 / tpr_for(cols));
        plan->variant = row_variant(op, aligned16(op.in[0]) && aligned16(op.out[0]));
        // Short rows leave most of the 16 elements per thread idle, and the general kernel's further reads hit the cache:
        // 131072 rows of bf16, registers / general: 33 columns 49 / 35 us, 64 46 / 36, 72 46 / 46, 128 46 / 52, 512 49 / 145;
        // in single elements 77 columns 51 / 47, 127 51 / 50, 129 54 / 61.
        if (cols <= (plan->variant == RV_SCALAR ? 128 : 64)) plan->variant = RV_ANY;
        break;
    case LITHOS_OP_ROPE_KV: {
        // dim = rows, n_q, n_kv, d, pos, cap
        const int64_t n_q = op.dim[1], n_kv = op.dim[2], d = op.dim[3], pos = op.dim[4], cap = op.dim[5];
        if (n_q <= 0 || n_kv <= 0 || d <= 0 || (d & 1) || pos < 0 || pos >= cap)
            return fail(LITHOS_EINVAL, "rope_kv: need n_q,n_kv,d > 0, d even, 0 <= pos < cap");
        if (!op.out[0] || !op.out[1]) return fail(LITHOS_EINVAL, "rope_kv: null cache pointer");
        blocks = ((uint64_t)rows * (n_q + 2 * n_kv) + 3) / 4;
        break;
    }
    case LITHOS_OP_SPIN:
        if (op.dim[1] < 0 || op.dim[1] > 100000000) return fail(LITHOS_EINVAL, "spin: ticks must be in [0, 1e8] (1 s)");
        blocks = rows;
        plan->threads = 1024;
        plan->wg_per_cu = 2;
        break;
    default:
        return fail(LITHOS_EINVAL, "unknown row op kind %d", op.kind);
    }
    if (blocks == 0 || blocks > 0x7fffffffull) return fail(LITHOS_EINVAL, "row op %d: grid out of range", op.kind);
    plan->grid = {(uint32_t)blocks, 1, 1};
    plan->total = (uint32_t)blocks;
    // resident workgroups per CU: asked of the runtime once per kernel (it feeds the atom quantum and
    // the occupancy filter of right-sizing); the constants above only serve if the query fails
    const void* fn = op.kind == LITHOS_OP_SPIN ? (const void*)spin_kernel : (const void*)row_kernel(op, plan->variant);
    plan->wg_per_cu = cached_occupancy(fn, (int)plan->threads, plan->wg_per_cu);
    return LITHOS_OK;
}

int rowops_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s)
{
    const dim3 grid(LITHOS_ATOM_LAUNCH_BLOCKS(atom)), block(plan.threads);
    if (op.kind == LITHOS_OP_SPIN) {
        LITHOS_HIP(launch_kernel(spin_kernel, grid, block, s, (uint64_t)op.dim[1], atom));
        return LITHOS_OK;
    }
    RowArgs a = make_args(op);
    if (op.kind == LITHOS_OP_SUM_SLICES) {
        a.aux[0] = op.dim[2]; a.aux[1] = op.dim[3]; a.aux[2] = op.ld[0]; a.aux[3] = op.ld[1];
        a.aux[4] = op.ld[2];
    } else if (op.kind == LITHOS_OP_ROPE_KV) {
        a.cols = op.dim[3];
        a.aux[0] = op.dim[1]; a.aux[1] = op.dim[2]; a.aux[2] = op.dim[4]; a.aux[3] = op.dim[5];
        a.p0 = nullptr; a.p1 = nullptr;
    }
    row_fn fn = row_kernel(op, plan.variant);
    if (!fn) return fail(LITHOS_EINVAL, "unknown row op kind %d", op.kind);
    LITHOS_HIP(launch_kernel(fn, grid, block, s, a, atom));
    return LITHOS_OK;
}

} // namespace lithos
