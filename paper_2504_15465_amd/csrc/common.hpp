// Host-side declarations shared by the library's translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <tuple>
#include <utility>
#include "../../include/lithos.h"
#include "atom_device.hpp"

namespace lithos {

template <typename Tuple, size_t... I>
inline void fill_ptrs(void** ptrs, Tuple& vals, std::index_sequence<I...>)
{
    ((ptrs[I] = (void*)&std::get<I>(vals)), ...);
}

void set_error(const char* fmt, ...);
int  fail(int code, const char* fmt, ...);

#define LITHOS_HIP(call)                                                                  \
    do {                                                                                  \
        hipError_t e_ = (call);                                                           \
        if (e_ != hipSuccess)                                                             \
            return ::lithos::fail(LITHOS_EHIP, "%s: %s (%s:%d)", #call,                   \
                                  hipGetErrorString(e_), __FILE__, __LINE__);             \
    } while (0)

// What an operator needs to be cut in atoms.
struct OpPlan {
    lithos_dim3 grid;       // logical grid
    uint32_t total;         // gx*gy*gz
    uint32_t threads;       // workgroup size
    uint32_t wg_per_cu;     // resident workgroups per CU (occupancy)
    int variant;            // kernel variant chosen by the validator
};

// Each operator family: validate + plan (no launch), and launch one atom.
int gemm_plan(const lithos_op_t& op, OpPlan* plan);
int gemm_square_tile(const lithos_op_t& op);     // of 64 and 128, by the number of tiles
int gemm_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s);
int rowops_plan(const lithos_op_t& op, OpPlan* plan);
int rowops_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s);
int attn_plan(const lithos_op_t& op, OpPlan* plan);
int attn_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s);
int attn_prefill_plan(const lithos_op_t& op, OpPlan* plan);
int attn_prefill_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s);
int spin_plan(const lithos_op_t& op, OpPlan* plan);
int spin_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s);
int probe_launch(uint32_t n_wg, uint32_t* dev_xcd, uint32_t* dev_hwid, hipStream_t s);

int op_plan(const lithos_op_t& op, OpPlan* plan);
int op_launch(const lithos_op_t& op, const OpPlan& plan, const AtomArgs& atom, hipStream_t s);

// hipLaunchKernel with a status code (the <<< >>> form reports errors only
// through the thread's sticky last-error slot, which hipEventQuery also sets).
template <typename... Params, typename... Args>
inline hipError_t launch_kernel(void (*k)(Params...), dim3 grid, dim3 block, hipStream_t s, Args... args)
{
    std::tuple<Params...> vals{static_cast<Params>(args)...};
    void* ptrs[sizeof...(Params)];
    fill_ptrs(ptrs, vals, std::index_sequence_for<Params...>{});
    return hipLaunchKernel(reinterpret_cast<const void*>(k), grid, block, ptrs, 0, s);
}

// hipOccupancyMaxActiveBlocksPerMultiprocessor for a kernel and workgroup size (no dynamic LDS), asked
// once per (device, kernel, size) and remembered; `fallback` if the runtime cannot say.
uint32_t cached_occupancy(const void* kernel, int threads, uint32_t fallback);

// fp32 -> bf16 bits, round to nearest even: one conversion instruction for two values (the integer form of
// the rounding took six for each, which bound the row kernels and the epilogues of short GEMMs).
typedef __bf16 lithos_bf16x2 __attribute__((ext_vector_type(2)));
typedef float lithos_f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const lithos_f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, lithos_bf16x2));
}

__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return (uint16_t)pack_bf16(f, f); }

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ void wave_lds_sync()
{
    // LDS operations of one wavefront complete in order; this only stops the compiler
    // from moving reads of other lanes' data across the writes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// GELU u * Phi(u).  |u| < 1.25: Phi = 1/2 + u P(u^2), 1.2e-8 of Phi(-|u|) at worst.  Beyond: max(u, 0) - |u| Phi(-|u|), where
// |u| Phi(-|u|) = exp(-u^2 / 2) R(t) with t = 1 / (1 + 0.3 |u|), 2.3e-8 relative up to |u| = 14, where the exponential leaves
// the normal numbers.  (Both fitted by iteratively reweighted least squares in float64, the coefficients rounded one after
// the other.)  Neither half serves alone: near 0 the second would subtract a number near u / 2 that carries the roundings
// of the reciprocal, the polynomial and the exponential, and 1 + erff cancels for u < -1.
// Measured on 4M uniform points a range against float64, worst / mean relative error (0.5 u (1 + erff) in brackets):
//   -5 .. -2    1.4e-6 / 2.1e-7  (4.8e-2 / 1.7e-3)     0 .. 0.5    1.2e-7 / 3.2e-8  (1.3e-7 / 3.3e-8)
//   -2 .. -1    3.7e-7 / 7.1e-8  (1.2e-6 / 1.7e-7)     0.5 .. 2    1.1e-7 / 2.4e-8  (1.4e-7 / 3.0e-8)
//   -1 .. -0.5  2.0e-7 / 4.0e-8  (2.7e-7 / 5.6e-8)     2 .. 4      6.5e-8 / 2.0e-8  (1.1e-7 / 2.7e-8)
//   -0.5 .. 0   1.3e-7 / 2.9e-8  (1.5e-7 / 3.1e-8)     4 .. 14     6.0e-8 / 4.3e-9  (1.0e-7 / 5.0e-9)
// and 2.4e-7 absolute at worst, for u in [4, 8) (4.5e-7).  22 instructions and two transcendentals; erff runs both of its
// branches in nearly every wavefront.  BRANCH: the last step under a condition instead of both results and a select, the
// same bits: bias + GELU of 16384 x 1024 bf16 20.0 us against 21.6 (erff: 38.7), but the 1003 x 3000 x 1160 GEMM's epilogue
// makes 28.4 of 26.5 us.
template <bool BRANCH = false>
__device__ __forceinline__ float gelu_erf(float u)
{
    const float z = u * u;
    float p = -6.449855391110759e-06f;
    p = fmaf(p, z, 0.00010947314149234444f);
    p = fmaf(p, z, -0.0011813343735411763f);
    p = fmaf(p, z, 0.009970515966415405f);
    p = fmaf(p, z, -0.06648968905210495f);
    p = fmaf(p, z, 0.398942232131958f);
    const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(u), 0.3f, 1.0f));
    float r = 0.1794036477804184f;
    r = fmaf(r, t, -0.43955719470977783f);
    r = fmaf(r, t, 0.15026725828647614f);
    r = fmaf(r, t, -0.2037215232849121f);
    r = fmaf(r, t, -0.04562024399638176f);
    r = fmaf(r, t, -0.039673078805208206f);
    r = fmaf(r, t, 0.0002813413448166102f);
    r = fmaf(r, t, 0.39893439412117004f);
    const float e = __builtin_amdgcn_exp2f(z * -0.72134752044448170368f);
    const float relu = fmaf(0.5f, fabsf(u), 0.5f * u);          // NaN at -infinity, as 0.5 u (1 + erff)
    if constexpr (BRANCH) {
        if (fabsf(u) < 1.25f) return u * fmaf(u, p, 0.5f);
        return fmaf(-e, r, relu);
    }
    const float near = u * fmaf(u, p, 0.5f), far = fmaf(-e, r, relu);
    return fabsf(u) < 1.25f ? near : far;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

} // namespace lithos
