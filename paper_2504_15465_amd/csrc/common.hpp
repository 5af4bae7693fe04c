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

// GELU u * Phi(u).  |u| < 1.25: Phi = 1/2 + u P(u^2), 1.2e-8 of Phi(-|u|) at worst.  Beyond: Phi(-|u|) = exp(-u^2 / 2) t Q(t)
// with t = 1 / (1 + |u| / 4), 8e-9 relative up to |u| = 14, where the exponential leaves the normal numbers; the upper
// half is 1 minus that.  (Both fitted by iteratively reweighted least squares in float64, the coefficients rounded one
// after the other.)  Neither half serves alone: near 0 the second would be 1 minus a number near 1/2 that carries the
// roundings of the reciprocal, the polynomial and the exponential, and 1 + erff cancels for u < -1.
// Measured on 4M uniform points a range against float64, worst / mean relative error (0.5 u (1 + erff) in brackets):
//   -5 .. -2    1.5e-6 / 2.2e-7  (4.8e-2 / 1.7e-3)     0 .. 0.5    1.2e-7 / 3.2e-8  (1.3e-7 / 3.3e-8)
//   -2 .. -1    5.2e-7 / 8.9e-8  (1.2e-6 / 1.7e-7)     0.5 .. 2    1.2e-7 / 2.6e-8  (1.4e-7 / 3.0e-8)
//   -1 .. -0.5  2.0e-7 / 4.0e-8  (2.7e-7 / 5.6e-8)     2 .. 4      9.7e-8 / 2.4e-8  (1.1e-7 / 2.7e-8)
//   -0.5 .. 0   1.3e-7 / 2.9e-8  (1.5e-7 / 3.1e-8)     4 .. 14     8.8e-8 / 4.7e-9  (1.0e-7 / 5.0e-9)
// and 3.8e-7 absolute at worst, for u in [4, 8) (4.5e-7).  26 instructions and two transcendentals without a branch; erff runs
// both of its branches in nearly every wavefront.  bias + GELU of 16384 x 1024 bf16: 20.7 us against 38.7.
__device__ __forceinline__ float gelu_erf(float u)
{
    const float z = u * u;
    float p = -6.449855391110759e-06f;
    p = fmaf(p, z, 0.00010947314149234444f);
    p = fmaf(p, z, -0.0011813343735411763f);
    p = fmaf(p, z, 0.009970515966415405f);
    p = fmaf(p, z, -0.06648968905210495f);
    p = fmaf(p, z, 0.398942232131958f);
    const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(u), 0.25f, 1.0f));
    float q = -0.04812637344002724f;
    q = fmaf(q, t, 0.11394011229276657f);
    q = fmaf(q, t, -0.029026754200458527f);
    q = fmaf(q, t, 0.09738033264875412f);
    q = fmaf(q, t, 0.07127942889928818f);
    q = fmaf(q, t, 0.0951959639787674f);
    q = fmaf(q, t, 0.099573515355587f);
    q = fmaf(q, t, 0.099742092192173f);
    q *= t;
    const float e = __builtin_amdgcn_exp2f(z * -0.72134752044448170368f);
    const float tail = fmaf(e, u >= 0.0f ? -q : q, u >= 0.0f ? 1.0f : 0.0f);
    return u * (fabsf(u) < 1.25f ? fmaf(u, p, 0.5f) : tail);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

} // namespace lithos
