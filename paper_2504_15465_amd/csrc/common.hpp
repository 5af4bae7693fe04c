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

// GELU u * Phi(u), Phi(u) = erfc(-u / sqrt 2) / 2, by one formula for every u: with x = |u| / sqrt 2,
// erfc(x) exp(x^2) = 1 - s P(s), s = p x / (1 + p x), P of degree 8 fitted (iteratively reweighted least
// squares, float64) to 8e-9 relative; the lower half of Phi then keeps its RELATIVE accuracy where
// 1 + erff cancels.  In float32, 4M points against float64: worst error 1.4e-7 relative for u > 0 (1.3e-7 with
// erff) and 2.4e-7 absolute overall (4.5e-7), mean for |u| < 3 8.5e-9 (1.1e-8).
// 21 instructions and two transcendentals without a branch; erff runs both of its branches in nearly
// every wavefront, which bound the bias + GELU row kernel (16384 x 1024 bf16: 51 us, 1.3 TB/s).
__device__ __forceinline__ float gelu_erf(float u)
{
    const float w = fminf(fabsf(u), 40.0f) * 0.261629509039022f;           // p / sqrt 2, p = 0.37; Phi is 0 or 1 long before 40
    const float s = w * __builtin_amdgcn_rcpf(w + 1.0f);
    float q = 0.06571311780777805f;
    q = fmaf(q, s, -0.2684981873662216f);
    q = fmaf(q, s, 0.31317405139724813f);
    q = fmaf(q, s, 0.14699449755866215f);
    q = fmaf(q, s, -0.34761325419640404f);
    q = fmaf(q, s, -0.9969110527035865f);
    q = fmaf(q, s, 3.292456271732396f);
    q = fmaf(q, s, -4.254981375949771f);
    q = fmaf(q, s, 3.049674549243907f);
    q = fmaf(q, -s, 1.0f);
    const float h = q * __builtin_amdgcn_exp2f(fmaf(u * u, -0.72134752044448170368f, -1.0f));   // erfc(x) / 2
    return u * (u >= 0.0f ? 1.0f - h : h);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

} // namespace lithos
