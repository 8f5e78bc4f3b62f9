// What the kernels of the fp32 convolution share: their parameters and the running maxima.
#pragma once
#include "q8_common.h"
#include "q8_conv_common.h"

namespace q8 {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kSlotStride = 32;         // a cache line apart

struct F32Params {
  const float* __restrict__ x;
  const float* __restrict__ w;
  const float* __restrict__ b;
  const float* __restrict__ res;
  float* __restrict__ y;
  unsigned* __restrict__ obs_sum;      // max |conv + bias| before the residual sum, or null
  unsigned* __restrict__ obs_out;      // max |y|, or null
  int N, H, W, C, K, R, S, sh, sw, ph, pw, dh, dw, Ho, Wo, M, rsc, out_cs, out_off, relu;
  int vec_y, vec_b;                    // output / residual rows, the bias take 16-byte accesses
  FastDiv by_img, by_row, by_c, by_s;
  int n_slots;                         // copies of each maximum, kSlotStride values apart
  int n_ptiles, n_ctiles;
};

[[maybe_unused]] constexpr int kOob = (int)0x80000000;   // beyond any descriptor (they span at most 2^31 - 1 bytes)


namespace {

// The workgroup's maxima into the copy of the two slots that it belongs to: one atomic per workgroup
// and slot, and only where the value there is smaller.  An atomic per wavefront on one address costs
// 3 ns each, 10 to 20 us of a launch of 25 in a first batch, where the slots are still low; the
// engine's 16 copies leave none of that.  `mx`: 2 * NW floats of LDS, whose last use every wavefront
// has left behind.
template <int NW>
__device__ __forceinline__ void observe_block(const F32Params& p, float m_sum, float m_out, float* mx) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (!p.obs_sum && !p.obs_out) return;
  for (int off = 32; off > 0; off >>= 1) {
    m_sum = fmaxf(m_sum, __shfl_xor(m_sum, off, 64));
    m_out = fmaxf(m_out, __shfl_xor(m_out, off, 64));
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    mx[wave] = m_sum;
    mx[NW + wave] = m_out;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned* slot = threadIdx.x == 0 ? p.obs_sum : p.obs_out;
    if (!slot) return;
    float m = 0.0f;
    for (int w = 0; w < NW; ++w) m = fmaxf(m, mx[threadIdx.x * NW + w]);
    slot += blockIdx.x % (unsigned)p.n_slots * kSlotStride;
    const unsigned bits = __float_as_uint(m);
    if (bits > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(slot, bits);
  }
#endif
}

}  // namespace

// The tiled kernel on LDS (q8_conv_f32_lds.hip).
int pick_f32_lds(long M, int K, int rsc, float* us);    // us: its estimate
int launch_f32_lds(int build, F32Params& p, hipStream_t stream);
const char* f32_lds_name(int build);
// The tiled kernel on the bf16 matrix instructions (q8_conv_f32_split.hip).
bool f32_split_pays(long M, int K, int rsc, float lds_us, bool lds);
int launch_f32_split(F32Params& p, hipStream_t stream);
const char* f32_split_name(long M, int K);

}  // namespace q8
