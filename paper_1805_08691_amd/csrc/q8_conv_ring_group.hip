// Independent layers of the main convolution kernel in one launch (see q8_conv_ring_kernel.h):
// the branches of a module that wait for the same tensors.
#include <utility>
#include "q8_conv_ring_kernel.h"

namespace q8 {
namespace {

struct RingGroupBuild {
  const char* name;
  int (*launch)(const ConvParams* const*, int, hipStream_t);
  int bp, bc;
  float base;
};
#define Q8_GROUP_ROW(WP, WC, TP, TC, BK, ST, US) \
  { "conv_i8_ring_group_kernel<" #WP "," #WC "," #TP "," #TC "," #BK "," #ST ">", \
    &launch_ring_group<WP, WC, TP, TC, BK, ST, 0>, WP * TP * 32, WC * TC * 32, US },
const RingGroupBuild kRingGroups[] = {
    Q8_GROUP_ROW(2, 2, 2, 1, 64, 4, 6.7f)     // 0: 128 pixels x 64 channels
    Q8_GROUP_ROW(2, 2, 1, 1, 128, 4, 6.2f)    // 1: 64 x 64, 128 reduction bytes per step
};
#undef Q8_GROUP_ROW
constexpr int kNumRingGroups = sizeof(kRingGroups) / sizeof(kRingGroups[0]);

}  // namespace

// us of a group as tiles of bp x bc: the chain of the longest tile or the operand bytes of all tiles
// at the rate of the chip (28 bytes per clock and CU, a sixth less where a step is not in one tap),
// 0.3 us per hundred workgroups, behind a launch; the rates are those of a single layer's estimate
// (ring_tiles_us), the base is fitted to Inception-v3 against the latency family's groups (us at 3 / 4 /
// 6 / 8 images: 322 / 353 / 425 / 487 with those alone, 320 / 355 / 405 / 437 with this choice).
// Measured on that network, a module's branches as launches of their own and together: 8 images
// 487 -> 437 us, 16: 727 -> 541, 32: 1043 -> 708, 64: 1285 -> 1046 (with the second pipeline from 18
// images on instead of from 48).  128 x 128 tiles of eight wavefronts: 561 at 16 images, 1096 at 64.
// Puts the layers with the longest tiles first, so that the launch does not end with them.
// -1: no build.
int pick_ring_group(const ConvParams** p, int n, float* us) {
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && p[j]->red_len > p[j - 1]->red_len; --j) std::swap(p[j], p[j - 1]);
  int best = -1;
  for (int v = 0; v < kNumRingGroups; ++v) {
    const RingGroupBuild& b = kRingGroups[v];
    float wg = 0.0f, feed = 0.0f, longest = 0.0f;
    for (int i = 0; i < n; ++i) {
      const float w = (float)(((p[i]->M + b.bp - 1L) / b.bp) * ((p[i]->K + b.bc - 1L) / b.bc));
      const float t =
          (float)((long)(b.bp + b.bc) * p[i]->red_len) * (p[i]->C % 64 == 0 ? 1.47e-5f : 1.8e-5f);
      wg += w;
      feed += w * t;
      longest = fmaxf(longest, t);
    }
    const float t = b.base + fmaxf(longest, feed / 256.0f) + 0.00312f * wg;
    if (wg < 2.0e9f && (best < 0 || t < *us)) { best = v; *us = t; }
  }
  return best;
}

int launch_ring_group_variant(int build, const ConvParams* const* p, int n, hipStream_t stream) {
  if (build < 0 || build >= kNumRingGroups || n < 1 || n > kMaxRingGroup)
    return Q8_EINVAL;
  return kRingGroups[build].launch(p, n, stream);
}

const char* ring_group_variant_name(int build) {
  return build >= 0 && build < kNumRingGroups ? kRingGroups[build].name : "unsupported";
}

}  // namespace q8
