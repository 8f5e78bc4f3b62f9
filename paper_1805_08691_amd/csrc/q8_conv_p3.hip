// The builds of the persistent 3x3 tile family (see q8_conv_p3_kernel.h, q8_conv_p3b_kernel.h)
// and their table.  A build asked for a layer it cannot take hands the layer to the generic kernel.
#include "q8_conv_p3_kernel.h"
#include "q8_conv_p3b_kernel.h"

namespace q8 {
namespace {

template <int PL>
int launch_p3_or_generic(ConvParams& p, hipStream_t stream) {
  if (p3_applicable<PL>(p)) return launch_p3<PL>(p, stream);
  return launch_ring<2, 2, 2, 2, 64, 3, 0>(p, stream);
}

int launch_p3b_or_generic(ConvParams& p, hipStream_t stream) {
  if (p3b_applicable(p)) return launch_p3b<0>(p, stream);
  return launch_ring<2, 2, 2, 1, 64, 2, 0>(p, stream);
}

struct P3Variant {
  const char* name;
  int (*launch)(ConvParams&, hipStream_t);
};
const P3Variant kP3Variants[] = {
    {"conv_i8_p3_kernel<4>", &launch_p3_or_generic<4>},     // maps up to 63 pixels wide
    {"conv_i8_p3_kernel<6>", &launch_p3_or_generic<6>},     // up to 127
    {"conv_i8_p3b_kernel", &launch_p3b_or_generic},         // 8 x 16 blocks (16 x 16 for K <= 32): any width
};
constexpr int kNumP3Variants = sizeof(kP3Variants) / sizeof(kP3Variants[0]);

}  // namespace

int num_p3_variants() { return kNumP3Variants; }
int launch_p3_variant(int variant, ConvParams& p, hipStream_t stream) {
  if (variant < 0 || variant >= kNumP3Variants) return Q8_EINVAL;
  return kP3Variants[variant].launch(p, stream);
}
bool p3_variant_takes(int variant, const ConvParams& p) {
  return variant == 0 ? p3_applicable<4>(p) : variant == 1 ? p3_applicable<6>(p) : p3b_applicable(p);
}
// The block-tiled build with a 2x2 maximum of stride 2 behind it, and whether it takes the layer and that many
// bytes of pooled pixels (Hp x Wp of them, cs bytes from one to the next, y 16-byte aligned).
bool p3b_pooled_takes(const ConvParams& p, size_t bytes) {
  return p3b_applicable(p) && !is_extended(p) && bytes < 0x7fffffffUL;
}
int launch_p3b_pooled(ConvParams& p, int8_t* y, int Hp, int Wp, int cs, int bytes, hipStream_t stream) {
  const P3bPool pool{y, bytes, Hp, Wp, cs};
  return launch_p3b<0, true>(p, stream, pool);
}
const char* p3_variant_name(int variant) {
  return variant >= 0 && variant < kNumP3Variants ? kP3Variants[variant].name : "unsupported";
}

}  // namespace q8
