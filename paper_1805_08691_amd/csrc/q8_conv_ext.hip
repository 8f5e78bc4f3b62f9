// The extended builds (unsigned activation codes, per-channel scales) of the 3x3 tile family, the
// persistent 3x3 kernel and the pointwise family that the dispatch chooses.  They share the plain
// builds' loops; only the tail differs (its scales, the code range, the bytes' sign bit), so the
// dispatch treats both alike.  Before they existed every such layer ran on the 128 x 128 ring: a
// ResNet-50 step with unsigned codes took 616 us at 13 images (two streams) and takes 392, 849 at
// 64 on one stream where the plain build takes 777.
#include "q8_conv_halo_kernel.h"
#include "q8_conv_p3b_kernel.h"
#include "q8_conv_pw_kernel.h"

namespace q8 {
namespace {

template <int WP, int WC, int TP, int TC, int PL, int KW, int ST>
int halo_ext(ConvParams& p, hipStream_t stream) {
  if (halo3_applicable<WP, WC, TP, TC, PL, KW>(p))
    return launch_halo3<WP, WC, TP, TC, PL, KW, ST, 1>(p, stream);
  return Q8_EUNSUPPORTED;
}

template <int TC, int KS>
int pw_ext(ConvParams& p, hipStream_t stream) {
  return pw_applicable<TC, KS, 1>(p) ? launch_pw<TC, KS, 1>(p, stream) : Q8_EUNSUPPORTED;
}

}  // namespace

// `family`: the variant's number inside its family.  Q8_EUNSUPPORTED, with nothing launched: there
// is no such build or it does not take the layer.
int launch_halo_ext(int family, ConvParams& p, hipStream_t stream) {
  switch (family) {     // the order of q8_conv_halo.hip's table
    case 0: return halo_ext<2, 2, 2, 1, 4, 1, 3>(p, stream);
    case 1: return halo_ext<2, 2, 2, 2, 4, 1, 3>(p, stream);
    case 2: return halo_ext<4, 2, 2, 2, 4, 1, 3>(p, stream);
    case 3: return halo_ext<4, 2, 2, 2, 8, 1, 3>(p, stream);
    case 4: return halo_ext<2, 2, 2, 1, 8, 1, 3>(p, stream);
    case 6: return halo_ext<2, 2, 1, 1, 2, 1, 3>(p, stream);
    case 9: return halo_ext<2, 2, 1, 2, 2, 2, 3>(p, stream);
    case 11: return halo_ext<2, 2, 1, 1, 2, 1, 9>(p, stream);
    case 10: return halo_ext<2, 2, 2, 1, 4, 2, 3>(p, stream);
    case 12: return halo_ext<2, 2, 1, 1, 2, 2, 9>(p, stream);
    case 14: return halo_ext<2, 2, 1, 1, 3, 2, 9>(p, stream);
    case 15: return halo_ext<2, 2, 1, 1, 3, 1, 9>(p, stream);
    case 16: return halo_ext<2, 2, 2, 1, 5, 2, 3>(p, stream);
    default: return Q8_EUNSUPPORTED;
  }
}
int launch_p3_ext(int family, ConvParams& p, hipStream_t stream) {
  return family == 2 && p3b_applicable(p) ? launch_p3b<1>(p, stream) : Q8_EUNSUPPORTED;
}
int launch_pw_ext(int family, ConvParams& p, hipStream_t stream) {
  switch (family) {     // the order of q8_conv_pw.hip's table
    case 0: return pw_ext<1, 1>(p, stream);
    case 2: return pw_ext<1, 2>(p, stream);
    case 3: return pw_ext<2, 2>(p, stream);
    case 5: return pw_ext<2, 4>(p, stream);
    default: return Q8_EUNSUPPORTED;
  }
}

}  // namespace q8
