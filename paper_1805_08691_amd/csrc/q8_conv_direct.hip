// The builds of the latency family (see q8_conv_direct_kernel.h) and their table.
#include <utility>
#include "q8_conv_direct_kernel.h"

namespace q8 {

namespace {
// Bytes of the start values: the bias, or the table with a row per rectangle of taps.
long start_bytes(const ConvParams& p) {
  const long rows = p.tap_sums ? (long)(p.R + 1) * (p.R + 1) * (p.S + 1) * (p.S + 1) : p.bias ? 1 : 0;
  return rows * p.K * 4;
}
}  // namespace

// The start values and the residual codes (as words) are read through descriptors.
bool direct_applicable(const ConvParams& p) {
  if (start_bytes(p) > 0x7fffffffL) return false;
  return !p.res || (p.res_bytes > 0 && p.res_cs % 4 == 0 && p.res_off % 4 == 0 && q8_aligned(p.res, 4));
}

namespace {

DirectParams direct_params(const ConvParams& p) {
  DirectParams d{};
  d.x = p.x; d.w = p.w; d.x_bytes = p.x_bytes; d.w_bytes = p.w_bytes;
  d.M = p.M; d.K = p.K; d.red_len = p.red_len; d.C = p.C;
  d.H = p.H; d.W = p.W; d.in_cs = p.in_cs; d.S = p.S;
  d.Wo = p.Wo; d.HoWo = p.Ho * p.Wo; d.stride_h = p.stride_h; d.stride_w = p.stride_w;
  d.pad_h = p.pad_h; d.pad_w = p.pad_w; d.dil_h = p.dil_h; d.dil_w = p.dil_w;
  d.by_img = FastDiv{p.div_img_m, p.div_img_s}; d.by_row = FastDiv{p.div_row_m, p.div_row_s};
  d.by_c = make_fast_div((unsigned)p.C); d.by_s = make_fast_div((unsigned)p.S);
  d.ptile_fastest = p.ptile_fastest; d.R = p.R;
  d.bias = p.bias; d.res = p.res; d.y = p.y; d.m = p.m; d.m_r = p.m_r; d.relu = p.relu;
  d.out_cs = p.out_cs; d.out_off = p.out_off; d.res_cs = p.res_cs; d.res_off = p.res_off;
  d.vec4 = p.vec4; d.f32_vec4 = p.f32_vec4; d.in_u8 = p.in_u8; d.out_u8 = p.out_u8; d.res_u8 = p.res_u8;
  d.tap_sums = p.tap_sums; d.m_vec = p.m_vec; d.y_f32 = p.y_f32; d.y_deq = p.y_deq; d.q_deq = p.q_deq;
  d.acc_dump = p.acc_dump;
  d.start_bytes = (int)start_bytes(p);
  d.res_bytes = p.res ? p.res_bytes : 0;
  d.mode = p.C % 64 != 0 ? 0 : p.R * p.S == 1 && (p.pad_h | p.pad_w) == 0 ? 2 : 1;
  return d;
}

template <int TP, int TC, int KW, int NB>
int launch_direct_group(const ConvParams* const* p, int n, hipStream_t stream) {
  DirectGroup g;
  g.n = n;
  long blocks = 0;
  for (int i = 0; i < n; ++i) {
    DirectParams& d = g.layer[i] = direct_params(*p[i]);
    d.n_ptiles = (d.M + TP * 16 - 1) / (TP * 16);
    d.n_ctiles = (d.K + TC * 16 - 1) / (TC * 16);
    g.first[i] = (int)blocks;
    blocks += (long)d.n_ptiles * d.n_ctiles;
    if (blocks > 0x7fffffffL) return Q8_EUNSUPPORTED;
  }
  hipLaunchKernelGGL((conv_i8_direct_group_kernel<TP, TC, KW, NB>), dim3((unsigned)blocks), dim3(KW * 64),
                     0, stream, g);
  return q8_launch_status();
}

template <int TP, int TC, int KW, int NB>
int launch_direct(const ConvParams& p, hipStream_t stream) {
  DirectParams d = direct_params(p);
  d.n_ptiles = (p.M + TP * 16 - 1) / (TP * 16);
  d.n_ctiles = (p.K + TC * 16 - 1) / (TC * 16);
  const long nblk = (long)d.n_ptiles * d.n_ctiles;
  if (nblk > 0x7fffffffL) return Q8_EUNSUPPORTED;
  auto kernel = d.mode == 0   ? conv_i8_direct_kernel<TP, TC, KW, NB, 0>
                : d.mode == 2 ? conv_i8_direct_kernel<TP, TC, KW, NB, 2>
                              : conv_i8_direct_kernel<TP, TC, KW, NB, 1>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)nblk), dim3(KW * 64), 0, stream, d);
  return q8_launch_status();
}

// us of a launch = base + per_wg * (workgroups beyond 256) / 100
//                 + per_byte * (operand bytes of one tile / 100 KB) * (tiles the busiest CU gets),
// fitted to launches behind one another with operands from the last-level cache: the layers of
// the three benchmark networks at batch 1 to 16 (over the 165 of them that the choice gives to this
// family, 2.4 ... 17 us: mean error 0.5 us, largest 1.8).  The operand term is 14 bytes per clock and CU, what gathered register loads reach here.
struct DirectVariant {
  const char* name;
  int (*launch)(const ConvParams&, hipStream_t);
  int (*launch_group)(const ConvParams* const*, int, hipStream_t);
  int bp, bc;
  float base, per_wg, per_byte;
};
#define Q8_DIRECT_ROW(TP, TC, KW, NB, A, B, C) \
  { "conv_i8_direct_kernel<" #TP "," #TC "," #KW "," #NB ">", &launch_direct<TP, TC, KW, NB>, \
    &launch_direct_group<TP, TC, KW, NB>, TP * 16, TC * 16, A, B, C },
const DirectVariant kDirectVariants[] = {
    Q8_DIRECT_ROW(1, 1, 8, 8, 2.70f, 0.178f, 2.32f)   // 0: 16 pixels x 16 channels, eight wavefronts
    Q8_DIRECT_ROW(1, 1, 4, 8, 2.69f, 0.024f, 2.36f)   // 1
    Q8_DIRECT_ROW(2, 1, 4, 6, 2.90f, 0.044f, 2.13f)   // 2: 32 x 16
    Q8_DIRECT_ROW(2, 2, 4, 4, 3.01f, 0.066f, 2.29f)   // 3: 32 x 32
};
#undef Q8_DIRECT_ROW
constexpr int kNumDirectVariants = sizeof(kDirectVariants) / sizeof(kDirectVariants[0]);

}  // namespace

int num_direct_variants() { return kNumDirectVariants; }
int launch_direct_variant(int variant, ConvParams& p, hipStream_t stream) {
  if (variant < 0 || variant >= kNumDirectVariants) return Q8_EINVAL;
  if (!direct_applicable(p)) return Q8_EUNSUPPORTED;
  return kDirectVariants[variant].launch(p, stream);
}
// The cheapest build for M pixels, K channels and red_len reduction bytes; *us its estimate.
int pick_direct(long M, int K, int red_len, float* us) {
  int best = -1;
  for (int v = 0; v < kNumDirectVariants; ++v) {
    const DirectVariant& d = kDirectVariants[v];
    const long wg = ((M + d.bp - 1) / d.bp) * ((K + d.bc - 1) / d.bc);
    const float t = d.base + d.per_wg * (float)(wg > 256 ? wg - 256 : 0) * 0.01f +
                    d.per_byte * (float)((long)(d.bp + d.bc) * red_len) * 1e-5f * (float)((wg + 255) / 256);
    if (best < 0 || t < *us) { best = v; *us = t; }
  }
  return best;
}
// The same for several independent layers in one launch: the busiest CU has the largest tile, or
// its share of all of them.  Puts the layers with the longest tiles first, so that the launch does not
// end with them.
int pick_direct_group(const ConvParams** p, int n, float* us) {
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && p[j]->red_len > p[j - 1]->red_len; --j) std::swap(p[j], p[j - 1]);
  int best = -1;
  for (int v = 0; v < kNumDirectVariants; ++v) {
    const DirectVariant& d = kDirectVariants[v];
    float wg = 0.0f, bytes = 0.0f, largest = 0.0f;
    for (int i = 0; i < n; ++i) {
      const float w = (float)(((p[i]->M + d.bp - 1) / d.bp) * (long)((p[i]->K + d.bc - 1) / d.bc));
      const float b = (float)((long)(d.bp + d.bc) * p[i]->red_len);
      wg += w;
      bytes += w * b;
      largest = b > largest ? b : largest;
    }
    const float share = bytes / 256.0f;
    const float t = d.base + 0.3f + d.per_wg * (wg > 256.0f ? wg - 256.0f : 0.0f) * 0.01f +
                    d.per_byte * 1e-5f * (wg > 256.0f ? share + 0.5f * largest : largest);
    if (best < 0 || t < *us) { best = v; *us = t; }
  }
  return best;
}
int launch_direct_group_variant(int variant, const ConvParams* const* p, int n, hipStream_t stream) {
  if (variant < 0 || variant >= kNumDirectVariants || n < 1 || n > kMaxGroup) return Q8_EINVAL;
  return kDirectVariants[variant].launch_group(p, n, stream);
}
const char* direct_variant_name(int variant) {
  return variant >= 0 && variant < kNumDirectVariants ? kDirectVariants[variant].name : "unsupported";
}

}  // namespace q8
