// q8_run_ops: a list of calls enqueued by one (see include/q8conv.h), with independent
// neighbours joined into one launch where the estimates say that it is shorter.
#include "q8_common.h"
#include "q8_conv_common.h"

namespace q8 {
int conv_fill_op(const q8_op* o, ConvParams& p, bool* empty);
int conv_choose(const q8_conv_desc* d, const ConvParams& p, float* us);
int conv_launch_chosen(int variant, ConvParams& p, hipStream_t s);
int first_direct_variant();
int num_direct_variants();
bool direct_applicable(const ConvParams& p);
int pick_direct_group(const ConvParams* const* p, int n, float* us);
int launch_direct_group_variant(int variant, const ConvParams* const* p, int n, hipStream_t stream);
int dequantize_list(const q8_op* ops, int n, hipStream_t stream);   // q8_elementwise.hip

namespace {

constexpr int kMaxGroup = 8;

int run_one(const q8_op& o, void* stream) {
  const q8_conv_desc& d = o.d;
  switch (o.kind) {
    case Q8_OP_CONV: {
      ConvParams p;
      bool empty = false;
      const int rc = conv_fill_op(&o, p, &empty);
      if (rc != Q8_OK || empty) return rc;
      float us = 0.0f;
      return conv_launch_chosen(conv_choose(&d, p, &us), p, (hipStream_t)stream);
    }
    case Q8_OP_HEAD:
      return q8_conv_image_f32_int8(&d, (const float*)o.x, o.H, o.W, o.C, o.top, o.left, o.q_x, o.p, o.w,
                                    (const int32_t*)o.bias, o.q_w, o.q_out, o.flags & Q8_OPF_POOL ? 1 : 0,
                                    (int8_t*)o.y, stream);
    case Q8_OP_POOL:
      return q8_pool_i8((const int8_t*)o.x, d.N, o.H, o.W, o.C, o.mode, o.R, o.S, o.stride, o.pad, o.Ho, o.Wo,
                        o.q_x, o.q_out, (int8_t*)o.y, d.out_c_stride, d.out_c_off, stream);
    case Q8_OP_MAXPOOL:
      return q8_maxpool_i8((const int8_t*)o.x, d.N, o.H, o.W, o.C, o.R, o.S, o.stride, o.pad, o.Ho, o.Wo,
                           (int8_t*)o.y, stream);
    case Q8_OP_QUANTIZE:
      return q8_quantize((const float*)o.x, o.n, o.q_x, o.p, (int8_t*)o.y, stream);
    case Q8_OP_QUANTIZE_PAD:
      return q8_quantize_pad_channels((const float*)o.x, o.n, o.C, o.Ho, o.q_x, o.p, (int8_t*)o.y, stream);
    case Q8_OP_QUANTIZE_IMAGE:
      return q8_quantize_image((const float*)o.x, d.N, o.H, o.W, o.C, o.q_x, o.p, (int8_t*)o.y, o.Ho, o.Wo,
                               o.top, o.left, stream);
    case Q8_OP_DEQUANTIZE:
      return o.flags & Q8_OPF_IN_U8 ? q8_dequantize_u8((const int8_t*)o.x, o.n, o.q_x, o.y_f32, stream)
                                    : q8_dequantize((const int8_t*)o.x, o.n, o.q_x, o.y_f32, stream);
    default:
      return Q8_EINVAL;
  }
}

// A run of independent ops on one stream.  The convolutions that would be launched as the latency
// family anyway go together, or all of them do, or none: whatever is estimated shortest.  Ops in
// front of a refused one are enqueued, those behind it are not: the convolutions, whose arguments
// are checked without a launch, therefore go behind the others.
int run_group(const q8_op* ops, int n, void* stream) {
  ConvParams p[kMaxGroup];
  const ConvParams *small[kMaxGroup], *all[kMaxGroup];
  int variant[kMaxGroup], n_small = 0, n_all = 0, n_conv = 0, refused = Q8_OK;
  bool is_small[kMaxGroup] = {}, waiting[kMaxGroup] = {};
  float us_each[kMaxGroup], us_small = 0.0f, us_all = 0.0f;
  const int first = first_direct_variant(), last = first + num_direct_variants();
  for (int i = 0; i < n && refused == Q8_OK; ++i) {
    if (ops[i].kind != Q8_OP_CONV) continue;
    bool empty = false;
    refused = conv_fill_op(&ops[i], p[i], &empty);
    if (refused != Q8_OK) n = i;
    else waiting[i] = !empty;
  }
  for (int i = 0; i < n; ++i) {
    if (ops[i].kind == Q8_OP_CONV) continue;
    const int rc = run_one(ops[i], stream);
    if (rc != Q8_OK) {
      refused = rc;
      n = i;
    }
  }
  for (int i = 0; i < n; ++i) {
    if (!waiting[i]) continue;
    ++n_conv;
    variant[i] = conv_choose(&ops[i].d, p[i], &us_each[i]);
    us_all += us_each[i];
    if (direct_applicable(p[i]) && p[i].S4 == 0) all[n_all++] = &p[i];
    if (variant[i] >= first && variant[i] < last) {
      is_small[i] = true;
      us_small += us_each[i];
      small[n_small++] = &p[i];
    }
  }
  float us_g = 0.0f, us_a = 0.0f;
  const int vs = n_small >= 2 ? pick_direct_group(small, n_small, &us_g) : -1;
  const int va = n_all >= 2 && n_all == n_conv ? pick_direct_group(all, n_all, &us_a) : -1;
  const float saved_small = vs >= 0 ? us_small - us_g : 0.0f, saved_all = va >= 0 ? us_all - us_a : 0.0f;
  if (saved_all > 0.0f && saved_all >= saved_small) {
    const int rc = launch_direct_group_variant(va, all, n_all, (hipStream_t)stream);
    return rc != Q8_OK ? rc : refused;
  }
  if (saved_small > 0.0f) {
    const int rc = launch_direct_group_variant(vs, small, n_small, (hipStream_t)stream);
    if (rc != Q8_OK) return rc;
    for (int i = 0; i < n; ++i) waiting[i] = waiting[i] && !is_small[i];
  }
  for (int i = 0; i < n; ++i) {
    if (!waiting[i]) continue;
    const int rc = conv_launch_chosen(variant[i], p[i], (hipStream_t)stream);
    if (rc != Q8_OK) return rc;
  }
  return refused;
}

}  // namespace
}  // namespace q8

extern "C" int q8_run_ops(const q8_op* ops, int n_ops, void* const* streams, int n_streams) {
  Q8_REQUIRE(n_ops >= 0 && (n_ops == 0 || (ops && streams && n_streams >= 1)), Q8_EINVAL);
  for (int i = 0; i < n_ops; ++i) Q8_REQUIRE(ops[i].stream >= 0 && ops[i].stream < n_streams, Q8_EINVAL);
  for (int i = 0; i < n_ops;) {
    const q8_op& o = ops[i];
    int j = i + 1;
    int rc;
    if (o.kind == Q8_OP_DEQUANTIZE) {
      while (j < n_ops && ops[j].kind == Q8_OP_DEQUANTIZE && ops[j].stream == o.stream) ++j;
      rc = q8::dequantize_list(ops + i, j - i, (hipStream_t)streams[o.stream]);
    } else if (o.group) {
      while (j < n_ops && j - i < q8::kMaxGroup && ops[j].group == o.group && ops[j].stream == o.stream &&
             ops[j].kind != Q8_OP_DEQUANTIZE)
        ++j;
      rc = j - i == 1 ? q8::run_one(o, streams[o.stream]) : q8::run_group(ops + i, j - i, streams[o.stream]);
    } else {
      rc = q8::run_one(o, streams[o.stream]);
    }
    if (rc != Q8_OK) return rc;
    i = j;
  }
  return Q8_OK;
}
