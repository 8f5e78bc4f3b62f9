// q8_run_ops: a list of calls enqueued by one (see include/q8conv.h), with independent
// neighbours joined into one launch where the estimates say that it is shorter.
#include "q8_common.h"
#include "q8_conv_common.h"

namespace q8 {
int conv_fill_op(const q8_op* o, ConvParams& p, bool* empty);
int conv_choose(const q8_conv_desc* d, const ConvParams& p, float* us, bool alone = false);
int conv_launch_chosen(int variant, ConvParams& p, hipStream_t s);
int first_direct_variant();
int num_direct_variants();
bool direct_applicable(const ConvParams& p);
int pick_direct_group(const ConvParams** p, int n, float* us);
int launch_direct_group_variant(int variant, const ConvParams* const* p, int n, hipStream_t stream);
int ring_group_takes(const q8_conv_desc* d, const ConvParams& p);
int pick_ring_group(const ConvParams** p, int n, float* us);
int launch_ring_group_variant(int build, const ConvParams* const* p, int n, hipStream_t stream);
const char* direct_variant_name(int variant);
const char* ring_group_variant_name(int build);
int first_p3_variant();
bool p3b_pooled_takes(const ConvParams& p, size_t bytes);
int launch_p3b_pooled(ConvParams& p, int8_t* y, int Hp, int Wp, int cs, int bytes, hipStream_t stream);
int num_bneck_builds();
const char* bneck_build_name(int build);
bool bneck_applicable(const ConvParams& a, const ConvParams& b, const ConvParams& c);
bool bneck_build_takes(int build, const ConvParams& a, const ConvParams& b, const ConvParams& c);
int pick_bneck(const ConvParams& a, const ConvParams& b, const ConvParams& c, float* us);
int launch_bneck(int build, const ConvParams& a, const ConvParams& b, const ConvParams& c, hipStream_t stream);
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

// The build for a block of three layers, -1: three launches.  shared: what the first layer's share of a launch
// with others takes less than a launch of its own; null: the block is marked, whoever marked it has asked.
// The estimates are of launches by themselves.  Inside a network (six blocks in a row with filters of their own; 486
// such networks of 64 to 1024 outer channels on 7 x 7 to 56 x 56 pixels, half of them with a projection beside each
// first layer) one launch and three lie apart from them by what goes with the middle channels and the launches
// replaced:
//  * no projection: below 1.15 of the three launches' estimate no block on 64 channels loses, below 0.95 none on 128.
//    (28 x 28 x 512 on one image, 0.96, gains 4 % there and costs ResNet-50 201.9 -> 204.2 us.)  256: three launches
//    are estimated up to a sixth too long while the last layer has at most two tiles of 64 x 64 per CU (1024 -> 256
//    -> 1024 on 14 x 14, 8 images 1.07 of their time at an estimated 0.89, 11 images 0.97 at 0.93);
//  * a projection: of 60, 87 and 96 on 64, 128 and 256 channels 0, 5 (up to 7 %) and 13 (up to 12 %) lose. Where the
//    first layer counted as a launch of its own, 2, 13 and 42 did, up to 29 %.
// ResNet-50, 8 images 295 -> 286 us, unsigned 319.5 -> 314.8.
// Unsigned or per-channel blocks of one or two images stay three launches: 9.7 us and 8.5 by themselves, but inside
// ResNet-50 209.0 and 211.9 with three of them (plain codes 203.0 and 200.9); two images unsigned 247.1 with three
// launches and 249.0, per channel 247.3 and 247.2; three per channel 303.6 and 275.6.
int block_choose(const q8_op* ops, const ConvParams* p, const float* shared) {
  float us = 0.0f, three = 0.0f;
  const int build = bneck_applicable(p[0], p[1], p[2]) ? pick_bneck(p[0], p[1], p[2], &us) : -1;
  if (build < 0) return -1;
  if (p[0].N <= 2 && (is_extended(p[0]) || is_extended(p[1]) || is_extended(p[2]))) return -1;
  for (int i = 0; i < 3; ++i) {
    float t = 0.0f;
    conv_choose(&ops[i].d, p[i], &t);
    three += t;
  }
  const long tiles = ((p[2].M + 63L) / 64) * ((p[2].K + 63) / 64);
  float most = (p[0].K == 64 ? 1.15f : 0.95f) * three;
  if (shared && *shared > 0.0f)
    most = fminf(most, (p[0].K == 256 ? 0.9f : 1.05f) * (three - *shared));
  else if (shared && p[0].K == 256 && tiles <= 512)
    most = 0.88f * three;
  return us < most ? build : -1;
}
int block_fill(const q8_op* ops, ConvParams* p, const float* shared = nullptr) {
  for (int i = 0; i < 3; ++i) {
    bool empty = false;
    if (ops[i].kind != Q8_OP_CONV || conv_fill_op(&ops[i], p[i], &empty) != Q8_OK || empty) return -1;
  }
  return block_choose(ops, p, shared);
}

// How the convolutions of a run of independent ops are launched: in part or in whole together, as
// the latency family or as the main kernel's group builds, or each by itself, whatever is estimated
// shortest.
struct GroupPlan {
  // Who may go where: every layer the latency family takes (all of them or none); those that it
  // would be launched as anyway (small); those whose tiled choice is the main kernel, the same with
  // the 3x3 family's, and of the former the ones that are not small.
  enum { kAllDirect, kSmallDirect, kTiled, kTiled3x3, kLargeTiled, kSets };
  ConvParams p[kMaxGroup];
  bool waiting[kMaxGroup] = {};        // convolutions that still have to be launched
  int variant[kMaxGroup];              // what each would be launched as on its own
  const ConvParams* set[kSets][kMaxGroup];
  int count[kSets] = {}, build[kSets], member[kMaxGroup] = {};
  int chosen[2] = {-1, -1};            // sets to launch together
  float less = 0.0f;                   // what that takes less than every layer on its own

  void choose(const q8_op* ops, int n) {
    const int first = first_direct_variant(), last = first + num_direct_variants();
    float alone[kSets] = {}, saved[kSets];
    int n_conv = 0;
    for (int i = 0; i < n; ++i) {
      if (!waiting[i]) continue;
      ++n_conv;
      float us = 0.0f;
      variant[i] = conv_choose(&ops[i].d, p[i], &us);
      const bool small = variant[i] >= first && variant[i] < last;
      const int tiled = ring_group_takes(&ops[i].d, p[i]);
      const bool in[kSets] = {direct_applicable(p[i]) && p[i].S4 == 0, small, tiled == 1, tiled != 0,
                              tiled == 1 && !small};
      for (int s = 0; s < kSets; ++s) {
        if (!in[s]) continue;
        member[i] |= 1 << s;
        set[s][count[s]++] = &p[i];
        alone[s] += us;
      }
    }
    for (int s = 0; s < kSets; ++s) {
      saved[s] = 0.0f;
      if (count[s] < 2 || (s == kAllDirect && count[s] != n_conv)) continue;
      float us = 0.0f;
      build[s] = s <= kSmallDirect ? pick_direct_group(set[s], count[s], &us)
                                   : pick_ring_group(set[s], count[s], &us);
      if (build[s] >= 0 && us < alone[s]) saved[s] = alone[s] - us;
    }
    int best = kAllDirect;
    for (int s : {kTiled, kTiled3x3})
      if (saved[s] > saved[best]) best = s;
    if (saved[best] > 0.0f && saved[best] >= saved[kSmallDirect] + saved[kLargeTiled]) {
      chosen[0] = best;
    } else {
      if (saved[kLargeTiled] > 0.0f) chosen[0] = kLargeTiled;
      if (saved[kSmallDirect] > 0.0f) chosen[1] = kSmallDirect;
    }
    for (int s : chosen)
      if (s >= 0) less += saved[s];
  }
};

// What the convolutions among independent ops take less together than on their own.
float group_less(const q8_op* ops, int n) {
  GroupPlan g;
  int m = 0;
  q8_op convs[kMaxGroup];
  for (int i = 0; i < n && m < kMaxGroup; ++i) {
    bool empty = false;
    if (ops[i].kind != Q8_OP_CONV || conv_fill_op(&ops[i], g.p[m], &empty) != Q8_OK || empty) continue;
    g.waiting[m] = true;
    convs[m++] = ops[i];
  }
  g.choose(convs, m);
  return g.less;
}

// A run of independent ops on one stream.  Ops in front of a refused one are enqueued, those behind
// it are not: the convolutions, whose arguments are checked without a launch, therefore go behind
// the others.
int run_group(const q8_op* ops, int n, void* stream) {
  GroupPlan g;
  int refused = Q8_OK;
  for (int i = 0; i < n && refused == Q8_OK; ++i) {
    if (ops[i].kind != Q8_OP_CONV) continue;
    bool empty = false;
    refused = conv_fill_op(&ops[i], g.p[i], &empty);
    if (refused != Q8_OK) n = i;
    else g.waiting[i] = !empty;
  }
  for (int i = 0; i < n; ++i) {
    if (ops[i].kind == Q8_OP_CONV) continue;
    const int rc = run_one(ops[i], stream);
    if (rc != Q8_OK) {
      refused = rc;
      n = i;
    }
  }
  g.choose(ops, n);
  for (int s : g.chosen) {
    if (s < 0) continue;
    const int rc = (s <= GroupPlan::kSmallDirect ? launch_direct_group_variant : launch_ring_group_variant)(
        g.build[s], g.set[s], g.count[s], (hipStream_t)stream);
    if (rc != Q8_OK) return rc;
    for (int i = 0; i < n; ++i) g.waiting[i] = g.waiting[i] && !(g.member[i] >> s & 1);
  }
  for (int i = 0; i < n; ++i) {
    if (!g.waiting[i]) continue;
    const int rc = conv_launch_chosen(g.variant[i], g.p[i], (hipStream_t)stream);
    if (rc != Q8_OK) return rc;
  }
  return refused;
}

// A bottleneck block: one launch where there is a build for it that is estimated shorter than three.
int run_block(const q8_op* ops, void* stream) {
  ConvParams p[3];
  const int build = block_fill(ops, p);
  if (build >= 0) return launch_bneck(build, p[0], p[1], p[2], (hipStream_t)stream);
  for (int i = 0; i < 3; ++i) {
    const int rc = run_one(ops[i], stream);
    if (rc != Q8_OK) return rc;
  }
  return Q8_OK;
}

// The 2x2 maximum with stride 2 as the kernel writes it: address of pooled pixel (0, 0), bytes from there on, bytes
// from one pixel to the next.
struct Pooled {
  int8_t* y;
  int bytes, cs;
};

// Whether pool is that maximum over conv's output and nothing else: no change of factor, no
// window without a pixel, every address in reach, and an output apart from all that the convolution reads and
// writes (a program may reuse the convolution's input there).
bool pool_behind(const q8_op& pool, const q8_op& conv, const ConvParams& p, Pooled* out) {
  const bool to_slice = pool.kind == Q8_OP_POOL;
  if (!(to_slice ? pool.mode == 0 && pool.q_x == pool.q_out && q8_finite_pos(pool.q_x) : pool.kind == Q8_OP_MAXPOOL))
    return false;
  const int cs = to_slice ? pool.d.out_c_stride : pool.C, c_off = to_slice ? pool.d.out_c_off : 0;
  if (pool.x != conv.y || pool.d.N != p.N || pool.H != p.Ho || pool.W != p.Wo || pool.C != p.K || p.out_cs != p.K ||
      p.out_off != 0 || pool.R != 2 || pool.S != 2 || pool.stride != 2 || pool.pad != 0 || pool.Ho < 1 || pool.Wo < 1 ||
      pool.Ho > (p.Ho + 1) / 2 || pool.Wo > (p.Wo + 1) / 2 || !pool.y || c_off < 0 || cs < c_off + pool.C ||
      (cs | c_off) % 16 || !q8_aligned(pool.y, 16))
    return false;
  const size_t bytes = (size_t)p.N * pool.Ho * pool.Wo * cs, table = (size_t)p.K * sizeof(int32_t);
  auto apart = [&](const void* b, size_t n) {
    const char *const a = (const char*)pool.y, *const c = (const char*)b;
    return !b || c + n <= a || a + bytes <= c;
  };
  if (!p3b_pooled_takes(p, bytes) || !apart(p.x, p.x_bytes) || !apart(p.w, p.w_bytes) || !apart(p.bias, table) ||
      !apart(p.y, (size_t)p.M * p.out_cs))
    return false;
  *out = {(int8_t*)pool.y + c_off, (int)(bytes - c_off), cs};
  return true;
}

// Whether work on one of two different handles waits for work enqueued on the other: the legacy default stream
// and streams that were not created to ignore it.
bool streams_wait(void* a, void* b) {
  auto legacy = [](void* s) { return s == nullptr || s == (void*)1; };             // (1: hipStreamLegacy)
  if (legacy(a) == legacy(b)) return legacy(a);
  unsigned flags = 0;
  return hipStreamGetFlags((hipStream_t)(legacy(a) ? b : a), &flags) != hipSuccess || !(flags & hipStreamNonBlocking);
}

// A list's convolutions that wait for the maximum behind them, to go into one launch with it at its place.
// A convolution goes behind ops of other streams only (streams wait for each other outside of a list only), and is
// enqueued by itself where one of those is refused: what stands in front of a refused op runs, what stands
// behind it does not.
struct Waiting {
  static constexpr int kAhead = 8;         // ops from a convolution to its maximum; convolutions that wait
  struct Entry {
    int conv, pool, variant;
    ConvParams p;
    Pooled pooled;
  };
  Entry entry[kAhead];
  int n = 0;

  // Op i, a convolution: the index of the op that goes into its launch, -1: none.
  static int behind(const q8_op* ops, int n_ops, void* const* streams, int i, const ConvParams& p, int variant,
                    Pooled* pooled) {
    if (variant != first_p3_variant() + 2) return -1;
    void* const own = streams[ops[i].stream];
    for (int j = i + 1; j < n_ops && j - i < kAhead; ++j) {
      void* const other = streams[ops[j].stream];
      if (other == own) return pool_behind(ops[j], ops[i], p, pooled) ? j : -1;
      if (streams_wait(own, other)) return -1;
    }
    return -1;
  }
  int run(const q8_op* ops, int n_ops, void* const* streams, int i) {
    const q8_op& o = ops[i];
    void* const stream = streams[o.stream];
    if (o.kind != Q8_OP_CONV || n == kAhead) return run_one(o, stream);
    bool empty = false;
    Entry& e = entry[n];
    const int rc = conv_fill_op(&o, e.p, &empty);
    if (rc != Q8_OK || empty) return rc;
    float us = 0.0f;
    e.variant = conv_choose(&o.d, e.p, &us);
    e.pool = behind(ops, n_ops, streams, i, e.p, e.variant, &e.pooled);
    if (e.pool < 0) return conv_launch_chosen(e.variant, e.p, (hipStream_t)stream);
    e.conv = i;
    ++n;
    return Q8_OK;
  }
  // Op i, if it is one of those maxima: both run.
  bool take(const q8_op* ops, void* const* streams, int i, int* rc) {
    for (int k = 0; k < n; ++k) {
      if (entry[k].pool != i) continue;
      Entry& e = entry[k];
      *rc = launch_p3b_pooled(e.p, e.pooled.y, ops[i].Ho, ops[i].Wo, e.pooled.cs, e.pooled.bytes,
                              (hipStream_t)streams[ops[i].stream]);
      for (--n; k < n; ++k) entry[k] = entry[k + 1];
      return true;
    }
    return false;
  }
  int refused(const q8_op* ops, void* const* streams, int code) {
    for (int k = 0; k < n; ++k) {
      const int rc = conv_launch_chosen(entry[k].variant, entry[k].p, (hipStream_t)streams[ops[entry[k].conv].stream]);
      if (rc != Q8_OK) return rc;
    }
    return code;
  }
};

}  // namespace
}  // namespace q8

extern "C" int q8_run_ops(const q8_op* ops, int n_ops, void* const* streams, int n_streams) {
  Q8_REQUIRE(n_ops >= 0 && (n_ops == 0 || (ops && streams && n_streams >= 1)), Q8_EINVAL);
  for (int i = 0; i < n_ops; ++i) Q8_REQUIRE(ops[i].stream >= 0 && ops[i].stream < n_streams, Q8_EINVAL);
  q8::Waiting waiting;
  for (int i = 0; i < n_ops;) {
    const q8_op& o = ops[i];
    int j = i + 1;
    int rc;
    if (waiting.take(ops, streams, i, &rc)) {
      // (its convolution ran with it)
    } else if (o.kind == Q8_OP_DEQUANTIZE) {
      while (j < n_ops && ops[j].kind == Q8_OP_DEQUANTIZE && ops[j].stream == o.stream) ++j;
      rc = q8::dequantize_list(ops + i, j - i, (hipStream_t)streams[o.stream]);
    } else if (o.kind == Q8_OP_CONV && (o.flags & Q8_OPF_BLOCK) && !o.group && i + 2 < n_ops &&
               ops[i + 1].stream == o.stream && ops[i + 2].stream == o.stream) {
      j = i + 3;
      rc = q8::run_block(ops + i, streams[o.stream]);
    } else if (o.group) {
      while (j < n_ops && j - i < q8::kMaxGroup && ops[j].group == o.group && ops[j].stream == o.stream &&
             ops[j].kind != Q8_OP_DEQUANTIZE)
        ++j;
      rc = j - i == 1 ? waiting.run(ops, n_ops, streams, i) : q8::run_group(ops + i, j - i, streams[o.stream]);
    } else {
      rc = waiting.run(ops, n_ops, streams, i);
    }
    if (rc != Q8_OK) return waiting.refused(ops, streams, rc);
    i = j;
  }
  return Q8_OK;
}

extern "C" const char* q8_group_variant(const q8_op* ops, int n_ops) {
  if (!ops || n_ops < 1 || n_ops > q8::kMaxGroup) return "unsupported";
  q8::GroupPlan g;
  for (int i = 0; i < n_ops; ++i) {
    bool empty = false;
    if (ops[i].kind != Q8_OP_CONV) continue;
    if (q8::conv_fill_op(&ops[i], g.p[i], &empty) != Q8_OK) return "unsupported";
    g.waiting[i] = !empty;
  }
  g.choose(ops, n_ops);
  const int s = g.chosen[0] >= 0 ? g.chosen[0] : g.chosen[1];
  if (s < 0) return "single launches";
  return s <= q8::GroupPlan::kSmallDirect ? q8::direct_variant_name(g.build[s])
                                          : q8::ring_group_variant_name(g.build[s]);
}

extern "C" const char* q8_block_variant(const q8_op* ops) {
  q8::ConvParams p[3];
  const int build = ops ? q8::block_fill(ops, p) : -1;
  return build >= 0 ? q8::bneck_build_name(build) : "single launches";
}

extern "C" int q8_block_pays(const q8_op* block, const q8_op* beside, int n_beside) {
  if (!block || n_beside < 0 || n_beside >= q8::kMaxGroup || (n_beside && !beside)) return 0;
  q8::ConvParams p[3];
  float shared = 0.0f;
  if (n_beside) {
    q8_op all[q8::kMaxGroup];
    all[0] = block[0];
    for (int i = 0; i < n_beside; ++i) all[i + 1] = beside[i];
    shared = q8::group_less(all, n_beside + 1) - q8::group_less(beside, n_beside);
  }
  if (!(shared > 0.0f)) shared = 0.0f;
  return q8::block_fill(block, p, &shared) >= 0;
}

extern "C" int q8_num_bottleneck_builds(void) { return q8::num_bneck_builds(); }

extern "C" const char* q8_bottleneck_build_name(int build) {
  return build >= 0 && build < q8::num_bneck_builds() ? q8::bneck_build_name(build) : "unsupported";
}

extern "C" int q8_run_bottleneck(const q8_op* ops, int build, void* stream) {
  Q8_REQUIRE(ops && build >= 0 && build < q8::num_bneck_builds(), Q8_EINVAL);
  q8::ConvParams p[3];
  for (int i = 0; i < 3; ++i) {
    bool empty = false;
    Q8_REQUIRE(ops[i].kind == Q8_OP_CONV, Q8_EINVAL);
    const int rc = q8::conv_fill_op(&ops[i], p[i], &empty);
    if (rc != Q8_OK) return rc;
    Q8_REQUIRE(!empty, Q8_EUNSUPPORTED);
  }
  Q8_REQUIRE(q8::bneck_applicable(p[0], p[1], p[2]) && q8::bneck_build_takes(build, p[0], p[1], p[2]), Q8_EUNSUPPORTED);
  return q8::launch_bneck(build, p[0], p[1], p[2], (hipStream_t)stream);
}

extern "C" int q8_joined_op(const q8_op* ops, int n_ops, void* const* streams, int n_streams, int i) {
  if (!ops || !streams || i < 0 || i >= n_ops || ops[i].kind != Q8_OP_CONV) return -1;
  for (int k = i; k < n_ops; ++k)
    if (ops[k].stream < 0 || ops[k].stream >= n_streams) return -1;
  q8::ConvParams p;
  q8::Pooled pooled;
  bool empty = false;
  float us = 0.0f;
  if (q8::conv_fill_op(&ops[i], p, &empty) != Q8_OK || empty) return -1;
  return q8::Waiting::behind(ops, n_ops, streams, i, p, q8::conv_choose(&ops[i].d, p, &us), &pooled);
}
