// Bottleneck blocks as one launch: the builds, which triples of layers they take, launch.
#include "q8_conv_bneck_kernel.h"

namespace q8 {
namespace {

constexpr int kLdsLimit = 163840;

// What a launch takes, us: L (u + v r + w f), L = base + per_step C / 64 + per_round K2 / MID the time of one
// strip, r the strips per CU, rounded up, f how full the last of them is (clocks fall and the L2s share as
// more CUs work).  u = 0 where one workgroup fills a CU; the others overlap two to four.
struct Build {
  const char* name;
  int mid, ap, bp, pitch, row_pad, threads, ring, xbuf, piece;
  int (*launch[2])(BneckParams&, unsigned, int, hipStream_t);
  float base, per_step, per_round, u, v, w;
};

template <int MID, int WP, int TA, int TB, int D, int XS, int GS, int OCC, int EXT>
int launch_build(BneckParams& q, unsigned grid, int lds, hipStream_t stream) {
  auto kernel = conv_i8_bneck_kernel<MID, WP, TA, TB, D, XS, GS, OCC, EXT>;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
  if (attr != hipSuccess) return Q8_EHIP;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(BneckShape<MID, WP, TA, TB, D, XS, GS>::NW * 64), lds, stream, q);
  return q8_launch_status();
}

#define Q8_BNECK(MID, WP, TA, TB, D, XS, GS, OCC, ...)                                                              \
  {"conv_i8_bneck_kernel<" #MID "," #WP "," #TA "," #TB "," #D "," #XS "," #GS "," #OCC ">", MID,                       \
   BneckShape<MID, WP, TA, TB, D, XS, GS>::AP, BneckShape<MID, WP, TA, TB, D, XS, GS>::BP,                     \
   BneckShape<MID, WP, TA, TB, D, XS, GS>::PITCH, BneckShape<MID, WP, TA, TB, D, XS, GS>::ROW_PAD, BneckShape<MID, WP, TA, TB, D, XS, GS>::NW * 64,             \
   BneckShape<MID, WP, TA, TB, D, XS, GS>::RING_BYTES, XS * BneckShape<MID, WP, TA, TB, D, XS, GS>::XCHUNK,    \
   GS * 64,                                                                                            \
   {launch_build<MID, WP, TA, TB, D, XS, GS, OCC, 0>, launch_build<MID, WP, TA, TB, D, XS, GS, OCC, 1>}, __VA_ARGS__}

// Fitted to 59 blocks of 10 x 10 ... 56 x 56 pixels at 1 to 64 images (error 3 % at the median, 12 % at most
// up to three strips per CU).
const Build kBuilds[] = {
    Q8_BNECK(256, 1, 3, 2, 3, 3, 2, 2, 11.4f, 0.25f, 1.3f, 0.0f, 1.0f, 0.36f),
    Q8_BNECK(256, 1, 2, 1, 2, 4, 2, 2, 7.7f, 0.24f, 0.92f, 0.0f, 1.0f, 0.37f),
    Q8_BNECK(128, 2, 3, 2, 2, 3, 2, 2, 8.1f, 0.3f, 1.25f, 0.0f, 1.0f, 0.34f),
    Q8_BNECK(128, 2, 2, 1, 2, 3, 2, 2, 6.2f, 0.15f, 0.8f, 0.0f, 1.0f, 0.27f),
    Q8_BNECK(64, 2, 4, 2, 2, 2, 1, 3, 5.4f, 0.28f, 0.9f, 0.42f, 0.6f, 0.05f),
    Q8_BNECK(64, 2, 3, 1, 2, 2, 1, 4, 4.3f, 0.24f, 0.65f, 0.55f, 0.5f, 0.05f),
};
#undef Q8_BNECK
constexpr int kNumBuilds = sizeof(kBuilds) / sizeof(kBuilds[0]);

struct Range {
  const char* lo;
  const char* hi;
};
Range range(const void* p, long bytes) { return {(const char*)p, (const char*)p + bytes}; }
bool apart(Range a, Range b) { return a.hi <= b.lo || b.hi <= a.lo; }

}  // namespace

int num_bneck_builds() { return kNumBuilds; }
const char* bneck_build_name(int build) { return kBuilds[build].name; }

// Whether the three layers form a block that one launch can take, whatever the build: shapes, tensors
// that follow one another, aligned rows, and outputs apart from everything the launch reads (a
// workgroup writes its pixels while another one still reads the rows beside them).
bool bneck_applicable(const ConvParams& a, const ConvParams& b, const ConvParams& c) {
  const int mid = a.K;
  if (mid != 64 && mid != 128 && mid != 256) return false;
  if (a.S4 || a.R != 1 || a.S != 1 || a.pad_h || a.pad_w || a.C % 64 || a.res) return false;
  if (b.R != 3 || b.S != 3 || b.stride_h != 1 || b.stride_w != 1 || b.pad_h != 1 || b.pad_w != 1 || b.dil_h != 1 ||
      b.dil_w != 1 || b.C != mid || b.K != mid || b.res)
    return false;
  if (c.R != 1 || c.S != 1 || c.stride_h != 1 || c.stride_w != 1 || c.pad_h || c.pad_w || c.C != mid || c.K % mid)
    return false;
  if (b.N != a.N || b.H != a.Ho || b.W != a.Wo || c.N != a.N || c.H != b.Ho || c.W != b.Wo) return false;
  if (b.x != a.y + a.out_off || b.in_cs != a.out_cs || c.x != b.y + b.out_off || c.in_cs != b.out_cs) return false;
  for (const ConvParams* p : {&a, &b, &c})
    if (p->acc_dump || p->y_f32 || p->y_deq || p->w2 || !p->vec16 || (long)p->M * p->out_cs >= 0x7fffffffL)
      return false;
  // (the codes between the layers are handed over as they are stored)
  if (a.out_u8 != b.in_u8 || b.out_u8 != c.in_u8) return false;
  if (c.res && (c.res_bytes <= 0 || (long)c.M * c.res_cs >= 0x7fffffffL)) return false;
  const Range reads[] = {range(a.x, a.x_bytes), range(a.w, a.w_bytes), range(b.w, b.w_bytes), range(c.w, c.w_bytes),
                         range(a.bias, a.bias ? 4L * a.K : 0), range(b.bias, b.bias ? 4L * b.K : 0),
                         range(c.bias, c.bias ? 4L * c.K : 0), range(c.res, c.res ? c.res_bytes : 0),
                         range(a.m_vec, a.m_vec ? 4L * a.K : 0), range(b.m_vec, b.m_vec ? 4L * b.K : 0),
                         range(c.m_vec, c.m_vec ? 4L * c.K : 0),
                         range(b.tap_sums, b.tap_sums ? 4L * 256 * b.K : 0)};
  const Range writes[] = {range(a.y, (long)a.M * a.out_cs), range(b.y, (long)b.M * b.out_cs),
                          range(c.y, (long)c.M * c.out_cs)};
  for (int i = 0; i < 3; ++i) {
    for (const Range& r : reads)
      if (r.lo && !apart(writes[i], r)) return false;
    for (int j = 0; j < i; ++j)
      if (!apart(writes[i], writes[j])) return false;
  }
  return true;
}

// Strips of whole rows: as many as the build's tiles hold, evenly many per strip.  0: not one.
static int bneck_rows(const Build& s, int H, int W) {
  int rows = s.bp / W;
  if (s.ap / W - 2 < rows) rows = s.ap / W - 2;
  if (rows < 1) return 0;
  if (rows > H) rows = H;
  const int strips = (H + rows - 1) / rows;
  return (H + strips - 1) / strips;
}
static int bneck_lds(const Build& s, int W, int K2, bool ext, int rows, int* params_off, int* tile_off) {
  int tile = s.xbuf;
  const int codes_a = (rows + 2) * ((W + 2) * s.pitch + s.row_pad), codes_b = s.bp * s.pitch;
  if (codes_a > tile) tile = codes_a;
  if (codes_b > tile) tile = codes_b;
  const auto whole = [](int k) { return (k * 4 + 1023) & ~1023; };
  *params_off = s.ring;
  *tile_off = s.ring + (2 * whole(s.mid) + whole(K2)) * (ext ? 2 : 1);
  return *tile_off + tile;
}

bool bneck_build_takes(int build, const ConvParams& a, const ConvParams& b, const ConvParams& c) {
  const Build& s = kBuilds[build];
  const int rows = a.K == s.mid && a.C % s.piece == 0 ? bneck_rows(s, b.H, b.W) : 0;
  int po, to;
  const bool ext = is_extended(a) || is_extended(b) || is_extended(c);
  return rows > 0 && c.K <= 8192 && bneck_lds(s, b.W, c.K, ext, rows, &po, &to) <= kLdsLimit &&
         (long)a.N * ((b.H + rows - 1) / rows) < 0x7fffffffL;
}

// The build estimated shortest, -1: none takes the block.
int pick_bneck(const ConvParams& a, const ConvParams& b, const ConvParams& c, float* us) {
  int best = -1;
  for (int i = 0; i < kNumBuilds; ++i) {
    const Build& s = kBuilds[i];
    if (!bneck_build_takes(i, a, b, c)) continue;
    const int rows = bneck_rows(s, b.H, b.W);
    const float strips = (float)((long)a.N * ((b.H + rows - 1) / rows)) / 256.0f, r = ceilf(strips);
    const float strip = s.base + s.per_step * (float)(a.C / 64) + s.per_round * (float)(c.K / s.mid);
    const float t = strip * (s.u + s.v * r + s.w * strips / r);
    if (best < 0 || t < *us) {
      best = i;
      *us = t;
    }
  }
  return best;
}

int launch_bneck(int build, const ConvParams& a, const ConvParams& b, const ConvParams& c, hipStream_t stream) {
  const Build& s = kBuilds[build];
  BneckParams q{};
  q.x = a.x; q.wa = a.w; q.wb = b.w; q.wc = c.w; q.res = c.res;
  q.ya = a.y; q.yb = b.y; q.yc = c.y;
  q.bias_a = a.bias; q.bias_b = b.bias; q.bias_c = c.bias; q.tap_sums = b.tap_sums;
  const auto tail = [](const ConvParams& p) { return BneckTail{p.m, p.m_r, p.relu, p.out_u8, p.res_u8, p.m_vec}; };
  q.a = tail(a); q.b = tail(b); q.c = tail(c);
  q.x_bytes = a.x_bytes;
  q.x_image = a.H * a.W * a.in_cs;
  q.x_row = a.stride_h * a.W * a.in_cs;
  q.x_pixel = a.stride_w * a.in_cs;
  q.wa_bytes = a.w_bytes; q.wb_bytes = b.w_bytes; q.wc_bytes = c.w_bytes; q.res_bytes = c.res_bytes;
  q.C = a.C; q.K2 = c.K; q.H = b.H; q.W = b.W; q.M = b.M;
  q.ya_cs = a.out_cs; q.ya_off = a.out_off; q.yb_cs = b.out_cs; q.yb_off = b.out_off;
  q.yc_cs = c.out_cs; q.yc_off = c.out_off; q.res_cs = c.res_cs; q.res_off = c.res_off;
  q.rows = bneck_rows(s, b.H, b.W);
  q.strips = (b.H + q.rows - 1) / q.rows;
  q.div_row_m = b.div_row_m; q.div_row_s = b.div_row_s;
  const FastDiv div = make_fast_div((unsigned)q.strips);
  q.div_strips_m = div.m;
  q.div_strips_s = div.s;
  const bool ext = is_extended(a) || is_extended(b) || is_extended(c);
  const int lds = bneck_lds(s, b.W, c.K, ext, q.rows, &q.params_off, &q.tile_off);
  return s.launch[ext](q, (unsigned)(a.N * q.strips), lds, stream);
}

}  // namespace q8
