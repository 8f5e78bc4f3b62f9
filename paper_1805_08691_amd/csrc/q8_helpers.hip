// Pooling helpers that only chain layers or feed calibration; none of them is part of the
// quantised arithmetic of arxiv 1805.08691.
#include "q8_common.h"
#include "q8_conv_common.h"

namespace {

constexpr int kThreads = 256;

template <typename T>
__device__ __forceinline__ T lowest();
template <>
__device__ __forceinline__ int8_t lowest<int8_t>() { return -128; }
template <>
__device__ __forceinline__ float lowest<float>() { return -3.402823466e38f; }

template <typename T>
__global__ __launch_bounds__(kThreads) void maxpool_kernel(const T* __restrict__ x, int N, int H,
                                                           int W, int C, int R, int S, int stride,
                                                           int pad, int Ho, int Wo,
                                                           T* __restrict__ y) {
  const size_t total = (size_t)N * Ho * Wo * C;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (size_t)gridDim.x * kThreads) {
    int c = (int)(i % C);
    size_t t = i / C;
    int wo = (int)(t % Wo); t /= Wo;
    int ho = (int)(t % Ho);
    int n = (int)(t / Ho);
    T best = lowest<T>();
    for (int r = 0; r < R; ++r) {
      int hi = ho * stride - pad + r;
      if ((unsigned)hi >= (unsigned)H) continue;
      for (int s = 0; s < S; ++s) {
        int wi = wo * stride - pad + s;
        if ((unsigned)wi >= (unsigned)W) continue;
        T v = x[(((size_t)n * H + hi) * W + wi) * C + c];
        best = v > best ? v : best;
      }
    }
    y[i] = best;
  }
}

typedef int v4i __attribute__((ext_vector_type(4)));
typedef short v2s __attribute__((ext_vector_type(2)));

// Workgroups go to the 8 XCDs round robin: renumber them so that each XCD owns one contiguous run of
// outputs.  Neighbouring output rows share input rows; with this they find them in their own L2 instead of
// fetching them once per XCD.
__device__ __forceinline__ unsigned xcd_run(unsigned bid, unsigned grid) {
  const unsigned xcd = bid % 8, idx = bid / 8, base = grid / 8, rem = grid % 8;
  return xcd * base + (xcd < rem ? xcd : rem) + idx;
}

// int8 pooling over WIN x WIN windows (MODE 0: maximum, 1: mean), 16 channels a
// lane and NO outputs of one row: the input columns that neighbouring windows share are loaded and
// reduced over the window's rows once.  A lane for every output was bound by its instructions, not by the
// bytes: three divisions by run-time numbers, nine addresses, nine selects of a neutral element, nine taps taken
// apart.  Here
//  * divisions are multiplications; a tap's address is one addition of a row and a column offset;
//  * nothing is selected.  Mean: a tap outside the image lies outside the buffer and reads as zeros.
//    Maximum: the taps' rows and columns are clamped into the image, and the clamped one lies in the
//    window too (every window holds a pixel of the image), so a tap comes twice;
//  * mean: bytes + 128, two to a word in 16-bit lanes, add up without carries (9 x 255); maximum: a word's
//    odd bytes are compared in place, whatever the bytes under them, and the even ones shifted up by eight.
// Before and after, us: 3 x 3 mean, 32 images of 35 x 35 x 288 11.8 / 7.5, 17 x 17 x 768 8.3 / 5.4, 8 x 8 x 2048
// 5.5 / 4.1 (one image of 35 x 35 x 288: 2.9 / 2.6); maximum 3 x 3, 64 images of 19 x 19 x 512 11.3 / 6.5; stride 2, 64
// images of 112 x 112 x 64 11.6 / 11.2 (5.8 TB/s); 2 x 2, 64 images of 300 x 300 x 64 89.7 / 81.9 (5.6 TB/s),
// one of 75 x 75 x 256 2.65 / 1.90.
struct PoolParams {
  int H, W, stride, pad_h, pad_w, Ho, Wo, C;      // C: channels = bytes of a pixel
  int x_bytes;
  unsigned total;                                 // lanes with work
  q8::FastDiv by_c, by_strip, by_row;             // of C / 16, strips of a row, rows
  int strips;
  float m, inv_count;
  int8_t* y;
  int out_cs, out_off;
};
#pragma clang fp contract(off)
template <int MODE, int WIN, int NO>
__global__ __launch_bounds__(kThreads) void pool_strip_kernel(const int8_t* __restrict__ x, const PoolParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int COLS = NO - 1 + WIN;
  const int stride = NO == 1 ? p.stride : 1;
  const unsigned i = xcd_run(blockIdx.x, gridDim.x) * kThreads + threadIdx.x;
  if (i >= p.total) return;
  const int t = q8::fast_div((int)i, p.by_c.m, p.by_c.s), c = ((int)i - t * (p.C >> 4)) << 4;
  const int u = q8::fast_div(t, p.by_strip.m, p.by_strip.s), wo = (t - u * p.strips) * NO;
  const int n = q8::fast_div(u, p.by_row.m, p.by_row.s), ho = u - n * p.Ho;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, p.x_bytes, 0x00020000);
  unsigned row[WIN], col[COLS];
#pragma unroll
  for (int r = 0; r < WIN; ++r) {
    const int h = ho * stride - p.pad_h + r;
    const int hc = MODE == 0 ? min(max(h, 0), p.H - 1) : h;
    row[r] = (unsigned)((n * p.H + hc) * p.W) * (unsigned)p.C;
    // beyond a mean's buffer of less than 2^30 bytes, and still so with either kind of column offset
    if (MODE == 1 && (unsigned)h >= (unsigned)p.H) row[r] = 0x40000000u;
  }
#pragma unroll
  for (int k = 0; k < COLS; ++k) {
    const int w = wo * stride - p.pad_w + k;
    const int wc = MODE == 0 ? min(max(w, 0), p.W - 1) : w;
    col[k] = (unsigned)(wc * p.C + c);
    if (MODE == 1 && (unsigned)w >= (unsigned)p.W) col[k] = 0x80000000u;
  }
  v4i tap[COLS][WIN];
#pragma unroll
  for (int k = 0; k < COLS; ++k)
#pragma unroll
    for (int r = 0; r < WIN; ++r)
      tap[k][r] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(row[r] + col[k]), 0, 0));
  // a column over the window's rows: odd and even bytes in 16-bit lanes
  unsigned odd[COLS][4], even[COLS][4];
  auto most = [](unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(v2s, a), __builtin_bit_cast(v2s, b)));
  };
#pragma unroll
  for (int k = 0; k < COLS; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < WIN; ++r) {
        const unsigned v = (unsigned)tap[k][r][q] ^ (MODE == 0 ? 0u : 0x80808080u);
        const unsigned o = MODE == 0 ? v : __builtin_amdgcn_perm(0u, v, 0x0c030c01u);
        const unsigned e = MODE == 0 ? v << 8 : v & 0x00ff00ffu;
        odd[k][q] = r == 0 ? o : MODE == 0 ? most(odd[k][q], o) : odd[k][q] + o;
        even[k][q] = r == 0 ? e : MODE == 0 ? most(even[k][q], e) : even[k][q] + e;
      }
  int8_t* const y = p.y + (((size_t)n * p.Ho + ho) * p.Wo + wo) * p.out_cs + p.out_off + c;
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    v4i out;
    unsigned so[4], se[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      so[q] = odd[k][q];
      se[q] = even[k][q];
#pragma unroll
      for (int s = 1; s < WIN; ++s) {
        so[q] = MODE == 0 ? most(so[q], odd[k + s][q]) : so[q] + odd[k + s][q];
        se[q] = MODE == 0 ? most(se[q], even[k + s][q]) : se[q] + even[k + s][q];
      }
    }
    if (MODE == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) out[q] = (int)__builtin_amdgcn_perm(so[q], se[q], 0x07030501u);
      if (p.m != 1.0f) {
        float f[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) f[e] = (float)(int8_t)((out[e >> 2] >> (8 * (e & 3))) & 0xff) * p.m;
        out = q8::pack16_signed(f);
      }
    } else if (WIN == 3 && p.m == 1.0f) {
      // A ninth of a whole number is 1/18 or more away from where Round changes, the fp32 product within
      // 4e-5 of it: 128 may be added before as well as behind.
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        unsigned w = 0;
        w = __builtin_amdgcn_cvt_pk_u8_f32((float)(se[q] & 0xffffu) * p.inv_count, 0, w);
        w = __builtin_amdgcn_cvt_pk_u8_f32((float)(so[q] & 0xffffu) * p.inv_count, 1, w);
        w = __builtin_amdgcn_cvt_pk_u8_f32((float)(se[q] >> 16) * p.inv_count, 2, w);
        w = __builtin_amdgcn_cvt_pk_u8_f32((float)(so[q] >> 16) * p.inv_count, 3, w);
        out[q] = (int)(w ^ 0x80808080u);
      }
    } else {
      float f[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f[4 * q + 0] = (float)((int)(se[q] & 0xffffu) - 128 * WIN * WIN) * p.inv_count;
        f[4 * q + 1] = (float)((int)(so[q] & 0xffffu) - 128 * WIN * WIN) * p.inv_count;
        f[4 * q + 2] = (float)((int)(se[q] >> 16) - 128 * WIN * WIN) * p.inv_count;
        f[4 * q + 3] = (float)((int)(so[q] >> 16) - 128 * WIN * WIN) * p.inv_count;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) f[e] = f[e] * p.m;
      out = q8::pack16_signed(f);
    }
    if (wo + k < p.Wo) *reinterpret_cast<v4i*>(y + (size_t)k * p.out_cs) = out;
  }
#endif
}

// General int8 pooling into a channel slice with a change of factor (see q8_pool_i8).
#pragma clang fp contract(off)
__global__ __launch_bounds__(kThreads) void pool_i8_kernel(const int8_t* __restrict__ x, int N, int H,
                                                           int W, int C, int mode, int R, int S,
                                                           int stride, int pad, int Ho, int Wo,
                                                           float m, float inv_count,
                                                           int8_t* __restrict__ y, int out_cs,
                                                           int out_off) {
  const size_t total = (size_t)N * Ho * Wo * C;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (size_t)gridDim.x * kThreads) {
    int c = (int)(i % C);
    size_t t = i / C;
    int wo = (int)(t % Wo); t /= Wo;
    int ho = (int)(t % Ho);
    int n = (int)(t / Ho);
    int best = -128, sum = 0;
    for (int r = 0; r < R; ++r) {
      int hi = ho * stride - pad + r;
      if ((unsigned)hi >= (unsigned)H) continue;
      for (int s2 = 0; s2 < S; ++s2) {
        int wi = wo * stride - pad + s2;
        if ((unsigned)wi >= (unsigned)W) continue;
        int v = x[(((size_t)n * H + hi) * W + wi) * C + c];
        best = v > best ? v : best;
        sum += v;
      }
    }
    float f = mode == 0 ? (float)best : (float)sum * inv_count;
    f = f * m;
    f = fminf(fmaxf(f, -128.0f), 127.0f);
    y[(((size_t)n * Ho + ho) * Wo + wo) * out_cs + out_off + c] = (int8_t)(int)rintf(f);
  }
}

// The same with 16 channels per lane (C, out_cs and out_off multiples of 16, 16-byte aligned tensors), any
// window: 16-byte loads and one 16-byte store, taps outside the image skipped.
template <int MODE>
__global__ __launch_bounds__(kThreads) void pool_i8_vec_kernel(const int8_t* __restrict__ x, int N,
                                                               int H, int W, int C16, int R,
                                                               int S, int stride, int pad, int Ho,
                                                               int Wo, float m, float inv_count,
                                                               int8_t* __restrict__ y, int out_cs,
                                                               int out_off) {
  // 32-bit index arithmetic: the host takes this kernel only below 2^31 items
  const unsigned total = (unsigned)N * Ho * Wo * C16;
  const unsigned bid = xcd_run(blockIdx.x, gridDim.x);
  for (unsigned i = bid * kThreads + threadIdx.x; i < total; i += gridDim.x * kThreads) {
    int c = (int)(i % (unsigned)C16);
    unsigned t = i / (unsigned)C16;
    int wo = (int)(t % (unsigned)Wo); t /= (unsigned)Wo;
    int ho = (int)(t % (unsigned)Ho);
    int n = (int)(t / (unsigned)Ho);
    // Two bytes per 32-bit word at a time, as 16-bit lanes.  Maximum: as in the strips.  Mean: the odd bytes
    // and the even bytes, each sign-extended by a packed arithmetic shift (a window of at most 128 taps cannot
    // overflow 16 bits).
    v2s acc_odd[4], acc_even[4];
    const short init = MODE == 0 ? (short)-32768 : (short)0;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc_odd[q] = acc_even[q] = v2s{init, init};
    auto take = [&](const v4i& v) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int w = v[q], w8 = w << 8;
        const v2s odd = __builtin_bit_cast(v2s, w), even = __builtin_bit_cast(v2s, w8);
        if (MODE == 0) {
          acc_odd[q] = __builtin_elementwise_max(acc_odd[q], odd);
          acc_even[q] = __builtin_elementwise_max(acc_even[q], even);
        } else {
          acc_odd[q] += odd >> 8;              // bytes 1 and 3
          acc_even[q] += even >> 8;            // bytes 0 and 2
        }
      }
    };
    for (int r = 0; r < R; ++r) {
      int hi = ho * stride - pad + r;
      if ((unsigned)hi >= (unsigned)H) continue;
      for (int s2 = 0; s2 < S; ++s2) {
        int wi = wo * stride - pad + s2;
        if ((unsigned)wi >= (unsigned)W) continue;
        take(*reinterpret_cast<const v4i*>(x + ((((size_t)n * H + hi) * W + wi) * C16 + c) * 16));
      }
    }
    v4i o = {};
    float f[16];
    if (MODE == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v2s odd = acc_odd[q], even = acc_even[q];
        o[q] = (int)__builtin_amdgcn_perm(__builtin_bit_cast(unsigned, odd), __builtin_bit_cast(unsigned, even),
                                          0x07030501u);
      }
    }
    if (MODE == 1 || m != 1.0f) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int sum = (e & 1) ? acc_odd[e >> 2][(e >> 1) & 1] : acc_even[e >> 2][(e >> 1) & 1];
        f[e] = MODE == 0 ? (float)(int8_t)((o[e >> 2] >> (8 * (e & 3))) & 0xff) : (float)sum * inv_count;
        f[e] = f[e] * m;
      }
      o = q8::pack16_signed(f);
    }
    *reinterpret_cast<v4i*>(y + (((size_t)n * Ho + ho) * Wo + wo) * out_cs + out_off + c * 16) = o;
  }
}

// fp32 twin for the calibration forward (max, or mean with padding counted as zeros).
__global__ __launch_bounds__(kThreads) void pool_f32_kernel(const float* __restrict__ x, int N, int H,
                                                            int W, int C, int mode, int R, int S,
                                                            int stride, int pad, int Ho, int Wo,
                                                            float* __restrict__ y, int out_cs,
                                                            int out_off) {
  const size_t total = (size_t)N * Ho * Wo * C;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (size_t)gridDim.x * kThreads) {
    int c = (int)(i % C);
    size_t t = i / C;
    int wo = (int)(t % Wo); t /= Wo;
    int ho = (int)(t % Ho);
    int n = (int)(t / Ho);
    float best = -3.402823466e38f, sum = 0.f;
    for (int r = 0; r < R; ++r) {
      int hi = ho * stride - pad + r;
      if ((unsigned)hi >= (unsigned)H) continue;
      for (int s2 = 0; s2 < S; ++s2) {
        int wi = wo * stride - pad + s2;
        if ((unsigned)wi >= (unsigned)W) continue;
        float v = x[(((size_t)n * H + hi) * W + wi) * C + c];
        best = fmaxf(best, v);
        sum += v;
      }
    }
    y[(((size_t)n * Ho + ho) * Wo + wo) * out_cs + out_off + c] =
        mode == 0 ? best : sum / (float)(R * S);
  }
}

// The same with four channels per lane, one output each: 16-byte accesses and divisions by multiplication; the values
// are taken in the same order.  Bound by memory.  3x3 maximum on 112 x 112 x 64 x 8 images 18.6 us with a value per
// lane, 9.3 so; the thirteen poolings of Inception-v3 on 8 images 231 and 120.
__global__ __launch_bounds__(kThreads) void pool_f32_vec_kernel(const float4* __restrict__ x, unsigned items, int H,
                                                                int W, int C4, int mode, int R, int S, int stride,
                                                                int pad, int Ho, int Wo, q8::FastDiv by_c,
                                                                q8::FastDiv by_wo, q8::FastDiv by_ho,
                                                                float4* __restrict__ y, int out_cs4, int out_off4) {
  const unsigned i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= items) return;
  const unsigned pix = (unsigned)q8::fast_div((int)i, by_c.m, by_c.s), c = i - pix * (unsigned)C4;
  const unsigned row = (unsigned)q8::fast_div((int)pix, by_wo.m, by_wo.s);
  const int wo = (int)(pix - row * (unsigned)Wo), n = q8::fast_div((int)row, by_ho.m, by_ho.s);
  const int h0 = ((int)row - n * Ho) * stride - pad, w0 = wo * stride - pad;
  const float4* const img = x + (size_t)n * H * W * C4 + c;
  constexpr float kLowest = -3.402823466e38f;
  float4 best{kLowest, kLowest, kLowest, kLowest}, sum{0.f, 0.f, 0.f, 0.f};
  for (int r = 0; r < R; ++r) {
    if ((unsigned)(h0 + r) >= (unsigned)H) continue;
    for (int s = 0; s < S; ++s) {
      if ((unsigned)(w0 + s) >= (unsigned)W) continue;
      const float4 v = img[((size_t)(h0 + r) * W + (w0 + s)) * C4];
      best = {fmaxf(best.x, v.x), fmaxf(best.y, v.y), fmaxf(best.z, v.z), fmaxf(best.w, v.w)};
      sum = {sum.x + v.x, sum.y + v.y, sum.z + v.z, sum.w + v.w};
    }
  }
  const float count = (float)(R * S);
  y[(size_t)pix * out_cs4 + out_off4 + c] =
      mode == 0 ? best : float4{sum.x / count, sum.y / count, sum.z / count, sum.w / count};
}

// int8 pooling with 16 channels per lane; false: not for these channels, addresses or sizes.
bool pool_i8_vec_launch(const int8_t* x, int N, int H, int W, int C, int mode, int R, int S, int stride,
                        int pad, int Ho, int Wo, float m, int8_t* y, int out_cs, int out_off, void* stream) {
  const size_t total = (size_t)N * Ho * Wo * C;
  if (C % 16 || out_cs % 16 || out_off % 16 || !q8_aligned(x, 16) || !q8_aligned(y, 16) ||
      (mode == 1 && R * S > 128) || total / 16 >= 0x7fffffffUL)
    return false;
  const float inv_count = 1.0f / (float)(R * S);
  // Strips: 3 x 3 windows and the maximum over 2 x 2, with any stride.  A tap's offset takes 31 bits, and a mean's
  // buffer ends where the taps outside the image are sent, so larger tensors go image by image or in bands of
  // rows.  (As the kernel for any window: 3 x 3 with stride 3 on one image of 35 x 35 x 288 4.3 us instead of 2.6.)
  // Two outputs a lane where windows share columns and more than three wavefronts of one output would
  // stand on a SIMD, one otherwise: one and two, 3 x 3 mean, one image of 35 x 35 x 288 2.61 / 2.96, eight
  // 3.52 / 3.79 (196608 outputs of 16 channels 3.58 / 3.80, 262144 4.06 / 3.96), 64 12.3 / 11.1; with four 64 take
  // 10.8; with two at stride 2 64 images of 112 x 112 x 64 12.5 instead of 11.2.
  const size_t row = (size_t)W * C, image = row * H, reach = mode == 0 ? 0x7fffffffUL : 0x40000000UL;
  const bool three = R == 3 && S == 3, two = R == 2 && S == 2 && mode == 0;
  if ((three || two) && (image < reach || row * (size_t)R < reach)) {
    const int no = three && stride == 1 && total / 16 > 3 * 1024 * 64 ? 2 : 1;
    auto kernel = two ? pool_strip_kernel<0, 2, 1>
                  : no == 2 ? (mode == 0 ? pool_strip_kernel<0, 3, 2> : pool_strip_kernel<1, 3, 2>)
                            : (mode == 0 ? pool_strip_kernel<0, 3, 1> : pool_strip_kernel<1, 3, 1>);
    const int images = image < reach ? (int)((reach - 1) / image) : 1;
    const int band = image < reach ? Ho : (int)(((reach - 1) / row - R) / stride) + 1;
    for (int n = 0; n < N; n += images)
      for (int ho = 0; ho < Ho; ho += band) {
        const int first = ho * stride - pad, top = first > 0 ? first : 0;      // the launch's first row of the image
        PoolParams p;
        p.H = H - top; p.W = W; p.stride = stride; p.pad_h = top - first; p.pad_w = pad;
        p.Ho = Ho - ho < band ? Ho - ho : band; p.Wo = Wo; p.C = C;
        const int some = N - n < images ? N - n : images;
        const size_t bytes = (some - 1) * image + (size_t)p.H * row;
        p.x_bytes = (int)(bytes < reach ? bytes : reach - 1);
        p.strips = (Wo + no - 1) / no;
        p.total = (unsigned)((size_t)some * p.Ho * p.strips * (C / 16));
        p.by_c = q8::make_fast_div((unsigned)(C / 16));
        p.by_strip = q8::make_fast_div((unsigned)p.strips);
        p.by_row = q8::make_fast_div((unsigned)p.Ho);
        p.m = m; p.inv_count = inv_count;
        p.y = y + ((size_t)n * Ho + ho) * Wo * out_cs;
        p.out_cs = out_cs; p.out_off = out_off;
        hipLaunchKernelGGL(kernel, dim3((p.total + kThreads - 1) / kThreads), dim3(kThreads), 0,
                           (hipStream_t)stream, x + (size_t)n * image + (size_t)top * row, p);
      }
    return true;
  }
  size_t vb = (total / 16 + kThreads - 1) / kThreads;
  if (vb > 65536) vb = 65536;
  hipLaunchKernelGGL((mode == 0 ? pool_i8_vec_kernel<0> : pool_i8_vec_kernel<1>), dim3((unsigned)vb),
                     dim3(kThreads), 0, (hipStream_t)stream, x, N, H, W, C / 16, R, S, stride, pad, Ho, Wo,
                     m, inv_count, y, out_cs, out_off);
  return true;
}

template <typename T>
int maxpool_launch(const T* x, int N, int H, int W, int C, int R, int S, int stride, int pad,
                   int Ho, int Wo, T* y, void* stream) {
  Q8_REQUIRE(N >= 0 && H >= 1 && W >= 1 && C >= 1 && R >= 1 && S >= 1 && stride >= 1 && pad >= 0 &&
                 Ho >= 0 && Wo >= 0, Q8_EINVAL);
  // every window must hold at least one in-image tap
  Q8_REQUIRE(pad < R && pad < S, Q8_EINVAL);
  Q8_REQUIRE(Ho == 0 || (long)(Ho - 1) * stride - pad < H, Q8_EINVAL);
  Q8_REQUIRE(Wo == 0 || (long)(Wo - 1) * stride - pad < W, Q8_EINVAL);
  size_t total = (size_t)N * Ho * Wo * C;
  if (total == 0) return Q8_OK;
  Q8_REQUIRE(x && y, Q8_EINVAL);
  if constexpr (sizeof(T) == 1) {
    if (pool_i8_vec_launch((const int8_t*)x, N, H, W, C, 0, R, S, stride, pad, Ho, Wo, 1.0f, (int8_t*)y, C, 0,
                           stream))
      return q8_launch_status();
  }
  size_t blocks = (total + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(maxpool_kernel<T>, dim3((unsigned)blocks), dim3(kThreads), 0,
                     (hipStream_t)stream, x, N, H, W, C, R, S, stride, pad, Ho, Wo, y);
  return q8_launch_status();
}

// Register-resident i8 MFMA loop: what the matrix cores sustain with no operand traffic
// (four independent accumulator chains per wave, four waves per block).
typedef int probe_v4i __attribute__((ext_vector_type(4)));
typedef int probe_v16i __attribute__((ext_vector_type(16)));
__global__ __launch_bounds__(256) void mfma_i8_probe_kernel(int iters, int32_t* sink) {
  probe_v4i a = {(int)threadIdx.x, 1, 2, 3}, b = {4, 5, 6, (int)blockIdx.x};
  probe_v16i c0 = {0}, c1 = {0}, c2 = {0}, c3 = {0};
  for (int i = 0; i < iters; ++i) {
    c0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c1, 0, 0, 0);
    c2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c2, 0, 0, 0);
    c3 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c3, 0, 0, 0);
  }
  int s = 0;
  for (int i = 0; i < 16; ++i) s += c0[i] + c1[i] + c2[i] + c3[i];
  if (s == 0x12345678) sink[0] = s;      // keeps the loop alive; practically never taken
}

}  // namespace

extern "C" {

int q8_maxpool_i8(const int8_t* x_dev, int N, int H, int W, int C, int R, int S, int stride, int pad,
                  int Ho, int Wo, int8_t* y_dev, void* stream) {
  return maxpool_launch<int8_t>(x_dev, N, H, W, C, R, S, stride, pad, Ho, Wo, y_dev, stream);
}
int q8_pool_i8(const int8_t* x_dev, int N, int H, int W, int C, int mode, int R, int S, int stride,
               int pad, int Ho, int Wo, float q_in, float q_out, int8_t* y_dev, int out_c_stride,
               int out_c_off, void* stream) {
  Q8_REQUIRE(q8_finite_pos(q_in) && q8_finite_pos(q_out), Q8_EINVAL);
  const float m = q_in / q_out;        // the rescale of Eq. A' between two factors, one fp32 division
  Q8_REQUIRE(N >= 0 && H >= 1 && W >= 1 && C >= 1 && R >= 1 && S >= 1 && stride >= 1 && pad >= 0 &&
                 Ho >= 0 && Wo >= 0 && (mode == 0 || mode == 1), Q8_EINVAL);
  Q8_REQUIRE(pad < R && pad < S && q8_finite_pos(m), Q8_EINVAL);
  Q8_REQUIRE(Ho == 0 || (long)(Ho - 1) * stride - pad < H, Q8_EINVAL);
  Q8_REQUIRE(Wo == 0 || (long)(Wo - 1) * stride - pad < W, Q8_EINVAL);
  Q8_REQUIRE(out_c_off >= 0 && out_c_stride >= out_c_off + C, Q8_EINVAL);
  size_t total = (size_t)N * Ho * Wo * C;
  if (total == 0) return Q8_OK;
  Q8_REQUIRE(x_dev && y_dev, Q8_EINVAL);
  const float inv_count = 1.0f / (float)(R * S);
  if (pool_i8_vec_launch(x_dev, N, H, W, C, mode, R, S, stride, pad, Ho, Wo, m, y_dev, out_c_stride,
                         out_c_off, stream))
    return q8_launch_status();
  size_t blocks = (total + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(pool_i8_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, (hipStream_t)stream,
                     x_dev, N, H, W, C, mode, R, S, stride, pad, Ho, Wo, m, inv_count, y_dev,
                     out_c_stride, out_c_off);
  return q8_launch_status();
}

int q8_pool_f32(const float* x_dev, int N, int H, int W, int C, int mode, int R, int S, int stride,
                int pad, int Ho, int Wo, float* y_dev, int out_c_stride, int out_c_off, void* stream) {
  Q8_REQUIRE(N >= 0 && H >= 1 && W >= 1 && C >= 1 && R >= 1 && S >= 1 && stride >= 1 && pad >= 0 &&
                 Ho >= 0 && Wo >= 0 && (mode == 0 || mode == 1), Q8_EINVAL);
  Q8_REQUIRE(pad < R && pad < S, Q8_EINVAL);
  Q8_REQUIRE(Ho == 0 || (long)(Ho - 1) * stride - pad < H, Q8_EINVAL);
  Q8_REQUIRE(Wo == 0 || (long)(Wo - 1) * stride - pad < W, Q8_EINVAL);
  Q8_REQUIRE(out_c_off >= 0 && out_c_stride >= out_c_off + C, Q8_EINVAL);
  size_t total = (size_t)N * Ho * Wo * C;
  if (total == 0) return Q8_OK;
  Q8_REQUIRE(x_dev && y_dev, Q8_EINVAL);
  if (C % 4 == 0 && out_c_stride % 4 == 0 && out_c_off % 4 == 0 && q8_aligned(x_dev, 16) && q8_aligned(y_dev, 16) &&
      total / 4 <= 0x7fffff00UL) {
    const unsigned items = (unsigned)(total / 4);
    hipLaunchKernelGGL(pool_f32_vec_kernel, dim3((items + kThreads - 1) / kThreads), dim3(kThreads), 0,
                       (hipStream_t)stream, reinterpret_cast<const float4*>(x_dev), items, H, W, C / 4, mode, R, S,
                       stride, pad, Ho, Wo, q8::make_fast_div((unsigned)C / 4), q8::make_fast_div((unsigned)Wo),
                       q8::make_fast_div((unsigned)Ho), reinterpret_cast<float4*>(y_dev), out_c_stride / 4,
                       out_c_off / 4);
    return q8_launch_status();
  }
  size_t blocks = (total + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(pool_f32_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, (hipStream_t)stream,
                     x_dev, N, H, W, C, mode, R, S, stride, pad, Ho, Wo, y_dev, out_c_stride,
                     out_c_off);
  return q8_launch_status();
}

int q8_maxpool_f32(const float* x_dev, int N, int H, int W, int C, int R, int S, int stride, int pad,
                   int Ho, int Wo, float* y_dev, void* stream) {
  return maxpool_launch<float>(x_dev, N, H, W, C, R, S, stride, pad, Ho, Wo, y_dev, stream);
}

int q8_probe_mfma_i8(int blocks, int iters, int32_t* sink_dev, void* stream) {
  Q8_REQUIRE(blocks >= 1 && blocks <= 65536 && iters >= 1 && iters <= (1 << 22) && sink_dev,
             Q8_EINVAL);
  hipLaunchKernelGGL(mfma_i8_probe_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     (hipStream_t)stream, iters, sink_dev);
  return q8_launch_status();
}

}  // extern "C"
