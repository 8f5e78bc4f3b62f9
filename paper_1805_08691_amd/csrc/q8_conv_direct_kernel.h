// Latency family of the int8 convolution (Eq. x / Eq. A' of arxiv 1805.08691): layers with few
// output tiles (small batches, small maps), where a launch is a chain of latencies -- kernel
// arguments, addresses, one trip to memory, the reduction, the store -- and not a rate.
//
// What bounds such a layer in the tiled kernels is the bytes ONE compute unit has to pull (30 per
// clock and CU) times the length of its chain of reduction steps: 7 x 7 x 512 3x3 on one image is
// 8 tiles of 64 x 64 with 590 KB each, 9 us on 8 of 256 CUs.  Here the output tile is as small as
// 16 x 16, so that the chip is filled, and the reduction of a tile is shared by KW wavefronts
// (Eq. x: integer sums regroup freely), each taking every KW-th 64-byte step.  Fragments go
// straight from memory into the MFMA's registers (v_mfma_i32_16x16x64_i8 wants 16 rows x 64 bytes,
// which is one load of a wavefront): no LDS, no barrier, up to NB steps requested before the
// first is used.  Partial sums meet in LDS once, and the tail is spread over the wavefronts.
//
// The kernel is kept small and is the same for every layer of a network's late part: cold
// instruction fetches count at this scale.
#pragma once
#include <type_traits>
#include "q8_common.h"
#include "q8_conv_common.h"

namespace q8 {

// What the kernel needs of ConvParams, in the order it needs it.
struct DirectParams {
  const int8_t* x;
  const int8_t* w;
  int x_bytes, w_bytes;
  int M, K, red_len, C;
  int H, W, in_cs, S;
  int Wo, HoWo, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w;
  FastDiv by_img, by_row, by_c, by_s;
  int n_ptiles, n_ctiles, ptile_fastest;
  int R, mode;                    // mode: the addressing build the layer takes in a group
  int start_bytes, res_bytes;     // descriptor sizes: start values (bias or table), residual
  const int32_t* bias;
  const int8_t* res;
  int8_t* y;
  float m, m_r;
  int relu, out_cs, out_off, res_cs, res_off;
  int vec4, f32_vec4, in_u8, out_u8, res_u8;
  const int32_t* tap_sums;
  const float* m_vec;
  float* y_f32;
  float* y_deq;
  float q_deq;
  int32_t* acc_dump;
};

// Independent layers in one launch: workgroup b belongs to the last layer l with first[l] <= b.
constexpr int kMaxGroup = 8;
struct DirectGroup {
  int n;
  int first[kMaxGroup];
  DirectParams layer[kMaxGroup];
};

namespace {

#if defined(__HIP_DEVICE_COMPILE__)
// Tail of Eq. A' for four consecutive channels [ch, ch + 4) of one pixel: v = accumulators
// (bias included).
__device__ __forceinline__ void direct_tail(const DirectParams& p, int pix, int ch, const v4i& v,
                                            unsigned res_word, const v4i& scale) {
  const int nvalid = p.K - ch;
  const size_t o = (size_t)pix * p.out_cs + p.out_off + ch;
  float t[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = (float)v[e] * __int_as_float(scale[e]);
  if (p.acc_dump) {
    int32_t* d = p.acc_dump + (size_t)pix * p.K + ch;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < nvalid) d[e] = v[e];
  }
  if (p.res) {
    const int add = p.res_u8 ? 128 : 0;            // stored byte + 128 = unsigned code
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float u = (float)((int)(int8_t)((res_word >> (8 * e)) & 0xff) + add) * p.m_r;
      t[e] = t[e] + u;
    }
  }
  if (p.y_f32) {                                   // Eq. D only: no clamp, no Round
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (p.relu) t[e] = fmaxf(t[e], 0.0f);
    if (p.f32_vec4 && nvalid >= 4) {
      *reinterpret_cast<float4*>(p.y_f32 + o) = float4{t[0], t[1], t[2], t[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nvalid) p.y_f32[o + e] = t[e];
    }
    return;
  }
  const float lo = (p.relu || p.out_u8) ? 0.0f : -128.0f, hi = p.out_u8 ? 255.0f : 127.0f;
  const int sub = p.out_u8 ? 128 : 0;              // unsigned code - 128 = stored byte
  int code[4];
  unsigned word = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    code[e] = (int)rintf(fminf(fmaxf(t[e], lo), hi)) - sub;
    word |= ((unsigned)code[e] & 0xffu) << (8 * e);
  }
  if (p.y_deq) {                                   // Eq. D on the codes just made
    float d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = p.q_deq * (float)code[e];
    if (p.f32_vec4 && nvalid >= 4) {
      *reinterpret_cast<float4*>(p.y_deq + o) = float4{d[0], d[1], d[2], d[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nvalid) p.y_deq[o + e] = d[e];
    }
  }
  if (p.vec4 && nvalid >= 4) {
    *reinterpret_cast<unsigned*>(p.y + o) = word;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < nvalid) p.y[o + e] = (int8_t)code[e];
  }
}

// Row of the start-value table of a pixel (see u8_start_index).
__device__ __forceinline__ int direct_start_index(const DirectParams& p, int pix) {
  const int n = fast_div(pix, p.by_img.m, p.by_img.s), rem = pix - n * p.HoWo;
  const int ho = fast_div(rem, p.by_row.m, p.by_row.s);
  const int hi0 = ho * p.stride_h - p.pad_h, wi0 = (rem - ho * p.Wo) * p.stride_w - p.pad_w;
  int r_lo = p.R, r_hi = 0, s_lo = p.S, s_hi = 0;
  for (int r = 0; r < p.R; ++r)
    if ((unsigned)(hi0 + r * p.dil_h) < (unsigned)p.H) { r_lo = min(r_lo, r); r_hi = r + 1; }
  for (int s = 0; s < p.S; ++s)
    if ((unsigned)(wi0 + s * p.dil_w) < (unsigned)p.W) { s_lo = min(s_lo, s); s_hi = s + 1; }
  if (r_hi <= r_lo || s_hi <= s_lo) r_lo = r_hi = s_lo = s_hi = 0;
  return ((r_lo * (p.R + 1) + r_hi) * (p.S + 1) + s_lo) * (p.S + 1) + s_hi;
}

constexpr int kDirectOob = (int)0x80000000;

// One tile of TP*16 pixels x TC*16 channels by the KW wavefronts of a workgroup.  MODE 2: 1 x 1
// filter without padding, C % 64 == 0 (the step is a scalar offset); 1: C % 64 == 0, a 64-byte step
// lies in one tap; 0: every lane finds the tap of its own 16-byte chunk.
template <int TP, int TC, int KW, int NB, int MODE>
__device__ __forceinline__ void conv_tile_direct(const DirectParams& p, const int bid_in, int* const lds) {
  constexpr int U = TP * TC;                      // units of the tail: MFMA tiles
  constexpr int OWN = (U + KW - 1) / KW;          // ... of which wavefront w finishes w, w + KW, ...
  // every argument the addresses need in one batch of scalar loads
  asm volatile("" ::"s"(p.x), "s"(p.w), "s"(p.M), "s"(p.K), "s"(p.H), "s"(p.HoWo), "s"(p.by_img.m),
               "s"(p.n_ptiles));
  const int lane = threadIdx.x & 63, row = lane & 15, quarter = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = p.n_ptiles * p.n_ctiles;
  int bid = bid_in;
  {
    const int xcd = bid % kNumXcd, idx = bid / kNumXcd, base = nblk / kNumXcd, rem = nblk % kNumXcd;
    bid = xcd * base + (xcd < rem ? xcd : rem) + idx;
  }
  int ptile, ctile;
  if (p.ptile_fastest) { ctile = bid / p.n_ptiles; ptile = bid - ctile * p.n_ptiles; }
  else { ptile = bid / p.n_ctiles; ctile = bid - ptile * p.n_ctiles; }
  const int pix0 = ptile * TP * 16, ch0 = ctile * TC * 16;

  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, p.w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_x =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, p.x_bytes, 0x00020000);

  // rows of the tile are dealt to channels so that a lane's accumulators of the TC tiles are
  // 4 TC consecutive channels of one pixel
  int a_off[TC];
#pragma unroll
  for (int i = 0; i < TC; ++i) {
    const int ch = ch0 + (row >> 2) * 4 * TC + i * 4 + (row & 3);
    a_off[i] = ch < p.K ? ch * p.red_len + quarter * 16 : kDirectOob;
  }
  int hi0[TP], wi0[TP], base[TP];
#pragma unroll
  for (int j = 0; j < TP; ++j) {
    const int pix = pix0 + j * 16 + row;
    hi0[j] = -(1 << 29);                          // beyond M: every tap outside the image
    wi0[j] = 0;
    base[j] = kDirectOob;
    if (pix < p.M) {
      const int n = fast_div(pix, p.by_img.m, p.by_img.s);
      const int rem = pix - n * p.HoWo;
      const int ho = fast_div(rem, p.by_row.m, p.by_row.s);
      hi0[j] = ho * p.stride_h - p.pad_h;
      wi0[j] = (rem - ho * p.Wo) * p.stride_w - p.pad_w;
      base[j] = ((n * p.H + hi0[j]) * p.W + wi0[j]) * p.in_cs + (MODE ? quarter * 16 : 0);
    }
  }
  const int nk = (p.red_len + 63) >> 6;
  v4i af[NB][TC], bf[NB][TP];
  auto load_step = [&](int st, auto buf_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value;
    // Steps behind the last one read filter values from beyond the descriptor, zeros.  Their scalar
    // offset is that of the first step: whichever way the range check counts a scalar offset, none
    // leads behind a pixel's channels or a filter.
    const int step_off = st < nk ? st * 64 : 0;
    if constexpr (MODE == 0) {
      const int k = st * 64 + quarter * 16;       // the lane's own 16-byte chunk and its tap
      const int tap = fast_div(k, p.by_c.m, p.by_c.s), c = k - tap * p.C;
      const int r = fast_div(tap, p.by_s.m, p.by_s.s), s = tap - r * p.S;
      const int dh = r * p.dil_h, dw = s * p.dil_w, delta = (dh * p.W + dw) * p.in_cs + c;
      const bool k_in = k < p.red_len;
#pragma unroll
      for (int j = 0; j < TP; ++j) {
        int off = base[j] + delta;
        asm volatile("" : "+v"(off));             // a select below, no branch
        const bool in = k_in & ((unsigned)(hi0[j] + dh) < (unsigned)p.H) &
                        ((unsigned)(wi0[j] + dw) < (unsigned)p.W);
        bf[BUF][j] = __builtin_bit_cast(
            v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, in ? off : kDirectOob, 0, 0));
      }
#pragma unroll
      for (int i = 0; i < TC; ++i)
        af[BUF][i] = __builtin_bit_cast(
            v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, k_in ? a_off[i] : kDirectOob, step_off, 0));
    } else {
      if constexpr (MODE == 2) {
#pragma unroll
        for (int j = 0; j < TP; ++j)
          bf[BUF][j] = __builtin_bit_cast(
              v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, base[j], step_off, 0));
      } else {
        const int tap = fast_div(st * 64, p.by_c.m, p.by_c.s), c = st * 64 - tap * p.C;
        const int r = fast_div(tap, p.by_s.m, p.by_s.s), s = tap - r * p.S;
        const int dh = r * p.dil_h, dw = s * p.dil_w, delta = (dh * p.W + dw) * p.in_cs + c;
#pragma unroll
        for (int j = 0; j < TP; ++j) {
          int off = base[j] + delta;
          asm volatile("" : "+v"(off));
          const bool in = (st < nk) & ((unsigned)(hi0[j] + dh) < (unsigned)p.H) &
                          ((unsigned)(wi0[j] + dw) < (unsigned)p.W);
          bf[BUF][j] = __builtin_bit_cast(
              v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, in ? off : kDirectOob, 0, 0));
        }
      }
#pragma unroll
      for (int i = 0; i < TC; ++i)
        af[BUF][i] = __builtin_bit_cast(
            v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, st < nk ? a_off[i] : kDirectOob, step_off, 0));
    }
  };
  v4i acc[TC][TP];
#pragma unroll
  for (int i = 0; i < TC; ++i)
#pragma unroll
    for (int j = 0; j < TP; ++j) acc[i][j] = v4i{0, 0, 0, 0};
  auto mma_step = [&](auto buf_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value;
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[BUF][i], bf[BUF][j], acc[i][j], 0, 0, 0);
  };
  using std::integral_constant;
  auto each_buf = [&](auto fn) __attribute__((always_inline)) {
    auto rec = [&](auto self, auto b_c) __attribute__((always_inline)) -> void {
      constexpr int BUF = decltype(b_c)::value;
      if constexpr (BUF < NB) {
        fn(b_c);
        self(self, integral_constant<int, BUF + 1>{});
      }
    };
    rec(rec, integral_constant<int, 0>{});
  };
  // The first NB steps of this wavefront are requested at once.  A wavefront with more of them
  // keeps NB in flight (steps behind the last add nothing, so the loop issues the same loads on
  // every path and its waits are exact); one with fewer issues what it has.
  // (may be zero or negative: nothing to do)
  const int n_mine = (nk - wave + KW - 1) / KW;
  each_buf([&](auto b_c) __attribute__((always_inline)) {
    if (decltype(b_c)::value < n_mine) load_step(wave + decltype(b_c)::value * KW, b_c);
  });

  // The tail's operands, requested behind the first operands: start values (the bias, or the
  // pixel's row of the table of start values), scales, residual codes.  Always issued, through
  // descriptors that read zeros where there is nothing.
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(p.tap_sums ? p.tap_sums : p.bias), 0, p.start_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_r =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.res, 0, p.res_bytes, 0x00020000);
  v4i start[OWN], scale[OWN];
  unsigned res_word[OWN];
#pragma unroll
  for (int k = 0; k < OWN; ++k) {
    const int u = wave + k * KW;
    const int ch = ch0 + quarter * 4 * TC + u / TP * 4, pix = pix0 + u % TP * 16 + row;
    const bool in = (ch < p.K) & (pix < p.M);
    const int idx = p.tap_sums && in ? direct_start_index(p, pix) : 0;
    start[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                                           rsrc_b, in ? (idx * p.K + ch) * 4 : kDirectOob, 0, 0));
    res_word[k] = __builtin_amdgcn_raw_buffer_load_b32(
        rsrc_r, in ? pix * p.res_cs + p.res_off + ch : kDirectOob, 0, 0);
  }
  if (p.m_vec) {
    const __amdgpu_buffer_rsrc_t rsrc_m =
        __builtin_amdgcn_make_buffer_rsrc((void*)p.m_vec, 0, p.K * 4, 0x00020000);
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const int ch = ch0 + quarter * 4 * TC + (wave + k * KW) / TP * 4;
      scale[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_m, ch * 4, 0, 0));
    }
  } else {
#pragma unroll
    for (int k = 0; k < OWN; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) scale[k][e] = __float_as_int(p.m);
  }

  if (n_mine > NB) {
    wait_vmcnt<0>();                 // (the conditional requests above leave no exact count)
    int k0 = 0;
    for (; k0 + NB < n_mine; k0 += NB)
      each_buf([&](auto b_c) __attribute__((always_inline)) {
        mma_step(b_c);
        load_step(wave + (k0 + decltype(b_c)::value + NB) * KW, b_c);
      });
    each_buf([&](auto b_c) __attribute__((always_inline)) { mma_step(b_c); });
  } else {
    each_buf([&](auto b_c) __attribute__((always_inline)) {
      if (decltype(b_c)::value < n_mine) mma_step(b_c);
    });
  }

#pragma unroll
  for (int u = 0; u < U; ++u)
    *reinterpret_cast<v4i*>(lds + ((u * KW + wave) * 64 + lane) * 4) = acc[u / TP][u % TP];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < OWN; ++k) {
    const int u = wave + k * KW;
    if (u >= U) break;
    v4i v = {0, 0, 0, 0};
#pragma unroll
    for (int g = 0; g < KW; ++g) v += *reinterpret_cast<const v4i*>(lds + ((u * KW + g) * 64 + lane) * 4);
    const int ch = ch0 + quarter * 4 * TC + u / TP * 4, pix = pix0 + u % TP * 16 + row;
    if (ch < p.K && pix < p.M) direct_tail(p, pix, ch, v + start[k], res_word[k], scale[k]);
  }
}
#endif  // __HIP_DEVICE_COMPILE__

template <int TP, int TC, int KW, int NB, int MODE>
__global__ __launch_bounds__(KW * 64) void conv_i8_direct_kernel(const DirectParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(16))) int lds[TP * TC * KW * 256];
  conv_tile_direct<TP, TC, KW, NB, MODE>(p, blockIdx.x, lds);
#endif
}

template <int TP, int TC, int KW, int NB>
__global__ __launch_bounds__(KW * 64) void conv_i8_direct_group_kernel(const DirectGroup g) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(16))) int lds[TP * TC * KW * 256];
  int l = 0;
  for (int i = 1; i < g.n; ++i) l = (int)blockIdx.x >= g.first[i] ? i : l;
  const DirectParams& p = g.layer[l];
  const int bid = blockIdx.x - g.first[l];
  if (p.mode == 2) conv_tile_direct<TP, TC, KW, NB, 2>(p, bid, lds);
  else if (p.mode == 1) conv_tile_direct<TP, TC, KW, NB, 1>(p, bid, lds);
  else conv_tile_direct<TP, TC, KW, NB, 0>(p, bid, lds);
#endif
}

}  // namespace
}  // namespace q8
