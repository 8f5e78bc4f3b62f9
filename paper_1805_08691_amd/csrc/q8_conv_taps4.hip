// The register-fed tile family of the int8 convolution (Eq. x / Eq. A' of arxiv 1805.08691): a
// network's first layer with up to four taps per filter row and four filter rows, over a 4-channel
// image that carries its own padding as a zero frame, K <= 64 output channels (a detector's 3x3
// on 300 x 300, Inception-v3's 3x3 / 2 on 299 x 299).
//
// Four taps x four channels are 16 bytes, half the depth of a 32 x 32 x 32 MFMA, and the 16 bytes that an output
// pixel reads of image row r are contiguous: lane (pixel, half h) loads those of row h into the operand's register
// layout as they lie in memory, then those of row 2 + h.  Every filter (two chunks of 16 bytes a channel) and the bias
// stay in registers, so there is no LDS and no barrier; a wavefront walks over runs of 32 pixels and requests
// the next run's bytes before it computes this one.  Taps beyond S (the next row's bytes, zeros past the tensor) and
// rows beyond R (the last row again) meet filter bytes that are zero.
//
// What bounds it: the stores, 64 bytes a pixel for 4 loaded (the caches serve a row's other two readings), and behind
// them the vector instructions, four for each code.  A lane has 16 consecutive channels of a pixel from either channel
// tile, runs of 32 bytes 64 apart; v_permlane16_swap exchanges them so that a store instruction writes 16 whole
// pixels, 1 KB in one run.  32 images, the general kernel and this one: 300 x 300 -> 64 channels 69.1 and 38.4 us
// (4.8 TB/s written), 149 x 149 -> 32 channels 18.0 and 8.7; two images 8.0 and 6.1.
#include "q8_conv_ring_kernel.h"

namespace q8 {
namespace {

// TC: channel tiles of 32.
template <int TC, int EXT>
__global__ __launch_bounds__(256, EXT ? 2 : 4) void conv_i8_taps4_kernel(const ConvParams p, int n_tiles) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, p.w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc((void*)p.y, 0, p.M * p.out_cs, 0x00020000);

  v4i af[TC][2];
  v16i bias_v[TC];
  float scales[TC][16] = {};
#pragma unroll
  for (int tc = 0; tc < TC; ++tc) {
    const int ch = tc * 32 + row_to_channel(col);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 2 * j + half;
      af[tc][j] = __builtin_amdgcn_raw_buffer_load_b128(
          rsrc_w, ch < p.K && r < p.R ? ch * p.red_len + r * 16 : kOobOffset, 0, 0);
    }
    int b[16];
    load_bias16(p, tc * 32 + 16 * half, b);
#pragma unroll
    for (int e = 0; e < 16; ++e) bias_v[tc][e] = b[e];
    if (EXT && p.m_vec) load_scale16(p, tc * 32 + 16 * half, scales[tc]);
  }

  // Pixel (n, ho, wo) of this lane and the byte its first tap lies at; a run further on all of them grow by
  // constants, with a carry from wo to ho and from ho to n: fewer and shorter instructions than two divisions.
  const int row_bytes = p.W * 4, step = gridDim.x * 4;
  const int r0 = min(half, p.R - 1) * row_bytes, r1 = min(2 + half, p.R - 1) * row_bytes;
  int tile = blockIdx.x * 4 + wave;
  int ho, wo;
  unsigned off;
  auto place = [&](int pix, int& h, int& w) {
    const int n = fast_div(pix, p.div_img_m, p.div_img_s), rem = pix - n * (p.Ho * p.Wo);
    h = fast_div(rem, p.div_row_m, p.div_row_s);
    w = rem - h * p.Wo;
    return (unsigned)(n * p.H + h * p.stride_h) * (unsigned)row_bytes + (unsigned)(w * p.stride_w) * 4u;
  };
  off = place(tile * 32 + col, ho, wo);
  int dh, dw;
  const unsigned d_off = __builtin_amdgcn_readfirstlane(place(step * 32, dh, dw));
  dh = __builtin_amdgcn_readfirstlane(dh);
  dw = __builtin_amdgcn_readfirstlane(dw);
  const unsigned d_row = (unsigned)p.stride_h * (unsigned)row_bytes - (unsigned)(p.Wo * p.stride_w) * 4u;
  const unsigned d_img = (unsigned)(p.H - p.Ho * p.stride_h) * (unsigned)row_bytes;
  auto load = [&](v4i (&x)[2]) {
    x[0] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, (int)(off + r0), 0, 0);
    x[1] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, (int)(off + r1), 0, 0);
  };
  // where this lane's stores go: pixel and first channel in a run (a pixel beyond M lies beyond the descriptor)
  const int st_col = TC == 2 ? lane & 15 : col, st_ch = TC == 2 ? (lane >> 5) * 16 + (lane >> 4 & 1) * 32 : half * 16;
  const unsigned st = st_ch < p.K ? (unsigned)(st_col * p.out_cs + p.out_off + st_ch) : 0x80000000u;

  auto run = [&](v4i (&x)[2], v4i (&next)[2]) {
    if (tile + step < n_tiles) {
      wo += dw;
      const bool row = wo >= p.Wo;
      wo -= row ? p.Wo : 0;
      ho += dh + (row ? 1 : 0);
      const bool img = ho >= p.Ho;
      ho -= img ? p.Ho : 0;
      off += d_off + (row ? d_row : 0u) + (img ? d_img : 0u);
      load(next);
    }
    v4i out[TC];
#pragma unroll
    for (int tc = 0; tc < TC; ++tc) {
      v16i acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[tc][0], x[0], bias_v[tc], 0, 0, 0);
      acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[tc][1], x[1], acc, 0, 0, 0);
      float t[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) t[e] = (float)acc[e] * (EXT && p.m_vec ? scales[tc][e] : p.m);
      if (EXT && p.out_u8) {
        out[tc] = pack16_nonneg(t, false, 255.0f);
#pragma unroll
        for (int a = 0; a < 4; ++a) out[tc][a] ^= 0x80808080;       // unsigned codes minus 128
      } else {
        out[tc] = p.relu ? pack16_nonneg(t, true, 127.0f) : pack16_signed(t);
      }
    }
    if constexpr (TC == 2) {        // rows of 16 lanes: 1 and 3 of the first with 0 and 2 of the second
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const auto s = __builtin_amdgcn_permlane16_swap((unsigned)out[0][a], (unsigned)out[1][a], false, false);
        out[0][a] = (int)s[0];
        out[1][a] = (int)s[1];
      }
    }
#pragma unroll
    for (int tc = 0; tc < TC; ++tc)
      __builtin_amdgcn_raw_buffer_store_b128(out[tc], rsrc_y, (int)(st + (unsigned)((tile * 32 + tc * 16) * p.out_cs)),
                                             0, 0);
    tile += step;
  };
  v4i xa[2], xb[2];
  load(xa);
  while (tile < n_tiles) {
    run(xa, xb);
    if (tile >= n_tiles) break;
    run(xb, xa);
  }
#endif
}

template <int TC, int EXT>
int launch_tiles(ConvParams& p, hipStream_t stream) {
  const int n_tiles = (int)((p.M + 31L) / 32), groups = (n_tiles + 3) / 4, most = 256 * (EXT ? 2 : 4);
  hipLaunchKernelGGL((conv_i8_taps4_kernel<TC, EXT>), dim3((unsigned)(groups < most ? groups : most)), dim3(256), 0,
                     stream, p, n_tiles);
  return q8_launch_status();
}

bool taps4_applicable(const ConvParams& p) {
  return p.S4 == 1 && p.S == 1 && p.C == 16 && p.in_cs == 4 && p.R <= 4 && p.K <= 64 && (p.K & 15) == 0 &&
         p.pad_h == 0 && p.pad_w == 0 && p.vec16 && !p.res && !p.acc_dump && !p.y_f32 && !p.y_deq && !p.in_u8 &&
         !p.res_u8 && !p.w2 && !p.tap_sums && (p.M + 32L) * p.out_cs < 0x7fffffffL;
}

}  // namespace

int launch_taps4_or_generic(ConvParams& p, hipStream_t stream) {
  const bool ext = is_extended(p);
  if (!taps4_applicable(p) || (ext && p.K <= 32))
    return ext ? launch_ring_ext_variant(8, p, stream) : launch_ring<2, 2, 2, 1, 64, 2, 0>(p, stream);
  if (p.K <= 32) return launch_tiles<1, 0>(p, stream);         // (extended: the host keeps to K > 32)
  return ext ? launch_tiles<2, 1>(p, stream) : launch_tiles<2, 0>(p, stream);
}

}  // namespace q8
