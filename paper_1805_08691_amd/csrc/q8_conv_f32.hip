// fp32 NHWC convolution + bias (+ residual) (+ ReLU): the forward that produces the real-valued
// activations calibration measures, with the max-abs of what it computes taken on the way.
// A helper around the quantised path, not part of it.
//
// This file: the register-fed builds, for channel counts and alignments that those on LDS and on the
// bf16 instructions (q8_conv_f32_lds.hip, q8_conv_f32_split.hip) do not take, and the host side.
// What bounds them: on large layers the fp32 matrix rate (122 of the 153 TF a library product of 8192 x 8192 x 8192
// reaches, 28 x 28 x 512 3x3 at batch 64); on small maps the operand loads, 11 to 14 bytes per clock and CU.  16 reduction bytes
// per lane feed four MFMAs of 32 clocks, so a wavefront loads its fragments straight into the MFMA's
// register layout (16 rows x 64 bytes a load), two stages ahead of the one it computes: no LDS and no
// barrier inside the loop.  ResNet-50 calibration on 8 images: 13.9 ms with the max-abs as passes over
// every tensor, 1.78 ms with these builds alone and an atomic per wavefront, 1.11 ms now.
//
// Small maps have few tiles (7 x 7 at batch 8: 392 pixels): KW groups of wavefronts then share
// the stages of one tile and add their accumulators through LDS in a fixed order.
#include "q8_conv_f32.h"

namespace q8 {
namespace {

// WP x WC wavefronts, each TP x TC MFMA tiles of 16 pixels x 16 channels; NC chunks of 64 bytes per
// row and stage, NB stages in registers.
// MODE 2: C % (16 NC) == 0, a stage lies in one tap; 1: C % 4 == 0, a 16-byte chunk lies
// in one tap; 0: any C, four single loads per chunk.
template <int WP, int WC, int TP, int TC, int KW, int NC, int NB, int MODE>
__global__ __launch_bounds__(WP * WC * KW * 64, 2) void conv_f32_mfma_kernel(const F32Params p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BP = WP * TP * 16, BC = WC * TC * 16, NW = WP * WC;
  constexpr int kXch = KW > 1 ? (KW - 1) * NW * TP * TC * 256 : 4;
  __shared__ __attribute__((aligned(16))) float xch[kXch];
  const int nblk = p.n_ptiles * p.n_ctiles;
  int bid = blockIdx.x;
  {   // every XCD takes a contiguous run of tiles, channel tile fastest (shared activations)
    const int xcd = bid % kNumXcd, idx = bid / kNumXcd, base = nblk / kNumXcd, rem = nblk % kNumXcd;
    bid = xcd * base + (xcd < rem ? xcd : rem) + idx;
  }
  const int ptile = bid / p.n_ctiles, ctile = bid - ptile * p.n_ctiles;
  const int pix0 = ptile * BP, ch0 = ctile * BC;
  const int lane = threadIdx.x & 63, row = lane & 15, quarter = lane >> 4;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kgroup = KW > 1 ? wave_all / NW : 0, wave = KW > 1 ? wave_all % NW : wave_all;
  const int wave_p = wave % WP, wave_c = wave / WP;

  // the activation descriptor starts at the tile's first image: offsets stay below 2^31
  // whatever the batch (the host checks the span of a tile's images)
  const int n0 = fast_div(pix0, p.by_img.m, p.by_img.s);
  const long img = (long)p.H * p.W * p.C;
  const long x_left = ((long)p.N - n0) * img * 4;
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(p.x + n0 * img), 0, (int)(x_left < 0x7fffffffL ? x_left : 0x7fffffffL), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, p.K * p.rsc * 4, 0x00020000);

  int a_off[TC];
#pragma unroll
  for (int i = 0; i < TC; ++i) {
    // rows are dealt to channels so that a lane's accumulators of the TC tiles are 4 TC
    // consecutive channels of one pixel
    const int ch = ch0 + wave_c * TC * 16 + (row >> 2) * 4 * TC + i * 4 + (row & 3);
    a_off[i] = ch < p.K ? ch * p.rsc * 4 + quarter * 16 : kOob;
  }
  int hi0[TP], wi0[TP], base[TP];
#pragma unroll
  for (int j = 0; j < TP; ++j) {
    const int pix = pix0 + (wave_p * TP + j) * 16 + row;
    hi0[j] = -(1 << 29);               // a pixel beyond M: every tap outside the image
    wi0[j] = base[j] = 0;
    if (pix < p.M) {
      const int n = fast_div(pix, p.by_img.m, p.by_img.s);
      const int rem = pix - n * (p.Ho * p.Wo);
      const int ho = fast_div(rem, p.by_row.m, p.by_row.s);
      hi0[j] = ho * p.sh - p.ph;
      wi0[j] = (rem - ho * p.Wo) * p.sw - p.pw;
      base[j] = (((n - n0) * p.H + hi0[j]) * p.W + wi0[j]) * p.C;
    }
  }

  v4f acc[TC][TP];
#pragma unroll
  for (int i = 0; i < TC; ++i)
#pragma unroll
    for (int j = 0; j < TP; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

  v4f af[NB][NC][TC], bf[NB][NC][TP];    // fragments of the stage computed and of NB - 1 in flight
  auto tap_offset = [&](int kidx, int j) {   // byte offset of reduction index kidx for row j
    const int tap = fast_div(kidx, p.by_c.m, p.by_c.s), c = kidx - tap * p.C;
    const int r = fast_div(tap, p.by_s.m, p.by_s.s), s = tap - r * p.S;
    const bool in = (kidx < p.rsc) & ((unsigned)(hi0[j] + r * p.dh) < (unsigned)p.H) &
                    ((unsigned)(wi0[j] + s * p.dw) < (unsigned)p.W);
    return in ? (base[j] + (r * p.dh * p.W + s * p.dw) * p.C + c) * 4 : kOob;
  };
  // Always issues the same number of loads (a stage behind the last one reads zeros), so the
  // waits in front of the MFMAs count exactly the loads of the stage they need.
  const int n_st = (p.rsc + NC * 16 - 1) / (NC * 16);
  auto load_stage = [&](int st, auto buf_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value;
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        // behind the end of a filter stands the next one, whose values must not meet this one's
        // sums, not even times zero (an infinity there)
        const int left = MODE == 2 ? 4 : p.rsc - (st * NC + c) * 16 - quarter * 4;
        const bool in = (st < n_st) & (left > 0);
        if constexpr (MODE != 0) {
          af[BUF][c][i] = __builtin_bit_cast(
              v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, (in ? a_off[i] : kOob) + c * 64,
                                                         st * NC * 64, 0));
        } else {
          // the 16 bytes may end behind the last filter: the whole offset in the vector operand,
          // which is what the range check compares with the descriptor's size, dword by dword
          af[BUF][c][i] = __builtin_bit_cast(
              v4f, __builtin_amdgcn_raw_buffer_load_b128(
                       rsrc_w, in ? a_off[i] + (st * NC + c) * 64 : kOob, 0, 0));
#pragma unroll
          for (int e = 1; e < 4; ++e) af[BUF][c][i][e] = e < left ? af[BUF][c][i][e] : 0.0f;
        }
      }
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      if constexpr (MODE == 2) {
        const int tap = fast_div(st * NC * 16, p.by_c.m, p.by_c.s), c0 = st * NC * 16 - tap * p.C;
        const int r = fast_div(tap, p.by_s.m, p.by_s.s), s = tap - r * p.S;
        const int delta = (r * p.dh * p.W + s * p.dw) * p.C + c0;
        int off = (base[j] + delta) * 4 + quarter * 16;
        asm volatile("" : "+v"(off));      // a select, no branch: the stage stays one region
        const bool in = (st < n_st) & ((unsigned)(hi0[j] + r * p.dh) < (unsigned)p.H) &
                        ((unsigned)(wi0[j] + s * p.dw) < (unsigned)p.W);
        off = in ? off : kOob;
#pragma unroll
        for (int c = 0; c < NC; ++c)
          bf[BUF][c][j] = __builtin_bit_cast(
              v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, off + c * 64, 0, 0));
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int kidx = (st * NC + c) * 16 + quarter * 4;
          if constexpr (MODE == 1) {
            bf[BUF][c][j] = __builtin_bit_cast(
                v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, tap_offset(kidx, j), 0, 0));
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              bf[BUF][c][j][e] = __builtin_bit_cast(
                  float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_x, tap_offset(kidx + e, j), 0, 0));
          }
        }
      }
    }
  };
  auto mma_stage = [&](auto buf_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int j = 0; j < TP; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[BUF][c][i][e], bf[BUF][c][j][e],
                                                             acc[i][j], 0, 0, 0);
  };
  using std::integral_constant;
  auto prologue = [&](auto self, auto b_c) __attribute__((always_inline)) -> void {
    constexpr int BUF = decltype(b_c)::value;
    if constexpr (BUF < NB - 1) {
      load_stage(kgroup + BUF * KW, b_c);
      self(self, integral_constant<int, BUF + 1>{});
    }
  };
  prologue(prologue, integral_constant<int, 0>{});
  // The residual values of the units this wavefront finishes, requested together: inside the tail
  // they were one trip to memory behind another (64 -> 256 channels on 56 x 56 x 8: 16 trips).
  // Lanes outside the output read the tensor's first values.  Behind the first operands where the
  // registers allow it, else behind the last.
  constexpr int U = TC * TP, OWN = U / KW;       // units: see the tail
  static_assert(U % KW == 0, "every group owns the same number of units");
  const int u0 = kgroup * OWN;
  auto unit_ch = [&](int u) { return ch0 + wave_c * TC * 16 + quarter * 4 * TC + u / TP * 4; };
  auto unit_pix = [&](int u) { return pix0 + (wave_p * TP + u % TP) * 16 + row; };
  const bool vec_res = p.res && p.vec_y;         // (then K % 4 == 0)
  v4f res_v[OWN];
  auto load_res = [&]() __attribute__((always_inline)) {
    if (vec_res) {
#pragma unroll
      for (int k = 0; k < OWN; ++k) {
        const int ch = unit_ch(u0 + k), pix = unit_pix(u0 + k);
        res_v[k] = *reinterpret_cast<const v4f*>(p.res + (ch < p.K && pix < p.M ? (size_t)pix * p.K + ch : 0));
      }
    }
  };
  constexpr bool kEarlyRes = OWN <= 4;
  if constexpr (kEarlyRes) load_res();
  // Full passes over the NB buffers.  The loads of a stage are spread between the MFMAs of the
  // stage computed meanwhile: a wavefront issues in order, and with 32 rows a load the address
  // unit takes long enough that a burst of them would keep the matrix unit waiting.
  const int n_mine = (n_st - kgroup + KW - 1) / KW;
  int k0 = 0;
  for (; k0 + NB <= n_mine; k0 += NB) {
    auto pass = [&](auto self, auto b_c) __attribute__((always_inline)) -> void {
      constexpr int BUF = decltype(b_c)::value;
      if constexpr (BUF < NB) {
        load_stage(kgroup + (k0 + BUF + NB - 1) * KW, integral_constant<int, (BUF + NB - 1) % NB>{});
        mma_stage(b_c);
        if constexpr (MODE == 2) {
          constexpr int kLoads = NC * (TC + TP), kMma = NC * 4 * TC * TP;
#pragma unroll
          for (int g = 0; g < kLoads; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                     // one VMEM read
            __builtin_amdgcn_sched_group_barrier(0x008, kMma / kLoads, 0);         // MFMAs
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        self(self, integral_constant<int, BUF + 1>{});
      }
    };
    pass(pass, integral_constant<int, 0>{});
  }
  auto rest = [&](auto self, auto b_c) __attribute__((always_inline)) -> void {
    constexpr int BUF = decltype(b_c)::value;
    if constexpr (BUF < NB - 1) {
      if (k0 + BUF < n_mine) mma_stage(b_c);
      self(self, integral_constant<int, BUF + 1>{});
    }
  };
  rest(rest, integral_constant<int, 0>{});

  // Units of the tail: one MFMA tile, four consecutive channels of a pixel per lane.  With KW groups
  // every wavefront hands the units it does not own to their owners through LDS, adds up its
  // own share and finishes it, so the tail is spread over all of them.
  if constexpr (!kEarlyRes) load_res();
  v4f own[OWN], bias[OWN];
#pragma unroll
  for (int k = 0; k < OWN; ++k) {
    const int ch = unit_ch(u0 + k);
    bias[k] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    if (p.b) {
      if (p.vec_b && ch + 4 <= p.K) {
        bias[k] = *reinterpret_cast<const v4f*>(p.b + ch);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (ch + e < p.K) bias[k][e] = p.b[ch + e];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const v4f v = acc[u / TP][u % TP];
    const int owner = u / OWN;
    if (kgroup == owner) {
      own[u % OWN] = v;
    } else if constexpr (KW > 1) {
      const int slot = (wave * U + u) * (KW - 1) + (kgroup < owner ? kgroup : kgroup - 1);
      *reinterpret_cast<v4f*>(xch + (slot * 64 + lane) * 4) = v;
    }
  }
  if constexpr (KW > 1) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < OWN; ++k)
#pragma unroll
      for (int g = 0; g < KW - 1; ++g)
        own[k] += *reinterpret_cast<const v4f*>(xch + (((wave * U + u0 + k) * (KW - 1) + g) * 64 + lane) * 4);
  }

  float m_sum = 0.0f, m_out = 0.0f;
#pragma unroll
  for (int k = 0; k < OWN; ++k) {
    const int u = u0 + k, ch = unit_ch(u), nvalid = p.K - ch;
    const int pix = unit_pix(u);
    if (nvalid <= 0 || pix >= p.M) continue;
    float* y = p.y + (size_t)pix * p.out_cs + p.out_off + ch;
    v4f v = own[k] + bias[k];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < nvalid) m_sum = fmaxf(m_sum, fabsf(v[e]));
    const bool whole = p.vec_y && nvalid >= 4;
    if (vec_res) {
      v += res_v[k];
    } else if (p.res) {
      const float* res = p.res + (size_t)pix * p.K + ch;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nvalid) v[e] += res[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (p.relu) v[e] = fmaxf(v[e], 0.0f);
      if (e < nvalid) m_out = fmaxf(m_out, fabsf(v[e]));
    }
    if (whole) {
      *reinterpret_cast<v4f*>(y) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nvalid) y[e] = v[e];
    }
  }
  __shared__ float mx[2 * NW * KW];
  observe_block<NW * KW>(p, m_sum, m_out, mx);
#endif
}

// Any size: one thread per output value.  Only for tensors the 32-bit offsets above cannot
// address (an image or the filters beyond 2 GiB, 2^31 output pixels).
__global__ __launch_bounds__(kThreads) void conv_f32_any_kernel(const F32Params p) {
  const size_t total = (size_t)p.N * p.Ho * p.Wo * p.K;
  float m_sum = 0.0f, m_out = 0.0f;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (size_t)gridDim.x * kThreads) {
    const int k = (int)(i % p.K);
    const size_t pix = i / p.K;
    const int wo = (int)(pix % p.Wo), ho = (int)(pix / p.Wo % p.Ho);
    const size_t n = pix / p.Wo / p.Ho;
    float v = 0.0f;
    for (int r = 0; r < p.R; ++r) {
      const long hi = (long)ho * p.sh - p.ph + (long)r * p.dh;
      if (hi < 0 || hi >= p.H) continue;
      for (int s = 0; s < p.S; ++s) {
        const long wi = (long)wo * p.sw - p.pw + (long)s * p.dw;
        if (wi < 0 || wi >= p.W) continue;
        const float* x = p.x + ((n * p.H + hi) * p.W + wi) * p.C;
        const float* w = p.w + (((size_t)k * p.R + r) * p.S + s) * p.C;
        for (int c = 0; c < p.C; ++c) v = fmaf(x[c], w[c], v);
      }
    }
    if (p.b) v += p.b[k];
    m_sum = fmaxf(m_sum, fabsf(v));
    if (p.res) v += p.res[pix * p.K + k];
    if (p.relu) v = fmaxf(v, 0.0f);
    m_out = fmaxf(m_out, fabsf(v));
    p.y[pix * p.out_cs + p.out_off + k] = v;
  }
  __shared__ float mx[2 * kThreads / 64];
  observe_block<kThreads / 64>(p, m_sum, m_out, mx);
}

template <int WP, int WC, int TP, int TC, int KW, int NC, int NB>
int launch_f32(F32Params& p, hipStream_t stream) {
  p.n_ptiles = (p.M + WP * TP * 16 - 1) / (WP * TP * 16);
  p.n_ctiles = (p.K + WC * TC * 16 - 1) / (WC * TC * 16);
  const long nblk = (long)p.n_ptiles * p.n_ctiles;
  if (nblk > 0x7fffffffL) return Q8_EUNSUPPORTED;
  auto kernel = p.C % (16 * NC) == 0 ? conv_f32_mfma_kernel<WP, WC, TP, TC, KW, NC, NB, 2>
                : p.C % 4 == 0 ? conv_f32_mfma_kernel<WP, WC, TP, TC, KW, NC, NB, 1>
                               : conv_f32_mfma_kernel<WP, WC, TP, TC, KW, NC, NB, 0>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)nblk), dim3(WP * WC * KW * 64), 0, stream, p);
  return q8_launch_status();
}

// One wavefront per maximum: the largest of its copies.
__global__ __launch_bounds__(64) void fold_slots_kernel(const float* __restrict__ spread, int n_slots,
                                                        float* __restrict__ out) {
  float m = 0.0f;
  for (int j = threadIdx.x; j < n_slots; j += 64)
    m = fmaxf(m, spread[((size_t)blockIdx.x * n_slots + j) * kSlotStride]);
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  if (threadIdx.x == 0) out[blockIdx.x] = m;
}

// The builds of the tiled kernel; MODE follows from the channel count.
struct F32Build {
  int (*launch)(F32Params&, hipStream_t);
  int nc;
  const char* name[3];
};
#define Q8_F32_NAME(WP, WC, TP, TC, KW, NC, NB, MODE) \
  "conv_f32_mfma_kernel<" #WP "," #WC "," #TP "," #TC "," #KW "," #NC "," #NB "," #MODE ">"
#define Q8_F32_ROW(WP, WC, TP, TC, KW, NC, NB) \
  { &launch_f32<WP, WC, TP, TC, KW, NC, NB>, NC, \
    { Q8_F32_NAME(WP, WC, TP, TC, KW, NC, NB, 0), Q8_F32_NAME(WP, WC, TP, TC, KW, NC, NB, 1), \
      Q8_F32_NAME(WP, WC, TP, TC, KW, NC, NB, 2) } },
const F32Build kF32Builds[] = {
    Q8_F32_ROW(4, 1, 4, 4, 1, 1, 3)   // 0: 256 pixels x 64 channels
    Q8_F32_ROW(2, 2, 4, 4, 1, 1, 3)   // 1: 128 x 128
    Q8_F32_ROW(1, 1, 4, 4, 4, 1, 3)   // 2: 64 x 64, its reduction shared by four wavefronts
    Q8_F32_ROW(1, 1, 2, 2, 4, 2, 3)   // 3: 32 x 32, the same
};
#undef Q8_F32_ROW
#undef Q8_F32_NAME

// The largest tile that still gives every CU one; below that the tile is shared by four
// groups of wavefronts (their SIMDs), first 64 x 64, then 32 x 32 where those leave CUs idle.
// (Short reductions shared by two groups of a 128 x 64 tile, or by none of a 64 x 64 tile of four
// wavefronts, are slower: 128 -> 512 on 28 x 28 x 8 48 and 50 us against 38, the maxima's slots at
// zero.)
// Up to 64 channels and many tiles: no sharing, whose exchange of accumulators then costs more
// than it hides (7x7 on 224 x 224 x 8, 1568 tiles of 64 x 64: 64 -> 46 us).
int pick_f32(long M, int K) {
  auto tiles = [&](long t) { return (M + t - 1) / t * ((K + t - 1) / t); };
  if (K <= 64 && K > 32 && tiles(64) >= 1024) return 0;
  if (K > 64 && tiles(128) >= 256) return 1;
  return K > 32 && tiles(64) >= 192 ? 2 : 3;
}

bool f32_desc_sane(const q8_conv_desc* d) {
  return d && d->N >= 0 && d->H >= 1 && d->W >= 1 && d->C >= 1 && d->K >= 1 && d->R >= 1 &&
         d->S >= 1 && d->stride_h >= 1 && d->stride_w >= 1 && d->pad_h >= 0 &&
         d->pad_w >= 0 && d->dil_h >= 1 && d->dil_w >= 1;
}

// Bytes that one tile of at most 256 pixels can reach: its images and the padding rows around them.
long f32_reach(const q8_conv_desc* d, long per_img) {
  return (255 / per_img + 2) * ((long)d->H * d->W * d->C * 4) +
         ((long)d->R * d->dil_h + d->pad_h + 1) * ((long)d->W + (long)d->S * d->dil_w) * d->C * 4;
}

// Whether the tiled kernel's 32-bit offsets reach everything it addresses.
bool f32_tiled(const q8_conv_desc* d, long M, long per_img) {
  const long rsc = (long)d->R * d->S * d->C;
  return !(M > 0x7fffff00L || rsc * d->K * 4 > 0x7fffffffL || f32_reach(d, per_img) > 0x7fffffffL ||
           d->H > (1 << 28) || (long)d->R * d->dil_h > (1 << 28));
}

// Whether the padding fits the 32-bit offsets of the builds whose descriptor starts at the image's first tap, pad_h
// rows and pad_w pixels in front of it, on both sides of the map, its columns too, which the register-fed builds do not
// count (in a descriptor of more than 2^31 - 1 bytes the out-of-range offset would lie inside).
bool f32_pad_fits(const q8_conv_desc* d, long per_img) {
  return f32_reach(d, per_img) + ((long)d->pad_h * d->W + 2L * d->pad_w) * d->C * 4 <= 0x7fffffffL;
}
// Whether the builds on LDS take the layer: whole 128-byte pieces of a tap, whole groups of a lane's
// channels, output (residual, bias) rows of 16-byte accesses.
bool f32_lds_takes(const q8_conv_desc* d, long per_img, int out_cs, int out_off) {
  return d->C % 32 == 0 && d->K % 16 == 0 && out_cs % 4 == 0 && out_off % 4 == 0 && f32_pad_fits(d, per_img);
}

// The layer's build, among those on LDS (0 ..), the ones on the bf16 matrix instructions (-1), or register-fed (-2).
// aligned: activations and filters are; rows: so are output (residual, bias) rows.
int pick_f32_tiled(const q8_conv_desc* d, long M, long per_img, int out_cs, int out_off, bool aligned, bool rows) {
  if (!aligned || d->C % 16 || !f32_pad_fits(d, per_img)) return -2;
  const int rsc = d->R * d->S * d->C;
  const bool lds = rows && f32_lds_takes(d, per_img, out_cs, out_off);
  float us;
  const int build = pick_f32_lds(M, d->K, rsc, &us);
  return f32_split_pays(M, d->K, rsc, us, lds) ? -1 : lds ? build : -2;
}

int conv_f32(const q8_conv_desc* d, const float* x, const float* w, const float* b, const float* res,
             float* y, int out_cs, int out_off, float* obs_sum, float* obs_out, int n_slots, hipStream_t stream) {
  Q8_REQUIRE(f32_desc_sane(d), Q8_EINVAL);
  F32Params p{};
  p.Ho = q8_conv_out_h(d); p.Wo = q8_conv_out_w(d);
  const long M = (long)d->N * p.Ho * p.Wo;
  if (M == 0) return Q8_OK;
  Q8_REQUIRE(x && w && y && out_off >= 0 && out_cs >= out_off + d->K, Q8_EINVAL);
  p.x = x; p.w = w; p.b = b; p.res = res; p.y = y;
  p.obs_sum = reinterpret_cast<unsigned*>(obs_sum); p.obs_out = reinterpret_cast<unsigned*>(obs_out);
  p.n_slots = n_slots;
  p.N = d->N; p.H = d->H; p.W = d->W; p.C = d->C; p.K = d->K; p.R = d->R; p.S = d->S;
  p.sh = d->stride_h; p.sw = d->stride_w; p.ph = d->pad_h; p.pw = d->pad_w;
  p.dh = d->dil_h; p.dw = d->dil_w;
  p.out_cs = out_cs; p.out_off = out_off; p.relu = d->relu ? 1 : 0;
  p.vec_y = (out_cs % 4 == 0 && out_off % 4 == 0 && q8_aligned(y, 16) &&
             (!res || (d->K % 4 == 0 && q8_aligned(res, 16)))) ? 1 : 0;
  p.vec_b = q8_aligned(b, 16) ? 1 : 0;
  const long per_img = (long)p.Ho * p.Wo;
  if (!f32_tiled(d, M, per_img)) {
    const size_t total = (size_t)M * d->K;
    const size_t blocks = (total + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(conv_f32_any_kernel, dim3((unsigned)(blocks < 65536 ? blocks : 65536)),
                       dim3(kThreads), 0, stream, p);
    return q8_launch_status();
  }
  p.M = (int)M; p.rsc = d->R * d->S * d->C;
  p.by_img = make_fast_div((unsigned)per_img); p.by_row = make_fast_div((unsigned)p.Wo);
  p.by_c = make_fast_div((unsigned)d->C); p.by_s = make_fast_div((unsigned)d->S);
  const int build = pick_f32_tiled(d, M, per_img, out_cs, out_off, q8_aligned(x, 16) && q8_aligned(w, 16),
                                   p.vec_y && p.vec_b);
  if (build >= 0) return launch_f32_lds(build, p, stream);
  if (build == -1) return launch_f32_split(p, stream);
  return kF32Builds[pick_f32(M, d->K)].launch(p, stream);
}

}  // namespace
}  // namespace q8

extern "C" {

int q8_conv_f32_ref(const q8_conv_desc* d, const float* x_dev, const float* w_dev,
                    const float* b_dev, const float* res_dev, float* y_dev, void* stream) {
  return q8::conv_f32(d, x_dev, w_dev, b_dev, res_dev, y_dev, d ? d->K : 0, 0, nullptr, nullptr,
                      1, (hipStream_t)stream);
}

int q8_conv_f32_observed(const q8_conv_desc* d, const float* x_dev, const float* w_dev,
                         const float* b_dev, const float* res_dev, float* y_dev,
                         float* maxabs_sum_dev, float* maxabs_out_dev, void* stream) {
  Q8_REQUIRE(q8_aligned(maxabs_sum_dev, 4) && q8_aligned(maxabs_out_dev, 4), Q8_EALIGN);
  return q8::conv_f32(d, x_dev, w_dev, b_dev, res_dev, y_dev,
                      d && d->out_c_stride ? d->out_c_stride : (d ? d->K : 0), d ? d->out_c_off : 0,
                      maxabs_sum_dev, maxabs_out_dev, 1, (hipStream_t)stream);
}

int q8_conv_f32_observed_spread(const q8_conv_desc* d, const float* x_dev, const float* w_dev,
                                const float* b_dev, const float* res_dev, float* y_dev,
                                float* maxabs_sum_dev, float* maxabs_out_dev, int n_slots, void* stream) {
  Q8_REQUIRE(n_slots >= 1, Q8_EINVAL);
  Q8_REQUIRE(q8_aligned(maxabs_sum_dev, 4) && q8_aligned(maxabs_out_dev, 4), Q8_EALIGN);
  return q8::conv_f32(d, x_dev, w_dev, b_dev, res_dev, y_dev,
                      d && d->out_c_stride ? d->out_c_stride : (d ? d->K : 0), d ? d->out_c_off : 0,
                      maxabs_sum_dev, maxabs_out_dev, n_slots, (hipStream_t)stream);
}

int q8_calibrate_fold(const float* spread_dev, int n_keys, int n_slots, float* out_dev, void* stream) {
  Q8_REQUIRE(n_keys >= 0 && n_slots >= 1 && (n_keys == 0 || (spread_dev && out_dev)), Q8_EINVAL);
  Q8_REQUIRE(q8_aligned(spread_dev, 4) && q8_aligned(out_dev, 4), Q8_EALIGN);
  if (n_keys == 0) return Q8_OK;
  hipLaunchKernelGGL(q8::fold_slots_kernel, dim3(n_keys), dim3(64), 0, (hipStream_t)stream, spread_dev, n_slots,
                     out_dev);
  return q8_launch_status();
}

const char* q8_conv_f32_variant(const q8_conv_desc* d) {
  if (!q8::f32_desc_sane(d)) return "unsupported";
  const long per_img = (long)q8_conv_out_h(d) * q8_conv_out_w(d), M = d->N * per_img;
  if (M > 0 && !q8::f32_tiled(d, M, per_img)) return "conv_f32_any_kernel";
  const int build = M > 0 ? q8::pick_f32_tiled(d, M, per_img, d->out_c_stride ? d->out_c_stride : d->K, d->out_c_off,
                                               true, true) : -2;
  if (build >= 0) return q8::f32_lds_name(build);
  if (build == -1) return q8::f32_split_name(M, d->K);
  const q8::F32Build& b = q8::kF32Builds[q8::pick_f32(M, d->K)];
  return b.name[d->C % (16 * b.nc) == 0 ? 2 : d->C % 4 == 0 ? 1 : 0];
}

}  // extern "C"
