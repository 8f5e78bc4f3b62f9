// fp32 convolution of calibration, the builds on LDS: C % 32 == 0, K % 16 == 0, aligned rows.
//
// What bounds the register-fed builds (q8_conv_f32.hip) on the layers of a calibration batch is not
// the matrix rate: gathered register loads reach 11 to 14 bytes per clock and CU, and a tile of two
// to eight stages is a chain of latencies with few wavefronts to hide it.  Here the operands go from
// memory straight into LDS (buffer_load ... lds) through a ring, as in the int8 kernel, and a
// wavefront owns one 32 x 32 tile of v_mfma_f32_32x32x2 (64 clocks for 256 bytes of operands), so
// that several small workgroups fit a CU.
//
// A reduction step is 64 bytes of every row, in one filter tap.  KW groups of WP x WC wavefronts take
// equal runs of a tile's steps, each with a ring of its own, and add their sums through LDS in a
// fixed order.  A value is the sum of four (build 0) or eight chains: against 64 bits no further off
// than the register-fed builds' four (14 x 14 x 256 3x3: 2.2e-7 of the 2-norm to 3.0e-7; with two chains
// build 0 was, 56 x 56 x 64 3x3 2.2e-7 to 1.6e-7).
//
// What bounds the loop is what a wavefront issues beside its eight MFMAs of 64 clocks a step: with
// one wavefront on a SIMD (few tiles) everything in front of the first and behind the last MFMA is
// time.  The loop has no vector instruction but the reads' own addresses (those are immediates:
// the ring is unrolled; the padding mask changes with the tap alone; steps behind the last one get
// empty descriptors), and reads, loads and the scalar bookkeeping stand between the MFMAs.  7 x 7 x
// 512 3x3 at batch 8 as 56 tiles of 64 x 64 (61 us of matrix work): 89 us with vector addresses, 87
// with scalar ones in front of the MFMAs, 72 with them between.  Times at batch 8, the register-fed
// builds' and these (us): 56 x 56 64 -> 64 3x3 29.7 and 24.6, 64 -> 256 + residual 28.3 and 21.5,
// 28 x 28 128 -> 512 + residual 24.7 and 16.5, 14 x 14 256 -> 256 3x3 35.5 and 22.3, 7 x 7 512 -> 512 3x3
// 34.9 and 24.2; 38 x 38 512 -> 512 3x3 572 and 407 (95 and 134 TF; a library product reaches 153).
#include <cmath>
#include "q8_conv_f32.h"
#include "q8_conv_ring_kernel.h"

namespace q8 {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kStepBytes = 64;       // of a row per reduction step

template <int WP, int WC, int KW, int ST>
__global__ __launch_bounds__(WP * WC * KW * 64) void conv_f32_lds_kernel(const F32Params p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NW = WP * WC, BP = WP * 32, BC = WC * 32, BK = kStepBytes;
  constexpr int CHUNKS = BK / 16, RPW = 64 / CHUNKS, NH = BK / 32;
  constexpr int A_LOADS = BC / RPW / NW, B_LOADS = BP / RPW / NW, LOADS = A_LOADS + B_LOADS;
  constexpr int A_BYTES = BC * BK, STAGE_BYTES = (BC + BP) * BK;
  constexpr int OWN = 4 / KW;                   // quarters of a lane's 16 channels that it finishes
  static_assert(BC % (RPW * NW) == 0 && BP % (RPW * NW) == 0, "every wavefront issues the same loads");
  static_assert(KW * ST * STAGE_BYTES >= KW * NW * 4096, "the exchange fits the ring");
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  const int nblk = p.n_ptiles * p.n_ctiles;
  int bid = blockIdx.x;
  {   // every XCD takes a contiguous run of tiles, channel tile fastest (shared activations)
    const int xcd = bid % kNumXcd, idx = bid / kNumXcd, base = nblk / kNumXcd, rem = nblk % kNumXcd;
    bid = xcd * base + (xcd < rem ? xcd : rem) + idx;
  }
  const int ptile = bid / p.n_ctiles, ctile = bid - ptile * p.n_ctiles;
  const int pix0 = ptile * BP, ch0 = ctile * BC;
  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kgroup = KW > 1 ? wave_all / NW : 0, wave = KW > 1 ? wave_all % NW : wave_all;
  const int wave_p = wave % WP, wave_c = wave / WP;

  // The activation descriptor starts at the tile's first image (see conv_f32_mfma_kernel), less the
  // first padding rows: a lane's offset of its pixel's first tap is then never negative and stays in
  // the vector offset; the tap's own goes into the scalar offset.  A tap outside the image gets a
  // vector offset out of range, which reads zeros.
  const int c_bytes = p.C * 4, x_shift = (p.ph * p.W + p.pw) * c_bytes;
  const int n0 = fast_div(pix0, p.by_img.m, p.by_img.s);
  const long img = (long)p.H * p.W * p.C;
  const long x_left = ((long)p.N - n0) * img * 4 + x_shift;
  const int8_t* const x_base = reinterpret_cast<const int8_t*>(p.x + n0 * img) - x_shift;
  const int x_bytes = (int)(x_left < 0x7fffffffL ? x_left : 0x7fffffffL), w_bytes = p.K * p.rsc * 4;

  // what this lane finishes: 4 OWN channels from ch on of pixel pix; its residual values first of
  // all, so that their trip to memory is the operands' trip too
  const int pix = pix0 + wave_p * 32 + (lane & 31);
  const int ch = ch0 + wave_c * 32 + 16 * (lane >> 5) + kgroup * 4 * OWN;
  const bool mine = ch < p.K && pix < p.M;          // (K % 16 == 0: all of a lane's channels or none)
  v4f res[OWN], bias[OWN];
#pragma unroll
  for (int q = 0; q < OWN; ++q) res[q] = bias[q] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  if (mine) {
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
      if (p.res) res[q] = *reinterpret_cast<const v4f*>(p.res + (size_t)pix * p.K + ch + 4 * q);
      if (p.b) bias[q] = *reinterpret_cast<const v4f*>(p.b + ch + 4 * q);
    }
  }

  // ---- loader: lane l of a load fills row l / CHUNKS, slot l % CHUNKS (swizzled, see swz)
  const int lrow = lane / CHUNKS;
  int a_off[A_LOADS], b_hi[B_LOADS], b_wi[B_LOADS], b_off[B_LOADS];
#pragma unroll
  for (int j = 0; j < A_LOADS; ++j) {
    const int row = (wave + NW * j) * RPW + lrow;
    const int c = ch0 + (row & ~31) + row_to_channel(row & 31);
    a_off[j] = c < p.K ? c * p.rsc * 4 + swz<CHUNKS>(row, lane % CHUNKS) * 16 : kOobOffset;
  }
#pragma unroll
  for (int j = 0; j < B_LOADS; ++j) {
    const int row = (wave + NW * j) * RPW + lrow, px = pix0 + row;
    b_hi[j] = -(1 << 29);                // a pixel beyond M: every tap outside the image
    b_wi[j] = b_off[j] = 0;
    if (px < p.M) {
      const int n = fast_div(px, p.by_img.m, p.by_img.s);
      const int rem = px - n * (p.Ho * p.Wo);
      const int ho = fast_div(rem, p.by_row.m, p.by_row.s);
      b_hi[j] = ho * p.sh - p.ph;
      b_wi[j] = (rem - ho * p.Wo) * p.sw - p.pw;
      b_off[j] = (((n - n0) * p.H + b_hi[j]) * p.W + b_wi[j]) * c_bytes + x_shift +
                 swz<CHUNKS>(row, lane % CHUNKS) * 16;
    }
  }
  int8_t* const ring = lds + kgroup * ST * STAGE_BYTES;
  // this group's steps, and where the next one to request lies in the reduction
  const int n_st = p.rsc / (BK / 4), n_mine = (n_st + KW - 1) / KW;
  int st = kgroup * n_mine;
  const int st_end = min(st + n_mine, n_st);
  const int dw_step = p.dw * c_bytes, dh_step = p.dh * p.W * c_bytes - p.S * dw_step;
  int tap = fast_div(st * (BK / 4), p.by_c.m, p.by_c.s), tap_c = st * BK - tap * c_bytes;
  int tap_r = fast_div(tap, p.by_s.m, p.by_s.s), tap_s = tap - tap_r * p.S;
  int tap_delta = (tap_r * p.dh * p.W + tap_s * p.dw) * c_bytes;
  bool tap_changed = false;
  int b_voff[B_LOADS];
  auto refresh_tap = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
      const bool in = ((unsigned)(b_hi[j] + tap_r * p.dh) < (unsigned)p.H) &
                      ((unsigned)(b_wi[j] + tap_s * p.dw) < (unsigned)p.W);
      b_voff[j] = in ? b_off[j] : kOobOffset;
    }
  };
  refresh_tap();
  // Load J of the next step into `buf`: scalar work only.  Behind the group's last step the
  // descriptors are empty: zeros, so that every step counts the same loads.
  auto load = [&](int buf, auto j_c) __attribute__((always_inline)) {
    constexpr int J = decltype(j_c)::value;
    int8_t* const stage = ring + buf * STAGE_BYTES;
    const bool any = st < st_end;
    if constexpr (J < A_LOADS) {
      const __amdgpu_buffer_rsrc_t rsrc =
          __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, any ? w_bytes : 0, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc, (__attribute__((address_space(3))) void*)(stage + (wave + NW * J) * 1024), 16, a_off[J],
          any ? st * BK : 0, 0, 0);
    } else {
      constexpr int B = J - A_LOADS;
      const __amdgpu_buffer_rsrc_t rsrc =
          __builtin_amdgcn_make_buffer_rsrc((void*)x_base, 0, any ? x_bytes : 0, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc, (__attribute__((address_space(3))) void*)(stage + A_BYTES + (wave + NW * B) * 1024), 16,
          b_voff[B], any ? tap_delta + tap_c : 0, 0, 0);
    }
  };
  auto advance = [&]() __attribute__((always_inline)) {
    ++st;
    tap_c += BK;
    tap_changed = tap_c == c_bytes;
    tap_c = tap_changed ? 0 : tap_c;
    tap_s += tap_changed ? 1 : 0;
    tap_delta += tap_changed ? dw_step : 0;
    const bool wrap = tap_s == p.S;
    tap_s = wrap ? 0 : tap_s;
    tap_r += wrap ? 1 : 0;
    tap_delta += wrap ? dh_step : 0;
  };
  const int frag = (lane & 31) * BK + swz<CHUNKS>(lane & 31, lane >> 5) * 16;
  int a_frag[NH], b_frag[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    a_frag[h] = kgroup * ST * STAGE_BYTES + ((wave_c * 32 * BK + frag) ^ (h * 32));
    b_frag[h] = kgroup * ST * STAGE_BYTES + ((A_BYTES + wave_p * 32 * BK + frag) ^ (h * 32));
    asm volatile("" : "+v"(a_frag[h]));    // in registers: the reads then add an immediate
    asm volatile("" : "+v"(b_frag[h]));
  }
  // SUMS chains of its own per wavefront: 2 KW or 4 KW of them, eight or (build 0) four for a value
  constexpr int SUMS = KW == 4 ? 2 : 4;
  v16f acc[SUMS];
#pragma unroll
  for (int c = 0; c < SUMS; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[c][e] = 0.0f;
  // The fragments of a whole step, two sets: those of step i + 1 are read while the MFMAs of step i run.
  v4f af[2][NH], bf[2][NH];
  using std::integral_constant;
  auto read = [&](auto buf_c, auto set_c, auto h_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value, SET = decltype(set_c)::value, H = decltype(h_c)::value;
    af[SET][H] = *reinterpret_cast<const v4f*>(lds + a_frag[H] + BUF * STAGE_BYTES);
    bf[SET][H] = *reinterpret_cast<const v4f*>(lds + b_frag[H] + BUF * STAGE_BYTES);
  };
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // the fragments this wavefront has asked for are in registers
    asm volatile("" ::: "memory");
    if constexpr (NW > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // prologue: ST steps requested, the first one's fragments read
  auto request = [&](auto self, int buf, auto j_c) __attribute__((always_inline)) -> void {
    constexpr int J = decltype(j_c)::value;
    if constexpr (J < LOADS) {
      load(buf, j_c);
      self(self, buf, integral_constant<int, J + 1>{});
    }
  };
#pragma unroll
  for (int i = 0; i < ST; ++i) {
    request(request, i, integral_constant<int, 0>{});
    advance();
    if (tap_changed) refresh_tap();
  }
  wait_vmcnt<(ST - 1) * LOADS>();
  meet();
  static_assert(NH == 2, "two sub-steps");
  read(integral_constant<int, 0>{}, integral_constant<int, 0>{}, integral_constant<int, 0>{});
  read(integral_constant<int, 0>{}, integral_constant<int, 0>{}, integral_constant<int, 1>{});
  // One step (its fragments are in registers, its ring buffer is read by all): with it the ST - 2 steps
  // behind the next one may still be in flight.
  auto step = [&](auto buf_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value, SET = BUF & 1;
    wait_vmcnt<(ST - 2) * LOADS>();
    meet();
    __builtin_amdgcn_sched_barrier(0);
    auto mma = [&](auto self, auto g_c) __attribute__((always_inline)) -> void {
      constexpr int G = decltype(g_c)::value, E = G / NH, H = G % NH;
      if constexpr (G < 4 * NH) {
        v16f& sum = acc[G % SUMS];
        sum = __builtin_amdgcn_mfma_f32_32x32x2f32(af[SET][H][E], bf[SET][H][E], sum, 0, 0, 0);
        if constexpr (G < NH) read(integral_constant<int, (BUF + 1) % ST>{}, integral_constant<int, SET ^ 1>{}, g_c);
        else if constexpr (G < NH + LOADS) load(BUF, integral_constant<int, G - NH>{});
        else if constexpr (G == NH + LOADS) advance();
        __builtin_amdgcn_sched_barrier(0);
        self(self, integral_constant<int, G + 1>{});
      }
    };
    static_assert(4 * NH > NH + LOADS, "one piece of work behind every MFMA");
    mma(mma, integral_constant<int, 0>{});
    if (tap_changed) refresh_tap();
  };
  static_assert(ST % 2 == 0, "the set of a step follows from its buffer");
  auto pass = [&](auto self, int n, auto buf_c) __attribute__((always_inline)) -> void {
    constexpr int BUF = decltype(buf_c)::value;
    if constexpr (BUF < ST) {
      if (BUF < n) {
        step(buf_c);
        self(self, n, integral_constant<int, BUF + 1>{});
      }
    }
  };
  int left = n_mine;
  for (; left >= ST; left -= ST) pass(pass, ST, integral_constant<int, 0>{});
  pass(pass, left, integral_constant<int, 0>{});
  wait_vmcnt<0>();                       // (the loads of steps behind the last: LDS is used again)

#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if constexpr (SUMS == 4) acc[0][e] = (acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e]);
    else acc[0][e] += acc[1][e];
  }
  v4f own[OWN];
  if constexpr (KW > 1) {
    __syncthreads();
    float* const xch = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v4f v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[0][4 * q + e];
      *reinterpret_cast<v4f*>(xch + (((wave * KW + kgroup) * 4 + q) * 64 + lane) * 4) = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
      own[q] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int g = 0; g < KW; ++g)
        own[q] += *reinterpret_cast<const v4f*>(xch + (((wave * KW + g) * 4 + kgroup * OWN + q) * 64 + lane) * 4);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) own[q][e] = acc[0][4 * q + e];
  }
  float m_sum = 0.0f, m_out = 0.0f;
  if (mine) {
    float* y = p.y + (size_t)pix * p.out_cs + p.out_off + ch;
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
      v4f v = own[q] + bias[q];
#pragma unroll
      for (int e = 0; e < 4; ++e) m_sum = fmaxf(m_sum, fabsf(v[e]));
      if (p.res) v += res[q];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p.relu) v[e] = fmaxf(v[e], 0.0f);
        m_out = fmaxf(m_out, fabsf(v[e]));
      }
      *reinterpret_cast<v4f*>(y + 4 * q) = v;
    }
  }
  __syncthreads();
  observe_block<NW * KW>(p, m_sum, m_out, reinterpret_cast<float*>(lds));
#endif
}

template <int WP, int WC, int KW, int ST>
int launch_lds(F32Params& p, hipStream_t stream) {
  constexpr int kLdsBytes = KW * ST * (WP + WC) * 32 * kStepBytes;
  p.n_ptiles = (p.M + WP * 32 - 1) / (WP * 32);
  p.n_ctiles = (p.K + WC * 32 - 1) / (WC * 32);
  const long nblk = (long)p.n_ptiles * p.n_ctiles;
  if (nblk > 0x7fffffffL) return Q8_EUNSUPPORTED;
  auto kernel = conv_f32_lds_kernel<WP, WC, KW, ST>;
  if constexpr (kLdsBytes > 65536) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (attr != hipSuccess) return Q8_EHIP;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)nblk), dim3(WP * WC * KW * 64), kLdsBytes, stream, p);
  return q8_launch_status();
}

struct F32LdsBuild {
  const char* name;
  int (*launch)(F32Params&, hipStream_t);
  int bp, bc;
};
#define Q8_F32_LDS_ROW(WP, WC, KW, ST) \
  { "conv_f32_lds_kernel<" #WP "," #WC "," #KW "," #ST ">", &launch_lds<WP, WC, KW, ST>, WP * 32, WC * 32 },
const F32LdsBuild kF32LdsBuilds[] = {
    Q8_F32_LDS_ROW(2, 2, 1, 4)    // 0: 64 pixels x 64 channels
    Q8_F32_LDS_ROW(1, 2, 2, 4)    // 1: 32 x 64, two groups
    Q8_F32_LDS_ROW(2, 1, 2, 4)    // 2: 64 x 32, two groups
    Q8_F32_LDS_ROW(1, 1, 4, 4)    // 3: 32 x 32, four groups
};
#undef Q8_F32_LDS_ROW
constexpr int kNumF32Lds = sizeof(kF32LdsBuilds) / sizeof(kF32LdsBuilds[0]);

}  // namespace

// The build whose estimate is lowest: 4.5 us of launch, prologue and tail, the matrix time of the tiles
// that the busiest CU gets (256 operations a clock at 2.4 GHz; 91 % of that are reached) and 0.6 us
// for each tile's own prologue and tail.  Fitted to ResNet-50's layers at batch 8 (deeper rings change
// nothing; two groups on 64 x 64 tiles, and 32 x 32 by two, are nowhere the best by more than 2 %).
int pick_f32_lds(long M, int K, int rsc, float* us_out) {
  int best = 0;
  float least = 0.0f;
  for (int v = 0; v < kNumF32Lds; ++v) {
    const F32LdsBuild& b = kF32LdsBuilds[v];
    const float n = (float)((M + b.bp - 1) / b.bp) * (float)((K + b.bc - 1) / b.bc) / 256.0f;
    const float tile = (float)(b.bp * b.bc) * (float)rsc * (1.1f * 2.0f / 256.0f / 2400.0f);
    const float us = 4.5f + (n < 8.0f ? ceilf(n) : n) * tile * (b.bp * b.bc == 1024 ? 1.05f : 1.0f) + 0.6f * n;
    if (v == 0 || us < least) { best = v; least = us; }
  }
  *us_out = least;
  return best;
}
int launch_f32_lds(int build, F32Params& p, hipStream_t stream) {
  return build >= 0 && build < kNumF32Lds ? kF32LdsBuilds[build].launch(p, stream) : Q8_EINVAL;
}
const char* f32_lds_name(int build) { return kF32LdsBuilds[build].name; }

}  // namespace q8
