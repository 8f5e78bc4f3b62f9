// fp32 convolution of calibration on the bf16 matrix instructions: C % 16 == 0, aligned activations and filters.
//
// v_mfma_f32_32x32x16_bf16 does 16 times the products per clock that the fp32 instruction does, and its
// products and sums are fp32.  A value of 24 significant bits is exactly the sum of three bf16 values h + m + l, each
// rounded to nearest (|m| <= 2^-9 |x|, |l| <= 2^-18 |x|), and of the nine products of two such sums six are taken: hh,
// hm + mh, hl + lh, mm.  What is left out is below 2^-26 of a product, an eighth of an fp32 product's own rounding
// error.  hh goes into one accumulator (one rounding for 16 products, where the fp32 instruction has
// eight), the other five into a second one of 2^-8 of its size.
//
// Against 64 bits the result is half as far off as the fp32 builds' (2-norms: 14 x 14 x 256 3x3 1.1e-7 and
// 2.2e-7, 7 x 7 x 512 3x3 1.5e-7 and 3.0e-7; over the 106 layers of the package's networks nowhere further off).
//
// What bounds it: splitting, 11 vector instructions for two values, behind the LDS reads.  A wavefront issues one of them in
// 8 clocks, two on a SIMD one in 4.3 (subtractions 2.5); four of them behind an MFMA of 35 clocks are free, eight cost
// 9.  So a wavefront has four MFMA tiles, for which it splits four fragments, and two wavefronts share a SIMD.
// (v_dot2_f32_bf16 would subtract without unpacking, but runs on the matrix pipe.  One or two tiles a wavefront are
// 10 to 40 % slower on large layers; 128 x 128 tiles of four wavefronts, where each fragment is split twice too, 5 %
// faster there, but with one chain per value further off than the fp32 builds.)  Where tiles are few the operands'
// way into LDS bounds the layer instead, and the fp32 builds with their smaller tiles stay (f32_split_pays).  Batch 8,
// the fp32 builds' and these (us): 150 x 150 128 -> 128 3x3 376 and 334, 38 x 38 512 -> 512 3x3 413 and 330 (105 % of
// the fp32 matrix rate), 19 x 19 512 -> 1024 dilated 199 and 157, 28 x 28 128 -> 128 23.0 and 18.8.
//
// The split is exact for zero and for 2^-110 <= |x| < 3.38e38; of smaller values it loses up to 2^-134 each, of a
// denormal perhaps all.  So it holds for a sum of at least 2^-60 whose operands are below 2^32 (2^-42 of the sum is lost
// for each product at worst), and for a sum of zero without denormal operands.  Where a workgroup has other sums
// (infinities, NaNs and values that bf16 rounds to infinity among them) it runs its reduction a second time on
// the fp32 instruction, for what the fp32 sum gives; where it has zeros it looks through its operands first.  Noting the
// largest operand, one instruction for two values, and the barrier behind which all know take 1.8 % (323 us of the 330
// above).  75 x 75 128 -> 256 177 us, with a zero in every tile 218 to 245, of NaNs or of values below 2^-60 326 to
// 364; the fp32 builds 190 to 210.
#include "q8_conv_f32.h"
#include "q8_conv_ring_kernel.h"

namespace q8 {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kSplitStep = 64;       // bytes of a row per reduction step
constexpr int kSplitStages = 2;      // steps of a wavefront's ring
constexpr float kSplitLeast = 0x1p-60f, kSplitLargest = 0x1p32f;

struct Split3 { v8bf h, m, l; };

__device__ __forceinline__ Split3 split3(v4f lo, v4f hi) {
  v4u h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float a = e < 2 ? lo[2 * e] : hi[2 * e - 4], b = e < 2 ? lo[2 * e + 1] : hi[2 * e - 3];
    const unsigned ph = __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{a, b}, v2bf));
    const float ra = a - __uint_as_float(ph << 16), rb = b - __uint_as_float(ph & 0xffff0000u);
    const unsigned pm = __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{ra, rb}, v2bf));
    const float sa = ra - __uint_as_float(pm << 16), sb = rb - __uint_as_float(pm & 0xffff0000u);
    h[e] = ph;
    m[e] = pm;
    l[e] = __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{sa, sb}, v2bf));
  }
  return {__builtin_bit_cast(v8bf, h), __builtin_bit_cast(v8bf, m), __builtin_bit_cast(v8bf, l)};
}

// A workgroup owns 64 pixels x 64 channels.  Its KW wavefronts take equal runs of the reduction steps, each with a ring of
// two steps and all four 32 x 32 tiles, and add their sums through LDS in a fixed order; they do not meet before.
template <int KW>
__global__ __launch_bounds__(KW * 64, 2) void conv_f32_split_kernel(const F32Params p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ST = kSplitStages, T = 2, B = T * 32, BK = kSplitStep, LOADS = B / 16;    // (loads of either operand)
  constexpr int A_BYTES = B * BK, STAGE_BYTES = 2 * B * BK;
  constexpr int QUADS = T * T * 4, OWN = QUADS / KW;        // groups of 4 channels of a lane; those that it finishes
  static_assert(QUADS % KW == 0, "the wavefronts finish equal parts");
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  const int nblk = p.n_ptiles * p.n_ctiles;
  int bid = blockIdx.x;
  {   // every XCD takes a contiguous run of tiles, channel tile fastest (shared activations)
    const int xcd = bid % kNumXcd, idx = bid / kNumXcd, base = nblk / kNumXcd, rem = nblk % kNumXcd;
    bid = xcd * base + (xcd < rem ? xcd : rem) + idx;
  }
  const int ptile = bid / p.n_ctiles, ctile = bid - ptile * p.n_ctiles;
  const int pix0 = ptile * B, ch0 = ctile * B;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // The descriptor starts at the tile's first image, less the first padding rows (see conv_f32_lds_kernel).
  const int c_bytes = p.C * 4, x_shift = (p.ph * p.W + p.pw) * c_bytes;
  const int n0 = fast_div(pix0, p.by_img.m, p.by_img.s);
  const long img = (long)p.H * p.W * p.C;
  const long x_left = ((long)p.N - n0) * img * 4 + x_shift;
  const int8_t* const x_base = reinterpret_cast<const int8_t*>(p.x + n0 * img) - x_shift;
  const int x_bytes = (int)(x_left < 0x7fffffffL ? x_left : 0x7fffffffL), w_bytes = p.K * p.rsc * 4;

  // ---- loader: lane l of a load fills row l / 4, slot l % 4 (swizzled)
  const int lrow = lane >> 2;
  int a_off[LOADS], b_hi[LOADS], b_wi[LOADS], b_off[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int row = j * 16 + lrow;
    const int c = ch0 + (row & ~31) + row_to_channel(row & 31);
    a_off[j] = c < p.K ? c * p.rsc * 4 + swz<4>(row, lane & 3) * 16 : kOobOffset;
  }
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int row = j * 16 + lrow, px = pix0 + row;
    b_hi[j] = -(1 << 29);                // a pixel beyond M: every tap outside the image
    b_wi[j] = b_off[j] = 0;
    if (px < p.M) {
      const int n = fast_div(px, p.by_img.m, p.by_img.s);
      const int rem = px - n * (p.Ho * p.Wo);
      const int ho = fast_div(rem, p.by_row.m, p.by_row.s);
      b_hi[j] = ho * p.sh - p.ph;
      b_wi[j] = (rem - ho * p.Wo) * p.sw - p.pw;
      b_off[j] = (((n - n0) * p.H + b_hi[j]) * p.W + b_wi[j]) * c_bytes + x_shift + swz<4>(row, lane & 3) * 16;
    }
  }
  // Behind the rings, what some lane has found: a sum that is taken again, a large operand, a sum of zero, a denormal.
  enum { kAgain, kLarge, kZero, kDenormal, kFlags };
  int* const found = reinterpret_cast<int*>(lds + KW * ST * STAGE_BYTES);
  if (threadIdx.x < kFlags) found[threadIdx.x] = 0;    // (a barrier follows before anyone sets one)
  auto any = [&](int flag) { return __builtin_amdgcn_readfirstlane(found[flag]) != 0; };
  int8_t* const ring = lds + wave * ST * STAGE_BYTES;
  // this group's steps, and where the next one to request lies in the reduction
  const int n_st = p.rsc / (BK / 4), n_mine = (n_st + KW - 1) / KW;
  const int st_end = min((wave + 1) * n_mine, n_st);
  const int dw_step = p.dw * c_bytes, dh_step = p.dh * p.W * c_bytes - p.S * dw_step;
  int st, tap_c, tap_r, tap_s, tap_delta, b_voff[LOADS];
  auto refresh_tap = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      const bool in = ((unsigned)(b_hi[j] + tap_r * p.dh) < (unsigned)p.H) &
                      ((unsigned)(b_wi[j] + tap_s * p.dw) < (unsigned)p.W);
      b_voff[j] = in ? b_off[j] : kOobOffset;
    }
  };
  auto begin = [&]() __attribute__((always_inline)) {
    st = wave * n_mine;
    const int tap = fast_div(st * (BK / 4), p.by_c.m, p.by_c.s);
    tap_c = st * BK - tap * c_bytes;
    tap_r = fast_div(tap, p.by_s.m, p.by_s.s);
    tap_s = tap - tap_r * p.S;
    tap_delta = (tap_r * p.dh * p.W + tap_s * p.dw) * c_bytes;
    refresh_tap();
  };
  // The loads of the next step into `buf`.  Behind the group's last step the descriptors are empty: zeros, so that
  // every step counts the same loads.
  auto request = [&](int buf) __attribute__((always_inline)) {
    int8_t* const stage = ring + buf * STAGE_BYTES;
    const bool any = st < st_end;
    const __amdgpu_buffer_rsrc_t rsrc_w =
        __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, any ? w_bytes : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_x =
        __builtin_amdgcn_make_buffer_rsrc((void*)x_base, 0, any ? x_bytes : 0, 0x00020000);
#pragma unroll
    for (int j = 0; j < LOADS; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc_w, (__attribute__((address_space(3))) void*)(stage + j * 1024), 16, a_off[j],
          any ? st * BK : 0, 0, 0);
#pragma unroll
    for (int j = 0; j < LOADS; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc_x, (__attribute__((address_space(3))) void*)(stage + A_BYTES + j * 1024), 16,
          b_voff[j], any ? tap_delta + tap_c : 0, 0, 0);
    ++st;
    tap_c += BK;
    if (tap_c == c_bytes) {
      tap_c = 0;
      ++tap_s;
      tap_delta += dw_step;
      if (tap_s == p.S) {
        tap_s = 0;
        ++tap_r;
        tap_delta += dh_step;
      }
      refresh_tap();
    }
  };
  const int frag = (lane & 31) * BK + swz<4>(lane & 31, lane >> 5) * 16;
  int a_frag[2], b_frag[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    a_frag[h] = wave * ST * STAGE_BYTES + (frag ^ (h * 32));
    b_frag[h] = wave * ST * STAGE_BYTES + ((A_BYTES + frag) ^ (h * 32));
    asm volatile("" : "+v"(a_frag[h]));    // in registers: the reads then add an immediate
    asm volatile("" : "+v"(b_frag[h]));
  }
  v16f acc[T][T], low[T][T];
  float large = 0.0f;                    // the largest operand that this lane has split
  unsigned small = ~0u;                  // 2 |bits| - 1 of the smallest but zero that it has looked at
  v4f af[T][2], bf[T][2];
  auto read = [&](int off) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < T; ++i) af[i][h] = *reinterpret_cast<const v4f*>(lds + a_frag[h] + off + i * 32 * BK);
#pragma unroll
      for (int j = 0; j < T; ++j) bf[j][h] = *reinterpret_cast<const v4f*>(lds + b_frag[h] + off + j * 32 * BK);
    }
  };
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // the fragments this wavefront has asked for are in registers
    asm volatile("" ::: "memory");
  };
  using std::integral_constant;
  // One step: its values are in registers or on their way.  Then its buffer is filled again, and the next step's values
  // are read while the last MFMAs run.  Fragments are split beside the MFMAs that do not need them yet: 1.5 % off.
  // kFp32: the products of the fp32 instruction instead.  kLook: none, the operands looked at.
  enum { kSplit, kFp32, kLook };
  auto step = [&](auto buf_c, auto mode_c) __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_c)::value, MODE = decltype(mode_c)::value;
    wait_vmcnt<(ST - 2) * 2 * LOADS>();
    meet();
    if constexpr (MODE != kSplit) {
      if constexpr (MODE == kFp32) {
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              acc[j][i] =
                  __builtin_amdgcn_mfma_f32_32x32x2f32(af[i][e / 4][e % 4], bf[j][e / 4][e % 4], acc[j][i], 0, 0, 0);
      } else {
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const unsigned a = __float_as_uint(af[i][e / 4][e % 4]), b = __float_as_uint(bf[i][e / 4][e % 4]);
            small = min(small, min((a << 1) - 1, (b << 1) - 1));
          }
      }
      __builtin_amdgcn_sched_barrier(0);
      request(BUF);
      read((BUF + 1) % ST * STAGE_BYTES);
      return;
    }
    Split3 a[T], b[T];
    auto split = [&](v4f lo, v4f hi) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; e += 2) {     // (fmaxf would quiet signalling NaNs first, two instructions more)
        asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(large) : "v"(lo[e]), "v"(lo[e + 1]));
        asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(large) : "v"(hi[e]), "v"(hi[e + 1]));
      }
      return split3(lo, hi);
    };
    auto mma = [&](int i, int j, int t) __attribute__((always_inline)) {     // product t of tile (i, j)
      v16f& sum = t == 2 ? acc[j][i] : low[j][i];
      const v8bf& u = t == 0 || t == 4 ? a[i].m : t == 1 ? a[i].l : a[i].h;
      const v8bf& v = t == 0 || t == 5 ? b[j].m : t == 3 ? b[j].l : b[j].h;
      sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u, v, sum, 0, 0, 0);
    };
    a[0] = split(af[0][0], af[0][1]);
    b[0] = split(bf[0][0], bf[0][1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 6; ++t) mma(0, 0, t);
    a[1] = split(af[1][0], af[1][1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 6; ++t) mma(1, 0, t);
    b[1] = split(bf[1][0], bf[1][1]);
    __builtin_amdgcn_sched_barrier(0);
    request(BUF);
    read((BUF + 1) % ST * STAGE_BYTES);
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int i = 0; i < T; ++i) mma(i, 1, t);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto pass = [&](auto self, int n, auto buf_c, auto mode_c) __attribute__((always_inline)) -> void {
    constexpr int BUF = decltype(buf_c)::value;
    if constexpr (BUF < ST) {
      if (BUF < n) {
        step(buf_c, mode_c);
        self(self, n, integral_constant<int, BUF + 1>{}, mode_c);
      }
    }
  };
  auto walk = [&](auto mode_c) __attribute__((always_inline)) {     // over the whole reduction
    begin();
#pragma unroll
    for (int i = 0; i < ST; ++i) request(i);
    wait_vmcnt<(ST - 1) * 2 * LOADS>();
    meet();
    read(0);
    int left = n_mine;
    for (; left >= ST; left -= ST) pass(pass, ST, integral_constant<int, 0>{}, mode_c);
    pass(pass, left, integral_constant<int, 0>{}, mode_c);
    wait_vmcnt<0>();                     // (the loads of steps behind the last: LDS is used again)
    __syncthreads();
  };
  // Its sums, into the exchange.  Quad q of a lane is channels 4 (q % 4) .. of its 16 in channel
  // tile q / 4 % T, pixel tile q / 4 / T; a wavefront finishes quads wave * OWN .., of one channel and one pixel tile.
  float* const xch = reinterpret_cast<float*>(lds);
  auto reduce = [&](auto mode_c) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][i][e] = low[j][i][e] = 0.0f;
    walk(mode_c);
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
      v4f v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[q / 4 / T][q / 4 % T][4 * (q % 4) + e];
        if constexpr (decltype(mode_c)::value == kSplit) v[e] += low[q / 4 / T][q / 4 % T][4 * (q % 4) + e];
      }
      *reinterpret_cast<v4f*>(xch + ((wave * QUADS + q) * 64 + lane) * 4) = v;
    }
  };
  auto total = [&](int o) {
    v4f v = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int g = 0; g < KW; ++g)
      v += *reinterpret_cast<const v4f*>(xch + ((g * QUADS + wave * OWN + o) * 64 + lane) * 4);
    return v;
  };
  reduce(integral_constant<int, kSplit>{});
  if (!(large < kSplitLargest)) found[kLarge] = 1;
  __syncthreads();
  v4f own[OWN];
#pragma unroll
  for (int o = 0; o < OWN; ++o) own[o] = total(o);
  auto pixel_of = [&](int o) { return pix0 + (wave * OWN + o) / 4 / T * 32 + (lane & 31); };
  auto channel_of = [&](int o) {
    const int q = wave * OWN + o;
    return ch0 + q / 4 % T * 32 + 16 * (lane >> 5) + 4 * (q % 4);
  };
  // The sums that the split cannot vouch for, and those of zero, for which it can where no operand is denormal.
  const bool all = any(kLarge);
  unsigned again = 0, zero = 0;
  float least = INFINITY, none = 0.0f;   // none: no number where some sum is infinite or none
#pragma unroll
  for (int o = 0; o < OWN; ++o)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      least = fminf(least, fabsf(own[o][e]));
      none = fmaf(own[o][e], 0.0f, none);
    }
  if (all || !(least >= kSplitLeast) || none != 0.0f) {
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
      if (pixel_of(o) >= p.M) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = fabsf(own[o][e]);
        if (channel_of(o) + e >= p.K || (!all && a >= kSplitLeast && a < INFINITY)) continue;
        (!all && a == 0.0f ? zero : again) |= 1u << (o * 4 + e);
      }
    }
    if (again) found[kAgain] = 1;
    if (zero) found[kZero] = 1;
  }
  __syncthreads();
  const bool some_again = any(kAgain), some_zero = any(kZero);
  if (some_again | some_zero) {
    bool second = some_again;
    if (some_zero) {
      walk(integral_constant<int, kLook>{});
      if (small < 0x00ffffffu) found[kDenormal] = 1;
      __syncthreads();
      if (any(kDenormal)) {
        again |= zero;
        second = true;
      }
    }
    if (second) {
      reduce(integral_constant<int, kFp32>{});
      __syncthreads();
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
        const v4f v = total(o);
#pragma unroll
        for (int e = 0; e < 4; ++e) own[o][e] = again >> (o * 4 + e) & 1 ? v[e] : own[o][e];
      }
      __syncthreads();
    }
  }
  float m_sum = 0.0f, m_out = 0.0f;
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int pix = pixel_of(o), ch = channel_of(o);
    if (pix >= p.M || ch >= p.K) continue;
    v4f v = own[o];
    float* const y = p.y + (size_t)pix * p.out_cs + p.out_off + ch;
    const float* const res = p.res ? p.res + (size_t)pix * p.K + ch : nullptr;
    auto relu_max = [&](float u) {
      if (p.relu) u = fmaxf(u, 0.0f);
      m_out = fmaxf(m_out, fabsf(u));
      return u;
    };
    if (p.vec_y && p.vec_b && ch + 4 <= p.K) {
      if (p.b) v += *reinterpret_cast<const v4f*>(p.b + ch);
#pragma unroll
      for (int e = 0; e < 4; ++e) m_sum = fmaxf(m_sum, fabsf(v[e]));
      if (res) v += *reinterpret_cast<const v4f*>(res);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = relu_max(v[e]);
      *reinterpret_cast<v4f*>(y) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (ch + e >= p.K) continue;
        float u = v[e];
        if (p.b) u += p.b[ch + e];
        m_sum = fmaxf(m_sum, fabsf(u));
        if (res) u += res[e];
        y[e] = relu_max(u);
      }
    }
  }
  observe_block<KW>(p, m_sum, m_out, reinterpret_cast<float*>(lds));
#endif
}

template <int KW>
int launch_split(F32Params& p, hipStream_t stream) {
  constexpr int kRingBytes = KW * kSplitStages * 2 * 64 * kSplitStep, kFlagBytes = 16;
  static_assert(kRingBytes == KW * 4 * 4096, "the exchange fits the rings");
  constexpr int kLdsBytes = kRingBytes + kFlagBytes;
  p.n_ptiles = (p.M + 63) / 64;
  p.n_ctiles = (p.K + 63) / 64;
  const long nblk = (long)p.n_ptiles * p.n_ctiles;
  if (nblk > 0x7fffffffL) return Q8_EUNSUPPORTED;
  auto kernel = conv_f32_split_kernel<KW>;
  if constexpr (kLdsBytes > 65536) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (attr != hipSuccess) return Q8_EHIP;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)nblk), dim3(KW * 64), kLdsBytes, stream, p);
  return q8_launch_status();
}

}  // namespace

// Whether the layer is faster here than with the builds of q8_conv_f32_lds.hip, by their estimate (which is
// low, by up to a quarter: hence the 1.1) and one fitted to the layers of the package's networks at 1, 3 and 8 images.
// n: 64 x 64 tiles per CU.  Up to one eight wavefronts share a tile; two workgroups of four wavefronts fit a CU.
// Of 106 layers 44 change: 41 take 0.59 to 0.99 of their time, three 1.00 to 1.02 (worst 1x1 512 -> 2048 on 7 x 7 x 8,
// 12.5 and 12.8 us).  K % 64: tiles are full.  Layers that those builds do not take (`lds` false) run
// register-fed, in 1.5 to 1.8 times that estimate where they are long: 3x3 80 -> 192 on 73 x 73 x 8 145 us, 86 here;
// 512 -> 84 on 38 x 38 x 8 146, 94.
//
// Where the reduction is short, or half of every tile lies beyond K, both kernels spend their time elsewhere and these
// estimates do not hold: of 489 layers drawn and chosen by them the 50 left out here took 1.09 of their time on average
// (0.86 to 1.33), the others 0.76.
bool f32_split_pays(long M, int K, int rsc, float lds_us, bool lds) {
  if (lds ? K % 64 != 0 || rsc < 16 * 16 : K <= 32 || rsc <= 8 * 16) return false;
  const float n = (float)((M + 63) / 64) * (float)((K + 63) / 64) / 256.0f;
  const float step = n <= 1.0f ? 0.139f : n <= 2.0f ? 0.29f : fmaxf(0.49f, 0.182f * n);
  const float us = (n <= 1.0f ? 7.0f : 9.0f) + 1.1f * n + step * (float)(rsc / 16);
  return lds ? us < 1.1f * lds_us : us > 30.0f && us < 1.5f * lds_us;
}
int launch_f32_split(F32Params& p, hipStream_t stream) {
  const long tiles = (p.M + 63L) / 64 * ((p.K + 63) / 64);
  return tiles <= 256 ? launch_split<8>(p, stream) : launch_split<4>(p, stream);
}
const char* f32_split_name(long M, int K) {
  return (M + 63) / 64 * ((K + 63) / 64) <= 256 ? "conv_f32_split_kernel<8>" : "conv_f32_split_kernel<4>";
}

}  // namespace q8
