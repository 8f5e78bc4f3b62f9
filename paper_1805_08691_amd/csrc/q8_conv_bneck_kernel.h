// A bottleneck block in one launch (Eq. x / Eq. A' / Eq. + of arxiv 1805.08691): a 1x1 layer (A) on
// MID output channels, the 3x3 layer (B, stride 1, padding 1) that reads it, and the 1x1 layer (C) behind
// that one with its fused sum, for MID = 64, 128 or 256.
//
// Three launches are three times a launch gap, a prologue that waits for its first operands, a ragged last
// round of workgroups and an epilogue.  Here a workgroup takes a strip of whole rows of one image
// through all three layers; the codes between them stay in LDS (and are written to their tensors once,
// for whoever reads those).  The strip's layer A covers one row more on either side, which neighbouring
// strips compute too.  us, three launches and one: 14 x 14, 1024 -> 256 -> 1024 at 64 images 34.4 and 28.8,
// at 32 23.9 and 20.9; 28 x 28, 512 -> 128 -> 512 at 32 25.1 and 20.1, at 13 17.4 and 12.0, at 4 13.2 and
// 11.1; 56 x 56, 256 -> 64 -> 256 at 13 19.7 and 15.2, at 4 15.4 and 8.5, at 64 56.8 and 57.0.  ResNet-50 64
// images 692 -> 645 us, 16 354 -> 320, 13 unsigned 428 -> 400, 4 296 -> 267.
//
// What bounds it, in clocks of a strip of four rows of 14 pixels (two pixel tiles a wavefront): 4400 until the
// first operands are there; layer A 10100 and B 12900, filters and input at 34 and 46 bytes a clock into LDS (matrix
// instructions 6300 and 9500); the tails of A and B 5600; layer C 11500, vector instructions of its
// tail (a matrix and a vector instruction of one wavefront hardly overlap, those of two do, so rounds stay
// a block of the one and then of the other).
//
//  * Filters: a wavefront owns 32 output channels in every layer, so it streams its own filter
//    rows, global -> LDS, into a ring that no other wavefront reads, through all three layers without a
//    pause and WITHOUT A BARRIER; only the steps of layer A meet, for the input chunk that all
//    wavefronts share.  A piece is G = 64 or 128 reduction bytes of the 32 rows.
//  * Fragments of the next 64 bytes are read while the last ones multiply.
//  * Layer A's codes lie in LDS as (rows + 2) x (W + 2) pixels with a frame of zeros, MID + 16
//    bytes apart and rows padded so that the strip's pixels i = row * W + column all follow one another
//    in banks: a tap is one scalar to add, no masks, and sixteen consecutive pixels read at one channel
//    touch every bank once (rows without that padding, 14 pixels wide: a third of the LDS cycles conflicts).
//  * Layer C's activations (a wavefront's TB pixel tiles x MID channels) are read from LDS once, into
//    registers, and serve all of its output channels, in rounds of 32 per wavefront.
// Every vector store is issued by every wavefront whatever its pixels (lanes without one go out of the
// buffer's range), so the waits for the ring can count them.
#pragma once
#include "q8_conv_ring_kernel.h"

namespace q8 {

// What the tail of a layer needs (as the members of ConvParams of the same names).
struct BneckTail {
  float m, m_r;
  int relu, out_u8, res_u8;
  const float* m_vec;
};

struct BneckParams {
  const int8_t *x, *wa, *wb, *wc, *res;
  int8_t *ya, *yb, *yc;
  const int32_t *bias_a, *bias_b, *bias_c, *tap_sums;
  BneckTail a, b, c;
  int x_bytes, x_image, x_row, x_pixel;          // input: bytes; of an image, of an output row's step, of a pixel's
  int wa_bytes, wb_bytes, wc_bytes, res_bytes;
  int C, K2, H, W, M;
  int ya_cs, ya_off, yb_cs, yb_off, yc_cs, yc_off, res_cs, res_off;
  int rows, strips;                              // output rows per strip, strips per image
  unsigned div_row_m, div_row_s, div_strips_m, div_strips_s;
  int params_off, tile_off;                      // LDS: biases and scales; input chunks / codes between the layers
};

namespace {

// WP wavefronts side by side on pixels; TA / TB pixel tiles of a wavefront in layer A / behind it; D
// pieces of GS * 64 bytes in a wavefront's filter ring, XS input chunks as long.
template <int MID_, int WP_, int TA_, int TB_, int D_, int XS_, int GS_>
struct BneckShape {
  static constexpr int MID = MID_, WP = WP_, TA = TA_, TB = TB_, D = D_, XS = XS_, GS = GS_;
  static constexpr int WC = MID / 32, NW = WC * WP;
  static constexpr int G = GS * 64, CHUNKS = G / 16, RPI = 64 / CHUNKS;    // rows a wave-wide load fills
  static constexpr int NKC = MID / 64;                          // 64-byte steps over MID channels
  static constexpr int AP = WP * TA * 32, BP = WP * TB * 32;    // pixels of layer A / of the strip, at most
  static constexpr int FL = 32 / RPI, PIECE = 32 * G;           // a piece: loads, bytes
  static constexpr int XL = (AP / RPI + NW - 1) / NW;           // input loads per wavefront and chunk
  static constexpr int XCHUNK = XL * NW * 1024;
  static constexpr int PITCH = MID + 16;
  static constexpr int ROW_PAD = (256 - 2 * PITCH % 256) % 256;  // (W + 2) PITCH + this = W PITCH modulo 256
  static constexpr int RING_BYTES = NW * D * PIECE;
  static_assert(XS >= D && NKC % GS == 0, "input chunks in flight");
  static_assert((D - 1) * (FL + XL) + (XS - D) * XL < 64 && (D - 1) * FL + 2 * TB < 64, "vmcnt is 6 bits");
  // LDS of one layer's biases (or scales): whole wave-wide loads
  static constexpr int param_bytes(int k) { return (k * 4 + 1023) & ~1023; }
};

template <int MID, int WP, int TA, int TB, int D, int XS, int GS, int OCC, int EXT>
__global__ __launch_bounds__(MID / 32 * WP * 64, OCC)
void conv_i8_bneck_kernel(const BneckParams q) {
#if defined(__HIP_DEVICE_COMPILE__)
  using Sh = BneckShape<MID, WP, TA, TB, D, XS, GS>;
  constexpr int NW = Sh::NW, NKC = Sh::NKC, XL = Sh::XL, FL = Sh::FL, G = Sh::G, PITCH = Sh::PITCH, PIECE = Sh::PIECE;
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_p = wave % WP, wave_c = wave / WP;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  auto rsrc_of = [](const void* base, int bytes) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
  };
  auto load_lds = [](__amdgpu_buffer_rsrc_t rsrc, int8_t* to, int off, int soff) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)to, 16, off, soff, 0, 0);
  };

  // ---- the strip (every XCD takes a contiguous run of them: neighbours share input rows)
  const int nblk = gridDim.x;
  int bid = blockIdx.x;
  {
    const int xcd = bid % kNumXcd, idx = bid / kNumXcd;
    const int base = nblk / kNumXcd, rem = nblk % kNumXcd;
    bid = xcd * base + (xcd < rem ? xcd : rem) + idx;
  }
  const int n = fast_div(bid, q.div_strips_m, q.div_strips_s);
  const int h0 = (bid - n * q.strips) * q.rows;
  const int H = q.H, W = q.W, TR = q.rows, K2 = q.K2;
  const int n_halo = (TR + 2) * W;                       // pixels of layer A
  const int n_own = min(TR, H - h0) * W;                 // pixels of the strip
  const int pix0 = (n * H + h0) * W;                     // its first output pixel

  const int row_bytes = (W + 2) * PITCH + Sh::ROW_PAD;   // of layer A's codes in LDS

  int8_t* const ring = lds + wave * (D * PIECE);
  int8_t* const params = lds + q.params_off;
  int8_t* const tile = lds + q.tile_off;
  constexpr int PB = Sh::param_bytes(MID);               // biases: layer A, B, C; then the scales
  const int scales_off = 2 * PB + Sh::param_bytes(K2);

  // ---- biases and scales into LDS, a wave-wide load at a time (the whole offset in the vector operand: that
  // is what the range check compares with the table's bytes, whichever way it counts a scalar offset)
  {
    auto copy = [&](const void* from, int k, int8_t* to, int first) __attribute__((always_inline)) {
      const int loads = Sh::param_bytes(k) >> 10;
      for (int i = (wave + NW - first) % NW; i < loads; i += NW)
        load_lds(rsrc_of(from, from ? k * 4 : 0), to + i * 1024, i * 1024 + lane * 16, 0);
    };
    copy(q.bias_a, MID, params, 0);
    copy(q.bias_b, MID, params + PB, 1);
    copy(q.bias_c, K2, params + 2 * PB, 2 % NW);
    if (EXT) {
      copy(q.a.m_vec, MID, params + scales_off, 0);
      copy(q.b.m_vec, MID, params + scales_off + PB, 1);
      copy(q.c.m_vec, K2, params + scales_off + 2 * PB, 2 % NW);
    }
  }

  // ---- the stream of filter pieces: layer A, layer B, then layer C in rounds of MID rows.  Load j of a
  // piece fills rows RPI j + lane / CHUNKS of this wavefront's 32; a segment's end is the rare case.
  const int gA = q.C / G;                                // pieces of layer A
  int f_ch[FL], f_chunk[FL], f_off[FL];
#pragma unroll
  for (int j = 0; j < FL; ++j) {
    const int row = Sh::RPI * j + lane / Sh::CHUNKS;
    f_ch[j] = wave_c * 32 + row_to_channel(row);
    f_chunk[j] = swz<Sh::CHUNKS>(row, lane % Sh::CHUNKS) * 16;
    f_off[j] = f_ch[j] * q.C + f_chunk[j];
  }
  __amdgpu_buffer_rsrc_t f_rsrc = rsrc_of(q.wa, q.wa_bytes);
  int f_soff = 0, f_left = gA, f_segment = 0, f_slot = 0;
  const int f_segments = 2 + K2 / MID;
  auto issue_filters = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < FL; ++j) load_lds(f_rsrc, ring + f_slot + j * 1024, f_off[j], f_soff);
    f_slot = f_slot == (D - 1) * PIECE ? 0 : f_slot + PIECE;
    f_soff += G;
    if (--f_left == 0) {
      ++f_segment;
      if (f_segment == 1) {
        f_rsrc = rsrc_of(q.wb, q.wb_bytes);
#pragma unroll
        for (int j = 0; j < FL; ++j) f_off[j] = f_ch[j] * (9 * MID) + f_chunk[j];
        f_soff = 0;
        f_left = 9 * MID / G;
      } else if (f_segment < f_segments) {
        f_rsrc = rsrc_of(q.wc, q.wc_bytes);
#pragma unroll
        for (int j = 0; j < FL; ++j) f_off[j] = f_ch[j] * MID + f_chunk[j];
        f_soff = (f_segment - 2) * (MID * MID);
        f_left = MID / G;
      } else {          // behind the last, each time: no bytes and no scalar offset, so nothing is read
        f_rsrc = rsrc_of(q.wc, 0);
        f_soff = 0;
        f_left = 1;
      }
    }
  };

  // ---- input loader: load j of a chunk fills pixels (wave + NW j) RPI + lane / CHUNKS of layer A
  const __amdgpu_buffer_rsrc_t rsrc_x = rsrc_of(q.x, q.x_bytes);
  int x_off[XL];
#pragma unroll
  for (int j = 0; j < XL; ++j) {
    const int i = (wave + NW * j) * Sh::RPI + lane / Sh::CHUNKS;
    const int hr = fast_div(i, q.div_row_m, q.div_row_s), col = i - hr * W, h = h0 - 1 + hr;
    x_off[j] = i < n_halo && (unsigned)h < (unsigned)H
                   ? n * q.x_image + h * q.x_row + col * q.x_pixel + swz<Sh::CHUNKS>(i & 31, lane % Sh::CHUNKS) * 16
                   : kOobOffset;
  }
  auto issue_x = [&](int chunk, int slot) __attribute__((always_inline)) {
    const bool in = chunk < gA;
#pragma unroll
    for (int j = 0; j < XL; ++j)
      load_lds(rsrc_x, tile + slot + (wave + NW * j) * 1024, in ? x_off[j] : kOobOffset, in ? chunk * G : 0);
  };
#pragma unroll
  for (int k = 0; k < D; ++k) {
    issue_filters();
    issue_x(k, k * Sh::XCHUNK);
  }
#pragma unroll
  for (int k = D; k < XS; ++k) issue_x(k, k * Sh::XCHUNK);

  auto meet = [&]() __attribute__((always_inline)) {     // bare: memory stays in flight
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto own_reads_done = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
  };
  auto load16 = [&](const int8_t* base, int ch, int (&v)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const v4i t = *reinterpret_cast<const v4i*>(base + (ch + 4 * a) * 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[4 * a + k] = t[k];
    }
  };
  auto load_scales = [&](int off, int ch, float (&mv)[16]) __attribute__((always_inline)) {
    int v[16];
    load16(params + scales_off + off, ch, v);
#pragma unroll
    for (int e = 0; e < 16; ++e) mv[e] = __int_as_float(v[e]);
  };

  const int own_ch = wave_c * 32 + 16 * frag_half;       // this lane's 16 channels of a round
  const int foff0 = frag_row * G + swz<Sh::CHUNKS>(frag_row, frag_half) * 16;
  int f_read = 0;                                        // ring slot of the piece read next
  auto next_piece = [&]() __attribute__((always_inline)) { f_read = f_read == (D - 1) * PIECE ? 0 : f_read + PIECE; };

  // ================================================================ layer A
  v4i af[2][2];                                          // [set][half] of a 64-byte step
  auto load_filter = [&](int set, int k) __attribute__((always_inline)) {    // step k of the piece
#pragma unroll
    for (int h = 0; h < 2; ++h)
      af[set][h] = *reinterpret_cast<const v4i*>(ring + f_read + (foff0 ^ ((2 * k + h) * 32)));
  };
  {
    v16i acc[TA];
    v4i bf[2][2][TA];
    int slot = 0;                          // of the input chunk read next
    auto load_step = [&](int set, int k) __attribute__((always_inline)) {
      load_filter(set, k);
      const int8_t* const xs = tile + slot + wave_p * (TA * 32 * G);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < TA; ++j)
          bf[set][h][j] = *reinterpret_cast<const v4i*>(xs + j * 32 * G + (foff0 ^ ((2 * k + h) * 32)));
    };
    wait_vmcnt<(D - 1) * (FL + XL) + (XS - D) * XL>();
    meet();
    {
      int b[16];
      load16(params, own_ch, b);
#pragma unroll
      for (int j = 0; j < TA; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = b[e];
    }
    load_step(0, 0);
    // step K of piece s, its fragments in set SET
    auto step = [&](int s, auto k_c, auto set_c) __attribute__((always_inline)) {
      constexpr int K = decltype(k_c)::value, SET = decltype(set_c)::value;
      own_reads_done();
      if constexpr (K + 1 < GS) {
        load_step(SET ^ 1, K + 1);
      } else {
        issue_filters();                   // of piece s + D, into the slot of piece s
        next_piece();
        if (s + 1 < gA) {
          // Younger than the next piece and input chunk: D - 1 pieces and the input chunks behind it
          // (only while there are any to request).
          if (s - 1 + XS >= gA) wait_vmcnt<(D - 1) * FL>();
          else if (s + 1 < D) wait_vmcnt<(D - 1) * FL + (XS - 2) * XL>();
          else wait_vmcnt<(D - 1) * FL + (XS > D ? D - 1 : D - 2) * XL>();
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          if (s + XS < gA) issue_x(s + XS, slot);
          slot = slot == (XS - 1) * Sh::XCHUNK ? 0 : slot + Sh::XCHUNK;
          load_step(SET ^ 1, 0);
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < TA; ++j)
          acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[SET][h], bf[SET][h][j], acc[j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    if constexpr (GS == 2) {
#pragma unroll 1
      for (int s = 0; s < gA; ++s) {
        step(s, c0, c0);
        step(s, c1, c1);
      }
    } else {
#pragma unroll 1
      for (int s = 0; s < gA; s += 2) {
        step(s, c0, c0);
        if (s + 1 < gA) step(s + 1, c0, c1);
      }
    }
    // the input chunks give way to the codes: nothing is on its way into them any more
    wait_vmcnt<0>();
    meet();
    for (int i = tid; i < (TR + 2) * 2 * (MID / 16); i += NW * 64) {     // the frame's two columns
      const int c = i % (MID / 16), r = i / (MID / 16);
      *reinterpret_cast<v4i*>(tile + (r >> 1) * row_bytes + (r & 1) * (W + 1) * PITCH + c * 16) = v4i{0, 0, 0, 0};
    }
    const __amdgpu_buffer_rsrc_t rsrc_y = rsrc_of(q.ya, q.M * q.ya_cs);
    float mv[16] = {};
    if (EXT && q.a.m_vec) load_scales(0, own_ch, mv);
#pragma unroll
    for (int j = 0; j < TA; ++j) {
      const int i = (wave_p * TA + j) * 32 + frag_row;
      const int hr = fast_div(i, q.div_row_m, q.div_row_s), col = i - hr * W, h = h0 - 1 + hr;
      const bool inside = (unsigned)h < (unsigned)H;
      int v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = acc[j][e];
      const int rw[4] = {0, 0, 0, 0};
      v4i codes = codes16_build<EXT>(q.a, v, rw, mv, false);
      if (!inside) codes = v4i{0, 0, 0, 0};
      if (i < n_halo) *reinterpret_cast<v4i*>(tile + hr * row_bytes + (col + 1) * PITCH + own_ch) = codes;
      const bool own = (unsigned)(i - W) < (unsigned)n_own;
      int off = (pix0 + i - W) * q.ya_cs + q.ya_off + own_ch;
      off = own ? off : kOobOffset;
      __builtin_amdgcn_raw_buffer_store_b128(codes, rsrc_y, off, 0, 0);
    }
    meet();
  }

  // ================================================================ layer B
  int own_pix[TB];                         // pixel of the strip
#pragma unroll
  for (int j = 0; j < TB; ++j) own_pix[j] = (wave_p * TB + j) * 32 + frag_row;
  {
    v16i acc[TB];
    int pbase[TB];
    {
      int b[16];
      load16(params + PB, own_ch, b);
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const int i = own_pix[j], ty = fast_div(i, q.div_row_m, q.div_row_s);
        pbase[j] = (i < TR * W ? ty * row_bytes + (i - ty * W) * PITCH : 0) + 16 * frag_half;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = b[e];
        if (EXT && q.tap_sums) {           // unsigned codes: the start values of the pixel's rectangle
          const int h = h0 + ty, w = i - ty * W;
          const int idx = i < n_own ? (((h == 0) * 4 + (h + 1 < H ? 3 : 2)) * 4 + (w == 0)) * 4 + (w + 1 < W ? 3 : 2) : 0;
          const v4i* const row = reinterpret_cast<const v4i*>(q.tap_sums + idx * MID + own_ch);
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const v4i t = row[a];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][4 * a + e] = t[e];
          }
        }
      }
    }
    v4i bf[2][2][TB];
    auto load_step = [&](int set, int k, const int8_t* base) __attribute__((always_inline)) {
      load_filter(set, k);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < TB; ++j) bf[set][h][j] = *reinterpret_cast<const v4i*>(base + pbase[j] + h * 32);
    };
    load_step(0, 0, tile);                 // (landed in front of layer A's tail)
    const int8_t* tap_base = tile;
    // one pass: the steps of one tap (of all of them where a tap is one step)
    constexpr int TAPS = NKC == 1 ? 9 : 1;
#pragma unroll 1
    for (int tap = 0; tap < 9; tap += TAPS) {
#pragma unroll
      for (int k = 0; k < TAPS * NKC; ++k) {
        const int set = k & 1, col = (tap + k / NKC) % 3;
        own_reads_done();
        if (k % GS == GS - 1) {            // the piece has been read: the one D behind it
          issue_filters();
          next_piece();
          // (counted: D - 1 pieces; the stores behind layer A only make it wait longer)
          wait_vmcnt<(D - 1) * FL>();
          asm volatile("" ::: "memory");
        }
        if (k % NKC == NKC - 1) tap_base += col == 2 ? row_bytes - 2 * PITCH : PITCH;
        if (tap + (k + 1) / NKC < 9) load_step(set ^ 1, (k + 1) % GS, tap_base + ((k + 1) % NKC) * 64);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < TB; ++j)
            acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[set][h], bf[set][h][j], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    meet();                                // layer A's codes have been read
    const __amdgpu_buffer_rsrc_t rsrc_y = rsrc_of(q.yb, q.M * q.yb_cs);
    float mv[16] = {};
    if (EXT && q.b.m_vec) load_scales(PB, own_ch, mv);
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      int v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = acc[j][e];
      const int rw[4] = {0, 0, 0, 0};
      const v4i codes = codes16_build<EXT>(q.b, v, rw, mv, false);
      *reinterpret_cast<v4i*>(tile + own_pix[j] * PITCH + own_ch) = codes;
      int off = (pix0 + own_pix[j]) * q.yb_cs + q.yb_off + own_ch;
      off = own_pix[j] < n_own ? off : kOobOffset;
      __builtin_amdgcn_raw_buffer_store_b128(codes, rsrc_y, off, 0, 0);
    }
    meet();
  }

  // ================================================================ layer C
  {
    constexpr int PIECES = NKC / GS;       // of a round
    v4i bf[NKC * 2][TB];                   // all of its activations
#pragma unroll
    for (int k = 0; k < NKC * 2; ++k)
#pragma unroll
      for (int j = 0; j < TB; ++j)
        bf[k][j] = *reinterpret_cast<const v4i*>(tile + own_pix[j] * PITCH + k * 32 + 16 * frag_half);
    const bool has_res = q.res != nullptr;
    const __amdgpu_buffer_rsrc_t rsrc_y = rsrc_of(q.yc, q.M * q.yc_cs);
    const __amdgpu_buffer_rsrc_t rsrc_r = rsrc_of(q.res, has_res ? q.res_bytes : 0);
    int r_off[TB], y_off[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const bool own = own_pix[j] < n_own;
      int r = (pix0 + own_pix[j]) * q.res_cs + q.res_off + own_ch;
      int y = (pix0 + own_pix[j]) * q.yc_cs + q.yc_off + own_ch;
      r_off[j] = own ? r : kOobOffset;
      y_off[j] = own ? y : kOobOffset;
    }
    const int rounds = K2 / MID;
    v4i res[TB], cf[2][2 * GS];            // residual codes of a round, fragments by piece
#pragma unroll
    for (int j = 0; j < TB; ++j) res[j] = v4i{0, 0, 0, 0};
    auto fetch_residual = [&](int round) __attribute__((always_inline)) {
      const int soff = (round < rounds ? round : rounds - 1) * MID;
#pragma unroll
      for (int j = 0; j < TB; ++j) res[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_r, r_off[j], soff, 0);
    };
    auto load_piece = [&](int set) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < 2 * GS; ++h) cf[set][h] = *reinterpret_cast<const v4i*>(ring + f_read + (foff0 ^ (h * 32)));
    };
    if (has_res) fetch_residual(0);
    wait_vmcnt<(D - 1) * FL + TB>();       // the first piece: behind it D - 1 pieces, the stores
    asm volatile("" ::: "memory");
    load_piece(0);
    auto run_round = [&](int round, auto set_c) __attribute__((always_inline)) {
      constexpr int SET = decltype(set_c)::value;
      v16i acc[TB];
      {
        int b[16];
        load16(params + 2 * PB, round * MID + own_ch, b);
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[j][e] = b[e];
      }
#pragma unroll
      for (int pc = 0; pc < PIECES; ++pc) {
        const int cs = PIECES == 1 ? SET : pc & 1;
        own_reads_done();
        issue_filters();
        next_piece();
        // Younger than the next piece: D - 1 pieces and, where a round began since it was requested, the
        // stores and residual loads in front of that round.
        if (pc >= D - 1) wait_vmcnt<(D - 1) * FL>();
        else if (has_res) wait_vmcnt<(D - 1) * FL + 2 * TB>();
        else wait_vmcnt<(D - 1) * FL + TB>();
        asm volatile("" ::: "memory");
        load_piece(cs ^ 1);
#pragma unroll
        for (int h = 0; h < 2 * GS; ++h)
#pragma unroll
          for (int j = 0; j < TB; ++j)
            acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cf[cs][h], bf[2 * GS * pc + h][j], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      float mv[16] = {};
      if (EXT && q.c.m_vec) load_scales(2 * PB, round * MID + own_ch, mv);
      v4i codes[TB];
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        int v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = acc[j][e];
        const int rw[4] = {res[j][0], res[j][1], res[j][2], res[j][3]};
        codes[j] = codes16_build<EXT>(q.c, v, rw, mv, has_res);
      }
#pragma unroll
      for (int j = 0; j < TB; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(codes[j], rsrc_y, y_off[j], round * MID, 0);
      if (has_res) fetch_residual(round + 1);
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
#pragma unroll 1
    for (int round = 0; round < rounds; round += 2) {
      run_round(round, c0);
      if (round + 1 < rounds) run_round(round + 1, c1);
    }
  }
  wait_vmcnt<0>();                         // (requests into LDS behind the last piece)
#endif
}

}  // namespace
}  // namespace q8
