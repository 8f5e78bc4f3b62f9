// The block-tiled build of the persistent 3x3 family (Eq. x / Eq. A' of arxiv 1805.08691):
// 3x3, stride 1, padding 0 or 1, 32 to 128 input channels in sixteens, maps of any width.  Extended layers: 32 and 64
// channels (128 would keep 36 registers of a lane in scratch; 80 and 96 fit, with 248, and are not built).
// A workgroup has 64 output channels (32 where K <= 32); layers of more are as many sets of walkers.
//
// The persistent 3x3 kernel (q8_conv_p3_kernel.h) cuts the output into runs of 128 consecutive
// pixels; the activations such a run reads are the run plus a whole map row on either side, so
// on a wide map (a detector's 300 x 300 first block) a tile would stage many times the pixels
// it computes.  Here a tile is a BLOCK of 8 rows x 16 columns of one image (16 x 16 where K <= 32) and
// its patch the input pixels around it.  Every patch row stands for one input position, so a position
// outside the image is simply a row of zeros in the patch (its load is sent out of the buffer's
// range): no per-tap masks, no selects -- the nine taps of output pixel (ty, tx) read patch rows
// (ty + r) * 18 + tx + s.  Workgroups walk over tiles with the next tile's patch in flight, and codes
// leave through a row-ordered staging tile (an output row of the block is 16 x K contiguous bytes).
//
// What bounds it is the LDS: a fragment of 1 KB per MFMA of 32 clocks and wavefront is all that four
// wavefronts can read.  So a wavefront keeps its 32 channels' filters in registers for the whole launch
// (72 of them, 36 where C = 32, 144 where C = 128: all of the 256 that two wavefronts per SIMD leave
// each), and an MFMA tile being two rows of the block, the rows that tap
// row r reads for one tile are those that row r - 2 reads for the next: five fragments serve the six
// (tap row, tile) pairs of a tap column.  30 LDS reads a tile and wavefront instead of 54, and nobody
// waits for a tile's stores.  64 -> 64 on 300 x 300 x 32 images 160 -> 133 us, on 56 x 56 x 32 9.2 -> 8.9;
// 32 -> 64 on 147 x 147 x 32 34.5 us in the general kernel (half a step per tap), 20.5 here, 32 -> 32 29.2 and
// 15.6 (48 MB: 9.3 us of a copy).  More than 64 channels, the best general build and this one: 64 -> 128 on
// 150 x 150 x 32 73.1 and 58.4, 64 -> 256 on 56 x 56 x 32 24.0 and 19.6, 32 -> 96 on 112 x 112 x 32 29.2 and 21.5,
// 128 -> 128 on 150 x 150 x 32 128 and 101 (2.1 POP/s).  Counts that fill no patch (48 of
// 64; 80, 96 and 112 of 128) have chunks of zeros in it, 80 and 96 three quarters of the products: 80 -> 192 on 71 x 71
// x 32 37.7 (the build chosen before: 43) and 30.1, 48 -> 64 on 150 x 150 x 8 14.0 and 10.7, 112 -> 128 there 33.4 and 26.6.
//
// POOL: the 2x2 maximum with stride 2 behind the layer in the same launch.  Blocks begin on even rows and columns,
// so every window lies in one staging tile: two rows of it in the lane that stores them, the other two in a lane
// of the same sixteen.  The pass that reads the layer's whole output again is gone, and so is its launch: two
// launches / one, us: 64 -> 64 on 300 x 300, 32 images 151 / 142, one 12.4 / 8.8; on 56 x 56 x 64 19.1 / 14.7;
// 32 -> 64 on 147 x 147 x 32 32.0 / 25.2.
#pragma once
#include "q8_conv_ring_kernel.h"

namespace q8 {
namespace {

template <int CB, int WC_>
struct P3bShape {
  static constexpr int NW = 4, WC = WC_, WP = NW / WC, TP = 2;
  static constexpr int TH = WP * TP * 2, TW = 16;                // output block
  static constexpr int PW = TW + 2, PATCH_PIX = (TH + 2) * PW;   // input positions around it
  static constexpr int BP = TH * TW, BC = WC * 32;
  static constexpr int CHUNKS = CB / 16, RPW = 64 / CHUNKS;      // rows per wave-wide load
  static constexpr int PL = (PATCH_PIX + NW * RPW - 1) / (NW * RPW);   // patch loads per wave
  static constexpr int PATCH_BYTES = PL * NW * 1024;
  static constexpr int S_BYTES = BP * BC;                        // staging: codes out
  // (the filters pass through LDS on their way to the registers, behind the first patch buffer)
  static constexpr int A_TAPS = CB <= 64 ? 9 : 3;                // at a time: 128 channels' nine would leave one workgroup a CU
  static constexpr int A_BYTES = A_TAPS * BC * CB, A_LOADS = A_BYTES / 1024;
  static constexpr int LDS_BYTES = PATCH_BYTES + (PATCH_BYTES + S_BYTES > A_BYTES ? PATCH_BYTES + S_BYTES : A_BYTES);
};

// The maximum's output for POOL: pooled rows and columns, address as of pooled pixel (0, 0, 0).
struct P3bPool {
  int8_t* y;
  int bytes, Hp, Wp, cs;
};

// p.n_ptiles = tiles in all (N * tiles_h * tiles_w); div_img and div_row divide a tile's number by the
// tiles of an image and of a row of them, n_ctiles (set by launch_p3b).
// NH: 32-byte halves of a tap that an MFMA takes.  PART: C <= 32 NH channels where the patch has CB, the chunks beyond
// C are zeros.
template <int CB, int WC, int EXT, bool POOL, int NH, bool PART>
__global__ __launch_bounds__(256, 2) void conv_i8_p3b_kernel(const ConvParams p, const P3bPool pool) {
#if defined(__HIP_DEVICE_COMPILE__)
  using Sh = P3bShape<CB, WC>;
  constexpr int NW = Sh::NW, WP = Sh::WP, TP = Sh::TP, BP = Sh::BP, BC = Sh::BC, CHUNKS = Sh::CHUNKS;
  constexpr int TH = Sh::TH, TW = Sh::TW, PW = Sh::PW, PL = Sh::PL;
  constexpr int SLOTS = BC / 16, NQ = 2 * TP + 1;
  static_assert(NH <= CB / 32 && (PART || NH == CB / 32), "the halves lie in the patch, without PART all of them");
  const int tap_bytes = PART ? p.C : CB;
  constexpr int STORES = BP * SLOTS / (NW * 64), ALL_STORES = STORES + POOL;
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  int8_t* const patch = lds;
  int8_t* const stage = lds + 2 * Sh::PATCH_BYTES;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_p = wave % WP, wave_c = wave / WP;
  const int H = p.H, W = p.W, Ho = p.Ho, Wo = p.Wo, pad = p.pad_h;
  // Every workgroup is a walker of its own over tiles walker, + walkers, ..., with 64 (32) channels from ch0 on;
  // those of one tile's channels are on the same XCD, a place apart.
  const int ch_tiles = (p.K + BC - 1) / BC, place = blockIdx.x / kNumXcd;
  const int ch0 = place % ch_tiles * BC, walkers = gridDim.x / ch_tiles;
  const int tiles_w = p.n_ctiles, tiles_img = ((Ho + TH - 1) / TH) * tiles_w;

  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, p.w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_x =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_y =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.y, 0, p.M * p.out_cs, 0x00020000);

  const int frag_row = lane & 31, frag_half = lane >> 5;
  // ---- patch loader: load j of this wave fills patch rows (wave + NW j) RPW + lane / CHUNKS; patch
  // row rho is input position (h0 - pad + rho / 18, w0 - pad + rho % 18) of the tile's image.
  // Slot of 16-byte chunk c in row rho, of the filters and, for 32 channels, of the patch: c ^ ((rho >> 2) & 3)
  // (32 channels: c ^ ((rho >> 3) & 1)), so that sixteen consecutive rows read at one chunk touch every bank once.
  auto slot_of = [](int rho, int chunk) {
    return CHUNKS == 8 ? chunk ^ ((rho >> 1) & 7) : CHUNKS == 4 ? chunk ^ ((rho >> 2) & 3) : chunk ^ ((rho >> 3) & 1);
  };
  // The patch of 64 and more channels by its column x alone (128: two columns fill the banks): an LDS read of 16
  // bytes serves lanes 0-3, 12-15, 20-23 and 24-27 together, i.e. columns 0-3 and 12-15 of one block row and 4-11 of the next.
  auto patch_slot = [&](int rho, int x, int chunk) {
    return CHUNKS == 8 ? chunk ^ ((x >> 1) & 7) : CHUNKS == 4 ? chunk ^ ((x >> 2) & 3) : slot_of(rho, chunk);
  };
  int pr_y[PL], pr_x[PL], pr_off[PL];          // ... and its offset from the block's
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    const int rho = (wave + NW * j) * Sh::RPW + lane / CHUNKS;
    pr_y[j] = rho < Sh::PATCH_PIX ? rho / PW : -4096;            // beyond the patch: never inside
    pr_x[j] = rho % PW;
    const int chunk = patch_slot(rho, pr_x[j], lane % CHUNKS) * 16;
    if (PART && chunk >= p.C) pr_y[j] = -4096;
    pr_off[j] = (pr_y[j] * W + pr_x[j]) * p.in_cs + chunk;
  }
  // tile number -> image and block origin
  auto tile_origin = [&](int tile, int& n, int& h0, int& w0) {
    n = fast_div(tile, p.div_img_m, p.div_img_s);
    const int rem = tile - n * tiles_img;
    const int th = fast_div(rem, p.div_row_m, p.div_row_s);
    h0 = th * TH;
    w0 = (rem - th * tiles_w) * TW;
  };
  auto issue_patch = [&](int tile, int buf) {
    int n, h0, w0;
    tile_origin(tile, n, h0, w0);
    const int origin = ((n * H + h0 - pad) * W + w0 - pad) * p.in_cs;
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      int off = origin + pr_off[j];
      asm volatile("" : "+v"(off));                              // a select, no branch
      const bool inside = ((unsigned)(h0 - pad + pr_y[j]) < (unsigned)H) & ((unsigned)(w0 - pad + pr_x[j]) < (unsigned)W);
      off = inside ? off : kOobOffset;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc_x,
          (__attribute__((address_space(3))) void*)(patch + buf * Sh::PATCH_BYTES + (wave + NW * j) * 1024),
          16, off, 0, 0, 0);
    }
  };

  int8_t* const filters = lds + Sh::PATCH_BYTES;
  auto load_filters = [&](int tap0) {
#pragma unroll
    for (int l = 0; l < Sh::A_LOADS; l += NW) {
      if (l + wave < Sh::A_LOADS) {
        const int row = ((l + wave) * Sh::RPW) % BC + lane / CHUNKS, tap = tap0 + (l + wave) * Sh::RPW / BC;
        const int ch = ch0 + (row & ~31) + row_to_channel(row & 31);
        const int chunk = slot_of(row, lane % CHUNKS) * 16;
        const int off = ch < p.K && (!PART || chunk < p.C) ? ch * p.red_len + chunk : kOobOffset;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrc_w, (__attribute__((address_space(3))) void*)(filters + (l + wave) * 1024), 16, off, tap * tap_bytes, 0, 0);
      }
    }
  };
  load_filters(0);
  int tile = place / ch_tiles * kNumXcd + blockIdx.x % kNumXcd;
  if (tile < p.n_ptiles) issue_patch(tile, 0);
  v16i bias_v;
  {
    int b[16];
    load_bias16(p, ch0 + wave_c * 32 + 16 * frag_half, b);
#pragma unroll
    for (int e = 0; e < 16; ++e) bias_v[e] = b[e];
  }
  float scales[16] = {};
  if (EXT && p.m_vec) load_scale16(p, ch0 + wave_c * 32 + 16 * frag_half, scales);

  // patch offsets of this lane's fragments, the same in every tile: fragment q of tap column s is the
  // two block rows from row 2 TP wave_p + q on, shifted by s columns
  // (from 64 channels on a slot is the column's alone, so the block's rows are a constant apart)
  constexpr int NQO = CHUNKS >= 4 ? 1 : NQ;
  int b_foff[3][NQO][NH];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int q = 0; q < NQO; ++q)
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int rho = (wave_p * TP * 2 + q + (frag_row >> 4)) * PW + (frag_row & 15) + s;
        b_foff[s][q][h] = rho * CB + patch_slot(rho, (frag_row & 15) + s, 2 * h + frag_half) * 16;
      }

  // Copy-out: a lane's two groups, half a block apart; for POOL in rows below one another (without it that order
  // costs 64 -> 64 on 300 x 300 x 32 images 115 -> 120 us).
  constexpr int LPR = TW * SLOTS;                 // lanes of a block row
  static_assert(STORES == 2 && NW * 64 / LPR * 2 == TH, "a lane stores two rows of a block");
  constexpr int DOWN = POOL ? 1 : TH / 2;
  const int out_y = tid / LPR * (POOL ? 2 : 1), out_x = tid % LPR / SLOTS, out_g = tid % SLOTS;
  // Bare barriers behind this wave's own LDS accesses: a fence would also wait for the patch in flight
  // and for the stores.
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // ---- the filters of this wavefront's 32 channels: fragment (tap, half) holds 16 bytes
  v4i af[9][NH];
#pragma unroll
  for (int t0 = 0; t0 < 9; t0 += Sh::A_TAPS) {
    if (t0) load_filters(t0);
    wait_vmcnt<0>();
    meet();
#pragma unroll
    for (int t = 0; t < Sh::A_TAPS; ++t)
#pragma unroll
      for (int h = 0; h < NH; ++h)
        af[t0 + t][h] = *reinterpret_cast<const v4i*>(filters + t * (BC * CB) + (wave_c * 32 + frag_row) * CB +
                                                      slot_of(frag_row, 2 * h + frag_half) * 16);
    meet();
  }
  for (int it = 0; tile < p.n_ptiles; ++it, tile += walkers) {
    const int buf = it & 1;
    const int next = tile + walkers;
    // the other patch buffer is free: every wave passed the barrier behind the last tile
    // This tile's patch has landed; younger than it are the last tile's STORES stores (always issued,
    // lanes outside the map out of range) and the next patch: nobody waits for the stores.
    if (next < p.n_ptiles) {
      issue_patch(next, buf ^ 1);
      if (it) wait_vmcnt<PL + ALL_STORES>();
      else wait_vmcnt<PL>();
    } else {
      if (it) wait_vmcnt<ALL_STORES>();
      else wait_vmcnt<0>();
    }
    meet();

    v16i acc[TP];
#pragma unroll
    for (int j = 0; j < TP; ++j) acc[j] = bias_v;
    if (EXT && p.tap_sums) {        // unsigned input codes: the start values of the pixel's rectangle
      int n, h0, w0;
      tile_origin(tile, n, h0, w0);
#pragma unroll
      for (int j = 0; j < TP; ++j) {
        const int i = (wave_p * TP + j) * 32 + frag_row, h = h0 + i / TW - pad, w = w0 + i % TW - pad;
        const int r_lo = h < 0, r_hi = h + 3 <= H ? 3 : 2, s_lo = w < 0, s_hi = w + 3 <= W ? 3 : 2;
        const int idx = h + pad < Ho && w + pad < Wo ? ((r_lo * 4 + r_hi) * 4 + s_lo) * 4 + s_hi : 0;
        int b[16];
        load_start16(p, idx, ch0 + wave_c * 32 + 16 * frag_half, b);
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = b[e];
      }
    }
    const int8_t* const pbase = patch + buf * Sh::PATCH_BYTES;
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        v4i bf[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          bf[q] = *reinterpret_cast<const v4i*>(pbase + b_foff[s][NQO == 1 ? 0 : q][h] +
                                                (NQO == 1 ? q * PW * CB : 0));
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int j = 0; j < TP; ++j)
            acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[r * 3 + s][h], bf[2 * j + r], acc[j], 0, 0, 0);
      }

    // ---- epilogue through the staging tile (free: the copy-out of the tile before ended in
    // front of a barrier)
    {
      const int slot = wave_c * 2 + (lane >> 5);
#pragma unroll
      for (int j = 0; j < TP; ++j) {
        const int row = (wave_p * TP + j) * 32 + (lane & 31);
        int v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = acc[j][e];
        const int rw[4] = {0, 0, 0, 0};
        *reinterpret_cast<v4i*>(stage + row * BC + ((slot ^ swz_out<SLOTS>(row)) << 4)) =
            codes16_build<EXT>(p, v, rw, scales, false);
      }
    }
    meet();
    {
      int n, h0, w0;
      tile_origin(tile, n, h0, w0);
      const int origin = ((n * Ho + h0) * Wo + w0) * p.out_cs + p.out_off + ch0;
      const bool in = (w0 + out_x < Wo) & (ch0 + out_g * 16 < p.K);
      v4i codes[STORES];
#pragma unroll
      for (int k = 0; k < STORES; ++k) {
        const int y = out_y + k * DOWN, row = y * TW + out_x;
        codes[k] = *reinterpret_cast<const v4i*>(stage + row * BC + ((out_g ^ swz_out<SLOTS>(row)) << 4));
        int off = origin + (y * Wo + out_x) * p.out_cs + out_g * 16;
        asm volatile("" : "+v"(off));
        off = in & (h0 + y < Ho) ? off : kOobOffset;
        __builtin_amdgcn_raw_buffer_store_b128(codes[k], rsrc_y, off, 0, 0);
      }
      if constexpr (POOL) {
        const __amdgpu_buffer_rsrc_t rsrc_p =
            __builtin_amdgcn_make_buffer_rsrc((void*)pool.y, 0, pool.bytes, 0x00020000);
        const bool below = h0 + out_y + 1 < Ho, beside = w0 + out_x + 1 < Wo;     // else the same pixel again
        v4i most;
#pragma unroll
        for (int q = 0; q < 4; ++q) {             // 16-bit lanes: odd bytes in place, even ones shifted
          auto larger = [](int u, int v) __attribute__((always_inline)) {
            typedef short v2s __attribute__((ext_vector_type(2)));
            return __builtin_bit_cast(int, __builtin_elementwise_max(__builtin_bit_cast(v2s, u), __builtin_bit_cast(v2s, v)));
          };
          // the pixel to the right is SLOTS lanes on, in the same row of 16 lanes for every even one
          auto right = [](int u) __attribute__((always_inline)) {
            return __builtin_amdgcn_update_dpp(u, u, 0x100 + SLOTS, 0xf, 0xf, false);
          };
          const int w = codes[0][q], w1 = below ? codes[1][q] : w;
          const int odd = larger(w, w1), even = larger(w << 8, w1 << 8);
          const int odd1 = right(odd), even1 = right(even);
          most[q] = (int)__builtin_amdgcn_perm((unsigned)larger(odd, beside ? odd1 : odd),
                                               (unsigned)larger(even, beside ? even1 : even), 0x07030501u);
        }
        const int hp = (h0 + out_y) / 2, wp = (w0 + out_x) / 2;
        int off = ((n * pool.Hp + hp) * pool.Wp + wp) * pool.cs + ch0 + out_g * 16;
        asm volatile("" : "+v"(off));
        off = in & (out_x % 2 == 0) & (hp < pool.Hp) & (wp < pool.Wp) ? off : kOobOffset;
        __builtin_amdgcn_raw_buffer_store_b128(most, rsrc_p, off, 0, 0);
      }
    }
    // every wave has read this tile's patch and the staging tile before the next pass
    // requests a patch into this buffer / writes codes into the staging tile
    meet();
  }
  wait_vmcnt<0>();
#endif
}

inline bool p3b_applicable(const ConvParams& p) {
  return p.R == 3 && p.S == 3 && p.stride_h == 1 && p.stride_w == 1 && p.dil_h == 1 && p.dil_w == 1 &&
         p.pad_h == p.pad_w && p.pad_h <= 1 && p3b_channels(p.C, is_extended(p)) && p.S4 == 0 && (p.K & 15) == 0 &&
         p.vec16 && !p.res && !p.acc_dump && !p.y_f32 && !p.y_deq && !p.w2 && (long)p.M * p.out_cs < 0x7fffffffL;
}

template <int CB, int WC, int EXT, bool POOL, int NH = CB / 32, bool PART = NH != CB / 32>
int launch_p3b_build(ConvParams& p, hipStream_t stream, const P3bPool& pool) {
  using Sh = P3bShape<CB, WC>;
  if (PART ? p.C > 32 * NH || p.C % 16 != 0 : p.C != CB) return Q8_EUNSUPPORTED;
  const long tiles_w = (p.Wo + Sh::TW - 1) / Sh::TW, tiles_h = (p.Ho + Sh::TH - 1) / Sh::TH;
  const long tiles = (long)p.N * tiles_h * tiles_w;
  if (tiles > 0x7fffffffL) return Q8_EUNSUPPORTED;
  p.n_ptiles = (int)tiles;
  p.n_ctiles = (int)tiles_w;
  const FastDiv img = make_fast_div((unsigned)(tiles_h * tiles_w)), row = make_fast_div((unsigned)tiles_w);
  p.div_img_m = img.m; p.div_img_s = img.s;
  p.div_row_m = row.m; p.div_row_s = row.s;
  auto kernel = conv_i8_p3b_kernel<CB, WC, EXT, POOL, NH, PART>;
  static const int resident = [&]() {
    int per_cu = 0, dev = 0, cus = 256;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      cus = prop.multiProcessorCount;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel),
                                                     256, Sh::LDS_BYTES) != hipSuccess || per_cu < 1)
      per_cu = 1;
    return per_cu * cus;
  }();
  // as many workgroups as stay resident, every one with the same number of tiles (+- 1); with several channel
  // tiles the walkers fill whole rows of XCDs (those of more than are resident follow them)
  const int ch_tiles = (p.K + Sh::BC - 1) / Sh::BC, most = resident / ch_tiles / kNumXcd * kNumXcd;
  const int places = ch_tiles == 1 ? resident : most < kNumXcd ? kNumXcd : most;
  const int passes = (p.n_ptiles + places - 1) / places;
  int walkers = (p.n_ptiles + passes - 1) / passes;
  if (ch_tiles > 1) walkers = (walkers + kNumXcd - 1) / kNumXcd * kNumXcd;
  if ((long)walkers * ch_tiles > 0x7fffffffL) return Q8_EUNSUPPORTED;
  const int grid = walkers * ch_tiles;
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), Sh::LDS_BYTES, stream, p, pool);
  return q8_launch_status();
}

// The build for p3b_channels: the smallest patch that holds C, and of it the halves that C reaches into.
template <int EXT, bool POOL = false>
int launch_p3b(ConvParams& p, hipStream_t stream, const P3bPool& pool = {}) {
  if constexpr (!EXT) {
    if (p.C > 112) return launch_p3b_build<128, 2, 0, POOL>(p, stream, pool);
    if (p.C > 96) return launch_p3b_build<128, 2, 0, POOL, 4, true>(p, stream, pool);
    if (p.C > 64) return launch_p3b_build<128, 2, 0, POOL, 3>(p, stream, pool);
    if (p.C > 32 && p.C < 64) return launch_p3b_build<64, 2, 0, POOL, 2, true>(p, stream, pool);
  }
  if (p.C > 32) return launch_p3b_build<64, 2, EXT, POOL>(p, stream, pool);
  if constexpr (!EXT) {                  // (the extended builds are kept to K > 32)
    if (p.K <= 32) return launch_p3b_build<32, 1, 0, POOL>(p, stream, pool);
  }
  return launch_p3b_build<32, 2, EXT, POOL>(p, stream, pool);
}

}  // namespace
}  // namespace q8
