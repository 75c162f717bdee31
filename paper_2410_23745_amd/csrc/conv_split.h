// fp32 contraction on the bf16 matrix cores, device side: parameter record, kernel template and launch helper.
// (fp32_parts.h: how a value is split, and which results are summed again.)
#pragma once
#include "conv_mfma.h"
#include "fp32_parts.h"

namespace syno {

struct SplitParams : MfmaPlace {
  int32_t x_bytes, w_bytes;          // one LDS buffer of the source rows and of the weights
  int32_t x_items;                   // X items (one pixel x 8 channels) per thread
  int32_t octet;                     // pixels between channel octets in LDS: a multiple of 16
  int32_t adjoint;                   // weights of backward-data: taps reversed (selects the instantiation)
  uint32_t m_slots;                  // ceil(2^32 / n_slots), 0 for 1
  int32_t phases;                    // 2x2 windows: output channels are (c, a, b) and the result is the image whose pixel (2h + a, 2w + b) of
                                     // channel c that is, in the place of the phase planes
};

namespace {

constexpr int kSplitChannels = 32;   // channels per chunk = one MFMA k-step per tap
// taps whose weights lie in LDS at a time: the nine of a 3x3 window go in as five and four
constexpr int split_taps(int T) { return T == 9 ? 5 : T; }
constexpr int split_subs(int T) { return T == 9 ? 2 : 1; }

// A 16 x 16 tile of results (pixels m0.. of the block, output channels o0.. of the group) with the fp32 matrix instructions,
// on the operands where they lie: for tiles with results that the parts cannot give, by the wave that stores them.  A tap's
// sum joins a result only where the tap lies inside the image.  Lane: pixels 4 * (lane / 16) + 0..3, channel lane % 16.
// Bound by the loads' round trips: 32x64x64 56x56 takes 139 us with one infinity in X and 330 of NaNs alone, 62 without.
template <int T, bool ADJ>
__device__ __forceinline__ floatx4 split_plain_tile(const SplitParams& p, const float* __restrict__ X, const float* __restrict__ W,
                                                    int g, int o0, int R0, int m0, int block_px, int lane) {
  auto place = [&](int m, int& n, int& h, int& w) {
    const int i = fdiv(m, p.m_wo);
    w = m - i * p.Wo;
    n = fdiv(R0 + i, p.m_ho);
    h = R0 + i - n * p.Ho;
  };
  auto row_of = [&](int h, int kh) { return p.h_wrap ? (h + p.h_shift + p.h_shift_g * g) % p.Hi : h * p.sh + kh - p.ph; };
  int n, h, w, at[T];
  place(min(m0 + (lane & 15), block_px - 1), n, h, w);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int kh = t / p.KW, r = row_of(h, kh), x = w * p.sw + t - kh * p.KW - p.pw;
    at[t] = n * p.xs_n + min(max(r, 0), p.Hi - 1) * p.Wi + min(max(x, 0), p.Wi - 1);
  }
  const float* const xg = X + (int64_t)g * p.Cg * p.xs_c;
  const float* const wo = W + (int64_t)g * p.ws_g + (int64_t)min(o0 + (lane & 15), p.Og - 1) * p.ws_o;
  floatx4 sum[T];
#pragma unroll
  for (int t = 0; t < T; ++t) sum[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < p.Cg; c0 += 4) {
    const int c = min(c0 + (lane >> 4), p.Cg - 1);
    const bool live = c0 + (lane >> 4) < p.Cg;
    const float *const xc = xg + (int64_t)c * p.xs_c, *const wc = wo + (int64_t)c * p.ws_c;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float a = xc[at[t]], b = wc[ADJ ? T - 1 - t : t];
      sum[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(live ? a : 0.f, live ? b : 0.f, sum[t], 0, 0, 0);
    }
  }
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    place(min(m0 + 4 * (lane >> 4) + j, block_px - 1), n, h, w);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int kh = t / p.KW, r = row_of(h, kh), x = w * p.sw + t - kh * p.KW - p.pw;
      if (r >= 0 && r < p.Hi && x >= 0 && x < p.Wi) v[j] += sum[t][j];
    }
  }
  return v;
}

// A workgroup (8 waves, one per CU) owns TR whole result rows x BN output channels, like conv_mfma, and walks the reduction
// in chunks of 32 channels, the weights of a 3x3 window in two groups of taps per chunk ("stages").
//  - X lies in LDS as [channel octet][row slot][pixel][part] 16-byte pieces: with the 48-byte pixel pitch and octets a
//    multiple of 256 bytes apart the 64 lanes of a fragment read meet no bank twice (a kernel of such reads alone: 4.4 cycles
//    each, 8.1 with any other distance; the writes of the staging do conflict), and taps and parts are constant offsets.
//  - W lies as [tap][part][channel octet][output channel].
//  - Staging is dealt evenly over the 512 threads, because a wave that stages more than its neighbours is waited for at the
//    next barrier: X items are single pixels x 8 channels (adjacent lanes adjacent pixels, XI items per thread), W items
//    BN/16 channels x T taps of one output channel (adjacent lanes adjacent output channels), one per thread.
//  - Values are split on their way into LDS: 11 vector instructions per pair, against 6 * 16 * TN cycles of matrix work per
//    fragment that every split value is read for.
//  - With two buffers a stage costs one barrier: the next stage is written, and the one after it requested, in pieces
//    between the tiles of the first k-step.  MODE 2: two buffers of X and W; 1: two of W; 0: one of either (what fits 160 KB).
// WM x WN x WK waves over pixels, output channels and taps; a wave has NTL (or NTL-1) x TN tiles of 16 x 16.  T: taps.
// ADJ: the weights of backward-data, read from the forward layout [forward output channel][output channel][reversed taps].
template <int WM, int WN, int WK, int NTL, int TN, int T, int MODE, int XI, bool ADJ>
__global__ __launch_bounds__(512) void conv_split(const SplitParams p, const float* __restrict__ X, const float* __restrict__ W,
                                                  float* __restrict__ out) {
  static_assert(WM * WN * WK == 8, "eight waves");
  constexpr int NT = 512, BN = WN * TN * 16;
  constexpr int CW = BN / 16;                      // channels of a weight item: BN * 32 / CW = 512 items
  constexpr int TS = split_taps(T), NSUB = split_subs(T);
  extern __shared__ __align__(16) unsigned char smem[];

  long long* const probe = reinterpret_cast<long long*>(((unsigned long long)p.probe_hi << 32) | p.probe_lo);
  if (probe && threadIdx.x == 0) {
    probe[(long long)blockIdx.x * 4 + 0] = wall_clock64();
    probe[(long long)blockIdx.x * 4 + 1] = clock64();
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int widx = __builtin_amdgcn_readfirstlane(tid >> 6);
  // waves w and w+4 share a SIMD: the second four take their pixel tiles (or taps) rotated, so that a wave with a tile or a
  // tap more meets one with less
  int wm, wn = 0, wk = 0;
  if constexpr (WM == 4) {
    wm = (widx + 2 * (widx >> 2)) & 3;
    if constexpr (WN == 2) wn = widx >> 2; else wk = widx >> 2;
  } else {
    wm = widx >> 2;
    wk = (widx + wm) & 3;
  }
  // (until the first load is out a call does nothing else: 5000 cycles with divisions and a walk over the images)
  int g, mb, nb;
  tile_of_block(p, blockIdx.x, g, mb, nb);
  const int R0 = mb * p.TR;
  const int rows = min(p.TR, p.rows_total - R0);

  const int n0 = div_by(R0, p.m_ho), h0 = R0 - n0 * p.Ho;
  // ---- what this thread stages: one weight item, XI X items
  const float* Wg = W + (int64_t)g * p.ws_g + (int64_t)nb * BN * p.ws_o;
  const char* wbase = reinterpret_cast<const char*>(Wg);
  const int w_o = tid & (BN - 1), w_c = tid / BN * CW;
  const uint32_t w_off = nb * BN + w_o < p.Og ? (uint32_t)(w_o * p.ws_o + w_c * p.ws_c) * 4u : 0u;
  const int w_loff = p.lds_w_off + ((w_c >> 3) * BN + w_o) * 16 + (w_c & 7) * 2;
  const char* xbase = reinterpret_cast<const char*>(X + (int64_t)g * p.Cg * p.xs_c);
  const int first_slots = (min(rows, p.Ho - h0) - 1) * p.sh + p.KH;
  const int shift = p.h_wrap ? (p.h_shift + p.h_shift_g * g) % p.Hi : 0;
  uint32_t x_off[XI];
  int x_loff[XI], x_cg[XI], x_zero[XI];
#pragma unroll
  for (int k = 0; k < XI; ++k) {
    const int per_cg = p.n_slots * p.Wi, idx = tid + k * NT;
    const int cg = div_by(idx, p.m_pcg), rem = idx - cg * per_cg;
    const int s = div_by(rem, p.m_vpr), x = rem - s * p.Wi;
    int n, r;
    row_of_slot(p, R0, n0, h0, first_slots, shift, s, n, r);
    const bool live = cg < 4 && (unsigned)r < (unsigned)p.Hi && n < p.n_images;
    const int at = (cg * p.octet + s * p.Wp + x + p.pw) * 48;
    x_cg[k] = cg * 8;
    x_off[k] = live ? (uint32_t)(n * p.xs_n + r * p.Wi + x + x_cg[k] * p.xs_c) * 4u : 0u;
    x_loff[k] = live ? at : -1;
    x_zero[k] = cg < 4 && !live ? at : -1;       // a row outside the image: zeroed once and never written
  }

  // values on their way from memory: those staged next, and (xn, wn) those after them where a stage is shorter than a
  // memory round trip
  constexpr bool XN = MODE == 2 && NSUB == 1, WN2 = MODE == 2;
  float xr[XI][8], xn[XN ? XI : 1][8], wr[CW * T], wn2[WN2 ? CW * T : 1];
  const int last = p.n_chunks - 1;

  // Loads are a wave-uniform base plus a 32-bit lane offset and stand in straight-line code (a load whose registers meet
  // other values at a branch's end is waited for right there): what has no source reads some valid element, and chunks past
  // the last one read it again.  A last chunk of fewer than 32 channels starts early, and the weights of the channels that
  // the chunk before has had are zero.
  constexpr int FW = 2;                            // pieces that a chunk's weights are requested in
  auto start_of = [&](int ch) {
    int c0 = __builtin_amdgcn_readfirstlane(min(min(ch, last) * kSplitChannels, p.Cg - kSplitChannels));
    asm volatile("" : "+s"(c0));      // (addresses are formed where they are used, not kept in registers from the chunk's start on)
    return c0;
  };
  const int64_t x_step = (int64_t)p.xs_c * 4, w_step = (int64_t)p.ws_c * 4;
  auto fetch_x = [&](int ch, auto k_c, float (&dst)[XI][8]) {           // item k
    constexpr int k = decltype(k_c)::value;
    const char* row = xbase + start_of(ch) * x_step;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      dst[k][j] = *reinterpret_cast<const float*>(row + x_off[k]);
      row += x_step;
    }
  };
  auto stage_x = [&](int ch, auto k_c) {
    constexpr int k = decltype(k_c)::value;
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) split_pair(xr[k][2 * j], xr[k][2 * j + 1], h[j], m[j], l[j]);
    if (x_loff[k] >= 0) {
      uint4* d = reinterpret_cast<uint4*>(smem + x_loff[k] + (MODE == 2 && (ch & 1) ? p.x_bytes : 0));
      d[0] = make_uint4(h[0], h[1], h[2], h[3]);
      d[1] = make_uint4(m[0], m[1], m[2], m[3]);
      d[2] = make_uint4(l[0], l[1], l[2], l[3]);
    }
    if constexpr (XN) {
#pragma unroll
      for (int j = 0; j < 8; ++j) xr[k][j] = xn[k][j];
    }
    __builtin_amdgcn_sched_barrier(0);             // (one piece's values at a time: registers)
  };
  // the weights of a whole chunk: CW channels x T taps, in memory order
  auto fetch_w = [&](int ch, auto part_c, auto& dst) {
    constexpr int part = decltype(part_c)::value;
    // N adjacent floats as 16- and 4-byte loads
    auto run = [&](const char* src, auto first_c, auto n_c) {
      constexpr int first = decltype(first_c)::value, N = decltype(n_c)::value;
      static_for<0, N / 4>([&](auto q_c) {
        constexpr int q = decltype(q_c)::value * 4;
        const f32x4_unaligned v = *reinterpret_cast<const f32x4_unaligned*>(src + 4 * q);
        dst[first + q] = v[0]; dst[first + q + 1] = v[1]; dst[first + q + 2] = v[2]; dst[first + q + 3] = v[3];
      });
      static_for<N / 4 * 4, N>([&](auto e_c) {
        constexpr int e = decltype(e_c)::value;
        dst[first + e] = *reinterpret_cast<const float*>(src + 4 * e);
      });
    };
    if constexpr (!ADJ) {
      if (part <= 0) run(wbase + start_of(ch) * (int64_t)(T * 4) + w_off, std::integral_constant<int, 0>{}, std::integral_constant<int, CW * T>{});
    } else {
      const char* row = wbase + (start_of(ch) + (part > 0 ? CW / FW : 0)) * w_step;
      static_for<0, CW>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        if (part >= 0 && j * FW / CW != part) return;
        run(row + w_off, std::integral_constant<int, j * T>{}, std::integral_constant<int, T>{});
        row += w_step;
      });
    }
  };
  // one tap of the weight item (the adjoint's taps are the reversed ones)
  auto stage_w = [&](int ch, auto tap_c, int buf) {
    constexpr int tap = decltype(tap_c)::value, i = tap >= TS ? tap - TS : tap;
    const bool live = p.Cg - kSplitChannels + w_c >= ch * kSplitChannels || ch * kSplitChannels <= p.Cg - kSplitChannels;
    uint32_t h[CW / 2], m[CW / 2], l[CW / 2];
#pragma unroll
    for (int j = 0; j < CW / 2; ++j) {
      constexpr int t = ADJ ? T - 1 - tap : tap;
      split_pair(live ? wr[2 * j * T + t] : 0.f, live ? wr[(2 * j + 1) * T + t] : 0.f, h[j], m[j], l[j]);
    }
    unsigned char* d = smem + w_loff + (buf ? p.w_bytes : 0) + i * kPlanes * 4 * BN * 16;
    auto put = [&](int plane, const uint32_t (&v)[CW / 2]) {
      if constexpr (CW == 2) *reinterpret_cast<uint32_t*>(d + plane * 4 * BN * 16) = v[0];
      else if constexpr (CW == 4) *reinterpret_cast<uint2*>(d + plane * 4 * BN * 16) = make_uint2(v[0], v[1]);
      else *reinterpret_cast<uint4*>(d + plane * 4 * BN * 16) = make_uint4(v[0], v[1], v[2], v[3]);
    };
    put(0, h); put(1, m); put(2, l);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto take_w = [&]() {                            // the weights after next become the next ones
    if constexpr (WN2) {
#pragma unroll
      for (int e = 0; e < CW * T; ++e) wr[e] = wn2[e];
    }
  };
  constexpr std::integral_constant<int, -1> all{};
  auto whole_x = [&](int ch) { static_for<0, XI>([&](auto i) { stage_x(ch, i); }); };
  auto load_x = [&](int ch, auto& dst) { static_for<0, XI>([&](auto i) { fetch_x(ch, i, dst); }); };
  auto first_w = [&](int ch, int buf) { static_for<0, TS>([&](auto i) { stage_w(ch, i, buf); }); };     // first group of taps
  auto rest_w = [&](int ch, int buf) { static_for<TS, T>([&](auto i) { stage_w(ch, i, buf); }); };

  fetch_w(0, all, wr);
  load_x(0, xr);
  if constexpr (WN2 && NSUB == 2) fetch_w(1, all, wn2);
  // while the first loads travel: what the window's padding reads is zeroed once and never written (rows outside the image, the
  // columns on either side of the rows)
  constexpr int XB = MODE == 2 ? 2 : 1;
#pragma unroll
  for (int k = 0; k < XI; ++k)
    if (x_zero[k] >= 0) {
#pragma unroll
      for (int b = 0; b < XB; ++b)
#pragma unroll
        for (int j = 0; j < 3; ++j) reinterpret_cast<uint4*>(smem + x_zero[k] + b * p.x_bytes)[j] = make_uint4(0, 0, 0, 0);
    }
  if (p.KW > 1)
    for (int i = tid; i < 4 * p.n_slots; i += NT) {
      const int cg = div_by(i, p.m_slots), s = i - cg * p.n_slots;
      for (int e = 0; e < p.KW - 1; ++e) {
        unsigned char* d = smem + (cg * p.octet + s * p.Wp + (e < p.pw ? e : p.Wi + e)) * 48;
#pragma unroll
        for (int b = 0; b < XB; ++b)
#pragma unroll
          for (int j = 0; j < 3; ++j) reinterpret_cast<uint4*>(d + b * p.x_bytes)[j] = make_uint4(0, 0, 0, 0);
      }
    }
  // ---- per-lane operand bases
  const int block_px = rows * p.Wo;
  const int MT = (block_px + 15) >> 4;
  const int tiles_base = MT / WM, tiles_extra = MT - tiles_base * WM;
  const int my_tiles = tiles_base + (wm < tiles_extra ? 1 : 0);
  const int my_first = wm * tiles_base + min(wm, tiles_extra);
  int a_base[NTL];
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    int m = (my_first + t) * 16 + (lane & 15);
    if (t >= my_tiles || m >= block_px) m = 0;
    const int i = div_by(m, p.m_wo), w = m - i * p.Wo;
    // (every image before the row's adds KH - sh slots)
    const int slot = p.h_wrap ? i : i * p.sh + (p.KH - p.sh) * div_by(h0 + i, p.m_ho);
    a_base[t] = (slot * p.Wp + w * p.sw + (lane >> 4) * p.octet) * 48;
  }
  const int b_base = p.lds_w_off + ((lane >> 4) * BN + wn * TN * 16 + (lane & 15)) * 16;

  floatx4 acc[NTL][TN];
#pragma unroll
  for (int t = 0; t < NTL; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u) acc[t][u] = floatx4{0.f, 0.f, 0.f, 0.f};

  // ---- the k-steps of one stage: this wave's share of its taps.  `P` pieces of staging work are done along with the first
  // k-step, spread over its tiles.
  auto multiply = [&](int ch, auto sub_c, int wbuf, auto pieces_c, auto&& piece) {
    constexpr int sub = decltype(sub_c)::value, n = sub ? T - TS : TS, P = decltype(pieces_c)::value;
    static_assert(n >= WK, "every wave has a k-step in every stage");
    const int q0 = wk * n / WK, q1 = (wk + 1) * n / WK;
    const int xoff = MODE == 2 && (ch & 1) ? p.x_bytes : 0;
    const int woff = b_base + (wbuf ? p.w_bytes : 0);
    auto a_off = [&](int q) {
      const int tap = sub * TS + q, kh = T == 4 ? tap / 2 : p.KW == 3 ? tap / 3 : tap, kw = T == 4 ? tap & 1 : p.KW == 3 ? tap - 3 * kh : 0;
      return xoff + (kh * p.Wp + kw) * 48;
    };
    uint4 a[2][kPlanes], b[TN][kPlanes];
    auto read_a = [&](uint4 (&d)[kPlanes], int base) {
#pragma unroll
      for (int s = 0; s < kPlanes; ++s) d[s] = *reinterpret_cast<const uint4*>(smem + base + s * 16);
    };
    auto read_b = [&](int q) {
#pragma unroll
      for (int u = 0; u < TN; ++u)
#pragma unroll
        for (int s = 0; s < kPlanes; ++s)
          b[u][s] = *reinterpret_cast<const uint4*>(smem + woff + u * 256 + (q * kPlanes + s) * 4 * BN * 16);
    };
    // The five small products of a tile are summed on their own and join its accumulator one tile later: two roundings at
    // the accumulator's magnitude per k-step instead of six (relative error 0.6 of it), and no wait for the matrix pipe.
    floatx4 small[TN];
    auto mfmas = [&](const uint4 (&x)[kPlanes], floatx4 (&c)[TN], floatx4 (&sum)[TN]) {
      constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int s = 0; s < 6; ++s)
#pragma unroll
        for (int u = 0; u < TN; ++u) {
          const bf16x8 av = __builtin_bit_cast(bf16x8, x[pa[s]]), bv = __builtin_bit_cast(bf16x8, b[u][pb[s]]);
          if (s == 5) c[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c[u], 0, 0, 0);
          else sum[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, s == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : sum[u], 0, 0, 0);
        }
    };
#pragma unroll
    for (int u = 0; u < TN; ++u) small[u] = floatx4{0.f, 0.f, 0.f, 0.f};
    int off = a_off(q0);
    read_b(q0);
    read_a(a[0], a_base[0] + off);
    auto kstep = [&](int q, auto first_c) {
      const int next = a_off(min(q + 1, q1 - 1));
      static_for<0, NTL>([&](auto t_c) {
        constexpr int t = decltype(t_c)::value;
        if constexpr (t + 1 < NTL) read_a(a[(t + 1) & 1], a_base[t + 1] + off);
        else read_a(a[(t + 1) & 1], a_base[0] + next);
        constexpr int before = (t + NTL - 1) % NTL;
        floatx4 sum[TN];
        if (t < NTL - 1 || NTL == 1 || my_tiles == NTL) {
          mfmas(a[t & 1], acc[t], sum);
#pragma unroll
          for (int u = 0; u < TN; ++u) { if constexpr (NTL > 1) acc[before][u] += small[u]; }
          // the next tile's reads go out before this one's products
          __builtin_amdgcn_sched_group_barrier(0x100, kPlanes, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 6 * TN, 0);
        } else {
#pragma unroll
          for (int u = 0; u < TN; ++u) { acc[before][u] += small[u]; sum[u] = floatx4{0.f, 0.f, 0.f, 0.f}; }
        }
#pragma unroll
        for (int u = 0; u < TN; ++u) {
          if constexpr (NTL > 1) small[u] = sum[u];
          else acc[0][u] += sum[u];
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(first_c)::value) static_for<t * P / NTL, (t + 1) * P / NTL>(piece);
      });
      if constexpr (NTL & 1) {
#pragma unroll
        for (int s = 0; s < kPlanes; ++s) a[0][s] = a[1][s];
      }
      if (q + 1 < q1) read_b(q + 1);
      off = next;
    };
    kstep(q0, std::true_type{});
    for (int q = q0 + 1; q < q1; ++q) kstep(q, std::false_type{});
#pragma unroll
    for (int u = 0; u < TN; ++u) { if constexpr (NTL > 1) acc[NTL - 1][u] += small[u]; }
  };

  // ---- the stages
  constexpr std::integral_constant<int, 0> s0{};
  constexpr std::integral_constant<int, 1> s1{};
  if constexpr (XN) load_x(1, xn);
  if constexpr (MODE == 2) whole_x(0);
  if constexpr (MODE >= 1) first_w(0, 0);
  if constexpr (MODE == 2) { if constexpr (XN) load_x(2, xn); else load_x(1, xr); }
  if constexpr (MODE >= 1 && NSUB == 1) {
    fetch_w(1, all, wr);
    if constexpr (WN2) fetch_w(2, all, wn2);
  }
  for (int ch = 0; ch < p.n_chunks; ++ch) {
    __syncthreads();
    if constexpr (MODE < 2) {                   // what has one buffer is written between two barriers
      whole_x(ch);
      if constexpr (MODE == 0) first_w(ch, 0);
      __syncthreads();
    }
    const int buf = MODE >= 1 && NSUB == 1 ? ch & 1 : 0;
    constexpr int FXP = MODE < 2 ? XI : 0;      // X of the next chunk is requested in the first stage, or staged in the last
    if constexpr (NSUB == 2 && MODE >= 1) {
      constexpr int P = FXP + (T - TS) + FW;
      multiply(ch, s0, 0, std::integral_constant<int, P>{}, [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        if constexpr (i < FXP) fetch_x(ch + 1, i_c, xr);
        else if constexpr (i < FXP + T - TS) stage_w(ch, std::integral_constant<int, TS + i - FXP>{}, 1);
        else {
          if constexpr (i == FXP + T - TS) take_w();
          if constexpr (WN2) fetch_w(ch + 2, std::integral_constant<int, i - FXP - (T - TS)>{}, wn2);
          else fetch_w(ch + 1, std::integral_constant<int, i - FXP - (T - TS)>{}, wr);
        }
      });
      __syncthreads();
      constexpr int XS = MODE == 2 ? XI : 0, Q = TS + 2 * XS;
      multiply(ch, s1, 1, std::integral_constant<int, Q>{}, [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        if constexpr (i < XS) stage_x(ch + 1, i_c);
        else if constexpr (i < 2 * XS) fetch_x(ch + 2, std::integral_constant<int, i - XS>{}, xr);
        else stage_w(ch + 1, std::integral_constant<int, i - 2 * XS>{}, 0);
      });
    } else if constexpr (NSUB == 2) {
      multiply(ch, s0, 0, std::integral_constant<int, XI>{}, [&](auto i_c) { fetch_x(ch + 1, i_c, xr); });
      __syncthreads();
      rest_w(ch, 0);
      __syncthreads();
      multiply(ch, s1, 0, std::integral_constant<int, FW>{}, [&](auto i_c) { fetch_w(ch + 1, i_c, wr); });
    } else if constexpr (MODE == 0) {
      multiply(ch, s0, 0, std::integral_constant<int, XI + FW>{}, [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        if constexpr (i < XI) fetch_x(ch + 1, i_c, xr);
        else fetch_w(ch + 1, std::integral_constant<int, i - XI>{}, wr);
      });
    } else {
      constexpr int XS = MODE == 2 ? XI : 0, P = XS + XI + TS + FW;
      multiply(ch, s0, buf, std::integral_constant<int, P>{}, [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        if constexpr (i < XS) stage_x(ch + 1, i_c);
        else if constexpr (i < XS + XI) {
          if constexpr (XN) fetch_x(ch + 3, std::integral_constant<int, i - XS>{}, xn);
          else fetch_x(ch + 1, std::integral_constant<int, i - XS>{}, xr);
        } else if constexpr (i < XS + XI + TS) stage_w(ch + 1, std::integral_constant<int, i - XS - XI>{}, buf ^ 1);
        else {
          if constexpr (i == XS + XI + TS) take_w();
          if constexpr (WN2) fetch_w(ch + 3, std::integral_constant<int, i - XS - XI - TS>{}, wn2);
          else fetch_w(ch + 2, std::integral_constant<int, i - XS - XI - TS>{}, wr);
        }
      });
    }
  }

  // ---- store: lane holds 4 consecutive pixels (rows of D) of one channel (column of D)
  const int img_px = p.Ho * p.Wo;
  bool odd = false;                // some result of this lane is none that the parts can give
  auto element = [&](int m, int o) -> int64_t {       // pixel m of the block, output channel o -> element of the result
    const int i = fdiv(m, p.m_wo), r = R0 + i, n = fdiv(r, p.m_ho);
    if constexpr (T == 4)
      if (p.phases) return (int64_t)n * p.os_n + (int64_t)(o >> 2) * (4 * p.os_o) + (2 * (r - n * p.Ho) + (o >> 1 & 1)) * (2 * p.Wo) + 2 * (m - i * p.Wo) + (o & 1);
    return (int64_t)n * p.os_n + (int64_t)(g * p.Og + o) * p.os_o + (r - n * p.Ho) * p.Wo + (m - i * p.Wo);
  };
  auto store = [&](int t, int u, floatx4 v) {
    const int m0 = (my_first + t) * 16 + 4 * (lane >> 4);
    const int o = nb * BN + (wn * TN + u) * 16 + (lane & 15);
    if (o >= p.Og || m0 >= block_px || t >= my_tiles) return;
    const int i0 = fdiv(m0, p.m_wo), rho = R0 + i0;
    const int n = fdiv(rho, p.m_ho), px = (rho - n * p.Ho) * p.Wo + (m0 - i0 * p.Wo);
    const int64_t off = (int64_t)n * p.os_n + (int64_t)(g * p.Og + o) * p.os_o + px;
    v *= kResultScale;
    // (one test for the four values; each is looked at again below)
    odd |= !trusted_result(fabsf(v[0]) + fabsf(v[1]) + fabsf(v[2]) + fabsf(v[3]));
    if constexpr (T == 4)
      if (p.phases && (p.Wo & 3) == 0) {
        // four pixels of a row of one phase: the lane beside this one has the same of the phase between them, and each of the two
        // stores four adjacent pixels of the image (the planes and their way back were 11 of 62 us at 32x64x56x56)
        const bool b = o & 1;
        const float give0 = b ? v[0] : v[2], give1 = b ? v[1] : v[3];
        const float take0 = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give0), 0xb1, 0xf, 0xf, true));
        const float take1 = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give1), 0xb1, 0xf, 0xf, true));
        const f32x4_unaligned w = {b ? take0 : v[0], b ? v[2] : take0, b ? take1 : v[1], b ? v[3] : take1};
        *reinterpret_cast<f32x4_unaligned*>(out + (element(m0, o & ~1) + (b ? 4 : 0))) = w;
        return;
      }
    if ((T != 4 || !p.phases) && m0 + 3 < block_px && px + 3 < img_px && (off & 3) == 0) {
      *reinterpret_cast<float4*>(out + off) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (m0 + j < block_px) out[element(m0 + j, o)] = v[j];
    }
  };
  int first_tile = 0, tile_step = 1;        // the tiles of this wave's area that it stores
  if constexpr (WK == 1) {
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) store(t, u, acc[t][u]);
  } else {
    // the waves that split the taps meet in LDS: [wave][tile][lane]; every one then adds up and stores a share of the tiles
    floatx4* red = reinterpret_cast<floatx4*>(smem);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) red[(((wk * WM + wm) * NTL + t) * TN + u) * 64 + lane] = acc[t][u];
    __syncthreads();
    first_tile = wk; tile_step = WK;
    for (int i = wk; i < NTL * TN; i += WK) {
      floatx4 v = red[(wm * NTL * TN + i) * 64 + lane];
#pragma unroll
      for (int k = 1; k < WK; ++k) v += red[((k * WM + wm) * NTL * TN + i) * 64 + lane];
      store(i / TN, i % TN, v);
    }
  }
  // (see split_pair; with phases a lane's results were stored by the lane beside it, in the same instructions)
  if (__any(odd)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll 1
    for (int i = first_tile; i < NTL * TN; i += tile_step) {
      const int t = i / TN, o0 = nb * BN + (wn * TN + i % TN) * 16, o = o0 + (lane & 15);
      const int m0 = (my_first + t) * 16, m = m0 + 4 * (lane >> 4);
      if (t >= my_tiles || o0 >= p.Og) continue;
      bool again[4], any = false;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        again[j] = o < p.Og && m + j < block_px && !trusted_result(out[element(m + j, o)]);
        any |= again[j];
      }
      if (!__any(any)) continue;
      const floatx4 v = split_plain_tile<T, ADJ>(p, X, W, g, o0, R0, m0, block_px, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (again[j]) out[element(m + j, o)] = v[j];
    }
  }
  if (probe && threadIdx.x == 0) {
    probe[(long long)blockIdx.x * 4 + 2] = wall_clock64();
    probe[(long long)blockIdx.x * 4 + 3] = clock64();
  }
}

template <int WM, int WN, int WK, int NTL, int TN, int T, int MODE, int XI, bool ADJ>
void launch_split_one(const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s) {
  auto kernel = conv_split<WM, WN, WK, NTL, TN, T, MODE, XI, ADJ>;
  static const hipError_t lds_opt_in =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
  (void)lds_opt_in;
  hipLaunchKernelGGL(kernel, dim3(p.n_mblocks * p.n_nblocks * p.G), dim3(512), p.lds_bytes, s, p, X, W, out);
}

// The instantiation with `tiles` = N, N-1, .. 1 pixel tiles per wave
template <int WM, int WN, int WK, int TN, int T, int MODE, int N>
void launch_split_tiles(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s) {
  if (tiles == N) {
    // X items per thread: 1, 2 or 4.  2x2 windows: backward-data only
    auto go = [&](auto xi_c) {
      constexpr int XI = decltype(xi_c)::value;
      if (T == 4 || p.adjoint) launch_split_one<WM, WN, WK, N, TN, T, MODE, XI, true>(p, X, W, out, s);
      else if constexpr (T != 4) launch_split_one<WM, WN, WK, N, TN, T, MODE, XI, false>(p, X, W, out, s);
    };
    if (p.x_items > 2) go(std::integral_constant<int, 4>{});
    else if (p.x_items > 1) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 1>{});
  } else if constexpr (N > 1) {
    launch_split_tiles<WM, WN, WK, TN, T, MODE, N - 1>(tiles, p, X, W, out, s);
  }
}

}  // namespace

// Launchers of the instantiations, one translation unit per tile configuration and window; `tiles`: pixel tiles per wave.
void launch_split_0_9(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_1_9(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_2_9(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_0_4(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_1_4(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_2_4(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_0_3(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_1_3(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);
void launch_split_3_1(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s);

}  // namespace syno
