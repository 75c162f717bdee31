// bf16 convolutions whose reduction takes several chunks of channels, forward and backward-data, device side: parameter record,
// kernel template, tile configurations and launch helper.
//   out[n, g*Og+o, h, w] = sum_{c,kh,kw} X[n, g*Cg+c, sh*h+kh-ph, sw*w+kw-pw] * W[g,o,c,kh,kw]      (zero outside the image)
// Backward-data is the same on the adjoint record (channel roles exchanged, taps reversed).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace syno {

struct FlowParams {
  int32_t Og, Cg, Ho, Wo, Hi, Wi, ph, pw, sh, sw, n_images;
  int32_t rows_total;                 // n_images * Ho
  int32_t xs_n, xs_c, xs_g;           // source strides: image, channel, group
  int32_t os_n, os_o, os_g;           // result strides
  int32_t ws_g, ws_o, ws_c;           // weight strides: group, this pass's output channel, its reduced channel; taps are adjacent
  // tiling
  int32_t TR, n_mblocks, n_nblocks, n_chunks, n_slots, Wp, vpr, octet;     // octet: pixels between channel octets in LDS
  int32_t img_slots;                  // row slots of a whole image
  int32_t x_bytes, w_bytes, lds_bytes, G;
  int32_t xcd_m, xcd_n, sm, sn, xcd_rows_first;      // as in conv_mfma; sm x sn tiles to an XCD
  int32_t out_bf16;
  int32_t phases;                     // 2x2 windows: the result is an image in the place of its phase planes, as in conv_split
  // ceil(2^32 / d), 0 for d = 1
  uint32_t m_tiles, m_nblocks, m_xcdn, m_sm, m_sn, m_ho, m_wo, m_pcg, m_vpr, m_img, m_edge;
  int32_t probe_lo, probe_hi;
};

// waves over pixels, output channels and k-steps; output tiles of 16 channels per wave; channel octets per chunk; most pixel tiles
// of 16 per wave
struct FlowConfig { int WM, WN, WK, TN, oct, max_tiles; };
constexpr int kNumFlowConfigs = 3;
constexpr FlowConfig kFlowConfigs[kNumFlowConfigs] = {{8, 1, 1, 2, 4, 4}, {4, 2, 1, 2, 4, 4}, {2, 1, 4, 2, 8, 4}};

namespace {

typedef float flow_f4 __attribute__((ext_vector_type(4)));
typedef float flow_f4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 flow_bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t flow_u2_any __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t flow_u4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t flow_u1_any __attribute__((aligned(2)));
#define SYNO_GLOBAL __attribute__((address_space(1)))
typedef const SYNO_GLOBAL char* flow_ptr;      // (keeps its address space through the empty asm statements below)

// n / d through m = ceil(2^32 / d), 0 for d = 1 (no branch)
__device__ __forceinline__ int flow_div(int n, uint32_t m) { return (int)__umulhi((uint32_t)n, m) + (n & (m ? 0 : -1)); }

// The same for any n below 2^31 (the estimate is at most one too large): a launch may have millions of blocks
__device__ __forceinline__ int flow_div_large(int n, int d, uint32_t m) {
  const int q = flow_div(n, m);
  return q - ((uint32_t)n < (uint32_t)q * (uint32_t)d ? 1 : 0);
}

template <int I, int N, class F>
__device__ __forceinline__ void flow_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    flow_for<I + 1, N>(f);
  }
}

__device__ __forceinline__ uint32_t flow_round_pair(float lo, float hi) {      // to nearest even
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  const f2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
}

// A workgroup (8 waves, one to a compute unit) owns TR whole result rows x BN output channels and walks the reduction in chunks of
// 8 * OCT channels.  X lies in LDS as [channel octet][row slot][pixel] 16-byte pieces, a row's slot with the window's zero columns
// around it, octets a multiple of 256 bytes apart; W as [tap][channel octet][output channel] pieces: fragments are single
// 16-byte reads free of bank conflicts, and taps constant offsets.
//  - What the chunked kernels before lost (cycles of a call of 39000 at 32x128x128 28x28, of which the products 7200): 5800 until
//    the first load was out, 1900 of every chunk for loads that touched 64 lines each (a lane took 8 channels x 9 taps, the
//    next lane the next output channel), 2400 for staging between two barriers, 2300 for adding up the waves that split a chunk.
//  - So: the first loads go out right after the block's place is known; a weight item is 2 channels x T taps, adjacent lanes
//    adjacent in memory (backward-data: T taps of one output channel in two rows), which pairs up into one dword per tap;
//    two LDS buffers, the next chunk staged out of registers between the k-steps of the present one while the loads of
//    the one after that and the next travel: one barrier per chunk and two chunks of time for a memory round trip.
//  - A row of taps (of one wave's share of a chunk) is summed by itself and joins the accumulators once: fewer roundings at
//    their magnitude than one per k-step.
// T taps, KW of them along a row.  ADJ: the weights of backward-data, read from the forward layout.  NTL: most pixel tiles per wave;
// a wave has that many or one less.  XI: X items (4 pixels x XC channels) per thread; four channels where a chunk's items are at most
// half the threads (half the load instructions, of which a compute unit takes one in 16 to 23 cycles).
template <int T, int KW, int WM, int WN, int WK, int NTL, int TN, int OCT, int XI, int XC, bool ADJ>
__global__ __launch_bounds__(512) void conv_flow_bf16(const FlowParams p, const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                                                      void* __restrict__ out) {
  static_assert(WM * WN * WK == 8, "eight waves");
  constexpr int KH = T / KW, BN = WN * TN * 16, KC = OCT * 8, STEPS = OCT / 4 * T;
  constexpr int WITEMS = BN * KC / 2, WI = (WITEMS + 511) / 512;
  constexpr int WD = ADJ ? (T + 1) / 2 : T;           // dwords of a weight item's row (ADJ: two rows)
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* const wl = smem + 2 * p.x_bytes;

  SYNO_GLOBAL long long* const probe = (SYNO_GLOBAL long long*)(((unsigned long long)(uint32_t)p.probe_hi << 32) | (uint32_t)p.probe_lo);
  if (probe && threadIdx.x == 0) {
    probe[(long long)blockIdx.x * 4 + 0] = wall_clock64();
    probe[(long long)blockIdx.x * 4 + 1] = clock64();
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // waves w and w + 4 share a SIMD: the second four take their pixel tiles in another order
  const int wk = WK == 1 ? 0 : wave & 3, wn = WN == 1 ? 0 : wave >> 2;
  const int wm = WM == 8 ? wave : WM == 4 ? (wave + 2 * wn) & 3 : wave >> 2;

  // ---- this block's tile
  const int tiles = p.n_mblocks * p.n_nblocks, g = flow_div_large(blockIdx.x, tiles, p.m_tiles), local = blockIdx.x - g * tiles;
  int mb, nb;
  if (p.xcd_m > 0) {
    const int xcd = local & 7, idx = local >> 3;
    const int xm = flow_div(xcd, p.m_xcdn), xn = xcd - xm * p.xcd_n;
    int im, in;
    if (p.xcd_rows_first) { in = flow_div_large(idx, p.sm, p.m_sm); im = idx - in * p.sm; }
    else { im = flow_div_large(idx, p.sn, p.m_sn); in = idx - im * p.sn; }
    mb = xm * p.sm + im;
    nb = xn * p.sn + in;
  } else {
    mb = flow_div_large(local, p.n_nblocks, p.m_nblocks);
    nb = local - mb * p.n_nblocks;
  }
  const int R0 = mb * p.TR, rows = min(p.TR, p.rows_total - R0);
  const int n0 = flow_div(R0, p.m_ho), h0 = R0 - n0 * p.Ho;

  // ---- what this thread stages: XI items of 4 adjacent pixels x XC channels (a row's last one is moved left to end with the row)
  const flow_ptr xbase = (flow_ptr)(X + (int64_t)g * p.xs_g);
  const int first_slots = (min(rows, p.Ho - h0) - 1) * p.sh + KH;     // of the first image; the others begin with their first row
  uint32_t x_off[XI];
  int x_dst[XI], x_oc[XI];
  bool x_live[XI];
#pragma unroll
  for (int k = 0; k < XI; ++k) {
    const int idx = XC == 8 ? tid + k * 512 : tid >> 1, per = p.n_slots * p.vpr, half = XC == 8 ? 0 : tid & 1;
    const int oc = flow_div(idx, p.m_pcg), rem = idx - oc * per, s = flow_div(rem, p.m_vpr);
    const int x = min((rem - s * p.vpr) * 4, p.Wi - 4);
    const int past = s - first_slots, j = flow_div(max(past, 0), p.m_img);
    const int n = past < 0 ? n0 : n0 + 1 + j;
    const int r = past < 0 ? h0 * p.sh + s - p.ph : past - j * p.img_slots - p.ph;
    x_oc[k] = oc * 8 + half * 4;
    x_live[k] = oc < OCT && (unsigned)r < (unsigned)p.Hi && n < p.n_images;
    x_off[k] = x_live[k] ? (uint32_t)(n * p.xs_n + r * p.Wi + x) * 2u : 0u;
    x_dst[k] = oc < OCT ? (oc * p.octet + s * p.Wp + x + p.pw) * 16 + half * 8 : -1;
  }
  // ---- and WI weight items: two reduced channels x T taps of one output channel
  const flow_ptr wbase = (flow_ptr)(W + (int64_t)g * p.ws_g);
  uint32_t w_off[WI];
  int w_dst[WI], w_c[WI];
  bool w_odd[WI];
#pragma unroll
  for (int k = 0; k < WI; ++k) {
    const int idx = tid + k * 512, rest = idx >> 6;
    const int pair = ADJ ? (idx >> 4) & 3 : idx & 3, lo = ADJ ? idx & 15 : (idx >> 2) & 15;
    const int oc = rest & (OCT - 1), o = (rest / OCT) * 16 + lo;
    const bool mine = WITEMS % 512 == 0 || idx < WITEMS;
    w_c[k] = oc * 8 + pair * 2;
    // (an output channel beyond the last is computed from the last one's weights and not stored)
    const int row = min(nb * BN + o, p.Og - 1);
    // (ADJ: a run of an odd number of taps is read in whole dwords at even elements, from the element before it where it begins at an odd one
    // - 16-byte loads at odd elements take seven times as long - or where it is the last of its row, which nothing may follow)
    w_odd[k] = ADJ && (T & 1) && ((row & 1) || row == p.Og - 1);
    w_off[k] = ((uint32_t)row * (uint32_t)p.ws_o - (w_odd[k] ? 1u : 0u)) * 2u;
    w_dst[k] = mine ? (oc * BN + o) * 16 + pair * 4 : -1;
  }

  struct Items { uint32_t x[XI][2 * XC], w[WI][ADJ ? 2 * WD : WD]; };
  // Loads are unconditional (what has no source reads some valid element and is zeroed when staged), chunks past the last one
  // read it again
  const uint32_t xc = (uint32_t)p.xs_c * 2u, wc = (uint32_t)p.ws_c * 2u;
  auto fetch_piece = [&](Items& v, int ch, auto piece_c) {        // two loads of an X item, or a part of a weight item
    constexpr int piece = decltype(piece_c)::value;
    const int c0 = min(ch, p.n_chunks - 1) * KC;
    if constexpr (piece < XC / 2 * XI) {
      constexpr int k = piece / (XC / 2), j0 = piece % (XC / 2) * 2;
      const uint32_t at = x_off[k] + (uint32_t)min(c0 + x_oc[k], p.Cg - XC) * xc;
      flow_ptr row = xbase + (uint64_t)j0 * xc;
#pragma unroll
      for (int j = j0; j < j0 + 2; ++j) {
        asm volatile("" : "+s"(row));      // (a uniform base and a 32-bit lane offset, not eight 64-bit lane addresses)
        const flow_u2_any d = *(const SYNO_GLOBAL flow_u2_any*)(row + at);
        row += xc;
        v.x[k][2 * j] = d[0];
        v.x[k][2 * j + 1] = d[1];
      }
    } else {
      // dwords q0 .. q1 of row `row`
      constexpr int k = (piece - XC / 2 * XI) / 2, half = (piece - XC / 2 * XI) & 1, row = ADJ ? half : 0, N = WD, split = N / 8 * 4;
      constexpr int q0 = ADJ ? 0 : half ? split : 0, q1 = ADJ ? N : half ? N : split;
      const uint32_t at = w_off[k] + (uint32_t)min(c0 + w_c[k], p.Cg - 2) * wc;
      flow_ptr base = wbase + (uint64_t)row * wc;
      asm volatile("" : "+s"(base));
      const flow_ptr src = base + at;
      constexpr int whole = q0 + (q1 - q0) / 4 * 4, pairs = whole + (q1 - whole) / 2 * 2;
      flow_for<0, (q1 - q0) / 4>([&](auto q_c) {
        constexpr int q = q0 + decltype(q_c)::value * 4;
        const flow_u4_any d = *(const SYNO_GLOBAL flow_u4_any*)(src + 4 * q);
        v.w[k][row * WD + q] = d[0]; v.w[k][row * WD + q + 1] = d[1]; v.w[k][row * WD + q + 2] = d[2]; v.w[k][row * WD + q + 3] = d[3];
      });
      if constexpr (pairs > whole) {
        const flow_u2_any d = *(const SYNO_GLOBAL flow_u2_any*)(src + 4 * whole);
        v.w[k][row * WD + whole] = d[0]; v.w[k][row * WD + whole + 1] = d[1];
      }
      flow_for<pairs, q1>([&](auto e_c) {
        constexpr int e = decltype(e_c)::value;
        v.w[k][row * WD + e] = *(const SYNO_GLOBAL flow_u1_any*)(src + 4 * e);
      });
    }
  };
  constexpr int FETCH = XC / 2 * XI + 2 * WI, STAGE = XI + WI;
  auto fetch = [&](Items& v, int ch) { flow_for<0, FETCH>([&](auto i) { fetch_piece(v, ch, i); }); };
  auto stage_x = [&](const Items& v, int ch, int buf, auto k_c) {
    constexpr int k = decltype(k_c)::value;
    {
      const bool live = x_live[k] && ch * KC + x_oc[k] < p.Cg;
      if (x_dst[k] >= 0) {
        unsigned char* const dst = smem + buf * p.x_bytes + x_dst[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;      // high or low halves of (second, first)
          uint32_t d[XC / 2];
#pragma unroll
          for (int h = 0; h < XC / 2; ++h) d[h] = __builtin_amdgcn_perm(v.x[k][4 * h + 2 + (i >> 1)], v.x[k][4 * h + (i >> 1)], live ? sel : 0x0c0c0c0cu);
          if constexpr (XC == 8) *reinterpret_cast<uint4*>(dst + i * 16) = make_uint4(d[0], d[1], d[2], d[3]);
          else *reinterpret_cast<uint2*>(dst + i * 16) = make_uint2(d[0], d[1]);
        }
      }
    }
  };
  auto stage_w = [&](const Items& v, int ch, int buf, auto k_c) {
    constexpr int k = decltype(k_c)::value;
    {
      const bool live = ch * KC + w_c[k] < p.Cg;
      if (WITEMS % 512 == 0 || w_dst[k] >= 0) {
        unsigned char* const dst = wl + buf * p.w_bytes + w_dst[k];
        uint32_t w[ADJ ? 2 * WD : WD];
#pragma unroll
        for (int i = 0; i < (ADJ ? 2 * WD : WD); ++i)
          w[i] = !ADJ || T % 2 == 0 ? v.w[k][i] : i % WD == WD - 1 ? v.w[k][i] >> (w_odd[k] ? 16 : 0) : __builtin_amdgcn_alignbit(v.w[k][i + 1 < 2 * WD ? i + 1 : i], v.w[k][i], w_odd[k] ? 16 : 0);
        flow_for<0, T>([&](auto t_c) {
          constexpr int t = decltype(t_c)::value;
          // channel 0's and channel 1's tap t: halves of these dwords
          constexpr int e0 = t, e1 = ADJ ? t : T + t;
          const uint32_t a = w[e0 >> 1], b = w[(ADJ ? WD : 0) + (e1 >> 1)];
          constexpr uint32_t sel = ((e0 & 1) ? 0x0302u : 0x0100u) | ((e1 & 1) ? 0x07060000u : 0x05040000u);
          *reinterpret_cast<uint32_t*>(dst + (ADJ ? T - 1 - t : t) * OCT * BN * 16) = __builtin_amdgcn_perm(b, a, live ? sel : 0x0c0c0c0cu);
        });
      }
    }
  };
  auto stage_piece = [&](const Items& v, int ch, int buf, auto piece_c) {
    constexpr int piece = decltype(piece_c)::value;
    if constexpr (piece < XI) stage_x(v, ch, buf, piece_c);
    else stage_w(v, ch, buf, std::integral_constant<int, piece - XI>{});
  };

  Items va, vb;
  fetch(va, 0);
  // ---- while it travels: the zero columns on either side of the rows (both buffers; never written again)
  if constexpr (KW > 1)
    for (int i = tid; i < OCT * p.n_slots; i += 512) {
      const int oc = flow_div(i, p.m_edge), s = i - oc * p.n_slots;
      unsigned char* const row = smem + (oc * p.octet + s * p.Wp) * 16;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int e = 0; e < KW - 1; ++e) *reinterpret_cast<uint4*>(row + b * p.x_bytes + (e < p.pw ? e : p.Wi + e) * 16) = make_uint4(0, 0, 0, 0);
      }
    }
  // ---- per-lane operand bases
  const int block_px = rows * p.Wo, MT = (block_px + 15) >> 4;
  const int base = MT / WM, extra = MT - base * WM;
  const int my_tiles = base + (wm < extra ? 1 : 0), my_first = wm * base + min(wm, extra);
  int a_base[NTL];
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    const int m = min((my_first + t) * 16 + (lane & 15), block_px - 1);
    const int i = flow_div(m, p.m_wo), w = m - i * p.Wo;
    const int slot = i * p.sh + (KH - p.sh) * flow_div(h0 + i, p.m_ho);      // (every image before this one adds KH - sh)
    a_base[t] = (slot * p.Wp + w * p.sw + (lane >> 4) * p.octet) * 16;
  }
  const int b_base = 2 * p.x_bytes + ((lane >> 4) * BN + wn * TN * 16 + (lane & 15)) * 16;

  fetch(vb, 1);

  flow_f4 acc[NTL][TN];
#pragma unroll
  for (int t = 0; t < NTL; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u) acc[t][u] = flow_f4{0.f, 0.f, 0.f, 0.f};

  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  const int row_pitch = p.Wp * 16;
  struct Frags { flow_bf8 a[NTL], b[TN]; };
  auto read = [&](Frags& f, int x_at, int w_at) {
#pragma unroll
    for (int u = 0; u < TN; ++u) f.b[u] = *reinterpret_cast<const flow_bf8*>(smem + b_base + w_at + u * 256);
#pragma unroll
    for (int t = 0; t < NTL; ++t) f.a[t] = *reinterpret_cast<const flow_bf8*>(smem + a_base[t] + x_at);
  };
  flow_f4 sum[NTL][TN];
#pragma unroll
  for (int u = 0; u < TN; ++u) sum[NTL - 1][u] = flow_f4{0.f, 0.f, 0.f, 0.f};
  const bool full = my_tiles == NTL;
  auto products = [&](const Frags& f, auto first_c, auto last_c) {        // all tiles but the last, or that one
    constexpr bool last = decltype(last_c)::value;
#pragma unroll
    for (int t = last ? NTL - 1 : 0; t < (last ? NTL : NTL - 1); ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u)
        sum[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[t], f.b[u], decltype(first_c)::value ? flow_f4{0.f, 0.f, 0.f, 0.f} : sum[t][u], 0, 0, 0);
  };
  auto join = [&]() {
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) {
        acc[t][u] += sum[t][u];
        asm volatile("" : "+v"(acc[t][u]));        // (here, and not where the next chunk's sums are added: registers)
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // a k-step's products with the next one's reads between them
  auto kstep = [&](const Frags& f, auto first_c, auto reads_c) {
    products(f, first_c, no);
    if constexpr (decltype(reads_c)::value) {
      constexpr int NM = (NTL - 1) * TN;
#pragma unroll
      for (int i = 0; i < NTL + TN; ++i) {
        if (i < NM) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      if constexpr (NM > NTL + TN) __builtin_amdgcn_sched_group_barrier(0x008, NM - NTL - TN, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (full) products(f, first_c, yes);
  };
  // the k-steps of a chunk, with P pieces of other work dealt out among them
  auto multiply = [&](int buf, auto pieces_c, auto&& piece) {
    constexpr int P = decltype(pieces_c)::value;
    int xb = buf * p.x_bytes, wb = buf * p.w_bytes;
    asm volatile("" : "+s"(xb), "+s"(wb));         // (addresses are formed where they are used, not kept in registers)
    Frags f[2];
    if constexpr (WK == 1) {
      read(f[0], xb, wb);
      flow_for<0, STEPS>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value, next = s + 1, tap = next % T, cg = next / T, kh = tap / KW, kw = tap - kh * KW;
        constexpr bool more = next < STEPS;
        if constexpr (more) read(f[next & 1], xb + cg * 4 * p.octet * 16 + kh * row_pitch + kw * 16, wb + (tap * OCT + cg * 4) * BN * 16);
        kstep(f[s & 1], std::integral_constant<bool, s % KW == 0>{}, std::integral_constant<bool, more>{});
        if constexpr (s % KW == KW - 1) join();
        flow_for<s * P / STEPS, (s + 1) * P / STEPS>(piece);
      });
    } else {
      // this wave's steps: wk, wk + WK, ... (at least one: the host sees to it)
      auto at = [&](int s, int& x_at, int& w_at) {
        const int cg = s / T, tap = s - cg * T, kh = tap / KW, kw = tap - kh * KW;
        x_at = xb + cg * 4 * p.octet * 16 + kh * row_pitch + kw * 16;
        w_at = wb + (tap * OCT + cg * 4) * BN * 16;
      };
      int x_at, w_at;
      at(wk, x_at, w_at);
      read(f[0], x_at, w_at);
      constexpr int MOST = (STEPS + WK - 1) / WK;
      flow_for<0, MOST>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        const int s = wk + i * WK;
        if constexpr (i + 1 < MOST) {
          at(min(s + WK, STEPS - 1), x_at, w_at);
          read(f[(i + 1) & 1], x_at, w_at);
        }
        if ((i + 1) * WK <= STEPS || s < STEPS) kstep(f[i & 1], std::integral_constant<bool, i == 0>{}, std::integral_constant<bool, (i + 1 < MOST)>{});
        flow_for<i * P / MOST, (i + 1) * P / MOST>(piece);
      });
      join();
    }
  };

  // ---- the chunks: `mine` held this one and is filled with the one after next, `next` holds the next one and is staged
  // (loads are not within branches: where a path might not have issued them the compiler waits for all of them)
  constexpr std::integral_constant<int, 0> b0{};
  constexpr std::integral_constant<int, 1> b1{};
  auto chunk = [&](int ch, auto buf_c, Items& mine, Items& next, bool more, auto fetch_c, auto stage_c) {
    constexpr int buf = decltype(buf_c)::value, F = decltype(fetch_c)::value ? FETCH : 0, S = decltype(stage_c)::value ? STAGE : 0;
    __syncthreads();
    multiply(buf, std::integral_constant<int, F + S>{}, [&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      if constexpr (i < F) fetch_piece(mine, ch + 2, i_c);
      else if (more) stage_piece(next, ch + 1, 1 - buf, std::integral_constant<int, i - F>{});
    });
  };
  flow_for<0, STAGE>([&](auto i) { stage_piece(va, 0, 0, i); });
  int ch = 0;
  for (; ch + 3 < p.n_chunks; ch += 2) {
    chunk(ch, b0, va, vb, true, yes, yes);
    chunk(ch + 1, b1, vb, va, true, yes, yes);
  }
  const int left = p.n_chunks - ch;            // 1 to 3 (where it is less than 3 the loads are for nothing)
  chunk(ch, b0, va, vb, left > 1, yes, yes);
  if (left > 1) {
    chunk(ch + 1, b1, vb, va, left > 2, no, yes);
    if (left > 2) chunk(ch + 2, b0, va, vb, false, no, no);
  }

  // ---- store: lane holds 4 consecutive pixels (rows of D) of one channel (column of D)
  const int img_px = p.Ho * p.Wo;
  auto store = [&](int t, int u, flow_f4 v) {
    const int m0 = (my_first + t) * 16 + 4 * (lane >> 4), o = nb * BN + (wn * TN + u) * 16 + (lane & 15);
    if (o >= p.Og || m0 >= block_px || t >= my_tiles) return;
    auto element = [&](int m, int& px) -> int64_t {       // pixel m of the block -> element of the result
      const int i = flow_div(m, p.m_wo), n = flow_div(h0 + i, p.m_ho);
      px = (h0 + i - n * p.Ho) * p.Wo + (m - i * p.Wo);
      if constexpr (T == 4)
        if (p.phases) return (int64_t)(n0 + n) * p.os_n + (int64_t)(o >> 2) * (4 * p.os_o) + (2 * (h0 + i - n * p.Ho) + (o >> 1 & 1)) * (2 * p.Wo) + 2 * (m - i * p.Wo) + (o & 1);
      return (int64_t)(n0 + n) * p.os_n + (int64_t)g * p.os_g + (int64_t)o * p.os_o + px;
    };
    int px;
    int64_t off = element(m0, px);
    bool four = m0 + 3 < block_px && px + 3 < img_px;
    if constexpr (T == 4)
      if (p.phases) {
        // four pixels of a row of one phase: the lane beside this one has the same of the phase between them, and each of the two
        // stores four adjacent pixels of the image
        four = (p.Wo & 3) == 0;
        const bool b = o & 1;
        const float take0 = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, b ? v[0] : v[2]), 0xb1, 0xf, 0xf, true));
        const float take1 = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, b ? v[1] : v[3]), 0xb1, 0xf, 0xf, true));
        if (four) {
          v = b ? flow_f4{take0, v[2], take1, v[3]} : flow_f4{v[0], take0, v[1], take1};
          off += b ? 3 : 0;            // (from the odd phase's first pixel to the pair after next)
        }
      }
    if (four) {
      if (p.out_bf16) {
        flow_u2_any d;
        d[0] = flow_round_pair(v[0], v[1]); d[1] = flow_round_pair(v[2], v[3]);
        *reinterpret_cast<flow_u2_any*>(reinterpret_cast<uint16_t*>(out) + off) = d;
      } else {
        *reinterpret_cast<flow_f4_any*>(reinterpret_cast<float*>(out) + off) = v;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (m0 + j < block_px) {
          const int64_t at = element(m0 + j, px);
          if (p.out_bf16) reinterpret_cast<uint16_t*>(out)[at] = (uint16_t)flow_round_pair(v[j], v[j]);
          else reinterpret_cast<float*>(out)[at] = v[j];
        }
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) store(t, u, acc[t][u]);
  } else {
    // the waves that split the k-steps meet in LDS: [wave][tile][lane]; every one then adds up and stores a share of the tiles
    flow_f4* const red = reinterpret_cast<flow_f4*>(smem);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) red[(((wk * WM + wm) * NTL + t) * TN + u) * 64 + lane] = acc[t][u];
    __syncthreads();
    for (int i = wk; i < NTL * TN; i += WK) {
      flow_f4 v = red[(wm * NTL * TN + i) * 64 + lane];
#pragma unroll
      for (int k = 1; k < WK; ++k) v += red[((k * WM + wm) * NTL * TN + i) * 64 + lane];
      store(i / TN, i % TN, v);
    }
  }
  if (probe && threadIdx.x == 0) {
    probe[(long long)blockIdx.x * 4 + 2] = wall_clock64();
    probe[(long long)blockIdx.x * 4 + 3] = clock64();
  }
}

constexpr int kFlowLdsBytes = 160 * 1024;

template <int T, int KW, int CFG, int NTL, int XI, int XC, bool ADJ>
void launch_flow_one(const FlowParams& p, const uint16_t* X, const uint16_t* W, void* out, hipStream_t s) {
  constexpr FlowConfig v = kFlowConfigs[CFG];
  auto kernel = conv_flow_bf16<T, KW, v.WM, v.WN, v.WK, NTL, v.TN, v.oct, XI, XC, ADJ>;
  static const hipError_t lds_opt_in =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kFlowLdsBytes);
  (void)lds_opt_in;
  hipLaunchKernelGGL(kernel, dim3(p.n_mblocks * p.n_nblocks * p.G), dim3(512), p.lds_bytes, s, p, X, W, out);
}

// The instantiation with `tiles` = N, N-1, .. 1 pixel tiles per wave and 1 or 2 X items per thread (0: items of half the channels)
template <int T, int KW, int CFG, bool ADJ, int N>
void launch_flow_tiles(int tiles, int x_items, const FlowParams& p, const uint16_t* X, const uint16_t* W, void* out, hipStream_t s) {
  if (tiles == N) {
    if (x_items == 0) launch_flow_one<T, KW, CFG, N, 1, 4, ADJ>(p, X, W, out, s);
    else if (x_items == 1) launch_flow_one<T, KW, CFG, N, 1, 8, ADJ>(p, X, W, out, s);
    else launch_flow_one<T, KW, CFG, N, 2, 8, ADJ>(p, X, W, out, s);
  } else if constexpr (N > 1) {
    launch_flow_tiles<T, KW, CFG, ADJ, N - 1>(tiles, x_items, p, X, W, out, s);
  }
}

}  // namespace

// Launchers of the instantiations, one translation unit per tile configuration
#define SYNO_FLOW_LAUNCHER(CFG) void launch_flow_##CFG(int taps, int tiles, int x_items, bool adjoint, const FlowParams& p, const uint16_t* X, const uint16_t* W, void* out, hipStream_t s)
SYNO_FLOW_LAUNCHER(0);
SYNO_FLOW_LAUNCHER(1);
SYNO_FLOW_LAUNCHER(2);

}  // namespace syno
