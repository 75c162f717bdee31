// bf16 convolutions in chunks of channels (conv_flow_bf16.h): which passes the kernel takes, tile choice and launch.
#include "conv_flow_bf16.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>

#include "plan.h"

namespace syno {
namespace {

constexpr int kCUs = 256;

struct FlowRecord : FlowParams { int32_t config, tiles, x_items, adjoint; };

// Record of contraction `which` for a tile configuration and TR output rows per block; false where the kernel does not take it.
bool fill_flow(const syno_plan* plan, int which, int cfg, int TR, FlowRecord& p) {
  const ConvLike& c = plan->conv;
  if (plan->in_dtype != SYNO_BF16 || cfg < 0 || cfg >= kNumFlowConfigs || TR < 1) return false;
  if (std::max(plan->x_elems, plan->out_elems) * 2 >= (1ll << 32)) return false;
  const FlowConfig& v = kFlowConfigs[cfg];
  const bool fwd = which == SYNO_FWD;
  const int T = c.KH * c.KW, BN = v.WN * v.TN * 16, KC = v.oct * 8;
  if (!(T == 9 && c.KH == 3) && !(T == 4 && c.KH == 2 && !fwd)) return false;
  if (c.h_wrap || c.w_wrap) return false;
  // forward-layout weights (taps adjacent, channels T apart), whole octets of the reduced channels, four pixels to a row
  if (c.ws_kw != 1 || c.ws_kh != c.KW || c.ws_c != T) return false;
  p = FlowRecord{};
  p.G = c.G; p.n_images = c.N;
  p.Ho = c.Ho; p.Wo = c.Wo; p.Hi = c.Hi; p.Wi = c.Wi;
  p.rows_total = c.N * c.Ho;
  const int plane = c.Hi * c.Wi;
  if (fwd) {
    p.Og = c.Og; p.Cg = c.Cg; p.ph = c.ph; p.pw = c.pw; p.sh = c.sh; p.sw = c.sw;
    p.os_o = c.Ho * c.Wo;
    p.ws_o = c.ws_o; p.ws_c = c.ws_c;
  } else {
    if (c.sh != 1 || c.sw != 1 || c.Cg < 2) return false;      // (one run of taps to a row could not be read in whole dwords)
    p.Og = c.Cg; p.Cg = c.Og; p.ph = c.KH - 1 - c.ph; p.pw = c.KW - 1 - c.pw; p.sh = p.sw = 1;
    p.os_o = plane;
    p.ws_o = c.ws_c; p.ws_c = c.ws_o;
  }
  if (c.sh > c.KH || (p.Cg & 7) || p.Wi < 4 || p.ph < 0 || p.pw < 0 || p.ph >= c.KH || p.pw >= c.KW) return false;
  p.ws_g = c.ws_g;
  p.xs_c = plane; p.xs_g = p.Cg * plane; p.xs_n = c.G * p.xs_g;
  p.os_g = p.Og * p.os_o; p.os_n = c.G * p.os_g;
  p.TR = TR;
  p.n_mblocks = (p.rows_total + TR - 1) / TR;
  p.n_nblocks = (p.Og + BN - 1) / BN;
  p.n_chunks = (p.Cg + KC - 1) / KC;
  // row slots: a run of r rows of one image takes (r-1)*sh + KH; blocks start at multiples of TR, which bounds the images in one
  const int images = p.Ho % TR == 0 ? 1 : TR % p.Ho == 0 ? TR / p.Ho : (TR + p.Ho - 2) / p.Ho + 1;
  p.n_slots = TR * p.sh + (c.KH - p.sh) * images;
  p.img_slots = (p.Ho - 1) * p.sh + c.KH;
  p.vpr = (p.Wi + 3) / 4;
  p.w_bytes = T * v.oct * BN * 16;
  // 16 pixels of a fragment that go over a row's end meet no bank twice where a row's slot is 16 pixels longer than the row
  // (2 longer: two of them do, and the read takes twice as long)
  for (const int pad : {p.Wo % 16 && p.sw == 1 ? 16 : c.KW - 1, c.KW - 1}) {
    p.Wp = p.Wi + pad;
    p.octet = (p.n_slots * p.Wp + 15) & ~15;
    p.x_bytes = v.oct * p.octet * 16;
    if (2 * (p.x_bytes + p.w_bytes) <= kFlowLdsBytes) break;
  }
  const int MT = (TR * p.Wo + 15) / 16;
  p.tiles = (MT + v.WM - 1) / v.WM;
  if (p.tiles > v.max_tiles) return false;
  const int64_t per = (int64_t)p.n_slots * p.vpr;
  p.x_items = v.oct * per <= 256 ? 0 : (int)((v.oct * per + 511) / 512);      // (0: items of four channels, see the kernel)
  if (p.x_items > 2) return false;
  p.lds_bytes = 2 * (p.x_bytes + p.w_bytes);
  if (v.WK > 1) p.lds_bytes = std::max(p.lds_bytes, 8 * p.tiles * v.TN * 1024);
  if (p.lds_bytes > kFlowLdsBytes) return false;
  const int64_t tiles = (int64_t)p.n_mblocks * p.n_nblocks, most = 1ll << 32;
  if (c.G * tiles >= (1ll << 23) || (int64_t)p.rows_total * p.Ho >= most) return false;
  auto magic = [](int64_t d) { return d == 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); };
  p.m_tiles = magic(tiles); p.m_nblocks = magic(p.n_nblocks);
  p.m_ho = magic(p.Ho); p.m_wo = magic(p.Wo); p.m_pcg = magic(per); p.m_vpr = magic(p.vpr); p.m_img = magic(p.img_slots);
  p.m_edge = magic(p.n_slots);
  // the tiles of a group dealt to the XCDs as in the other contraction kernels: the split that fetches the fewest bytes
  if (tiles % 8 == 0) {
    const double src = 2.0 * c.N * p.Cg * plane, wts = 2.0 * p.Og * p.Cg * T, fits = 2.0 * 1024 * 1024;
    double fewest = 0;
    for (int a = 1; a <= 8; a *= 2) {
      const int b = 8 / a;
      if (p.n_mblocks % a || p.n_nblocks % b) continue;
      const int sm = p.n_mblocks / a, sn = p.n_nblocks / b;
      for (int rows_first = 0; rows_first < 2; ++rows_first) {
        double bytes = b * src + a * wts;
        if ((int64_t)sm * sn > 32) {
          if (!rows_first && wts / b > fits) bytes += a * wts * (sm - 1);
          if (rows_first && src / a > fits) bytes += b * src * (sn - 1);
        }
        if (p.xcd_m == 0 || bytes < fewest) {
          fewest = bytes;
          p.xcd_m = a; p.xcd_n = b; p.sm = sm; p.sn = sn;
          p.xcd_rows_first = (int64_t)sm * sn <= 32 ? wts > src : rows_first;
        }
      }
    }
    p.m_xcdn = magic(p.xcd_n); p.m_sm = magic(p.sm); p.m_sn = magic(p.sn);
  }
  p.config = cfg;
  p.adjoint = !fwd;
  p.out_bf16 = plan->out_dtype == SYNO_BF16;
  const uintptr_t probe = reinterpret_cast<uintptr_t>(plan->opt.clock_probe);
  p.probe_lo = (int32_t)(uint32_t)probe;
  p.probe_hi = (int32_t)(uint32_t)(probe >> 32);
  return true;
}

// Estimated duration in microseconds: least squares over 23000 passes of 8 to 512 channels (standard deviation 9 %).  A round of
// workgroups costs its ends and per chunk: the busiest SIMD's products, LDS reads, load instructions, and the stores.
double flow_cost(const FlowRecord& p, const ConvLike& c) {
  const FlowConfig& v = kFlowConfigs[p.config];
  const int T = c.KH * c.KW, BN = v.WN * v.TN * 16, steps = v.oct / 4 * T;
  const int MT = (std::min(p.TR, p.rows_total) * p.Wo + 15) / 16, base = MT / v.WM, extra = MT % v.WM;
  double simd[4] = {0, 0, 0, 0}, reads = 0;
  for (int w = 0; w < 8; ++w) {
    const int wk = v.WK == 1 ? 0 : w & 3, wn = v.WN == 1 ? 0 : w >> 2;
    const int wm = v.WM == 8 ? w : v.WM == 4 ? (w + 2 * wn) & 3 : w >> 2;
    const int mine = (steps - wk + v.WK - 1) / v.WK, tiles = base + (wm < extra ? 1 : 0);
    simd[w & 3] += 16.0 * mine * tiles * v.TN;
    reads += mine * (p.tiles + v.TN);
  }
  struct Weights { double call, round, chunk, product, read, x, w, stored, moved; };
  constexpr Weights of[kNumFlowConfigs] = {{3.0, 0.63, 0.065, 3.24e-4, 1.42e-3, 0.0695, 0.056, 0.312, 0.0034},
                                           {2.1, 1.89, 0, 1.15e-4, 2.82e-3, 0.0503, 0.12, 0.245, 0.0099},
                                           {2.0, 2.49, 0, 2.12e-4, 3.15e-3, 0.0813, 0.108, 0.4, 0.0039}};
  const Weights& q = of[p.config];
  const double blocks = (double)p.n_mblocks * p.n_nblocks * p.G, rounds = std::ceil(blocks / kCUs);
  const double x_loads = p.x_items ? 8 * p.x_items : 4, w_items = BN * v.oct * 8 / 1024.0;
  const double chunk = q.chunk + q.product * *std::max_element(simd, simd + 4) + q.read * reads + q.x * x_loads + q.w * w_items;
  const double bytes = v.oct * 16.0 * p.n_slots * p.Wi + 2.0 * BN * v.oct * 8 * T, stored = 4.0 * p.n_images * p.os_n;
  return q.call + rounds * (q.round + p.n_chunks * chunk) + q.stored * 1e-6 * stored + q.moved * 1e-6 * p.n_chunks * blocks * bytes;
}

}  // namespace

// Fills launch[which] with the tiles of the lowest estimate; false where the kernel does not take the pass.  `named`: the one configuration
// asked for, or -1; `rows`: the rows per block asked for, or 0.  On 30000 passes drawn (8 to 512
// channels, 1 to 128 images of 5 to 64 pixels, strides 1 and 2) it takes 1 / 1.47 (forward), 1 / 1.79 (backward-data) and 1 / 1.45 (stride 2)
// of the other kernels' time in the mean.  `*sure`: not one of the forward passes in several rounds of workgroups that wider or
// narrower panels of output channels, or a single chunk, may suit better (0.72 to 1.7 times as fast).
bool flow_configure(syno_plan* plan, int which, int named, int rows, bool* sure) {
  const ConvLike& c = plan->conv;
  FlowRecord best{}, p;
  double least = 1e300;
  for (int cfg = 0; cfg < kNumFlowConfigs; ++cfg)
    for (int TR = 1; TR <= c.N * c.Ho && TR * c.Wo <= 16 * 32; ++TR) {
      if ((named >= 0 && cfg != named) || (rows > 0 && TR != rows)) continue;
      if (!fill_flow(plan, which, cfg, TR, p)) continue;
      const double cost = flow_cost(p, c);
      if (cost < least) { least = cost; best = p; }
    }
  if (least >= 1e300) return false;
  const bool one_round = (int64_t)best.n_mblocks * best.n_nblocks * best.G <= kCUs, strided = best.sh > 1 || best.sw > 1;
  *sure = named >= 0 || best.adjoint || one_round ||
          !(best.Cg <= 32 || (best.Og > 32 && best.Og <= 48) || (best.Cg <= 64 && best.Og > 128) || (strided && best.Og <= 32));
  Launch& L = plan->launch[which];
  static_assert(sizeof(FlowRecord) <= sizeof(L.params), "parameter record does not fit");
  memcpy(L.params, &best, sizeof best);
  L.params_ready = true;
  L.variant = -2 - best.config;
  L.workspace = 0;
  L.cycles = least * 2400;
  L.roundings = (double)best.Cg * c.KH * c.KW / 32;
  return true;
}

bool flow_store_phases(syno_plan* plan) {
  FlowRecord p;
  memcpy(&p, plan->launch[SYNO_BWD_DATA].params, sizeof p);
  p.phases = 1;
  memcpy(plan->launch[SYNO_BWD_DATA].params, &p, sizeof p);
  return true;
}

std::string flow_describe(const syno_plan* plan, int which) {
  FlowRecord p;
  memcpy(&p, plan->launch[which].params, sizeof p);
  const FlowConfig& v = kFlowConfigs[p.config];
  char b[256];
  snprintf(b, sizeof b, "in-chunks tiles=%d rows/block=%d BN=%d KC=%d weights=direct waves=%dx%dx%d grid=%d lds=%dB slots=%d", p.config, p.TR, v.WN * v.TN * 16,
           v.oct * 8, v.WM, v.WN, v.WK, p.n_mblocks * p.n_nblocks * p.G, p.lds_bytes, p.n_slots);
  std::string d = b;
  if (p.xcd_m > 0) d += " tiles-per-xcd=" + std::to_string(p.sm) + "x" + std::to_string(p.sn) + (p.xcd_rows_first ? "(rows first)" : "");
  return d;
}

syno_status launch_flow(const syno_plan* plan, int which, const void* A, const void* B, void* out, hipStream_t stream) {
  FlowRecord p;
  memcpy(&p, plan->launch[which].params, sizeof p);
  const uint16_t *X = static_cast<const uint16_t*>(A), *W = static_cast<const uint16_t*>(B);
  (p.config == 0 ? launch_flow_0 : p.config == 1 ? launch_flow_1 : launch_flow_2)(plan->conv.KH * plan->conv.KW, p.tiles, p.x_items, p.adjoint, p, X, W, out, stream);
  return hipGetLastError() == hipSuccess ? SYNO_OK : SYNO_ERR_HIP;
}

}  // namespace syno
