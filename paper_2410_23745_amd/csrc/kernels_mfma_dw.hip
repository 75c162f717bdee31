// MFMA backward-weight contraction for convolution-like operators (bf16 or fp32 inputs, fp32 result):
//   dW[g,o,c,kh,kw] = sum_{n,h,w} G[n, g*Og+o, h, w] * X[n, g*Cg+c, row(h,g)+kh-ph, w+kw-pw]
// Kernels in this file:
//   dw_stream_bf16              bf16 (dw_stream_bf16.h)
//   dw_rows_bf16                bf16, windows of three rows on rows of 14 pixels, many channels and images (dw_rows_bf16.h)
//   dw_split                    fp32 on the bf16 matrix cores (dw_split.h)
//   dw_mfma_f32                 any supported window; the source rows of a chunk come from a table in LDS
//   dw_rows_f32                 windows with a row extent (KH = 3): eight waves in two halves that alternate between
//                               multiplying one LDS buffer and staging the next chunk into the other
//   dw_reduce_slots, _tiles     fixed-order sum of the split partials into dW
// A GEMM per group and tap with M = o, N = c and the reduction over the pixels (n,h,w), which is the
// contiguous axis of both operands - exactly what the matrix instructions want.
//
// Both operands are staged pixel-contiguous into LDS.  In the kernels of this file rows have a pitch of W plus at least
// one zero column: that column is the zero padding of the window on either side, so a tap is a pure
// shift of the X index by (kw - pw) elements and needs no mask.  G has zeros in its pad columns, so
// whatever X holds there never contributes.  With a window along h as well (KH = 3) a chunk of rows stays inside one image,
// X is staged with its KH-1 halo rows (zero outside the image), and tap kh is a further shift by kh whole rows.
//
// The pixel axis is split over workgroups (split-K); each writes its tile of sums into the workspace in
// the register layout of the accumulators (coalesced 16-byte stores) and a second kernel adds the partials
// in a fixed order and scatters them into dW, so the result does not depend on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>

#include "fp32_parts.h"
#include "plan.h"

namespace syno {

struct DwParams {
  int32_t G, Og, Cg, H, W, KH, KW, ph, pw;
  int32_t rows_total;                  // N*H
  int32_t h_wrap, h_shift, h_shift_g;  // X row = (h + h_shift + h_shift_g*g) mod H when wrapped, else h
  int32_t plane, gs_n, xs_n;           // H*W; image strides of G and X
  int32_t ws_g, ws_o, ws_c, ws_kh, ws_kw;   // dW strides
  int32_t w_elems;                     // elements of dW
  int32_t n_tiles, ct, slots;          // workgroup tiles (g, o block, c block); c-tiles per wave; 8 * ct * KH*KW
  int32_t pitch, TRK, CP, CPp;         // LDS row pitch, rows per chunk, chunk length (multiple of 32), LDS channel pitch
  int32_t CPg;                         // fp32 kernel: channel pitch of the G tile (it has no halo rows); CPp is X's
  int32_t rows_per_split, n_splits, n_oblk, n_cblk;
  int32_t n_xrows;                     // rows of X staged per chunk: TRK + KH - 1
  int32_t cpi;                         // KH > 1: chunks per image (chunks do not cross images); else 0
  int32_t ipc, n_images;               // bf16 rows, cpi == 1: whole images per chunk, each with its own halo rows; images
  int32_t chunks_per_split, n_chunks;
  int32_t items;                       // 64 * n_xrows * W/2 dword items per tensor per chunk
  uint32_t magic_w2, magic_rw2;        // ceil(2^32/d) for d = items per row and n_xrows * items per row (0 for d = 1)
  int32_t lds_x_off, lds_tab_off, lds_bytes;
  // fp32 kernel for windows with a row extent (chunks inside one image, source rows affine in the staged row):
  int32_t direct;                      // that kernel takes this plan
  int32_t ni_g, ni_x;                  // staging items per thread of G and of X
  int32_t mode;                        // pixels per staging item: 4, 2, 1, or a whole row of 7 or 14
  int32_t lds_buf;                     // bytes of one LDS buffer (G tile, then X tile at lds_x_off); there are two
  uint32_t magic_cpi;                  // ceil(2^32/d) for d = cpi (0 for d = 1); magic_w2 is for the items per row
  // fp32 on the bf16 matrix cores (dw_split.h): `pitch` pixels per stream row, CPp LDS elements per X channel
  int32_t parts;                       // that kernel takes this plan
  int32_t stream_reach, stream_ring;   // pixels of X read beyond a chunk on either side; pixels in the ring
  uint32_t m_pitch, m_rows;            // ceil(2^32/d) for d = pitch and d = the rows of an image in the stream
  uint32_t m_groups;                   // the same for the items of an X channel in a chunk with its window (dw_split.h)
  // bf16 (dw_stream_bf16.h): channels of a workgroup's tile, whose slots are (output-channel tile, input-channel tile, tap)
  int32_t stream, tile_o, tile_c;
  int32_t narrow;                      // rows of the image have 1, 2 or 3 pixels, and the record's H x W are 8-pixel items of them (else 0)
  uint32_t g_last, x_last;             // byte offset of the last place in G and X with 8 elements behind it
  int32_t tail_chunk;                  // chunks from here on may hold items that reach past the tensor's end
};

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
// f(integral_constant<int, I>) for I = 0 .. N-1
template <int I, int N, class F>
__device__ __forceinline__ void for_blocks(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    for_blocks<I + 1, N>(f);
  }
}

__device__ __forceinline__ uint32_t alignbit16(uint32_t hi, uint32_t lo) { return __builtin_amdgcn_alignbit(hi, lo, 16); }

template <int KH, int KW, int CT>
__device__ __forceinline__ void dw_finish(const DwParams& p, float* __restrict__ partial, int g, int ob, int cb, int split,
                                          int widx, int lane, const floatx4 (&acc)[2][CT][KH * KW]);

// The k-steps of one staged chunk: 4 pixels each; the fragments of the next step are read while the MFMAs of the
// current one issue (one wave per SIMD here, so nothing else would cover the LDS latency).
template <int KH, int KW, int CT>
__device__ __forceinline__ void dw_f32_chunk(const DwParams& p, const float* gl, const float* xl, const int (&a_base)[2],
                                             const int (&b_base)[CT], floatx4 (&acc)[2][CT][KH * KW], int first = 0,
                                             int stride = 1) {
  constexpr int T = KH * KW;
  const int steps = p.CP >> 2;
  auto read = [&](int st, float (&a)[2], float (&b)[CT * T]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = gl[a_base[i] + st * 4];
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
      for (int kh = 0; kh < KH; ++kh)
#pragma unroll
        for (int t = 0; t < KW; ++t) b[i * T + kh * KW + t] = xl[b_base[i] + st * 4 + kh * p.pitch + t];
  };
  auto mfmas = [&](const float (&a)[2], const float (&b)[CT * T]) {
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int ao = 0; ao < 2; ++ao)
          acc[ao][i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ao], b[i * T + t], acc[ao][i][t], 0, 0, 0);
  };
  auto interleave = [&]() {       // (left to the compiler when a step has only a handful of MFMAs)
    if constexpr (CT * T >= 6)
#pragma unroll
    for (int i = 0; i < CT * T; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);     // 2 MFMAs
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // 1 LDS read
    }
  };
  // the wave takes steps first, first + stride, ... (waves that share an output tile split the steps between them)
  float fa0[2], fb0[CT * T], fa1[2], fb1[CT * T];
  int st = first;
  if (st >= steps) return;
  read(st, fa0, fb0);
  for (; st + 2 * stride < steps; st += 2 * stride) {
    // one fragment read of the next step after every second MFMA of the current one: the reads issue in the
    // shadow of the matrix pipe and a whole step lies between a fragment's read and its use
    read(st + stride, fa1, fb1); mfmas(fa0, fb0); interleave();
    read(st + 2 * stride, fa0, fb0); mfmas(fa1, fb1); interleave();
  }
  if (st + stride < steps) { read(st + stride, fa1, fb1); mfmas(fa0, fb0); mfmas(fa1, fb1); }
  else mfmas(fa0, fb0);
}

// Leaves the workgroup's sums: in dW itself when there is one split, else in the workspace in accumulator layout.
template <int KH, int KW, int CT>
__device__ __forceinline__ void dw_finish(const DwParams& p, float* __restrict__ partial, int g, int ob, int cb, int split,
                                              int widx, int lane, const floatx4 (&acc)[2][CT][KH * KW]) {
  constexpr int CX = 32 * CT, T = KH * KW;
  const int wo = widx >> 1, wc = widx & 1;
  // One split only (large dW, few pixels): nothing to add up, the sums go straight into dW (`partial` is dW then):
  // lane holds 4 consecutive o (rows of D) at one c (column).
  if (p.n_splits == 1) {
    float* dw = partial + (int64_t)g * p.ws_g;
#pragma unroll
    for (int ao = 0; ao < 2; ++ao)
#pragma unroll
      for (int i = 0; i < CT; ++i) {
        const int c = cb * CX + (CT * wc + i) * 16 + (lane & 15);
        if (c >= p.Cg) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int o = ob * 64 + (2 * wo + ao) * 16 + 4 * (lane >> 4) + v;
          if (o >= p.Og) continue;
#pragma unroll
          for (int t = 0; t < T; ++t)
            dw[(int64_t)o * p.ws_o + (int64_t)c * p.ws_c + (t / KW) * p.ws_kh + (t % KW) * p.ws_kw] = acc[ao][i][t][v];
        }
      }
    return;
  }
  // partial[split][tile][slot][lane]: every accumulator register quadruple goes out as it is, one 16-byte store
  // per lane (1 KB per wave and slot); the reduction kernel knows which weights a (slot, lane) holds
  constexpr int SLOTS = 8 * CT * T;
  const int tile = (g * p.n_oblk + ob) * p.n_cblk + cb;
  floatx4* dst = reinterpret_cast<floatx4*>(partial) +
                 ((int64_t)split * p.n_tiles + tile) * (SLOTS * 64) + (widx * 2 * CT * T) * 64 + lane;
#pragma unroll
  for (int ao = 0; ao < 2; ++ao)
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
      for (int t = 0; t < T; ++t) dst[((ao * CT + i) * T + t) * 64] = acc[ao][i][t];
}

#include "dw_split.h"
#include "dw_stream_bf16.h"

// fp32 inputs: the same contraction with v_mfma_f32_16x16x4_f32, whose K-step is 4 consecutive pixels (lane ->
// row l%16, pixel l/16).  Operands are single dwords, so a tap is any element shift and nothing has to be cut;
// staging moves items of VEC adjacent pixels of a row (4 when W is a multiple of 4, else 2 or 1), at most
// kF32Items per thread and tensor, which wait in registers while the previous chunk is computed.
constexpr int kF32Items = 18;     // staging items per thread, tensor and chunk
constexpr int kGuardF = 4;       // zero floats in front of each X channel row
constexpr int kRowsThreads = 512;
constexpr int kRowsBatches = 2;   // staging batches (of 28 floats per thread and tensor) a chunk may need   // staging items per thread and tensor of the kernel for windows with a row extent

template <int KH, int KW, int CT, int VEC>
__global__ __launch_bounds__(256) void dw_mfma_f32(const DwParams p, const float* __restrict__ Gt,
                                                   const float* __restrict__ Xt, float* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* gl = reinterpret_cast<float*>(smem);                   // [64][CPg]
  float* xl = reinterpret_cast<float*>(smem + p.lds_x_off);     // [32*CT][CPp], data starts at kGuardF
  int* row_tab = reinterpret_cast<int*>(smem + p.lds_tab_off);  // [2][n_xrows]
  constexpr int CX = 32 * CT, T = KH * KW;

  const int tid = threadIdx.x, lane = tid & 63;
  const int widx = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = widx >> 1, wc = widx & 1;
  int bid = blockIdx.x;
  const int split = bid % p.n_splits; bid /= p.n_splits;
  const int cb = bid % p.n_cblk; bid /= p.n_cblk;
  const int ob = bid % p.n_oblk;
  const int g = bid / p.n_oblk;
  const int chunk_begin = split * p.chunks_per_split;
  const int chunk_end = min(p.n_chunks, chunk_begin + p.chunks_per_split);
  {
    uint4* z = reinterpret_cast<uint4*>(smem);
    const int n16 = p.lds_tab_off >> 4;
    for (int i = tid; i < n16; i += 256) z[i] = make_uint4(0, 0, 0, 0);
  }
  const int o_lim = p.Og - ob * 64, c_lim = min(p.Cg - cb * CX, CX);
  const float* Gg = Gt + (int64_t)(g * p.Og + ob * 64) * p.plane;
  const float* Xg = Xt + (int64_t)(g * p.Cg + cb * CX) * p.plane;

  floatx4 acc[2][CT][T];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[a][b][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  int a_base[2], b_base[CT];     // element indices
#pragma unroll
  for (int a = 0; a < 2; ++a) a_base[a] = ((2 * wo + a) * 16 + (lane & 15)) * p.CPg + (lane >> 4);
#pragma unroll
  for (int b = 0; b < CT; ++b) b_base[b] = ((CT * wc + b) * 16 + (lane & 15)) * p.CPp + (lane >> 4) + kGuardF - p.pw;

  // ---- staging items of this thread (the same for every chunk): VEC pixels of (channel, row)
  typedef float vec_t __attribute__((ext_vector_type(VEC == 1 ? 2 : VEC), aligned(4)));
  int it_off[kF32Items], it_r[kF32Items], it_lo[kF32Items], it_lg[kF32Items];
  {
    const int WV = p.W / VEC;                        // items per row
#pragma unroll
    for (int k = 0; k < kF32Items; ++k) {
      const int idx = tid + k * 256;
      const int ch = __umulhi((uint32_t)idx, p.magic_rw2);
      const int rem = idx - ch * (p.n_xrows * WV);
      const int r = p.magic_w2 ? __umulhi((uint32_t)rem, p.magic_w2) : rem;   // (one item per row: no division)
      const int j = (rem - r * WV) * VEC;
      const bool used = idx < p.items;
      it_off[k] = ch * p.plane + j;
      // bit 30 / 29: this channel exists in G / in X
      it_r[k] = used ? (r | (ch < o_lim ? (1 << 30) : 0) | (ch < c_lim ? (1 << 29) : 0)) : -1;
      it_lo[k] = (used && ch < CX) ? ch * p.CPp + r * p.pitch + j + kGuardF : -1;
      it_lg[k] = (used && r < p.TRK) ? ch * p.CPg + r * p.pitch + j : -1;
    }
  }
  float gr[kF32Items][VEC], xr[kF32Items][VEC];
  // source rows of chunk q: tab[r] = G row offset, tab[n_xrows + r] = X row offset (-1: none, zeros)
  auto rows_of = [&](int q, int tab) {     // tab: offset of the table inside row_tab (an index, so that LDS stays LDS)
    if (tid < p.n_xrows) {
      int go = -1, xo = -1;
      if (KH == 1) {
        const int rho = q * p.TRK + tid;
        if (rho < p.rows_total) {
          const int n = rho / p.H, h = rho - n * p.H;
          const int r = p.h_wrap ? (h + p.h_shift + p.h_shift_g * g) % p.H : h;
          go = n * p.gs_n + h * p.W;
          xo = n * p.xs_n + r * p.W;
        }
      } else {
        const int n = q / p.cpi, h0 = (q - n * p.cpi) * p.TRK;
        const int rows = min(p.TRK, p.H - h0);
        if (tid < rows) go = n * p.gs_n + (h0 + tid) * p.W;
        const int hx = h0 - p.ph + tid;
        if (tid < rows + KH - 1 && hx >= 0 && hx < p.H) xo = n * p.xs_n + hx * p.W;
      }
      row_tab[tab + tid] = go;
      row_tab[tab + p.n_xrows + tid] = xo;
    }
  };
  // global -> registers.  Every item is loaded unconditionally (items without a source read the block's first
  // elements) so that the requests go out back to back; what has no source is zeroed on the way to LDS.
  uint32_t g_ok = 0, x_ok = 0;           // bit k: item k of the chunk in flight has a source in G / in X
  auto load = [&](int tab) {
    g_ok = 0; x_ok = 0;
#pragma unroll
    for (int k = 0; k < kF32Items; ++k) {
      const int r = it_r[k] >= 0 ? (it_r[k] & 0xffff) : 0;
      const int go = row_tab[tab + r], xo = row_tab[tab + p.n_xrows + r];
      const bool gv = it_r[k] >= 0 && go >= 0 && (it_r[k] >> 30);
      const bool xv = it_r[k] >= 0 && xo >= 0 && ((it_r[k] >> 29) & 1);
      g_ok |= gv ? (1u << k) : 0u;
      x_ok |= xv ? (1u << k) : 0u;
      const float* gs = Gg + (gv ? go + it_off[k] : 0);
      const float* xs = Xg + (xv ? xo + it_off[k] : 0);
      if constexpr (VEC == 1) {
        gr[k][0] = *gs;
        xr[k][0] = *xs;
      } else {
        const vec_t a = *reinterpret_cast<const vec_t*>(gs);
        const vec_t b = *reinterpret_cast<const vec_t*>(xs);
#pragma unroll
        for (int e = 0; e < VEC; ++e) { gr[k][e] = a[e]; xr[k][e] = b[e]; }
      }
    }
  };
  auto store = [&]() {                   // registers -> LDS
#pragma unroll
    for (int k = 0; k < kF32Items; ++k) {
      if (it_lg[k] >= 0)
#pragma unroll
        for (int e = 0; e < VEC; ++e) gl[it_lg[k] + e] = ((g_ok >> k) & 1) ? gr[k][e] : 0.f;
      if (it_lo[k] >= 0)
#pragma unroll
        for (int e = 0; e < VEC; ++e) xl[it_lo[k] + e] = ((x_ok >> k) & 1) ? xr[k][e] : 0.f;
    }
  };

  // The next chunk travels global -> registers while the current one is computed out of LDS.
  const int tab[2] = {0, 2 * p.n_xrows};
  if (chunk_begin < chunk_end) {
    rows_of(chunk_begin, tab[0]);
    __syncthreads();                     // (also: the zero fill is complete)
    load(tab[0]);
  }
  for (int q = chunk_begin; q < chunk_end; ++q) {
    const bool more = q + 1 < chunk_end;
    const int next = ((q - chunk_begin + 1) & 1) ? tab[1] : tab[0];
    __syncthreads();                     // the previous chunk is fully consumed
    store();
    if (more) rows_of(q + 1, next);
    __syncthreads();
    if (more) load(next);
    dw_f32_chunk<KH, KW, CT>(p, gl, xl, a_base, b_base, acc);
  }
  dw_finish<KH, KW, CT>(p, partial, g, ob, cb, split, widx, lane, acc);
}

// fp32, windows with a row extent (KH = 3).  A chunk is TRK rows of ONE image, so the source of staged row r is
// row h0 + r of G and row h0 - 1 + r of X: one uniform base per chunk and tensor plus an offset that depends only on
// the item; nothing is looked up, and every load is a uniform base plus a 32-bit lane offset.
//
// Eight waves in two halves that trade places: while one half (4 waves, one per SIMD, each with its own part of the
// output tile) multiplies the chunk that lies in one LDS buffer, the other half fetches the next chunk from memory
// and lays it out in the second buffer; after one barrier the halves swap roles.  So each half computes every other
// chunk of the workgroup's share and stages the chunks it will compute itself; the matrix pipes always have a wave
// that issues MFMAs, and the memory round trips, the address arithmetic and the LDS writes of the staging all run
// beside them.  The sums of the two halves meet in LDS at the end.
// Staging goes in batches of up to 28 floats per thread and tensor: items of adjacent pixels of a row (a whole row of
// 7 or 14 pixels, else 4, 2 or 1 pixels), G (64 channels x TRK rows) and X (32*CT channels x TRK + 2 rows) together.  Rows that a chunk does not have (the halo above the
// first and below the last row of an image, the missing rows of an image's last chunk) are loaded from a safe
// address and written as zeros; items beyond the list or the group's channels go to 4 KB of LDS nobody reads.
template <int KW, int CT, int MODE>
__global__ __launch_bounds__(kRowsThreads) void dw_rows_f32(const DwParams p, const float* __restrict__ Gt,
                                                            const float* __restrict__ Xt, float* __restrict__ partial) {
  constexpr int KH = 3, CX = 32 * CT, T = KH * KW;
  // A staging item is MODE adjacent pixels of one staged row: 4, 2 or 1 (what the width divides by), or a whole row
  // of 7 or 14 pixels, moved as pieces of 4, 2 and 1.
  constexpr int FL = MODE;                                          // floats per item
  constexpr int NB = MODE == 7 ? 4 : MODE == 14 ? 2 : 7;            // items per thread and batch
  constexpr int NI = NB * kRowsBatches;                             // items per thread and chunk at most
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t dump = (uint32_t)p.lds_tab_off;                // behind the two buffers

  const int tid = threadIdx.x, lane = tid & 63, htid = tid & 255;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int widx = wave & 3, half = wave >> 2;
  const int wo = widx >> 1, wc = widx & 1;
  int bid = blockIdx.x;
  const int split = bid % p.n_splits; bid /= p.n_splits;
  const int cb = bid % p.n_cblk; bid /= p.n_cblk;
  const int ob = bid % p.n_oblk;
  const int g = bid / p.n_oblk;
  const int chunk_begin = split * p.chunks_per_split;
  const int chunk_end = min(p.n_chunks, chunk_begin + p.chunks_per_split);
  {
    uint4* z = reinterpret_cast<uint4*>(smem);
    const int n16 = p.lds_tab_off >> 4;
    for (int i = tid; i < n16; i += kRowsThreads) z[i] = make_uint4(0, 0, 0, 0);
  }
  const int o_lim = p.Og - ob * 64, c_lim = min(p.Cg - cb * CX, CX);
  const float* Gg = Gt + (int64_t)(g * p.Og + ob * 64) * p.plane;
  const float* Xg = Xt + (int64_t)(g * p.Cg + cb * CX) * p.plane;

  floatx4 acc[2][CT][T];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[a][b][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  int a_base[2], b_base[CT];     // element indices inside a buffer's G and X tile
#pragma unroll
  for (int a = 0; a < 2; ++a) a_base[a] = ((2 * wo + a) * 16 + (lane & 15)) * p.CPg + (lane >> 4);
#pragma unroll
  for (int b = 0; b < CT; ++b) b_base[b] = ((CT * wc + b) * 16 + (lane & 15)) * p.CPp + (lane >> 4) + kGuardF - p.pw;

  // ---- this thread's staging items, worked out once.  256 threads of a half share a tensor's channels evenly
  // (4 threads per G channel, 256 / CX per X channel); a thread takes every 4th (8th) item of its channel.  Per
  // item: the byte offset from the chunk's first source row, and the LDS byte offset inside a buffer with the staged
  // row in the top byte (row 255: never).
  uint32_t g_off[NI], g_put[NI], x_off[NI], x_put[NI];
  {
    const int WR = p.W / FL;                     // items per row
    auto plan_items = [&](uint32_t (&off)[NI], uint32_t (&put)[NI], int tpc_log2, int rows_staged, int ch_lim,
                          int ch_pitch, int lds_first, uint32_t safe) {
      const int ch = htid >> tpc_log2, sub = htid & ((1 << tpc_log2) - 1);
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const int i = sub + (k << tpc_log2);
        const int r = p.magic_w2 ? (int)__umulhi((uint32_t)i, p.magic_w2) : i;
        const int j = (i - r * WR) * FL;
        const bool exists = r < rows_staged && ch < ch_lim;
        off[k] = exists ? (uint32_t)(ch * p.plane + r * p.W + j) * 4 : safe;
        // (items that never carry data write to a spare area behind the buffers, each lane to its own 64 bytes)
        put[k] = exists ? ((uint32_t)(lds_first + ch * ch_pitch + r * p.pitch + j) * 4) | ((uint32_t)r << 24)
                        : (dump + (uint32_t)lane * 64) | (255u << 24);
      }
    };
    plan_items(g_off, g_put, 2, p.TRK, o_lim, p.CPg, 0, 0u);
    plan_items(x_off, x_put, CT == 1 ? 3 : 2, p.n_xrows, c_lim, p.CPp, kGuardF + (p.lds_x_off >> 2), (uint32_t)p.W * 4);
  }
  // Pieces of an item: float offset and width.  Source rows are only element-aligned; in LDS a row of 7 starts on a
  // 32-byte boundary (pitch 8), every other layout is element-aligned as well.
  typedef float f4_t __attribute__((ext_vector_type(4), aligned(4)));
  typedef float f2_t __attribute__((ext_vector_type(2), aligned(4)));
  typedef float f4a_t __attribute__((ext_vector_type(4), aligned(16)));
  typedef float f2a_t __attribute__((ext_vector_type(2), aligned(8)));
  auto load_item = [&](float (&v)[FL], const char* src) {
    const float* f = reinterpret_cast<const float*>(src);
    int o = 0;
#pragma unroll
    for (; o + 4 <= FL; o += 4) { const f4_t t = *reinterpret_cast<const f4_t*>(f + o); v[o] = t[0]; v[o + 1] = t[1]; v[o + 2] = t[2]; v[o + 3] = t[3]; }
    if constexpr (FL % 4 >= 2) { const f2_t t = *reinterpret_cast<const f2_t*>(f + o); v[o] = t[0]; v[o + 1] = t[1]; o += 2; }
    if constexpr (FL % 2 == 1) v[o] = f[o];
  };
  auto store_item = [&](const float (&v)[FL], unsigned char* dst) {
    float* f = reinterpret_cast<float*>(dst);
    int o = 0;
#pragma unroll
    for (; o + 4 <= FL; o += 4) {
      if constexpr (MODE == 7) *reinterpret_cast<f4a_t*>(f + o) = f4a_t{v[o], v[o + 1], v[o + 2], v[o + 3]};
      else *reinterpret_cast<f4_t*>(f + o) = f4_t{v[o], v[o + 1], v[o + 2], v[o + 3]};
    }
    if constexpr (FL % 4 >= 2) {
      if constexpr (MODE == 7) *reinterpret_cast<f2a_t*>(f + o) = f2a_t{v[o], v[o + 1]};
      else *reinterpret_cast<f2_t*>(f + o) = f2_t{v[o], v[o + 1]};
      o += 2;
    }
    if constexpr (FL % 2 == 1) f[o] = v[o];
  };
  // One batch of one tensor: up to NB items, requested back to back; staged rows [r_lo, r_hi) exist in this chunk.
  struct Batch { float v[NB][FL]; };
  auto fetch = [&](Batch& bt, const char* src_base, const uint32_t* off, const uint32_t* put, int count, uint32_t safe,
                   int r_lo, int r_hi) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      if (k >= count) break;
      const bool ok = ((put[k] >> 24) - (uint32_t)r_lo) < (uint32_t)(r_hi - r_lo);
      load_item(bt.v[k], src_base + (ok ? off[k] : safe));
    }
  };
  auto put_batch = [&](Batch& bt, uint32_t buf, const uint32_t* put, int count, int r_lo, int r_hi) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      if (k >= count) break;
      const bool ok = ((put[k] >> 24) - (uint32_t)r_lo) < (uint32_t)(r_hi - r_lo);
      const bool never = (put[k] >> 24) == 255u;
#pragma unroll
      for (int e = 0; e < FL; ++e) bt.v[k][e] = ok ? bt.v[k][e] : 0.f;
      store_item(bt.v[k], smem + (put[k] & 0xffffffu) + (never ? 0u : buf));
    }
  };
  // Stages chunk q (rows [h0, h0 + rows) of image n) into the buffer at byte offset `buf`; run by the 256 threads of
  // one half.  The batches of G and X are requested together, then written.
  auto stage = [&](int q, uint32_t buf) {
    const int n = p.magic_cpi ? (int)__umulhi((uint32_t)q, p.magic_cpi) : q;
    const int h0 = (q - n * p.cpi) * p.TRK;
    const int rows = min(p.TRK, p.H - h0);
    const char* gb = reinterpret_cast<const char*>(Gg) + ((int64_t)n * p.gs_n + (int64_t)h0 * p.W) * 4;
    // (one row above the chunk; when the chunk starts an image that row is not read: staged row 0 does not exist then
    // and the safe offset points at the chunk's first row)
    const char* xb = reinterpret_cast<const char*>(Xg) + ((int64_t)n * p.xs_n + (int64_t)(h0 - 1) * p.W) * 4;
    const int x_lo = h0 == 0 ? 1 : 0, x_hi = min(rows + 2, p.H - h0 + 1);
#pragma unroll
    for (int b = 0; b < NI / NB; ++b) {
      const int ng = p.ni_g - b * NB, nx = p.ni_x - b * NB;       // (uniform) items of this batch
      if (ng <= 0 && nx <= 0) break;
      Batch bg, bx;
      fetch(bg, gb, g_off + b * NB, g_put + b * NB, ng, 0u, 0, rows);
      fetch(bx, xb, x_off + b * NB, x_put + b * NB, nx, (uint32_t)p.W * 4, x_lo, x_hi);
      put_batch(bg, buf, g_put + b * NB, ng, 0, rows);
      put_batch(bx, buf, x_put + b * NB, nx, x_lo, x_hi);
    }
  };

  __syncthreads();                                   // LDS is zeroed
  if (half == 0 && chunk_begin < chunk_end) stage(chunk_begin, 0u);
  __syncthreads();
  for (int q = chunk_begin; q < chunk_end; ++q) {
    const int par = (q - chunk_begin) & 1;
    if (par == half) {
      const unsigned char* cur = smem + par * p.lds_buf;
      dw_f32_chunk<KH, KW, CT>(p, reinterpret_cast<const float*>(cur), reinterpret_cast<const float*>(cur + p.lds_x_off),
                               a_base, b_base, acc);
    } else if (q + 1 < chunk_end) {
      stage(q + 1, (uint32_t)((par ^ 1) * p.lds_buf));
    }
    __syncthreads();
  }
  // the sums of the two halves meet in LDS: the upper waves leave theirs there, the lower ones add them
  floatx4* red = reinterpret_cast<floatx4*>(smem) + (widx * 2 * CT * T) * 64 + lane;
  if (half) {
#pragma unroll
    for (int ao = 0; ao < 2; ++ao)
#pragma unroll
      for (int i = 0; i < CT; ++i)
#pragma unroll
        for (int t = 0; t < T; ++t) red[((ao * CT + i) * T + t) * 64] = acc[ao][i][t];
  }
  __syncthreads();
  if (half) return;
#pragma unroll
  for (int ao = 0; ao < 2; ++ao)
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[ao][i][t] += red[((ao * CT + i) * T + t) * 64];
  dw_finish<KH, KW, CT>(p, partial, g, ob, cb, split, widx, lane, acc);
}

#include "dw_rows_bf16.h"

// Channels of the first element of 16 x 16 tile `sub` of a workgroup's tile (ob, cb)
struct TilePlace { int o, c; };
__device__ __forceinline__ TilePlace tile_place(const DwParams& p, int ob, int cb, int sub) {
  if (p.stream) {
    const int ct = p.tile_c >> 4, ao = sub / ct;
    return {ob * p.tile_o + ao * 16, cb * p.tile_c + (sub - ao * ct) * 16};
  }
  const int i = sub % p.ct, ao = (sub / p.ct) & 1, wave = sub / (p.ct * 2);
  return {ob * 64 + (2 * (wave >> 1) + ao) * 16, cb * 32 * p.ct + (p.ct * (wave & 1) + i) * 16};
}

// Adds the split partials kept in the accumulator layout of the contraction kernels, in 64 bits, and writes the sums into dW (up
// to 256 partials in 32 bits were half of a weight gradient's error: fp32 64x16x16 28x28 1.6e-7 -> 8.2e-8 relative, 2x2 32x64x64 28x28
// 1.6e-7 -> 6.5e-8, bf16 1x1 32x64x64 56x56 1.6e-7 -> 7.6e-8; the reads bound these kernels, calls take 0 to 0.5 us longer);
// the variant for few splits of a large dW.  A block owns one 16 (o) x 16 (c) tile with all its T taps: T
// consecutive slots of 64 quadruples, slot = sub*T + t, where `sub` names the o-tile and the c-tile (tile_place); lane l of a quadruple holds rows 4*(l>>4) .. +3 (o) of column l&15 (c).  Wave j adds the
// splits, in order, for taps j, j+4, ...; then the threads walk the tile in (o, c, tap) order, which is contiguous in
// dW for the usual weight layouts, so dW is written in whole lines.
constexpr int kMaxTaps = 9;
__global__ __launch_bounds__(256) void dw_reduce_tiles(const DwParams p, const float4* __restrict__ partial,
                                                       float* __restrict__ dW) {
  __shared__ float sums[kMaxTaps][64][4];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int T = p.KH * p.KW;
  const int subs = p.slots / T;                    // 16x16 tiles per workgroup tile
  const int tile = blockIdx.x / subs, sub = blockIdx.x - tile * subs;
  const int64_t n4 = (int64_t)p.n_tiles * p.slots * 64;
  for (int t = grp; t < T; t += 4) {
    const int64_t e = ((int64_t)tile * p.slots + sub * T + t) * 64 + lane;
    const float4 f = partial[e];
    double x = f.x, y = f.y, z = f.z, w = f.w;
    for (int k = 1; k < p.n_splits; ++k) {
      const float4 v = partial[(int64_t)k * n4 + e];
      x += v.x; y += v.y; z += v.z; w += v.w;
    }
    *reinterpret_cast<float4*>(sums[t][lane]) = make_float4((float)x, (float)y, (float)z, (float)w);
  }
  __syncthreads();
  int q = tile;
  const int cb = q % p.n_cblk; q /= p.n_cblk;
  const int ob = q % p.n_oblk;
  const int g = q / p.n_oblk;
  const TilePlace at = tile_place(p, ob, cb, sub);
  const int c0 = at.c;
  // thread = (row ol, 16 threads per row); a row is 16*T consecutive (c, tap) pairs
  const int ol = threadIdx.x >> 4, o = at.o + ol;
  if (o >= p.Og) return;
  const uint32_t inv_t = (65536u + T - 1) / T;      // rem / T for rem < 16 * kMaxTaps
  const int64_t row = (int64_t)g * p.ws_g + (int64_t)o * p.ws_o;
  for (int rem = threadIdx.x & 15; rem < 16 * T; rem += 16) {
    const int cl = (int)(((uint32_t)rem * inv_t) >> 16), t = rem - cl * T;
    const int c = c0 + cl;
    if (c >= p.Cg) continue;
    const int kh = t / p.KW;
    dW[row + (int64_t)c * p.ws_c + kh * p.ws_kh + (t - kh * p.KW) * p.ws_kw] = sums[t][(ol >> 2) * 16 + cl][ol & 3];
  }
}

// The same sums for many splits and few tiles: a block owns one slot (64 quadruples, one tap of a 16x16 tile), which
// keeps enough blocks in flight when dW is small; the stores are scattered, which does not matter at that size.
// W waves take turns with the partials: 4, or 16 from 72 partials on where there are at most 256 slots: the chains of loads are then a
// fourth as long (weight gradients of one tile, the whole call: 72 to 95 partials 1.04 to 1.09 times as fast, from 96 on 1.03 to 1.13;
// 48 to 71 0.98 to 1.01, 24 to 47 0.99; with 600 slots 16 waves each take longer to start than they save).
template <int W>
__global__ __launch_bounds__(W * 64) void dw_reduce_slots(const DwParams p, const float4* __restrict__ partial,
                                                          float* __restrict__ dW) {
  __shared__ double4 sums[W][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t n4 = (int64_t)p.n_tiles * p.slots * 64;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  double4 s = make_double4(0., 0., 0., 0.);
#pragma unroll 4
  for (int k = grp; k < p.n_splits; k += W) {
    const float4 v = partial[(int64_t)k * n4 + e];
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  sums[grp][lane] = s;
  __syncthreads();
  if (grp != 0) return;
  double4 all = make_double4(0., 0., 0., 0.);
#pragma unroll
  for (int j = 0; j < W; j += 4) {
    const double4 a = sums[j][lane], b = sums[j + 1][lane], c4 = sums[j + 2][lane], d = sums[j + 3][lane];
    all.x += (a.x + b.x) + (c4.x + d.x); all.y += (a.y + b.y) + (c4.y + d.y); all.z += (a.z + b.z) + (c4.z + d.z); all.w += (a.w + b.w) + (c4.w + d.w);
  }
  const float r[4] = {(float)all.x, (float)all.y, (float)all.z, (float)all.w};
  const int T = p.KH * p.KW;
  int q = blockIdx.x;
  const int slot = q % p.slots; q /= p.slots;
  const int cb = q % p.n_cblk; q /= p.n_cblk;
  const int ob = q % p.n_oblk;
  const int g = q / p.n_oblk;
  const int t = slot % T, sub = slot / T;
  const TilePlace at = tile_place(p, ob, cb, sub);
  const int c = at.c + (lane & 15);
  if (c >= p.Cg) return;
  const int64_t base = (int64_t)g * p.ws_g + (int64_t)c * p.ws_c + (t / p.KW) * p.ws_kh + (t % p.KW) * p.ws_kw;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int o = at.o + 4 * (lane >> 4) + v;
    if (o < p.Og) dW[base + (int64_t)o * p.ws_o] = r[v];
  }
}

uint32_t magic_of(int d) { return (uint32_t)(((1ull << 32) + d - 1) / d); }

// bf16: the stream kernel's tile of sums per window - output-channel and input-channel tiles of 16 per wave, waves side by side
// along the input channels (the other waves share the k-steps)
struct StreamTile { int no, nc, wc; };
constexpr StreamTile stream_tile(int T, bool wide) {
  return T == 1 ? StreamTile{4, 4, 1} : T <= 4 ? StreamTile{2, 2, wide ? 2 : 1} : StreamTile{2, 1, 2};
}

// (cost: us, as the splits are chosen by)
bool fill_dw_stream(const syno_plan* plan, DwParams& p, double* cost_out) {
  const ConvLike& c = plan->conv;
  p = DwParams{};
  p.G = c.G; p.Og = c.Og; p.Cg = c.Cg; p.H = c.Ho; p.W = c.Wo; p.KH = c.KH; p.KW = c.KW; p.ph = c.ph; p.pw = c.pw;
  p.rows_total = c.N * c.Ho; p.n_images = c.N;
  p.h_wrap = c.h_wrap; p.h_shift = c.h_shift; p.h_shift_g = c.h_shift_g;
  p.plane = c.Ho * c.Wo;
  p.gs_n = c.G * c.Og * p.plane; p.xs_n = c.G * c.Cg * p.plane;
  if (std::min(plan->out_elems, plan->x_elems) < 8) return false;     // (the kernel reads 8 elements at a time)
  p.g_last = (uint32_t)(plan->out_elems - 8) * 2u; p.x_last = (uint32_t)(plan->x_elems - 8) * 2u;
  p.ws_g = c.ws_g; p.ws_o = c.ws_o; p.ws_c = c.ws_c; p.ws_kh = c.ws_kh; p.ws_kw = c.ws_kw;
  p.w_elems = (int32_t)plan->w_elems;
  p.stream = 1;
  // Rows are filled up to 8 pixels.  Nothing couples the pixels of a 1x1 window, so an image is one row then; a column of pixels under
  // a column of taps is a row under a row of taps; and rows of up to 3 pixels go several to an item where only neighbours along w
  // are read (us, each row filled up and so; the kernels before filled rows up to 2 or 4): 1x1 32x256x256 196x1 45 -> 14, 7x8x64 13x13
  // 13.8 -> 10.7; 3x1 32x256x256 196x1 89 -> 17; 1x3 196x1 82 -> 26, 98x2 35 -> 26.
  const bool one_row = !c.h_wrap && c.KW == 1 && (c.KH == 1 || (c.KH == 3 && c.Wo == 1));
  if (one_row) {
    p.H = 1; p.W = p.plane;
    if (c.KH == 3) { p.KH = 1; p.KW = 3; p.ws_kw = p.ws_kh; }
  } else if (!c.h_wrap && c.KH == 1 && c.KW == 3 && c.Wo <= 3) {
    p.narrow = c.Wo;
    p.W = c.Wo == 3 ? 6 : 4;
    p.H = (p.plane + p.W - 1) / p.W;
  }
  p.pitch = (p.W + 7) & ~7;
  const int T = p.KH * p.KW, rows = p.H + p.KH / 2;
  if (p.KH > 1 && kBfChunk + 2 * (p.KH / 2) * p.pitch > 64 * 8) return false;      // (an X channel's units are one wave's lanes)
  p.CPp = stream_x_pitch(p.KH, p.pitch);
  const int64_t stream = (int64_t)c.N * rows * p.pitch;
  if (stream >= (1ll << 31) - 16 * kBfChunk) return false;      // (positions, also of what is requested past the end)
  auto set_tile = [&](bool wide) {
    const StreamTile t = stream_tile(T, wide);
    p.tile_o = 16 * t.no; p.tile_c = 16 * t.nc * t.wc;
    p.slots = t.no * t.nc * t.wc * T;
    p.lds_bytes = std::max(2 * p.tile_o * stream_g_pitch(p.KW) + 2 * p.tile_c * p.CPp, 8 * t.no * t.nc * T * 1024);
    return p.lds_bytes <= 160 * 1024;
  };
  // windows of three taps: 64 input channels to a workgroup where every compute unit walks at least 8 chunks of them, so that each of
  // G's pixels is staged half as often (us, 32 and 64 channels; the kernels before had 64): gshift 64x512 28x28 in 2 groups 126, 97;
  // 3x1 128x512x512 7x7 58, 52; 1x3 16x512x512 28x28 67, 55; with fewer chunks the larger sums cost more: 3x1 64x128x128 28x28 (7) 23.2, 24.3,
  // 32x256x256 14x14 (4) 16.8, 17.5)
  const bool wide = T == 3 && !p.narrow &&
                    (stream / kBfChunk) * c.G * ((c.Og + 31) / 32) * ((c.Cg + 63) / 64) >= 8 * 256;
  if (!(wide && set_tile(true)) && !set_tile(false)) return false;
  // quotients by multiplication where they are exact
  if ((stream + 16 * kBfChunk) * std::max(p.pitch, rows) < (1ll << 32)) { p.m_pitch = magic_of(p.pitch); p.m_rows = magic_of(rows); }
  p.n_chunks = (int)((stream + kBfChunk - 1) / kBfChunk);
  p.tail_chunk = (int)std::max<int64_t>(0, ((int64_t)(c.N - 1) * rows - p.KH) * p.pitch / kBfChunk - 1);      // (the last image's)
  p.n_oblk = (c.Og + p.tile_o - 1) / p.tile_o;
  p.n_cblk = (c.Cg + p.tile_c - 1) / p.tile_c;
  const int64_t tiles = (int64_t)c.G * p.n_oblk * p.n_cblk;
  if (tiles * p.n_chunks >= (1ll << 31)) return false;
  p.n_tiles = (int)tiles;
  // splits of the stream: rounds of 256 workgroups, each the start and end of a kernel and its chunks, against a second kernel
  // that reads the sums back (us; a chunk of unaligned rows' loads takes longer.  With 0.4 us a chunk six chunks of 7x8x64 13x13
  // 1x1 stayed in one workgroup: 22.5 us, in six 14.8; nine taps' whole rows of dW out of LDS cost one split 2.5 us: 2x128x128 14x14 in one
  // 13.6, in two 11.9)
  const double ends = 8., second = T == 9 ? -.9 : 1.6, chunk = T == 9 ? 1.7 : p.W % 8 == 0 ? 1.2 : 1.7;
  int64_t splits = 1;
  double best = 0;
  for (int64_t s = 1; s <= p.n_chunks && (s == 1 || s * tiles <= 256); ++s) {
    const int64_t per = (p.n_chunks + s - 1) / s;
    const double cost = (double)((s * tiles + 255) / 256) * (ends + per * chunk) + (s > 1 ? second + (double)s * tiles * p.slots * 2048. / 4e6 : 0.);
    if (s == 1 || cost < best) { best = cost; splits = s; }
  }
  // (the option counts workgroups of 64 output and 64, from 5 taps on 32, input channels, as the fp32 kernels')
  const int64_t blocks = (int64_t)c.G * ((c.Og + 63) / 64) * ((c.Cg + (T <= 3 ? 63 : 31)) / (T <= 3 ? 64 : 32));
  if (plan->opt.dw_workgroups > 0) splits = std::max<int64_t>(1, std::min<int64_t>(p.n_chunks, plan->opt.dw_workgroups / blocks));
  while (splits > 1 && splits * tiles * p.slots * 1024 > (int64_t)SYNO_STATIC_SCRATCH_BYTES) splits /= 2;      // (an option may ask for more)
  p.chunks_per_split = (int)((p.n_chunks + splits - 1) / splits);
  p.n_splits = (p.n_chunks + p.chunks_per_split - 1) / p.chunks_per_split;
  // (windows of three taps: a long run's chunks are shorter than the few that the rule above is for)
  const double rounds = (double)((tiles * p.n_splits + 255) / 256);
  *cost_out = T == 3 ? rounds * (9. + p.chunks_per_split * (p.tile_c == 64 ? 1.4 : .93)) + (p.n_splits > 1 ? (double)p.n_splits * tiles * p.slots * 2048. / 4e6 : 0.) : best;
  return true;
}

// bf16 rows of 14 pixels under a window of three rows (dw_rows_bf16.h): chunks of an image's rows, or of several small images, as large as a
// thread's list of rows and two LDS buffers allow.
bool fill_dw_rows_bf16(const syno_plan* plan, DwParams& p, double* cost_out) {
  const ConvLike& c = plan->conv;
  if (c.KH != 3 || c.KW > 3 || c.KW == 2 || c.Wo != 14) return false;
  DwParams base{};
  base.G = c.G; base.Og = c.Og; base.Cg = c.Cg; base.H = c.Ho; base.W = c.Wo; base.KH = c.KH; base.KW = c.KW; base.ph = c.ph; base.pw = c.pw;
  base.rows_total = c.N * c.Ho; base.n_images = c.N;
  base.plane = c.Ho * c.Wo;
  base.gs_n = c.G * c.Og * base.plane; base.xs_n = c.G * c.Cg * base.plane;
  base.ws_g = c.ws_g; base.ws_o = c.ws_o; base.ws_c = c.ws_c; base.ws_kh = c.ws_kh; base.ws_kw = c.ws_kw;
  base.w_elems = (int32_t)plan->w_elems;
  base.direct = 1;
  base.pitch = 16;
  const int T = c.KH * c.KW, cx = T == 3 ? 64 : 32;
  auto skew = [](int v) { v = (v + 7) & ~7; return (v & 31) == 0 ? v + 8 : v; };
  auto cfg = [&](int t, int ipc, DwParams& o) {     // t rows of an image per chunk, or ipc whole images
    o = base;
    o.ipc = ipc;
    o.n_xrows = ipc > 1 ? ipc * (c.Ho + 2) : t + 2;
    o.TRK = ipc > 1 ? o.n_xrows - 2 : t;
    o.CP = (o.TRK * o.pitch + 31) & ~31;
    o.CPg = skew(o.CP + 8);
    o.CPp = skew(std::max(o.CP, o.n_xrows * o.pitch) + 2 * o.pitch + 48);
    o.ni_g = ((ipc > 1 ? o.n_xrows : t) + 3) / 4;
    o.ni_x = (o.n_xrows + 256 / cx - 1) / (256 / cx);
    o.lds_x_off = 64 * o.CPg * 2;
    o.lds_buf = o.lds_x_off + cx * o.CPp * 2;
    o.lds_tab_off = 2 * o.lds_buf;
    o.lds_bytes = std::max(o.lds_tab_off + 4096, 4 * 2 * (cx / 32) * T * 1024);
    return std::max(o.ni_g, o.ni_x) <= 2 * kRowsBatches && o.lds_bytes <= 160 * 1024 && o.n_xrows <= 254;
  };
  int t = c.Ho;
  while (t > 1 && !cfg(t, 1, p)) --t;
  if (!cfg(t, 1, p)) return false;
  if (t == c.Ho) {                 // whole images: as many per chunk as fit
    int m = 1;
    DwParams more;
    while (m < c.N && cfg(c.Ho, m + 1, more)) { p = more; ++m; }
    p.cpi = 1;
    p.n_chunks = (c.N + p.ipc - 1) / p.ipc;
  } else {
    p.cpi = (c.Ho + t - 1) / t;
    t = (c.Ho + p.cpi - 1) / p.cpi;       // chunks of an image about equally long
    cfg(t, 1, p);
    p.cpi = (c.Ho + t - 1) / t;
    p.n_chunks = c.N * p.cpi;
  }
  if ((int64_t)p.n_chunks * p.cpi >= (1ll << 32)) return false;      // (exact quotients)
  p.magic_cpi = magic_of(p.cpi);
  p.n_oblk = (c.Og + 63) / 64;
  p.n_cblk = (c.Cg + cx - 1) / cx;
  const int64_t tiles = (int64_t)c.G * p.n_oblk * p.n_cblk;
  if (tiles * p.n_chunks >= (1ll << 31)) return false;
  p.n_tiles = (int)tiles;
  p.ct = cx / 32;
  p.slots = 8 * p.ct * T;
  const int64_t target = plan->opt.dw_workgroups > 0 ? plan->opt.dw_workgroups : 256;
  int64_t splits = std::max<int64_t>(1, std::min<int64_t>(p.n_chunks, target / std::max<int64_t>(1, tiles)));
  while (splits > 1 && splits * tiles * p.slots * 1024 > (int64_t)SYNO_STATIC_SCRATCH_BYTES) splits /= 2;
  p.chunks_per_split = (int)((p.n_chunks + splits - 1) / splits);
  p.n_splits = (p.n_chunks + p.chunks_per_split - 1) / p.chunks_per_split;
  const double rounds = (double)((tiles * p.n_splits + 255) / 256), images = (double)c.N * p.chunks_per_split / p.n_chunks * c.Ho / 14.;
  *cost_out = rounds * (T == 3 ? 11. + 1.87 * images : 13. + 1.75 * images) + (p.n_splits > 1 ? (double)p.n_splits * tiles * p.slots * 2048. / 4e6 : 0.);
  return true;
}

// bf16: the stream, or the rows where their estimate is the lower one
bool fill_dw_bf16(const syno_plan* plan, DwParams& p) {
  double stream, rows;
  DwParams r;
  if (!fill_dw_stream(plan, p, &stream)) return false;
  if (fill_dw_rows_bf16(plan, r, &rows) && rows < stream) p = r;
  return true;
}

// fp32 configuration: element items, k-steps of 4 pixels, channel pitch = 4 * odd floats so that the 16 rows x 4
// pixels of a fragment read fall into 64 distinct banks.
bool fill_dw_f32_as(const syno_plan* plan, DwParams& p, bool direct) {
  const ConvLike& c = plan->conv;
  p = DwParams{};
  p.G = c.G; p.Og = c.Og; p.Cg = c.Cg; p.H = c.Ho; p.W = c.Wo; p.KH = c.KH; p.KW = c.KW; p.ph = c.ph; p.pw = c.pw;
  p.rows_total = c.N * c.Ho;
  p.h_wrap = c.h_wrap; p.h_shift = c.h_shift; p.h_shift_g = c.h_shift_g;
  p.plane = c.Ho * c.Wo;
  p.gs_n = c.G * c.Og * p.plane; p.xs_n = c.G * c.Cg * p.plane;
  p.ws_g = c.ws_g; p.ws_o = c.ws_o; p.ws_c = c.ws_c; p.ws_kh = c.ws_kh; p.ws_kw = c.ws_kw;
  p.w_elems = (int32_t)plan->w_elems;
  p.pitch = c.Wo + std::max(1, std::max(c.pw, c.KW - 1 - c.pw));     // at least one zero column between rows
  const int cx = (c.KH * c.KW <= 3) ? 64 : 32, halo = c.KH - 1;
  // rows per chunk: about 200 staged pixels per channel, a bounded number of staging batches per thread, and
  // both tiles within LDS
  const int vec = (c.Wo % 4 == 0) ? 4 : (c.Wo % 2 == 0) ? 2 : 1;
  // windows with a row extent go to the kernel that derives its source rows from the chunk's position and keeps
  // two chunks in LDS (one being multiplied, one being staged); the others look rows up in a table
  const int budget = kF32Items * vec * 256;        // table kernel: floats per tensor and chunk
  int trk = std::max(1, 200 / p.pitch);
  if (direct && c.Ho * p.pitch <= 256) trk = c.Ho;     // small images whole
  if (c.KH > 1) trk = std::min(trk, c.Ho);
  auto pitch_of = [&](int elems) { int v = (elems + 3) & ~3; return ((v >> 2) & 1) ? v : v + 4; };   // 4 * odd
  auto lds_need = [&](int t) {
    if (direct)      // both buffers, the spare 16 bytes
      return (int64_t)2 * (64 * pitch_of(((t * p.pitch + 3) & ~3) + 4) + cx * pitch_of((t + halo) * p.pitch + kGuardF + 8)) * 4 + 4096;
    return (int64_t)64 * (t * p.pitch + 16) * 4 + (int64_t)cx * ((t + halo) * p.pitch + halo * p.pitch + 32) * 4;
  };
  // staging items of that kernel: whole rows of 7 or 14 pixels, else `vec` pixels; 4 threads per G channel and
  // 256 / cx per X channel share a channel's items
  const int mode = (c.Wo == 7 || c.Wo == 14) ? c.Wo : vec;
  const int ni_cap = (mode == 7 ? 4 : mode == 14 ? 2 : 7) * kRowsBatches;
  auto items_g = [&](int t) { return (t * (c.Wo / mode) + 3) / 4; };
  auto items_x = [&](int t) { return ((t + halo) * (c.Wo / mode) + 256 / cx - 1) / (256 / cx); };
  auto over = [&](int t) {
    if (direct) return lds_need(t) > 160 * 1024 || std::max(items_g(t), items_x(t)) > ni_cap || t + halo > 254;
    return 64 * (t + halo) * c.Wo > budget || lds_need(t) > 140 * 1024;
  };
  while (trk > 1 && over(trk)) --trk;
  if (over(trk)) return false;
  if (c.KH > 1) {
    p.cpi = (c.Ho + trk - 1) / trk;
    trk = (c.Ho + p.cpi - 1) / p.cpi;
    p.n_chunks = c.N * p.cpi;
  } else {
    trk = std::min(trk, p.rows_total);
    p.n_chunks = (p.rows_total + trk - 1) / trk;
  }
  p.TRK = trk;
  p.n_xrows = trk + halo;
  p.CP = (p.TRK * p.pitch + 3) & ~3;
  if (direct) {
    // the last k-step reads G up to CP - 1 and X up to n_xrows * pitch + 7 (its guard included)
    p.CPg = pitch_of(p.CP + 4);
    p.CPp = pitch_of(p.n_xrows * p.pitch + kGuardF + 8);
  } else {
    p.CPp = (std::max(p.CP, p.n_xrows * p.pitch) + halo * p.pitch + c.KW + kGuardF + 4 + 3) & ~3;
    if (((p.CPp >> 2) & 1) == 0) p.CPp += 4;
    p.CPg = (p.CP + 4 + 3) & ~3;
    if (((p.CPg >> 2) & 1) == 0) p.CPg += 4;
  }
  p.items = 64 * p.n_xrows * (c.Wo / vec);
  p.magic_w2 = magic_of(c.Wo / vec);
  p.magic_rw2 = magic_of(p.n_xrows * (c.Wo / vec));
  p.n_oblk = (c.Og + 63) / 64;
  p.n_cblk = (c.Cg + cx - 1) / cx;
  const int tiles = c.G * p.n_oblk * p.n_cblk;
  p.n_tiles = tiles;
  p.ct = cx / 32;
  p.slots = 8 * p.ct * c.KH * c.KW;
  const int target = plan->opt.dw_workgroups > 0 ? plan->opt.dw_workgroups : 256;
  int splits = std::max(1, std::min(p.n_chunks, target / std::max(1, tiles)));
  while (splits > 1 && (int64_t)splits * tiles * p.slots * 1024 > (40ll << 20)) splits /= 2;
  p.chunks_per_split = (p.n_chunks + splits - 1) / splits;
  p.rows_per_split = p.chunks_per_split * p.TRK;
  p.n_splits = (p.n_chunks + p.chunks_per_split - 1) / p.chunks_per_split;
  p.lds_x_off = 64 * p.CPg * 4;
  p.lds_tab_off = p.lds_x_off + cx * p.CPp * 4;
  p.lds_bytes = p.lds_tab_off + ((2 * 2 * p.n_xrows * 4 + 15) & ~15);     // two row tables (current and next chunk)
  if (direct) {
    p.mode = mode;
    p.direct = 1;
    p.ni_g = items_g(p.TRK);
    p.ni_x = items_x(p.TRK);
    p.magic_w2 = magic_of(c.Wo / mode);
    p.magic_cpi = magic_of(p.cpi);
    p.lds_buf = p.lds_x_off + cx * p.CPp * 4;
    p.lds_tab_off = 2 * p.lds_buf;            // the 4 KB that retired items write to
    // (the final sum of the two halves needs 4 waves x 2*ct*taps accumulators x 1 KB of LDS)
    p.lds_bytes = std::max(p.lds_tab_off + 4096, 4 * 2 * p.ct * c.KH * c.KW * 1024);
    return p.lds_bytes <= 160 * 1024;
  }
  return p.lds_bytes <= 144 * 1024 && 64 * p.CPp < (1 << 30) && p.n_xrows <= 256 && p.n_xrows <= 256 &&
         (int64_t)64 * p.n_xrows * c.Wo * std::max(c.Wo, p.n_xrows * c.Wo) < (1ll << 32);
}

// Windows with a row extent take the kernel with the alternating wave halves when their rows fit its item lists,
// else (and all other windows) the kernel that looks its rows up in a table.
bool fill_dw_f32(const syno_plan* plan, DwParams& p) {
  if (plan->conv.KH == 2) return false;          // (not instantiated)
  if (plan->conv.KH == 3 && fill_dw_f32_as(plan, p, true)) return true;
  return fill_dw_f32_as(plan, p, false);
}

// fp32 on the bf16 matrix cores: windows of 1 or 3 along either axis, or 2x2 (errors against 64 bits 0.34 to 0.79 of the index
// program's, which had it before, largest 0.28 to 0.77; on the fp32 instructions 0.9 to 4.2), rows not cyclic.  Images of up to 4 columns, of whose
// rows at least half would be filling, and a single chunk of pixels, where there is nothing to overlap the splitting with,
// stay with the fp32 instructions: 64x256x256 64x1 3x1 86 us against 52, 1x1024x1024 7x7 50.5 against 45; from 7 columns
// and two chunks on this one is ahead (2x512x512 7x7 26.5 against 26.4, 4x512x512 29.9 against 31.1, 32x64x64 56x56 59 against 86).
bool fill_dw_split(const syno_plan* plan, DwParams& p) {
  const ConvLike& c = plan->conv;
  if (c.h_wrap || c.Wo <= 4) return false;
  if (c.KH == 2 ? c.KW != 2 : (c.KH != 1 && c.KH != 3) || (c.KW != 1 && c.KW != 3)) return false;
  if (std::max(plan->x_elems, plan->out_elems) * 4 >= kNoPixel) return false;        // byte offsets
  p = DwParams{};
  p.G = c.G; p.Og = c.Og; p.Cg = c.Cg; p.H = c.Ho; p.W = c.Wo; p.KH = c.KH; p.KW = c.KW; p.ph = c.ph; p.pw = c.pw;
  p.rows_total = c.N * c.Ho; p.n_images = c.N;
  p.plane = c.Ho * c.Wo;
  p.gs_n = c.G * c.Og * p.plane; p.xs_n = c.G * c.Cg * p.plane;
  p.ws_g = c.ws_g; p.ws_o = c.ws_o; p.ws_c = c.ws_c; p.ws_kh = c.ws_kh; p.ws_kw = c.ws_kw;
  p.w_elems = (int32_t)plan->w_elems;
  p.parts = 1;
  p.pitch = (c.Wo + 7) & ~7;
  p.TRK = 1;
  const int T = c.KH * c.KW;
  p.ct = T == 9 ? 1 : 2;
  const int cx = 32 * p.ct;
  p.stream_reach = (c.KH > 1 ? p.pitch : 0) + (c.KW > 1 ? 8 : 0);
  p.stream_ring = 2 * kStreamChunk + 2 * p.stream_reach;
  int units = p.stream_ring / 8;
  while ((units & 3) != 2) ++units;
  p.CPp = units * 8;
  const int64_t stream = (int64_t)c.N * (c.Ho + 1) * p.pitch;
  // (exact quotients, also for the positions that are requested past the end)
  if ((stream + 4096) * std::max(p.pitch, c.Ho + 1) >= (1ll << 32)) return false;
  p.m_pitch = magic_of(p.pitch); p.m_rows = magic_of(c.Ho + 1);
  p.m_groups = magic_of((kStreamChunk + 2 * p.stream_reach) / (p.ct == 1 ? 4 : 8));
  p.n_chunks = (int)((stream + kStreamChunk - 1) / kStreamChunk);
  if (p.n_chunks < 2) return false;
  p.n_oblk = (c.Og + 63) / 64;
  p.n_cblk = (c.Cg + cx - 1) / cx;
  const int tiles = c.G * p.n_oblk * p.n_cblk;
  p.n_tiles = tiles;
  p.slots = 8 * p.ct * T;
  const int target = plan->opt.dw_workgroups > 0 ? plan->opt.dw_workgroups : 256;
  int splits = std::max(1, std::min(p.n_chunks, target / std::max(1, tiles)));
  while (splits > 1 && (int64_t)splits * tiles * p.slots * 1024 > (40ll << 20)) splits /= 2;
  p.chunks_per_split = (p.n_chunks + splits - 1) / splits;
  p.rows_per_split = 0;
  p.n_splits = (p.n_chunks + p.chunks_per_split - 1) / p.chunks_per_split;
  p.lds_bytes = std::max(2 * 64 * kGUnits * 16 + kPlanes * cx * p.CPp * 2, 4 * 2 * p.ct * T * 1024);
  return p.lds_bytes <= 160 * 1024;
}

bool fill_any(const syno_plan* plan, DwParams& p) {
  if (plan->in_dtype == SYNO_BF16) return fill_dw_bf16(plan, p);
  // (a named variant of the fp32 contraction kernel asks for the fp32 instructions)
  if (plan->opt.mfma_variant > 0 && fill_dw_f32(plan, p)) return true;
  return fill_dw_split(plan, p) || fill_dw_f32(plan, p);
}

}  // namespace

bool mfma_dw_supports(const syno_plan* p) {
  if (!p->conv_like) return false;
  if (p->in_dtype != SYNO_BF16 && p->in_dtype != SYNO_F32) return false;
  const ConvLike& c = p->conv;
  if (c.sh != 1 || c.sw != 1 || c.w_wrap) return false;
  // windows: 1, 3 or 5 along an axis or 2x2, at most 9 taps (each tap is a set of accumulators); a 5-wide window along the
  // row only with fp32 inputs (the bf16 kernels cut their shifted fragments for 3-wide windows)
  if ((c.KH == 2) != (c.KW == 2)) return false;
  if (c.KH != 1 && ((c.KH != 2 && c.KH != 3 && c.KH != 5) || c.h_wrap || c.ph != c.KH / 2 || c.ws_kh < 0)) return false;
  if (c.Wi != c.Wo || c.Hi != c.Ho) return false;
  if (c.KW > 3 && !(c.KW == 5 && p->in_dtype == SYNO_F32)) return false;
  if (c.KH * c.KW > 9) return false;
  if (c.pw != c.KW / 2) return false;
  if (c.ws_kw < 0 || (c.Og == 1 && c.Cg == 1)) return false;
  DwParams dp;
  return fill_any(p, dp);
}

void mfma_dw_configure(syno_plan* plan) {
  DwParams dp;
  Launch& L = plan->launch[SYNO_BWD_WEIGHT];
  static_assert(sizeof(DwParams) <= sizeof(L.params), "parameter record does not fit");
  L.params_ready = fill_any(plan, dp);
  memcpy(L.params, &dp, sizeof dp);
  L.variant = 0;
  // one tile of fp32 sums (`slots` of 1 KB) per workgroup (whole tiles also where Og or Cg end inside one)
  L.workspace = dp.n_splits == 1 ? 0 : (size_t)dp.n_splits * dp.n_tiles * dp.slots * 1024;
  // problems that only dw_split takes (the fp32 instructions' kernels stage whole rows, which are too wide here): whatever
  // workspace it, or a plan around it, needs, the entry point without one has them on the index program
  DwParams f32;
  L.static_generic = dp.parts && !fill_dw_f32(plan, f32);
}

std::string mfma_dw_describe(const syno_plan* plan) {
  if (!plan->launch[SYNO_BWD_WEIGHT].params_ready) return "unconfigured";
  DwParams p;
  memcpy(&p, plan->launch[SYNO_BWD_WEIGHT].params, sizeof p);
  char b[256];
  if (p.stream) {
    snprintf(b, sizeof b, "stream pixels/chunk=%d pitch=%d chunks=%d splits=%d grid=%d lds=%dB tile=%dx%d", kBfChunk, p.pitch, p.n_chunks, p.n_splits,
             p.n_tiles * p.n_splits, p.lds_bytes, p.tile_o, p.tile_c);
    return b;
  }
  if (p.parts) {
    snprintf(b, sizeof b, "bf16-parts pixels/chunk=%d pitch=%d chunks=%d splits=%d grid=%d lds=%dB", kStreamChunk, p.pitch, p.n_chunks, p.n_splits,
             p.G * p.n_oblk * p.n_cblk * p.n_splits, p.lds_bytes);
    return b;
  }
  snprintf(b, sizeof b, "rows/chunk=%d(+%d) pitch=%d chunks=%d splits=%d grid=%d lds=%dB", p.TRK, p.KH - 1, p.pitch, p.n_chunks,
           p.n_splits, p.G * p.n_oblk * p.n_cblk * p.n_splits, p.lds_bytes);
  return b;
}

namespace {
// Launch of one instantiation; the opt-in to more than 64 KB of dynamic LDS is made once per instantiation.
template <typename K, typename T>
void launch_dw_kernel(K kernel, int grid, const DwParams& p, const T* G, const T* X, float* dst, hipStream_t stream,
                      int threads = 256) {
  static const hipError_t lds_opt_in =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (lds_opt_in != hipSuccess) return;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), p.lds_bytes, stream, p, G, X, dst);
}
}  // namespace

// A = G (upstream gradient), B = X, out = dW (fp32), ws = n_splits partial copies of dW.
syno_status launch_mfma_dw(const syno_plan* plan, const void* A, const void* B, void* out, void* ws, hipStream_t stream) {
  if (!plan->launch[SYNO_BWD_WEIGHT].params_ready) return SYNO_ERR_UNSUPPORTED;
  DwParams p;
  memcpy(&p, plan->launch[SYNO_BWD_WEIGHT].params, sizeof p);
  if (!ws && p.n_splits > 1) return SYNO_ERR_WORKSPACE;
  const int grid = p.G * p.n_oblk * p.n_cblk * p.n_splits;
  float* const dst = p.n_splits == 1 ? static_cast<float*>(out) : static_cast<float*>(ws);
  using std::integral_constant;
  auto by_window = [&](auto go) {
    if (p.KH == 2) go(integral_constant<int, 2>{}, integral_constant<int, 2>{}, integral_constant<int, 2>{});
    else if (p.KH == 3 && p.KW == 3) go(integral_constant<int, 3>{}, integral_constant<int, 3>{}, integral_constant<int, 1>{});
    else if (p.KH == 5) go(integral_constant<int, 5>{}, integral_constant<int, 1>{}, integral_constant<int, 1>{});
    else if (p.KW == 5) go(integral_constant<int, 1>{}, integral_constant<int, 5>{}, integral_constant<int, 1>{});
    else if (p.KH == 3) go(integral_constant<int, 3>{}, integral_constant<int, 1>{}, integral_constant<int, 2>{});
    else if (p.KW == 3) go(integral_constant<int, 1>{}, integral_constant<int, 3>{}, integral_constant<int, 2>{});
    else go(integral_constant<int, 1>{}, integral_constant<int, 1>{}, integral_constant<int, 2>{});
  };
  if (plan->in_dtype == SYNO_F32) {
    const float* Gf = static_cast<const float*>(A);
    const float* Xf = static_cast<const float*>(B);
    by_window([&](auto kh_c, auto kw_c, auto ct_c) {
      constexpr int kh = decltype(kh_c)::value, kw = decltype(kw_c)::value, ct = decltype(ct_c)::value;
      if (p.parts) {
        if constexpr (kh <= 3 && kw <= 3) {
          if (p.W % 8 == 0) launch_dw_kernel(dw_split<kh, kw, ct, 4, true>, grid, p, Gf, Xf, dst, stream, 512);
          else if (p.W % 4 == 0) launch_dw_kernel(dw_split<kh, kw, ct, 4, false>, grid, p, Gf, Xf, dst, stream, 512);
          else if (p.W % 2 == 0) launch_dw_kernel(dw_split<kh, kw, ct, 2, false>, grid, p, Gf, Xf, dst, stream, 512);
          else launch_dw_kernel(dw_split<kh, kw, ct, 1, false>, grid, p, Gf, Xf, dst, stream, 512);
        }
      } else if constexpr (kh == 2) {            // (no kernel on the fp32 instructions)
      } else if (kh == 3 && p.direct) {
        if constexpr (kh == 3) {
        if (p.mode == 4) launch_dw_kernel(dw_rows_f32<kw, ct, 4>, grid, p, Gf, Xf, dst, stream, kRowsThreads);
        else if (p.mode == 7) launch_dw_kernel(dw_rows_f32<kw, ct, 7>, grid, p, Gf, Xf, dst, stream, kRowsThreads);
        else if (p.mode == 14) launch_dw_kernel(dw_rows_f32<kw, ct, 14>, grid, p, Gf, Xf, dst, stream, kRowsThreads);
        else if (p.mode == 2) launch_dw_kernel(dw_rows_f32<kw, ct, 2>, grid, p, Gf, Xf, dst, stream, kRowsThreads);
        else launch_dw_kernel(dw_rows_f32<kw, ct, 1>, grid, p, Gf, Xf, dst, stream, kRowsThreads);
        }
      } else {
        if (p.W % 4 == 0) launch_dw_kernel(dw_mfma_f32<kh, kw, ct, 4>, grid, p, Gf, Xf, dst, stream);
        else if (p.W % 2 == 0) launch_dw_kernel(dw_mfma_f32<kh, kw, ct, 2>, grid, p, Gf, Xf, dst, stream);
        else launch_dw_kernel(dw_mfma_f32<kh, kw, ct, 1>, grid, p, Gf, Xf, dst, stream);
      }
    });
  } else {
    const uint16_t* G = static_cast<const uint16_t*>(A);
    const uint16_t* X = static_cast<const uint16_t*>(B);
    by_window([&](auto kh_c, auto kw_c, auto) {
      constexpr int kh = decltype(kh_c)::value, kw = decltype(kw_c)::value;
      if (p.direct) {
        if constexpr (kh == 3) launch_dw_kernel(dw_rows_bf16<kw, kw == 1 ? 2 : 1>, grid, p, G, X, dst, stream, kRowsThreads);
      } else if constexpr (kw <= 3) {          // (5-wide rows: mfma_dw_supports refuses them)
        auto stream_kernel = [&](auto wide_c) {
          constexpr StreamTile t = stream_tile(kh * kw, decltype(wide_c)::value);
          if (p.W % 8 == 0) launch_dw_kernel(dw_stream_bf16<kh, kw, t.no, t.nc, t.wc, true>, grid, p, G, X, dst, stream, 512);
          else launch_dw_kernel(dw_stream_bf16<kh, kw, t.no, t.nc, t.wc, false>, grid, p, G, X, dst, stream, 512);
        };
        if constexpr (kh * kw == 3) {
          constexpr StreamTile t = stream_tile(3, false);
          if (p.narrow) {
            if constexpr (kw == 3) launch_dw_kernel(dw_stream_bf16<1, 3, t.no, t.nc, t.wc, false, true>, grid, p, G, X, dst, stream, 512);
          } else if (p.tile_c == 64) {
            stream_kernel(std::true_type{});
          } else {
            stream_kernel(std::false_type{});
          }
        } else {
          stream_kernel(std::false_type{});
        }
      }
    });
  }
  // many splits of a small dW: one block per slot keeps the device busy; few splits, or a dW with at least one 16x16
  // tile per compute unit: one block per tile with all its taps writes dW in whole lines
  if (p.n_splits == 1) {
    // (written by the contraction itself)
  } else if (p.n_splits > 4 && p.n_tiles * (p.slots / (p.KH * p.KW)) < 256)
  {
    const int blocks = p.n_tiles * p.slots;
    const float4* const parts = reinterpret_cast<const float4*>(ws);
    if (p.n_splits >= 72 && blocks <= 256) hipLaunchKernelGGL(dw_reduce_slots<16>, dim3(blocks), dim3(1024), 0, stream, p, parts, static_cast<float*>(out));
    else hipLaunchKernelGGL(dw_reduce_slots<4>, dim3(blocks), dim3(256), 0, stream, p, parts, static_cast<float*>(out));
  }
  else
    hipLaunchKernelGGL(dw_reduce_tiles, dim3(p.n_tiles * (p.slots / (p.KH * p.KW))), dim3(256), 0, stream, p,
                       reinterpret_cast<const float4*>(ws), static_cast<float*>(out));
  return hipGetLastError() == hipSuccess ? SYNO_OK : SYNO_ERR_HIP;
}

}  // namespace syno
