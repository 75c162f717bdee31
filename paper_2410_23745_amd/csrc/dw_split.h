// Backward-weight of fp32 convolutions on the bf16 matrix cores (every value as three bf16 parts, fp32_parts.h).
// Included by kernels_mfma_dw.hip, which owns the parameter record and the kernels that add the splits up.
//
// The reduction axis is a stream of pixels: all rows of all images one after the other, each row `pitch` pixels (a multiple
// of 8, at least the width) and one row of zeros after each image, which is the window's padding below that image and above
// the next one.  A tap along h is a shift by whole rows of the stream; a tap along w a shift by one pixel, cut out of an
// aligned 16-byte read and one element of its neighbour, which counts as zero at a row's ends.  Every source row is so
// staged once, whatever the window.
//  - A workgroup (8 waves) owns 64 output x 32*CT input channels and a range of 64-pixel chunks.  G's chunks go through two
//    LDS buffers, X's through a ring that holds the window's rows around the chunk and the chunk staged next:
//    [channel][8 pixels][part] 16-byte units, channels 2 (mod 4) units apart, which keeps the fragment reads free of bank
//    conflicts (a kernel of such reads alone: 4.4 cycles per 1 KB, 8.1 otherwise), and the parts at constant offsets.
//  - One barrier per chunk.  A chunk is two k-steps of 32 pixels, one per half of the waves; the next chunk is written, and
//    the one after it requested, between the taps.  The halves' sums meet in LDS at the end.
//  - Bound: 96 cycles of matrix work per 16x16 tile, tap and k-step, against some 200 vector instructions per wave and
//    chunk (splitting, cutting, addresses), which have to fit beside it: positions are kept by addition, and pixels that
//    do not exist are buffer loads past the end, which give zeros.  Filling (a
//    pitch above the width, the zero rows) costs 2 % at 56x56, 18 % at 28, 22 % at 14, 31 % at 7.  Issuing the requests
//    earlier, a second set of registers for them, and interleaving the vector work with the matrix instructions by hand
//    each left the times as they are: 890 to 990 TFLOP/s of bf16 products in the kernel by itself, filling included, where a
//    large library product has 1190 (matrix units occupied 0.36 to 0.40 of the time at the nominal clock, by the counters).
//  - Measured, with the kernel that adds the splits up, against the fp32 instructions (batch 32): 64 channels at 56x56 86 ->
//    59 us, 128 at 28 89 -> 64, 256 at 14 94 -> 69, 512 at 7 89 -> 71; 1x1 64 -> 256 at 56 93 -> 49; 3x1 96 -> 64 at 56
//    85 -> 44.  Error against 64 bits 1.4e-7 to 1.7e-7 of the largest weight's gradient, before 3.3e-7 to 3.8e-7.
#pragma once

constexpr int kStreamChunk = 64;                 // pixels
constexpr int kGUnits = 26;                      // LDS distance of G's channels in 16-byte units: 8 x 3 parts, and 2 (mod 4)
constexpr uint32_t kNoPixel = 1u << 31;          // an offset beyond every tensor here: a buffer load answers it with zeros

// All taps of a 16 x 16 tile (output channels o0.., input channels c0.. of the group) over the stream's pixels begin..end-1
// with the fp32 matrix instructions, on the tensors where they lie: for tiles with sums that the parts cannot give.  A
// pixel whose tap lies outside the image counts as zero in both operands.  Lane: output channels 4 * (lane / 16) + 0..3,
// input channel lane % 16.  Each workgroup does its own pixels again, so that one infinity costs one split's share: 153 us
// at 32x64x64 56x56, 330 where all of G is NaN, 69 without.
template <int KH, int KW>
__device__ __forceinline__ void dw_plain_tile(const DwParams& p, const float* __restrict__ Gt, const float* __restrict__ Xt, int g,
                                              int o0, int c0, int begin, int end, int lane, floatx4 (&sum)[KH * KW]) {
  constexpr int NX = 4 + KW - 1;                 // the pixels of a row that the taps of four read
  const float* const gch = Gt + (int64_t)(g * p.Og + min(o0 + (lane & 15), p.Og - 1)) * p.plane;
  const float* const xch = Xt + (int64_t)(g * p.Cg + min(c0 + (lane & 15), p.Cg - 1)) * p.plane;
#pragma unroll
  for (int t = 0; t < KH * KW; ++t) sum[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = begin; s0 < end; s0 += 16) {
    const int s = s0 + 4 * (lane >> 4);          // four pixels of one row (its pitch is a multiple of 8)
    const int row = (int)__umulhi((uint32_t)s, p.m_pitch), n = (int)__umulhi((uint32_t)row, p.m_rows);
    const int h = row - n * (p.H + 1), w = s - row * p.pitch;
    const bool live = n < p.n_images && h < p.H;
    const float* const gr = gch + (live ? (int64_t)n * p.gs_n + h * p.W : 0);
    float gv[4], xv[KH][NX];
#pragma unroll
    for (int e = 0; e < 4; ++e) gv[e] = gr[live && w + e < p.W ? w + e : 0];
#pragma unroll
    for (int kh = 0; kh < KH; ++kh) {
      const int hx = h + kh - p.ph;
      const bool in = live && hx >= 0 && hx < p.H;
      const float* const xr = xch + (in ? (int64_t)n * p.xs_n + hx * p.W : 0);
#pragma unroll
      for (int e = 0; e < NX; ++e) {
        const int wx = w + e - p.pw;
        xv[kh][e] = xr[in && wx >= 0 && wx < p.W ? wx : 0];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int kh = 0; kh < KH; ++kh)
#pragma unroll
        for (int kw = 0; kw < KW; ++kw) {
          const int hx = h + kh - p.ph, wx = w + e + kw - p.pw;
          const bool in = live && w + e < p.W && hx >= 0 && hx < p.H && wx >= 0 && wx < p.W;
          sum[kh * KW + kw] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? gv[e] : 0.f, in ? xv[kh][e + kw] : 0.f, sum[kh * KW + kw], 0, 0, 0);
        }
  }
}

// VEC: pixels per load (4, 2 or 1, what the width divides by).  EDGE: rows without a zero pixel between them (widths that
// are multiples of 8), whose ends the taps must not reach across.
template <int KH, int KW, int CT, int VEC, bool EDGE>
__global__ __launch_bounds__(512) void dw_split(const DwParams p, const float* __restrict__ Gt, const float* __restrict__ Xt,
                                                float* __restrict__ partial) {
  constexpr int T = KH * KW, CX = 32 * CT, NT = 512;
  constexpr int XE = CT == 1 ? 4 : 8;            // pixels of an X item: CX * 64 / XE = 512 items per chunk, as of G's 8-pixel ones
  constexpr int GBYTES = 64 * kGUnits * 16, UNIT = kPlanes * 16;      // UNIT: bytes of 8 pixels
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* const xl = smem + 2 * GBYTES;
  const int x_row = p.CPp / 8 * UNIT;            // bytes of an X channel

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int widx = wave & 3, half = wave >> 2, wo = widx >> 1, wc = widx & 1;
  int bid = blockIdx.x;
  const int split = bid % p.n_splits; bid /= p.n_splits;
  const int cb = bid % p.n_cblk; bid /= p.n_cblk;
  const int ob = bid % p.n_oblk;
  const int g = bid / p.n_oblk;
  const int chunk_begin = split * p.chunks_per_split;
  const int chunk_end = min(p.n_chunks, chunk_begin + p.chunks_per_split);
  const int B = p.stream_reach;                  // pixels of X that a chunk reads on either side of its own (a multiple of 8)

  // channels beyond the tensor's read the last one (their sums are never stored)
  const auto gbase = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Gt + (int64_t)(g * p.Og + ob * 64) * p.plane), 0, (int)kNoPixel, 0x00020000);
  const auto xbase = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Xt + (int64_t)(g * p.Cg + cb * CX) * p.plane), 0, (int)kNoPixel, 0x00020000);
  const int o_last = p.Og - ob * 64 - 1, c_last = p.Cg - cb * CX - 1;

  // A stream position: its column, its row within the image (H: the row of zeros), the image, and the byte offset there
  struct Place { int col, r, n; uint32_t at; };
  auto place = [&](int s, uint32_t channel, int image_stride) {
    const int row = s >= 0 ? (int)__umulhi((uint32_t)s, p.m_pitch) : 0, n = (int)__umulhi((uint32_t)row, p.m_rows), r = row - n * (p.H + 1);
    const int col = s - row * p.pitch;
    return Place{col, s >= 0 ? r : p.H, n, channel + (uint32_t)(n * image_stride + r * p.W + col) * 4u};
  };
  const int d_row = kStreamChunk / p.pitch, d_col = kStreamChunk - d_row * p.pitch;
  auto next_chunk = [&](Place& q, int image_stride) {
    q.col += d_col; q.r += d_row; q.at += (uint32_t)(d_row * p.W + d_col) * 4u;
    if (q.col >= p.pitch) { q.col -= p.pitch; ++q.r; q.at += (uint32_t)(p.W - p.pitch) * 4u; }
    while (q.r > p.H) { q.r -= p.H + 1; ++q.n; q.at += (uint32_t)(image_stride - (p.H + 1) * p.W) * 4u; }
  };
  // requests n pixels of one channel
  auto request = [&](__amdgpu_buffer_rsrc_t base, const Place& q, auto& v) {
    constexpr int N = sizeof(v) / 4;
    const int left = q.r < p.H && q.n < p.n_images ? p.W - q.col : 0;
#pragma unroll
    for (int e = 0; e < N / VEC; ++e) {
      const int at = left > e * VEC ? (int)q.at + e * VEC * 4 : (int)kNoPixel;
      if constexpr (VEC == 4) {
        const auto t = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(base, at, 0, 0));
        v[4 * e] = t[0]; v[4 * e + 1] = t[1]; v[4 * e + 2] = t[2]; v[4 * e + 3] = t[3];
      } else if constexpr (VEC == 2) {
        const auto t = __builtin_bit_cast(f32x2_any, __builtin_amdgcn_raw_buffer_load_b64(base, at, 0, 0));
        v[2 * e] = t[0]; v[2 * e + 1] = t[1];
      } else {
        v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(base, at, 0, 0));
      }
    }
  };
  // splits n pixels and lays their parts out
  auto lay = [&](unsigned char* dst, const auto& v) {
    constexpr int N = sizeof(v) / 4;
    uint32_t h[N / 2], m[N / 2], l[N / 2];
#pragma unroll
    for (int j = 0; j < N / 2; ++j) split_pair(v[2 * j], v[2 * j + 1], h[j], m[j], l[j]);
    auto put = [&](unsigned char* d, const uint32_t (&w)[N / 2]) {
      if constexpr (N == 8) *reinterpret_cast<uint4*>(d) = make_uint4(w[0], w[1], w[2], w[3]);
      else *reinterpret_cast<uint2*>(d) = make_uint2(w[0], w[1]);
    };
    put(dst, h);
    put(dst + 16, m);
    put(dst + 32, l);
  };
  auto bytes_of = [&](int px) { return (px >> 3) * UNIT + (px & 7) * 2; };      // of a pixel's first part within its channel

  // this thread's items of a chunk
  const int g_ch = tid >> 3, g_px = (tid & 7) * 8, x_ch = tid / (64 / XE), x_px = (tid & (64 / XE - 1)) * XE;
  unsigned char* const g_put = smem + g_ch * kGUnits * 16 + bytes_of(g_px);
  Place g_at = place(chunk_begin * kStreamChunk + g_px, (uint32_t)min(g_ch, o_last) * (uint32_t)p.plane * 4u, p.gs_n);
  Place x_at = place(chunk_begin * kStreamChunk + B + x_px, (uint32_t)min(x_ch, c_last) * (uint32_t)p.plane * 4u, p.xs_n);
  float gr[8], xr[XE];
  // the next chunk of G, and the pixels of X that its window reaches beyond the one before
  auto fetch = [&]() {
    next_chunk(g_at, p.gs_n);
    next_chunk(x_at, p.xs_n);
    request(gbase, g_at, gr);
    request(xbase, x_at, xr);
  };
  // ring position of a chunk's first pixel; positions are kept by addition
  const int ring = p.stream_ring;
  auto wrap = [&](int pos) { return pos >= ring ? pos - ring : pos; };

  // ---- the first chunk's G and its whole window of X: all of a round's requests before anything is waited for (one by one
  // they cost a memory round trip each, 4 at 56x56)
  int base = 0;                        // ring position of the current chunk's first pixel
  {
    // items of X on their way at a time (a wave's 64 exist or do not: their number is a multiple of 64).  Odd widths, whose items are
    // single loads: one with G's, and the windows' others after it (whole calls of 3x3 windows 1 / 1.01 of the time with three, 1x1 the same)
    constexpr int IN = VEC == 1 && T > 1 ? 1 : 3;
    const int groups = (kStreamChunk + 2 * B) / XE, all = CX * groups;
    request(gbase, g_at, gr);
    for (int i0 = tid; i0 < all; i0 += IN * NT) {
      float v[IN][XE];
      int put[IN];
#pragma unroll
      for (int e = 0; e < IN; ++e) {
        const int i = i0 + e * NT;
        if (i >= all) break;
        const int ch = (int)__umulhi((uint32_t)i, p.m_groups), q = i - ch * groups, pos = q * XE - B;
        put[e] = ch * x_row + bytes_of(pos < 0 ? pos + ring : pos);
        request(xbase, place(chunk_begin * kStreamChunk + pos, (uint32_t)min(ch, c_last) * (uint32_t)p.plane * 4u, p.xs_n), v[e]);
      }
      if (i0 == tid) lay(g_put, gr);
#pragma unroll
      for (int e = 0; e < IN; ++e)
        if (i0 + e * NT < all) lay(xl + put[e], v[e]);
    }
    fetch();
  }
  int col = ((chunk_begin * kStreamChunk + half * 32 + (lane >> 4) * 8) % p.pitch);   // column of this lane's 8 pixels
  const int col_step = kStreamChunk % p.pitch;

  floatx4 acc[2][CT][T];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[a][b][t] = floatx4{0.f, 0.f, 0.f, 0.f};

  struct Row { uint4 cur[kPlanes]; uint32_t prev[kPlanes], next[kPlanes]; };    // 8 pixels of X and their neighbours
  const int ring_bytes = ring / 8 * UNIT;
  auto around = [&](int at) { return at >= ring_bytes ? at - ring_bytes : at < 0 ? at + ring_bytes : at; };
  for (int ch = chunk_begin; ch < chunk_end; ++ch) {
    __syncthreads();
    const int buf = (ch - chunk_begin) & 1;
    const unsigned char* const ga = smem + buf * GBYTES + ((2 * wo) * 16 + (lane & 15)) * kGUnits * 16 + (half * 4 + (lane >> 4)) * UNIT;
    const unsigned char* const xa = xl + (CT * wc * 16 + (lane & 15)) * x_row;
    const int here = around((base / 8 + half * 4 + (lane >> 4)) * UNIT), up = p.pitch / 8 * UNIT;
    uint4 a[2][kPlanes];
    Row row[2];
    auto read_row = [&](auto b_c, Row& d) {          // block b: input-channel tile b / KH, window row b % KH
      constexpr int b = decltype(b_c)::value, i = b / KH, kh = b % KH;
      const int pos = KH == 1 || kh == 1 ? here : around(here + (kh - 1) * up);
      const unsigned char* const r = xa + i * 16 * x_row;
      const unsigned char *const at = r + pos, *const left = r + around(pos - UNIT), *const right = r + around(pos + UNIT);
#pragma unroll
      for (int s = 0; s < kPlanes; ++s) {
        d.cur[s] = *reinterpret_cast<const uint4*>(at + s * 16);
        if constexpr (KW > 1) {
          d.prev[s] = *reinterpret_cast<const uint32_t*>(left + s * 16 + 12);
          d.next[s] = *reinterpret_cast<const uint32_t*>(right + s * 16);
        }
      }
    };
    const bool first_col = EDGE && col == 0, last_col = EDGE && col == p.pitch - 8;
    // staging work between the taps: the next chunk into LDS, then the requests for the one after it
    auto piece = [&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      if constexpr (i == 0) lay(g_put + (buf ^ 1) * GBYTES, gr);
      else if constexpr (i == 1) lay(xl + x_ch * x_row + bytes_of(wrap(wrap(base + kStreamChunk + B) + x_px)), xr);
      else fetch();
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int NBLK = CT * KH, P = 3;
#pragma unroll
    for (int ao = 0; ao < 2; ++ao)
#pragma unroll
      for (int s = 0; s < kPlanes; ++s) a[ao][s] = *reinterpret_cast<const uint4*>(ga + ao * 16 * kGUnits * 16 + s * 16);
    read_row(std::integral_constant<int, 0>{}, row[0]);
    for_blocks<0, NBLK>([&](auto b_c) {
      constexpr int b = decltype(b_c)::value, i = b / KH, kh = b % KH;
      if constexpr (b + 1 < NBLK) read_row(std::integral_constant<int, b + 1>{}, row[(b + 1) & 1]);
      const Row& x = row[b & 1];
      for_blocks<0, KW>([&](auto kw_c) {
        constexpr int kw = decltype(kw_c)::value, t = kh * KW + kw;
        uint4 f[kPlanes];
#pragma unroll
        for (int s = 0; s < kPlanes; ++s) {
          const uint4 c = x.cur[s];
          if constexpr (KW == 1 || kw == 1) f[s] = c;
          else if constexpr (kw == 0) f[s] = make_uint4(alignbit16(c.x, first_col ? 0u : x.prev[s]), alignbit16(c.y, c.x), alignbit16(c.z, c.y), alignbit16(c.w, c.z));
          else f[s] = make_uint4(alignbit16(c.y, c.x), alignbit16(c.z, c.y), alignbit16(c.w, c.z), alignbit16(last_col ? 0u : x.next[s], c.w));
        }
        // the small products are summed by themselves, so that a k-step rounds the large sum twice and not six times
        constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
        floatx4 small[2] = {};
#pragma unroll
        for (int s = 0; s < 5; ++s)
#pragma unroll
          for (int ao = 0; ao < 2; ++ao)
            small[ao] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[ao][pa[s]]), __builtin_bit_cast(bf16x8, f[pb[s]]), small[ao], 0, 0, 0);
#pragma unroll
        for (int ao = 0; ao < 2; ++ao)
          acc[ao][i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[ao][0]), __builtin_bit_cast(bf16x8, f[0]), acc[ao][i][t], 0, 0, 0) + small[ao];
        __builtin_amdgcn_sched_barrier(0);
        constexpr int done = i * T + t, all = CT * T;
        for_blocks<done * P / all, (done + 1) * P / all>(piece);
      });
    });
    base = wrap(base + kStreamChunk);
    col += col_step;
    if (col >= p.pitch) col -= p.pitch;
  }

  // ---- the halves' sums meet in LDS
  __syncthreads();
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
  uint32_t odd = 0;                              // tiles of this wave with a sum that the parts cannot give
#pragma unroll
  for (int ao = 0; ao < 2; ++ao)
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      bool any = false;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const floatx4 v = (acc[ao][i][t] + red[((ao * CT + i) * T + t) * 64]) * kResultScale;
        acc[ao][i][t] = v;
        any |= !trusted_result(fabsf(v[0]) + fabsf(v[1]) + fabsf(v[2]) + fabsf(v[3]));
      }
      odd |= (uint32_t)(__any(any) != 0) << (ao * CT + i);
    }
  dw_finish<KH, KW, CT>(p, partial, g, ob, cb, split, widx, lane, acc);
  // (see split_pair)
  while (odd) {
    const int q = __builtin_ctz(odd), i = q % CT, ao = q / CT;
    odd &= odd - 1;
    const int o0 = ob * 64 + (2 * wo + ao) * 16, c0 = cb * CX + (CT * wc + i) * 16;
    const int o = o0 + 4 * (lane >> 4), c = c0 + (lane & 15);
    if (o0 >= p.Og || c0 >= p.Cg) continue;
    floatx4 v[T];
    dw_plain_tile<KH, KW>(p, Gt, Xt, g, o0, c0, chunk_begin * kStreamChunk, chunk_end * kStreamChunk, lane, v);
    const int tile = (g * p.n_oblk + ob) * p.n_cblk + cb;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      // its place, as dw_finish has it
      float* at = partial + (int64_t)g * p.ws_g + (int64_t)o * p.ws_o + (int64_t)c * p.ws_c + (t / KW) * p.ws_kh + (t % KW) * p.ws_kw;
      if (p.n_splits > 1) at = partial + ((((int64_t)split * p.n_tiles + tile) * (8 * CT * T) + (widx * 2 * CT + q) * T + t) * 64 + lane) * 4;
      const int64_t step = p.n_splits > 1 ? 1 : p.ws_o;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (o + j < p.Og && c < p.Cg && !trusted_result(at[j * step])) at[j * step] = v[t][j];
    }
  }
}
