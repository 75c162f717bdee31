// Backward-weight of bf16 convolutions.  Included by kernels_mfma_dw.hip, which owns the parameter record and the kernels
// that add the splits up.
//
// The reduction axis is a stream of pixels: all rows of all images one after the other, each row `pitch` pixels (the width
// rounded up to a multiple of 8) and, for windows with a row extent, KH / 2 rows of zeros after each image, which are the
// window's padding below that image and above the next one.  A tap along h is a shift of X by whole rows of the stream.  A tap
// along w is a shift of G by one pixel the other way, cut out of an aligned 16-byte read and one element of its neighbour
// (which counts as zero across a row's ends): G's shifted fragments serve every row of the window and every input channel.
//  - A workgroup (8 waves) owns 16*NO output x 16*NC*WC input channels and a range of chunks of 256 pixels; the waves of one
//    column of input channels share a chunk's k-steps of 32 pixels among themselves (8 / WC of them, whose sums meet in LDS at the
//    end).  Small tiles of sums, because every workgroup's go to memory and back where a reduction is split: with 64 x 32
//    channels per workgroup the splits of a 3x3 window were 19 MB, with 32 x 32 9.4 MB.
//  - Two LDS buffers; X's hold the chunk with the rows its window reaches (staged again with the next chunk: a ring saved those
//    loads and cost more in address arithmetic).  Channels are 2 (mod 4) 16-byte units apart, so that the fragment reads
//    are free of bank conflicts.
//  - One barrier per chunk; the next chunk is written to LDS out of registers, and the requests for the one after it follow: by
//    half of the waves before their products, by the other half after theirs, so that a SIMD's two waves take turns.
//  - Bound: a wave has 36 matrix instructions (576 cycles, 3x3) per chunk and a vector instruction occupies its SIMD for 4, so
//    what is neither has to stay below about 150 of those: positions are kept by addition.  A load instruction of a wave occupies the
//    compute unit's address path for 16 cycles, whatever it moves, so an item of 8 pixels is one 16-byte load at element
//    alignment, whose pixels beyond the row's end are masked (in aligned loads of 2 pixels the 14-pixel rows of the grouped
//    shift-unfold operator took 24.6 us instead of 16.4).
//  - Measured (us with the kernel that adds the splits up; the kernels before staged chunks of rows through a table, every load
//    waited for): 128 channels 3x3 28x28 batch 32 35 -> 28, 27x136x140 57x56 144 -> 65, grouped shift-unfold 256 channels 14x14
//    batch 128 22.8 -> 17.9, 38x24x320 38x38 61 -> 30, 1x1 23x256x24 49x26 23 -> 15; 7x8x64 13x13 1x1, six workgroups, 12.9 -> 14.8.
//    A chunk takes 1.7 us, of which the matrix instructions 0.5: vector and load issue of the staging, barriers.
#pragma once

constexpr int kBfChunk = 256, kBfUnits = kBfChunk / 8;     // pixels, 16-byte units
// LDS: bytes of a G channel (with a unit of the neighbouring pixels on either side for taps along w), of an X channel
constexpr int stream_units(int n) { return n + ((2 - n) & 3); }      // the next that is 2 (mod 4)
constexpr int stream_g_pitch(int KW) { return stream_units(kBfUnits + (KW > 1 ? 2 : 0)) * 16; }
constexpr int stream_x_pitch(int KH, int pitch) { return stream_units(kBfUnits + KH / 2 * 2 * (pitch / 8)) * 16; }

// FULL: the width is a multiple of 8 (items exist whole or not at all, and are 16-byte aligned)
template <int KH, int KW, int NO, int NC, int WC, bool FULL>
__global__ __launch_bounds__(512) void dw_stream_bf16(const DwParams p, const uint16_t* __restrict__ Gt, const uint16_t* __restrict__ Xt,
                                                      float* __restrict__ dst) {
  constexpr int T = KH * KW, KP = 8 / WC, CT = NC * WC, GO = 16 * NO, CX = 16 * CT, KS = kBfChunk / 32 / KP;
  constexpr int GP = stream_g_pitch(KW), HALO = KW > 1 ? 1 : 0;
  constexpr int XL = KH > 1 ? 64 : 32, XK = CX * XL / 512;      // lanes along an X channel's units, channels per thread
  extern __shared__ __align__(16) unsigned char smem[];
  const int x_pitch = p.CPp, x_buf = CX * x_pitch;              // bytes
  unsigned char* const xl = smem + 2 * GO * GP;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wc = wave % WC, kp = wave / WC;
  // each XCD takes a run of (split, tile) pairs: the tiles of one split read the same pixels
  const int all = p.n_tiles * p.n_splits, per = all / 8, more = all % 8, xcd = blockIdx.x % 8;
  const int id = xcd * per + min(xcd, more) + blockIdx.x / 8, split = id / p.n_tiles, tile = id - split * p.n_tiles;
  const int cb = tile % p.n_cblk, ob = tile / p.n_cblk % p.n_oblk, g = tile / (p.n_cblk * p.n_oblk);
  const int chunk_begin = split * p.chunks_per_split, chunk_end = min(p.n_chunks, chunk_begin + p.chunks_per_split);
  const int B = KH / 2 * p.pitch;               // pixels of X that the window reaches on either side

  // Where an item lies in the stream: its column, row within the image, image; chunks advance it by addition
  const int rows = p.H + KH / 2;                // of an image in the stream
  struct Place { int col, r, n; };
  auto place = [&](int s) {
    const int back = s < 0 ? 1 : 0;              // (what lies before the stream counts as the image before the first)
    s += back * p.pitch * rows;
    const int row = (int)(p.m_pitch ? __umulhi((uint32_t)s, p.m_pitch) : (uint32_t)s / (uint32_t)p.pitch);
    const int n = (int)(p.m_rows ? __umulhi((uint32_t)row, p.m_rows) : (uint32_t)row / (uint32_t)rows);
    return Place{s - row * p.pitch, row - n * rows, n - back};
  };
  const int d_rows = kBfChunk / p.pitch, d_col = kBfChunk - d_rows * p.pitch, d_n = d_rows / rows, d_r = d_rows - d_n * rows;
  auto advance = [&](Place& q) {
    q.col += d_col; q.r += d_r; q.n += d_n;
    if (q.col >= p.pitch) { q.col -= p.pitch; ++q.r; }
    if (q.r >= rows) { q.r -= rows; ++q.n; }
  };
  // pixels that exist from q on, at most 8, and the byte offset there in its channel (cyclic rows: X's is `shift` further)
  auto left_of = [&](const Place& q) { return q.r < p.H && (unsigned)q.n < (unsigned)p.n_images ? max(0, min(8, p.W - q.col)) : 0; };
  auto offset_of = [&](const Place& q, int image_stride, int shift) {
    int r = q.r + shift;
    if (KH == 1) r = r >= p.H ? r - p.H : r;
    return ((uint32_t)q.n * (uint32_t)image_stride + (uint32_t)(r * p.W + q.col)) * 2u;
  };
  const int shift = KH == 1 && p.h_wrap ? (p.h_shift + p.h_shift_g * g) % p.H : 0;

  // 8 pixels of a channel from byte `at` of a tensor on.  Rows end anywhere, so the last item of a tensor may reach past it:
  // it is read from `last`, the last place with 8 elements, and laid out element by element afterwards (`mend`).
  typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
  auto request = [&](const uint16_t* tensor, uint32_t at, int left, uint32_t last) {
    at = left > 0 ? at : 0u;
    if constexpr (FULL) return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(tensor) + at);
    const u32x4_any v = *reinterpret_cast<const u32x4_any*>(reinterpret_cast<const char*>(tensor) + min(at, last));
    return make_uint4(v[0], v[1], v[2], v[3]);
  };
  auto keep = [&](const uint4& v, int left) {
    auto mask = [&](int e) { return FULL ? (left > 0 ? ~0u : 0u) : left >= e + 2 ? ~0u : left == e + 1 ? 0xffffu : 0u; };
    return make_uint4(v.x & mask(0), v.y & mask(2), v.z & mask(4), v.w & mask(6));
  };
  auto mend = [&](unsigned char* put, const uint16_t* tensor, uint32_t at, int left, uint32_t last) {
    if (left <= 0 || at <= last) return;
#pragma clang loop vectorize(disable) unroll(disable)
    for (int e = 0; e < left; ++e) reinterpret_cast<uint16_t*>(put)[e] = tensor[at / 2 + e];
  };

  // this thread's items of a chunk (channels beyond the tensor's read the last one: their sums are never stored): of G, unit
  // tid % 32 of channels tid / 32 + 16 k, and for the first threads one of the neighbouring units; of X, unit tid % XL of
  // channels tid / XL + 512 / XL * k
  const uint32_t g_last = p.g_last, x_last = p.x_last;
  const int o_first = g * p.Og + ob * GO, c_first = g * p.Cg + cb * CX, o_last = p.Og - ob * GO - 1, c_last = p.Cg - cb * CX - 1;
  const int g_unit = tid & (kBfUnits - 1), g_ch0 = tid / kBfUnits, x_unit = tid & (XL - 1), x_ch0 = tid / XL;
  const bool x_mine = x_unit * 8 < kBfChunk + 2 * B, h_mine = HALO && tid < 2 * GO;
  uint32_t g_ch[NO], x_ch[XK];
#pragma unroll
  for (int k = 0; k < NO; ++k) g_ch[k] = (uint32_t)(o_first + min(g_ch0 + 16 * k, o_last)) * (uint32_t)p.plane * 2u;
#pragma unroll
  for (int k = 0; k < XK; ++k) x_ch[k] = (uint32_t)(c_first + min(x_ch0 + 512 / XL * k, c_last)) * (uint32_t)p.plane * 2u;
  const uint32_t h_ch = (uint32_t)(o_first + min(tid >> 1, o_last)) * (uint32_t)p.plane * 2u;
  const int first_px = chunk_begin * kBfChunk;
  Place g_at = place(first_px + g_unit * 8), x_at = place(first_px - B + x_unit * 8), h_at = place(first_px + (tid & 1 ? kBfChunk : -8));
  struct Items { uint4 g[NO], h, x[XK]; int gl, hl, xl; uint32_t go, ho, xo; };
  auto fetch = [&](Items& s) {
    s.gl = left_of(g_at);
    s.go = offset_of(g_at, p.gs_n, 0);
    s.xl = x_mine ? left_of(x_at) : 0;
    s.xo = offset_of(x_at, p.xs_n, shift);
#pragma unroll
    for (int k = 0; k < NO; ++k) s.g[k] = request(Gt, g_ch[k] + s.go, s.gl, g_last);
#pragma unroll
    for (int k = 0; k < XK; ++k) s.x[k] = request(Xt, x_ch[k] + s.xo, s.xl, x_last);
    advance(g_at);
    advance(x_at);
    if constexpr (HALO) {
      s.hl = h_mine ? left_of(h_at) : 0;
      s.ho = offset_of(h_at, p.gs_n, 0);
      s.h = request(Gt, h_ch + s.ho, s.hl, g_last);
      advance(h_at);
    }
  };
  unsigned char* const g_put = smem + g_ch0 * GP + (g_unit + HALO) * 16;
  unsigned char* const h_put = smem + (tid >> 1) * GP + (tid & 1 ? kBfUnits + 1 : 0) * 16;
  unsigned char* const x_put = xl + x_ch0 * x_pitch + x_unit * 16;
  // chunk: of the items (only the last image's may reach past a tensor's end)
  auto lay = [&](const Items& s, int buf, int chunk) {
    auto g_to = [&](int k) { return g_put + (buf * GO + 16 * k) * GP; };
    auto x_to = [&](int k) { return x_put + buf * x_buf + 512 / XL * k * x_pitch; };
#pragma unroll
    for (int k = 0; k < NO; ++k) *reinterpret_cast<uint4*>(g_to(k)) = keep(s.g[k], s.gl);
#pragma unroll
    for (int k = 0; k < XK; ++k)
      if (KH == 1 || x_mine) *reinterpret_cast<uint4*>(x_to(k)) = keep(s.x[k], s.xl);
    if (HALO && h_mine) *reinterpret_cast<uint4*>(h_put + buf * GO * GP) = keep(s.h, s.hl);
    if (!FULL && chunk >= p.tail_chunk) {
#pragma unroll
      for (int k = 0; k < NO; ++k) mend(g_to(k), Gt, g_ch[k] + s.go, s.gl, g_last);
#pragma unroll
      for (int k = 0; k < XK; ++k) mend(x_to(k), Xt, x_ch[k] + s.xo, s.xl, x_last);
      if (HALO) mend(h_put + buf * GO * GP, Gt, h_ch + s.ho, s.hl, g_last);
    }
  };

  // (the nine taps' sums leave registers for one chunk on its way, the others' for two)
  constexpr int SETS = T == 9 ? 1 : 2;
  Items next[SETS];
  {
    Items first;
    fetch(first);
#pragma unroll
    for (int k = 0; k < SETS; ++k) fetch(next[k]);
    lay(first, 0, chunk_begin);
  }

  floatx4 acc[NO][NC][T];
#pragma unroll
  for (int a = 0; a < NO; ++a)
#pragma unroll
    for (int b = 0; b < NC; ++b)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[a][b][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  int col[KS];                                   // column of this lane's 8 pixels of k-step ks
  if constexpr (KW > 1) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) col[ks] = place(first_px + (ks * KP + kp) * 32 + (lane >> 4) * 8).col;
  }
  const unsigned char* const ga = smem + (lane & 15) * GP + (kp * 4 + (lane >> 4) + HALO) * 16;
  const unsigned char* const xa = xl + (wc * NC * 16 + (lane & 15)) * x_pitch + (kp * 4 + (lane >> 4)) * 16;

  struct GRead { uint4 cur; uint32_t prev, next; };    // 8 pixels of G and their neighbours
  auto multiply = [&](int buf) {
    const unsigned char* const gb = ga + buf * GO * GP;
    const unsigned char* const xb = xa + buf * x_buf;
    constexpr int NBLK = KS * NC * KH;
    GRead gr[NO];
    uint4 row[2];
    auto read_g = [&](auto ks_c) {
      constexpr int ks = decltype(ks_c)::value;
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        const unsigned char* at = gb + i * 16 * GP + ks * KP * 64;
        gr[i].cur = *reinterpret_cast<const uint4*>(at);
        if constexpr (KW > 1) {
          gr[i].prev = *reinterpret_cast<const uint32_t*>(at - 4);
          gr[i].next = *reinterpret_cast<const uint32_t*>(at + 16);
        }
      }
    };
    auto read_row = [&](auto b_c) {              // block b: k-step, input-channel tile, window row
      constexpr int b = decltype(b_c)::value, ks = b / (NC * KH), i = b / KH % NC, kh = b % KH;
      row[b & 1] = *reinterpret_cast<const uint4*>(xb + i * 16 * x_pitch + kh * p.pitch * 2 + ks * KP * 64);
    };
    uint4 a[KW][NO];                             // G's fragments, shifted for the taps along w
    auto shift_g = [&](auto ks_c) {
      constexpr int ks = decltype(ks_c)::value;
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        const GRead& v = gr[i];
        const uint4 c = v.cur;
        if constexpr (KW == 1) {
          a[0][i] = c;
        } else {
          // tap kw pairs X's pixel q with G's q - kw + 1
          const uint32_t prev = col[ks] == 0 ? 0u : v.prev, next = col[ks] == p.pitch - 8 ? 0u : v.next;
          a[0][i] = make_uint4(alignbit16(c.y, c.x), alignbit16(c.z, c.y), alignbit16(c.w, c.z), alignbit16(next, c.w));
          a[1][i] = c;
          if constexpr (KW == 3) a[KW - 1][i] = make_uint4(alignbit16(c.x, prev), alignbit16(c.y, c.x), alignbit16(c.z, c.y), alignbit16(c.w, c.z));
        }
      }
    };
    read_row(std::integral_constant<int, 0>{});
    for_blocks<0, NBLK>([&](auto b_c) {
      constexpr int b = decltype(b_c)::value, ks = b / (NC * KH), i = b / KH % NC, kh = b % KH;
      if constexpr (b + 1 < NBLK) {
        read_row(std::integral_constant<int, b + 1>{});
      }
      if constexpr (b % (NC * KH) == 0) { read_g(std::integral_constant<int, ks>{}); shift_g(std::integral_constant<int, ks>{}); }
      const bf16x8 x = __builtin_bit_cast(bf16x8, row[b & 1]);
#pragma unroll
      for (int kw = 0; kw < KW; ++kw)
#pragma unroll
        for (int ao = 0; ao < NO; ++ao)
          acc[ao][i][kh * KW + kw] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[kw][ao]), x, acc[ao][i][kh * KW + kw], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (KW > 1) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        col[ks] += d_col;
        if (col[ks] >= p.pitch) col[ks] -= p.pitch;
      }
    }
  };
  // The two waves of a SIMD take turns: one stages (the next chunk into LDS, then the requests for the one SETS after it) while
  // the other multiplies.  (The requests of the last rounds lie past this split's chunks: pixels of the next split, or none.)
  const bool early = wave >= 4;
  auto step = [&](int ch, Items& s) {
    const int buf = (ch - chunk_begin) & 1;
    __syncthreads();
    if (early) { lay(s, buf ^ 1, ch + 1); fetch(s); }
    __builtin_amdgcn_sched_barrier(0);
    multiply(buf);
    if (!early) { lay(s, buf ^ 1, ch + 1); fetch(s); }
  };
  int ch = chunk_begin;
  if constexpr (SETS == 2)
    for (; ch + 1 < chunk_end; ch += 2) {
      step(ch, next[0]);
      step(ch + 1, next[1]);
    }
  for (; ch < chunk_end; ++ch) step(ch, next[0]);

  // ---- the sums of the waves that shared the k-steps meet in LDS
  __syncthreads();
  floatx4* const red = reinterpret_cast<floatx4*>(smem);
  constexpr int SLOTS = NO * CT * T, MINE = NO * NC * T;
#pragma unroll
  for (int ao = 0; ao < NO; ++ao)
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int t = 0; t < T; ++t) red[(wave * MINE + (ao * NC + i) * T + t) * 64 + lane] = acc[ao][i][t];
  __syncthreads();
  // slot: (output-channel tile, input-channel tile, tap)
  auto at_slot = [&](int slot) {
    const int t = slot % T, ci = slot / T % CT, ao = slot / (T * CT);
    return (ci / NC * MINE + (ao * NC + ci % NC) * T + t) * 64;
  };
  if (p.n_splits > 1) {
    floatx4* const out = reinterpret_cast<floatx4*>(dst) + ((int64_t)split * p.n_tiles + tile) * SLOTS * 64;
    for (int i = tid; i < SLOTS * 64; i += 512) {
      const floatx4* r = red + at_slot(i >> 6) + (i & 63);
      floatx4 s = r[0];
#pragma unroll
      for (int k = 1; k < KP; ++k) s += r[k * WC * MINE * 64];
      out[i] = s;
    }
  } else {
    // whole rows of dW in (input channel, tap) order, which is contiguous for the usual layouts
    for (int i = tid; i < GO * CX * T; i += 512) {
      const int t = i % T, c = i / T % CX, o = i / (T * CX);
      if (ob * GO + o >= p.Og || cb * CX + c >= p.Cg) continue;
      const float* r = reinterpret_cast<const float*>(red + at_slot((o / 16 * CT + c / 16) * T + t) + ((o & 15) >> 2) * 16 + (c & 15)) + (o & 3);
      float s = r[0];
#pragma unroll
      for (int k = 1; k < KP; ++k) s += r[k * WC * MINE * 256];
      dst[(int64_t)g * p.ws_g + (int64_t)(ob * GO + o) * p.ws_o + (int64_t)(cb * CX + c) * p.ws_c + (t / KW) * p.ws_kh + (t % KW) * p.ws_kw] = s;
    }
  }
}
