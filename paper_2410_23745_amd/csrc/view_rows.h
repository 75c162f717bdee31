// Pure views whose rows are rows of X: the innermost axis walks X's elements one by one (from any place on, cyclically where a
// Shift wraps it), the weight does not depend on it, and every other axis adds a multiple of its index to either offset -
// scales per channel, cyclic shifts along rows, transposed or repeated outer axes.  Included by kernels_view.hip.
//
// A workgroup takes passes of R rows: a thread per row works out the offsets and reads the weight, one pass ahead, and all
// threads move the rows of this one, four pieces each, all loads on their way before the first store.  Pieces are 4 elements
// where the rows divide into them - 16-byte loads at element alignment (a piece that the wrap cuts takes a second one) -
// else single ones, adjacent lanes on adjacent elements.
//  - Bound: memory.  The general kernel's chain of table reads, exchanged offsets and four scalar loads and stores a run took
//    49 us at 64x128x56x56 fp32 (205 MB), this one 42; rows whose length is no multiple of 4 went element by element:
//    2x433x56x50 24 us -> 6, 2x423x45x29 17 -> 5.  Weight gradients 64x128x56x56 63 -> 44, 5x321x35x34 27 -> 8.
#pragma once

struct ViewRows {
  int32_t n_outer, L, k, rows, R;            // L: row length; element c of a row is X's (c + k) mod L of it
  int32_t bx, bw;                            // constant parts of the offsets
  int32_t size[kMaxAxes], sx[kMaxAxes], sw[kMaxAxes];
  uint32_t magic[kMaxAxes], m_l;             // division_magic of the sizes and of a row's pieces
};

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t u16x4_any __attribute__((ext_vector_type(4), aligned(2)));

// four adjacent elements at any element
template <bool BF>
__device__ __forceinline__ void load_any(const void* base, int off, float (&v)[4]) {
  if constexpr (BF) {
    const u16x4_any t = *reinterpret_cast<const u16x4_any*>(static_cast<const uint16_t*>(base) + off);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __uint_as_float((uint32_t)t[i] << 16);
  } else {
    const f32x4_any t = *reinterpret_cast<const f32x4_any*>(static_cast<const float*>(base) + off);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = t[i];
  }
}

// V elements from s on of the row of L elements at `row`, cyclically
template <int V, bool BF>
__device__ __forceinline__ void load_cyclic(const void* base, int row, int s, int L, float (&v)[V]) {
  if constexpr (V == 1) {
    v[0] = load_one<BF>(base, row + s);
  } else {
    const int over = s - (L - 4);            // elements past the row's end
    load_any<BF>(base, row + min(s, L - 4), v);
    if (over > 0) {
      float b[4];
      load_any<BF>(base, row, b);
      const float a[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = over == 1 ? (i < 3 ? a[i < 3 ? i + 1 : 3] : b[0]) : over == 2 ? (i < 2 ? a[i + 2 > 3 ? 3 : i + 2] : b[i < 2 ? 0 : i - 2]) : (i < 1 ? a[3] : b[i < 1 ? 0 : i - 1]);
      }
    }
  }
}

// the forward pass, or (SCATTER) the way back from the result to X: dst[x(o)] = src[o] * W[w(o)]
template <bool IBF, bool OBF, bool SCATTER, int V>
__global__ __launch_bounds__(kThreads) void view_rows(const ViewRows p, const void* __restrict__ src, const void* __restrict__ Wt,
                                                      void* __restrict__ dst) {
  __shared__ int x_of[2][kThreads];
  __shared__ float w_of[2][kThreads];
  const int tid = threadIdx.x, pieces = p.L / V, k = SCATTER && p.k ? p.L - p.k : p.k;
  auto decode = [&](int row0, int buf) {
    if (tid >= p.R || row0 + tid >= p.rows) return;
    uint32_t rest = (uint32_t)(row0 + tid);
    int x = p.bx, w = p.bw;
    for (int j = p.n_outer - 1; j >= 0; --j) {
      const uint32_t q = div_magic(rest, (uint32_t)p.size[j], p.magic[j]);
      const int d = (int)(rest - q * (uint32_t)p.size[j]);
      rest = q;
      x += d * p.sx[j];
      w += d * p.sw[j];
    }
    x_of[buf][tid] = x;
    w_of[buf][tid] = load_one<IBF>(Wt, w);
  };
  const int step = gridDim.x * p.R;          // (the host keeps rows + step below 2^31)
  int buf = 0;
  decode(blockIdx.x * p.R, 0);
  __syncthreads();
  for (int row0 = blockIdx.x * p.R; row0 < p.rows; row0 += step, buf ^= 1) {
    const int n = min(p.R, p.rows - row0) * pieces;
    for (int u0 = 0; u0 < n; u0 += 4 * kThreads) {
      float v[4][V];
      int row[4], c[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = min(u0 + j * kThreads + tid, n - 1);
        row[j] = (int)div_magic((uint32_t)u, (uint32_t)pieces, p.m_l);
        c[j] = (u - row[j] * pieces) * V;
        int s = c[j] + k;
        s = s >= p.L ? s - p.L : s;
        load_cyclic<V, IBF>(src, SCATTER ? (row0 + row[j]) * p.L : x_of[buf][row[j]], s, p.L, v[j]);
      }
      if (u0 == 0 && row0 + step < p.rows) decode(row0 + step, buf ^ 1);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (u0 + j * kThreads + tid >= n) continue;
        const float w = w_of[buf][row[j]];
#pragma unroll
        for (int i = 0; i < V; ++i) v[j][i] *= w;
        const int at = SCATTER ? x_of[buf][row[j]] + c[j] : (row0 + row[j]) * p.L + c[j];
        if constexpr (V == 1) {
          store_one<OBF>(dst, at, v[j][0]);
        } else if constexpr (!SCATTER) {
          store_run<4, OBF>(dst, at, v[j]);
        } else if constexpr (OBF) {
          const uint32_t lo = pack_bf16x2(v[j][0], v[j][1]), hi = pack_bf16x2(v[j][2], v[j][3]);
          *reinterpret_cast<u16x4_any*>(static_cast<uint16_t*>(dst) + at) = u16x4_any{(uint16_t)lo, (uint16_t)(lo >> 16), (uint16_t)hi, (uint16_t)(hi >> 16)};
        } else {
          *reinterpret_cast<f32x4_any*>(static_cast<float*>(dst) + at) = f32x4_any{v[j][0], v[j][1], v[j][2], v[j][3]};
        }
      }
    }
    __syncthreads();
  }
}

// The weight gradient of such a view: what view_grad_long computes (a workgroup per combination of the axes that the weight
// depends on and slice of the rows of the others), on whole rows.
struct ViewRowsGrad {
  ViewRows v;                                // n_outer: the axes that are summed; rows: of one combination
  int32_t sg[kMaxAxes];                      // their strides in G
  int32_t n_carry, c_size[kMaxAxes], c_sg[kMaxAxes], c_sx[kMaxAxes], c_sw[kMaxAxes];
  int32_t n_combo, n_splits, chunk;          // slices of `chunk` rows
};

template <bool IBF, int V>
__global__ __launch_bounds__(kThreads) void view_rows_grad(const ViewRowsGrad q, const void* __restrict__ G, const void* __restrict__ X,
                                                           double* __restrict__ partial, int* __restrict__ t_index, float* __restrict__ target) {
  __shared__ int x_of[2][kThreads], g_of[2][kThreads];
  __shared__ double wave_sum[kThreads / 64];
  const ViewRows& p = q.v;
  const int tid = threadIdx.x, pieces = p.L / V, combo = blockIdx.x / q.n_splits, slice = blockIdx.x - combo * q.n_splits;
  int x0 = p.bx, g0 = 0, t0 = p.bw;
  int rest_c = combo;
  for (int j = q.n_carry - 1; j >= 0; --j) {
    const int d = rest_c % q.c_size[j];
    rest_c /= q.c_size[j];
    x0 += d * q.c_sx[j];
    g0 += d * q.c_sg[j];
    t0 += d * q.c_sw[j];
  }
  const int begin = slice * q.chunk, end = min(p.rows, begin + q.chunk);
  auto decode = [&](int row0, int buf) {
    if (tid >= p.R || row0 + tid >= end) return;
    uint32_t rest = (uint32_t)(row0 + tid);
    int x = x0, g = g0;
    for (int j = p.n_outer - 1; j >= 0; --j) {
      const uint32_t r = div_magic(rest, (uint32_t)p.size[j], p.magic[j]);
      const int d = (int)(rest - r * (uint32_t)p.size[j]);
      rest = r;
      x += d * p.sx[j];
      g += d * q.sg[j];
    }
    x_of[buf][tid] = x;
    g_of[buf][tid] = g;
  };
  double acc = 0.0;                          // (64 bits: see view_grad_long)
  int buf = 0;
  decode(begin, 0);
  __syncthreads();
  for (int row0 = begin; row0 < end; row0 += p.R, buf ^= 1) {
    const int n = min(p.R, end - row0) * pieces;
    for (int u0 = 0; u0 < n; u0 += 4 * kThreads) {
      float g[4][V], x[4][V];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = min(u0 + j * kThreads + tid, n - 1), row = (int)div_magic((uint32_t)u, (uint32_t)pieces, p.m_l);
        const int c = (u - row * pieces) * V;
        int s = c + p.k;
        s = s >= p.L ? s - p.L : s;
        load_run<V, IBF>(G, g_of[buf][row] + c, g[j]);
        load_cyclic<V, IBF>(X, x_of[buf][row], s, p.L, x[j]);
      }
      if (u0 == 0 && row0 + p.R < end) decode(row0 + p.R, buf ^ 1);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (u0 + j * kThreads + tid >= n) continue;
#pragma unroll
        for (int i = 0; i < V; ++i) acc = fma((double)g[j][i], (double)x[j][i], acc);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) acc += __shfl_down(acc, d, 64);
  if ((tid & 63) == 0) wave_sum[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double t = wave_sum[0];
    for (int w = 1; w < kThreads / 64; ++w) t += wave_sum[w];
    if (q.n_splits == 1) {
      target[t0] = (float)t;
    } else {
      partial[blockIdx.x] = t;
      if (slice == 0) t_index[combo] = t0;
    }
  }
}

// pieces per row and rows per pass (four pieces per thread)
inline int view_rows_width(const ViewRows& p) { return p.L % 4 == 0 ? 4 : 1; }
inline void view_rows_pass(ViewRows& p) {
  const int pieces = p.L / view_rows_width(p);
  p.m_l = division_magic(pieces);
  p.R = std::max(1, std::min(kThreads, 4 * kThreads / pieces));
}

// Whether the view is one of rows; then its record for the forward pass
inline bool fill_view_rows(const syno_plan* plan, ViewRows& p) {
  const ViewStream& vs = plan->view;
  p = ViewRows{};
  if (vs.n_red != 0 || vs.n_axes < 1 || std::max(plan->out_elems, plan->x_elems) > (int64_t(1) << 30)) return false;
  const int last = vs.n_axes - 1;
  p.n_outer = last;
  p.L = vs.size[last];
  int64_t rows = 1;
  for (int i = 0; i < last; ++i) {
    int first[2], one[2] = {0, 0}, off[2];
    table_entry(vs, i, 0, first);
    if (vs.size[i] > 1) {
      table_entry(vs, i, 1, one);
      p.sx[i] = one[0] - first[0];
      p.sw[i] = one[1] - first[1];
    }
    for (int o = 2; o < vs.size[i]; ++o) {
      table_entry(vs, i, o, off);
      if (off[0] != first[0] + o * p.sx[i] || off[1] != first[1] + o * p.sw[i]) return false;
    }
    p.bx += first[0];
    p.bw += first[1];
    p.size[i] = vs.size[i];
    p.magic[i] = division_magic(vs.size[i]);
    rows *= vs.size[i];
  }
  // the innermost axis: the smallest offset is the row's start
  int first[2], off[2], least = 0;
  table_entry(vs, last, 0, first);
  for (int o = 0; o < p.L; ++o) {
    table_entry(vs, last, o, off);
    least = o == 0 ? off[0] : std::min(least, off[0]);
    if (off[1] != first[1]) return false;
  }
  p.k = first[0] - least;
  if (p.k >= p.L) return false;
  for (int o = 0; o < p.L; ++o) {
    table_entry(vs, last, o, off);
    if (off[0] != least + (o + p.k) % p.L) return false;
  }
  p.bx += least;
  p.bw += first[1];
  p.rows = (int32_t)rows;
  view_rows_pass(p);
  return true;
}
