// Matrix products of bf16 operands, out[m,n] = sum_k A(m,k) B(k,n), each operand stored with either axis contiguous: the
// forward product and both gradients of a matrix-product graph read their operands where they lie, without packed or
// transposed copies.
//  - A workgroup (8 waves) owns a BM x BN tile; steps of 64 k go through two LDS buffers, filled by loads that write LDS
//    directly while the other buffer is multiplied: one barrier per step.  Pieces outside the operand are loads past the end
//    of the buffer, which give zeros.
//  - LDS: an operand with k contiguous lies as rows of 64 k (128 bytes, the 16-byte units of a row permuted by the row's
//    number, so that the b128 fragment reads of 16 rows meet every bank once); one with k as the slow axis lies as rows of
//    BM (BN) values and is read with the transposing 8-byte reads, its 32-byte units permuted likewise.
//  - Bound: the matrix units.  256 x 192 takes 56 KB per 1536 cycles of them, 128 x 192 and 128 x 128 (smaller products, and
//    those that fill the last round of workgroups better) 40 KB per 768 and 32 KB per 512, near what the L2s deliver.
//    8192x3072x3072 runs at 900 TFLOP/s (a large library product: 1190).  Rings of 3 and 4 buffers changed the small tiles by
//    -8 to +8 %; the sum of a step by itself costs 5 to 10 % and halves the error (2.7e-7 -> 1.1e-7 at 2048x2048x2048).
//  - The matrix instruction takes B's fragment as its rows, so that a lane's four results are neighbours along n: 16-byte stores.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

#include "plan.h"

namespace syno {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
#define SYNO_LDS __attribute__((address_space(3)))

struct GemmParams {
  int32_t M, N, K;               // of this product
  int32_t lda, ldb;              // elements between rows of the operands as stored
  int32_t config, n_m, n_n, splits, steps_per_split;
  long long* probe;              // the plan's clock probe (4 values per workgroup), or null
};

constexpr int kStepK = 64, kThreads = 512;
constexpr uint32_t kOutside = 1u << 31;          // an offset beyond every operand here

// permutation of a row's 32-byte units in a tile whose rows are WIDTH values of one k: the rows that a transposing read
// touches at a time (0-3 and 8-11, 4-7 and 12-15, ...) fall on different banks
template <int WIDTH>
__device__ __forceinline__ int swizzle(int k) {
  return WIDTH % 128 == 0 ? (k & 3) | ((k >> 1) & 4) : ((k >> 1) & 1) | ((k >> 2) & 2);
}

typedef int intx4 __attribute__((ext_vector_type(4)));

// 16 bytes per lane from `src` + offset + step to LDS address `lds` + 16 * lane.  Written out because the compiler waits for
// its own direct loads before the next read of LDS, whichever buffer that reads; nothing but LDS is written, and the
// caller waits (vmcnt) and meets the other waves before that buffer is read.  m0, the address's register, is the compiler's
// own and is said to be overwritten (it warns that it will not keep the value across, which is what is meant).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(intx4 src, uint32_t lds, uint32_t offset, uint32_t step) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(offset), "s"(src), "s"(step) : "memory", "m0");
}
#pragma clang diagnostic pop
// a raw buffer over everything below kOutside bytes from `base` on
__device__ __forceinline__ intx4 buffer_at(const void* base) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  return intx4{__builtin_amdgcn_readfirstlane((int)(uint32_t)a), __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff), (int)kOutside, 0x00020000};
}

// Requests one step of an operand: EXT rows (columns) from `first` on, `left` k from the step's first on.
template <int EXT, bool KSLOW>
struct Stage {
  static constexpr int kLoads = EXT / 64;        // per wave: 1 KB each
  uint32_t at[kLoads];
  int k_of[kLoads];                              // where in the step this lane's piece lies along k
  __device__ __forceinline__ void init(int wave, int lane, int first, int extent, int ld) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int q = j * 8 + wave;
      int e, k;
      if constexpr (!KSLOW) {
        const int row = q * 8 + (lane >> 3);
        k = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
        e = first + row;
        at[j] = (uint32_t)e * (uint32_t)ld * 2u + k * 2u;
      } else {
        const int unit = q * 64 + lane, row = unit / (EXT / 8), in = unit - row * (EXT / 8);
        k = row;
        e = first + ((in >> 1) ^ swizzle<EXT>(row)) * 16 + (in & 1) * 8;
        at[j] = (uint32_t)k * (uint32_t)ld * 2u + (uint32_t)e * 2u;
      }
      if (e >= extent) at[j] = kOutside;
      k_of[j] = k;
    }
  }
  __device__ __forceinline__ void request(intx4 src, uint32_t lds, int wave, uint32_t step_at, int left) const {
#pragma unroll
    for (int j = 0; j < kLoads; ++j)
      load_to_lds(src, lds + (j * 8 + wave) * 1024, k_of[j] < left ? at[j] : kOutside, step_at);
  }
};

// the fragment of 16 rows (columns) from `tile` * 16 on, k = 32 * half + 8 * (lane >> 4) + 0..7
template <int EXT, bool KSLOW>
__device__ __forceinline__ bf16x8 fragment(const unsigned char* lds, int tile, int half, int lane) {
  const int r = lane & 15, g = lane >> 4;
  if constexpr (!KSLOW) {
    const int row = tile * 16 + r;
    return *reinterpret_cast<const bf16x8*>(lds + row * 128 + (((half * 4 + g) ^ ((row >> 1) & 7)) * 16));
  } else {
    const int k = 32 * half + 8 * g + (r >> 2);
    const unsigned char* at = lds + k * (EXT * 2) + ((tile ^ swizzle<EXT>(k)) * 32) + (r & 3) * 8;
    union { shortx4 s[2]; bf16x8 v; } f;
    f.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SYNO_LDS shortx4*)at);
    f.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SYNO_LDS shortx4*)(at + 4 * EXT * 2));     // (k + 4: the same permutation)
    return f.v;
  }
}

template <int BM, int BN, int WM, bool AS, bool BS, typename OutT>
__global__ __launch_bounds__(kThreads, BM * BN <= 128 * 128 ? 4 : 2) void gemm_bf16(const GemmParams p, const void* __restrict__ A, const void* __restrict__ B,
                                                      OutT* __restrict__ out, float* __restrict__ partial) {
  constexpr int WN = 8 / WM, MT = BM / WM / 16, NT = BN / WN / 16, ABYTES = BM * 128, STAGE = (BM + BN) * 128;
  extern __shared__ __align__(1024) unsigned char smem[];
  long long* const probe = p.probe ? p.probe + (int64_t)blockIdx.x * 4 : nullptr;
  if (probe && threadIdx.x == 0) {
    probe[0] = wall_clock64();
    probe[1] = clock64();
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // each XCD takes a run of tiles (neighbours share A's rows), walked in columns of 8 tile rows
  const int tiles = p.n_m * p.n_n, all = tiles * p.splits, per = all / 8, rest = all % 8, x = blockIdx.x % 8;
  int id = x * per + min(x, rest) + blockIdx.x / 8;
  const int split = id / tiles;
  id -= split * tiles;
  const int band = id / (8 * p.n_n), rows = min(8, p.n_m - band * 8), in = id - band * 8 * p.n_n;
  const int m0 = (band * 8 + in % rows) * BM, n0 = (in / rows) * BN;
  const int k_begin = split * p.steps_per_split * kStepK, k_end = min(p.K, k_begin + p.steps_per_split * kStepK);

  const intx4 ra = buffer_at(A), rb = buffer_at(B);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(SYNO_LDS unsigned char*)smem;
  Stage<BM, AS> sa;
  Stage<BN, BS> sb;
  sa.init(wave, lane, m0, p.M, p.lda);
  sb.init(wave, lane, n0, p.N, p.ldb);
  const uint32_t da = AS ? (uint32_t)p.lda * 2u : 2u, db = BS ? (uint32_t)p.ldb * 2u : 2u;      // bytes from one k to the next
  auto request = [&](int buf, int k) {
    sa.request(ra, lds0 + buf * STAGE, wave, (uint32_t)k * da, k_end - k);
    sb.request(rb, lds0 + buf * STAGE + ABYTES, wave, (uint32_t)k * db, k_end - k);
  };

  floatx4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // 128 x 128 tiles: the next step's fragments are read while this one is multiplied.  1.03 times as fast over 100 products; the
  // larger tiles, whose steps last longer than what that hides, lost 1 % with it.
  if constexpr (BM * BN <= 128 * 128) {
    // The fragments of a step are in registers when it begins, so that its buffer is free behind one barrier and is filled again while
    // the step is multiplied; the next step's are read between its rows of tiles, into the registers of the rows before.
    bf16x8 a[2][MT], b[2][NT];
    auto read_a = [&](int buf, int i) {
#pragma unroll
      for (int h = 0; h < 2; ++h) a[h][i] = fragment<BM, AS>(smem + buf * STAGE, wm * MT + i, h, lane);
    };
    auto read_b = [&](int buf, int j) {
#pragma unroll
      for (int h = 0; h < 2; ++h) b[h][j] = fragment<BN, BS>(smem + buf * STAGE + ABYTES, wn * NT + j, h, lane);
    };
    constexpr int LOADS = BM / 64 + BN / 64;               // of a wave and step
    const int steps = (k_end - k_begin + kStepK - 1) / kStepK;
    // this wave's part of a step is in LDS, and every other's
    auto meet = [&]() {
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    request(0, k_begin);
    if (steps > 1) {
      request(1, k_begin + kStepK);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    meet();
#pragma unroll
    for (int j = 0; j < NT; ++j) read_b(0, j);
#pragma unroll
    for (int i = 0; i < MT; ++i) read_a(0, i);
    int buf = 0;                                           // of the step that is multiplied: its fragments have been read
    auto multiply = [&](auto more_c, int next) {
      constexpr bool more = decltype(more_c)::value;
      // a step's products are summed by themselves first: the long sum is rounded once per step, to nearest
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if constexpr (more) { if (i > 0) read_a(next, i - 1); }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          floatx4 s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[0][i], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          acc[i][j] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[1][j], a[1][i], s, 0, 0, 0);
          if constexpr (more) { if (i == MT - 1) read_b(next, j); }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (more) read_a(next, MT - 1);
    };
    for (int t = 0; t + 1 < steps; ++t) {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      meet();                                              // step t + 1 is in LDS, and step t's buffer has been read by all
      if (t + 2 < steps) request(buf, k_begin + (t + 2) * kStepK);
      buf ^= 1;
      multiply(std::true_type{}, buf);
    }
    multiply(std::false_type{}, 0);
  } else {
    request(0, k_begin);
    int buf = 0;
    for (int k = k_begin; k < k_end; k += kStepK, buf ^= 1) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's part of the step is in LDS,
      __syncthreads();                                       // and every other's; the other buffer has been read
      if (k + kStepK < k_end) request(buf ^ 1, k + kStepK);
      const unsigned char *la = smem + buf * STAGE, *lb = la + ABYTES;
      bf16x8 a[2][MT], b[2][NT];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int j = 0; j < NT; ++j) b[h][j] = fragment<BN, BS>(lb, wn * NT + j, h, lane);
#pragma unroll
        for (int i = 0; i < MT; ++i) a[h][i] = fragment<BM, AS>(la, wm * MT + i, h, lane);
      }
      // a step's products are summed by themselves first: the long sum is rounded once per step, to nearest
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          floatx4 s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[0][i], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          acc[i][j] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[1][j], a[1][i], s, 0, 0, 0);
        }
    }
  }
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = m0 + (wm * MT + i) * 16 + r;
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n = n0 + (wn * NT + j) * 16 + 4 * g;
      if (n >= p.N) continue;
      const int64_t at = (int64_t)m * p.N + n;
      if (p.splits > 1) {
        *reinterpret_cast<floatx4*>(partial + (int64_t)split * p.M * p.N + at) = acc[i][j];
      } else if constexpr (sizeof(OutT) == 4) {
        *reinterpret_cast<floatx4*>(out + at) = acc[i][j];
      } else {
        union { __hip_bfloat16 v[4]; uint2 u; } o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o.v[v] = __float2bfloat16(acc[i][j][v]);
        *reinterpret_cast<uint2*>(out + at) = o.u;
      }
    }
  }
  if (probe && threadIdx.x == 0) {
    probe[2] = wall_clock64();
    probe[3] = clock64();
  }
}

// out = the sum of the splits (n: a multiple of 4)
template <typename OutT>
__global__ __launch_bounds__(256) void gemm_sum(const float* __restrict__ partial, OutT* __restrict__ out, int64_t n, int splits) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  floatx4 s = *reinterpret_cast<const floatx4*>(partial + i);
  for (int k = 1; k < splits; ++k) s += *reinterpret_cast<const floatx4*>(partial + k * n + i);
  if constexpr (sizeof(OutT) == 4) {
    *reinterpret_cast<floatx4*>(out + i) = s;
  } else {
    union { __hip_bfloat16 v[4]; uint2 u; } o;
#pragma unroll
    for (int v = 0; v < 4; ++v) o.v[v] = __float2bfloat16(s[v]);
    *reinterpret_cast<uint2*>(out + i) = o.u;
  }
}

constexpr int kConfigs = 3, kTiles[kConfigs][3] = {{256, 192, 4}, {128, 192, 2}, {128, 128, 4}};      // BM, BN, waves along m

template <int CFG, bool AS, bool BS, typename OutT>
syno_status launch_tiles(const GemmParams& p, const void* A, const void* B, OutT* out, float* partial, hipStream_t stream) {
  constexpr int BM = kTiles[CFG][0], BN = kTiles[CFG][1], lds = 2 * (BM + BN) * 128;
  auto kernel = gemm_bf16<BM, BN, kTiles[CFG][2], AS, BS, OutT>;
  static const hipError_t opt_in =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (opt_in != hipSuccess) return SYNO_ERR_HIP;
  hipLaunchKernelGGL(kernel, dim3(p.n_m * p.n_n * p.splits), dim3(kThreads), lds, stream, p, A, B, out, partial);
  if (p.splits > 1) {
    const int64_t n = (int64_t)p.M * p.N;
    hipLaunchKernelGGL(gemm_sum<OutT>, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, stream, partial, out, n, p.splits);
  }
  return hipGetLastError() == hipSuccess ? SYNO_OK : SYNO_ERR_HIP;
}

template <bool AS, bool BS, typename OutT>
syno_status launch_layout(const GemmParams& p, const void* A, const void* B, void* out, void* ws, hipStream_t stream) {
  OutT* const o = static_cast<OutT*>(out);
  float* const w = static_cast<float*>(ws);
  switch (p.config) {
    case 0: return launch_tiles<0, AS, BS, OutT>(p, A, B, o, w, stream);
    case 1: return launch_tiles<1, AS, BS, OutT>(p, A, B, o, w, stream);
    default: return launch_tiles<2, AS, BS, OutT>(p, A, B, o, w, stream);
  }
}
}  // namespace

// Takes bf16 products whose contiguous axes are multiples of 8 (16-byte pieces), unless the caller names a tile, a row count
// or a number of splits of the convolution kernels.  Against those at every size measured (us, before -> now; forward, dX,
// dW): 64x128x128 9.8, 12.5, 5.0 -> 4.0, 3.9, 4.3; 264x200x1032 28, 17, 16 -> 8.7, 5.6, 5.9; 1000x1024x512 20, 29, 27 -> 9,
// 13, 13; 8192x128x128 13, 17, 66 -> 5.4, 5.3, 14; 8192x2304x768 116, 112, 118 -> 52, 38, 48; 8192x3072x3072 498, 456, 589
// -> 171, 165, 186 (M x N x K).  The tile and the splits are those of the lowest estimate in cycles: rounds of 256
// workgroups, each its steps (matrix instructions, or what the L2s deliver) and 4000 cycles at its ends; splits also the pass
// over their sums.  Named one by one on seven products, no other choice was faster by more than 6 %.
bool gemm_configure(syno_plan* plan, int which, int64_t M, int64_t K, int64_t N) {
  const syno_plan_options& o = plan->opt;
  if (plan->in_dtype != SYNO_BF16 || o.mfma_splits || o.mfma_rows || o.mfma_variant) return false;
  if (K % 8 || N % 8 || std::max({M * K, K * N, M * N}) * 4 >= (int64_t)kOutside) return false;
  GemmParams p{};
  p.M = (int)(which == SYNO_BWD_WEIGHT ? K : M);
  p.N = (int)(which == SYNO_BWD_DATA ? K : N);
  p.K = (int)(which == SYNO_FWD ? K : which == SYNO_BWD_DATA ? N : M);
  p.lda = (int)(which == SYNO_BWD_DATA ? N : K);
  p.ldb = (int)N;
  p.probe = static_cast<long long*>(o.clock_probe);
  const int steps = (p.K + kStepK - 1) / kStepK;
  auto take = [&](int c, int splits) {
    p.config = c;
    p.n_m = (p.M + kTiles[c][0] - 1) / kTiles[c][0];
    p.n_n = (p.N + kTiles[c][1] - 1) / kTiles[c][1];
    p.steps_per_split = (steps + splits - 1) / splits;
    p.splits = (steps + p.steps_per_split - 1) / p.steps_per_split;
  };
  const int64_t sums = (int64_t)p.M * p.N * 4;     // bytes of one split's
  auto cheapest = [&](int64_t limit) {
    double best = 1e30;
    int best_c = -1, best_splits = 0;
    for (int c = 0; c < kConfigs; ++c)
      for (int splits = 1; splits <= 16 && splits <= steps; ++splits) {      // (43 splits of 8192x128x128's dW: 19 us, 16: 14)
        take(c, splits);
        if (p.splits != splits) continue;
        const int64_t blocks = (int64_t)p.n_m * p.n_n * splits;
        if (blocks >= (1 << 30) || (splits > 1 && splits * sums > limit)) continue;
        const double step = std::max(kTiles[c][0] * kTiles[c][1] / 32., (kTiles[c][0] + kTiles[c][1]) * 3.2);
        const double cost = (double)((blocks + 255) / 256) * (p.steps_per_split * step + 4000.) + (splits > 1 ? 6000. + splits * sums * 2 / 1800. : 0.);
        if (cost < best) { best = cost; best_c = c; best_splits = splits; }
      }
    if (best_c >= 0) take(best_c, best_splits);
    return best_c >= 0;
  };
  if (!cheapest(64ll << 20)) return false;
  // The weight gradient's sums have to fit the scratch of the entry point without a workspace.  Where that refuses the cheapest
  // choice: the small tiles, two workgroups of which a compute unit holds, in as many splits as one such round and the scratch
  // have room for (us, the refused choice -> this, and in brackets the cheapest one by the estimate that fits: 11136x8432x200
  // 68 -> 73 (77), 23992x17816x96 217 -> 196 (234), 16384x2048x768 72 -> 70 (82), 16136x13584x216 146 -> 188 (240)).
  constexpr int64_t scratch = SYNO_STATIC_SCRATCH_BYTES;
  if (which == SYNO_BWD_WEIGHT && p.splits > 1 && p.splits * sums > scratch) {
    take(2, 1);
    const int64_t splits = std::min<int64_t>({2 * 256 / ((int64_t)p.n_m * p.n_n), scratch / sums, steps});
    if (splits >= 2) take(2, (int)splits);
    else if (!cheapest(scratch)) return false;
  }
  Launch& L = plan->launch[which];
  static_assert(sizeof(GemmParams) <= sizeof(L.params), "parameter record does not fit");
  memcpy(L.params, &p, sizeof p);
  L.workspace = p.splits > 1 ? (size_t)p.splits * p.M * p.N * 4 : 0;
  return true;
}

std::string gemm_describe(const syno_plan* plan, int which) {
  GemmParams p;
  memcpy(&p, plan->launch[which].params, sizeof p);
  char b[128];
  snprintf(b, sizeof b, "as it is: tiles=%dx%d grid=%d reduction-splits=%d", kTiles[p.config][0], kTiles[p.config][1], p.n_m * p.n_n * p.splits, p.splits);
  return b;
}

// A: X (forward, backward-weight: here the operands come as G, X) or G (backward-data).
syno_status launch_gemm(const syno_plan* plan, int which, const void* A, const void* B, void* out, void* ws, hipStream_t stream) {
  GemmParams p;
  memcpy(&p, plan->launch[which].params, sizeof p);
  const bool f32 = which == SYNO_BWD_WEIGHT || plan->out_dtype == SYNO_F32;
  if (which == SYNO_FWD) return f32 ? launch_layout<false, true, float>(p, A, B, out, ws, stream) : launch_layout<false, true, __hip_bfloat16>(p, A, B, out, ws, stream);
  if (which == SYNO_BWD_DATA) return f32 ? launch_layout<false, false, float>(p, A, B, out, ws, stream) : launch_layout<false, false, __hip_bfloat16>(p, A, B, out, ws, stream);
  return launch_layout<true, true, float>(p, B, A, out, ws, stream);
}

}  // namespace syno
