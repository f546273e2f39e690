// Kernels for few token rows: the GEMMs of the expert at M <= 64 rows (short
// chunks, the sequential baseline, the time-MLP) and the attention of small
// grids.  At these sizes a kernel is a chain of latencies (dispatch, first
// loads, a reduction, the stores), not arithmetic or bandwidth, so both
// kernels take one pass: every operand goes straight from memory into MFMA
// registers, the reduction dimension is split over the waves of a workgroup,
// and the waves' sums meet once in LDS.  No second kernel reduces partials.
#include "fv_internal.h"

namespace fv {

namespace {

// Output columns of a 16-column group g.  Linear: 16 g + i.  Paired (packed
// QKV and gate/up matrices, whose partners sit 32 columns apart in every 64):
// i < 8 the first partners 64 (g / 4) + 8 (g % 4) + i, i >= 8 their partners,
// so lanes l and l ^ 32 of the output tile hold a pair.
template <bool PAIR>
__device__ __forceinline__ int few_col(int g, int i) {
  if (!PAIR) return 16 * g + i;
  return 64 * (g >> 2) + 8 * (g & 3) + (i & 7) + 32 * (i >> 3);
}

// C[M][N] = A[M][K] Bt[N][K]^T for M <= 64 (RT 16-row tiles; more rows by
// grid.y).  A workgroup owns CG 16-column groups and one k slice (blockIdx.z
// of KS); its KW waves split that slice, each wave loading its pieces of the
// weights and of A directly as MFMA fragments (a wave's whole share of a
// 1024-deep product is one batch of loads), and the KW partial tiles are
// added through LDS in wave order.  The product is formed transposed
// (weights as the A operand): a lane then holds four consecutive columns of
// one row.  Wave w < RT * CG finishes tile w; what its epilogue reads is
// requested before the main loop.
template <typename T, int RT, int CG, int KW, class Epi>
__global__ __launch_bounds__(64 * KW) void few_gemm_kernel(const T* __restrict__ A,
                                                           const T* __restrict__ Bt, int M, int N,
                                                           int K, int KS, Epi epi) {
  static_assert(RT * CG <= KW, "one output tile per wave");
  if (epi.skipped()) return;
  constexpr int EPV = 16 / (int)sizeof(T);
  constexpr int U = 4;  // 64-byte k blocks per batch of loads
  __shared__ f32x4 red[KW][RT * CG][64];
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g0 = blockIdx.x * CG, row0 = blockIdx.y * 16 * RT, kz = blockIdx.z;
  const int nb = K / (4 * EPV);
  const int z0 = (kz * nb) / KS, zn = ((kz + 1) * nb) / KS - z0;
  const int b0 = z0 + (wave * zn) / KW, b1 = z0 + ((wave + 1) * zn) / KW;

  const T* wp[CG];
  const T* ap[RT];
#pragma unroll
  for (int j = 0; j < CG; ++j)
    wp[j] = Bt + tile_off<T>(few_col<Epi::kPair>(g0 + j, c), q * EPV, K);
  // rows past M re-read row M - 1 (in bounds, and few cache lines more)
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int r = min(row0 + 16 * i + c, M - 1);
    ap[i] = A + (Epi::kTiledA ? tile_off<T>(r, q * EPV, K) : (size_t)r * K + q * EPV);
  }
  // the tile this wave finishes; a wave with none requests an existing one's
  // epilogue inputs (a column past N would be out of bounds) and leaves them
  const int ti = wave % RT, tj = min(wave / RT, CG - 1);
  const int orow = row0 + 16 * ti + c;
  typename Epi::Pre pre;
  epi.begin(min(orow, M - 1), pre);

  f32x4 acc[RT][CG];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CG; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (b0 >= b1) epi.prepare(min(orow, M - 1), g0 + tj, lane, pre);  // no block of its own
  for (int b = b0; b < b1; b += U) {
    // loads past the wave's last block re-read it (in bounds, not
    // multiplied); the weights, which may come from HBM, go first
    u32x4 w[U][CG], a[U][RT];
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int j = 0; j < CG; ++j)
        w[s][j] = *reinterpret_cast<const u32x4*>(wp[j] + (size_t)min(b + s, b1 - 1) * (64 * EPV));
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int i = 0; i < RT; ++i)
        a[s][i] = *reinterpret_cast<const u32x4*>(
            ap[i] + (size_t)min(b + s, b1 - 1) * (Epi::kTiledA ? 64 * EPV : 4 * EPV));
    __builtin_amdgcn_sched_barrier(0);
    if (b == b0) epi.prepare(min(orow, M - 1), g0 + tj, lane, pre);
#pragma unroll
    for (int s = 0; s < U; ++s)
      if (b + s < b1)
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < CG; ++j) acc[i][j] = mma64(w[s][j], a[s][i], acc[i][j], T());
  }
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CG; ++j) red[wave][j * RT + i][lane] = acc[i][j];
  __syncthreads();
  if (wave >= RT * CG) return;
  f32x4 v = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < KW; ++w) v += red[w][wave][lane];
  epi.apply(v, pre, orow, g0 + tj, lane, kz, M);
}

// ---------------------------------------------------------------- epilogues
// begin, prepare: request what the lane's part of the tile needs from memory,
// before and after the operand loads; apply: lane (q, c) gets row `row` (c)
// and the four columns few_col(g, 4q .. 4q + 3).
struct FewPartial {  // fp32 split partials [KS][M][N] for the fused residual reduction
  static constexpr bool kPair = false, kTiledA = true;
  struct Pre {};
  float* ws;
  int N;
  __device__ bool skipped() const { return false; }
  __device__ void begin(int, Pre&) const {}
  __device__ void prepare(int, int, int, Pre&) const {}
  __device__ void apply(f32x4 v, Pre, int row, int g, int lane, int kz, int M) const {
    if (row < M)
      *reinterpret_cast<f32x4*>(ws + ((size_t)kz * M + row) * N + 16 * g + 4 * (lane >> 4)) = v;
  }
};

template <typename T>
struct FewBiasSilu {
  static constexpr bool kPair = false, kTiledA = false;
  typedef f32x4 Pre;
  T* out;
  const float* bias;
  int ldo;
  const int* skip;
  __device__ bool skipped() const { return skip && *skip; }
  __device__ void begin(int, Pre&) const {}
  __device__ void prepare(int, int g, int lane, Pre& b) const {
    b = *reinterpret_cast<const f32x4*>(bias + 16 * g + 4 * (lane >> 4));
  }
  __device__ void apply(f32x4 v, Pre b, int row, int g, int lane, int, int M) const {
    if (row < M)
      store4<T>(out + (size_t)row * ldo + 16 * g + 4 * (lane >> 4), silu_f(v[0] + b[0]),
                silu_f(v[1] + b[1]), silu_f(v[2] + b[2]), silu_f(v[3] + b[3]));
  }
};

struct FewBiasF32 {
  static constexpr bool kPair = false, kTiledA = false;
  typedef f32x4 Pre;
  float* out;
  const float* bias;
  int ldo;
  const int* skip;
  __device__ bool skipped() const { return skip && *skip; }
  __device__ void begin(int, Pre&) const {}
  __device__ void prepare(int, int g, int lane, Pre& b) const {
    b = *reinterpret_cast<const f32x4*>(bias + 16 * g + 4 * (lane >> 4));
  }
  __device__ void apply(f32x4 v, Pre b, int row, int g, int lane, int, int M) const {
    if (row < M)
      *reinterpret_cast<f32x4*>(out + (size_t)row * ldo + 16 * g + 4 * (lane >> 4)) = v + b;
  }
};

// first partner's value in x0, second's in x1, for lanes l and l ^ 32 alike
__device__ __forceinline__ void pair_of(f32x4 v, f32x4& x0, f32x4& x1) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const auto s =
        __builtin_amdgcn_permlane32_swap(__float_as_uint(v[e]), __float_as_uint(v[e]), false, false);
    x0[e] = __uint_as_float(s[0]);
    x1[e] = __uint_as_float(s[1]);
  }
}

template <typename T>
struct FewGeglu {
  static constexpr bool kPair = true, kTiledA = true;
  struct Pre {};
  T* out;
  int ldo;
  __device__ bool skipped() const { return false; }
  __device__ void begin(int, Pre&) const {}
  __device__ void prepare(int, int, int, Pre&) const {}
  __device__ void apply(f32x4 v, Pre, int row, int g, int lane, int, int M) const {
    f32x4 x0, x1;
    pair_of(v, x0, x1);
    if (row < M && lane < 32)
      store4<T>(out + tile_off<T>(row, 8 * g + 4 * (lane >> 4), ldo), gelu_tanh_f(x0[0]) * x1[0],
                gelu_tanh_f(x0[1]) * x1[1], gelu_tanh_f(x0[2]) * x1[2], gelu_tanh_f(x0[3]) * x1[3]);
  }
};

template <typename T>
struct FewGelu {
  static constexpr bool kPair = false, kTiledA = true;
  struct Pre {};
  T* out;
  int ldo;
  __device__ bool skipped() const { return false; }
  __device__ void begin(int, Pre&) const {}
  __device__ void prepare(int, int, int, Pre&) const {}
  __device__ void apply(f32x4 v, Pre, int row, int g, int lane, int, int M) const {
    if (row < M)
      store4<T>(out + tile_off<T>(row, 16 * g + 4 * (lane >> 4), ldo), gelu_tanh_f(v[0]),
                gelu_tanh_f(v[1]), gelu_tanh_f(v[2]), gelu_tanh_f(v[3]));
  }
};

// Rotary + arena scatter of the packed QKV product (see EpiQkv): lanes below
// 32 store the first half of each rotated pair, the others the second; value
// columns are stored element by element into V^T (16 lanes: 16 tokens of one
// feature row).
template <typename T>
struct FewQkv {
  static constexpr bool kPair = true, kTiledA = true;
  struct Pre {
    int b, len, arow;
    f32x4 cs, sn;
  };
  QkvArgs<T> a;
  __device__ bool skipped() const { return false; }
  __device__ void begin(int row, Pre& p) const {
    p.b = row / a.tokens;
    p.len = a.len[p.b];
  }
  __device__ void prepare(int row, int g, int lane, Pre& p) const {
    const int tok = row - p.b * a.tokens;
    p.arow = buffer_row0(p.len) + tok;
    // (value columns read, and ignore, a valid table entry)
    const int half = a.head_dim / 2, c0 = 64 * (g >> 2);
    const int d = 32 * ((c0 % a.head_dim) >> 6) + 8 * (g & 3) + 4 * ((lane >> 4) & 1);
    p.cs = *reinterpret_cast<const f32x4*>(a.rcos + (size_t)(p.len + tok) * half + d);
    p.sn = *reinterpret_cast<const f32x4*>(a.rsin + (size_t)(p.len + tok) * half + d);
  }
  __device__ void apply(f32x4 v, const Pre& p, int row, int g, int lane, int, int M) const {
    const int dh = a.head_dim, half = dh / 2;
    const int qd = a.n_q_heads * dh, kd = a.n_kv_heads * dh, c0 = 64 * (g >> 2);
    f32x4 x0, x1;
    pair_of(v, x0, x1);
    if (row >= M) return;
    const bool second = lane >= 32;
    if (c0 < qd + kd) {
      const bool isq = c0 < qd;
      const int cc = isq ? c0 : c0 - qd, head = cc / dh;
      const int d = 32 * ((cc - head * dh) >> 6) + 8 * (g & 3) + 4 * ((lane >> 4) & 1);
      T* dst = isq ? a.q + (size_t)row * qd + head * dh
                   : a.karena + (((size_t)p.b * a.n_kv_heads + head) * a.S + p.arow) * dh;
      const f32x4 y = second ? x1 * p.cs + x0 * p.sn : x0 * p.cs - x1 * p.sn;
      store4<T>(dst + d + (second ? half : 0), y[0], y[1], y[2], y[3]);
    } else {
      const int cc = c0 - qd - kd + 8 * (g & 3) + 4 * ((lane >> 4) & 1) + (second ? 32 : 0);
      const int head = cc / dh, d = cc - head * dh;
      T* base = a.vtarena + (((size_t)p.b * a.n_kv_heads + head) * dh + d) * a.S + p.arow;
#pragma unroll
      for (int e = 0; e < 4; ++e) base[(size_t)e * a.S] = from_f32<T>(v[e]);
    }
  }
};

template <typename T, int RT, int CG, int KW, class Epi>
void few_launch(const T* A, const T* Bt, int M, int N, int K, int KS, const Epi& epi,
                hipStream_t s) {
  const dim3 grid(N / (16 * CG), (M + 16 * RT - 1) / (16 * RT), KS);
  hipLaunchKernelGGL((few_gemm_kernel<T, RT, CG, KW, Epi>), grid, dim3(64 * KW), 0, s, A, Bt, M, N,
                     K, KS, epi);
}

// Row tiles by M; 4 waves where a wave's share would fall under two k
// blocks; two column groups per workgroup (they share the A fragments) once
// one would give more than about 320 workgroups; four in fp32 at 17 to 32 rows
// past 1280 column groups (28672 columns, k 2048, 17 rows: 70 -> 57 us; 26624
// columns, k 1024, 33.6 -> 33.3; slower in bf16 and at 16 rows or fewer).
template <typename T, class Epi>
void few_run(const T* A, const T* Bt, int M, int N, int K, int KS, const Epi& epi, hipStream_t s) {
  if (M <= 0) return;
  const int nb = K * (int)sizeof(T) / 64 / KS;
  const bool two = (long)(N / 16) * KS > 320 && N % 32 == 0;
  if constexpr (sizeof(T) == 4)
    if (M > 16 && M <= 32 && (long)(N / 16) * KS > 1280 && N % 64 == 0)
      return few_launch<T, 2, 4, 8>(A, Bt, M, N, K, KS, epi, s);
#define FV_FEW(RT)                                                   \
  if (nb <= 16 && !(two && RT > 2))                                   \
    two ? few_launch<T, RT, (RT > 2 ? 1 : 2), 4>(A, Bt, M, N, K, KS, epi, s) \
        : few_launch<T, RT, 1, 4>(A, Bt, M, N, K, KS, epi, s);       \
  else if (two)                                                      \
    few_launch<T, RT, 2, 8>(A, Bt, M, N, K, KS, epi, s);             \
  else                                                               \
    few_launch<T, RT, 1, 8>(A, Bt, M, N, K, KS, epi, s);
  if (M <= 16) {
    FV_FEW(1)
  } else if (M <= 32) {
    FV_FEW(2)
  } else if (M <= 48) {
    FV_FEW(3)
  } else {
    FV_FEW(4)
  }
#undef FV_FEW
}

}  // namespace

// k slices of an output or down projection at few rows: each workgroup's
// waves take four k blocks each, in at most 8 waves.
int few_splits(int N, int K, int esz) {
  const int nb = K * esz / 64;
  int ks = 2;
  while (ks < 8 && nb / ks > 32 && (long)(N / 16) * ks * 2 <= 512) ks *= 2;
  if (ks < 4 && nb / 4 >= 8 && (long)(N / 16) * 4 <= 512) ks = 4;
  return ks;
}

template <typename T>
void few_partials(const T* A, const T* Bt, float* ws, int M, int N, int K, int ks, hipStream_t s) {
  few_run(A, Bt, M, N, K, ks, FewPartial{ws, N}, s);
}
template <typename T>
void few_bias_silu(const T* A, const T* Bt, const float* bias, T* out, int M, int N, int K,
                   hipStream_t s, const int* skip) {
  few_run(A, Bt, M, N, K, 1, FewBiasSilu<T>{out, bias, N, skip}, s);
}
template <typename T>
void few_bias_f32(const T* A, const T* Bt, const float* bias, float* out, int M, int N, int K,
                  hipStream_t s, const int* skip) {
  few_run(A, Bt, M, N, K, 1, FewBiasF32{out, bias, N, skip}, s);
}
template <typename T>
void few_qkv(const T* A, const T* Bt, const QkvArgs<T>& qa, int M, int N, int K, hipStream_t s) {
  few_run(A, Bt, M, N, K, 1, FewQkv<T>{qa}, s);
}
template <typename T>
void few_geglu(const T* A, const T* Bt, T* out, int M, int N, int K, hipStream_t s) {
  few_run(A, Bt, M, N, K, 1, FewGeglu<T>{out, N / 2}, s);
}
template <typename T>
void few_gelu(const T* A, const T* Bt, T* out, int M, int N, int K, hipStream_t s) {
  few_run(A, Bt, M, N, K, 1, FewGelu<T>{out, N}, s);
}

#define FV_INSTANTIATE(T)                                                                         \
  template void few_partials<T>(const T*, const T*, float*, int, int, int, int, hipStream_t);     \
  template void few_bias_silu<T>(const T*, const T*, const float*, T*, int, int, int, hipStream_t, \
                                 const int*);                                                     \
  template void few_bias_f32<T>(const T*, const T*, const float*, float*, int, int, int,          \
                                hipStream_t, const int*);                                         \
  template void few_qkv<T>(const T*, const T*, const QkvArgs<T>&, int, int, int, hipStream_t);    \
  template void few_geglu<T>(const T*, const T*, T*, int, int, int, hipStream_t);                 \
  template void few_gelu<T>(const T*, const T*, T*, int, int, int, hipStream_t);
FV_INSTANTIATE(bf16_t)
FV_INSTANTIATE(float)
#undef FV_INSTANTIATE

}  // namespace fv
