// MFMA GEMMs of the action expert with fused epilogues.
//
// Every linear layer of the expert (time-MLP, FiLM maps, packed QKV, output
// projection, packed gate/up, down projection) is C = A * W with A the
// activations [M][K] (row-major) and W stored output-major as Bt [N][K].
//
// Two main loops.  The bf16 tiles 256x256, 128x128 and 64x128 use
// gemm_dma_kernel: k-tiles go from memory straight into a ring of LDS stages
// with the direct-to-LDS loads (see there).  The fp32 tiles, the bf16 256x128
// tile and bf16 products of 2^22 k or more use gemm_kernel, described here.
// Products of at most 64 rows have kernels of their own (fv_few.hip).
//
// gemm_kernel block: NW waves (2, 4 or 8).  Tile BM x BN; k is staged through
// LDS 128 bytes per row (64 bf16 / 32 fp32) at a time in two buffers.  While a wave
// multiplies the tile in one buffer with 32x32 MFMA instructions, the
// registers holding the next tile are written to the other buffer piece by
// piece between k-steps, and every freed register piece immediately issues
// its global load of the tile after that; the MFMA operands of the next
// k-step are read from LDS while the current k-step's MFMAs run, and the
// instruction order interleaves MFMAs with those reads, stores and loads.
// One barrier per k-tile.  Rows of A beyond M re-read row M-1 (never
// stored).  Large grids walk their tiles in an order that keeps the blocks
// each of the chip's 8 dies runs together on shared operands.
//
// Split-K (KS > 1): block z of a tile accumulates k-tiles [z*nk/KS,
// (z+1)*nk/KS) and writes its partial tile to a workspace; a second, small
// kernel sums the KS partials of each tile in split order (so the result
// does not depend on scheduling) and runs the epilogue.  The partials are
// fp32, except those of the direct-to-LDS kernel with no epilogue (EpiNone,
// the output and down projections), which are bf16 and are summed by the
// fused residual reduction (resid_norm_kernel).  The kernel
// boundary makes the partials visible across the chip's separate L2 caches
// without device-wide cache flushes inside the GEMM.
//
// Epilogues consume the accumulators in registers:
//  * bias + SiLU (time-MLP), bias to fp32 (FiLM maps);
//  * QKV: queries and keys are rotated (half-split rotary pairs) and keys and
//    values are written straight into the layer's K / V^T arena at row
//    buffer_row0(len[b]) + token (the prefix length rounded up to 8), so
//    attention reads [prefix ; buffer] from one arena;
//  * gated residual h += gate[chunk] * acc;
//  * GeGLU gelu(g) * u and plain GELU.
// Element-type outputs of the QKV and GELU epilogues are transposed within
// each group of four lanes first, so a lane stores four consecutive columns
// of one row at once.
// Paired epilogues rely on the weight packing: columns [64p, 64p+32) and
// [64p+32, 64p+64) of a packed matrix hold the two partners of a pair, which
// then sit in the same lane and register of two adjacent 32-column tiles.
#include <stdexcept>
#include <type_traits>

#include "fv_internal.h"

namespace fv {

namespace {

// 32x32 MFMA per element type: bf16 32x32x16 (8 k per lane), fp32 32x32x2
// (1 k per lane).  Output layout (both): lane l, register r holds
// row 8*(r/4) + 4*(l/32) + r%4, column l%32 of the 32x32 tile.
template <typename T> struct Mf32;
template <> struct Mf32<bf16_t> {
  static constexpr int KG = 8, KM = 16;
  typedef bf16x8 frag;
  __device__ static __forceinline__ frag load(const bf16_t* p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(p));
  }
  __device__ static __forceinline__ f32x16 mma(frag a, frag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mf32<float> {
  static constexpr int KG = 1, KM = 2;
  typedef float frag;
  __device__ static __forceinline__ frag load(const float* p) { return *p; }
  __device__ static __forceinline__ f32x16 mma(frag a, frag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};

__device__ __forceinline__ int acc_row(int r, int lane) {
  return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

// Registers 4q .. 4q+3 of a 32x32 accumulator hold four consecutive rows of
// the lane's column.  quad_rows transposes each such 4x4 block within its
// group of four lanes: lane l gets back row 8q + 4 (l / 32) + (l & 3) at the
// columns (l & 28) .. (l & 28) + 3 of the 32-column block, so a row's four
// outputs leave as one store instead of four 2-byte ones.  Every lane of the
// wave must be active.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ f32x4 quad_rows(float x0, float x1, float x2, float x3, int lane) {
  const bool b0 = lane & 1, b1 = lane & 2;
  // lanes l, l^1 trade: each then holds two adjacent columns of the rows
  // (l & 1) and 2 + (l & 1)
  const float r1 = dpp_mov<0xB1>(b0 ? x0 : x1);  // quad_perm [1,0,3,2]
  const float r2 = dpp_mov<0xB1>(b0 ? x2 : x3);
  const float z0 = b0 ? r1 : x0, z1 = b0 ? x1 : r1;
  const float z2 = b0 ? r2 : x2, z3 = b0 ? x3 : r2;
  // lanes l, l^2 trade column pairs
  const float t1 = dpp_mov<0x4E>(b1 ? z0 : z2);  // quad_perm [2,3,0,1]
  const float t2 = dpp_mov<0x4E>(b1 ? z1 : z3);
  return b1 ? f32x4{t1, t2, z2, z3} : f32x4{z0, z1, t1, t2};
}
// store of the four transposed values at p (4-element aligned when `vec`)
template <typename T>
__device__ __forceinline__ void store_quad(T* p, const f32x4& u, bool vec) {
  if (vec) {
    store4<T>(p, u[0], u[1], u[2], u[3]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = from_f32<T>(u[e]);
  }
}

// Output tile of this block.  Block b of a launch runs on XCD b % 8 (the
// chip's 8 dies, each with its own L2).  When the grid is large enough, the
// (x, y) block index is remapped so that each die takes a contiguous range
// of tiles, walked in groups kTileGroup row panels tall, column by column:
// the tiles a die runs together then share A row panels and weight column
// blocks in its L2 instead of fetching them from memory once per die.
// Split-K grids (gridDim.z k slices dividing the 8 dies) give each die one
// k slice and a contiguous range of its column blocks, every row tile of
// them: a die then fetches its slice of A and its share of the weights, not
// the whole A of every slice.
constexpr int kTileGroup = 8;
__device__ __forceinline__ void tile_of(int& tm, int& tn, int& kz) {
  const int nN = gridDim.x, nM = gridDim.y, nK = gridDim.z, nb = nN * nM;
  kz = blockIdx.z;
  if (nK > 1 && 8 % nK == 0 && nN % (8 / nK) == 0) {
    const int dpk = 8 / nK;  // dies per k slice
    const int lin = (blockIdx.z * nM + blockIdx.y) * nN + blockIdx.x;
    const int x = lin & 7, s = lin >> 3;
    kz = x / dpk;
    tm = s % nM;
    tn = (x % dpk) * (nN / dpk) + s / nM;
    return;
  }
  if (nb < 64) {
    tm = blockIdx.y;
    tn = blockIdx.x;
    return;
  }
  const int b = blockIdx.y * nN + blockIdx.x;
  const int per = nb >> 3, rem = nb & 7;  // dies x < rem take per + 1 tiles
  const int x = b & 7, s = b >> 3;
  const int L = x * per + min(x, rem) + s;
  const int gsz = kTileGroup * nN;
  const int g = L / gsz, i = L - g * gsz;
  const int gm = min(kTileGroup, nM - g * kTileGroup);
  tm = g * kTileGroup + i % gm;
  tn = i / gm;
}

// Epilogues with a run-time skip flag (Epi::skipped()): the whole launch
// returns at once when it is set (every workgroup reads the same flag).
template <class Epi, class = void>
struct EpiSkip {
  __device__ static bool skip(const Epi&) { return false; }
};
template <class Epi>
struct EpiSkip<Epi, std::void_t<decltype(&Epi::skipped)>> {
  __device__ static bool skip(const Epi& e) { return e.skipped(); }
};

template <typename T, int BM, int BN, int NW, int WGM, class Epi>
__global__ __launch_bounds__(64 * NW) void gemm_kernel(const T* __restrict__ A,
                                                       const T* __restrict__ Bt, int M, int N,
                                                       int K, int KS, float* __restrict__ ws,
                                                       Epi epi) {
  if (EpiSkip<Epi>::skip(epi)) return;
  using MF = Mf32<T>;
  constexpr int NT = 64 * NW;
  constexpr int WGN = NW / WGM;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / 32, FN = WTN / 32;
  constexpr int EPV = 16 / (int)sizeof(T);  // elements per 16-byte vector
  constexpr int BK = 8 * EPV;               // 128 bytes of k per row and stage
  constexpr int LDR = BK + EPV;             // LDS row pitch (one vector of padding)
  constexpr int NA = BM * 8 / NT, NB = BN * 8 / NT, NP = NA + NB;  // 16-byte pieces per thread
  constexpr int NSTEP = BK / MF::KM;        // k-steps per stage
  static_assert(FM >= 1 && FN >= 1 && WGM * WGN == NW, "bad tile");
  static_assert((BM * 8) % NT == 0 && (BN * 8) % NT == 0 && NSTEP % 2 == 0, "bad tile");
  __shared__ __attribute__((aligned(16))) T sm[2 * (BM + BN) * LDR];  // [buf][A rows ; B rows]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  int tm, tn, kz;
  tile_of(tm, tn, kz);
  const int m0 = tm * BM, n0 = tn * BN;
  const int arow = wm * WTM, brow = BM + wn * WTN;  // fragment rows in the stage
  const int nk_all = K / BK;
  const int kt0 = (kz * nk_all) / KS, kt1 = ((kz + 1) * nk_all) / KS;
  const int klast = (kt1 - 1) * BK;

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};

  // Thread piece p: 16 bytes of row r, k-vector c of a stage (A rows first).
  // Consecutive threads take consecutive vectors of a row of A, consecutive
  // rows of a weight tile: its loads are then contiguous, which counts where the
  // weights come from memory (fp32, 4 streams of 100 tokens, 4 layers of width
  // 512: 426 us a pass, 433 with consecutive vectors of a row, though a product
  // alone, its weights in cache, is 2-3 % slower).
  const T* gp[NP];
  int lp[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const bool isa = p < NA;
    const int vi = tid + NT * (isa ? p : p - NA);
    const int r = isa ? vi >> 3 : (vi >> 7) * 16 + (vi & 15);
    const int c = isa ? vi & 7 : (vi >> 4) & 7;
    gp[p] = isa ? A + (size_t)min(m0 + r, M - 1) * K + c * EPV
                : Bt + tile_off<T>(n0 + r, c * EPV, K);
    lp[p] = (isa ? r : BM + r) * LDR + c * EPV;
  }

  // offset of k for piece p: the weights' tiles put 16 rows' k side by side
  auto koff = [](int p, int k) __attribute__((always_inline)) {
    return p < NA ? (size_t)k : tile_k(k);
  };

  // Prologue: stage kt0 into LDS buffer 0, stage kt0+1 into registers.
  u32x4 rg[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) rg[p] = *reinterpret_cast<const u32x4*>(gp[p] + koff(p, kt0 * BK));
#pragma unroll
  for (int p = 0; p < NP; ++p) *reinterpret_cast<u32x4*>(&sm[lp[p]]) = rg[p];
  {
    const int k1 = min((kt0 + 1) * BK, klast);
#pragma unroll
    for (int p = 0; p < NP; ++p) rg[p] = *reinterpret_cast<const u32x4*>(gp[p] + koff(p, k1));
  }
  __syncthreads();

  // Fragments are double-buffered: those of k-step ks+1 are read while the
  // MFMAs of k-step ks run.  The next stage's register pieces go to the
  // other LDS buffer during k-steps 0..NSTEP-2 (each freed register then
  // loads its piece of the stage after that); one barrier, placed before the
  // last k-step, publishes the new stage, whose first fragments are read
  // while the last k-step's MFMAs run.
  const int lr = lane & 31, lk = MF::KG * (lane >> 5);
  typename MF::frag af[2][FM], bfr[2][FN];
  auto read_frags = [&](int slot, int buf, int ks) __attribute__((always_inline)) {
    const T* base = sm + buf * (BM + BN) * LDR + ks * MF::KM + lk;
#pragma unroll
    for (int i = 0; i < FM; ++i) af[slot][i] = MF::load(base + (arow + 32 * i + lr) * LDR);
#pragma unroll
    for (int j = 0; j < FN; ++j) bfr[slot][j] = MF::load(base + (brow + 32 * j + lr) * LDR);
  };
  read_frags(0, 0, 0);
  for (int kt = kt0; kt < kt1; ++kt) {
    const int cur = (kt - kt0) & 1;
    const int knext = min((kt + 2) * BK, klast);  // unconditional prefetch (clamped)
    T* const nxt = sm + (cur ^ 1) * (BM + BN) * LDR;
#pragma unroll
    for (int ks = 0; ks < NSTEP; ++ks) {
      const int cb = ks & 1;
      if (ks + 1 < NSTEP) {
        read_frags(cb ^ 1, cur, ks + 1);
      } else {
        __syncthreads();
        read_frags(cb ^ 1, cur ^ 1, 0);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = MF::mma(af[cb][i], bfr[cb][j], acc[i][j]);
      int nw = 0;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (ks + 1 == NSTEP || (p * (NSTEP - 1)) / NP != ks) continue;
        *reinterpret_cast<u32x4*>(&nxt[lp[p]]) = rg[p];
        rg[p] = *reinterpret_cast<const u32x4*>(gp[p] + koff(p, knext));
        ++nw;
      }
      // issue order: one fragment read after each MFMA, then one LDS store
      // and one global load per MFMA, then the remaining MFMAs
      constexpr int nrd = FM + FN < FM * FN ? FM + FN : FM * FN;
#pragma unroll
      for (int q = 0; q < nrd; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        if (q < nw && nrd + q < FM * FN) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
      }
#pragma unroll
      for (int q = 0; q < FM * FN; ++q)
        if (q >= nrd + nw) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  }
  const int ar = wm * WTM, bc = wn * WTN;

  if (KS > 1) {
    // Partial tile -> workspace, row-major [KS][M][N] fp32 (lanes of a row
    // write 32 consecutive columns); summed in split order afterwards.
    float* part = ws + (size_t)kz * M * N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int col = n0 + bc + 32 * j + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + ar + 32 * i + acc_row(r, lane);
          if (row < M) part[(size_t)row * N + col] = acc[i][j][r];
        }
      }
    return;
  }
  epi.template apply<FM, FN>(acc, m0 + ar, n0 + bc, lane, M);
}

// Epilogues with an LDS-staged form (Epi::kStaged) use it in the direct-to-LDS
// kernel, whose stage buffers are free after the main loop.
template <class Epi, class = void>
struct EpiStaged { static constexpr bool value = false; };
template <class Epi>
struct EpiStaged<Epi, std::void_t<decltype(Epi::kStaged)>> { static constexpr bool value = Epi::kStaged; };
template <class Epi>
constexpr bool epi_staged() { return EpiStaged<Epi>::value; }

// ------------------------------------------------- direct-to-LDS bf16 GEMM
// BM x BN output tile per block of NW waves (WGM along M).  The A and W
// k-tiles (64 k = 128 bytes per row) go from memory straight to LDS with the
// direct-to-LDS loads (no staging registers, no LDS store instructions) into
// a ring of NS stages; 16-byte piece c of A's stage row r sits at piece
// c ^ ((r / 2) % 8), which keeps the MFMA fragment reads conflict-free
// without padding; W's tiles keep their layout, in which a fragment read is
// runs of 256 bytes.  One barrier per k-tile, after every wave's last fragment
// reads of the tile; the loads of tile k + NS are issued right after it into
// the stage just consumed, so NS - 1 tiles are in flight while one is
// multiplied.  Fragments of k-step s + LA are read during the MFMAs of
// k-step s (LA = 2 for the 32x64 wave tiles, 1 for 128x64), so the barrier
// comes LA - 1 k-steps before the end of a tile, once the wave has issued
// its last read of it.  Split-K (KS > 1) with EpiNone writes bf16 partials,
// four columns of a row per store (summed in fp32 by resid_norm_kernel);
// with any other epilogue it writes fp32 partials as gemm_kernel does.
// The loads are buffer loads (lds_dma16), and a k-step's fragments are read in
// the order the MFMAs take them, so that the first MFMA waits for two reads,
// not for all: gate/up at 32000 rows 535 -> 515 us, the projections with the
// gated residual 262 -> 255.
//   * 256x256, 8 waves (128x64 wave tiles), 2 stages: large M (batch 64);
//   * 128x128, 8 waves and 64x128, 4 waves (32x64 wave tiles), 3 stages
//     (2 for 128x128 grids of several rounds): medium M (batch 1), where the
//     deeper ring hides the load latency.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {  // at most N vector memory ops outstanding
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
__device__ __forceinline__ void wait_lgkmcnt0() {
  __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
}

template <int BM, int BN, int NW, int WGM, int NS>
constexpr int dma_lds_bytes() {
  return NS * (BM + BN) * 128;
}

struct EpiNone;  // partials only (split-K feeding the fused residual reduction)

template <int BM, int BN, int NW, int WGM, int NS, class Epi>
__global__ __launch_bounds__(64 * NW) void gemm_dma_kernel(const bf16_t* __restrict__ A,
                                                           const bf16_t* __restrict__ Bt, int M,
                                                           int N, int K, int KS,
                                                           float* __restrict__ ws, Epi epi) {
  if (EpiSkip<Epi>::skip(epi)) return;
  constexpr int WGN = NW / WGM, WTM = BM / WGM, WTN = BN / WGN, FM = WTM / 32, FN = WTN / 32;
  constexpr int BK = 64, NSTEP = 4;
  // k-steps whose fragments are read ahead: two for the 32x64 wave tiles,
  // whose two MFMAs per k-step are shorter than an LDS read (QKV at batch 1
  // 10.4 -> 10.2 us); one where a k-step has 8 MFMAs
  constexpr int LA = FM * FN >= 4 ? 1 : 2;
  constexpr int STAGE = (BM + BN) * 128;        // bytes
  constexpr int NI = (BM + BN) * 8 / (64 * NW);  // direct loads per wave per stage
  static_assert(NI * 64 * NW == (BM + BN) * 8 && FM >= 1 && FN >= 1 && NS >= 2, "bad tile");
  extern __shared__ __attribute__((aligned(16))) bf16_t dma_smem[];
  unsigned char* smem = reinterpret_cast<unsigned char*>(dma_smem);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WGM, wn = wave / WGM;
  int tm, tn, kz;
  tile_of(tm, tn, kz);
  // uniform, though divided in vector registers: scalar from here on
  tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn);
  kz = __builtin_amdgcn_readfirstlane(kz);
  const int m0 = tm * BM, n0 = tn * BN;
  const int nk_all = K / BK;
  const int kt0 = (kz * nk_all) / KS, kt1 = ((kz + 1) * nk_all) / KS;

  // lane's piece of each of the wave's loads (load L = NI wave + i of a
  // stage), as byte offsets without k: 8 rows of A, 128 bytes each, or one
  // 1 KB weight tile (16 columns by 32 k; the two of a k-tile side by side),
  // stored as it comes
  const lds_src srca = lds_source(A + (size_t)m0 * K);
  const lds_src srcb = lds_source(Bt + (size_t)n0 * K);
  int off[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int L = NI * wave + i, r = 8 * L + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    off[i] = L < BM / 8 ? 2 * (min(r, M - 1 - m0) * K + 8 * c)
                        : ((L - BM / 8) / 2 * (K / 32) + (L & 1)) * 1024 + 16 * lane;
  }
  auto issue = [&](int kt, int stage) __attribute__((always_inline)) {
    unsigned char* st = smem + stage * STAGE + 1024 * NI * wave;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bool isa = NI * wave + i < BM / 8;
      lds_dma16(isa ? srca : srcb, st + 1024 * i, off[i], kt * (isa ? 128 : 2048));
    }
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};
  const int lr = lane & 31, lg = lane >> 5;
  const int swz = (lr >> 1) & 7;  // rows 32 i + lr of any fragment share it
  const int arow = wm * WTM;
  // column lr of the wave's weight tiles: 16-column group, then column in it
  const int bcol = BM * 64 + (wn * (WTN / 16) + (lr >> 4)) * 1024 + 8 * (lr & 15);
  // fragment slots: the k-step index within the tile when reading LA > 1
  // steps ahead, else alternate
  constexpr int NSL = LA == 1 ? 2 : NSTEP;
  u32x4 af[NSL][FM], bfr[NSL][FN];
  auto read_frags = [&](int slot, int stage, int ks) __attribute__((always_inline)) {
    const bf16_t* st = reinterpret_cast<const bf16_t*>(smem + stage * STAGE);
    const int co = 8 * ((2 * ks + lg) ^ swz);
    auto read_a = [&](int i) __attribute__((always_inline)) {
      af[slot][i] = *reinterpret_cast<const u32x4*>(st + (arow + 32 * i + lr) * 64 + co);
    };
    // in the order of use: the first MFMA then waits for two reads, not all
    read_a(0);
#pragma unroll
    for (int j = 0; j < FN; ++j)
      bfr[slot][j] = *reinterpret_cast<const u32x4*>(st + bcol + 2048 * j + 128 * (2 * ks + lg));
#pragma unroll
    for (int i = 1; i < FM; ++i) read_a(i);
  };

#pragma unroll
  for (int p = 0; p < NS; ++p)
    if (kt0 + p < kt1) issue(kt0 + p, p);
  if (kt1 - kt0 >= NS)
    wait_vmcnt<(NS - 1) * NI>();  // tile kt0 landed, the next NS - 1 may be in flight
  else
    wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int p = 0; p < LA; ++p) read_frags(p % NSL, 0, p);
  int stage = 0;
  for (int kt = kt0; kt < kt1; ++kt) {
    const int nstage = stage + 1 == NS ? 0 : stage + 1;
#pragma unroll
    for (int ks = 0; ks < NSTEP; ++ks) {
      const int cb = ks % NSL;
      const int rs = ks + LA;  // k-step read now (rs >= NSTEP: of tile kt + 1)
      if (rs < NSTEP) {
        read_frags(rs % NSL, stage, rs);
      } else {
        if (rs == NSTEP) {
          // this wave's loads of tile kt + 1 landed (later ones may still
          // fly) and its reads of tile kt, all issued by now, completed; after
          // the barrier both hold for every wave, and this stage is free for
          // tile kt + NS
          if (kt + NS - 1 < kt1)
            wait_vmcnt<(NS - 2) * NI>();
          else
            wait_vmcnt<0>();
          wait_lgkmcnt0();
          __builtin_amdgcn_s_barrier();
          if (kt + NS < kt1) issue(kt + NS, stage);
        }
        if (kt + 1 < kt1) read_frags(rs % NSL, nstage, rs - NSTEP);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, af[cb][i]), __builtin_bit_cast(bf16x8, bfr[cb][j]),
              acc[i][j], 0, 0, 0);
      if (rs != NSTEP) {  // one fragment read after each MFMA
        constexpr int nrd = FM + FN < FM * FN ? FM + FN : FM * FN;
#pragma unroll
        for (int q = 0; q < nrd; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int q = nrd; q < FM * FN; ++q) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      }
    }
    stage = nstage;
  }
  const int ar = wm * WTM, bc = wn * WTN;
  if (KS > 1) {
    if constexpr (std::is_same<Epi, EpiNone>::value) {
      // partials for the fused residual reduction: bf16, four columns of a
      // row per store (the sum over splits and the residual stay fp32)
      bf16_t* part = reinterpret_cast<bf16_t*>(ws) + (size_t)kz * M * N;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int col = n0 + bc + 32 * j + (lane & 28);
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4 u = quad_rows(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1],
                                      acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3], lane);
            const int row = m0 + ar + 32 * i + 8 * q4 + 4 * (lane >> 5) + (lane & 3);
            if (row < M) store4<bf16_t>(part + (size_t)row * N + col, u[0], u[1], u[2], u[3]);
          }
        }
    } else {
      float* part = ws + (size_t)kz * M * N;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int col = n0 + bc + 32 * j + lr;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = m0 + ar + 32 * i + acc_row(r, lane);
            if (row < M) part[(size_t)row * N + col] = acc[i][j][r];
          }
        }
    }
    return;
  }
  if constexpr (epi_staged<Epi>()) {
    __syncthreads();  // every wave is done with the k-tile stages
    epi.template apply_staged<FM, FN, NW, NS * STAGE>(acc, reinterpret_cast<float*>(smem), m0 + ar,
                                                      n0 + bc, lane, wave, M);
  } else {
    epi.template apply<FM, FN>(acc, m0 + ar, n0 + bc, lane, M);
  }
}

// Sum of the KS split partials of each tile, in split order, followed by the
// epilogue; same block shape and register layout as the GEMM that wrote them.
template <int BM, int BN, int NW, int WGM, class Epi>
__global__ __launch_bounds__(64 * NW) void gemm_reduce_kernel(const float* __restrict__ ws, int M,
                                                              int N, int KS, Epi epi) {
  if (EpiSkip<Epi>::skip(epi)) return;
  constexpr int WGN = NW / WGM;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / 32, FN = WTN / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int row0 = blockIdx.y * BM + wm * WTM, col0 = blockIdx.x * BN + wn * WTN;
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};
  for (int z = 0; z < KS; ++z) {  // split order; loads within a split are independent
    const float* part = ws + (size_t)z * M * N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int col = col0 + 32 * j + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = min(row0 + 32 * i + acc_row(r, lane), M - 1);
          acc[i][j][r] += part[(size_t)row * N + col];
        }
      }
  }
  epi.template apply<FM, FN>(acc, row0, col0, lane, M);
}

// ----------------------------------------------------------------- epilogues
// Raw split partials only (no epilogue, no reduction); the caller reduces them.
struct EpiNone {
  template <int FM, int FN>
  __device__ void apply(f32x16 (&)[FM][FN], int, int, int, int) const {}
};

// Element (i, j, r) of a wave's accumulators sits at
//   row = row0 + 32 i + acc_row(r, lane),   col = col0 + 32 j + lane % 32.

template <typename T>
struct EpiBiasSilu {
  T* out; const float* bias; int ldo;
  const int* skip;  // nullptr, or a flag that skips the launch when set
  __device__ bool skipped() const { return skip && *skip; }
  template <int FM, int FN>
  __device__ void apply(f32x16 (&acc)[FM][FN], int row0, int col0, int lane, int M) const {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = col0 + 32 * j + (lane & 31);
      const float b = bias[col];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + 32 * i + acc_row(r, lane);
          if (row < M) out[(size_t)row * ldo + col] = from_f32<T>(silu_f(acc[i][j][r] + b));
        }
    }
  }
};

struct EpiBiasF32 {
  float* out; const float* bias; int ldo;
  const int* skip;  // nullptr, or a flag that skips the launch when set
  __device__ bool skipped() const { return skip && *skip; }
  template <int FM, int FN>
  __device__ void apply(f32x16 (&acc)[FM][FN], int row0, int col0, int lane, int M) const {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = col0 + 32 * j + (lane & 31);
      const float b = bias[col];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + 32 * i + acc_row(r, lane);
          if (row < M) out[(size_t)row * ldo + col] = acc[i][j][r] + b;
        }
    }
  }
};

template <typename T>
struct EpiQkv {
  QkvArgs<T> a;
  // The query columns of rows of at most two streams, the bulk of the product
  // (rows from row_hi on are the second stream's; pos_lo and pos_hi: rotary
  // position minus row of each).  Table and output addresses are a uniform
  // base and a 32-bit lane offset that moves by uniform steps from row to
  // row: an address of its own per element is a long VALU chain after the
  // main loop (64 streams of 500 tokens, 2 layers, 3047 -> 3000 us together
  // with the attention merge's slots by split count; a batch-1 step unchanged).
  // Rows past M read a clamped table entry and are not stored.
  __device__ __forceinline__ void rotate_q(const f32x16& v0, const f32x16& v1, int row0, int c0,
                                           int lane, int M, int row_hi, int pos_lo,
                                           int pos_hi) const {
    const int dh = a.head_dim, half = dh / 2, qd = a.n_q_heads * dh;
    const int head = c0 / dh, dlo = 32 * ((c0 - head * dh) >> 6) + (lane & 31);
    const int lrow = 4 * (lane >> 5), k4 = lane & 3;
    const char* __restrict__ rcos = reinterpret_cast<const char*>(a.rcos);
    const char* __restrict__ rsin = reinterpret_cast<const char*>(a.rsin);
    const int step = 4 * half;  // bytes of a table row
    const int off_lo = pos_lo * step, off_hi = pos_hi * step;
    const uint32_t off_max = (uint32_t)a.S * step - 4;
    const int lane_off = (row0 + lrow) * step + 4 * dlo;
    float cs[16], sn[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ro = 8 * (r >> 2) + (r & 3);
      const uint32_t off = min(
          (uint32_t)(lane_off + ro * step + (lrow >= row_hi - row0 - ro ? off_hi : off_lo)), off_max);
      cs[r] = *reinterpret_cast<const float*>(rcos + off);
      sn[r] = *reinterpret_cast<const float*>(rsin + off);
    }
    T* qb = a.q + (size_t)row0 * qd + head * dh;  // uniform
    const uint32_t lo = (uint32_t)((lrow + k4) * qd + (dlo & ~3));
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      float y0[4], y1[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * q4 + e;
        y0[e] = v0[r] * cs[r] - v1[r] * sn[r];
        y1[e] = v1[r] * cs[r] + v0[r] * sn[r];
      }
      const f32x4 u0 = quad_rows(y0[0], y0[1], y0[2], y0[3], lane);
      const f32x4 u1 = quad_rows(y1[0], y1[1], y1[2], y1[3], lane);
      if (row0 + 8 * q4 + lrow + k4 >= M) continue;
      T* dst = qb + (size_t)8 * q4 * qd + lo;
      store4<T>(dst, u0[0], u0[1], u0[2], u0[3]);
      store4<T>(dst + half, u1[0], u1[1], u1[2], u1[3]);
    }
  }
  template <int FM, int FN>
  __device__ void apply(f32x16 (&acc)[FM][FN], int row0, int col0, int lane, int M) const {
    static_assert(FN % 2 == 0, "QKV epilogue needs column pairs");
    row0 = __builtin_amdgcn_readfirstlane(row0);  // a wave's rows and columns
    col0 = __builtin_amdgcn_readfirstlane(col0);
    const int dh = a.head_dim, half = dh / 2;
    const int qd = a.n_q_heads * dh, kd = a.n_kv_heads * dh;
    const float* __restrict__ rcos = a.rcos;
    const float* __restrict__ rsin = a.rsin;
    // (stream, arena row) of a token row: b = row / tokens,
    // buffer_row0(len[b]) + row - b tokens.  The wave's rows span at most two
    // streams when tokens >= 32 FM: their two lengths are read once (no
    // per-row lookup ahead of the rotary tables); otherwise every row looks
    // its stream up.
    const int ntok = a.tokens;
    const int b_lo = __builtin_amdgcn_readfirstlane(min(row0, M - 1) / ntok);
    const int b_hi = __builtin_amdgcn_readfirstlane(min(row0 + 32 * FM - 1, M - 1) / ntok);
    const bool two = b_hi - b_lo <= 1;
    const int len_lo = buffer_row0(a.len[b_lo]), len_hi = buffer_row0(a.len[b_hi]);
    const int gap_lo = len_lo - a.len[b_lo], gap_hi = len_hi - a.len[b_hi];
    const int row_hi = b_hi * ntok;
    // rotary position of a token = its arena row minus its stream's alignment gap
    auto gap_of = [&](int b) __attribute__((always_inline)) {
      if (two) return b == b_hi ? gap_hi : gap_lo;
      const int P = a.len[b];
      return buffer_row0(P) - P;
    };
    auto locate = [&](int row) __attribute__((always_inline)) {
      row = min(row, M - 1);
      if (two) {
        const bool hi = row >= row_hi;
        const int b = hi ? b_hi : b_lo;
        return int2{b, (hi ? len_hi : len_lo) + row - b * ntok};
      }
      const int b = row / ntok;
      return int2{b, buffer_row0(a.len[b]) + row - b * ntok};
    };
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int j = 0; j < FN; j += 2) {
        const int c0 = col0 + 32 * j;  // first packed column of the pair group
        if (two && c0 < qd) {
          rotate_q(acc[i][j], acc[i][j + 1], row0 + 32 * i, c0, lane, M, row_hi,
                   a.len[b_lo] - b_lo * ntok, a.len[b_hi] - b_hi * ntok);
          continue;
        }
        int2 rp[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) rp[r] = locate(row0 + 32 * i + acc_row(r, lane));
        if (c0 < qd + kd) {
          const bool isq = c0 < qd;
          const int cc = isq ? c0 : c0 - qd;
          const int head = cc / dh;
          const int dlo = 32 * ((cc - head * dh) >> 6) + (lane & 31);
          float cs[16], sn[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int pos = rp[r].y - gap_of(rp[r].x);
            cs[r] = rcos[(size_t)pos * half + dlo];
            sn[r] = rsin[(size_t)pos * half + dlo];
          }
          // rotated pair (d, d + dh/2) per register, then each group of
          // four rows transposed so a lane writes 4 features of one row
          const int d0 = dlo & ~3, k4 = lane & 3;
          // (stream, arena row) of the row each lane writes (K rows only)
          int2 pw[4];
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            pw[q4] = isq ? int2{0, 0} : locate(row0 + 32 * i + 8 * q4 + 4 * (lane >> 5) + k4);
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            float y0[4], y1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int r = 4 * q4 + e;
              const float x0 = acc[i][j][r], x1 = acc[i][j + 1][r];
              y0[e] = x0 * cs[r] - x1 * sn[r];
              y1[e] = x1 * cs[r] + x0 * sn[r];
            }
            const f32x4 u0 = quad_rows(y0[0], y0[1], y0[2], y0[3], lane);
            const f32x4 u1 = quad_rows(y1[0], y1[1], y1[2], y1[3], lane);
            const int row = row0 + 32 * i + 8 * q4 + 4 * (lane >> 5) + k4;
            if (row >= M) continue;
            T* dst = isq ? a.q + (size_t)row * qd + head * dh
                         : a.karena + (((size_t)pw[q4].x * a.n_kv_heads + head) * a.S + pw[q4].y) * dh;
            store4<T>(dst + d0, u0[0], u0[1], u0[2], u0[3]);
            store4<T>(dst + d0 + half, u1[0], u1[1], u1[2], u1[3]);
          }
        } else {
          // V^T rows: registers 4q..4q+3 of a lane are 4 consecutive tokens,
          // written as one 4-element run when they are valid rows of one stream
          const int cc = c0 - qd - kd;
          const int g = cc / dh, d = cc - g * dh + (lane & 31);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int rowq = row0 + 32 * i + acc_row(4 * q, lane);
            const bool run = rowq + 3 < M && rp[4 * q].x == rp[4 * q + 3].x &&
                             (rp[4 * q].y & 3) == 0;  // aligned 4-element run
            if (run) {
              T* base = a.vtarena + ((size_t)rp[4 * q].x * a.n_kv_heads + g) * dh * a.S + rp[4 * q].y;
              store4<T>(base + (size_t)d * a.S, acc[i][j][4 * q], acc[i][j][4 * q + 1],
                        acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
              store4<T>(base + (size_t)(d + 32) * a.S, acc[i][j + 1][4 * q],
                        acc[i][j + 1][4 * q + 1], acc[i][j + 1][4 * q + 2],
                        acc[i][j + 1][4 * q + 3]);
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int r = 4 * q + e;
                if (rowq + e >= M) continue;
                T* base = a.vtarena + ((size_t)rp[r].x * a.n_kv_heads + g) * dh * a.S + rp[r].y;
                base[(size_t)d * a.S] = from_f32<T>(acc[i][j][r]);
                base[(size_t)(d + 32) * a.S] = from_f32<T>(acc[i][j + 1][r]);
              }
            }
          }
        }
      }
    }
  }
};

struct EpiGatedResid {
  static constexpr bool kStaged = true;
  float* h; const float* mod; int mod_ld, gate_off, chunk_len, ldh;
  const int* period;  // FiLM-row sharing flag (film_row), or nullptr
  // Direct-to-LDS kernels: the accumulators go through the (idle) LDS so that
  // h is read and written as whole-row 16-byte pieces, in passes of PI
  // 32-row slabs per wave; `smem` holds NW x PI x 32 x WTN floats.
  template <int FM, int FN, int NW, int LDS_BYTES>
  __device__ void apply_staged(f32x16 (&acc)[FM][FN], float* smem, int row0, int col0, int lane,
                               int wave, int M) const {
    constexpr int WTN = 32 * FN;
    constexpr int PI_MAX = LDS_BYTES / (NW * 32 * WTN * 4);
    constexpr int PI = PI_MAX >= FM ? FM : (PI_MAX >= 2 && FM % 2 == 0 ? 2 : 1);
    static_assert(PI >= 1 && FM % PI == 0, "staging does not fit");
    constexpr int C4 = WTN / 4;                // 16-byte pieces per row
    constexpr int PER = PI * 32 * C4 / 64;     // pieces per lane and pass
    const int per = film_period(period);
    float* cs = smem + wave * PI * 32 * WTN;
    float* __restrict__ hh = h;
    const float* __restrict__ mm = mod;
#pragma unroll
    for (int i0 = 0; i0 < FM; i0 += PI) {
      if (i0 > 0) __syncthreads();  // every wave done reading the last pass
#pragma unroll
      for (int ii = 0; ii < PI; ++ii)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            cs[(32 * ii + acc_row(r, lane)) * WTN + 32 * j + (lane & 31)] = acc[i0 + ii][j][r];
      __syncthreads();
#pragma unroll
      for (int q0 = 0; q0 < PER; q0 += 8) {
        f32x4 hv[8], gv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {  // independent loads first
          if (q0 + q >= PER) break;
          const int idx = (q0 + q) * 64 + lane, rr = idx / C4, c4 = idx - rr * C4;
          const int row = min(row0 + 32 * i0 + rr, M - 1);
          hv[q] = *reinterpret_cast<const f32x4*>(hh + (size_t)row * ldh + col0 + 4 * c4);
          const size_t mrow = (size_t)film_row(row / chunk_len, per) * mod_ld;
          gv[q] = *reinterpret_cast<const f32x4*>(mm + mrow + gate_off + col0 + 4 * c4);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (q0 + q >= PER) break;
          const int idx = (q0 + q) * 64 + lane, rr = idx / C4, c4 = idx - rr * C4;
          const int row = row0 + 32 * i0 + rr;
          const f32x4 a4 = *reinterpret_cast<const f32x4*>(cs + rr * WTN + 4 * c4);
          if (row < M)
            *reinterpret_cast<f32x4*>(hh + (size_t)row * ldh + col0 + 4 * c4) = hv[q] + gv[q] * a4;
        }
      }
    }
  }
  template <int FM, int FN>
  __device__ void apply(f32x16 (&acc)[FM][FN], int row0, int col0, int lane, int M) const {
    const int per = film_period(period);
    float* __restrict__ hh = h;
    const float* __restrict__ mm = mod;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int col = col0 + 32 * j + (lane & 31);
        float hv[16], gv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {  // independent loads first
          const int row = min(row0 + 32 * i + acc_row(r, lane), M - 1);
          hv[r] = hh[(size_t)row * ldh + col];
          gv[r] = mm[(size_t)film_row(row / chunk_len, per) * mod_ld + gate_off + col];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + 32 * i + acc_row(r, lane);
          if (row < M) hh[(size_t)row * ldh + col] = hv[r] + gv[r] * acc[i][j][r];
        }
      }
  }
};

template <typename T>
struct EpiGeglu {
  T* out; int ldo;
  template <int FM, int FN>
  __device__ void apply(f32x16 (&acc)[FM][FN], int row0, int col0, int lane, int M) const {
    static_assert(FN % 2 == 0, "GeGLU epilogue needs column pairs");
    const bool vec = (ldo & 3) == 0;
#pragma unroll
    for (int j = 0; j < FN; j += 2) {
      const int col = ((col0 + 32 * j) >> 1) + (lane & 28);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            y[e] = gelu_tanh_f(acc[i][j][4 * q4 + e]) * acc[i][j + 1][4 * q4 + e];
          const f32x4 u = quad_rows(y[0], y[1], y[2], y[3], lane);
          const int row = row0 + 32 * i + 8 * q4 + 4 * (lane >> 5) + (lane & 3);
          if (row < M) store_quad<T>(out + (size_t)row * ldo + col, u, vec);
        }
    }
  }
};

template <typename T>
struct EpiGelu {
  T* out; int ldo;
  template <int FM, int FN>
  __device__ void apply(f32x16 (&acc)[FM][FN], int row0, int col0, int lane, int M) const {
    const bool vec = (ldo & 3) == 0;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = col0 + 32 * j + (lane & 28);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = gelu_tanh_f(acc[i][j][4 * q4 + e]);
          const f32x4 u = quad_rows(y[0], y[1], y[2], y[3], lane);
          const int row = row0 + 32 * i + 8 * q4 + 4 * (lane >> 5) + (lane & 3);
          if (row < M) store_quad<T>(out + (size_t)row * ldo + col, u, vec);
        }
    }
  }
};

// ------------------------------------------ few-row GEMM, weights streamed
// out[m][n] = sum_k A[m][k] W[n][k] + bias[n] in fp32, bf16 operands, for
// M <= 16 rows and a weight matrix far larger than the memory-side cache
// (the FiLM maps of every norm at small batch), so the kernel is a stream of
// the weights at HBM rate.  A wave owns 16 output columns at a time, whose
// weight tiles are one contiguous range, and multiplies them with MFMA
// 16x16x32 tiles: a 128-element k batch is four tiles, each one contiguous
// 1 KB load.  A stays in registers.  The weight pieces of
// the next three batches (across the end of a column group, the next
// group's first three) are in flight while one batch is multiplied.
constexpr int kStreamRows = 16;
template <int NB>
__global__ __launch_bounds__(256) void stream_bias_f32_kernel(const bf16_t* __restrict__ A,
                                                              const bf16_t* __restrict__ Bt,
                                                              const float* __restrict__ bias,
                                                              float* __restrict__ out, int M,
                                                              int N, const int* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int K = 128 * NB, R = 4, AHEAD = 3;  // ring slots; batches in flight
  static_assert(NB % R == 0 && AHEAD < R, "ring");
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int G = N / 16, stride = gridDim.x * 4;
  int g = blockIdx.x + gridDim.x * (threadIdx.x >> 6);
  if (g >= G) return;  // whole waves
  // rows m >= M repeat row M - 1: every load is in bounds and unconditional,
  // and those rows are never stored
  bf16x8 a[NB][4];
  const bf16_t* arow = A + (size_t)min(c, M - 1) * K + 8 * q;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int p = 0; p < 4; ++p)
      a[b][p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(arow + 128 * b + 32 * p));
  auto wrow = [&](int gg) { return Bt + (size_t)16 * gg * K + 8 * lane; };
  const bf16_t* cur = wrow(g);
  u16x8 w[R][4];
#pragma unroll
  for (int b = 0; b < AHEAD; ++b)
#pragma unroll
    for (int p = 0; p < 4; ++p) w[b][p] = *reinterpret_cast<const u16x8*>(cur + 2048 * b + 512 * p);
  for (;;) {
    // the last group's look-ahead re-reads its own first batches (cache
    // hits) instead of another group's weights
    const bf16_t* nxt = g + stride < G ? wrow(g + stride) : cur;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int ib = b + AHEAD;
      const bf16_t* src = ib < NB ? cur + 2048 * ib : nxt + 2048 * (ib - NB);
#pragma unroll
      for (int p = 0; p < 4; ++p) w[ib % R][p] = *reinterpret_cast<const u16x8*>(src + 512 * p);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < 4; ++p)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[b][p], __builtin_bit_cast(bf16x8, w[b % R][p]),
                                                      acc, 0, 0, 0);
    }
    const int n = 16 * g + c;
    const float bn = bias[n];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 4 * q + r;
      if (m < M) out[(size_t)m * N + n] = acc[r] + bn;
    }
    g += stride;
    if (g >= G) break;
    cur = nxt;
  }
}

template <int NB>
void launch_stream_bias_f32(const bf16_t* A, const bf16_t* Bt, const float* bias, float* out,
                            int M, int N, hipStream_t s, const int* skip) {
  // one workgroup of four waves per CU, every wave about G / 1024 column
  // groups (a cold read of the FiLM weights: 48.5 us against 50.4 with two
  // workgroups per CU, and 46.6 for a plain streaming read of the same bytes)
  const int G = N / 16, blocks = std::min(256, (G + 3) / 4);
  hipLaunchKernelGGL((stream_bias_f32_kernel<NB>), dim3(blocks), dim3(256), 0, s, A, Bt, bias, out,
                     M, N, skip);
}

// -------------------------------------------------------------- tile choice
// Tile shapes (BM x BN, waves); every wave owns a sub-tile at least 64
// columns wide, so paired epilogues find both partners of a 64-column pair
// group in one wave.
enum Tile { T256x128w8 = 0, T128x128w8 = 1, T64x128w4 = 2, T256x256big = 3, TFew = 4 };
constexpr int kTileBM[] = {256, 128, 64, 256};
constexpr int kTileBN[] = {128, 128, 128, 256};

template <typename T, int BM, int BN, int NW, int WGM, class Epi>
void launch_tile(const T* A, const T* Bt, int M, int N, int K, const GemmPlan& p,
                 const GemmWork& w, const Epi& epi, hipStream_t s) {
  dim3 grid(N / BN, (M + BM - 1) / BM, p.ks);
  hipLaunchKernelGGL((gemm_kernel<T, BM, BN, NW, WGM, Epi>), grid, dim3(64 * NW), 0, s, A, Bt, M,
                     N, K, p.ks, w.ws, epi);
  if (p.ks > 1 && !std::is_same<Epi, EpiNone>::value)
    hipLaunchKernelGGL((gemm_reduce_kernel<BM, BN, NW, WGM, Epi>), dim3(grid.x, grid.y),
                       dim3(64 * NW), 0, s, w.ws, M, N, p.ks, epi);
}

// Direct-to-LDS instances: (tile, waves, stages) of the bf16 tiles that use it.
#define FV_DMA_TILES(X) \
  X(256, 256, 8, 2, 2)  \
  X(128, 128, 8, 4, 3)  \
  X(128, 128, 8, 4, 2)  \
  X(64, 128, 4, 2, 3)

template <int BM, int BN, int NW, int WGM, int NS, class Epi>
hipError_t allow_dma_lds() {
  return hipFuncSetAttribute(
      reinterpret_cast<const void*>(&gemm_dma_kernel<BM, BN, NW, WGM, NS, Epi>),
      hipFuncAttributeMaxDynamicSharedMemorySize, dma_lds_bytes<BM, BN, NW, WGM, NS>());
}

template <int BM, int BN, int NW, int WGM, int NS, class Epi>
void launch_dma(const bf16_t* A, const bf16_t* Bt, int M, int N, int K, const GemmPlan& p,
                const GemmWork& w, const Epi& epi, hipStream_t s) {
  dim3 grid(N / BN, (M + BM - 1) / BM, p.ks);
  hipLaunchKernelGGL((gemm_dma_kernel<BM, BN, NW, WGM, NS, Epi>), grid, dim3(64 * NW),
                     (dma_lds_bytes<BM, BN, NW, WGM, NS>()), s, A, Bt, M, N, K, p.ks, w.ws, epi);
  // the 256x256 tile never splits k (plan_gemm), so it has no reduction
  if constexpr (BM * BN < 256 * 256 && !std::is_same<Epi, EpiNone>::value)
    if (p.ks > 1)
      hipLaunchKernelGGL((gemm_reduce_kernel<BM, BN, NW, WGM, Epi>), dim3(grid.x, grid.y),
                         dim3(64 * NW), 0, s, w.ws, M, N, p.ks, epi);
}

// Launches the tile kernel of plan p (not TFew).  The 128x128 tile of the
// direct-to-LDS kernel takes three stages when the grid fits the chip with one
// workgroup per CU (the deeper ring hides load latency, measured 1568 against
// 1864 us per batch-1 step with two), two stages otherwise (two workgroups
// then fit per CU and overlap each other).
template <typename T, class Epi>
void run_tile(const T* A, const T* Bt, int M, int N, int K, const GemmPlan& p, const GemmWork& w,
              const Epi& epi, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    if (p.dma) {
      const bool rounds = (long)p.tiles * p.ks > 256;
      switch (p.tile) {
        case T256x256big: return launch_dma<256, 256, 8, 2, 2>(A, Bt, M, N, K, p, w, epi, s);
        case T128x128w8:
          return rounds ? launch_dma<128, 128, 8, 4, 2>(A, Bt, M, N, K, p, w, epi, s)
                        : launch_dma<128, 128, 8, 4, 3>(A, Bt, M, N, K, p, w, epi, s);
        case T64x128w4: return launch_dma<64, 128, 4, 2, 3>(A, Bt, M, N, K, p, w, epi, s);
      }
    }
  }
  switch (p.tile) {
    case T256x128w8: return launch_tile<T, 256, 128, 8, 4>(A, Bt, M, N, K, p, w, epi, s);
    case T128x128w8: return launch_tile<T, 128, 128, 8, 4>(A, Bt, M, N, K, p, w, epi, s);
    case T64x128w4: return launch_tile<T, 64, 128, 4, 2>(A, Bt, M, N, K, p, w, epi, s);
  }
  throw std::logic_error("GEMM plan without a tile kernel");
}

template <typename T, class Epi>
void run_gemm(const T* A, const T* Bt, int M, int N, int K, const GemmWork& w, const Epi& epi,
              hipStream_t s) {
  if (M > 0) run_tile(A, Bt, M, N, K, plan_gemm(M, N, K, sizeof(T) == 2), w, epi, s);
}

}  // namespace

namespace {

// Tile by row count: large M takes 256x256 tiles (fewer re-reads of A and
// W) when that still gives about 200 blocks and no mostly idle second round,
// else 128x128 (bf16; two workgroups per CU); medium M takes 128x128 tiles
// when that still gives about 200 blocks (96 for an output or down
// projection), else 64x128.  ks is the widest split: where a grid has fewer
// than 128 tiles, a power of two with at least 4 k-tiles per split and at
// most about 320 blocks, so that every CU streams its share of the weights;
// with `reduce_fused` (the output and down projections, whose split sum is
// fused into the next kernel at no extra launch) also for grids of up to 160
// tiles.
GemmPlan tile_plan(int M, int N, int K, bool bf16, bool reduce_fused) {
  GemmPlan p;
  if (N % 128 || M <= 0) return p;
  const int bk = bf16 ? 64 : 32, nk = K / bk;
  auto ntiles = [&](int t) { return ((M + kTileBM[t] - 1) / kTileBM[t]) * (N / kTileBN[t]); };
  // 256x256 tiles run one workgroup per CU, 128x128 tiles two.  A grid of
  // two rounds of 256x256 tiles whose second round is mostly idle (under 72
  // of 256 tiles) takes 128x128 tiles instead: measured per step, batch 16
  // (QKV, 64 tiles in round two) 7.82 -> 7.67 ms, batch 36 (output and
  // down projections, 28) 17.67 -> 17.00, batch 40 (60) 19.03 -> 18.73;
  // slower at batch 44 (88) and 48 (120).  Two full rounds are best on
  // 256x256 tiles, also below 4096 rows (4000 rows, gate/up 83.6 -> 73.1 us).
  const long n256 = ntiles(T256x256big);
  // the direct-to-LDS kernel's byte offsets (512 K) are 32-bit
  const bool dma = bf16 && K < 1 << 22;
  if (dma && M >= 2048 && N % 256 == 0 && n256 >= 200 && !(n256 > 256 && n256 < 328)) {
    p.tile = T256x256big;
  } else if (M >= 4096) {
    p.tile = bf16 && N % 256 == 0 ? T128x128w8 : T256x128w8;
  } else if (M > 256) {
    // (an output or down projection takes 128x128 tiles from 96 of them on:
    // with k split in two they beat 64x128 tiles, batch 3 2790 -> 2722 us)
    // 128x128 from 200 tiles on, except narrow products whose 64x128 tiles fit
    // one round of two workgroups per CU where the 128x128 tiles hardly fill
    // theirs or just pass it (4-layer passes, 128x128 / 64x128: QKV at 1155
    // rows, 200 tiles, 514 / 502 us; a plain MLP's up product at 1300 rows,
    // 264 tiles, 352 / 342).  In between the larger tiles read less: QKV at
    // 1300 rows, 220 tiles, 507 / 520; 4096 columns of gate/up at 1000 rows,
    // 256 tiles, 291 / 295.  N > K leaves out the projections back to the
    // width (8 streams of 500 tokens: 1020 us on 128x128 tiles, 1067 on
    // 64x128).
    const int t128 = ntiles(T128x128w8);
    const bool narrow = bf16 && N > K && N <= 4096 && ntiles(T64x128w4) <= 512 &&
                        (t128 <= 208 || t128 > 256);
    if (reduce_fused && bf16 && t128 >= 96)
      p.tile = T128x128w8;
    else
      p.tile = t128 >= 200 && !narrow ? T128x128w8 : T64x128w4;
  } else {
    p.tile = T64x128w4;
  }
  p.dma = dma && p.tile != T256x128w8;
  p.tiles = ntiles(p.tile);
  p.ks = 1;
  if ((p.tiles < 128 || (reduce_fused && p.tiles <= 160)) && p.tile != T256x256big)
    while ((long)p.tiles * p.ks * 2 <= 320 && nk / (p.ks * 2) >= 4 && p.ks < 8) p.ks *= 2;
  return p;
}

// Split of a bf16 product whose partials take a reduction kernel of their own:
// the power of two up to `widest` that costs least, in us.  A k-tile takes
// 0.30; a reduction 3.7 for two splits and 4.6 for more, 0.45 per MB of
// partials, and 2 where the split grid passes one workgroup per CU (a launch,
// unsplit / split in 4: gate/up of 384 columns at 80 rows and k 1920
// 12.2 / 10.4, QKV of 512 columns at 80 rows and k 1792 13.6 / 12.5; of 2560
// columns at 192 rows and k 1024 10.7 / 15.3).
int cheapest_split(int M, int N, int nk, int tiles, int widest) {
  const double mb = 4e-6 * M * N;
  int best = 1;
  double least = 0.30 * nk;
  for (int ks = 2; ks <= widest; ks *= 2) {
    const double t = 0.30 * nk / ks + (ks == 2 ? 3.7 : 4.6) + 0.45 * mb * ks +
                     ((long)tiles * ks > 256 ? 2.0 : 0.0);
    if (t < least) {
      best = ks;
      least = t;
    }
  }
  return best;
}

}  // namespace

GemmPlan plan_gemm(int M, int N, int K, bool bf16, bool reduce_fused) {
  GemmPlan p;
  if (N % 128 == 0 && M > 0 && few_rows(M)) {
    p.tile = TFew;
    p.ks = reduce_fused ? few_splits(N, K, bf16 ? 2 : 4) : 1;
    p.tiles = N / 16;
    p.ws_floats = reduce_fused ? (size_t)p.ks * M * N : 0;
    return p;
  }
  p = tile_plan(M, N, K, bf16, reduce_fused);
  // (fp32 k-tiles take 1.2 us: the widest split, 416 us against 452 without
  // for 4 layers of width 512 at 400 rows)
  if (bf16 && !reduce_fused) p.ks = cheapest_split(M, N, K / 64, p.tiles, p.ks);
  p.ws_floats = p.ks > 1 ? (size_t)p.ks * M * N : 0;
  return p;
}

size_t widest_split_floats(int M, int N, int K, bool bf16, bool reduce_fused) {
  const GemmPlan p = tile_plan(M, N, K, bf16, reduce_fused);
  return p.ks > 1 ? (size_t)p.ks * M * N : 0;
}

template <typename T>
int gemm_partials(const T* A, const T* Bt, int M, int N, int K, const GemmWork& w,
                  hipStream_t s, bool* bf16_parts) {
  const GemmPlan p = plan_gemm(M, N, K, sizeof(T) == 2, true);
  *bf16_parts = gemm_partials_bf16(p);
  if (p.tile == TFew)
    few_partials(A, Bt, w.ws, M, N, K, p.ks, s);
  else if (p.ks > 1)
    run_tile(A, Bt, M, N, K, p, w, EpiNone{}, s);
  return p.ks;
}

template <typename T>
void gemm_bias_silu(const T* A, const T* Bt, const float* bias, T* out, int M, int N, int K,
                    const GemmWork& w, hipStream_t s, const int* skip) {
  if (few_rows(M)) return few_bias_silu(A, Bt, bias, out, M, N, K, s, skip);
  run_gemm(A, Bt, M, N, K, w, EpiBiasSilu<T>{out, bias, N, skip}, s);
}
template <typename T>
void gemm_bias_f32(const T* A, const T* Bt, const float* bias, float* out, int M, int N, int K,
                   const GemmWork& w, hipStream_t s, const int* skip) {
  if constexpr (sizeof(T) == 2) {
    if (M <= kStreamRows && N % 16 == 0) {
      switch (K) {
        case 512: launch_stream_bias_f32<4>(A, Bt, bias, out, M, N, s, skip); return;
        case 1024: launch_stream_bias_f32<8>(A, Bt, bias, out, M, N, s, skip); return;
        default: break;
      }
    }
  }
  // Every workgroup of the one-pass kernel reads all rows of A, so past 32 rows
  // a wide product (the FiLM maps of more than a few layers) is faster on the
  // tiles, one row tile and no split (bf16, width 1024, 64 rows: 18 layers, 112640
  // columns, 86 us one-pass, 46 on tiles; 8192 columns 7.5 / 11.1; width 512,
  // 13312 columns, 9.1 / 9.1 at 48 rows).
  const bool wide = M > 32 && N > 16384;
  if (few_rows(M) && !wide) return few_bias_f32(A, Bt, bias, out, M, N, K, s, skip);
  const GemmPlan p = few_rows(M) ? tile_plan(M, N, K, sizeof(T) == 2, false)
                                 : plan_gemm(M, N, K, sizeof(T) == 2);
  run_tile(A, Bt, M, N, K, p, w, EpiBiasF32{out, bias, N, skip}, s);
}
template <typename T>
void gemm_qkv(const T* A, const T* Bt, const QkvArgs<T>& qa, int M, int N, int K,
              const GemmWork& w, hipStream_t s) {
  if (few_rows(M)) return few_qkv(A, Bt, qa, M, N, K, s);
  run_gemm(A, Bt, M, N, K, w, EpiQkv<T>{qa}, s);
}
template <typename T>
void gemm_gated_resid(const T* A, const T* Bt, float* h, const float* mod, int mod_ld,
                      int gate_off, int chunk_len, int M, int N, int K, const GemmWork& w,
                      hipStream_t s, const int* period) {
  run_gemm(A, Bt, M, N, K, w, EpiGatedResid{h, mod, mod_ld, gate_off, chunk_len, N, period}, s);
}
template <typename T>
void gemm_geglu(const T* A, const T* Bt, T* out, int M, int N, int K, const GemmWork& w,
                hipStream_t s) {
  if (few_rows(M)) return few_geglu(A, Bt, out, M, N, K, s);
  run_gemm(A, Bt, M, N, K, w, EpiGeglu<T>{out, N / 2}, s);
}
template <typename T>
void gemm_gelu(const T* A, const T* Bt, T* out, int M, int N, int K, const GemmWork& w,
               hipStream_t s) {
  if (few_rows(M)) return few_gelu(A, Bt, out, M, N, K, s);
  run_gemm(A, Bt, M, N, K, w, EpiGelu<T>{out, N}, s);
}

// The direct-to-LDS kernels' dynamic LDS exceeds the default limit; every
// (tile, epilogue) instance is raised once per device before any launch.
template <class Epi>
hipError_t allow_dma_all() {
  hipError_t e = hipSuccess;
#define FV_ALLOW(BM, BN, NW, WGM, NS) \
  if (e == hipSuccess) e = allow_dma_lds<BM, BN, NW, WGM, NS, Epi>();
  FV_DMA_TILES(FV_ALLOW)
#undef FV_ALLOW
  return e;
}

hipError_t gemm_prepare() {
  const hipError_t e[] = {allow_dma_all<EpiBiasSilu<bf16_t>>(), allow_dma_all<EpiBiasF32>(),
                          allow_dma_all<EpiQkv<bf16_t>>(),      allow_dma_all<EpiGatedResid>(),
                          allow_dma_all<EpiGeglu<bf16_t>>(),    allow_dma_all<EpiGelu<bf16_t>>(),
                          allow_dma_all<EpiNone>()};
  for (hipError_t x : e)
    if (x != hipSuccess) return x;
  return hipSuccess;
}

#define FV_INSTANTIATE(T)                                                                        \
  template void gemm_bias_silu<T>(const T*, const T*, const float*, T*, int, int, int,           \
                                  const GemmWork&, hipStream_t, const int*);                     \
  template void gemm_bias_f32<T>(const T*, const T*, const float*, float*, int, int, int,        \
                                 const GemmWork&, hipStream_t, const int*);                      \
  template void gemm_qkv<T>(const T*, const T*, const QkvArgs<T>&, int, int, int,                \
                            const GemmWork&, hipStream_t);                                       \
  template void gemm_gated_resid<T>(const T*, const T*, float*, const float*, int, int, int,     \
                                    int, int, int, const GemmWork&, hipStream_t, const int*);    \
  template void gemm_geglu<T>(const T*, const T*, T*, int, int, int, const GemmWork&,            \
                              hipStream_t);                                                      \
  template void gemm_gelu<T>(const T*, const T*, T*, int, int, int, const GemmWork&, hipStream_t); \
  template int gemm_partials<T>(const T*, const T*, int, int, int, const GemmWork&, hipStream_t, \
                                bool*);
FV_INSTANTIATE(bf16_t)
FV_INSTANTIATE(float)
#undef FV_INSTANTIATE

}  // namespace fv
