// fp32 GEMM on v_mfma_f32_32x32x2_f32 for gfx950 (storage type SK_F32), the accuracy path
// of the library.  Same contract as the bf16 GEMM.  4 waves as 2 x 2; a wave owns T x T MFMA
// blocks of 32 x 32: tiles of 64 x 64 (T = 1) or 128 x 128 (T = 2).  k chunks of 32, LDS
// double-buffered.
//
// What bounds it: the matrix pipe (64 cycles per MFMA; hipBLASLt's 8192^3 product reaches
// 153 TFLOP/s on this chip) once the loads are early enough.  A chunk is 16 MFMAs of a 64 x 64
// tile's wave, 1024 cycles, about a trip to far memory, so two register sets keep the loads of the
// chunk two ahead in flight behind the LDS stores of the next one.  A work-group alone on a CU
// still takes 1600 cycles a chunk (one wave per SIMD waits for its own LDS reads and barriers);
// two or more share the pipe at 85 % of its rate, so the planner splits the contraction until
// there are.  Measured, 16-wide chunks with one set of loads in flight -> this kernel:
// [4096 x 3072] . [3072 x 128] 57 -> 34 us (94 TFLOP/s), [4096 x 128] . [128 x 3072] 42 -> 36 us,
// [8192 x 4096] . [4096 x 512] 250-260 us (132-137 TFLOP/s).
//
// Lane layout of v_mfma_f32_32x32x2_f32 (D = P . Q), lane l:
//   P: row l % 32, k = l / 32;   Q: col l % 32, k = l / 32;
//   D: col l % 32, rows 8 * (r / 4) + 4 * (l / 32) + r % 4, r = 0..15.
// Which k of a chunk an MFMA takes, and which row of the tile a block's row is, is free as long
// as both operands agree and the stores follow, and the LDS reads are cut for it: in a group of
// 8 k the half-wave l / 32 holds k = 4 (l / 32) + 0..3 for four MFMAs, which is one 16-byte
// read of a k-contiguous operand; an operand contiguous along m (n) with two blocks per wave
// gives block i the rows 2 r + i, which makes its read one 8-byte read for both blocks.
#include "sk_bf16_tile.h"
#include "sk_launch.h"

namespace sk {

// One operand chunk, EXT rows (m or n) by F32_BK k; KC: source [ext, K], stored [EXT][F32_BK]
// with 16-byte pieces swizzled by row; otherwise source [K, ext], stored [F32_BK][EXT + 8].
template <int T, bool KC>
struct F32Chunk {
  static constexpr int EXT = 64 * T;
  static constexpr int LD = KC ? F32_BK : EXT + 8;   // (k rows 4 apart, read together, 32 banks apart)
  static constexpr int ELEMS = KC ? EXT * F32_BK : F32_BK * LD;
  static constexpr int PPR = (KC ? F32_BK : EXT) / 4;           // 16-byte pieces of a row
  static constexpr int PIECES = EXT * F32_BK / 4 / 256;         // per thread
  static __device__ __forceinline__ int piece_of(int row, int pc) { return KC ? pc ^ ((row >> 1) & 7) : pc; }

  // Global -> registers, branch free: everything outside the matrix or the k range reads as zero.
  static __device__ __forceinline__ void load(uint4 (&r)[PIECES], const float* __restrict__ g, int64_t ld,
                                              int e0, int e_total, int k0, int k_end, int k_total, int tid) {
    const int64_t rows = KC ? e_total : k_total;
    const GWindow w = make_window(g, KC ? (int64_t)e0 * ld + k0 : (int64_t)k0 * ld + e0, rows * ld, 4);
    const unsigned ldb = (unsigned)ld * 4u;
#pragma unroll
    for (int v = 0; v < PIECES; ++v) {
      const int q = v * 256 + tid, row = q / PPR, col = (q % PPR) * 4;
      const bool ok = KC ? k0 + col < k_end : (e0 + col < e_total && k0 + row < k_end);
      r[v] = window_load16(w, ok ? (unsigned)row * ldb + (unsigned)col * 4u : OOB_OFFSET);
    }
  }
  static __device__ __forceinline__ void store(float* tile, const uint4 (&r)[PIECES], int tid) {
#pragma unroll
    for (int v = 0; v < PIECES; ++v) {
      const int q = v * 256 + tid, row = q / PPR;
      *reinterpret_cast<uint4*>(tile + row * LD + piece_of(row, q % PPR) * 4) = r[v];
    }
  }
  // f[i][j]: block i's operand value for MFMA j of k group g (8 k); w: index of the wave's 32 T rows
  static __device__ __forceinline__ void read(float (&f)[T][4], const float* tile, int w, int g, int lane) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int row = (w * T + i) * 32 + (lane & 31);
        const float4 v = *reinterpret_cast<const float4*>(tile + row * LD + piece_of(row, g * 2 + (lane >> 5)) * 4);
        f[i][0] = v.x; f[i][1] = v.y; f[i][2] = v.z; f[i][3] = v.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float* p = tile + (g * 8 + (lane >> 5) * 4 + j) * LD + (w * 32 + (lane & 31)) * T;
        if constexpr (T == 2) {
          const float2 v = *reinterpret_cast<const float2*>(p);
          f[0][j] = v.x; f[1][j] = v.y;
        } else {
          f[0][j] = *p;
        }
      }
    }
  }
  // row (column) of the wave's 32 T that row r of block i is
  static __device__ __forceinline__ int place(int i, int r) { return KC ? i * 32 + r : r * T + i; }
};

// The work of one work-group, index `block` of the product's own; a device function so that one launch
// can carry the work-groups of two products.
template <int T, bool A_KC, bool B_KC, bool COLSUM>
struct F32Tile {
  typedef F32Chunk<T, A_KC> CA;
  typedef F32Chunk<T, B_KC> CB;
  static constexpr int STAGE = CA::ELEMS + CB::ELEMS;
  static __device__ __forceinline__ void run(const GemmArgs& p, int block, float* lds);
};

template <int T, bool A_KC, bool B_KC, bool COLSUM>
__device__ __forceinline__ void F32Tile<T, A_KC, B_KC, COLSUM>::run(const GemmArgs& p, const int block, float* const lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles = p.tiles_m * p.tiles_n;
  const int id = xcd_remap(block, tiles * p.splits);
  const int split = id / tiles;
  int tile_m, tile_n;
  tile_coords(id - split * tiles, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * CA::EXT, n0 = tile_n * CB::EXT;
  const int k_begin = split * p.k_per_split;
  const int k_end = (k_begin + p.k_per_split < p.K) ? k_begin + p.k_per_split : p.K;
  const float* __restrict__ A = static_cast<const float*>(p.A);
  const float* __restrict__ B = static_cast<const float*>(p.B);

  f32x16 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // Column sums of B ride on the vector ALU, which the MFMAs leave idle: this lane's k only,
  // the two half-waves are added at the end.  (Every wave forms them, one in two of the first
  // row of tiles writes them: as MFMAs against ones they cost those waves as much as the product.)
  float csum[T];
#pragma unroll
  for (int j = 0; j < T; ++j) csum[j] = 0.f;

  // this lane's bias values, through a window of N elements (none without a bias: zeros)
  const GWindow bias_w = make_window(p.bias, 0, p.bias != nullptr ? p.N : 0, 4);
  float bv[T];
#pragma unroll
  for (int n = 0; n < T; ++n)
    bv[n] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
        bias_w.rsrc, (n0 + wn * 32 * T + CB::place(n, lane & 31)) * 4, 0, 0));

  uint4 ra0[CA::PIECES], rb0[CB::PIECES], ra1[CA::PIECES], rb1[CB::PIECES];
  auto load = [&](uint4 (&a)[CA::PIECES], uint4 (&b)[CB::PIECES], int k0) {   // (past the range: zeros)
    CA::load(a, A, p.lda, m0, p.M, k0, k_end, p.K, tid);
    CB::load(b, B, p.ldb, n0, p.N, k0, k_end, p.K, tid);
  };
  auto store = [&](float* s, const uint4 (&a)[CA::PIECES], const uint4 (&b)[CB::PIECES]) {
    CA::store(s, a, tid);
    CB::store(s + CA::ELEMS, b, tid);
  };
  // The fragments of a k group are read one group ahead of its MFMAs, the first group of the
  // next chunk behind the last MFMAs of the current one (so the barrier sits one group before
  // the end of a chunk); loads, LDS reads and LDS stores are spread between the MFMAs.
  float fa0[T][4], fb0[T][4], fa1[T][4], fb1[T][4];
  auto read = [&](const float* s, int g, float (&a)[T][4], float (&b)[T][4]) {
    CA::read(a, s, wm, g, lane);
    CB::read(b, s + CA::ELEMS, wn, g, lane);
  };
  auto mma = [&](const float (&a)[T][4], const float (&b)[T][4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int n = 0; n < T; ++n)
          acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][j], b[n][j], acc[i][n], 0, 0, 0);
    if (COLSUM) {
#pragma unroll
      for (int n = 0; n < T; ++n) csum[n] += (b[n][0] + b[n][1]) + (b[n][2] + b[n][3]);
    }
  };
  constexpr int NM = 4 * T * T, ND = (A_KC ? T : 4) + (B_KC ? T : 4);
  constexpr int PA = CA::PIECES, PB = CB::PIECES;
  // One chunk: its MFMAs out of `s`, the loads of the chunk two ahead into (la, lb), the next
  // chunk, loaded an iteration ago into (sa, sb), to the other LDS buffer.
  auto iteration = [&](const float* s, float* next, uint4 (&la)[PA], uint4 (&lb)[PB], const uint4 (&sa)[PA],
                       const uint4 (&sb)[PB], int k0) {
    __builtin_amdgcn_sched_barrier(0);
    read(s, 1, fa1, fb1);
    CA::load(la, A, p.lda, m0, p.M, k0 + 2 * F32_BK, k_end, p.K, tid);
    mma(fa0, fb0);
    sched_phase<NM, ND, PA, 0>();
    read(s, 2, fa0, fb0);
    CB::load(lb, B, p.ldb, n0, p.N, k0 + 2 * F32_BK, k_end, p.K, tid);
    mma(fa1, fb1);
    sched_phase<NM, ND, PB, 0>();
    read(s, 3, fa1, fb1);
    store(next, sa, sb);
    mma(fa0, fb0);
    sched_phase<NM, ND, 0, PA + PB>();
    __syncthreads();
    read(next, 0, fa0, fb0);
    mma(fa1, fb1);
    sched_phase<NM, ND, 0, 0>();
  };
  load(ra0, rb0, k_begin);
  load(ra1, rb1, k_begin + F32_BK);
  store(lds, ra0, rb0);
  __syncthreads();
  read(lds, 0, fa0, fb0);
  // (an odd last chunk outside the loop: a way out of its middle makes the compiler wait for every
  // load at the top)
  int k0 = k_begin;
  for (; k0 + F32_BK < k_end; k0 += 2 * F32_BK) {
    iteration(lds, lds + STAGE, ra0, rb0, ra1, rb1, k0);
    iteration(lds + STAGE, lds, ra1, rb1, ra0, rb0, k0 + F32_BK);
  }
  if (k0 < k_end) iteration(lds, lds + STAGE, ra0, rb0, ra1, rb1, k0);

  // Results leave branch free through a window on the rows from m0 on (rows past M fall outside,
  // columns past N are pointed there): under a bounds branch each, every store waited for the
  // one before it.
  const GWindow cw = make_window(p.C, ((int64_t)split * p.M + m0) * p.ldc, (int64_t)(split + 1) * p.M * p.ldc, 4);
  constexpr bool PAIRS = !B_KC && T == 2;   // the wave's two blocks interleave by column: 8-byte stores
  int gn[T];
#pragma unroll
  for (int n = 0; n < T; ++n) gn[n] = n0 + wn * 32 * T + CB::place(n, lane & 31);
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = wm * 32 * T + CA::place(i, 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3));
      float v[T];
#pragma unroll
      for (int n = 0; n < T; ++n) v[n] = acc[i][n][r] * p.scale + bv[n];
      auto off = [&](int n) { return gn[n] < p.N ? (int)(((unsigned)row * (unsigned)p.ldc + (unsigned)gn[n]) * 4u) : (int)OOB_OFFSET; };
      if constexpr (PAIRS) {   // (N is a multiple of 16: both columns or neither)
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 w = {__builtin_bit_cast(unsigned, v[0]), __builtin_bit_cast(unsigned, v[T - 1])};
        __builtin_amdgcn_raw_buffer_store_b64(w, cw.rsrc, off(0), 0, 0);
      } else {
#pragma unroll
        for (int n = 0; n < T; ++n)
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v[n]), cw.rsrc, off(n), 0, 0);
      }
    }
  if (COLSUM) {
    if (p.colsum != nullptr && m0 == 0 && wm == 0) {
      float* out = p.colsum + (int64_t)split * p.N;
#pragma unroll
      for (int n = 0; n < T; ++n) {
        const float s = csum[n] + __shfl_xor(csum[n], 32);
        if (lane < 32 && gn[n] < p.N) out[gn[n]] = s;
      }
    }
  }
}

template <int T, bool A_KC, bool B_KC, bool COLSUM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmArgs p) {
  typedef F32Tile<T, A_KC, B_KC, COLSUM> G;
  __shared__ __attribute__((aligned(16))) float lds[2 * G::STAGE];
  G::run(p, blockIdx.x, lds);
}

// Two independent products in one launch: the first groups_a work-groups are GA's on `a`, the rest
// GB's on `b`.  The backward pass has two such pairs, and each has a partner that leaves most of the
// chip idle by itself or is over in a launch's own time.
template <class GA, class GB>
__global__ __launch_bounds__(256) void dual_gemm_f32_kernel(const GemmArgs a, const GemmArgs b, const int groups_a) {
  __shared__ __attribute__((aligned(16))) float lds[2 * (GA::STAGE > GB::STAGE ? GA::STAGE : GB::STAGE)];
  if ((int)blockIdx.x < groups_a) GA::run(a, blockIdx.x, lds);
  else GB::run(b, (int)blockIdx.x - groups_a, lds);
}

template <int T, bool A_KC, bool B_KC, bool COLSUM>
static hipError_t launch_one(GemmArgs a, hipStream_t s) {
  a.tiles_m = (a.M + 64 * T - 1) / (64 * T);
  a.tiles_n = (a.N + 64 * T - 1) / (64 * T);
  const long long grid = (long long)a.tiles_m * a.tiles_n * a.splits;
  if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  // (the result is always addressed as slabs [M, ldc], one per k range: one slab when not split)
  note_gemm(a, A_KC, B_KC, 4, 4, true);
  static const std::string name =
      kernel_label("gemm_f32_kernel", {lbl(T), lbl(A_KC), lbl(B_KC), lbl(COLSUM)});
  return launch_kernel(name.c_str(), gemm_work(a, 4, 4, true), gemm_f32_kernel<T, A_KC, B_KC, COLSUM>,
                       dim3((unsigned)grid), dim3(256), s, a);
}

template <bool A_KC, bool B_KC, bool COLSUM>
static hipError_t launch_tiles(int tile, const GemmArgs& a, hipStream_t s) {
  switch (tile) {
    case TILE_64x64: return launch_one<1, A_KC, B_KC, COLSUM>(a, s);
    case TILE_128x128: return launch_one<2, A_KC, B_KC, COLSUM>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_f32(GemmKind kind, int tile, const GemmArgs& a, hipStream_t s) {
  switch (kind) {
    case GEMM_NN: return launch_tiles<true, false, false>(tile, a, s);
    case GEMM_NT: return launch_tiles<true, true, false>(tile, a, s);
    case GEMM_TN_F32: return launch_tiles<false, false, true>(tile, a, s);
    default: return hipErrorInvalidValue;
  }
}

template <class GA, class GB>
static hipError_t launch_pair(int T, GemmArgs a, GemmArgs b, Work work, hipStream_t s) {
  for (GemmArgs* g : {&a, &b}) {
    g->tiles_m = (g->M + 64 * T - 1) / (64 * T);
    g->tiles_n = (g->N + 64 * T - 1) / (64 * T);
  }
  const long long ga = (long long)a.tiles_m * a.tiles_n * a.splits, gb = (long long)b.tiles_m * b.tiles_n * b.splits;
  if (ga <= 0 || gb <= 0 || ga + gb > 0x7fffffffLL) return hipErrorInvalidValue;
  return launch_kernel("dual_gemm_f32_kernel", work, dual_gemm_f32_kernel<GA, GB>, dim3((unsigned)(ga + gb)), dim3(256), s, a, b, (int)ga);
}

hipError_t launch_dual_gemm_f32(GemmKind kind_a, const GemmArgs& a, GemmKind kind_b, const GemmArgs& b, int tile, hipStream_t s) {
  bool akc, bkc, f32;
  gemm_kind_traits(kind_a, akc, bkc, f32);
  note_gemm(a, akc, bkc, 4, 4, true);
  gemm_kind_traits(kind_b, akc, bkc, f32);
  note_gemm(b, akc, bkc, 4, 4, true);
  Work work = gemm_work(a, 4, 4, true);
  const Work wb = gemm_work(b, 4, 4, true);
  work.flops += wb.flops;
  work.bytes += wb.bytes;
  const bool big = tile == TILE_128x128;
  if (!big && tile != TILE_64x64) return hipErrorInvalidValue;
  if (kind_a == GEMM_NT && kind_b == GEMM_NN)
    return big ? launch_pair<F32Tile<2, true, true, false>, F32Tile<2, true, false, false>>(2, a, b, work, s)
               : launch_pair<F32Tile<1, true, true, false>, F32Tile<1, true, false, false>>(1, a, b, work, s);
  if (kind_a == GEMM_TN_F32 && kind_b == GEMM_NT)
    return big ? launch_pair<F32Tile<2, false, false, true>, F32Tile<2, true, true, false>>(2, a, b, work, s)
               : launch_pair<F32Tile<1, false, false, true>, F32Tile<1, true, true, false>>(1, a, b, work, s);
  return hipErrorInvalidValue;
}

}  // namespace sk
