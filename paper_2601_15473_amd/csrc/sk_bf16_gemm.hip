// bf16 MFMA GEMM with fp32 accumulation for gfx950: the contraction every
// two-pass plan of the SKLinear forward/backward is made of.
//
//   C[M, N] = scale * (A . B) (+ bias[n]),   or raw fp32 split-K partial slabs.
//
// (The 256 x 256 tile is a kernel of its own: sk_bf16_gemm256.hip.)  One work-group of 2 x 2
// waves owns a BM x BN tile; each wave a (BM/2) x (BN/2) sub-tile of 32x32 MFMA blocks.
// Operands go global -> registers -> LDS (double buffered, one barrier per 64-wide k chunk), or
// straight into a ring of chunks in LDS (sk_bf16_ring.h), and are read from LDS directly in the
// MFMA fragment layout; operands whose contiguous dimension is not k are read with
// the LDS transpose read.  Results leave straight from registers: fp32 as 16-byte
// pieces, bf16 in whole lines through a wave-private strip of LDS.
#include "sk_bf16_ring.h"
#include "sk_launch.h"

namespace sk {

// One tile configuration of the GEMM: its work-group size, its LDS footprint and its body
// (the work of one work-group, given the group's index in the launch and LDS of at
// least LDS_BYTES).  The body is a device function so that one launch can carry the
// work-groups of two independent GEMMs (dual_gemm_kernel below).
template <int BM, int BN, bool A_KC, bool B_KC, typename OutT, bool COLSUM>
struct GemmTile {
  static constexpr int NTH = 256, WAVES_N = 2;
  typedef OpTile<BM, A_KC, BK, NTH> TA;
  typedef OpTile<BN, B_KC, BK, NTH> TB;
  static constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;
  static constexpr int STAGE = TA::ELEMS + TB::ELEMS;
  static constexpr int LDS_BYTES = 2 * STAGE * 2;
  // bf16 results leave through a wave-private strip of LDS (32 rows of the wave's sub-tile at
  // a time, see the epilogue), carved out of a main buffer that is idle by then.
  static constexpr int WAVE_STRIP = 32 * WN * 2;
  static_assert((NTH / 64) * WAVE_STRIP <= STAGE * 2, "the waves' strips fit one main buffer");
  static __device__ __forceinline__ void run(const GemmArgs& p, int block, unsigned char* smem);
};

template <int BM, int BN, bool A_KC, bool B_KC, typename OutT, bool COLSUM>
__device__ __forceinline__ void
GemmTile<BM, BN, A_KC, B_KC, OutT, COLSUM>::run(const GemmArgs& p, int block, unsigned char* const smem) {
  bf16* const lds = reinterpret_cast<bf16*>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  const int tiles = p.tiles_m * p.tiles_n;
  const int id = xcd_remap(block, tiles * p.splits);
  const int split = id / tiles;
  int tile_m, tile_n;
  tile_coords(id - split * tiles, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int k_begin = split * p.k_per_split;
  const int k_end = (k_begin + p.k_per_split < p.K) ? k_begin + p.k_per_split : p.K;
  const int nk = (k_end - k_begin + BK - 1) / BK;

  const bf16* __restrict__ A = static_cast<const bf16*>(p.A);
  const bf16* __restrict__ B = static_cast<const bf16*>(p.B);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  f32x16 csum[COLSUM ? TN : 1];
  if (COLSUM) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) csum[j][r] = 0.f;
  }
  // Column sums of B ride on the MFMA: an all-ones fragment in place of A's.
  const bool do_colsum = COLSUM && p.colsum != nullptr && tile_m == 0 && wm == 0;
  bf16x8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (bf16)1.0f;

  // One k step (16 wide): fragments of the four steps of a chunk are read one step
  // ahead of the MFMAs that use them (two fragment sets), so LDS latency hides
  // behind the matrix pipe.
  bf16x8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
  auto read = [&](const bf16* As, int ks, bf16x8 (&fa)[TM], bf16x8 (&fb)[TN]) {
    const bf16* Bs = As + TA::ELEMS;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = read_frag<A_KC, TA::LD>(As, wm * WM + i * 32, ks, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = read_frag<B_KC, TB::LD>(Bs, wn * WN + j * 32, ks, lane);
  };
  auto mma = [&](const bf16x8 (&fa)[TM], const bf16x8 (&fb)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    if (COLSUM) {
      if (do_colsum) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
          csum[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], ones, csum[j], 0, 0, 0);
      }
    }
  };
  // Work per chunk and thread: NMMA MFMAs and NDSR fragment reads per k step.  Each k step is one scheduling
  // phase in which the other instructions are spread evenly between the MFMAs
  // (sched_phase), so they issue in the shadow of the matrix pipe instead of in a
  // burst that stalls it (the texture path takes 16 cycles per 16-byte-per-lane load).
  constexpr int NDSR = (A_KC ? TM : 2 * TM) + (B_KC ? TN : 2 * TN);
  constexpr int NMMA = TM * TN;

  // This lane's bias values (four columns per 8-column group of each 32-column block),
  // fetched before the main loop so the epilogue does not wait for them; through a
  // buffer window of N elements (none without a bias), so no lane needs a branch.
  constexpr bool HAS_BIAS = sizeof(OutT) == 2;
  uint2 bias_r[HAS_BIAS ? TN : 1][4];
  if constexpr (HAS_BIAS) {
    const GWindow bias_w = make_window(p.bias, 0, p.bias != nullptr ? p.N : 0, 2);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const int gn = n0 + wn * WN + j * 32 + q * 8 + (lane >> 5) * 4;
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(bias_w.rsrc, gn * 2, 0, 0);
        bias_r[j][q] = make_uint2(v.x, v.y);
      }
  }

  {
    // An iteration is too short to cover a load's latency, so two
    // register sets keep the loads of chunk kc + 2 in flight while chunk kc + 1,
    // loaded one iteration earlier, is stored.  (Four and six sets were measured on the
    // shapes of this layer and were no faster.)
    uint4 ra0[TA::PIECES], rb0[TB::PIECES], ra1[TA::PIECES], rb1[TB::PIECES];
    TA::load(ra0, A, p.lda, m0, p.M, k_begin, k_end, p.K, tid);
    TB::load(rb0, B, p.ldb, n0, p.N, k_begin, k_end, p.K, tid);
    TA::load(ra1, A, p.lda, m0, p.M, k_begin + BK, k_end, p.K, tid);
    TB::load(rb1, B, p.ldb, n0, p.N, k_begin + BK, k_end, p.K, tid);
    TA::store(lds, ra0, tid);
    TB::store(lds + TA::ELEMS, rb0, tid);
    __syncthreads();
    auto iteration = [&](const bf16* As, bf16* An, uint4 (&la)[TA::PIECES], uint4 (&lb)[TB::PIECES],
                         uint4 (&sa)[TA::PIECES], uint4 (&sb)[TB::PIECES], int k0) {
      // loads into (la, lb) for chunk k0, A's during k step 0 and B's during k step 1 (in
      // one burst they hold the waves at the memory pipe's queue; measured 1 % on the
      // [8192 x 1024..4096] shapes); stores from (sa, sb), loaded an iteration ago
      __builtin_amdgcn_sched_barrier(0);
      read(As, 1, fa1, fb1);
      TA::load(la, A, p.lda, m0, p.M, k0, k_end, p.K, tid);
      mma(fa0, fb0);
      sched_phase<NMMA, NDSR, TA::PIECES, 0>();
      read(As, 2, fa0, fb0);
      TB::load(lb, B, p.ldb, n0, p.N, k0, k_end, p.K, tid);
      mma(fa1, fb1);
      TA::store(An, sa, tid);
      sched_phase<NMMA, NDSR, TB::PIECES, TA::PIECES>();
      read(As, 3, fa1, fb1);
      mma(fa0, fb0);
      TB::store(An + TA::ELEMS, sb, tid);
      sched_phase<NMMA, NDSR, 0, TB::PIECES>();
      // the barrier one k step before the end of the chunk: the first fragments of the
      // next chunk come in behind the last step's MFMAs, not behind the barrier
      __syncthreads();
      read(An, 0, fa0, fb0);
      mma(fa1, fb1);
      sched_phase<NMMA, NDSR, 0, 0>();
    };
    read(lds, 0, fa0, fb0);
    for (int kc = 0; kc < nk; kc += 2) {
      iteration(lds, lds + STAGE, ra0, rb0, ra1, rb1, k_begin + (kc + 2) * BK);
      // an all-zero chunk when nk is odd
      iteration(lds + STAGE, lds, ra1, rb1, ra0, rb0, k_begin + (kc + 3) * BK);
    }
  }

  // ---- epilogue: accumulators -> global ----
  // Lane l owns output row l % 32 of each 32-row block and, for q = 0..3, the four
  // columns 8 q + 4 (l / 32) .. +3 of each 32-column block.
  //   fp32: those 16 bytes are stored as they are (32-byte row segments, merged by the L2).
  //   bf16: the two half-waves exchange the halves of neighbouring column groups
  //     (v_permlane32_swap), after which every lane holds eight consecutive columns; the
  //     wave then turns each 32-row block of its sub-tile over through a strip of LDS that
  //     only it touches (no barrier: one wave's LDS operations execute in order), so that
  //     eight consecutive lanes hold one whole row of the sub-tile and a store instruction
  //     writes complete 128-byte lines.  Stored straight from registers the same data left as
  //     32 scattered 32-byte segments per instruction, which the store path takes four
  //     times as long to work through: with the stores switched off the [8192 x 512] .
  //     [512 x 4096] product of BERT-large took 37 us instead of 50, and most of that gap
  //     stayed when the stores went to a cache-resident scratch target instead, i.e. it was
  //     the instructions, not the bytes.  Pieces are XOR-swizzled by row so that neither the
  //     column-wise writes nor the row-wise reads collide on LDS banks.
  OutT* __restrict__ C = static_cast<OutT*>(p.C) +
                         (sizeof(OutT) == 4 ? (int64_t)split * p.M * p.ldc : (int64_t)0);
  const float scale = p.scale;
  const int wn0 = n0 + wn * WN;  // first global column of this wave
  const int n_store = p.n_store > 0 ? p.n_store : p.N;

  if constexpr (sizeof(OutT) == 4) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int gm = m0 + wm * WM + i * 32 + (lane & 31);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int gn = wn0 + j * 32 + q * 8 + (lane >> 5) * 4;
          if (gm < p.M && gn < n_store)
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + (int64_t)gm * p.ldc + gn) =
                make_float4(acc[i][j][q * 4 + 0] * scale, acc[i][j][q * 4 + 1] * scale,
                            acc[i][j][q * 4 + 2] * scale, acc[i][j][q * 4 + 3] * scale);
        }
    }
  } else {
    constexpr int PPRW = WN / 8;        // 16-byte pieces per row of the wave's sub-tile
    constexpr int RPI = 64 / PPRW;      // rows one store instruction covers
    constexpr int ROW_BYTES = WN * 2;
    // The strips live in the main buffer.  The last k step still read fragments after the
    // loop's last barrier, so one more comes first.
    __syncthreads();
    unsigned char* const strip = smem + wave * WAVE_STRIP;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row_w = lane & 31;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
          uint2 w[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int q = 2 * pr + h;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[i][j][q * 4 + e] * scale;
            const uint2 bb = bias_r[j][q];
            v[0] += bf16_bits_to_float(bb.x & 0xffffu);
            v[1] += bf16_bits_to_float(bb.x >> 16);
            v[2] += bf16_bits_to_float(bb.y & 0xffffu);
            v[3] += bf16_bits_to_float(bb.y >> 16);
            w[h].x = pack_bf16x2(v[0], v[1]);
            w[h].y = pack_bf16x2(v[2], v[3]);
          }
          typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
          const u32x2 s0 = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
          const u32x2 s1 = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
          // columns j * 32 + 16 pr + 8 (l / 32) .. + 7 of the sub-tile: piece 4 j + 2 pr + l / 32
          const int piece = j * 4 + pr * 2 + (lane >> 5);
          *reinterpret_cast<uint4*>(strip + row_w * ROW_BYTES + ((piece ^ (row_w & (PPRW - 1))) * 16)) =
              make_uint4(s0.x, s1.x, s0.y, s1.y);
        }
#pragma unroll
      for (int r0 = 0; r0 < 32; r0 += RPI) {
        const int row_r = r0 + lane / PPRW, piece = lane % PPRW;
        const uint4 v = *reinterpret_cast<const uint4*>(strip + row_r * ROW_BYTES + ((piece ^ (row_r & (PPRW - 1))) * 16));
        const int gm = m0 + wm * WM + i * 32 + row_r;
        const int gn = wn0 + piece * 8;
        if (gm < p.M && gn < n_store)
          *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(C) + (int64_t)gm * p.ldc + gn) = v;
      }
    }
  }

  if (COLSUM) {
    // every D column of csum holds the same sums; lanes 0 and 32 write them out
    if (do_colsum && (lane & 31) == 0) {
      float* out = p.colsum + (int64_t)split * p.N;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int gn = wn0 + j * 32 + q * 8 + (lane >> 5) * 4;
          if (gn < p.N)
            *reinterpret_cast<float4*>(out + gn) = make_float4(
                csum[j][q * 4 + 0], csum[j][q * 4 + 1], csum[j][q * 4 + 2], csum[j][q * 4 + 3]);
        }
    }
  }
}

// RING: the tile on a ring of chunks, for launches of one round.
template <int BM, int BN, bool A_KC, bool B_KC, typename OutT, bool COLSUM, bool RING = false>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const GemmArgs p) {
  typedef typename std::conditional<RING, RingTile<BM, BN, A_KC, B_KC, OutT, COLSUM>, GemmTile<BM, BN, A_KC, B_KC, OutT, COLSUM>>::type G;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[G::LDS_BYTES];
  G::run(p, blockIdx.x, smem);
}

// Whether a tile has a ring, for the launches of one round on which it is ahead.  Past a round two or more staged
// work-groups on a CU hide each other's waits as well, and a ring takes their room ([11752 x 3344] . [3344 x 2032] and the like on
// 128 x 128 rings in place of 256 x 256 tiles or staged ones: 4 to 10 % behind).  It is behind for bf16 results of 128 x 64
// ([4001 x 384] . [384 x 768] 9.8 : 8.5 us) and for 64 x 128 (dY . U^T of [4096 x 3072], R = 128, in four ranges 12.3 : 12.0).
template <int BM, int BN, typename OutT>
constexpr bool has_ring() { return BM == BN || (BM == 128 && sizeof(OutT) == 4); }

// Two independent GEMMs in one launch: the first `groups_a` work-groups run GA on `a`, the
// rest run GB on `b`.  For small problems a kernel's fixed cost (launch, first trip to
// memory, drain) is as large as its work, and two kernels that do not depend on each
// other can share it; the chip co-schedules both kinds of work-group on every CU.
template <class GA, class GB>
__global__ __launch_bounds__(256) void dual_gemm_kernel(const GemmArgs a, const GemmArgs b,
                                                        const int groups_a) {
  constexpr int BYTES = GA::LDS_BYTES > GB::LDS_BYTES ? GA::LDS_BYTES : GB::LDS_BYTES;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[BYTES];
  if ((int)blockIdx.x < groups_a) GA::run(a, blockIdx.x, smem);
  else GB::run(b, (int)blockIdx.x - groups_a, smem);
}

// Sums the split-K slabs in index order; see ReduceArgs.
// (One piece per thread and no bounds test inside the slab loop: as many work-groups as
// pieces allow matters more here than loads per thread.)
__global__ __launch_bounds__(256) void reduce_splits_kernel(const ReduceArgs p) {
  int64_t i4 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  const float* __restrict__ part = p.part;
  float* __restrict__ out = p.out;
  int64_t n = p.n;
  float scale = p.scale;
  int splits = p.splits;
  if (i4 >= n) {  // second segment
    i4 -= n;
    part = p.part2; out = p.out2; n = p.n2; scale = p.scale2; splits = p.splits2;
    if (i4 >= n) return;
  }
  float4 s = sum_slabs(part + i4, n, splits);
  s.x *= scale; s.y *= scale; s.z *= scale; s.w *= scale;
  *reinterpret_cast<float4*>(out + i4) = s;
}

// Sum of split-K slabs in index order, rounded once to bf16 (an intermediate that the
// next GEMM reads as an operand).
// (`second` is for two products of one launch; the sum of one alone takes 0.3 us longer with it as an argument.)
__device__ __forceinline__ void reduce_to_bf16(const RoundedSum& p, int64_t i4) {
  const float4 s = sum_slabs(p.part + i4, p.n, p.splits);
  uint2 w;
  w.x = pack_bf16x2(s.x, s.y);
  w.y = pack_bf16x2(s.z, s.w);
  *reinterpret_cast<uint2*>(static_cast<bf16*>(p.out) + i4) = w;
}
__global__ __launch_bounds__(256) void reduce_to_bf16_kernel(const RoundedSum p) {
  const int64_t i4 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 < p.n) reduce_to_bf16(p, i4);
}
__global__ __launch_bounds__(256) void reduce_two_to_bf16_kernel(const RoundedSum p, const RoundedSum second) {
  const int64_t i4 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 < p.n) reduce_to_bf16(p, i4);
  else if (i4 - p.n < second.n) reduce_to_bf16(second, i4 - p.n);
}

// Up to three fp32 arrays, whole or in slabs, rounded to bf16, one behind the other over the work-groups.  Bound by the launch:
// 246 k numbers (a two-sided BERT-base layer's gradients) 2.7 us, through torch's fused copy 13.6.  The sums of their ranges here instead of
// ahead of it are two launches less of that layer's six backward.
__global__ __launch_bounds__(256) void round_gradients_kernel(const RoundArgs p) {
  int64_t i4 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
#pragma unroll
  for (int s = 0; s < RoundArgs::MAX; ++s) {
    if (i4 < p.n[s]) {
      const float* const from = p.from[s] + i4;
      unsigned short* const to = p.to[s] + i4;
      if (i4 + 4 <= p.n[s]) {
        float4 v = sum_slabs(from, p.stride[s], p.splits[s]);
        v.x *= p.scale[s]; v.y *= p.scale[s]; v.z *= p.scale[s]; v.w *= p.scale[s];
        *reinterpret_cast<uint2*>(to) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
      } else {
        for (int e = 0; i4 + e < p.n[s]; ++e) to[e] = (unsigned short)pack_bf16x2(from[e] * p.scale[s], 0.f);
      }
      return;
    }
    i4 -= (p.n[s] + 3) / 4 * 4;
  }
}

template <typename OutT>
static std::string out_label() { return sizeof(OutT) == 2 ? "bf16" : "float"; }

template <int BM, int BN, bool A_KC, bool B_KC, typename OutT, bool COLSUM>
static hipError_t launch_cfg(GemmArgs a, hipStream_t s) {
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + BN - 1) / BN;
  const long long total = (long long)a.tiles_m * a.tiles_n * a.splits;
  if (total <= 0 || total > 0x7fffffffLL || (A_KC && !within_window(BM, a.lda, BK, 2)) || (B_KC && !within_window(BN, a.ldb, BK, 2)))
    return hipErrorInvalidValue;
  note_gemm(a, A_KC, B_KC, 2, sizeof(OutT), sizeof(OutT) == 4);
  static const std::string name = kernel_label("gemm_bf16_kernel", {lbl(BM), lbl(BN), lbl(A_KC), lbl(B_KC), out_label<OutT>(), lbl(COLSUM)});
  const Work work = gemm_work(a, 2, sizeof(OutT), sizeof(OutT) == 4);
  if constexpr (has_ring<BM, BN, OutT>()) {
    if (total <= NUM_CUS * RingTile<BM, BN, A_KC, B_KC, OutT, COLSUM>::PER_CU) {
      static const std::string ring = kernel_label("gemm_bf16_kernel", {lbl(BM), lbl(BN), lbl(A_KC), lbl(B_KC), out_label<OutT>(), lbl(COLSUM), lbl(true)});
      return launch_kernel(ring.c_str(), work, gemm_bf16_kernel<BM, BN, A_KC, B_KC, OutT, COLSUM, true>, dim3((unsigned)total), dim3(256), s, a);
    }
  }
  return launch_kernel(name.c_str(), work, gemm_bf16_kernel<BM, BN, A_KC, B_KC, OutT, COLSUM>, dim3((unsigned)total), dim3(256), s, a);
}

// Tiles that have a ring only.
template <int BM, int BN, bool A_KC, bool B_KC>
static hipError_t launch_ring(GemmArgs a, hipStream_t s) {
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + BN - 1) / BN;
  const long long total = (long long)a.tiles_m * a.tiles_n;
  if (a.splits != 1 || total <= 0 || total > 0x7fffffffLL || (A_KC && !within_window(BM, a.lda, BK, 2)) || (B_KC && !within_window(BN, a.ldb, BK, 2)))
    return hipErrorInvalidValue;
  note_gemm(a, A_KC, B_KC, 2, 2, false);
  static const std::string name = kernel_label("gemm_bf16_kernel", {lbl(BM), lbl(BN), lbl(A_KC), lbl(B_KC), "bf16", lbl(false), lbl(true)});
  return launch_kernel(name.c_str(), gemm_work(a, 2, 2, false), gemm_bf16_kernel<BM, BN, A_KC, B_KC, bf16, false, true>, dim3((unsigned)total), dim3(256), s, a);
}

template <bool A_KC, bool B_KC, typename OutT, bool COLSUM>
static hipError_t launch_tiles(int tile, const GemmArgs& a, hipStream_t s) {
  switch (tile) {
    case TILE_128x128: return launch_cfg<128, 128, A_KC, B_KC, OutT, COLSUM>(a, s);
    case TILE_128x64: return launch_cfg<128, 64, A_KC, B_KC, OutT, COLSUM>(a, s);
    case TILE_64x128: return launch_cfg<64, 128, A_KC, B_KC, OutT, COLSUM>(a, s);
    case TILE_64x64: return launch_cfg<64, 64, A_KC, B_KC, OutT, COLSUM>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_bf16(GemmKind kind, int tile, const GemmArgs& a, hipStream_t s) {
  if (tile == TILE_256x256) return launch_gemm256_bf16(kind, a, s);
  if (tile == TILE_256x128 && kind == GEMM_NN) return launch_ring<256, 128, true, false>(a, s);
  if (tile == TILE_256x128 && kind == GEMM_NT) return launch_ring<256, 128, true, true>(a, s);
  switch (kind) {
    case GEMM_NN: return launch_tiles<true, false, bf16, false>(tile, a, s);
    case GEMM_NT: return launch_tiles<true, true, bf16, false>(tile, a, s);
    case GEMM_TN_F32: return launch_tiles<false, false, float, true>(tile, a, s);
    case GEMM_TN_F32_PLAIN: return launch_tiles<false, false, float, false>(tile, a, s);
    case GEMM_NN_F32: return launch_tiles<true, false, float, false>(tile, a, s);
    case GEMM_TT: return launch_tiles<false, true, bf16, false>(tile, a, s);
    case GEMM_NN_F32_COLSUM: return launch_tiles<true, false, float, true>(tile, a, s);
    case GEMM_NT_F32: return launch_tiles<true, true, float, false>(tile, a, s);
    case GEMM_TT_F32: return launch_tiles<false, true, float, false>(tile, a, s);
    default: return hipErrorInvalidValue;
  }
}

namespace {
typedef GemmTile<64, 64, true, true, bf16, false> NT_64x64;
typedef GemmTile<128, 64, true, true, bf16, false> NT_128x64;
typedef GemmTile<128, 128, true, true, bf16, false> NT_128x128;
typedef GemmTile<64, 64, true, true, float, false> NTF_64x64;
typedef GemmTile<64, 128, true, true, float, false> NTF_64x128;
typedef GemmTile<128, 128, true, true, float, false> NTF_128x128;
typedef GemmTile<64, 64, false, true, bf16, false> TT_64x64;
typedef GemmTile<128, 128, false, true, bf16, false> TT_128x128;
typedef GemmTile<64, 64, false, true, float, false> TTF_64x64;
typedef GemmTile<64, 128, false, true, float, false> TTF_64x128;
typedef GemmTile<128, 64, false, true, float, false> TTF_128x64;
typedef GemmTile<128, 128, false, true, float, false> TTF_128x128;
typedef GemmTile<128, 64, true, false, float, true> NNFC_128x64;
typedef GemmTile<128, 128, true, false, float, true> NNFC_128x128;
typedef RingTile<64, 64, true, true, bf16, false> RING_NT_64x64;
typedef RingTile<64, 64, true, true, float, false> RING_NTF_64x64;
typedef RingTile<64, 64, false, true, bf16, false> RING_TT_64x64;
typedef RingTile<64, 64, false, true, float, false> RING_TTF_64x64;

// The pairs of (kind, tile) the dual kernel is built for, the ones the backward pass's plans produce, with the kernel
// of each and, for those on 64 x 64 tiles, the one on rings.  The first should be the longer-running GEMM: its
// work-groups are dispatched first and the other's fill in beside them.
typedef void (*DualKernel)(GemmArgs, GemmArgs, int);
struct DualPair { GemmKind ka; int ta; GemmKind kb; int tb; DualKernel staged, ring; };
const DualPair kDualPairs[] = {
    // narrow sketch: R in 65..128, R <= 64; of a long input, Z^T in ranges as well
    {GEMM_NT_F32, TILE_64x128, GEMM_TT, TILE_64x64, dual_gemm_kernel<NTF_64x128, TT_64x64>, nullptr},
    {GEMM_NT_F32, TILE_64x64, GEMM_TT, TILE_64x64, dual_gemm_kernel<NTF_64x64, TT_64x64>, dual_gemm_kernel<RING_NTF_64x64, RING_TT_64x64>},
    {GEMM_NT_F32, TILE_64x64, GEMM_TT_F32, TILE_64x128, dual_gemm_kernel<NTF_64x64, TTF_64x128>, nullptr},
    {GEMM_NT_F32, TILE_64x128, GEMM_TT_F32, TILE_128x128, dual_gemm_kernel<NTF_64x128, TTF_128x128>, nullptr},
    {GEMM_NT_F32, TILE_64x128, GEMM_TT_F32, TILE_128x64, dual_gemm_kernel<NTF_64x128, TTF_128x64>, nullptr},
    // wide sketch, dY.U^T beside Z^T: both whole, the one, the other or both in ranges
    {GEMM_NT, TILE_128x128, GEMM_TT, TILE_128x128, dual_gemm_kernel<NT_128x128, TT_128x128>, nullptr},
    {GEMM_NT_F32, TILE_128x128, GEMM_TT, TILE_128x128, dual_gemm_kernel<NTF_128x128, TT_128x128>, nullptr},
    {GEMM_NT, TILE_128x128, GEMM_TT_F32, TILE_128x128, dual_gemm_kernel<NT_128x128, TTF_128x128>, nullptr},
    {GEMM_NT_F32, TILE_128x128, GEMM_TT_F32, TILE_128x128, dual_gemm_kernel<NTF_128x128, TTF_128x128>, nullptr},
    {GEMM_NT, TILE_64x64, GEMM_TT, TILE_64x64, dual_gemm_kernel<NT_64x64, TT_64x64>, dual_gemm_kernel<RING_NT_64x64, RING_TT_64x64>},
    {GEMM_NT, TILE_64x64, GEMM_TT_F32, TILE_64x64, dual_gemm_kernel<NT_64x64, TTF_64x64>, dual_gemm_kernel<RING_NT_64x64, RING_TTF_64x64>},
    {GEMM_NT_F32, TILE_64x64, GEMM_TT_F32, TILE_64x64, dual_gemm_kernel<NTF_64x64, TTF_64x64>, dual_gemm_kernel<RING_NTF_64x64, RING_TTF_64x64>},
    // wide sketch, Z^T.dY beside G.S^T
    {GEMM_NN_F32_COLSUM, TILE_128x64, GEMM_NT, TILE_128x128, dual_gemm_kernel<NNFC_128x64, NT_128x128>, nullptr},
    {GEMM_NN_F32_COLSUM, TILE_128x128, GEMM_NT, TILE_128x128, dual_gemm_kernel<NNFC_128x128, NT_128x128>, nullptr},
    {GEMM_NN_F32_COLSUM, TILE_128x64, GEMM_NT, TILE_128x64, dual_gemm_kernel<NNFC_128x64, NT_128x64>, nullptr},
    {GEMM_NN_F32_COLSUM, TILE_128x64, GEMM_NT, TILE_64x64, dual_gemm_kernel<NNFC_128x64, NT_64x64>, nullptr},
};
const DualPair* dual_pair(GemmKind ka, int ta, GemmKind kb, int tb) {
  for (const DualPair& p : kDualPairs)
    if (p.ka == ka && p.ta == ta && p.kb == kb && p.tb == tb) return &p;
  return nullptr;
}
}  // namespace

bool dual_gemm_supported(GemmKind kind_a, int tile_a, GemmKind kind_b, int tile_b) {
  return dual_pair(kind_a, tile_a, kind_b, tile_b) != nullptr;
}

hipError_t launch_dual_gemm_bf16(GemmKind kind_a, int tile_a, GemmArgs a, GemmKind kind_b, int tile_b,
                                 GemmArgs b, hipStream_t s) {
  const DualPair* const pair = dual_pair(kind_a, tile_a, kind_b, tile_b);
  if (pair == nullptr) return hipErrorInvalidValue;
  int bm, bn;
  tile_dims(tile_a, bm, bn);
  a.tiles_m = (a.M + bm - 1) / bm;
  a.tiles_n = (a.N + bn - 1) / bn;
  tile_dims(tile_b, bm, bn);
  b.tiles_m = (b.M + bm - 1) / bm;
  b.tiles_n = (b.N + bn - 1) / bn;
  const long long ga = (long long)a.tiles_m * a.tiles_n * a.splits;
  const long long gb = (long long)b.tiles_m * b.tiles_n * b.splits;
  if (ga <= 0 || gb <= 0 || ga + gb > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(ga + gb)), block(256);
  Work work;
  {
    bool akc, bkc, f32;
    gemm_kind_traits(kind_a, akc, bkc, f32);
    note_gemm(a, akc, bkc, 2, f32 ? 4 : 2, f32);
    work = gemm_work(a, 2, f32 ? 4 : 2, f32);
    gemm_kind_traits(kind_b, akc, bkc, f32);
    note_gemm(b, akc, bkc, 2, f32 ? 4 : 2, f32);
    const Work wb = gemm_work(b, 2, f32 ? 4 : 2, f32);
    work.flops += wb.flops;
    work.bytes += wb.bytes;
  }
  // 64 x 64 tiles in one round, two work-groups to a CU: on the ring, as a product by itself.  Backward pass, us, staged : ring,
  // narrow sketches: 2925 tokens, 1584 -> 2480, R = 64 29.6 : 26.6; 1024, 1024 -> 1024, R = 64 19.6 : 17.5; 2901, 304 -> 3824, R = 16 20.1 : 20.4;
  // wide ones: 1600, 2464 -> 1536, R = 256 30.6 : 25.3; 1507, 3120 -> 464, R = 512 36.9 : 31.6; 4096, 768 -> 768, R = 256 (512
  // work-groups) 24.5 : 23.5.  (On rings of their own the 128 x 64 and the 128 x 128 tiles of the other pairs are level with the staged
  // ones: 150 layers with the latter, 1.0000 of the time, 0.98 to 1.02.)
  const bool ring = pair->ring != nullptr && ga + gb <= NUM_CUS * RING_NT_64x64::PER_CU;
  return launch_kernel(ring ? "dual_gemm_kernel<ring>" : "dual_gemm_kernel", work, ring ? pair->ring : pair->staged, grid, block, s, a, b, (int)ga);
}

__global__ __launch_bounds__(256) void reduce_splits_2d_kernel(const float* __restrict__ part,
                                                               float* __restrict__ out, int rows, int cols,
                                                               int64_t ld_out, int splits, float scale) {
  const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
  const int r = blockIdx.y;
  if (c >= cols) return;
  const int64_t n = (int64_t)rows * cols, at = (int64_t)r * cols + c;
  const float4 s = sum_slabs(part + at, n, splits);
  *reinterpret_cast<float4*>(out + (int64_t)r * ld_out + c) =
      make_float4(s.x * scale, s.y * scale, s.z * scale, s.w * scale);
}

hipError_t launch_reduce_splits_2d(const float* part, float* out, int rows, int cols, int64_t ld_out,
                                   int splits, float scale, hipStream_t s) {
  if (rows < 1 || rows > 65535 || cols < 4 || (cols & 3) != 0 || splits < 1) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((cols / 4 + 255) / 256), (unsigned)rows);
  note_matrix(part, (int64_t)splits * rows, cols, cols, 4, false);
  note_matrix(out, rows, cols, ld_out, 4, true);
  return launch_kernel("reduce_splits_2d_kernel", Work{0.0, 4.0 * rows * cols * (splits + 1)}, reduce_splits_2d_kernel, grid, dim3(256), s, part, out, rows,
                       cols, ld_out, splits, scale);
}

hipError_t launch_reduce_to_bf16(const RoundedSum& a, const RoundedSum& b, hipStream_t s) {
  const int64_t groups = ((a.n + b.n) / 4 + 255) / 256;
  if (groups == 0) return hipSuccess;
  if (a.n < 0 || b.n < 0 || ((a.n | b.n) & 3) != 0 || (a.n > 0 && a.splits < 1) || (b.n > 0 && b.splits < 1) || groups > 0x7fffffffLL) return hipErrorInvalidValue;
  Work work{0.0, 0.0};
  for (const RoundedSum& r : {a, b}) {
    if (r.n == 0) continue;
    note_matrix(r.part, r.splits, r.n, r.n, 4, false);
    note_matrix(r.out, 1, r.n, r.n, 2, true);
    work.bytes += (double)r.n * (4.0 * r.splits + 2.0);
  }
  if (a.n > 0 && b.n > 0) return launch_kernel("reduce_two_to_bf16_kernel", work, reduce_two_to_bf16_kernel, dim3((unsigned)groups), dim3(256), s, a, b);
  return launch_kernel("reduce_to_bf16_kernel", work, reduce_to_bf16_kernel, dim3((unsigned)groups), dim3(256), s, a.n > 0 ? a : b);
}

hipError_t launch_reduce_splits(const ReduceArgs& a, hipStream_t s) {
  const int64_t groups = ((a.n + a.n2) / 4 + 255) / 256;
  if (groups <= 0) return hipSuccess;
  note_reduce(a);
  return launch_kernel("reduce_splits_kernel", reduce_work(a), reduce_splits_kernel, dim3((unsigned)groups), dim3(256), s, a);
}

hipError_t launch_round_gradients(const RoundArgs& a, hipStream_t s) {
  int64_t pieces = 0;
  Work work{0.0, 0.0};
  for (int i = 0; i < RoundArgs::MAX; ++i) {
    if (a.n[i] == 0) continue;
    if (a.n[i] < 0 || a.splits[i] < 1 || (a.splits[i] > 1 && (a.n[i] & 3) != 0)) return hipErrorInvalidValue;
    pieces += (a.n[i] + 3) / 4;
    note_matrix(a.from[i], a.splits[i], a.n[i], a.stride[i], 4, false);
    note_matrix(a.to[i], 1, a.n[i], a.n[i], 2, true);
    work.bytes += (double)a.n[i] * (4.0 * a.splits[i] + 2.0);
  }
  const int64_t groups = (pieces + 255) / 256;
  if (groups <= 0) return hipSuccess;
  if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
  return launch_kernel("round_gradients_kernel", work, round_gradients_kernel, dim3((unsigned)groups), dim3(256), s, a);
}

}  // namespace sk
