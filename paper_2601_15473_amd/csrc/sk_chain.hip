// The "expand" half of SKLinear for small sketch widths (bf16, R <= 512), with the
// R-wide intermediate resident on chip, and optionally the "sketch" half fused in
// front of it:
//
//   C[M, N] = scale * Zt . B2 (+ bias),   Zt = the bf16 R-wide intermediate of a
//   64-token tile, either
//     - computed here:  Zt = bf16(A[64 tokens, K1] . B1)            (FUSED), or
//     - read from the workspace: bf16 [M, R], or the sum of fp32 split-K slabs.
//
// A work-group (256 threads, 4 waves) owns one token tile and one slice of the N
// range.  Zt sits in LDS once and every wave lifts the whole of it into registers
// as MFMA fragments; the waves then split each BN-wide tile of N four ways, so a B2
// fragment is read from LDS by exactly one wave and used for all 32-row blocks.
// Three kernels share that plan:
//   chain_ring (R <= 128, both stages fused, 64-token tiles: what the automatic plans launch there but for narrow sketches in
//     more than a round): every operand straight into LDS, on a ring of chunks in stage 1 and of whole tiles of B2 in stage 2;
//   chain_small (R <= 128, every other launch of the automatic plans): B2 arrives through registers one whole [R x 128] tile at
//     a time, double buffered across tile boundaries;
//     in both, output tiles leave one step later through LDS, in whole rows (chain_small_kernel), in short runs
//     straight from registers (chain_short_kernel);
//   chain_kernel (R <= 512, forced plans only): B2 streams in 64-row chunks and the output
//     tile is re-laid out through LDS into whole rows.
#include "sk_bf16_ring.h"
#include "sk_launch.h"

namespace sk {

constexpr int CH_BM = 64;

template <int RT, int BN, bool B2_KC, bool FUSED, bool B1_KC>
struct ChainLds {
  typedef OpTile<BN, B2_KC> TB2;
  typedef OpTile<CH_BM, true> TA;
  typedef OpTile<RT, B1_KC> TB1;
  static constexpr int Z_LD = RT + 8;
  static constexpr int Z_BYTES = CH_BM * Z_LD * 2;
  static constexpr int OUT_LD = BN * 2 + 8;                       // bytes per staged output row
  static constexpr int S2_BYTES = 2 * TB2::ELEMS * 2 + CH_BM * OUT_LD;
  static constexpr int S1_BYTES = FUSED ? 2 * (TA::ELEMS + TB1::ELEMS) * 2 : 0;
  static constexpr int BYTES = Z_BYTES + (S1_BYTES > S2_BYTES ? S1_BYTES : S2_BYTES);
};

template <int RT, int BN, bool B2_KC, bool FUSED, bool B1_KC>
__global__ __launch_bounds__(256) void chain_kernel(const ChainArgs p) {
  typedef ChainLds<RT, BN, B2_KC, FUSED, B1_KC> L;
  typedef typename L::TB2 TB2;
  constexpr int KC = RT / 64;            // k chunks of stage 2
  constexpr int WN = BN / 4, TN = WN / 32;
  __shared__ __attribute__((aligned(16))) unsigned char smem[L::BYTES];
  bf16* const Zs = reinterpret_cast<bf16*>(smem);
  unsigned char* const work = smem + L::Z_BYTES;
  bf16* const Bbuf = reinterpret_cast<bf16*>(work);
  unsigned char* const ostage = work + 2 * TB2::ELEMS * 2;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // all slices of one token tile run on the same XCD, so its L2 fetches the tile once
  const int wg = xcd_remap(blockIdx.x, p.tiles_m * p.n_slices);
  const int tile_m = wg / p.n_slices, slice = wg % p.n_slices;
  const int m0 = tile_m * CH_BM;

  // this work-group's run of BN-wide tiles
  const int n_tiles = (p.N + BN - 1) / BN;
  const int per_slice = (n_tiles + p.n_slices - 1) / p.n_slices;
  const int t_begin = slice * per_slice;
  const int t_end = (t_begin + per_slice < n_tiles) ? t_begin + per_slice : n_tiles;
  const int my_tiles = t_end - t_begin;
  if (my_tiles <= 0) return;  // uniform over the work-group

  const bf16* __restrict__ B2 = static_cast<const bf16*>(p.B2);
  uint4 rb[TB2::PIECES];
  // first B2 chunk goes in flight before anything else
  TB2::load(rb, B2, p.ldb2, t_begin * BN, p.N, 0, p.R, p.R, tid);

  // ---------------- the intermediate tile Zt -> LDS ----------------
  if (FUSED) {
    typedef typename L::TA TA;
    typedef typename L::TB1 TB1;
    constexpr int STAGE = TA::ELEMS + TB1::ELEMS;
    constexpr int TN1 = RT / 64;  // waves 2 x 2: each 32 rows x RT/2 columns
    bf16* const s1 = reinterpret_cast<bf16*>(work);
    const bf16* __restrict__ A = static_cast<const bf16*>(p.A);
    const bf16* __restrict__ B1 = static_cast<const bf16*>(p.B1);
    const int wm = wave >> 1, wn = wave & 1;
    f32x16 acc1[TN1];
#pragma unroll
    for (int j = 0; j < TN1; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc1[j][r] = 0.f;
    uint4 ra[TA::PIECES], rb1[TB1::PIECES];
    const int nk = (p.K1 + BK - 1) / BK;
    TA::load(ra, A, p.lda, m0, p.M, 0, p.K1, p.K1, tid);
    TB1::load(rb1, B1, p.ldb1, 0, p.R, 0, p.K1, p.K1, tid);
    TA::store(s1, ra, tid);
    TB1::store(s1 + TA::ELEMS, rb1, tid);
    __syncthreads();
    for (int kc = 0; kc < nk; ++kc) {
      const bf16* As = s1 + (kc & 1) * STAGE;
      const bf16* Bs = As + TA::ELEMS;
      const bool more = kc + 1 < nk;
      if (more) {
        TA::load(ra, A, p.lda, m0, p.M, (kc + 1) * BK, p.K1, p.K1, tid);
        TB1::load(rb1, B1, p.ldb1, 0, p.R, (kc + 1) * BK, p.K1, p.K1, tid);
      }
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        const bf16x8 fa = read_frag<true, TA::LD>(As, wm * 32, ks, lane);
#pragma unroll
        for (int j = 0; j < TN1; ++j) {
          const bf16x8 fb = read_frag<B1_KC, TB1::LD>(Bs, wn * (RT / 2) + j * 32, ks, lane);
          acc1[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa, acc1[j], 0, 0, 0);
        }
      }
      if (more) {
        bf16* An = s1 + ((kc + 1) & 1) * STAGE;
        TA::store(An, ra, tid);
        TB1::store(An + TA::ELEMS, rb1, tid);
      }
      __syncthreads();
    }
    // round once to bf16: lane owns row l % 32 and 4 consecutive columns per q
#pragma unroll
    for (int j = 0; j < TN1; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = wn * (RT / 2) + j * 32 + q * 8 + (lane >> 5) * 4;
        uint2 w;
        w.x = pack_bf16x2(acc1[j][q * 4 + 0], acc1[j][q * 4 + 1]);
        w.y = pack_bf16x2(acc1[j][q * 4 + 2], acc1[j][q * 4 + 3]);
        *reinterpret_cast<uint2*>(Zs + (wm * 32 + (lane & 31)) * L::Z_LD + c) = w;
      }
  } else if (p.z_splits == 0) {
    // bf16 [M, R] from the workspace; columns >= R and rows >= M read as zero
    const bf16* __restrict__ Z = static_cast<const bf16*>(p.Z);
    constexpr int PPR = RT / 8;
#pragma unroll
    for (int i = 0; i < (CH_BM * PPR) / 256; ++i) {
      const int piece = i * 256 + tid;
      const int r = piece / PPR, c = (piece % PPR) * 8;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (m0 + r < p.M && c < p.R) v = *reinterpret_cast<const uint4*>(Z + (int64_t)(m0 + r) * p.R + c);
      *reinterpret_cast<uint4*>(Zs + r * L::Z_LD + c) = v;
    }
  } else {
    // sum of fp32 split-K slabs, slabs added in index order, rounded once to bf16
    const float* __restrict__ Zp = static_cast<const float*>(p.Z);
    constexpr int PPR = RT / 4;
#pragma unroll 2
    for (int i = 0; i < (CH_BM * PPR) / 256; ++i) {
      const int piece = i * 256 + tid;
      const int r = piece / PPR, c = (piece % PPR) * 4;
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m0 + r < p.M && c < p.R) {
        const float* src = Zp + (int64_t)(m0 + r) * p.R + c;
        s = *reinterpret_cast<const float4*>(src);
        for (int k = 1; k < p.z_splits; ++k) {
          const float4 v = *reinterpret_cast<const float4*>(src + (int64_t)k * p.z_slab);
          s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
      }
      uint2 w;
      w.x = pack_bf16x2(s.x, s.y);
      w.y = pack_bf16x2(s.z, s.w);
      *reinterpret_cast<uint2*>(Zs + r * L::Z_LD + c) = w;
    }
  }
  __syncthreads();  // Zt complete; stage-1 buffers (aliasing Bbuf) are free

  // every wave lifts all of Zt into registers, in MFMA fragment layout
  bf16x8 fa[2][RT / 16];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < RT / 16; ++ks)
      fa[i][ks] = read_frag_rowmajor<L::Z_LD>(Zs, i * 32, ks, lane);

  TB2::store(Bbuf, rb, tid);
  __syncthreads();

  // ---------------- stage 2: stream B2, one BN-wide output tile at a time ----------------
  f32x16 acc[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  bf16* __restrict__ C = static_cast<bf16*>(p.C);
  const bf16* __restrict__ bias = static_cast<const bf16*>(p.bias);
  const float scale = p.scale;
  const int n_it = my_tiles * KC;
  int it = 0;
  for (int jt = 0; jt < my_tiles; ++jt) {
    const int n0 = (t_begin + jt) * BN;
#pragma unroll
    for (int c = 0; c < KC; ++c, ++it) {
      const bf16* Bs = Bbuf + (it & 1) * TB2::ELEMS;
      const bool more = it + 1 < n_it;
      if (more) {
        const int nn0 = (c + 1 < KC) ? n0 : n0 + BN;
        const int k0 = (c + 1 < KC) ? (c + 1) * 64 : 0;
        TB2::load(rb, B2, p.ldb2, nn0, p.N, k0, p.R, p.R, tid);
      }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const bf16x8 fb = read_frag<B2_KC, TB2::LD>(Bs, wave * WN + j * 32, ks, lane);
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa[i][c * 4 + ks], acc[i][j], 0, 0, 0);
        }
      }
      if (c == KC - 1) {
        // tile finished: scale, bias, round, re-lay out through LDS, store whole rows
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int cc = wave * WN + j * 32 + q * 8 + (lane >> 5) * 4;  // column in the tile
              float v[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                v[e] = acc[i][j][q * 4 + e] * scale;
                acc[i][j][q * 4 + e] = 0.f;
              }
              if (bias != nullptr && n0 + cc < p.N) {
                const uint2 bb = *reinterpret_cast<const uint2*>(bias + n0 + cc);
                v[0] += bf16_bits_to_float(bb.x & 0xffffu);
                v[1] += bf16_bits_to_float(bb.x >> 16);
                v[2] += bf16_bits_to_float(bb.y & 0xffffu);
                v[3] += bf16_bits_to_float(bb.y >> 16);
              }
              uint2 w;
              w.x = pack_bf16x2(v[0], v[1]);
              w.y = pack_bf16x2(v[2], v[3]);
              *reinterpret_cast<uint2*>(ostage + (i * 32 + (lane & 31)) * L::OUT_LD + cc * 2) = w;
            }
        __syncthreads();
        constexpr int PPR = BN / 4;  // 8-byte pieces per output row
#pragma unroll
        for (int s = 0; s < (CH_BM * PPR) / 256; ++s) {
          const int idx = s * 256 + tid;
          const int r = idx / PPR, pc = idx % PPR;
          const int gm = m0 + r, gn = n0 + pc * 4;
          if (gm < p.M && gn < p.N)
            *reinterpret_cast<uint2*>(C + (int64_t)gm * p.ldc + gn) =
                *reinterpret_cast<const uint2*>(ostage + r * L::OUT_LD + pc * 8);
        }
      }
      if (more) TB2::store(Bbuf + ((it + 1) & 1) * TB2::ELEMS, rb, tid);
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Narrow sketches (R <= 128): the same chain, shaped for memory-level parallelism.
// These shapes are bound by bytes and latency, not flops, so the kernel keeps two loads
// in flight per thread at all times (two register sets, prefetch distance two).
//   - The token tile is MB = 64 rows, or 128 when the launcher asks for it (many
//     tokens: half the B2 traffic and LDS reads per MFMA in stage 2).
//   - stage 1 (waves 2 x 2) walks K1 in 64-wide chunks (x chunk + B1 chunk per step);
//   - stage 2 takes B2 one whole [R x 128] tile at a time (no k loop inside a tile).
//     A 64-lane LDS instruction costs the CU about 9 cycles, a transposing read
//     twice that per fragment, so the waves split the tile's columns 1 x 4: every
//     wave holds all rows of Zt in registers and each B2 fragment is read from LDS
//     exactly once.  A finished tile is turned over in LDS and leaves one step later, a
//     store instruction writing four whole 256-byte rows.
//   - In both stages each k step is one scheduling phase: fragment reads of the next
//     step, the step's MFMAs, a share of the global loads of the chunk / tile two
//     ahead and of the LDS stores of the next one.  A wave that issues its loads in
//     one burst waits at the memory pipe's queue while LDS and MFMA idle.
// ---------------------------------------------------------------------------
constexpr int CS_BN = 128;

// Finished output tiles kept in LDS: two, and one where that lets two work-groups share a CU, at one
// more barrier a step ([40000 x 384] -> 384, R = 32, forward 22.4 -> 17.4 us; 65536 tokens, 768 wide 39.7 ->
// 32.8; 3072 wide, runs of 24 tiles, 103 -> 108).
constexpr int chain_outs(int mb, int rt) { return mb == 128 && rt == 64 ? 1 : 2; }

template <int MB, int RT, bool B2_KC, bool FUSED, bool B1_KC, bool SHORT>
struct SmallLds {
  typedef OpTile<CS_BN, B2_KC, RT> TB2;
  typedef OpTile<MB, true> TA;
  typedef OpTile<RT, B1_KC> TB1;
  static constexpr int Z_LD = RT + 8;
  static constexpr int Z_BYTES = MB * Z_LD * 2;
  // finished output tiles, over Zt (which is in registers by then), then the B2 tiles
  static constexpr int OUTS = SHORT ? 0 : chain_outs(MB, RT);
  static constexpr int OUT_BYTES = MB * CS_BN * 2;
  // (without either, Zt lies where the second B2 tile goes once everybody has it in registers: 64 KB in all for R = 128)
  static constexpr bool OVER_B2 = SHORT && !FUSED;
  static constexpr int Z_AT = OVER_B2 ? TB2::ELEMS * 2 : 0;
  static constexpr int HEAD_BYTES = OVER_B2 ? 0 : Z_BYTES > OUTS * OUT_BYTES ? Z_BYTES : OUTS * OUT_BYTES;
  static constexpr int S2_BYTES = 2 * TB2::ELEMS * 2;
  static constexpr int S1_BYTES = FUSED ? 2 * (TA::ELEMS + TB1::ELEMS) * 2 : 0;   // (behind Zt)
  static constexpr int S1_END = Z_AT + Z_BYTES + S1_BYTES;
  static constexpr int BYTES = S1_END > HEAD_BYTES + S2_BYTES ? S1_END : HEAD_BYTES + S2_BYTES;
};

// Scheduling of one stage-2 tile of the narrow kernel: per k step the fragment reads of
// the next step (ND LDS reads), the step's NM MFMAs, one or two of the KS + 4 global loads
// and one of the KS LDS stores.
template <int KS, int ND, int NM, int I = 0>
__device__ __forceinline__ void sched_stage2() {
  if constexpr (I < KS) {
    if constexpr (I + 1 < KS) __builtin_amdgcn_sched_group_barrier(0x100, ND, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, NM, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, I < 4 ? 2 : 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
    sched_stage2<KS, ND, NM, I + 1>();
  } else {
    __builtin_amdgcn_sched_barrier(0);
  }
}

// SHORT: for runs of few output tiles, which leave straight from registers as they are finished.
// LEAN: one B2 tile fetched ahead of the slabs of Zt instead of two, for a launch that shares registers (256 with the slabs, else 272).
template <int MB, int RT, bool B2_KC, bool FUSED, bool B1_KC, bool SHORT, bool LEAN = false>
__device__ __forceinline__ void chain_small(const ChainArgs& p, const int block, unsigned char* const smem) {
  static_assert(MB == 64 || MB == 128, "token tiles are 64 or 128 rows");
  typedef SmallLds<MB, RT, B2_KC, FUSED, B1_KC, SHORT> L;
  typedef typename L::TB2 TB2;
  constexpr int KS = RT / 16;
  constexpr int MT = MB / 32;   // 32-row blocks of the token tile (stage 2: all of them in every wave)
  // stage 1: waves 2 x 2, each MB/2 rows x RT/2 columns of Zt (a 1 x 4 grid, with fewer
  // LDS reads per MFMA when B1 is read transposed, measured no faster)
  constexpr int WM1 = MB / 2, WN1 = RT / 2;
  constexpr int TM1 = WM1 / 32, TN1 = WN1 / 32;
  bf16* const Zs = reinterpret_cast<bf16*>(smem + L::Z_AT);
  bf16* const Bbuf = reinterpret_cast<bf16*>(smem + L::HEAD_BYTES);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;  // stage-1 wave grid
  const int wg = xcd_remap(block, p.tiles_m * p.n_slices);
  const int tile_m = wg / p.n_slices, slice = wg % p.n_slices;
  const int m0 = tile_m * MB;

  const int n_tiles = (p.N + CS_BN - 1) / CS_BN;
  const int per_slice = (n_tiles + p.n_slices - 1) / p.n_slices;
  const int t_begin = slice * per_slice;
  const int t_end = (t_begin + per_slice < n_tiles) ? t_begin + per_slice : n_tiles;
  const int my_tiles = t_end - t_begin;
  // The reduction this launch carries along goes to the work-groups with the least tile
  // work: those of the slices that got fewer tiles than the rest (often none at all, when
  // the tiles do not divide over the slices), or to everybody when all slices are equal.
  const bool has_tail = p.tail.n + p.tail.n2 > 0;
  const int first_light = n_tiles / per_slice;           // slices below this one are full
  const int n_light = p.n_slices - first_light;
  const bool tail_here = has_tail && (n_light == 0 || slice >= first_light);
  const int tail_rank = n_light == 0 ? wg : tile_m * n_light + (slice - first_light);
  const int tail_ranks = p.tiles_m * (n_light == 0 ? p.n_slices : n_light);
  if (my_tiles <= 0) {  // uniform over the work-group
    if (tail_here) reduce_splits_part(p.tail, tail_rank, tail_ranks, tid);
    return;
  }

  const bf16* __restrict__ B2 = static_cast<const bf16*>(p.B2);
  uint4 rb0[TB2::PIECES], rb1[TB2::PIECES];
  // B2 tile jt of this work-group; tiles past its run load as zeros (all lanes masked)
  auto load_b2 = [&](uint4 (&r)[TB2::PIECES], int jt) {
    TB2::load(r, B2, p.ldb2, (t_begin + jt) * CS_BN, jt < my_tiles ? p.N : 0, 0, p.R, p.R, tid);
  };
  // The first two B2 tiles go in flight early: before anything else when the intermediate
  // comes from memory, behind the first two chunks of stage 1 when it is computed here
  // (their 64 KB per work-group would hold up the start of stage 1 by ~0.7 us otherwise).
  if (!FUSED) {
    load_b2(rb0, 0);
    if (!LEAN) load_b2(rb1, 1);
  }

  // bias through a buffer window of N elements (zero elements when there is no bias:
  // every load then returns zero)
  const GWindow bias_w = make_window(p.bias, 0, p.bias != nullptr ? p.N : 0, 2);
  // this lane's 4 x 4 bias values of tile jt; always fetched one tile ahead of its use
  // (a tile's MFMAs are shorter than a trip to L2)
  auto load_bias = [&](uint2 (&bv)[4], int jt) {
    const int n0 = (t_begin + jt) * CS_BN;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cc = wave * 32 + q * 8 + (lane >> 5) * 4;
      typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
      const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(bias_w.rsrc, (n0 + cc) * 2, 0, 0);
      bv[q] = make_uint2(v.x, v.y);
    }
  };
  uint2 bv0[4], bv1[4];
  load_bias(bv0, 0);

  // this work-group's share of the carried reduction, while its own first loads are in flight
  if (tail_here) reduce_splits_part(p.tail, tail_rank, tail_ranks, tid);

  // ---------------- the intermediate tile Zt -> LDS ----------------
  if (FUSED) {
    typedef typename L::TA TA;
    typedef typename L::TB1 TB1;
    constexpr int STAGE = TA::ELEMS + TB1::ELEMS;
    bf16* const s1 = reinterpret_cast<bf16*>(smem + L::Z_BYTES);
    const bf16* __restrict__ A = static_cast<const bf16*>(p.A);
    const bf16* __restrict__ B1 = static_cast<const bf16*>(p.B1);
    f32x16 acc1[TM1][TN1];
#pragma unroll
    for (int i = 0; i < TM1; ++i)
#pragma unroll
      for (int j = 0; j < TN1; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc1[i][j][r] = 0.f;
    uint4 xa0[TA::PIECES], xb0[TB1::PIECES], xa1[TA::PIECES], xb1[TB1::PIECES];
    const int nk = (p.K1 + BK - 1) / BK;
    // chunks past K1 load as zeros, so the loop needs no branch around its loads
    auto load_a = [&](uint4 (&r)[TA::PIECES], int kc) {
      TA::load(r, A, p.lda, m0, p.M, kc * BK, p.K1, p.K1, tid);
    };
    constexpr int HB = TB1::PIECES / 2;
    auto load_b_lo = [&](uint4 (&r)[TB1::PIECES], int kc) {
      TB1::template load<0, HB>(r, B1, p.ldb1, 0, p.R, kc * BK, p.K1, p.K1, tid);
    };
    auto load_b_hi = [&](uint4 (&r)[TB1::PIECES], int kc) {
      TB1::template load<HB, TB1::PIECES>(r, B1, p.ldb1, 0, p.R, kc * BK, p.K1, p.K1, tid);
    };
    bf16x8 fa0[TM1], fa1[TM1], fb0[TN1], fb1[TN1];
    auto rd = [&](const bf16* As, int ks, bf16x8 (&fa)[TM1], bf16x8 (&fb)[TN1]) {
#pragma unroll
      for (int i = 0; i < TM1; ++i) fa[i] = read_frag<true, TA::LD>(As, wm * WM1 + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < TN1; ++j)
        fb[j] = read_frag<B1_KC, TB1::LD>(As + TA::ELEMS, wn * WN1 + j * 32, ks, lane);
    };
    auto mm = [&](const bf16x8 (&fa)[TM1], const bf16x8 (&fb)[TN1]) {
#pragma unroll
      for (int i = 0; i < TM1; ++i)
#pragma unroll
        for (int j = 0; j < TN1; ++j)
          acc1[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc1[i][j], 0, 0, 0);
    };
    // LDS read instructions of one k step: one per x fragment, one (k-contiguous B1) or
    // two (transposing reads) per B1 fragment
    constexpr int NDS = TM1 + TN1 * (B1_KC ? 1 : 2);
    constexpr int NM1 = TM1 * TN1;
    // One chunk: MFMAs on the chunk in `As`, the loads of the chunk two ahead (into la,
    // lb) and the LDS stores of the next chunk (from sa, sb, loaded an iteration ago)
    // spread between them -- issued in one burst the loads hold every wave at the
    // memory pipe's queue while LDS and MFMA sit idle.
    auto iteration = [&](const bf16* As, bf16* An, uint4 (&la)[TA::PIECES], uint4 (&lb)[TB1::PIECES],
                         uint4 (&sa)[TA::PIECES], uint4 (&sb)[TB1::PIECES], int kc_load) {
      rd(As, 0, fa0, fb0);
      __builtin_amdgcn_sched_barrier(0);
      rd(As, 1, fa1, fb1);
      load_a(la, kc_load);
      mm(fa0, fb0);
      sched_phase<NM1, NDS, TA::PIECES, 0>();
      rd(As, 2, fa0, fb0);
      load_b_lo(lb, kc_load);
      mm(fa1, fb1);
      sched_phase<NM1, NDS, HB, 0>();
      rd(As, 3, fa1, fb1);
      load_b_hi(lb, kc_load);
      mm(fa0, fb0);
      TA::store(An, sa, tid);
      sched_phase<NM1, NDS, TB1::PIECES - HB, TA::PIECES>();
      mm(fa1, fb1);
      TB1::store(An + TA::ELEMS, sb, tid);
      sched_phase<NM1, 0, 0, TB1::PIECES>();
      __syncthreads();
    };
    load_a(xa0, 0);
    load_b_lo(xb0, 0);
    load_b_hi(xb0, 0);
    load_a(xa1, 1);
    load_b_lo(xb1, 1);
    load_b_hi(xb1, 1);
    load_b2(rb0, 0);
    load_b2(rb1, 1);
    TA::store(s1, xa0, tid);
    TB1::store(s1 + TA::ELEMS, xb0, tid);
    __syncthreads();
    for (int kc = 0; kc < nk; kc += 2) {
      // chunk kc sits in buffer 0; set 1 holds chunk kc + 1 (in flight or landed)
      iteration(s1, s1 + STAGE, xa0, xb0, xa1, xb1, kc + 2);
      iteration(s1 + STAGE, s1, xa1, xb1, xa0, xb0, kc + 3);  // an all-zero chunk when nk is odd
    }
#pragma unroll
    for (int i = 0; i < TM1; ++i)
#pragma unroll
      for (int j = 0; j < TN1; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = wn * WN1 + j * 32 + q * 8 + (lane >> 5) * 4;
          uint2 w;
          w.x = pack_bf16x2(acc1[i][j][q * 4 + 0], acc1[i][j][q * 4 + 1]);
          w.y = pack_bf16x2(acc1[i][j][q * 4 + 2], acc1[i][j][q * 4 + 3]);
          *reinterpret_cast<uint2*>(Zs + (wm * WM1 + i * 32 + (lane & 31)) * L::Z_LD + c) = w;
        }
  } else if (p.z_splits == 0) {
    const bf16* __restrict__ Z = static_cast<const bf16*>(p.Z);
    constexpr int PPR = RT / 8;
#pragma unroll
    for (int i = 0; i < (MB * PPR) / 256; ++i) {
      const int piece = i * 256 + tid;
      const int r = piece / PPR, c = (piece % PPR) * 8;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (m0 + r < p.M && c < p.R) v = *reinterpret_cast<const uint4*>(Z + (int64_t)(m0 + r) * p.R + c);
      *reinterpret_cast<uint4*>(Zs + r * L::Z_LD + c) = v;
    }
  } else {
    // Sum of the fp32 split-K slabs in index order, rounded once to bf16.  The loads
    // are branch free (buffer windows, one per slab; a masked lane reads zero) and go
    // out four slabs x all pieces of the thread at a time, so the whole tile costs one
    // or two trips to memory instead of one per piece.
    const float* __restrict__ Zp = static_cast<const float*>(p.Z);
    constexpr int PPR = RT / 4;
    constexpr int NP = (64 * PPR) / 256;  // pieces of four floats per thread and 64 rows
    constexpr int MAXS = 8, GROUP = 4;
    for (int h = 0; h < MB / 64; ++h) {  // 64 rows at a time: bounds the registers in flight
    unsigned off[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int piece = i * 256 + tid;
      const int r = h * 64 + piece / PPR, c = (piece % PPR) * 4;
      off[i] = c < p.R ? (unsigned)(r * p.R + c) * 4u : OOB_OFFSET;  // rows past M fall outside
    }
    float4 sum[NP];
#pragma unroll
    for (int g = 0; g < MAXS / GROUP; ++g) {
      if (g * GROUP < p.z_splits) {  // uniform
        f32x4 v[GROUP][NP];
#pragma unroll
        for (int k = 0; k < GROUP; ++k) {
          const int sp = g * GROUP + k;
          // slabs past z_splits: an empty window, every lane reads zero
          const int64_t origin = (int64_t)sp * p.z_slab + (int64_t)m0 * p.R;
          const GWindow w = make_window(Zp, origin, sp < p.z_splits ? (int64_t)sp * p.z_slab + (int64_t)p.M * p.R : origin, 4);
#pragma unroll
          for (int i = 0; i < NP; ++i)
            v[k][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(w.rsrc, (int)off[i], 0, 0));
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
#pragma unroll
          for (int k = 0; k < GROUP; ++k) {
            if (g == 0 && k == 0) sum[i] = make_float4(v[0][i].x, v[0][i].y, v[0][i].z, v[0][i].w);
            else { sum[i].x += v[k][i].x; sum[i].y += v[k][i].y; sum[i].z += v[k][i].z; sum[i].w += v[k][i].w; }
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int piece = i * 256 + tid;
      const int r = h * 64 + piece / PPR, c = (piece % PPR) * 4;
      uint2 w;
      w.x = pack_bf16x2(sum[i].x, sum[i].y);
      w.y = pack_bf16x2(sum[i].z, sum[i].w);
      *reinterpret_cast<uint2*>(Zs + r * L::Z_LD + c) = w;
      // (asked for: the token tile's first work-group leaves its columns behind)
      if (p.z_out != nullptr && slice == 0 && c >= p.z_first && c < p.R && m0 + r < p.M)
        *reinterpret_cast<uint2*>(static_cast<bf16*>(p.z_out) + (int64_t)(m0 + r) * (p.R - p.z_first) + (c - p.z_first)) = w;
    }
    }  // h
  }
  if (LEAN) load_b2(rb1, 1);   // (its registers held slabs)
  __syncthreads();  // Zt complete; stage-1 buffers (aliasing Bbuf) are free

  // all rows of Zt, as MFMA fragments, in every wave for the rest of the kernel
  bf16x8 fa[MT][KS];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[i][ks] = read_frag_rowmajor<L::Z_LD>(Zs, i * 32, ks, lane);

  TB2::store(Bbuf, rb0, tid);
  __syncthreads();

  const float scale = p.scale;

  // Finished tiles leave through LDS, in whole rows: wave w stores rows MB / 4 * w .. of what all
  // waves have put into the tile's buffer by the barrier that ends its step.  (Straight
  // from registers a store instruction wrote 32-byte segments of 32 rows: 8192 wide, 4096
  // tokens, R = 16, where the stores are what bounds it, forward expansion 22.1 -> 18.1 us, 3.7
  // TB/s, input gradient 19.8 -> 17.1; level where the first contraction dominates.)  The 16-byte
  // pieces of a row are XOR-swizzled by row, so neither side conflicts; rows past M and columns
  // past N fall outside the window.
  const GWindow out_w = make_window(p.C, (int64_t)m0 * p.ldc, (int64_t)p.M * p.ldc, 2);
  constexpr int ROWS_OUT = MB / 16;   // store instructions per wave and tile
  auto tile_read = [&](const unsigned char* buf, uint4 (&v)[ROWS_OUT]) {
#pragma unroll
    for (int u = 0; u < ROWS_OUT; ++u) {
      const int row = wave * (MB / 4) + u * 4 + (lane >> 4);
      v[u] = *reinterpret_cast<const uint4*>(buf + row * 256 + (((lane & 15) ^ (row & 15)) * 16));
    }
  };
  auto tile_store = [&](int jt, const uint4 (&v)[ROWS_OUT]) {
    const int gn = (t_begin + jt) * CS_BN + (lane & 15) * 8;
    const unsigned row = (unsigned)(wave * (MB / 4) + (lane >> 4));
    const unsigned at = jt >= 0 && jt < my_tiles && gn < p.N ? (row * (unsigned)p.ldc + (unsigned)gn) * 2u : OOB_OFFSET;
#pragma unroll
    for (int u = 0; u < ROWS_OUT; ++u) window_store16(out_w, at + (unsigned)(u * 8) * (unsigned)p.ldc, v[u]);
  };

  // One [MB x 128] output tile (wave w owns columns 32 w .. 32 w + 31 of it) from the B2
  // tile in `Bs`.  Between its MFMAs go the loads of the tile two ahead (into rl), the
  // next tile's bias (into bvn) and the LDS stores of the next tile (from rs, loaded one
  // step ago, into Bn): issued in one burst, the loads hold every wave at the memory
  // pipe's queue while LDS and MFMA sit idle.
  // The tile before it leaves from `done`; its own result goes to `out`.
  auto step = [&](int jt, const bf16* Bs, bf16* Bn, const uint2 (&bv)[4], uint2 (&bvn)[4],
                  uint4 (&rl)[TB2::PIECES], uint4 (&rs)[TB2::PIECES], const unsigned char* done, unsigned char* out) {
    uint4 leaving[ROWS_OUT];
    if constexpr (!SHORT) tile_read(done, leaving);
    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    bf16x8 fb = read_frag<B2_KC, TB2::LD>(Bs, wave * 32, 0, lane);
    __builtin_amdgcn_sched_barrier(0);
    load_bias(bvn, jt + 1);
    load_b2(rl, jt + 2);
    // (an LDS store may not pass an LDS read in the compiler's eyes, so each k step's
    // store sits where the schedule wants it: after the reads of the step that follows;
    // reading the fragments two steps ahead instead of one measured no faster)
    static_for<0, KS>([&](auto ksc) {
      constexpr int ks = decltype(ksc)::value;
      bf16x8 fbn = fb;
      if (ks + 1 < KS) fbn = read_frag<B2_KC, TB2::LD>(Bs, wave * 32, ks + 1, lane);
#pragma unroll
      for (int i = 0; i < MT; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa[i][ks], acc[i], 0, 0, 0);
      TB2::template store<ks, ks + 1>(Bn, rs, tid);
      fb = fbn;
    });
    sched_stage2<KS, B2_KC ? 1 : 2, MT>();
    if constexpr (!SHORT) tile_store(jt - 1, leaving);
    // A lane holds, per 8-column group q, the four columns 8 q + 4 (l / 32) .. +3 of its row;
    // exchanging the upper half-wave's part of an even group with the lower half-wave's part
    // of the odd group next to it (v_permlane32_swap) leaves every lane with eight
    // consecutive columns: 16 bytes, piece 4 w + 2 pr + l / 32 of the tile's row.
    auto rows_out = [&](const f32x16& acc, int row0) {
      const int row = row0 + (lane & 31);
#pragma unroll
      for (int pr = 0; pr < 2; ++pr) {
        uint2 w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int q = 2 * pr + h;
          const float b0 = bf16_bits_to_float(bv[q].x & 0xffffu), b1 = bf16_bits_to_float(bv[q].x >> 16);
          const float b2 = bf16_bits_to_float(bv[q].y & 0xffffu), b3 = bf16_bits_to_float(bv[q].y >> 16);
          w[h].x = pack_bf16x2(acc[q * 4 + 0] * scale + b0, acc[q * 4 + 1] * scale + b1);
          w[h].y = pack_bf16x2(acc[q * 4 + 2] * scale + b2, acc[q * 4 + 3] * scale + b3);
        }
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 s0 = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
        const u32x2 s1 = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
        const int piece = wave * 4 + pr * 2 + (lane >> 5);
        const uint4 v = make_uint4(s0.x, s1.x, s0.y, s1.y);
        if constexpr (SHORT) {
          const int gn = (t_begin + jt) * CS_BN + piece * 8;
          window_store16(out_w, gn < p.N ? ((unsigned)row * (unsigned)p.ldc + (unsigned)gn) * 2u : OOB_OFFSET, v);
        } else {
          *reinterpret_cast<uint4*>(out + row * 256 + ((piece ^ (row & 15)) * 16)) = v;
        }
      }
    };
    if (L::OUTS == 1) __syncthreads();   // (everybody has read the tile before it)
#pragma unroll
    for (int i = 0; i < MT; ++i) rows_out(acc[i], i * 32);
    __syncthreads();
  };

  unsigned char* const out0 = smem;
  unsigned char* const out1 = smem + (L::OUTS == 2 ? L::OUT_BYTES : 0);
  for (int jt = 0; jt < my_tiles; jt += 2) {
    // tile jt sits in buffer 0; set 1 holds tile jt + 1
    step(jt, Bbuf, Bbuf + TB2::ELEMS, bv0, bv1, rb0, rb1, out1, out0);
    // (behind an odd last tile a step on zeros, 2000 cycles, would hold up its stores: [2048 x 768] -> 768,
    // R = 128, forward 11.4 us with it, 10.8 without)
    if (jt + 1 < my_tiles) step(jt + 1, Bbuf + TB2::ELEMS, Bbuf, bv1, bv0, rb1, rb0, out0, out1);
  }
  if constexpr (!SHORT) {
    uint4 leaving[ROWS_OUT];
    tile_read(my_tiles & 1 ? out0 : out1, leaving);
    tile_store(my_tiles - 1, leaving);
  }
}
// The same chain with both stages fused, for token tiles of 64 rows: every operand goes straight into LDS.
//   - stage 1 runs on a ring of four 64-wide chunks of x and B1 (as sk_bf16_ring.h: two phases of two k steps a chunk,
//     one barrier, the loads up to four chunks ahead);
//   - stage 2 on a ring of whole [R x 128] tiles of B2, each with its bias: a phase multiplies half of a tile's
//     k steps and reads the other half, or the first half of the next tile; a finished tile is turned over in LDS and
//     leaves in the second phase of the next step (runs of few tiles: straight from registers).
// What it waits for: loads through registers, two chunks or tiles ahead, left a work-group alone on its CU 1110 cycles
// a chunk (256 of MFMAs) and 2090 a tile (512).  Forward, us, before : now: 4096 tokens, 768 -> 3072, R = 128
// 18.4 : 16.2; 768 -> 768, R = 128 11.8 : 9.7, R = 32 9.5 : 8.1; 1119, 944 -> 496, R = 32 9.2 : 7.0.
template <int RT, bool KC, bool SHORT>
struct ChainRing {
  static constexpr int KS = RT / 16, KH = KS / 2;
  static constexpr int S1 = 4, SLOT1 = (64 + RT) * 128, L1A = 2, L1B = RT / 32, L1 = L1A + L1B;
  static constexpr int S2 = RT == 128 ? 3 : 4, SLOT2 = RT * 256, L2 = RT / 16 + 1;   // (a tile's loads and its bias)
  static constexpr int Z_LD = RT + 8, Z_BYTES = 64 * Z_LD * 2, OUT_BYTES = 64 * 256;
  static constexpr int HEAD = SHORT ? (Z_BYTES + 1023) / 1024 * 1024 : 2 * OUT_BYTES;   // Zt, then two finished tiles
  static constexpr int RING = S1 * SLOT1 > S2 * SLOT2 ? S1 * SLOT1 : S2 * SLOT2;
  static constexpr int BIAS_AT = HEAD + RING, BIAS_TILES = 2 * S2;
  static constexpr int BYTES = BIAS_AT + BIAS_TILES * 256;
  static constexpr int STORES = 4;                                                   // of a wave per step
  static_assert(Z_BYTES <= HEAD && BYTES <= 160 * 1024, "LDS of a compute unit");
};

template <int RT, bool KC, bool SHORT>
__device__ __forceinline__ void chain_ring(const ChainArgs& p) {
  typedef ChainRing<RT, KC, SHORT> L;
  typedef Panels<true> PA;
  typedef Panels<KC> PB;
  constexpr int TN1 = RT / 64;   // stage 1: waves 2 x 2, each 32 rows x RT / 2 columns of Zt
  constexpr int KS = L::KS, KH = L::KH;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[L::BYTES];
  // (what the loads write is invisible to the compiler: it must not take smem for unwritten)
  asm volatile("" ::"v"((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem) : "memory");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int wg = xcd_remap(blockIdx.x, p.tiles_m * p.n_slices);
  const int tile_m = wg / p.n_slices, slice = wg % p.n_slices;
  const int m0 = tile_m * 64;
  const int n_tiles = (p.N + CS_BN - 1) / CS_BN;
  const int per_slice = (n_tiles + p.n_slices - 1) / p.n_slices;
  const int t_begin = slice * per_slice;
  const int t_end = (t_begin + per_slice < n_tiles) ? t_begin + per_slice : n_tiles;
  const int my_tiles = t_end - t_begin;
  if (my_tiles <= 0) return;  // uniform over the work-group

  // ---------------- stage 1: Zt = A . B1 ----------------
  {
    const unsigned lda = (unsigned)p.lda * 2u, ldb = (unsigned)p.ldb1 * 2u;   // bytes
    const unsigned va = PA::load_offset(wave, lane, lda), vb = PB::load_offset(wave, lane, ldb);
    const int lane_k = PA::load_k(wave, lane);
    const unsigned step_b = KC ? 128u : ldb * 64u, panel_b = KC ? ldb * 64u : 128u;
    u32x4 a_src = scalar(descriptor(p.A, (int64_t)m0 * p.lda, (int64_t)p.M * p.lda, 2));
    u32x4 b_src = scalar(descriptor(p.B1, 0, KC ? (int64_t)p.R * p.ldb1 : (int64_t)p.K1 * p.ldb1, 2));
    unsigned a_off = 0, b_off = 0, s_slot = L::HEAD;
    int left = p.K1;
    auto load_a = [&](int i) { load_to_lds(s_slot + i * 4096 + wave * 1024, lane_k < left ? va : OOB_OFFSET, a_src, a_off + (i ? lda * 32u : 0u)); };
    auto load_b = [&](int i) {
      load_to_lds(s_slot + 8192 + i * 4096 + wave * 1024, KC ? (lane_k < left ? vb : OOB_OFFSET) : vb, b_src,
                  b_off + (i & 1 ? ldb * 32u : 0u) + (i >> 1) * panel_b);
    };
    auto next_chunk = [&]() {
      left -= 64;
      a_off += 128u; b_off += step_b;
      if (left <= 0) a_src.z = b_src.z = 0;   // past the last chunk nothing is fetched
      s_slot = s_slot + L::SLOT1 == L::HEAD + L::S1 * L::SLOT1 ? L::HEAD : s_slot + L::SLOT1;
    };
    bf16x8 fa[2][2], fb[2][2][TN1];
    const unsigned a_read = PA::read_address(0, lane) + wm * 4096;
    const unsigned b_0 = PB::read_address(0, lane);
    const unsigned b_read = 8192 + (KC ? b_0 + wn * TN1 * 4096 : TN1 == 2 ? b_0 + wn * 8192 : b_0 ^ (wn << 6));
    auto read_a = [&](int set, int s, unsigned slot, int ks) { fa[set][s] = PA::frag(slot + a_read, 0, ks); };
    auto read_b = [&](int set, int s, int j, unsigned slot, int ks) { fb[set][s][j] = PB::frag(slot + b_read, j, ks); };
#pragma unroll
    for (int c = 0; c < L::S1; ++c) {
#pragma unroll
      for (int i = 0; i < L::L1A; ++i) load_a(i);
      if (c == L::S1 - 1) break;   // (the last chunk's loads of B1 are the first phase's)
#pragma unroll
      for (int i = 0; i < L::L1B; ++i) load_b(i);
      next_chunk();
    }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((L::S1 - 2) * L::L1 + L::L1A) : "memory");   // chunk 0
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      read_a(0, s, L::HEAD, s);
#pragma unroll
      for (int j = 0; j < TN1; ++j) read_b(0, s, j, L::HEAD, s);
    }
    f32x16 acc[TN1];
#pragma unroll
    for (int j = 0; j < TN1; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    unsigned c_slot = L::HEAD;
    const int nk = (p.K1 + 63) / 64;
    for (int kc = 0; kc < nk; ++kc) {
      const unsigned n_slot = c_slot + L::SLOT1 == L::HEAD + L::S1 * L::SLOT1 ? L::HEAD : c_slot + L::SLOT1;
      auto phase = [&](auto h_c) {   // (see sk_bf16_ring.h)
        constexpr int H = decltype(h_c)::value, NM = 2 * TN1, NR = 2 * (1 + TN1), NL = H == 0 ? L::L1B : L::L1A;
        const unsigned slot = H == 0 ? c_slot : n_slot;
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, NM>([&](auto tc) {
          constexpr int t = decltype(tc)::value;
          static_for<t * NR / NM, (t + 1) * NR / NM>([&](auto rc) {
            constexpr int r = decltype(rc)::value, s = r / (1 + TN1), e = r % (1 + TN1);
            if constexpr (e < TN1) read_b(1 - H, s, e, slot, 2 * (1 - H) + s);
            else read_a(1 - H, s, slot, 2 * (1 - H) + s);
          });
          static_for<t * NL / NM, (t + 1) * NL / NM>([&](auto lc) {
            if constexpr (H == 0) load_b(decltype(lc)::value);
            else load_a(decltype(lc)::value);
          });
          constexpr int s = t / TN1, j = t % TN1;
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[H][s][j], fa[H][s], acc[j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        });
      };
      phase(IntC<0>{});
      next_chunk();
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((L::S1 - 2) * L::L1) : "memory");
      phase(IntC<1>{});
      c_slot = n_slot;
    }
    // rounded once to bf16; columns past R are zeros (B1 may hold anything there: its rows' neighbours)
    bf16* const Zs = reinterpret_cast<bf16*>(smem);
#pragma unroll
    for (int j = 0; j < TN1; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = wn * (RT / 2) + j * 32 + q * 8 + (lane >> 5) * 4;
        uint2 w;
        w.x = c < p.R ? pack_bf16x2(acc[j][q * 4 + 0], acc[j][q * 4 + 1]) : 0u;
        w.y = c < p.R ? pack_bf16x2(acc[j][q * 4 + 2], acc[j][q * 4 + 3]) : 0u;
        *reinterpret_cast<uint2*>(Zs + (wm * 32 + (lane & 31)) * L::Z_LD + c) = w;
      }
  }
  // Zt complete, stage 1's ring read by everybody and nothing under way into it
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  // ---------------- stage 2: one [64 x 128] output tile a step ----------------
  const unsigned ldb2 = (unsigned)p.ldb2 * 2u;
  const unsigned v2 = PB::load_offset(wave, lane, ldb2);
  const int lane_k2 = PA::load_k(wave, lane);
  u32x4 b2_src{}, bias_src{};
  auto set_tile = [&](int jt) {   // (past the run: nothing to fetch)
    const int n0 = (t_begin + jt) * CS_BN;
    b2_src = scalar(descriptor(p.B2, KC ? (int64_t)n0 * p.ldb2 : (int64_t)n0, jt >= my_tiles ? 0 : KC ? (int64_t)p.N * p.ldb2 : (int64_t)(p.R - 1) * p.ldb2 + p.N, 2));
    bias_src = scalar(descriptor(p.bias, n0, p.bias != nullptr && jt < my_tiles ? p.N : 0, 2));
  };
  // load i of the tile into `slot`: 32 lines of panel (n panel, k panel)
  auto load2 = [&](int i, unsigned slot) {
    const int kp = i >> 2, np = (i >> 1) & 1, h = i & 1;
    load_to_lds(slot + (unsigned)((np * (RT / 64) + kp) * 8192 + h * 4096) + wave * 1024, KC ? (lane_k2 + kp * 64 < p.R ? v2 : OOB_OFFSET) : v2, b2_src,
                (h ? ldb2 * 32u : 0u) + (KC ? np * ldb2 * 64u + kp * 128u : kp * ldb2 * 64u + np * 128u));
  };
  auto load_bias = [&](int jt) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(L::BIAS_AT + (jt % L::BIAS_TILES) * 256), "v"(lane * 4), "s"(bias_src) : "m0");
  };
#pragma unroll
  for (int t = 0; t < L::S2; ++t) {
    set_tile(t);
    load_bias(t);
#pragma unroll
    for (int i = 0; i < L::L2 - 1; ++i) load2(i, L::HEAD + t * L::SLOT2);
  }
  // all rows of Zt, as MFMA fragments, in every wave for the rest of the kernel
  bf16x8 fz[2][KS];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fz[i][ks] = read_frag_rowmajor<L::Z_LD>(reinterpret_cast<const bf16*>(smem), i * 32, ks, lane);
  bf16x8 f2[2][KH];
  const unsigned b2_0 = PB::read_address(0, lane);
  const unsigned b2_read = (wave >> 1) * (RT / 64) * 8192 + (KC ? b2_0 + (wave & 1) * 4096 : b2_0 ^ ((wave & 1) << 6));
  auto read2 = [&](int set, int s, unsigned slot, int ks) { f2[set][s] = PB::frag(slot + b2_read + (ks >> 2) * 8192, 0, ks & 3); };
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((L::S2 - 1) * L::L2) : "memory");   // tile 0; Zt is in registers
#pragma unroll
  for (int s = 0; s < KH; ++s) read2(0, s, L::HEAD, s);

  const float scale = p.scale;
  const GWindow out_w = make_window(p.C, (int64_t)m0 * p.ldc, (int64_t)p.M * p.ldc, 2);
  // whole rows of the finished tile jt (none if jt is not one): wave w stores rows 16 w .. + 15
  auto tile_out = [&](int jt) {
    const unsigned char* const buf = smem + (jt & 1) * L::OUT_BYTES;
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = wave * 16 + u * 4 + (lane >> 4);
      v[u] = *reinterpret_cast<const uint4*>(buf + row * 256 + (((lane & 15) ^ (row & 15)) * 16));
    }
    const int gn = (t_begin + jt) * CS_BN + (lane & 15) * 8;
    const unsigned at = jt >= 0 && gn < p.N ? ((unsigned)(wave * 16 + (lane >> 4)) * (unsigned)p.ldc + (unsigned)gn) * 2u : OOB_OFFSET;
#pragma unroll
    for (int u = 0; u < 4; ++u) window_store16(out_w, at + (unsigned)(u * 8) * (unsigned)p.ldc, v[u]);
  };
  unsigned c_slot = L::HEAD;
  for (int jt = 0; jt < my_tiles; ++jt) {
    const unsigned n_slot = c_slot + L::SLOT2 == L::HEAD + L::S2 * L::SLOT2 ? L::HEAD : c_slot + L::SLOT2;
    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    set_tile(jt + L::S2);
    auto phase = [&](auto h_c) {
      constexpr int H = decltype(h_c)::value;
      const unsigned slot = H == 0 ? c_slot : n_slot;
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, KH>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        read2(1 - H, s, slot, KH * (1 - H) + s);
        if constexpr (H == 1) {   // this tile's slot is free
          if constexpr (s == 0) load_bias(jt + L::S2);
          static_for<s*(L::L2 - 1) / KH, (s + 1) * (L::L2 - 1) / KH>([&](auto lc) { load2(decltype(lc)::value, c_slot); });
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[H][s], fz[i][KH * H + s], acc[i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    phase(IntC<0>{});
    // This tile is in registers, the tile before it in LDS, the next tile has landed: younger than its loads are those of S2 - 2
    // tiles and, once it was not among the first S2, the stores of S2 - 1 steps.
    if (jt + 1 >= L::S2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((L::S2 - 2) * L::L2 + (L::S2 - 1) * L::STORES) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((L::S2 - 2) * L::L2) : "memory");
    phase(IntC<1>{});
    if constexpr (!SHORT) tile_out(jt - 1);
    // ---- this wave's 32 columns of the tile (see chain_small) ----
    const unsigned char* const bias = smem + L::BIAS_AT + (jt % L::BIAS_TILES) * 256 + wave * 64;
    unsigned char* const out = smem + (jt & 1) * L::OUT_BYTES;
    uint2 bv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bv[q] = *reinterpret_cast<const uint2*>(bias + (q * 8 + (lane >> 5) * 4) * 2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = i * 32 + (lane & 31);
#pragma unroll
      for (int pr = 0; pr < 2; ++pr) {
        uint2 w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int q = 2 * pr + h;
          const float b0 = bf16_bits_to_float(bv[q].x & 0xffffu), b1 = bf16_bits_to_float(bv[q].x >> 16);
          const float b2 = bf16_bits_to_float(bv[q].y & 0xffffu), b3 = bf16_bits_to_float(bv[q].y >> 16);
          w[h].x = pack_bf16x2(acc[i][q * 4 + 0] * scale + b0, acc[i][q * 4 + 1] * scale + b1);
          w[h].y = pack_bf16x2(acc[i][q * 4 + 2] * scale + b2, acc[i][q * 4 + 3] * scale + b3);
        }
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 s0 = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
        const u32x2 s1 = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
        const int piece = wave * 4 + pr * 2 + (lane >> 5);
        const uint4 v = make_uint4(s0.x, s1.x, s0.y, s1.y);
        if constexpr (SHORT) {
          const int gn = (t_begin + jt) * CS_BN + piece * 8;
          window_store16(out_w, gn < p.N ? ((unsigned)row * (unsigned)p.ldc + (unsigned)gn) * 2u : OOB_OFFSET, v);
        } else {
          *reinterpret_cast<uint4*>(out + row * 256 + ((piece ^ (row & 15)) * 16)) = v;
        }
      }
    }
    c_slot = n_slot;
  }
  // the last tile leaves; no load may land in LDS that is someone else's
  if constexpr (!SHORT) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    tile_out(my_tiles - 1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// RING: both stages on rings of loads (chain_ring), for fused launches of 64-row tiles.
template <int MB, int RT, bool B2_KC, bool FUSED, bool B1_KC, bool RING, bool SHORT>
__device__ __forceinline__ void chain_body(const ChainArgs& p) {
  if constexpr (RING) {
    chain_ring<RT, B2_KC, SHORT>(p);
  } else {
    __shared__ __attribute__((aligned(16))) unsigned char smem[SmallLds<MB, RT, B2_KC, FUSED, B1_KC, SHORT>::BYTES];
    chain_small<MB, RT, B2_KC, FUSED, B1_KC, SHORT>(p, blockIdx.x, smem);
  }
}
template <int MB, int RT, bool B2_KC, bool FUSED, bool B1_KC, bool RING = false>
__global__ __launch_bounds__(256, chain_outs(MB, RT) == 1 ? 2 : 1) void chain_small_kernel(const ChainArgs p) {
  chain_body<MB, RT, B2_KC, FUSED, B1_KC, RING, false>(p);
}
template <int MB, int RT, bool B2_KC, bool FUSED, bool B1_KC, bool RING = false>
__global__ __launch_bounds__(256) void chain_short_kernel(const ChainArgs p) {
  chain_body<MB, RT, B2_KC, FUSED, B1_KC, RING, true>(p);
}

// Z^T . dY in ranges of tokens beside the expansion of dX over runs of 64-row tiles (long ones, which leave through LDS, up to R = 64),
// in one launch: the first `groups_a` work-groups and the rest, two to a CU (72 KB of LDS and 240 registers at most).  Each of
// the two by itself is a round of work-groups that wait for their first operands and for their last stores, one reading
// dY, the other writing dX; beside each other they wait at the same time.  The sum of the ranges, which the expansion carried while it came
// last, has a launch of its own again (2 to 3 us).  Backward pass, us, expansion behind : beside: 4096 tokens, 768 -> 3072, R = 128 35.0 : 34.0;
// 2048, 768 -> 768, R = 128 22.9 : 21.2; 1000, 512 -> 1024, R = 48 15.0 : 12.7; x . S in ranges: 418, 3616 -> 272, R = 80 21.0 : 15.7; 62 of 150 layers of
// 300 to 16384 tokens, 256 to 4096 wide, take it with short runs, in 0.89 of the time.  Long runs: 9295, 960 -> 1504, R = 16 35.8 : 32.3; 4096, 8192 -> 8192,
// R = 16 67.8 : 65.8; 36 of 150 such layers 0.95, 48 of 80 of 4096 to 8192 wide, R 16 to 96, 0.94.  (R = 128 with long runs would be one to a CU.)
template <int BM, int RT, bool SHORT = true>
__global__ __launch_bounds__(256, 2) void factor_beside_expand_kernel(const GemmArgs a, const ChainArgs c, const int groups_a) {
  typedef RingTile<BM, 64, true, false, float, true> G;
  typedef SmallLds<64, RT, true, false, true, SHORT> L;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[G::LDS_BYTES > L::BYTES ? G::LDS_BYTES : L::BYTES];
  if ((int)blockIdx.x < groups_a) G::run(a, blockIdx.x, smem);
  else chain_small<64, RT, true, false, true, SHORT, true>(c, (int)blockIdx.x - groups_a, smem);
}

bool chain_supported(int R) { return R >= 16 && R <= 512; }

// Flops and bytes of a chain launch: both contractions when the first one is fused in,
// otherwise the second one with the intermediate (or its slabs) read from memory; the
// reduction it may carry along counts by its bytes.
static Work chain_work(const ChainArgs& a, bool fused) {
  Work w;
  w.flops = 2.0 * a.M * a.R * ((fused ? a.K1 : 0) + (double)a.N);
  w.bytes = 2.0 * ((double)a.R * a.N + (double)a.M * a.N) + (a.bias != nullptr ? 2.0 * a.N : 0.0);
  if (fused) w.bytes += 2.0 * ((double)a.M * a.K1 + (double)a.K1 * a.R);
  else w.bytes += (double)a.M * a.R * (a.z_splits == 0 ? 2.0 : 4.0 * a.z_splits);
  w.bytes += reduce_work(a.tail).bytes;
  return w;
}

template <int RT, int BN, bool B2_KC, bool FUSED, bool B1_KC>
static hipError_t launch_one(const ChainArgs& a, hipStream_t s) {
  const long long grid = (long long)a.tiles_m * a.n_slices;
  if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  static const std::string name =
      kernel_label("chain_kernel", {lbl(RT), lbl(BN), lbl(B2_KC), lbl(FUSED), lbl(B1_KC)});
  return launch_kernel(name.c_str(), chain_work(a, FUSED), chain_kernel<RT, BN, B2_KC, FUSED, B1_KC>, dim3((unsigned)grid), dim3(256),
                       s, a);
}

static bool brief_runs(const ChainArgs& a, int mb) {
  const int run = ((a.N + CS_BN - 1) / CS_BN + a.n_slices - 1) / a.n_slices;
  return run <= (mb == 64 ? 3 : 2) || a.tiles_m == 1;
}

template <int MB, int RT, bool B2_KC, bool FUSED, bool B1_KC>
static hipError_t launch_small_mb(const ChainArgs& a, hipStream_t s) {
  const long long grid = (long long)a.tiles_m * a.n_slices;
  if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  // Runs of up to three tiles (two of 128 rows) are over before whole rows pay for the trip through LDS, the
  // barrier behind the last tile and the room for them, us, through LDS : straight: [9007 x 144] -> 208, R = 112,
  // runs of 2, 8.2 : 7.8; [84448 x 64] -> 176, R = 48, runs of 2 of 128 rows, 17.1 : 15.7; [2048 x 768] -> 768,
  // R = 128, runs of 1, 10.9 : 10.8; [40000 x 384] -> 384, R = 32, runs of 3 of 128 rows, 17.6 : 18.2; [4096 x 1024] ->
  // 2048, R = 64, runs of 4, 13.9 : 14.2; [30000 x 768] -> 768, R = 64, runs of 6, 19.3 : 20.6.
  // A lone token tile has next to nothing to store beside the weights it reads ([1 x 528] -> 131072, R = 128,
  // runs of 4, 13.5 : 12.4).
  const bool brief = brief_runs(a, MB);
  // Fused launches of 64-row tiles run on rings but for those of a narrow sketch in more than a round: there the rings and the
  // finished tiles would leave room for one work-group on a CU (of short runs, two) instead of two and more, us, on rings : without:
  // [12128 x 1728] -> 3872, R = 16, 46.2 : 35.6; [11483 x 624] -> 3328, R = 32, 29.7 : 23.9; short runs, [17339 x 512] -> 176, R = 32,
  // 11.5 : 10.6; [22078 x 112] -> 192, R = 32, 9.2 : 8.6.
  const bool ring = RT > 64 || grid <= NUM_CUS;
  const Work work = chain_work(a, FUSED);
  if constexpr (FUSED && MB == 64) {
    if (ring) {
      static const std::string names[2] = {kernel_label("chain_small_kernel", {lbl(MB), lbl(RT), lbl(B2_KC), lbl(FUSED), lbl(B1_KC), lbl(true)}),
                                           kernel_label("chain_short_kernel", {lbl(MB), lbl(RT), lbl(B2_KC), lbl(FUSED), lbl(B1_KC), lbl(true)})};
      return brief ? launch_kernel(names[1].c_str(), work, chain_short_kernel<MB, RT, B2_KC, FUSED, B1_KC, true>, dim3((unsigned)grid), dim3(256), s, a)
                   : launch_kernel(names[0].c_str(), work, chain_small_kernel<MB, RT, B2_KC, FUSED, B1_KC, true>, dim3((unsigned)grid), dim3(256), s, a);
    }
  }
  if constexpr (!(FUSED && MB == 64 && RT > 64)) {
    if (brief) {
      static const std::string name =
          kernel_label("chain_short_kernel", {lbl(MB), lbl(RT), lbl(B2_KC), lbl(FUSED), lbl(B1_KC)});
      return launch_kernel(name.c_str(), work, chain_short_kernel<MB, RT, B2_KC, FUSED, B1_KC>, dim3((unsigned)grid), dim3(256), s, a);
    }
    static const std::string name =
        kernel_label("chain_small_kernel", {lbl(MB), lbl(RT), lbl(B2_KC), lbl(FUSED), lbl(B1_KC)});
    return launch_kernel(name.c_str(), work, chain_small_kernel<MB, RT, B2_KC, FUSED, B1_KC>, dim3((unsigned)grid), dim3(256), s, a);
  }
  return hipErrorInvalidValue;
}

template <int RT, bool B2_KC, bool FUSED, bool B1_KC>
static hipError_t launch_small(const ChainArgs& a, hipStream_t s) {
  return a.bm == 128 ? launch_small_mb<128, RT, B2_KC, FUSED, B1_KC>(a, s)
                     : launch_small_mb<64, RT, B2_KC, FUSED, B1_KC>(a, s);
}

template <bool B_KC, bool FUSED>
static hipError_t launch_rt(const ChainArgs& a, hipStream_t s) {
  constexpr int BN = 128;
  if (a.z_splits > 8) return hipErrorInvalidValue;
  if (a.R <= 64) return launch_small<64, B_KC, FUSED, B_KC>(a, s);
  if (a.R <= 128) return launch_small<128, B_KC, FUSED, B_KC>(a, s);
  if (a.R <= 192) return launch_one<192, BN, B_KC, FUSED, B_KC>(a, s);
  if (a.R <= 256) return launch_one<256, BN, B_KC, FUSED, B_KC>(a, s);
  if (!FUSED) {  // the fused form needs LDS for both stages: R <= 256 only
    if (a.R <= 384) return launch_one<384, BN, B_KC, false, B_KC>(a, s);
    if (a.R <= 512) return launch_one<512, BN, B_KC, false, B_KC>(a, s);
  }
  return hipErrorInvalidValue;
}

int chain_bn(int R) { return R <= 128 ? CS_BN : 128; }

static void note_chain(bool b_kc, bool fused, const ChainArgs& a) {
  if (!tracing()) return;
  if (fused) {
    note_matrix(a.A, a.M, a.K1, a.lda, 2, false);
    note_matrix(a.B1, b_kc ? a.R : a.K1, b_kc ? a.K1 : a.R, a.ldb1, 2, false);
  } else if (a.z_splits == 0) {
    note_matrix(a.Z, a.M, a.R, a.R, 2, false);
  } else {   // fp32 slabs [M, R], z_slab elements apart
    note_matrix(a.Z, 1, (int64_t)(a.z_splits - 1) * a.z_slab + (int64_t)a.M * a.R, 0, 4, false);
  }
  note_matrix(a.B2, b_kc ? a.N : a.R, b_kc ? a.R : a.N, a.ldb2, 2, false);
  if (a.bias != nullptr) note_matrix(a.bias, 1, a.N, a.N, 2, false);
  note_matrix(a.C, a.M, a.N, a.ldc, 2, true);
  note_matrix(a.z_out, a.M, a.R - a.z_first, a.R - a.z_first, 2, true);
  note_reduce(a.tail);
}

hipError_t launch_chain_bf16(bool b_kc, bool fused, ChainArgs a, hipStream_t s) {
  if (!chain_supported(a.R) || a.n_slices < 1 || (fused && a.R > CHAIN_FUSED_MAX_R))
    return hipErrorInvalidValue;
  if (a.bm == 0) a.bm = CH_BM;
  if (a.bm != CH_BM && !(a.bm == 128 && a.R <= 128)) return hipErrorInvalidValue;
  if (fused && a.tail.n + a.tail.n2 > 0) return hipErrorInvalidValue;   // (no plan asks a fused launch to carry one)
  if (a.z_out != nullptr && (fused || a.z_splits == 0 || a.R > 128)) return hipErrorInvalidValue;
  a.tiles_m = (a.M + a.bm - 1) / a.bm;
  note_chain(b_kc, fused, a);
  if (b_kc) return fused ? launch_rt<true, true>(a, s) : launch_rt<true, false>(a, s);
  return fused ? launch_rt<false, true>(a, s) : launch_rt<false, false>(a, s);
}

// Up to two work-groups a CU in all: past that the two kinds queue (of six layers with 513 to 768 three were 7 % ahead, three 1 to 3 % behind).
bool factor_beside_expand_supported(int tile, const GemmArgs& a, const ChainArgs& c) {
  const int tiles_m = (c.M + 63) / 64;
  int bm, bn;
  tile_dims(tile, bm, bn);
  if ((tile != TILE_64x64 && tile != TILE_128x64) || c.bm != 64 || c.R > 128 || (c.R > 64) != (tile == TILE_128x64) || c.z_splits > 8) return false;
  ChainArgs t = c;
  t.tiles_m = tiles_m;
  const long long groups = (long long)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * a.splits + (long long)tiles_m * c.n_slices;
  return (brief_runs(t, 64) || c.R <= 64) && groups <= 2 * NUM_CUS;
}

template <int BM, int RT, bool SHORT = true>
static hipError_t launch_beside(GemmArgs a, const ChainArgs& c, hipStream_t s) {
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + 63) / 64;
  const int ga = a.tiles_m * a.tiles_n * a.splits;
  note_gemm(a, true, false, 2, 4, true);
  note_chain(true, false, c);
  Work work = gemm_work(a, 2, 4, true);
  const Work wc = chain_work(c, false);
  work.flops += wc.flops;
  work.bytes += wc.bytes;
  static const std::string name = kernel_label("factor_beside_expand_kernel", {lbl(BM), lbl(RT), lbl(SHORT)});
  return launch_kernel(name.c_str(), work, factor_beside_expand_kernel<BM, RT, SHORT>, dim3((unsigned)(ga + c.tiles_m * c.n_slices)), dim3(256), s, a, c, ga);
}

hipError_t launch_factor_beside_expand(int tile, GemmArgs a, ChainArgs c, hipStream_t s) {
  if (!factor_beside_expand_supported(tile, a, c) || c.tail.n + c.tail.n2 > 0 || !within_window(128, a.lda, 64, 2)) return hipErrorInvalidValue;
  c.tiles_m = (c.M + 63) / 64;
  if (tile == TILE_128x64) return launch_beside<128, 128>(a, c, s);
  return brief_runs(c, 64) ? launch_beside<64, 64>(a, c, s) : launch_beside<64, 64, false>(a, c, s);
}

}  // namespace sk
