// The bf16 GEMM tiles (same contract as sk_bf16_gemm.hip) on a ring of chunks in LDS: for launches of one round,
// whose work-groups have a CU to themselves or share it with one other.
#pragma once
#include "sk_bf16_lds.h"

namespace sk {

// Operands go from global memory straight into a ring of SLOTS 64-wide chunks in LDS, up to SLOTS chunks ahead.
// A chunk is two phases of two k steps: a phase multiplies what the one before has read and reads
// what the next will multiply, and the one barrier of a chunk lies between them -- behind it the next
// chunk is in LDS and this one's slot is free for the loads.
//
// A work-group with no other beside it waits for its loads: through registers, two chunks ahead, a chunk takes 750 cycles
// (64 x 64 tiles) to 1350 (128 x 128) where its MFMAs take 128 to 512.  Here (us, cold operands): 64 x 64 tiles, [4001 x 768] .
// [768 x 384] 10.2 -> 8.3; 128 x 128, S^T . x^T of [8192 x 1024] and R = 512 15.4 -> 12.5; Z^T . dY of
// [8192 x 4096] in two ranges 51.3 -> 45.1; [8192 x 1024] . [1024 x 512] 16.3 -> 14.8.  What bounds it now is the fill: with
// neither reads nor MFMAs the same loops take 80 to 95 % of the time (35 to 57 GB/s a CU, a chunk of a
// 128 x 128 tile 0.58 us), and neither more slots nor tiles that start at different k changed that.  A 256 x 128 tile, a wave's part 128 x 64,
// fills three quarters as much for the same products, 0.83 us a chunk: for expansions of one round (choose_expansion_tile).
template <int BM, int BN, bool A_KC, bool B_KC, typename OutT, bool COLSUM>
struct RingTile {
  static constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;   // waves 2 x 2
  static constexpr int SLOTS = BM == BN ? 4 : 3;
  static constexpr int A_BYTES = BM * 128, SLOT = (BM + BN) * 128;
  static constexpr int LDS_BYTES = SLOTS * SLOT;
  static constexpr int PER_CU = LDS_BYTES <= 80 * 1024 ? 2 : 1;
  static constexpr int LA = BM / 32, LB = BN / 32, LOADS = LA + LB;           // of a wave per chunk
  static constexpr int AHEAD = (SLOTS - 2) * LOADS;                           // loads in flight at a barrier
  static constexpr int STRIP = 32 * WN * 2;                                   // a wave's, for bf16 results
  static_assert(LDS_BYTES <= 160 * 1024 && 4 * STRIP <= LDS_BYTES && AHEAD + LOADS <= 63, "LDS of a compute unit, the load counter");
  static __device__ __forceinline__ void run(const GemmArgs& p, int block, unsigned char* smem);   // (smem: the kernel's only LDS, from address 0)
};

template <int BM, int BN, bool A_KC, bool B_KC, typename OutT, bool COLSUM>
__device__ __forceinline__ void
RingTile<BM, BN, A_KC, B_KC, OutT, COLSUM>::run(const GemmArgs& p, const int block, unsigned char* const smem) {
  typedef Panels<A_KC> PA;
  typedef Panels<B_KC> PB;
  // (what the loads write is invisible to the compiler: it must not take smem for unwritten)
  asm volatile("" ::"v"((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem) : "memory");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles = p.tiles_m * p.tiles_n;
  const int id = xcd_remap(block, tiles * p.splits), split = p.splits > 1 ? id / tiles : 0;
  int tile_m, tile_n;
  tile_coords(id - split * tiles, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int k0 = split * p.k_per_split, k_end = k0 + p.k_per_split < p.K ? k0 + p.k_per_split : p.K;
  const int nk = (k_end - k0 + 63) / 64;

  // This lane's bias values (see sk_bf16_gemm.hip), through a buffer window of N elements (none without a bias)
  constexpr bool BF16_OUT = sizeof(OutT) == 2;
  uint2 bias_r[BF16_OUT ? TN : 1][4];
  if constexpr (BF16_OUT) {
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

  // ---- the stream of chunks to load ----
  const unsigned lda = (unsigned)p.lda * 2u, ldb = (unsigned)p.ldb * 2u;   // bytes
  const unsigned va = PA::load_offset(wave, lane, lda), vb = PB::load_offset(wave, lane, ldb);
  const int lane_k = Panels<true>::load_k(wave, lane);   // (lines 32 and 64 further down: the same)
  const unsigned step_a = A_KC ? 128u : lda * 64u, step_b = B_KC ? 128u : ldb * 64u;        // next chunk
  const unsigned panel_a = A_KC ? lda * 64u : 128u, panel_b = B_KC ? ldb * 64u : 128u;      // next panel
  const int64_t a_total = A_KC ? (int64_t)p.M * p.lda : (int64_t)(p.K - 1) * p.lda + p.M;
  const int64_t b_total = B_KC ? (int64_t)p.N * p.ldb : (int64_t)(p.K - 1) * p.ldb + p.N;
  u32x4 a_src = scalar(descriptor(p.A, A_KC ? (int64_t)m0 * p.lda + k0 : (int64_t)k0 * p.lda + m0, a_total, 2));
  u32x4 b_src = scalar(descriptor(p.B, B_KC ? (int64_t)n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + n0, b_total, 2));
  unsigned a_off = 0, b_off = 0, s_slot = 0;   // the stream's chunk: byte offsets from the origins, slot
  int left = k_end - k0;                       // k left from it on
  // Past the k range a k-contiguous operand reads as zero; the other kind has only rows past the array there, and what it
  // reads past its m or n are rows or columns of the result that are not stored.
  auto load_a = [&](int i) {
    load_to_lds(s_slot + i * 4096 + wave * 1024, A_KC ? (lane_k < left ? va : OOB_OFFSET) : va, a_src,
                a_off + (i & 1 ? lda * 32u : 0u) + (i >> 1) * panel_a);
  };
  auto load_b = [&](int i) {
    load_to_lds(s_slot + A_BYTES + i * 4096 + wave * 1024, B_KC ? (lane_k < left ? vb : OOB_OFFSET) : vb, b_src,
                b_off + (i & 1 ? ldb * 32u : 0u) + (i >> 1) * panel_b);
  };
  // Offsets are 32-bit: an operand that is not k-contiguous takes its origin along whenever a chunk starts
  // 1 GB behind it, one whose rows are 8 MB apart or more with every chunk.
  auto rebase = [](u32x4& src, unsigned& off, const void* base, int64_t elements) {
    const uint64_t at = ((uint64_t)src.y << 32 | src.x) + off;
    src = descriptor((const void*)at, 0, ((int64_t)((uint64_t)base - at) >> 1) + elements, 2);
    off = 0;
  };
  auto next_chunk = [&]() {
    left -= 64;
    a_off += step_a; b_off += step_b;
    if (A_KC ? p.lda > 1 << 22 : a_off >= 1u << 30) rebase(a_src, a_off, p.A, a_total);
    if (B_KC ? p.ldb > 1 << 22 : b_off >= 1u << 30) rebase(b_src, b_off, p.B, b_total);
    if (left <= 0) a_src.z = b_src.z = 0;   // past the last chunk nothing is fetched
    s_slot = s_slot + SLOT == SLOTS * SLOT ? 0 : s_slot + SLOT;
  };

  // ---- fragments: two sets of two k steps ----
  bf16x8 fa[2][2][TM], fb[2][2][TN];
  const unsigned a_0 = PA::read_address(0, lane), b_0 = PB::read_address(0, lane);
  const unsigned a_read = A_KC || TM >= 2 ? a_0 + wm * TM * 4096 : a_0 ^ (wm << 6);
  const unsigned b_read = A_BYTES + (B_KC || TN >= 2 ? b_0 + wn * TN * 4096 : b_0 ^ (wn << 6));
  auto read_a = [&](int set, int s, int i, unsigned slot, int ks) { fa[set][s][i] = PA::frag(slot + a_read, i, ks); };
  auto read_b = [&](int set, int s, int j, unsigned slot, int ks) { fb[set][s][j] = PB::frag(slot + b_read, j, ks); };

#pragma unroll
  for (int c = 0; c < SLOTS; ++c) {
#pragma unroll
    for (int i = 0; i < LA; ++i) load_a(i);
    if (c == SLOTS - 1) break;   // (the last chunk's loads of B are the first phase's)
#pragma unroll
    for (int i = 0; i < LB; ++i) load_b(i);
    next_chunk();
  }
  // chunk 0: all but SLOTS - 2 chunks and A's loads of the last
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(AHEAD + LA) : "memory");
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int i = 0; i < TM; ++i) read_a(0, s, i, 0, s);
#pragma unroll
    for (int j = 0; j < TN; ++j) read_b(0, s, j, 0, s);
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // column sums of B ride on the MFMA: an all-ones fragment in place of A's
  f32x16 csum[COLSUM ? TN : 1];
  const bool do_colsum = COLSUM && p.colsum != nullptr && tile_m == 0 && wm == 0;
  bf16x8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (bf16)1.0f;
  if constexpr (COLSUM) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) csum[j][r] = 0.f;
  }

  unsigned c_slot = 0;   // where the chunk being multiplied lies
  for (int kc = 0; kc < nk; ++kc) {
    const unsigned n_slot = c_slot + SLOT == SLOTS * SLOT ? 0 : c_slot + SLOT;
    // H = 0: multiplies k steps 0, 1, reads 2, 3 of this chunk, B's loads of the stream's chunk;
    // H = 1: multiplies 2, 3, reads 0, 1 of the next chunk, A's loads of the stream's next
    auto phase = [&](auto h_c) {
      constexpr int H = decltype(h_c)::value;
      constexpr int NM = 2 * TM * TN, NR = 2 * (TM + TN), NL = H == 0 ? LB : LA;
      const unsigned slot = H == 0 ? c_slot : n_slot;
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, NM>([&](auto tc) {   // reads and loads spread between the MFMAs
        constexpr int t = decltype(tc)::value;
        static_for<t * NR / NM, (t + 1) * NR / NM>([&](auto rc) {
          constexpr int r = decltype(rc)::value, s = r / (TM + TN), e = r % (TM + TN);
          if constexpr (e < TN) read_b(1 - H, s, e, slot, 2 * (1 - H) + s);
          else read_a(1 - H, s, e - TN, slot, 2 * (1 - H) + s);
        });
        static_for<t * NL / NM, (t + 1) * NL / NM>([&](auto lc) {
          if constexpr (H == 0) load_b(decltype(lc)::value);
          else load_a(decltype(lc)::value);
        });
        constexpr int s = t / (TM * TN), i = t % (TM * TN) / TN, j = t % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[H][s][j], fa[H][s][i], acc[i][j], 0, 0, 0);
        if constexpr (COLSUM && i == 0) {
          if (do_colsum) csum[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[H][s][j], ones, csum[j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    phase(IntC<0>{});
    next_chunk();
    // this chunk is in registers, and all but the SLOTS - 2 youngest chunks have landed: the next one has
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(AHEAD) : "memory");
    phase(IntC<1>{});
    c_slot = n_slot;
  }

  // ---- epilogue (see sk_bf16_gemm.hip): fp32 straight from registers, bf16 through a strip of LDS, branch free ----
  // No load may land in LDS any more, in the strips' room or in what is someone else's, and nobody may read it as a chunk.
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  const float scale = p.scale;
  const int wn0 = n0 + wn * WN, n_store = p.n_store > 0 ? p.n_store : p.N;
  if constexpr (!BF16_OUT) {
    float* const C = static_cast<float*>(p.C);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t row = (int64_t)split * p.M + m0 + wm * WM + i * 32;
      const GWindow w = make_window(C, row * p.ldc + wn0, (int64_t)(split + 1) * p.M * p.ldc, 4);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = j * 32 + q * 8 + (lane >> 5) * 4;
          const f32x4 v = {acc[i][j][q * 4 + 0] * scale, acc[i][j][q * 4 + 1] * scale, acc[i][j][q * 4 + 2] * scale, acc[i][j][q * 4 + 3] * scale};
          window_store16(w, wn0 + c < n_store ? ((unsigned)(lane & 31) * (unsigned)p.ldc + (unsigned)c) * 4u : OOB_OFFSET, __builtin_bit_cast(uint4, v));
        }
    }
  } else {
    constexpr int PPRW = WN / 8, RPI = 64 / PPRW, ROW_BYTES = WN * 2;
    unsigned char* const strip = smem + wave * STRIP;
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
            const uint2 b = bias_r[j][q];
            w[h].x = pack_bf16x2(acc[i][j][q * 4 + 0] * scale + bf16_bits_to_float(b.x & 0xffffu), acc[i][j][q * 4 + 1] * scale + bf16_bits_to_float(b.x >> 16));
            w[h].y = pack_bf16x2(acc[i][j][q * 4 + 2] * scale + bf16_bits_to_float(b.y & 0xffffu), acc[i][j][q * 4 + 3] * scale + bf16_bits_to_float(b.y >> 16));
          }
          typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
          const u32x2 s0 = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
          const u32x2 s1 = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
          const int piece = j * 4 + pr * 2 + (lane >> 5);
          *reinterpret_cast<uint4*>(strip + row_w * ROW_BYTES + ((piece ^ (row_w & (PPRW - 1))) * 16)) = make_uint4(s0.x, s1.x, s0.y, s1.y);
        }
      const GWindow w = make_window(p.C, (int64_t)(m0 + wm * WM + i * 32) * p.ldc + wn0, (int64_t)p.M * p.ldc, 2);
      uint4 v[32 / RPI];
#pragma unroll
      for (int u = 0; u < 32 / RPI; ++u) {
        const int row_r = u * RPI + lane / PPRW, piece = lane % PPRW;
        v[u] = *reinterpret_cast<const uint4*>(strip + row_r * ROW_BYTES + ((piece ^ (row_r & (PPRW - 1))) * 16));
      }
#pragma unroll
      for (int u = 0; u < 32 / RPI; ++u) {
        const int row_r = u * RPI + lane / PPRW, c = (lane % PPRW) * 8;
        window_store16(w, wn0 + c < n_store ? ((unsigned)row_r * (unsigned)p.ldc + (unsigned)c) * 2u : OOB_OFFSET, v[u]);
      }
    }
  }
  if constexpr (COLSUM) {
    if (do_colsum) {   // (every column of csum holds the same sums: lanes 0 and 32 write them)
      const GWindow w = make_window(p.colsum, (int64_t)split * p.N + wn0, (int64_t)(split + 1) * p.N, 4);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = {csum[j][q * 4 + 0], csum[j][q * 4 + 1], csum[j][q * 4 + 2], csum[j][q * 4 + 3]};
          window_store16(w, (lane & 31) == 0 ? (unsigned)(j * 32 + q * 8 + (lane >> 5) * 4) * 4u : OOB_OFFSET, __builtin_bit_cast(uint4, v));
        }
    }
  }
}

}  // namespace sk
