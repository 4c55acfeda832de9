// bf16 GEMM for few rows of A (a handful of tokens): C = scale * (A . B) + bias, A [M, K], B [K, N] or
// [N, K], result in bf16.
//
// What bounds it is streaming B once: a row or sixty-four of A make next to no work of it.  So
// a work-group owns few columns (32 or 64) over the whole contraction, and its four waves share
// that: wave w takes the 64-wide k chunks w, w + 4, ... through a ring of its own in LDS, filled
// by direct loads that only the wave itself waits for -- no barrier until the four partial sums
// meet (in wave order) at the end, and up to 150 KB per CU in flight, which is what the
// trip to HBM times a CU's share of its bandwidth asks for.  A long first contraction (past K = 3072, the
// planner's few_rows_splits) is cut into two to eight ranges, each on XCDs of its own, that leave fp32
// slabs for another launch to sum; everything else is one launch without slabs.
#include "sk_bf16_lds.h"
#include "sk_launch.h"

namespace sk {

// A8: rows of A per work-group in eights (as many as a load instruction fills), NB: 32-column blocks.
template <int A8, int NB, bool B_KC>
struct FewRows {
  static constexpr int BM = 8 * A8, BN = 32 * NB, MB = (BM + 31) / 32;
  static constexpr int A_BYTES = A8 * 1024, B_BYTES = NB * 4096, SLOT = A_BYTES + B_BYTES;
  static constexpr int LOADS = A8 + 4 * NB;                        // per chunk and wave
  static constexpr int WAVE_LDS = 40960;                           // a quarter of the CU's
  static constexpr int SLOTS = WAVE_LDS / SLOT < 8 ? WAVE_LDS / SLOT : 8;
  static constexpr int PLD = BN + 4;                               // floats per row of a partial sum
  static_assert((SLOTS - 1) * LOADS <= 63, "the load counter ends at 63");
  static_assert(4 * MB * 32 * PLD * 4 <= 4 * WAVE_LDS, "the partial sums fit");
  static_assert(A8 * 8 <= 64 && NB <= 2, "one panel each");
};

template <int A8, int NB, bool B_KC>
__global__ __launch_bounds__(256) void gemm_bf16_few_rows_kernel(const GemmArgs p) {
  typedef FewRows<A8, NB, B_KC> G;
  constexpr int MB = G::MB;
  constexpr bool HALF = NB == 1 && !B_KC;   // 32 columns: lines of 64 bytes, which need no swizzle
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * G::WAVE_LDS];
  // (what the loads write is invisible to the compiler: it must not take smem for unwritten)
  asm volatile("" ::"v"((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem) : "memory");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Row tiles of the same columns side by side; k ranges by XCD (work-groups go to the eight in turn).
  int wg, split = 0;
  if (p.splits > 1) {
    const int per = 8 / p.splits, xcd = blockIdx.x & 7;   // XCDs to a range
    split = xcd / per;
    wg = ((int)blockIdx.x >> 3) * per + xcd % per;
    if (wg >= p.tiles_m * p.tiles_n) return;
  } else {
    wg = xcd_remap(blockIdx.x, p.tiles_m * p.tiles_n);
  }
  const int m0 = wg % p.tiles_m * G::BM, n0 = wg / p.tiles_m * G::BN;
  const int k_begin = split * p.k_per_split;
  const int k_end = k_begin + p.k_per_split < p.K ? k_begin + p.k_per_split : p.K;
  const unsigned lda = (unsigned)p.lda * 2u, ldb = (unsigned)p.ldb * 2u;

  const u32x4 a_src = descriptor(p.A, (int64_t)m0 * p.lda, (int64_t)p.M * p.lda, 2);
  // (lines of a k-contiguous operand 8 further down swizzle differently, 16 further down alike)
  const unsigned va = Panels<true>::load_offset(0, lane, lda), va2 = Panels<true>::load_offset(1, lane, lda) - 8u * lda;
  const int ka = Panels<true>::load_k(0, lane), ka2 = Panels<true>::load_k(1, lane);
  const unsigned vb = HALF ? (unsigned)(lane >> 2) * ldb + (lane & 3) * 16u : Panels<B_KC>::load_offset(0, lane, ldb);
  const unsigned vb2 = Panels<B_KC>::load_offset(1, lane, ldb) - 8u * ldb;
  const int n_chunks = (k_end - k_begin + 63) / 64, mine = (n_chunks - wave + 3) / 4;
  const unsigned ring = wave * G::WAVE_LDS;

  // The i-th of this wave's chunks into its slot.  Past the contraction A reads as zero (and B, k
  // contiguous); rows of B there lie past the array.
  auto issue = [&](int i, unsigned slot) {
    const int k0 = k_begin + (wave + 4 * i) * 64;
    const bool in = k0 + ka < k_end, in2 = k0 + ka2 < k_end;
#pragma unroll
    for (int r = 0; r < A8; ++r)
      load_to_lds(slot + r * 1024, r & 1 ? (in2 ? va2 : OOB_OFFSET) : (in ? va : OOB_OFFSET), a_src, (unsigned)k0 * 2u + (unsigned)r * 8u * lda);
    const int64_t b_at = B_KC ? (int64_t)n0 * p.ldb : (int64_t)k0 * p.ldb + n0;
    const u32x4 b_src = descriptor(p.B, b_at, B_KC ? (int64_t)p.N * p.ldb : (int64_t)(p.K - 1) * p.ldb + p.N, 2);
#pragma unroll
    for (int r = 0; r < 4 * NB; ++r) {
      const unsigned to = slot + G::A_BYTES + r * 1024;
      if constexpr (B_KC)
        load_to_lds(to, r & 1 ? (in2 ? vb2 : OOB_OFFSET) : (in ? vb : OOB_OFFSET), b_src,
                    (unsigned)k0 * 2u + (unsigned)r * 8u * ldb);
      else
        load_to_lds(to, vb, b_src, (unsigned)r * (HALF ? 16u : 8u) * ldb);
    }
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
  for (int s = 0; s < G::SLOTS; ++s)
    if (s < mine) issue(s, ring + s * G::SLOT);
  const unsigned a_read = Panels<true>::read_address(0, lane);
  const unsigned b_read = HALF ? (unsigned)(((lane >> 5) * 8 + ((lane & 15) >> 2)) * 64 + (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2)
                               : Panels<B_KC>::read_address(0, lane);
  unsigned slot = ring;
  for (int i = 0; i < mine; ++i) {
    if (i + G::SLOTS <= mine) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((G::SLOTS - 1) * G::LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bf16x8 fa[MB][4], fb[NB][4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int m = 0; m < MB; ++m) fa[m][ks] = Panels<true>::frag(slot + a_read, m, ks);
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        if constexpr (HALF) {
          const unsigned at = slot + G::A_BYTES + b_read + ks * 1024;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(at));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(at + 256));
          typedef short s16x8 __attribute__((ext_vector_type(8)));
          const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          fb[n][ks] = __builtin_bit_cast(bf16x8, both);
        } else {
          fb[n][ks] = Panels<B_KC>::frag(slot + G::A_BYTES + b_read, n, ks);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot is in registers: refill it
    if (i + G::SLOTS < mine) issue(i + G::SLOTS, slot);
    slot = slot + G::SLOT == ring + G::SLOTS * G::SLOT ? ring : slot + G::SLOT;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[n][ks], fa[m][ks], acc[m][n], 0, 0, 0);
  }

  // the four partial sums, added in wave order
  float* const part = reinterpret_cast<float*>(smem);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(part + (wave * MB * 32 + m * 32 + (lane & 31)) * G::PLD + n * 32 + q * 8 + (lane >> 5) * 4) =
            make_float4(acc[m][n][q * 4 + 0], acc[m][n][q * 4 + 1], acc[m][n][q * 4 + 2], acc[m][n][q * 4 + 3]);
  __syncthreads();
  constexpr int PPR = G::BN / 4;
  for (int q = tid; q < G::BM * PPR; q += 256) {
    const int row = q / PPR, col = q % PPR * 4, gm = m0 + row, gn = n0 + col;
    if (gm >= p.M || gn >= p.N) continue;
    float4 s = *reinterpret_cast<const float4*>(part + row * G::PLD + col);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 v = *reinterpret_cast<const float4*>(part + (w * MB * 32 + row) * G::PLD + col);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    if (p.splits > 1) {
      *reinterpret_cast<float4*>(static_cast<float*>(p.C) + ((int64_t)split * p.M + gm) * p.ldc + gn) = s;
      continue;
    }
    uint2 b = make_uint2(0u, 0u);
    if (p.bias != nullptr) b = *reinterpret_cast<const uint2*>(static_cast<const bf16*>(p.bias) + gn);
    uint2 o;
    o.x = pack_bf16x2(s.x * p.scale + bf16_bits_to_float(b.x & 0xffffu), s.y * p.scale + bf16_bits_to_float(b.x >> 16));
    o.y = pack_bf16x2(s.z * p.scale + bf16_bits_to_float(b.y & 0xffffu), s.w * p.scale + bf16_bits_to_float(b.y >> 16));
    *reinterpret_cast<uint2*>(static_cast<bf16*>(p.C) + (int64_t)gm * p.ldc + gn) = o;
  }
}

template <int A8, int NB, bool B_KC>
static hipError_t launch_one(GemmArgs a, hipStream_t s) {
  typedef FewRows<A8, NB, B_KC> G;
  a.tiles_m = (a.M + G::BM - 1) / G::BM;
  a.tiles_n = (a.N + G::BN - 1) / G::BN;
  const long long tiles = (long long)a.tiles_m * a.tiles_n;
  const long long grid = a.splits > 1 ? (tiles + 8 / a.splits - 1) / (8 / a.splits) * 8 : tiles;
  if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  const bool slabs = a.splits > 1;
  note_gemm(a, true, B_KC, 2, slabs ? 4 : 2, slabs);
  static const std::string name = kernel_label("gemm_bf16_few_rows_kernel", {lbl(A8), lbl(NB), lbl(B_KC)});
  return launch_kernel(name.c_str(), gemm_work(a, 2, slabs ? 4 : 2, slabs), gemm_bf16_few_rows_kernel<A8, NB, B_KC>,
                       dim3((unsigned)grid), dim3(256), s, a);
}

template <int NB, bool B_KC>
static hipError_t launch_rows(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 8) return launch_one<1, NB, B_KC>(a, s);
  if (a.M <= 16) return launch_one<2, NB, B_KC>(a, s);
  if (a.M <= 32) return launch_one<4, NB, B_KC>(a, s);
  return launch_one<8, NB, B_KC>(a, s);
}

hipError_t launch_gemm_few_rows_bf16(GemmKind kind, const GemmArgs& a, hipStream_t s) {
  if ((kind != GEMM_NN && kind != GEMM_NT) || (a.splits != 1 && a.splits != 2 && a.splits != 4 && a.splits != 8) ||
      (a.splits > 1 && a.k_per_split % 64 != 0))
    return hipErrorInvalidValue;
  // 32 columns per work-group until those make more than a round
  const bool wide = a.splits > 1 || (long long)((a.M + 63) / 64) * ((a.N + 31) / 32) > NUM_CUS;
  if (kind == GEMM_NN) return wide ? launch_rows<2, false>(a, s) : launch_rows<1, false>(a, s);
  return wide ? launch_rows<2, true>(a, s) : launch_rows<1, true>(a, s);
}

}  // namespace sk
