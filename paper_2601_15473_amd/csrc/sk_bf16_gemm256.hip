// The 256 x 256 tile of the bf16 MFMA GEMM (same contract as sk_bf16_gemm.hip) and the column
// sums of dY that go with it.
//
// Four waves as 2 x 2, one per SIMD; a wave owns 128 x 128 of the tile (4 x 4 MFMA blocks, all 256
// accumulation registers).  Operands go from global memory straight into LDS
// (buffer_load_dwordx4 ... lds) in 64-wide k chunks, two chunks of 64 KB in LDS.
//
// What bounds it is how long the matrix pipe waits, and three things decide that:
//   - whole lines.  A chunk's rows are 128 bytes; the same loop on 32-wide chunks asked the L2 for
//     every line twice (88 M requests instead of 45 M for [16384 x 11008] . [11008 x 2048]) and ran a
//     third slower.
//   - loads that are early AND spread.  A phase is half a chunk: a wave multiplies A blocks 2 h and
//     2 h + 1 with all four B blocks (32 MFMAs, 1024 cycles), reads the A blocks of the next phase and
//     half of the B blocks of the NEXT chunk into a second register set, and loads into what the
//     phase before has read -- so a slot is refilled as soon as it is in registers, one to one and a
//     half chunks before it is needed, one load per four MFMAs, and the barrier of a phase leaves 16
//     of the wave's loads in flight.  (One barrier and one burst of loads per chunk: a half slower.)
//   - nothing else in the in-order load counter.  Stores retire through it as well, so the loads
//     of the next tile's first phase go out ahead of a tile's stores, and the first three phases
//     behind an epilogue wait for what lies before the stores only ([8192 x 512] . [512 x 4096], two
//     tiles per work-group: 53 -> 39 us).  For the same reason no register may be spilled here: the
//     compiler's wait for a reload is a wait for every load.
// The loads are inline assembly because the compiler would wait for all of them ahead of every
// LDS read; what waits on what is spelled out at the barriers.
//
// Measured against the eight-wave loop it replaces (operands through registers, MFMAs 55 % of
// the cycles; now 76 %), random data, us: [16384 x 4096] . S [4096 x 2048] 242 -> 208, [16384 x 2048] .
// U [2048 x 11008] 710 -> 580, [16384 x 11008] . U^T 705 -> 557-590, [16384 x 2048] . S^T 250 -> 212,
// S^T . x^T 255 -> 207, [8192 x 512] . [512 x 4096] 49 -> 39.  Long launches run into the power limit
// (1.6 GHz instead of 2.1), which is why the last ones gain least.
#include "sk_bf16_lds.h"
#include "sk_launch.h"

namespace sk {

constexpr int CHUNK = 65536;                      // bytes of a chunk in LDS: A's 32 KB, then B's
constexpr int STRIPS = 2 * CHUNK;                 // then 8 KB per wave for its results (and bias values)
constexpr int GEMM256_LDS = STRIPS + 4 * 8192;    // all of a CU's LDS

// The work of one work-group: tiles block, block + stride, ... below `total`.  `smem` must be the
// kernel's only LDS (it then starts at LDS address 0), and the kernel's first argument a GemmArgs.
// k ranges but the last are multiples of 128, at least 256 long; n_store is set.  FAR: for operands
// that are not k-contiguous and span more than 2 GB over a tile's k range, and bf16 results that do
// over its rows.
template <bool A_KC, bool B_KC, typename OutT, bool FAR>
__device__ __forceinline__ void gemm256_tiles(unsigned char* const smem, const int block, const int stride, const int total) {
  typedef Panels<A_KC> PA;
  typedef Panels<B_KC> PB;
  // (what the loads write is invisible to the compiler: it must not take smem for unwritten)
  asm volatile("" ::"v"((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem) : "memory");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // The arguments, loaded anew where they are used: held in scalar registers throughout they crowd
  // out the main loop's own values.
  typedef const __attribute__((address_space(4))) GemmArgs* ArgPtr;
  auto args = []() {
    ArgPtr q = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    return q;
  };
  struct Tile {
    int split, m0, n0, k_len;
    u32x4 a, b;   // the operands from the tile's first row and k on
  };
  auto locate = [&](int blk, bool any) {
    const ArgPtr q = args();
    Tile t;
    const int tiles = q->tiles_m * q->tiles_n;
    const int id = xcd_remap(blk, tiles * q->splits);
    t.split = id / tiles;
    int tm, tn;
    tile_coords(id - t.split * tiles, q->tiles_m, q->tiles_n, tm, tn);
    t.m0 = tm * 256;
    t.n0 = tn * 256;
    const int k0 = t.split * q->k_per_split;
    const int k1 = k0 + q->k_per_split < q->K ? k0 + q->k_per_split : q->K;
    t.k_len = k1 - k0;
    const int64_t oa = A_KC ? (int64_t)t.m0 * q->lda + k0 : (int64_t)k0 * q->lda + t.m0;
    const int64_t ob = B_KC ? (int64_t)t.n0 * q->ldb + k0 : (int64_t)k0 * q->ldb + t.n0;
    // (an operand that is not k-contiguous may be a column range of a wider array: it ends with its
    // last row's last column)
    t.a = descriptor(q->A, oa, !any ? 0 : A_KC ? (int64_t)q->M * q->lda : (int64_t)(q->K - 1) * q->lda + q->M, 2);
    t.b = descriptor(q->B, ob, !any ? 0 : B_KC ? (int64_t)q->N * q->ldb : (int64_t)(q->K - 1) * q->ldb + q->N, 2);
    return t;
  };

  // ---- the two streams of chunks to load, running ahead of the one being multiplied ----
  const unsigned lda = (unsigned)args()->lda * 2u, ldb = (unsigned)args()->ldb * 2u;   // bytes
  const unsigned va = PA::load_offset(wave, lane, lda), vb = PB::load_offset(wave, lane, ldb);
  const int lane_k = Panels<true>::load_k(wave, lane);   // (lines 32 and 64 further down: the same)
  const unsigned step_a = A_KC ? 128u : lda * 64u, step_b = B_KC ? 128u : ldb * 64u;        // next chunk
  const unsigned panel_a = A_KC ? lda * 64u : 128u, panel_b = B_KC ? ldb * 64u : 128u;      // next panel
  Tile here = locate(block, true);
  u32x4 a_src = here.a, b_src = here.b;
  unsigned a_off = 0, b_off = 0;              // byte offset of the chunk in there
  int a_left = here.k_len, b_left = here.k_len;   // k left from it on
  // Load i (of 4) of panels h and h + 2: lines 32 (i & 1) + 8 wave .. of panel h + 2 (i >> 1).  Past the
  // k range a k-contiguous operand reads as zero; the other kind has only rows past the array
  // there, and what it reads past its m or n are rows or columns of the result that are not stored.
  auto lds_of = [&](int i, int h) { return (unsigned)((i >> 1) * 16384 + h * 8192 + (i & 1) * 4096) + (unsigned)wave * 1024u; };
  auto load_a = [&](int i, int h, unsigned chunk) {
    load_to_lds(chunk + lds_of(i, h), A_KC ? (lane_k < a_left ? va : OOB_OFFSET) : va, a_src,
                a_off + (h ? panel_a : 0u) + (i & 1 ? lda * 32u : 0u) + (i & 2 ? 2 * panel_a : 0u));
  };
  auto load_b = [&](int i, int h, unsigned chunk) {
    load_to_lds(chunk + 32768u + lds_of(i, h), B_KC ? (lane_k < b_left ? vb : OOB_OFFSET) : vb, b_src,
                b_off + (h ? panel_b : 0u) + (i & 1 ? ldb * 32u : 0u) + (i & 2 ? 2 * panel_b : 0u));
  };

  // Offsets are 32-bit: far operands take their origin along whenever a chunk starts 1 GB behind
  // it (64 rows are 128 MB at most).  (For all operands the two compares a chunk cost 0.3 %.)
  auto move_on = [](u32x4& src, unsigned& off, const void* base, int64_t total) {
    const uint64_t at = ((uint64_t)src.y << 32 | src.x) + off;
    src = descriptor((const void*)at, 0, ((int64_t)((uint64_t)base - at) >> 1) + total, 2);
    off = 0;
  };
  auto move_a = [&]() {
    if (!FAR || A_KC || a_off < (1u << 30)) return;
    const ArgPtr q = args();
    move_on(a_src, a_off, q->A, (int64_t)(q->K - 1) * q->lda + q->M);
  };
  auto move_b = [&]() {
    if (!FAR || B_KC || b_off < (1u << 30)) return;
    const ArgPtr q = args();
    move_on(b_src, b_off, q->B, (int64_t)(q->K - 1) * q->ldb + q->N);
  };

  bf16x8 fa[2][2][4], fb[2][4][4];   // fragments [set][block][k step]
  unsigned a_read = PA::read_address(wm, lane), b_read = 32768 + PB::read_address(wn, lane);
  // (opaque, or every address of either chunk is kept in a register of its own)
  auto flip = [](unsigned& address) {
    address ^= CHUNK;
    asm volatile("" : "+v"(address));
  };

  // ---- prologue: chunk 0, and what the main loop expects to be under way ----
  {
    auto a4 = [&](int h, unsigned chunk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) load_a(i, h, chunk);
    };
    auto b4 = [&](int h, unsigned chunk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) load_b(i, h, chunk);
    };
    a4(0, 0); b4(0, 0); b4(1, 0); a4(1, 0);
    a_off += step_a; b_off += step_b; a_left -= 64; b_left -= 64;
    b4(0, CHUNK);
    a4(0, CHUNK); b4(1, CHUNK);
    asm volatile("s_waitcnt vmcnt(12)\n\ts_barrier" ::: "memory");   // chunk 0
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[0][i][ks] = PA::frag(a_read, i, ks);
#pragma unroll
      for (int i = 0; i < 4; ++i) fb[0][i][ks] = PB::frag(b_read, i, ks);
    }
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // B blocks 0, 1 of chunk 1
    a4(1, CHUNK);
    b_off += step_b; b_left -= 64;
    b4(0, 0);
    a_off += step_a; a_left -= 64;
    a4(0, 0); b4(1, 0);
    b_off += step_b; b_left -= 64;
    flip(b_read);
  }

  unsigned chunk_lds = 0;   // where the chunk being multiplied lies
  for (int blk = block; blk < total; blk += stride) {
    const bool has_next = blk + stride < total;
    const Tile next = locate(has_next ? blk + stride : blk, has_next);
    if constexpr (sizeof(OutT) == 2) {
      // the wave's 128 bias values (zeros without a bias) wait for the epilogue in its strip
      const ArgPtr q = args();
      const u32x4 bias = descriptor(q->bias, here.n0 + wn * 128, q->bias != nullptr ? q->N : 0, 2);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(STRIPS + wave * 8192), "v"(lane_again() * 4), "s"(bias) : "m0");
    }
    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // chunks, in pairs (the second B register set) and at least four (the streams cross into the
    // next tile two and three chunks ahead); those past the k range are zeros
    const int nk = here.k_len > 256 ? (here.k_len + 127) / 128 * 2 : 4;

    // Chunk kc, its B fragments in set P.  FIRST: 1 for the first of a tile (its first phase's loads
    // are out already), 2 for the second, 0 for the rest.
    auto chunk = [&](auto set_c, auto first_c, int kc) {
      constexpr int P = decltype(set_c)::value, FIRST = decltype(first_c)::value;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1) flip(a_read);
        if (h == 0 && FIRST != 1 && kc + 2 == nk) { a_src = next.a; a_off = 0; a_left = next.k_len; }
        const unsigned a_to = chunk_lds, b_to = h == 0 ? chunk_lds : chunk_lds ^ CHUNK;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int ks = t >> 1, i = t & 1;
          fa[1 - h][i][ks] = PA::frag(a_read, h == 0 ? 2 + i : i, ks);
          fb[1 - P][2 * h + i][ks] = PB::frag(b_read, 2 * h + i, ks);
          if (!(FIRST == 1 && h == 0)) {
            if (i == 0) load_a(ks, h, a_to);
            else load_b(ks, 1 - h, b_to);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[2 * h + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[P][j][ks], fa[h][i][ks], acc[2 * h + i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (h == 0) {
          if (FIRST != 1) {
            b_off += step_b; b_left -= 64;
            if (kc + 3 == nk) { b_src = next.b; b_off = 0; b_left = next.k_len; }
            move_b();
          }
        } else {
          a_off += step_a; a_left -= 64;
          move_a();
        }
        // This phase's reads done, and the loads two phases back and older: what the next phase
        // reads.  Behind an epilogue 32 (bf16) or 64 (fp32) stores and the bias load lie in between:
        // 8 + 8 + 33 younger ones in all three phases (the counter ends at 63).
        if (FIRST == 1 || (FIRST == 2 && h == 0)) {
          if (blk == block) asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
          else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(sizeof(OutT) == 2 ? 49 : 63) : "memory");
        } else {
          asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
      }
      flip(b_read);
      chunk_lds ^= CHUNK;
      asm volatile("" : "+s"(chunk_lds));
    };
    chunk(IntC<0>{}, IntC<1>{}, 0);
    chunk(IntC<1>{}, IntC<2>{}, 1);
    for (int kc = 2; kc < nk; kc += 2) {
      chunk(IntC<0>{}, IntC<0>{}, kc);
      chunk(IntC<1>{}, IntC<0>{}, kc + 1);
    }

    // the loads of the next tile's first phase, ahead of this tile's stores
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) { load_a(i, 0, chunk_lds); load_b(i, 1, chunk_lds); }
    b_off += step_b; b_left -= 64;

    // ---- epilogue ----
    // Lane l owns row l % 32 of each 32-row block and, for q = 0..3, columns 8 q + 4 (l / 32) .. + 3 of each
    // 32-column block.  fp32 leaves like that, 16 bytes a lane; bf16 is turned over a 32-row
    // block at a time through the wave's strip of LDS (no barrier: a wave's LDS operations execute
    // in order), so that a store instruction writes four whole rows of 256 bytes.  All stores
    // are branch free; what lies outside the result is dropped at the window.
    __builtin_amdgcn_sched_barrier(0);
    const ArgPtr q = args();
    const int el = lane_again();
    const float scale = q->scale;
    if constexpr (sizeof(OutT) == 2) {
      unsigned char* const strip = smem + STRIPS + wave * 8192;
      // (far results, Z^T over millions of tokens: a window for every 32 rows, 256 of which pass 2 GB)
      const GWindow all = make_window(q->C, (int64_t)here.m0 * q->ldc, (int64_t)q->M * q->ldc, 2);
      const unsigned ldc = (unsigned)q->ldc * 2u;
      uint2 bias[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          bias[j][e] = *reinterpret_cast<const uint2*>(strip + (j * 32 + e * 8 + (el >> 5) * 4) * 2);
      const int gn = here.n0 + wn * 128 + (el & 15) * 8;
      const unsigned at = gn < q->n_store ? (unsigned)((FAR ? 0 : wm * 128) + (el >> 4)) * ldc + (unsigned)gn * 2u : OOB_OFFSET;
      unsigned char* const wr = strip + (el & 31) * 256;
      const unsigned char* const rd = strip + (el >> 4) * 256;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        GWindow out = all;
        if constexpr (FAR) out = make_window(q->C, (int64_t)(here.m0 + wm * 128 + i * 32) * q->ldc, (int64_t)q->M * q->ldc, 2);
        // (the accumulators stay in their own registers until their block is due: copied out ahead
        // they crowd out what the next tile's main loop needs)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[i][j]));
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int pr = 0; pr < 2; ++pr) {
            uint2 w[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int e = 2 * pr + h;
              const uint2 b = bias[j][e];
              w[h].x = pack_bf16x2(acc[i][j][e * 4 + 0] * scale + bf16_bits_to_float(b.x & 0xffffu),
                                   acc[i][j][e * 4 + 1] * scale + bf16_bits_to_float(b.x >> 16));
              w[h].y = pack_bf16x2(acc[i][j][e * 4 + 2] * scale + bf16_bits_to_float(b.y & 0xffffu),
                                   acc[i][j][e * 4 + 3] * scale + bf16_bits_to_float(b.y >> 16));
            }
            // half-waves exchange: eight consecutive columns, piece 4 j + 2 pr + l / 32 of the row
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 s0 = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
            const u32x2 s1 = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
            const int piece = j * 4 + pr * 2 + (el >> 5);
            *reinterpret_cast<uint4*>(wr + ((piece ^ (el & 15)) * 16)) = make_uint4(s0.x, s1.x, s0.y, s1.y);
          }
        __builtin_amdgcn_sched_barrier(0);
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          v[u] = *reinterpret_cast<const uint4*>(rd + u * 1024 + (((el & 15) ^ ((u * 4 + (el >> 4)) & 15)) * 16));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) window_store16(out, at + (unsigned)((FAR ? 0 : i * 32) + u * 4) * ldc, v[u]);
      }
    } else {
      const GWindow out = make_window(q->C, ((int64_t)here.split * q->M + here.m0) * q->ldc, (int64_t)(here.split + 1) * q->M * q->ldc, 4);
      const unsigned ldc = (unsigned)q->ldc * 4u;
      const unsigned row = (unsigned)(wm * 128 + (el & 31)) * ldc;
      const int col = here.n0 + wn * 128 + (el >> 5) * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          asm volatile("" : "+a"(acc[i][j]));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int gn = col + j * 32 + e * 8;
            const f32x4 v = {acc[i][j][e * 4 + 0] * scale, acc[i][j][e * 4 + 1] * scale, acc[i][j][e * 4 + 2] * scale, acc[i][j][e * 4 + 3] * scale};
            window_store16(out, gn < q->n_store ? row + (unsigned)(i * 32) * ldc + (unsigned)gn * 4u : OOB_OFFSET, __builtin_bit_cast(uint4, v));
          }
        }
    }
    here = next;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load may land in LDS that is someone else's
}

// One work-group per CU (the tile takes all of its LDS) walks the tiles index, index + grid, ...
template <int BM, int BN, int CHUNKS, int STEPS, bool A_KC, bool B_KC, typename OutT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_crew_kernel(const GemmArgs, const int total) {
  static_assert(BM == 256 && BN == 256 && CHUNKS == 2 && STEPS == 4, "256 x 256, two chunks of four k steps in LDS");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[GEMM256_LDS];
  gemm256_tiles<A_KC, B_KC, OutT, false>(smem, blockIdx.x, gridDim.x, total);
}
template <bool A_KC, bool B_KC, typename OutT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_far_kernel(const GemmArgs, const int total) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[GEMM256_LDS];
  gemm256_tiles<A_KC, B_KC, OutT, true>(smem, blockIdx.x, gridDim.x, total);
}

// ---- column sums ----
// Column sums of a dense row-major bf16 matrix [rows, cols] in fp32, the row range cut
// into `splits` runs of rows_per_split (out[s][c] = sum of rows of run s; fixed order).
// One work-group owns 512 columns of one run: a wave reads one whole 1 KB row segment
// per instruction (lane = 8 columns), sixteen of them in flight, the four waves stride over the
// rows, and their four partial sums meet in LDS and are added in wave order.
// (As a loop unrolled sixteen times by the compiler the last rows of a run, up to fifteen a wave, were one trip each: backward pass of 8192 tokens,
// 3072 -> 8192, R = 2048, 648 us, now 640; 9001, 4096 -> 8192 915 : 909; level where the sums ride beside a round of tiles.)
constexpr int COLSUM_COLS = 512;
__device__ __forceinline__ void colsum_body(const unsigned short* __restrict__ in, float* __restrict__ out,
                                            int rows, int cols, int rows_per_split, int bx, int by, float* part) {
  constexpr int NW = 4, AHEAD = 16, PLD = COLSUM_COLS + 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = bx * COLSUM_COLS + lane * 8;
  const int r_begin = by * rows_per_split;
  const int r_end = (r_begin + rows_per_split < rows) ? r_begin + rows_per_split : rows;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (c < cols) {
    for (int r = r_begin + wave; r < r_end; r += AHEAD * NW) {
      uint4 v[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {   // (past the run: its last row again, not added)
        const int at = r + u * NW < r_end ? r + u * NW : r_end - 1;
        v[u] = *reinterpret_cast<const uint4*>(in + (int64_t)at * cols + c);
      }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const bool in_run = r + u * NW < r_end;
        const unsigned w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] += in_run ? __builtin_bit_cast(float, w[e] << 16) : 0.f;
          acc[2 * e + 1] += in_run ? __builtin_bit_cast(float, w[e] & 0xffff0000u) : 0.f;
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[wave * PLD + lane * 8 + e] = acc[e];
  __syncthreads();
  for (int i = tid; i < COLSUM_COLS; i += 64 * NW) {
    const int gc = bx * COLSUM_COLS + i;
    if (gc < cols) {
      float s = part[i];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += part[w * PLD + i];   // in wave order
      out[(int64_t)by * cols + gc] = s;
    }
  }
}

__global__ __launch_bounds__(256) void colsum_bf16_kernel(const unsigned short* __restrict__ in,
                                                          float* __restrict__ out, int rows,
                                                          int cols, int rows_per_split) {
  __shared__ float part[4 * (COLSUM_COLS + 8)];
  colsum_body(in, out, rows, cols, rows_per_split, blockIdx.x, blockIdx.y, part);
}

// A launch of the GEMM that does not fill the chip, with the column sums riding along:
// work-groups past the GEMM's own run the column-sum body on the CUs the GEMM leaves free --
// one streams from HBM while the other multiplies.
template <bool A_KC, bool B_KC, typename OutT, bool FAR>
__device__ __forceinline__ void gemm256_with_colsum(const int gemm_groups, const ColsumArgs& c) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[GEMM256_LDS];
  if ((int)blockIdx.x < gemm_groups) {
    gemm256_tiles<A_KC, B_KC, OutT, FAR>(smem, blockIdx.x, gemm_groups, gemm_groups);
  } else {
    const int w = blockIdx.x - gemm_groups;
    colsum_body(static_cast<const unsigned short*>(c.in), c.out, c.rows, c.cols, c.rows_per_split,
                w % c.col_groups, w / c.col_groups, reinterpret_cast<float*>(smem));
  }
}
template <int BM, int BN, int CHUNKS, int STEPS, bool A_KC, bool B_KC, typename OutT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_with_colsum_kernel(
    const GemmArgs, const int gemm_groups, const ColsumArgs c) {
  static_assert(BM == 256 && BN == 256 && CHUNKS == 2 && STEPS == 4, "256 x 256, two chunks of four k steps in LDS");
  gemm256_with_colsum<A_KC, B_KC, OutT, false>(gemm_groups, c);
}
template <bool A_KC, bool B_KC, typename OutT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_far_with_colsum_kernel(
    const GemmArgs, const int gemm_groups, const ColsumArgs c) {
  gemm256_with_colsum<A_KC, B_KC, OutT, true>(gemm_groups, c);
}

bool gemm256_supported(GemmKind kind, const GemmArgs& a) {
  bool a_kc, b_kc, f32;
  gemm_kind_traits(kind, a_kc, b_kc, f32);
  if (kind == GEMM_NN_F32_COLSUM || kind == GEMM_TN_F32) return false;   // no registers for the sums
  if (kind == GEMM_NT_F32 || kind == GEMM_TT_F32) return false;          // (no plan splits these on this tile)
  // ranges but the last: whole pairs of chunks (their zero chunks would be the next range's rows)
  if (a.splits > 1 && (a.k_per_split % 128 != 0 || a.k_per_split < 256)) return false;
  // byte offsets from a tile's origin are 32-bit: 256 rows of a k-contiguous operand, over the whole
  // k range, a few chunks of the other kind (is_far)
  const int64_t range = (int64_t)(a.splits > 1 ? a.k_per_split : a.K) + 512;
  if (!(a_kc ? within_window(256, a.lda, range, 2) : a.lda <= 1 << 20)) return false;
  if (!(b_kc ? within_window(256, a.ldb, range, 2) : a.ldb <= 1 << 20)) return false;
  // ... and rows of the result: all 256, or 32 where there is a variant for far ones
  return within_window(f32 || (a_kc && b_kc) ? 256 : 32, a.ldc, a.n_store > 0 ? a.n_store : a.N, f32 ? 4 : 2);
}

// Whether an operand that is not k-contiguous spans more over a tile's k range than offsets reach, or the
// result over its rows.
static bool is_far(bool a_kc, bool b_kc, const GemmArgs& a, int osize) {
  const int64_t range = (int64_t)(a.splits > 1 ? a.k_per_split : a.K) + 512;
  return (!a_kc && range * a.lda * 2 > 0x7fffffffLL) || (!b_kc && range * a.ldb * 2 > 0x7fffffffLL) ||
         !within_window(256, a.ldc, a.n_store > 0 ? a.n_store : a.N, osize);
}

template <bool A_KC, bool B_KC, typename OutT>
static hipError_t launch_crew(GemmArgs a, hipStream_t s) {
  a.tiles_m = (a.M + 255) / 256;
  a.tiles_n = (a.N + 255) / 256;
  if (a.n_store <= 0) a.n_store = a.N;
  const long long total = (long long)a.tiles_m * a.tiles_n * a.splits;
  if (total <= 0 || total > 0x7fffffffLL - NUM_CUS) return hipErrorInvalidValue;
  constexpr bool F32 = sizeof(OutT) == 4;
  note_gemm(a, A_KC, B_KC, 2, sizeof(OutT), F32);
  const dim3 grid((unsigned)(total < NUM_CUS ? total : NUM_CUS));
  const Work work = gemm_work(a, 2, sizeof(OutT), F32);
  if constexpr (!A_KC || !B_KC) {
    if (is_far(A_KC, B_KC, a, sizeof(OutT))) {
      static const std::string far = kernel_label("gemm_bf16_far_kernel", {lbl(A_KC), lbl(B_KC), F32 ? "float" : "bf16"});
      return launch_kernel(far.c_str(), work, gemm_bf16_far_kernel<A_KC, B_KC, OutT>, grid, dim3(256), s, a, (int)total);
    }
  }
  static const std::string name = kernel_label("gemm_bf16_crew_kernel", {lbl(256), lbl(256), lbl(2), lbl(4), lbl(A_KC), lbl(B_KC), F32 ? "float" : "bf16"});
  return launch_kernel(name.c_str(), work, gemm_bf16_crew_kernel<256, 256, 2, 4, A_KC, B_KC, OutT>, grid, dim3(256), s, a, (int)total);
}

hipError_t launch_gemm256_bf16(GemmKind kind, const GemmArgs& a, hipStream_t s) {
  if (!gemm256_supported(kind, a)) return hipErrorInvalidValue;
  switch (kind) {
    case GEMM_NN: return launch_crew<true, false, bf16>(a, s);
    case GEMM_NT: return launch_crew<true, true, bf16>(a, s);
    case GEMM_TT: return launch_crew<false, true, bf16>(a, s);
    case GEMM_NN_F32: return launch_crew<true, false, float>(a, s);
    case GEMM_TN_F32_PLAIN: return launch_crew<false, false, float>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm256_with_colsum(GemmArgs a, const void* in, float* out, int rows, int cols, int splits,
                                      int rows_per_split, hipStream_t s) {
  if (!gemm256_supported(GEMM_NN_F32, a)) return hipErrorInvalidValue;
  a.tiles_m = (a.M + 255) / 256;
  a.tiles_n = (a.N + 255) / 256;
  if (a.n_store <= 0) a.n_store = a.N;
  ColsumArgs c;
  c.in = in; c.out = out; c.rows = rows; c.cols = cols; c.rows_per_split = rows_per_split;
  c.col_groups = (cols + COLSUM_COLS - 1) / COLSUM_COLS;
  const long long gg = (long long)a.tiles_m * a.tiles_n * a.splits;
  const long long grid = gg + (long long)c.col_groups * splits;
  if (gg <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  note_gemm(a, true, false, 2, 4, true);
  note_matrix(in, rows, cols, cols, 2, false);
  note_matrix(out, splits, cols, cols, 4, true);
  Work work = gemm_work(a, 2, 4, true);
  work.bytes += (double)rows * cols * 2 + (double)splits * cols * 4;
  return is_far(true, false, a, 4)
             ? launch_kernel("gemm_bf16_far_with_colsum_kernel<true, false, float>", work,
                             gemm_bf16_far_with_colsum_kernel<true, false, float>, dim3((unsigned)grid), dim3(256), s, a, (int)gg, c)
             : launch_kernel("gemm_bf16_with_colsum_kernel<256, 256, 2, 4, true, false, float>", work,
                             gemm_bf16_with_colsum_kernel<256, 256, 2, 4, true, false, float>,
                             dim3((unsigned)grid), dim3(256), s, a, (int)gg, c);
}

hipError_t launch_colsum_bf16(const void* in, float* out, int rows, int cols, int splits,
                              int rows_per_split, hipStream_t s) {
  const dim3 grid((unsigned)((cols + COLSUM_COLS - 1) / COLSUM_COLS), (unsigned)splits);
  note_matrix(in, rows, cols, cols, 2, false);
  note_matrix(out, splits, cols, cols, 4, true);
  return launch_kernel("colsum_bf16_kernel", Work{0.0, (double)rows * cols * 2 + (double)splits * cols * 4},
                       colsum_bf16_kernel, grid, dim3(256), s,
                       static_cast<const unsigned short*>(in), out, rows, cols, rows_per_split);
}

}  // namespace sk
