// libsk's C ABI (include/sk.h): argument validation, per-shape plan, launches.
// Validation runs before any HIP call, so error paths work without a GPU.
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <string>

#include <vector>

#include "../../include/sk.h"
#include "../../include/sk_debug.h"
#include "sk_launch.h"

// Scratch of sk_linear_bwd_weight_noalloc (SK_NOALLOC_SCRATCH_BYTES, include/sk.h): device
// memory that belongs to the loaded code object (one copy per GPU, held until the process
// ends), so that entry point needs no workspace from its caller and no allocation of its
// own.  In host code this name is only a handle for hipGetSymbolAddress; kernels are given
// the address that call returns.
static __device__ __align__(256) unsigned char scratch[SK_NOALLOC_SCRATCH_BYTES];

namespace {

using namespace sk;

constexpr size_t WS_ALIGN = 256;

thread_local std::string g_hip_error;
std::atomic<int> g_plan{0};

// Forced plan parameters (sk_set_tuning; negative = the planner chooses).
std::atomic<int> g_tune[SK_TUNE_COUNT] = {{-1}, {-1}, {-1}, {-1}, {-1}, {-1}, {-1}, {-1}};
int tune(sk_tune_knob knob) { return g_tune[knob].load(std::memory_order_relaxed); }
// The tile a knob forces (the values past the list stand for the 256 x 256 tile as well), or -1.
int forced_tile(sk_tune_knob knob) {
  const int t = tune(knob);
  return t < 0 ? -1 : t < TILE_COUNT ? t : t <= 7 ? TILE_256x256 : -1;
}

// The calling thread's launch trace or kernel timer (include/sk_debug.h); null otherwise.
struct Hooks : LaunchHooks {
  bool trace = false;
  std::vector<sk_trace_access> accesses;
  std::vector<std::string> launches;      // trace mode: the kernels, and their work-groups in `groups`
  // profile mode
  std::vector<hipEvent_t> events;       // 2 per kernel: before, after
  std::vector<std::string> names;
  std::vector<unsigned> groups;
  std::vector<Work> work;
  int max_kernels = 0;
  bool recording = false;               // the current launch got its `before` event

  bool tracing() const override { return trace; }
  void access(const void* p, uint64_t bytes, bool write) override {
    sk_trace_access a;
    a.address = (uint64_t)reinterpret_cast<uintptr_t>(p);
    a.bytes = bytes;
    a.write = write ? 1 : 0;
    a.launch = (int)launches.size();
    accesses.push_back(a);
  }
  void launch_recorded(const char* name, unsigned g) override {
    launches.push_back(name);
    groups.push_back(g);
  }
  void before(const char* name, unsigned g, double flops, double bytes, hipStream_t s) override {
    recording = (int)names.size() < max_kernels;
    if (!recording) return;
    if (hipEventRecord(events[2 * names.size()], s) != hipSuccess) { recording = false; return; }
    names.push_back(name);
    groups.push_back(g);
    work.push_back(Work{flops, bytes});
  }
  void after(hipStream_t s) override {
    if (recording) (void)hipEventRecord(events[2 * names.size() - 1], s);
    recording = false;
  }
};
thread_local Hooks* g_hooks = nullptr;

size_t align_up(size_t v) { return (v + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN; }

sk_status hip_fail(hipError_t e, const char* what) {
  g_hip_error = std::string(what) + ": " + hipGetErrorString(e);
  return SK_ERR_HIP;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct Shape {
  int64_t T, in, out;
  int l, k, R;
  sk_dtype dtype;
  size_t esize;
};

// Checks everything that does not involve pointers.
sk_status check_shape(int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k,
                      sk_dtype dtype, Shape& s) {
  if (tokens < 1 || in < 1 || out < 1 || l < 1 || k < 1) return SK_ERR_INVALID_ARG;
  if (dtype != SK_F32 && dtype != SK_BF16) return SK_ERR_UNSUPPORTED;
  const int64_t R = (int64_t)l * k;
  if ((in & 15) || (out & 15) || (R & 15)) return SK_ERR_UNSUPPORTED;
  // index arithmetic inside the kernels is 32-bit per dimension
  if (tokens > (1 << 24) || in > (1 << 20) || out > (1 << 20) || R > (1 << 16))
    return SK_ERR_UNSUPPORTED;
  s.T = tokens; s.in = in; s.out = out; s.l = l; s.k = k; s.R = (int)R; s.dtype = dtype;
  s.esize = dtype == SK_BF16 ? 2 : 4;
  return SK_OK;
}

}  // namespace

namespace sk {
LaunchHooks* launch_hooks() { return g_hooks; }
}  // namespace sk

namespace {

// Room for slabs behind the recomputed Z of a factor gradient: a shape that fits the fixed scratch
// of sk_linear_bwd_weight_noalloc without splits is not split past it, one that does not has no limit.
size_t slab_room(size_t z_bytes) {
  return z_bytes < SK_NOALLOC_SCRATCH_BYTES ? SK_NOALLOC_SCRATCH_BYTES - z_bytes : SIZE_MAX;
}

// Tile choice for the general GEMM (measured on MI355X).  256 x 256 where its rounds of 256
// work-groups are modelled to end before 128 x 128's (two work-groups per CU): a round takes
// 6 us + 0.0215 us per k against 4.2 + 0.0165 for 512 of the smaller tiles, on top of 6 and 5 us a
// launch (fitted), so 192 of the big tiles already win (measured, K = 320: 18.6 against 18.7 us; K = 2048:
// 49 against 60), 128 do not (K = 512: 19.5 against 16.3), and one more than a round has no use for
// them.  Otherwise the largest tile that still gives every CU a work-group without being mostly
// padding, the smallest when the problem cannot fill the chip.
double big_tiles_us(int64_t M, int64_t N, double k, int splits) {
  const int64_t big = ((M + 255) / 256) * ((N + 255) / 256) * splits;
  return 6.0 + (double)((big + NUM_CUS - 1) / NUM_CUS) * (6.0 + 0.0215 * k);
}
int64_t small_tiles(int64_t M, int64_t N) { return ((M + 127) / 128) * ((N + 127) / 128); }
double small_tiles_us(int64_t tiles, double k) {
  const double halves = (double)((tiles + NUM_CUS - 1) / NUM_CUS);   // half rounds: one work-group per CU
  return 5.0 + (halves < 2 ? 2 : halves) / 2 * (4.2 + 0.0165 * k);
}
int choose_tile(int64_t M, int64_t N, int64_t K, int splits) {
  if (const int t = forced_tile(SK_TUNE_TILE); t >= 0) return t;  // forced (tests, sweeps)
  const int64_t m_cap = (M + 63) / 64 * 64, n_cap = (N + 63) / 64 * 64;
  if (K / splits > 128 && m_cap >= 256 && n_cap >= 256) {
    const double k = (double)K / splits;
    if (big_tiles_us(M, N, k, splits) < small_tiles_us(small_tiles(M, N) * splits, k)) return TILE_256x256;
  }
  static const int order[] = {TILE_128x128, TILE_128x64, TILE_64x128, TILE_64x64};
  for (int i = 0; i < (int)(sizeof(order) / sizeof(order[0])); ++i) {
    const int t = order[i];
    int bm, bn;
    tile_dims(t, bm, bn);
    if (bm > m_cap || bn > n_cap) continue;
    const int64_t wgs = ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * splits;
    if (wgs >= NUM_CUS) return t;
  }
  return TILE_64x64;
}
// ... of a bf16 result in a launch of its own: where 128 x 64 or 64 x 128 tiles make more than a round and 128 x 128 ones no more than
// one, those.  They run on the ring then, a chunk in 0.5 us on 50 to 100 % of the CUs; the smaller ones run on the staged loop, one or two to a CU,
// and fill 48 KB for the 32 of the larger.  Calls, us, 128 x 64 : 128 x 128: forward, 4001 tokens, 768 -> 768, R = 384 17.0 : 15.7; expansions of
// 144 to 1008, 30 of 600 to 12000 tokens 0.83 to 0.95 of the call; first contractions of 256 to 4600, 30 layers of 2400 to 16384 tokens, R 192 to 1008,
// forward 0.76 to 0.96 (2689 tokens, 3664 -> 320, R = 976 54.8 : 41.5), input gradient 0.85 to 1.00, factor gradient 0.82 to 1.00.  Where 64 x 64 is chosen (128 x 64 does
// not make a round) it stays: 1.03 to 1.11.
// Exactly one round of the smaller ones has every CU fetching, of the larger ones (at most) half of them, which is behind where the operands come from memory
// or the walk is short: 120 such layers, times the smaller tiles' call: x . S and expansions forward 0.97 to 1.08 over 160 to 1536, 0.88 to 0.97 over 2048 and more (three of 18 at
// 1.01 to 1.03); input gradient 0.98 to 1.10 (4075 tokens, 512 -> 256, R = 1200 20.9 : 23.0), level from 2048 on; S^T . x^T 0.85 to 0.95 where x is in the
// Infinity Cache from the call before, 1.03 to 1.11 where it is not (4079 tokens, 2560 -> 1536, R = 480 43.4 : 48.2), as in training.  So those stay, but for
// forward ones over 2048 and more.  (A result at most 64 wide never makes more of the smaller ones than of 128 x 128, half of each padding.)
int lone_tile(GemmKind kind, int t, int64_t M, int64_t N, int64_t K) {
  if ((t != TILE_128x64 && t != TILE_64x128) || K <= 128 || small_tiles(M, N) > NUM_CUS) return t;
  int bm, bn;
  tile_dims(t, bm, bn);
  const int64_t groups = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  return groups > NUM_CUS || (kind == GEMM_NN && K >= 2048) ? TILE_128x128 : t;
}

// ... of an expansion in a launch of its own: also 256 x 128 on a ring, while those make one round and 128 x 128 tiles more than one.  A launch takes
// 6.5 us + 0.0148 a k then (fitted), against the staged tiles' 9.2 + 0.0165, and fills 24 KB a chunk and 128 x 128 of the result where
// those fill 32.  180 layers with a short input, 600 to 16384 tokens, expansions of 144 to 2048 to 512 to 8192, us, 128 x 128 or 256 x 256 : 256 x 128: 2272
// tokens, R = 1968, 1856 out 43.1 : 36.7; 3220, 448, 1376 17.0 : 14.7; 1615, 256, 3488 13.1 : 12.5; 0.89 of the time above R = 256 (0.78 to 1.04,
// two behind, both of 12000 tokens to 528 and 560), 0.93 below (0.90 to 0.98).  Not for the first contractions, whose operands come
// from memory and not from the launch before: 0.84 to 1.09 of the time there, level over 40 layers.  Past a round each round costs 8 us again.
int choose_expansion_tile(GemmKind kind, int64_t M, int64_t N, int64_t K) {
  int t = choose_tile(M, N, K, 1);
  if (tune(SK_TUNE_TILE) >= 0 || K <= 128) return t;
  t = lone_tile(kind, t, M, N, K);
  const int64_t mid = (M + 255) / 256 * ((N + 127) / 128), small = small_tiles(M, N);
  if (mid > NUM_CUS || small <= NUM_CUS) return t;
  const double us = 6.5 + 0.0148 * (double)K;
  return us < (t == TILE_256x256 ? big_tiles_us(M, N, (double)K, 1) : small_tiles_us(small, (double)K)) ? TILE_256x128 : t;
}

// fp32 contraction [M, N] over K: tile and split of the contraction (fp32 slabs, summed by one
// more launch), the pair with the least modelled time.  Measured rates of one CU: a lone 64 x 64
// work-group 0.39 TFLOP/s, two or more 0.52; 128 x 128 tiles 0.50 and 0.53, at 2 us more before
// the first and behind the last MFMA; 6 us for the launch that sums the slabs, which are written
// and read at 4 TB/s.  [4096 x 3072] . [3072 x 128]: 64 x 64 unsplit 66 us, 2 ranges 38 + sum,
// 4 ranges 34 + sum, 8 ranges 33 + longer sum; 128 x 128, 8 ranges, 36 + sum.  [8192 x 512] .
// [512 x 4096]: 128 x 128 264 us, 64 x 64 276-292.
struct F32Plan {
  int tile, splits, k_per_split;
  size_t slab_bytes;   // of the slabs (0 when not split)
};
F32Plan plan_f32(int64_t M, int64_t N, int64_t K, int forced_splits, size_t max_slabs = SIZE_MAX) {
  static const int cand[] = {TILE_64x64, TILE_128x128};
  const int forced = tune(SK_TUNE_TILE);
  const bool force_tile = forced == TILE_64x64 || forced == TILE_128x128;
  const unsigned k = (unsigned)K;
  unsigned from = 1, most = k / 128 < 16 ? k / 128 : 16;   // ranges of at least 128
  if (most < 1) most = 1;
  if (forced_splits >= 0) from = most = forced_splits < 1 ? 1 : (forced_splits > (int)most ? most : forced_splits);
  struct Best {
    int64_t tiles;
    double time;
    unsigned splits, kps;
  } b[2];
  for (int c = 0; c < 2; ++c) {
    int bm, bn;
    tile_dims(cand[c], bm, bn);
    b[c] = Best{((M + bm - 1) / bm) * ((N + bn - 1) / bn), -1.0, 0, 0};
  }
  // (a call asks for several plans, a workspace query for up to two per 16 columns: the ranges are
  // worked out once for both tiles)
  for (unsigned sp = from; sp <= most; ++sp) {
    const unsigned kps = ((k + sp - 1) / sp + F32_BK - 1) / F32_BK * F32_BK;
    const unsigned splits = (k + kps - 1) / kps;
    if (splits > 1 && forced_splits < 0 && align_up((size_t)splits * M * N * 4) > max_slabs) continue;
    const double sum = splits > 1 ? 6.0e-6 + splits * (double)M * N * 8.0 / 4.0e12 : 0.0;
    for (int c = 0; c < 2; ++c) {
      const int64_t per_cu = (b[c].tiles * splits + NUM_CUS - 1) / NUM_CUS;
      const double time = (c == 0 ? per_cu * (double)kps * (2.0 * 64 * 64) / (per_cu > 1 ? 0.52e12 : 0.39e12)
                                  : per_cu * (double)kps * (2.0 * 128 * 128) / (per_cu > 1 ? 0.53e12 : 0.50e12) + 2.0e-6) + sum;
      if (b[c].time < 0.0 || time < b[c].time) { b[c].time = time; b[c].splits = splits; b[c].kps = kps; }
    }
  }
  const int c = force_tile ? (forced == cand[1]) : b[1].time < b[0].time;
  F32Plan f{};
  f.tile = cand[c]; f.splits = (int)b[c].splits; f.k_per_split = (int)b[c].kps;
  f.slab_bytes = f.splits > 1 ? align_up((size_t)f.splits * M * N * 4) : 0;
  return f;
}
F32Plan plan_f32_first(int64_t M, int64_t N, int64_t K, size_t max_slabs = SIZE_MAX) {
  return plan_f32(M, N, K, tune(SK_TUNE_SSPLITS), max_slabs);
}

// A first contraction of the layer run as a general GEMM: bf16 [M, N] result (the narrow
// intermediate, or its transpose), contraction length K.  Over a long K a small output
// leaves the choice between small tiles that fill the chip unsplit and large tiles split
// over K into fp32 slabs, which one more small kernel sums into the bf16 result.  The same
// rates as the token-split model rank the two (per work-group flop/s by tile; slabs written
// and re-read at 4 TB/s; 5 us for the extra launch), and the split form has to win by a
// tenth to be taken (measured on the 8192-wide layers: modelled ratios of 0.85 paid, 0.95
// did not).  8192-wide layer, R = 256, 4096 tokens: 54 us unsplit on 64 x 64 tiles.
struct FirstPlan {
  int tile, splits, k_per_split;
  size_t slab_bytes;   // fp32 slabs (0 when not split)
  bool few;            // the few-rows kernel
};

// Splits of a GEMM_NN or GEMM_NT [M, N] over K on the few-rows kernel, 0 where the tiles are the better
// choice.  Up to 64 rows it wins everywhere (one kernel each, us, against the tiles: [8 x 2048] .
// [2048 x 11008] 12 : 15, [64 x 1024] . [1024 x 512] 4.5 : 8); above, every 64 rows stream B again,
// and it wins while that is less than a round of short work-groups ([131 x 768] . [768 x 128] 4 : 7,
// [128 x 384] . [384 x 8192] level, [512 x 512] . [512 x 4096] 11 : 8).  An expansion wide enough for more
// rounds pays each round's start (a work-group takes a CU's LDS): calls with 528 in and 32768 out, R = 16,
// 8.6 : 8.9 at 32 tokens, 8.4 : 7.7 at 8, 131072 out 10.8 : 22.0 and 9.8 : 17.2.  Its columns lie a row of B apart,
// which for a power-of-two row is one L2 channel an XCD: past K = 3072 a first contraction gives each
// XCD a k range instead ([8 x 4096] . [4096 x 2048] 17.5 us in one range, 6.6 + 4 for the sum in eight).
int few_rows_splits(int64_t M, int64_t N, int64_t K, bool first) {
  if (M > 256 || tune(SK_TUNE_TILE) >= 0) return 0;
  const int64_t tiles = (M + 63) / 64 * ((N + 63) / 64);
  int splits = first && K > 3072 ? 8 : 1;
  while (splits > 1 && M <= 64 && tiles * splits > NUM_CUS) splits /= 2;
  if (M > 64 && (tiles > 160 || tiles * splits > NUM_CUS || tiles * K / 64 / splits > 1024)) return 0;
  if (!first && tiles > (M > 16 ? 1 : 2) * NUM_CUS) return 0;
  return splits;
}

FirstPlan plan_first(GemmKind kind, int64_t M, int64_t N, int64_t K) {
  FirstPlan f{};
  if (const int sp = kind != GEMM_TT ? few_rows_splits(M, N, K, true) : 0; sp > 0) {
    f.few = true;
    f.splits = sp;
    f.k_per_split = (int)(((K + sp - 1) / sp + 63) / 64 * 64);
    f.slab_bytes = sp > 1 ? align_up((size_t)sp * M * N * 4) : 0;
    return f;
  }
  f.tile = choose_tile(M, N, K, 1);
  f.splits = 1;
  f.k_per_split = (int)((K + 63) / 64 * 64);
  f.slab_bytes = 0;
  auto rate = [](int bm, int bn) {
    return bm * bn >= 256 * 256 ? 5.0e12 : bm * bn >= 128 * 128 ? 3.5e12 : bm * bn >= 128 * 64 ? 2.2e12 : 1.5e12;
  };
  auto time_of = [&](int tile, int64_t splits, int64_t kps) {
    int bm, bn;
    tile_dims(tile, bm, bn);
    const int64_t wgs = ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * splits;
    const int64_t rounds = (wgs + NUM_CUS - 1) / NUM_CUS;
    double t = rounds * (double)kps * 2.0 * bm * bn / rate(bm, bn);
    if (splits > 1) t += splits * (double)M * N * 8.0 / 4.0e12 + 5.0e-6;
    return t;
  };
  if (tune(SK_TUNE_TILE) >= 0) return f;  // a forced tile is taken as it is
  const double t_plain = time_of(f.tile, 1, K);
  double best = t_plain * 0.9;
  static const int cand[] = {TILE_128x128, TILE_128x64, TILE_64x128};
  for (int c = 0; c < 3; ++c) {
    int bm, bn;
    tile_dims(cand[c], bm, bn);
    if (bm > (M + 63) / 64 * 64 || bn > (N + 63) / 64 * 64) continue;
    for (int64_t sp = 2; sp <= 8; ++sp) {
      int64_t kps = (K + sp - 1) / sp;
      kps = (kps + 63) / 64 * 64;
      if (kps < 512) break;
      const int64_t sp_eff = (K + kps - 1) / kps;
      if (sp_eff < 2) continue;
      const double t = time_of(cand[c], sp_eff, kps);
      if (t < best) { best = t; f.tile = cand[c]; f.splits = (int)sp_eff; f.k_per_split = (int)kps; }
    }
  }
  if (f.splits > 1) f.slab_bytes = align_up((size_t)f.splits * M * N * 4);
  else f.tile = lone_tile(kind, f.tile, M, N, K);
  return f;
}

struct WeightPlan {
  int tile;
  int splits;
  int k_per_split;
  int64_t ldz;         // bf16: row stride of Z^T [R, ldz]
  bool own_colsum;     // db from its own kernel (the big tile has no registers for it)
  int colsum_splits;   // rows of column-sum partials: `splits`, or the own kernel's row runs
  int colsum_rows;     // tokens per row run of the own kernel
  // Uneven split (big tile only): the first head_cols output columns are one full round
  // of tiles over all tokens, straight into dU; only the rest is split over the tokens.
  int head_cols;       // 0: the whole output is split evenly (`splits`)
  int z_tile;          // bf16: tile of the GEMM that recomputes Z^T
  int z_splits;        // split of that GEMM over `in` (fp32 slabs, summed into bf16 Z^T)
  int z_k_per_split;
  // workspace: Z | slabs of dU | of db | of Z, while that fits the fixed scratch of
  // sk_linear_bwd_weight_noalloc; past it the slabs of Z, dead once summed, share the room of the
  // others.  Z^T . dY writing into lines that the sum before it has just read takes up to 2 us longer:
  // [2275 x 4800 -> 1040], R = 272, 35.3 us shared, 33.5 apart; [4096 x 8192 -> 1024], R = 128, 34.0, 32.2.
  // With more than 32 MiB in all (the L2s' 8 x 4 MiB) thirteen shapes measured the same either way.
  size_t z_bytes, part_bytes, csum_bytes, zpart_bytes;
  size_t zpart_at() const {
    const size_t behind = z_bytes + part_bytes + csum_bytes;
    return behind + zpart_bytes <= SK_NOALLOC_SCRATCH_BYTES ? behind : z_bytes;
  }
  size_t total() const {
    const size_t du_end = z_bytes + part_bytes + csum_bytes, z_end = zpart_at() + zpart_bytes;
    return du_end > z_end ? du_end : z_end;
  }
};

// A contraction over the token axis with a small fp32 output [M, N] (a weight gradient):
// tile and split of the tokens.  Every split writes and re-reads a slab of the output,
// so: as few splits as fill the chip, at least 256 tokens each, summed in a fixed
// order (deterministic).
struct TokenPlan {
  int tile;
  bool big_tile;       // 256 x 256: no registers left for column sums in the kernel
  int splits, k_per_split;
};

// Split count with the least modelled time for one tile shape: rounds of work-groups over
// the chip x tokens per split x the tile's time per token, plus writing and re-reading one
// fp32 slab per split.  Rates are measured ones (flop/s one work-group sustains; HBM
// bytes/s); the model only has to rank the candidates.
struct SplitChoice {
  double time;
  int64_t splits, kps;
};
static SplitChoice best_split(int64_t M, int64_t N, int64_t T, int bm, int bn) {
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const double wg_rate = bm * bn >= 256 * 256 ? 5.0e12
                         : bm * bn >= 128 * 128 ? 3.5e12 : bm * bn >= 128 * 64 ? 2.2e12 : 1.5e12;
  const double t_token = 2.0 * bm * bn / wg_rate;
  const double t_slab = (double)M * N * 8.0 / 4.0e12;
  int64_t max_splits = (T + 255) / 256;   // at least 256 tokens each
  if (max_splits > 32) max_splits = 32;
  const int64_t unit = bm * bn >= 256 * 256 ? 128 : 64;   // of a range: what the tile's kernel takes
  SplitChoice c{-1.0, 1, (T + unit - 1) / unit * unit};
  for (int64_t sp = 1; sp <= max_splits; ++sp) {
    int64_t k = (T + sp - 1) / sp;
    k = (k + unit - 1) / unit * unit;
    const int64_t sp_eff = (T + k - 1) / k;
    const int64_t rounds = (tiles * sp_eff + NUM_CUS - 1) / NUM_CUS;
    const double t = rounds * k * t_token + (sp_eff > 1 ? sp_eff * t_slab + 2.0e-6 : 0.0);
    if (c.time < 0.0 || t < c.time) { c.time = t; c.splits = sp_eff; c.kps = k; }
  }
  return c;
}

// `lda`: stride of the first operand's rows where it is k-contiguous (bf16 Z^T, a row of which is all
// tokens long), 0 where it is not.  Its rows of a tile have to lie within a window: past 4.2 million
// tokens 256 rows do not, past 8.4 million 128.
TokenPlan plan_tokens(int64_t M, int64_t N, int64_t T, sk_dtype dtype, bool tunable, int64_t lda,
                      size_t room = SIZE_MAX) {
  TokenPlan w{};
  if (dtype != SK_BF16) {
    const size_t sums = align_up((size_t)16 * N * 4);   // the column sums' slabs, at the most splits
    const F32Plan f = plan_f32(M, N, T, tunable ? tune(SK_TUNE_WSPLITS) : -1,
                               room == SIZE_MAX ? room : (room > sums ? room - sums : 0));
    w.tile = f.tile; w.splits = f.splits; w.k_per_split = f.k_per_split;
    return w;
  }
  int bm, bn;
  auto in_window = [&](int tile) {
    tile_dims(tile, bm, bn);
    return lda == 0 || within_window(bm, lda, bm == 256 ? T + 512 : 64, 2);
  };
  {
    w.tile = M <= 64 ? TILE_64x64 : in_window(TILE_128x64) ? TILE_128x64 : TILE_64x128;
    if (((M + 255) / 256) * ((N + 255) / 256) >= NUM_CUS && in_window(TILE_256x256)) {
      w.tile = TILE_256x256;
    } else if (w.tile == TILE_128x64) {
      // 128 x 64 or 128 x 128, whichever the model has finishing first: the narrower
      // tile fills the chip with fewer token splits (few tokens: c1, c2), the square one
      // moves fewer bytes per flop (from half a chip of tiles on, or many tokens:
      // [65536 x 768 -> 3072], R = 128 measured 152 -> 132 us)
      if (best_split(M, N, T, 128, 128).time < best_split(M, N, T, 128, 64).time)
        w.tile = TILE_128x128;
    }
    if (const int t = tunable ? forced_tile(SK_TUNE_WTILE) : -1; t >= 0 && in_window(t)) w.tile = t;  // forced
    w.big_tile = w.tile == TILE_256x256;
    tile_dims(w.tile, bm, bn);
  }
  const SplitChoice c = best_split(M, N, T, bm, bn);
  int64_t splits = c.splits, kps = c.kps;
  int64_t max_splits = (T + 255) / 256;
  if (max_splits > 32) max_splits = 32;
  if (const int f = tunable ? tune(SK_TUNE_WSPLITS) : -1; f >= 0) {  // forced (clamped to 1..max)
    splits = f < 1 ? 1 : (f > max_splits ? max_splits : f);
    const int64_t unit = w.big_tile ? 128 : 64;
    kps = ((T + splits - 1) / splits + unit - 1) / unit * unit;
    splits = (T + kps - 1) / kps;
  }
  w.splits = (int)splits;
  w.k_per_split = (int)kps;
  return w;
}

// dU = Z^T . dY with Z recomputed: where its pieces live in the workspace.
WeightPlan plan_weight(const Shape& s) {
  WeightPlan w{};
  w.ldz = s.dtype == SK_BF16 ? (s.T + 63) / 64 * 64 : s.R;
  w.z_bytes = align_up((size_t)(s.dtype == SK_BF16 ? s.R * w.ldz * 2 : s.T * s.R * 4));
  const TokenPlan t = plan_tokens(s.R, s.out, s.T, s.dtype, true, w.ldz, slab_room(w.z_bytes));
  w.tile = t.tile;
  w.own_colsum = t.big_tile;
  w.z_splits = 1;
  w.z_k_per_split = (int)s.in;
  if (s.dtype == SK_BF16) {
    // Z^T [R, T] recomputed as a general GEMM over `in` (plan_first: split over a long
    // `in` when its tiles are few -- the paper's 8192-wide layers at R = 16: 64 tiles of
    // 64 x 64 walking 128 chunks each took 51 us, four ranges and the sum take 17)
    const FirstPlan f = plan_first(GEMM_TT, s.R, s.T, s.in);
    w.z_tile = f.tile;
    w.z_splits = f.splits;
    w.z_k_per_split = f.k_per_split;
    w.zpart_bytes = w.z_splits > 1 ? align_up((size_t)w.z_splits * s.R * w.ldz * 4) : 0;
  } else {
    const F32Plan f = plan_f32_first(s.T, s.R, s.in, slab_room(w.z_bytes));   // Z = x . S_cat, split like any first GEMM
    w.z_splits = f.splits;
    w.zpart_bytes = f.slab_bytes;
  }
  const int64_t splits = t.splits, kps = t.k_per_split;
  w.splits = (int)splits;
  w.k_per_split = (int)kps;
  w.colsum_splits = w.splits;
  w.colsum_rows = w.k_per_split;
  if (w.own_colsum) {
    // the column-sum kernel splits the tokens by itself, enough to fill the chip
    const int64_t col_groups = (s.out + 511) / 512;
    int64_t cs = (4 * NUM_CUS + col_groups - 1) / col_groups;
    const int64_t max_cs = (s.T + 127) / 128;
    if (cs > max_cs) cs = max_cs;
    if (cs > 48) cs = 48;
    if (cs < 1) cs = 1;
    int64_t rows = (s.T + cs - 1) / cs;
    rows = (rows + 31) / 32 * 32;
    w.colsum_rows = (int)rows;
    w.colsum_splits = (int)((s.T + rows - 1) / rows);
  }
  w.head_cols = 0;
  if (w.own_colsum && splits > 1 && s.R <= 65535 && tune(SK_TUNE_WSPLITS) < 0) {
    // More tiles than CUs but fewer than two rounds (c4: 344 tiles of 256 x 256): a round of
    // whole-token tiles covering as many tile columns as fit, then the remaining columns
    // split over the tokens so that they fill one more, shorter round.  Against the even
    // split that is the same MFMA time with a fraction of the slabs (c4: 2 x 90 MB -> 2 x 23 MB).
    const int64_t tm = (s.R + 255) / 256, tn = (s.out + 255) / 256;
    const int64_t head_tn = NUM_CUS / tm;
    if (tm * tn > NUM_CUS && tm * tn < 2 * NUM_CUS && head_tn >= 1 && head_tn < tn &&
        head_tn * tm * 4 >= NUM_CUS * 3) {
      const int64_t tail_tiles = (tn - head_tn) * tm;
      int64_t sp = NUM_CUS / tail_tiles;
      if (sp > (s.T + 1023) / 1024) sp = (s.T + 1023) / 1024;
      if (sp > 8) sp = 8;
      if (sp >= 2) {
        int64_t k2 = ((s.T + sp - 1) / sp + 127) / 128 * 128;
        w.head_cols = (int)(head_tn * 256);
        w.splits = (int)((s.T + k2 - 1) / k2);
        w.k_per_split = (int)k2;
      }
    }
  }
  const int64_t split_cols = s.out - w.head_cols;
  w.part_bytes = w.splits > 1 ? align_up((size_t)w.splits * s.R * split_cols * 4) : 0;
  w.csum_bytes = w.colsum_splits > 1 ? align_up((size_t)w.colsum_splits * s.out * 4) : 0;
  return w;
}

// Kernel plans of the forward and the input gradient.
enum Plan : int {
  PLAN_AUTO = 0,
  PLAN_FUSED = 1,         // one kernel, intermediate tile never leaves the chip (bf16, R <= 256)
  PLAN_TWO_GEMM = 2,      // two general GEMMs, bf16/fp32 intermediate through the workspace
  PLAN_SPLIT_EXPAND = 3,  // split-K sketch GEMM into fp32 slabs, then the expand kernel that
                          // sums them on the way into LDS (bf16, R <= 512)
};

// Shape of the expand/fused launch: rows of a token tile and the number of N slices (one
// work-group per CU).
struct ChainShape {
  int bm, slices;
};
ChainShape chain_shape(int64_t T, int64_t N, int R, bool share_cu) {
  ChainShape c;
  // 128-row token tiles halve the B2 traffic and the LDS reads per MFMA of stage 2; they
  // pay once their tiles alone fill the chip (measured on [T x 768 -> 3072], R = 128:
  // forward -14..16 % from 65536 tokens on, +17 % at 4096 tokens, where they double the
  // number of work-groups that repeat stage 1)
  c.bm = (R <= 128 && T >= 128 * (int64_t)NUM_CUS) ? 128 : 64;
  if (const int v = tune(SK_TUNE_BM); v == 64 || (v == 128 && R <= 128)) c.bm = v;  // forced
  const int64_t tiles_m = (T + c.bm - 1) / c.bm;
  const int64_t n_tiles = (N + chain_bn(R) - 1) / chain_bn(R);
  int64_t sl = NUM_CUS / tiles_m;
  // share_cu: the expansion alone (no first contraction to repeat per slice, no carried
  // reduction to deal out) of a sketch up to 64 wide is small enough in LDS for two
  // work-groups per CU (8192-wide layer, R = 16: input gradient 39.8 -> 33.5 us)
  if (share_cu && R <= 64) sl = 2 * NUM_CUS / tiles_m;
  // No work-group walks more than 24 output tiles: with many tokens and a wide output every
  // CU otherwise streams its own 64 rows end to end, 16384 rows are being written at once
  // and the stores crawl ([65536 x 8192 -> 8192], R = 128: forward 1030 us with one run of
  // 64 tiles per token tile, 550 us with four runs of 16)
  if (sl < (n_tiles + 23) / 24) sl = (n_tiles + 23) / 24;
  if (const int v = tune(SK_TUNE_SLICES); v >= 0) sl = v;  // forced (clamped below)
  if (sl > n_tiles) sl = n_tiles;
  if (sl < 1) sl = 1;
  c.slices = (int)sl;
  return c;
}

Plan pick_plan(const Shape& s, sk_op op, bool workspace) {
  const int forced = g_plan.load(std::memory_order_relaxed);
  const bool chain_ok = s.dtype == SK_BF16 && chain_supported(s.R);
  const bool fused_ok = chain_ok && s.R <= CHAIN_FUSED_MAX_R;
  switch (forced) {
    case PLAN_FUSED: return fused_ok ? PLAN_FUSED : (chain_ok ? PLAN_SPLIT_EXPAND : PLAN_TWO_GEMM);
    case PLAN_TWO_GEMM: return PLAN_TWO_GEMM;
    case PLAN_SPLIT_EXPAND: return chain_ok ? PLAN_SPLIT_EXPAND : PLAN_TWO_GEMM;
    default: break;
  }
  // automatic (measured on MI355X): the on-chip plans win while the sketch is narrow
  // (R <= 128: the layer is bound by bytes and by launch count); wider sketches run
  // faster as two general GEMMs with large tiles.  One fused kernel recomputes the first
  // contraction once per N slice, which is cheap while length x slices stays small: up to
  // about 6000 (the forward of an up-projection at 4096 tokens: 768 x 4; its input
  // gradient, 3072 long, from two slices down, i.e. from 6144 tokens on, where it
  // measured level at two slices and 16-20 % ahead at one).  Beyond that the first
  // contraction is split over its length instead and the expansion sums the slabs.
  const int64_t k1 = op == SK_OP_FWD ? s.in : s.out;
  const int64_t n2 = op == SK_OP_FWD ? s.out : s.in;
  // Few tokens: two launches of the few-rows kernel beat the single fused one past a short first
  // contraction ([8 x 768] -> 768, R = 32: 6.6 us against 8.1; [131 x 768] -> 3072, R = 128: 8.4 against
  // 11.8 split), which stays for callers without a workspace.  A walk of the fused kernel takes two chunks
  // at a time, 0.65 us (forward) or 0.55 each up to R = 64, 0.85 or 0.7 above, on top of 4.1 to 5 us; the two
  // launches take 6.2 to 7 us whatever they do.  1 to 256 tokens, 64 to 8192 wide, fused : few rows: K = 128
  // 4.7-5.7 : 6.2-7.8, K = 384, R = 32, 5.9-6.2 : 6.2-7.1, K = 512 the forward of 1 to 16 tokens 6.6-6.9 : 6.2
  // and the rest 6.2-7.3 : 6.7-8.3, K = 640 level but for the gradient past 32 tokens, 6.8-7.9 : 7.1-8.7; R = 128, K = 256 6.2-7.5 : 6.9-8.1, K = 384 7.0-8.5 : 6.9-8.5.
  if (s.dtype == SK_BF16 && workspace && few_rows_splits(s.T, s.R, k1, true) > 0 && few_rows_splits(s.T, n2, s.R, false) > 0) {
    const int64_t walk = (k1 + 127) / 128;
    const bool brief = s.R > 64 ? walk <= 2 : walk <= 3 + (op != SK_OP_FWD) + (s.T > 32);
    if (s.R <= 128 && brief) return PLAN_FUSED;
    // Past 32 tokens a narrow sketch's first launch, one work-group per 64 rows, takes 1.9 us per 1000 of
    // the contraction: beyond 1792 the split sketch is ahead (42 tokens, 672 out, R = 16: K = 1536 9.2 split :
    // 8.8, 2048 9.2 : 9.6, 2944 9.8 : 11.3, 4096 10.5 : 11.4), where the chain plans would take it.
    if (s.R > 64 || s.T <= 32 || k1 <= 1792 || k1 * chain_shape(s.T, n2, s.R, false).slices <= 6144) return PLAN_TWO_GEMM;
  }
  if (chain_ok && s.R <= 128) {
    // ... and, the walk of a work-group on rings being the shorter one, a contraction of up to 1536 in one round of them at
    // any number of slices past the few tokens above (fused : split, us: 4053 tokens, 1280 -> 2144, R = 48 13.1 : 17.3; 3813,
    // 1344 <- 2912, R = 128 18.5 : 25.0; 1064, 1344 -> 5168, R = 128 13.5 : 17.0; 417, 1408 <- 832, R = 64 8.9 : 9.2; 300,
    // 1792 -> 4096, R = 32 10.1 : 9.0; from 2500 on split is ahead nearly always, 1693, 3520 <- 496 15.8 : 9.6).
    const ChainShape c = chain_shape(s.T, n2, s.R, false);
    const int64_t groups = (s.T + c.bm - 1) / c.bm * c.slices;
    const bool one_round = groups <= NUM_CUS;
    // Past a round a longer walk is fused where no slice repeats it and no round is nearly empty: above R = 64 at any number
    // of work-groups, up to R = 64 from one and a half rounds on (such work-groups share a CU, so a few past a round make it
    // last twice as long).  470 layers of 8192 to 70000 tokens, contractions of 1552 to 6144, time fused over split, median (least to most):
    // 64-row tiles R > 64 0.94 (0.82-1.02), R <= 64 up to 1.5 rounds 1.06 (0.91-1.20); 128-row tiles R > 64 0.87 (0.70-1.00), R <= 64
    // up to 1.5 rounds 1.04 (0.93-1.20), past it 0.88 (0.80-1.02); two and more slices, 64 rows 1.12 (0.95-1.57), 128 rows 1.02 (0.92-1.29).
    // Input gradient of 65536 tokens, 768 -> 3072, R = 128 125 : 147 us; of 10442, 5136 -> 2928, R = 64 (two slices) 75 : 48.
    const bool long_walk = c.slices == 1 && (s.R > 64 || groups * 2 > 3 * NUM_CUS);
    // (a caller without a workspace has no other plan)
    if (k1 * c.slices <= 6144 ? one_round || k1 <= 1536 || long_walk || !workspace : one_round && k1 <= 1536 && s.T > 256) return PLAN_FUSED;
    return PLAN_SPLIT_EXPAND;
  }
  return PLAN_TWO_GEMM;
}

// Split of the first contraction (M = tokens, N = R, contraction length K) so that a
// skinny output still fills the chip: fp32 slabs, one per k range, summed in order by
// the consumer.  splits == 1 means the bf16 result is written directly.
struct SketchPlan {
  int tile, splits, k_per_split;
  size_t bytes;
};

SketchPlan plan_sketch(const Shape& s, int64_t K) {
  SketchPlan q{};
  q.tile = s.R <= 64 ? TILE_64x64 : (s.R <= 256 ? TILE_64x128 : TILE_128x128);
  if (const int t = tune(SK_TUNE_STILE);  // forced
      t == TILE_64x64 || t == TILE_64x128 || t == TILE_128x128 || t == TILE_128x64)
    q.tile = t;
  int bm, bn;
  tile_dims(q.tile, bm, bn);
  const int64_t tiles = ((s.T + bm - 1) / bm) * ((s.R + bn - 1) / bn);
  // one work-group per CU; two for the 64 x 64 tile (R <= 64), whose work-groups are small
  // enough to share a CU and, streaming a long x from HBM, need the loads in flight of
  // two (8192-wide layer, R = 16: forward 36.8 -> 33.5 us)
  const int64_t want = s.R <= 64 ? 2 * NUM_CUS : NUM_CUS;
  int64_t splits = (want + tiles - 1) / tiles;
  if (const int v = tune(SK_TUNE_SSPLITS); v >= 0) splits = v;  // forced (clamped below)
  const int64_t max_splits = K / 128 > 0 ? K / 128 : 1;   // at least two k chunks each
  if (splits > max_splits) splits = max_splits;
  if (splits > 8) splits = 8;
  if (splits < 1) splits = 1;
  int64_t kps = (K + splits - 1) / splits;
  kps = (kps + 63) / 64 * 64;
  splits = (K + kps - 1) / kps;
  q.splits = (int)splits;
  q.k_per_split = (int)kps;
  q.bytes = splits > 1 ? align_up((size_t)splits * s.T * s.R * 4) : align_up((size_t)s.T * s.R * 2);
  return q;
}

// Workspace of the first-stage gradient for nc columns: G = dY . U_sub^T [T, nc] in the
// storage type, then the token-split slabs of dA [in, nc].
size_t first_stage_bytes(const Shape& s, int64_t nc) {
  const TokenPlan t = plan_tokens(s.in, nc, s.T, s.dtype, false, 0);
  const size_t da_slabs = t.splits > 1 ? align_up((size_t)t.splits * s.in * nc * 4) : 0;
  // slabs of G when its GEMM is split over `out`: dead once summed, so they share the
  // region of the dA slabs
  size_t g_slabs;
  if (s.dtype == SK_BF16) {
    g_slabs = plan_first(GEMM_NT, s.T, nc, s.out).slab_bytes;
  } else {
    g_slabs = plan_f32_first(s.T, nc, s.out).slab_bytes;
  }
  return align_up((size_t)s.T * nc * s.esize) + (da_slabs > g_slabs ? da_slabs : g_slabs);
}

// Both gradients of a narrow sketch in one pass over x and dY (sk_bwd_narrow.hip): a
// work-group per tile of 32 or 64 tokens produces its rows of dX outright and leaves one
// fp32 slab of dU_cat (and of dbias) behind, which a second kernel sums; G never leaves the
// chip and three launches become two.  A work-group is four waves on a CU of its own, so
// nothing hides its latencies but its own prefetching, and it takes 13-18 us for its tile
// whatever the token count; a second round of work-groups doubles that.  Measured on MI355X
// (in = out = 768, R = 32, backward call; 32-token tiles / 64-token tiles / the three-launch
// schedule, us): 512 tokens 16.2 / - / 20.7, 2048 18.4 / 22.1 / 22.6, 4096 21.1 / 24.4 /
// 23.2, 8192 25.9 / 27.5 / 30.5, 12288 41.4 / 30.7 / 35.4, 16384 46.3 / 34.8 / 38.8, 20480
// - / 52.9 / 44.5; R = 64 (a variant of the kernel since removed) lost at every size.
// A sweep over in = 64..768 and out = 64..3072 at 256..16384 tokens (same call, one pass
// over three launches): out <= 256 0.63-0.84, out = 768 0.80-1.04, out = 1024 0.83-1.14
// (R = 16: 0.82-1.03), out = 2048 1.06-1.31, out = 3072 1.20-1.59 -- a work-group walks all
// of `out`, and the walk is what it cannot hide.
// So: R <= 32, out <= 896 (1024 for R = 16), one round of work-groups, slabs of at most 32 MiB, and not where bwd_both
// has the gradients share launches instead (`shares` there).
struct NarrowPlan {
  bool ok;
  int tm, tiles_m;   // tokens per work-group (32 or 64), work-groups
  size_t du_bytes, db_bytes;
  size_t total() const { return du_bytes + db_bytes; }
};

NarrowPlan plan_narrow(const Shape& s) {
  NarrowPlan n{};
  const int forced = tune(SK_TUNE_NARROW_BWD);
  if (s.dtype != SK_BF16 || g_plan.load(std::memory_order_relaxed) != PLAN_AUTO || forced == 0) return n;
  if (s.in > narrow_bwd_max_in(s.R)) return n;   // (0 for a sketch the kernel does not serve)
  // 32-token tiles while they make one round of work-groups with slabs under the cap, 64-token
  // tiles beyond; only while a work-group's walk over `out` stays short
  for (int tm = 32; tm <= 64; tm *= 2) {
    if ((forced == 32 || forced == 64) && tm != forced) continue;
    const int64_t tiles_m = (s.T + tm - 1) / tm;
    const size_t du = (size_t)tiles_m * s.R * s.out * 4;
    const bool fits = du <= ((size_t)32 << 20) && tiles_m <= NUM_CUS && s.out <= (s.R <= 16 ? 1024 : 896);
    if (forced < 0 && !fits) continue;
    if (forced > 0 && forced != 32 && forced != 64 && !fits && tm == 32) continue;   // forced without a tile height: 64 unless 32 fits
    n.ok = true;
    n.tm = tm;
    n.tiles_m = (int)tiles_m;
    n.du_bytes = align_up(du);
    n.db_bytes = align_up((size_t)tiles_m * s.out * 4);
    return n;
  }
  return n;
}

// Backward pass of a wide sketch in shared launches: dY.U^T beside Z^T on one tile, each in ranges or not, the sums of those in a launch,
// then Z^T.dY beside G.S^T.
struct WidePlan {
  int tile;                      // of the first two, -1: none
  int g_splits, g_k_per_split;   // ranges of dY.U^T
  int du_tile, dx_tile;
};

// Apart, the two gradients of a layer take five to seven launches, most of which leave CUs without a work-group or with one that waits;
// beside each other two to four.  The ranges of Z^T and of the tokens stay those of the separate calls (dU and db come out
// the same), those of dY.U^T are as many as its slabs have room for.  The first two have one result size, so one tile
// serves both, the one with the least modelled time: all chunks at the rate of a CU with company (its fill: 0.62 us
// a chunk of a 128 x 128 tile, 0.27 of a 64 x 64 one) or the longest walk of a CU (0.65, 0.36 by itself, of more than a round half way between
// an even share of them and the whole number that the fullest CU has), whichever is more, and slabs at 4 TB/s and 2.5 us for the launch
// that sums them.  64 x 64 tiles past two work-groups a CU run on the staged loop, which long walks of dY.U^T keep waiting: 0.33.
// (Fitted to the first launch and its sums of 250 layers over every tile and range: 1.017 of the best choice's time at the mean, one in eight more than 5 %
// behind; without the fullest CU and the staged rate 1.031 and one in five, up to 1.5.)  Backward pass, us, those two out : in: 7024 tokens,
// 256 -> 6000, R = 192 104 : 86; 1383, 96 -> 7408, R = 992 105 : 86; 2142, 1360 -> 2992, R = 576 58.7 : 50.7; 110 of 1200 layers took another pair, in 0.95
// of the time (0.82 to 1.04).
// Backward pass, us, apart : shared: 735 tokens, 560 -> 592, R = 432 23.2 : 14.7; 2777, 3376 -> 4800,
// R = 1360 202 : 155; 2302, 3744 -> 7200, R = 672 151 : 117; 99 of 150 layers of 512 to 16384 tokens, 512 to 4096 wide, R 144 to
// 512, were apart, now 0.78 of the time, 24 of 50 of 2048 to 16384 tokens, R 512 to 2048, 0.86, all of 257 to 600 tokens 0.69, the rest within
// 2 %.  Layers that shared launches before on tiles of two models of their own: 0.997 (0.87 to 1.02).  390 more layers of up to 400
// inputs and 2000 to 8192 outputs, where there is little to share: 0.86, eight of them 2 to 6 % behind.
// None where one of the first two takes the 256 x 256 tile by itself (see sk_linear_bwd), or where dX does and is modelled more than 24 us ahead on it:
// 12520 tokens, 7296 -> 144, R = 352 223 : 234; 14077, 8080 -> 1216, R = 320 302 : 317; ten such layers 0.99 to 1.05, from 15 to 24 us 0.80 to 1.04 (mean 0.95).
WidePlan plan_wide(const Shape& s, const WeightPlan& w, const FirstPlan& first) {
  WidePlan best{-1, 1, 0, 0, 0};
  if (tune(SK_TUNE_TILE) >= 0 || choose_tile(s.T, s.R, s.out, 1) == TILE_256x256 || choose_tile(s.R, s.T, s.in, 1) == TILE_256x256) return best;
  best.du_tile = w.tile;
  best.dx_tile = choose_tile(s.T, s.in, s.R, 1);
  if (best.dx_tile == TILE_256x256 && small_tiles_us(small_tiles(s.T, s.in), (double)s.R) - big_tiles_us(s.T, s.in, (double)s.R, 1) > 24.0) return best;
  if (w.tile == TILE_128x128 || best.dx_tile == TILE_256x256) best.dx_tile = TILE_128x128;
  else if (best.dx_tile == TILE_64x128) best.dx_tile = TILE_128x64;
  if (!dual_gemm_supported(GEMM_NN_F32_COLSUM, best.du_tile, GEMM_NT, best.dx_tile)) return best;
  double least = -1.0;
  const double z_walk = (double)((s.in / w.z_splits + 63) / 64);
  for (const int tile : {TILE_128x128, TILE_64x64}) {
    const int side = tile == TILE_128x128 ? 128 : 64;
    const int64_t tiles = ((s.T + side - 1) / side) * ((s.R + side - 1) / side);
    for (int sp = 1; sp <= first.splits; ++sp) {
      const int64_t kps = ((s.out + sp - 1) / sp + 63) / 64 * 64;
      if ((s.out + kps - 1) / kps != sp) continue;
      const bool staged = tiles * (sp + w.z_splits) > 2 * NUM_CUS && w.z_splits == 1 && s.out >= 1024;
      const double shared = tile == TILE_128x128 ? 0.62 : staged ? 0.33 : 0.27, alone = tile == TILE_128x128 ? 0.65 : 0.36;
      auto walks = [&](int64_t groups, double chunks) {
        const double deep = 0.5 * ((double)groups / NUM_CUS + (double)((groups + NUM_CUS - 1) / NUM_CUS));
        return chunks * (groups > NUM_CUS && deep * shared > alone ? deep * shared : alone);
      };
      const double g_walk = (double)(kps / 64), all = tiles * (sp * g_walk + w.z_splits * z_walk) * shared / NUM_CUS;
      const double g_us = walks(tiles * sp, g_walk), z_us = walks(tiles * w.z_splits, z_walk), longest = g_us > z_us ? g_us : z_us;
      const double us = (all > longest ? all : longest) + (sp > 1 ? (w.z_splits > 1 ? 0.0 : 2.5) + sp * (double)s.T * s.R * 8.0 / 4.0e6 : 0.0);
      if (least < 0.0 || us < least) { least = us; best.tile = tile; best.g_splits = sp; best.g_k_per_split = (int)kps; }
    }
  }
  return best;
}

size_t workspace_for(sk_op op, const Shape& s) {
  const size_t mid = align_up((size_t)s.T * s.R * s.esize);  // Z or G
  switch (op) {
    case SK_OP_FWD:
    case SK_OP_BWD_INPUT: {
      // the maximum over the plans, so one buffer serves whichever is selected
      size_t need = mid;
      if (s.dtype == SK_BF16)   // two GEMMs with the first one split: slabs behind the intermediate
        need += plan_first(op == SK_OP_FWD ? GEMM_NN : GEMM_NT, s.T, s.R, op == SK_OP_FWD ? s.in : s.out).slab_bytes;
      else
        need += plan_f32_first(s.T, s.R, op == SK_OP_FWD ? s.in : s.out).slab_bytes;
      if (s.dtype == SK_BF16 && chain_supported(s.R)) {
        const size_t b = plan_sketch(s, op == SK_OP_FWD ? s.in : s.out).bytes;
        if (b > need) need = b;
      }
      return need;
    }
    case SK_OP_BWD_WEIGHT:
      return plan_weight(s).total();
    case SK_OP_BWD: {
      const size_t two = workspace_for(SK_OP_BWD_INPUT, s) + workspace_for(SK_OP_BWD_WEIGHT, s);
      const NarrowPlan n = plan_narrow(s);
      return n.ok && n.total() > two ? n.total() : two;
    }
    case SK_OP_BWD_TWO_SIDED:   // both gradients' | what the first-stage gradient of half the columns takes by itself
      return s.R % 32 == 0 ? workspace_for(SK_OP_BWD, s) + first_stage_bytes(s, s.R / 2) : 0;
    case SK_OP_BWD_WEIGHT_FIRST: {
      // the maximum over every admissible column count (narrow ranges split the tokens
      // further), so one buffer serves any range
      size_t need = 0;
      for (int64_t nc = 16; nc <= s.R; nc += 16) {
        const size_t b = first_stage_bytes(s, nc);
        if (b > need) need = b;
      }
      return need;
    }
  }
  return 0;
}

hipError_t gemm(const Shape& s, GemmKind kind, GemmArgs a, hipStream_t st) {
  if (s.dtype == SK_BF16 && few_rows_splits(a.M, a.N, a.K, false) > 0) return launch_gemm_few_rows_bf16(kind, a, st);
  if (s.dtype == SK_BF16) return launch_gemm_bf16(kind, choose_expansion_tile(kind, a.M, a.N, a.K), a, st);
  return launch_gemm_f32(kind, plan_f32(a.M, a.N, a.K, 1).tile, a, st);
}

// The first of the two GEMMs of a call: as it is, or (bf16, plan_first) split over its
// contraction into fp32 slabs at `slabs` that are then summed into the bf16 result a.C.
hipError_t first_gemm(const Shape& s, GemmKind kind, GemmKind kind_slabs, GemmArgs a, void* slabs,
                      hipStream_t st, size_t max_slabs = SIZE_MAX) {
  if (s.dtype != SK_BF16) {
    const F32Plan f = plan_f32_first(a.M, a.N, a.K, max_slabs);
    if (f.splits == 1) return launch_gemm_f32(kind, f.tile, a, st);
    // fp32: the same kernel writes the slabs (one per range of the contraction); summed in order
    float* out = static_cast<float*>(a.C);
    a.C = slabs; a.splits = f.splits; a.k_per_split = f.k_per_split;
    const hipError_t e = launch_gemm_f32(kind, f.tile, a, st);
    if (e != hipSuccess) return e;
    ReduceArgs r{};
    r.part = static_cast<const float*>(slabs); r.out = out; r.n = (int64_t)a.M * a.N; r.scale = 1.0f;
    r.splits = a.splits; r.splits2 = 1; r.scale2 = 1.0f;
    return launch_reduce_splits(r, st);
  }
  const FirstPlan f = plan_first(kind, a.M, a.N, a.K);
  if (f.splits == 1) return f.few ? launch_gemm_few_rows_bf16(kind, a, st) : launch_gemm_bf16(kind, f.tile, a, st);
  void* out = a.C;
  a.C = slabs; a.splits = f.splits; a.k_per_split = f.k_per_split;
  const hipError_t e = f.few ? launch_gemm_few_rows_bf16(kind, a, st) : launch_gemm_bf16(kind_slabs, f.tile, a, st);
  if (e != hipSuccess) return e;
  return launch_reduce_to_bf16(static_cast<const float*>(slabs), out, (int64_t)a.M * a.N, f.splits, st);
}

// C[M,N] = scale * (A[M,K] . B) + bias through the workspace-free single GEMM.
GemmArgs dense_args(const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc,
                    int64_t M, int64_t N, int64_t K, float scale, const void* bias) {
  GemmArgs a{};
  a.A = A; a.B = B; a.C = C; a.bias = bias; a.colsum = nullptr;
  a.lda = lda; a.ldb = ldb; a.ldc = ldc;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)((K + 63) / 64 * 64);
  a.splits = 1;
  a.scale = scale;
  return a;
}


// The last columns of G = dY . U_cat^T in the storage type, as a backward pass may leave them behind: `at` is null where
// its schedule does not form them.  With them the two-sided layer's first-stage gradient is one product instead of two:
// 4096 tokens, 768 -> 3072, R = 128, the whole backward pass 52.1 -> 39.9 us, seventeen drawn layers 1.18 times as fast.
struct GColumns {
  int64_t first;     // the first column asked for
  void* room;        // [tokens, R - first] in the storage type, for a schedule that keeps G elsewhere
  const void* at;
  int64_t ld;
  void take(const unsigned char* G, const Shape& s) {   // from the whole of G
    at = G + (size_t)first * s.esize;
    ld = s.R;
  }
};

// Where a backward pass leaves the gradients of the factors, the bias and the first stage for a launch that sums and rounds them: finished in
// fp32 (splits 1), or in slabs where its schedule would end with a launch for their sum.
struct Unrounded {
  struct Part {
    const float* at;
    int64_t stride;
    int splits;
    float scale;
  } du, db, da;
};

// Two fp32 products of the backward pass in one launch where both take the same tile, else in two.
hipError_t gemm_pair_f32(GemmKind kind_a, int tile_a, const GemmArgs& a, GemmKind kind_b, int tile_b, const GemmArgs& b, hipStream_t st) {
  if (tile_a == tile_b) return launch_dual_gemm_f32(kind_a, a, kind_b, b, tile_a, st);
  const hipError_t e = launch_gemm_f32(kind_a, tile_a, a, st);
  return e != hipSuccess ? e : launch_gemm_f32(kind_b, tile_b, b, st);
}

// sk_linear_bwd in fp32 (workspaces laid out as those of the two separate calls).
sk_status bwd_f32(const Shape& s, const void* x, const void* dY, const void* S_cat, const void* U_cat, void* dX, float* dU_cat,
                  float* dbias, unsigned char* ws_in, unsigned char* ws_w, GColumns* want, hipStream_t hs) {
  g_hip_error.clear();
  if (want) want->take(ws_in, s);
  const float scale = 1.0f / (float)s.l;
  const WeightPlan w = plan_weight(s);
  const F32Plan gp = plan_f32_first(s.T, s.R, s.out), zp = plan_f32_first(s.T, s.R, s.in, slab_room(w.z_bytes));
  float* const G = reinterpret_cast<float*>(ws_in);
  float* const g_slabs = reinterpret_cast<float*>(ws_in + align_up((size_t)s.T * s.R * 4));
  float* const Z = reinterpret_cast<float*>(ws_w);
  float* const z_slabs = reinterpret_cast<float*>(ws_w + w.zpart_at());
  float* const part = reinterpret_cast<float*>(ws_w + w.z_bytes);
  float* const cpart = reinterpret_cast<float*>(ws_w + w.z_bytes + w.part_bytes);

  GemmArgs g = dense_args(dY, s.out, U_cat, s.out, gp.splits > 1 ? g_slabs : G, s.R, s.T, s.R, s.out, 1.0f, nullptr);
  g.splits = gp.splits; g.k_per_split = gp.k_per_split;
  GemmArgs z = dense_args(x, s.in, S_cat, s.R, zp.splits > 1 ? z_slabs : Z, s.R, s.T, s.R, s.in, 1.0f, nullptr);
  z.splits = zp.splits; z.k_per_split = zp.k_per_split;
  hipError_t e = gemm_pair_f32(GEMM_NT, gp.tile, g, GEMM_NN, zp.tile, z, hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (dY.U^T beside x.S)");
  if (gp.splits > 1 || zp.splits > 1) {
    const int64_t n = s.T * s.R;
    ReduceArgs r{};
    r.part = g_slabs; r.out = G; r.n = gp.splits > 1 ? n : 0; r.splits = gp.splits; r.scale = 1.0f;
    r.part2 = z_slabs; r.out2 = Z; r.n2 = zp.splits > 1 ? n : 0; r.splits2 = zp.splits; r.scale2 = 1.0f;
    e = launch_reduce_splits(r, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (sums of G and Z)");
  }
  GemmArgs du{};
  du.A = Z; du.lda = s.R; du.B = dY; du.ldb = s.out; du.ldc = s.out;
  du.M = s.R; du.N = (int)s.out; du.K = (int)s.T;
  du.splits = w.splits; du.k_per_split = w.k_per_split;
  if (w.splits == 1) { du.C = dU_cat; du.colsum = dbias; du.scale = scale; }
  else { du.C = part; du.colsum = dbias ? cpart : nullptr; du.scale = 1.0f; }
  const GemmArgs dx = dense_args(G, s.R, S_cat, s.R, dX, s.in, s.T, s.in, s.R, scale, nullptr);
  e = gemm_pair_f32(GEMM_TN_F32, w.tile, du, GEMM_NT, plan_f32(s.T, s.in, s.R, 1).tile, dx, hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (Z^T.dY beside G.S^T)");
  if (w.splits > 1) {
    ReduceArgs r{};
    r.part = part; r.out = dU_cat; r.n = (int64_t)s.R * s.out; r.splits = w.splits; r.scale = scale;
    r.part2 = cpart; r.out2 = dbias; r.n2 = dbias ? s.out : 0; r.splits2 = w.splits; r.scale2 = 1.0f;
    e = launch_reduce_splits(r, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (sum of splits)");
  }
  return SK_OK;
}

// dA = (1 / l) . x^T . G for nc columns of G [tokens, nc], rows ldg apart; `part`: the slabs of split tokens.
sk_status first_stage_gradient(const Shape& s, const void* x, const void* G, int64_t ldg, int64_t nc, float* dA, float* part, hipStream_t hs,
                               Unrounded* later = nullptr) {
  // dA = scale * x^T . G, the token axis split in order
  const TokenPlan t = plan_tokens(s.in, nc, s.T, s.dtype, false, 0);
  GemmArgs a{};
  a.A = x; a.lda = s.in;
  a.B = G; a.ldb = ldg;
  a.ldc = nc;
  a.M = (int)s.in; a.N = (int)nc; a.K = (int)s.T;
  a.splits = t.splits; a.k_per_split = t.k_per_split;
  a.bias = nullptr; a.colsum = nullptr;
  const float scale = 1.0f / (float)s.l;
  if (t.splits == 1) { a.C = dA; a.scale = scale; }
  else { a.C = part; a.scale = 1.0f; }
  hipError_t e = s.dtype == SK_BF16 ? launch_gemm_bf16(GEMM_TN_F32_PLAIN, t.tile, a, hs)
                       : launch_gemm_f32(GEMM_TN_F32, t.tile, a, hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight_first (x^T.G)");
  if (t.splits > 1 && later) {
    later->da = {part, (int64_t)s.in * nc, t.splits, scale};
  } else if (t.splits > 1) {
    ReduceArgs r{};
    r.part = part; r.out = dA; r.n = (int64_t)s.in * nc; r.scale = scale;
    r.n2 = 0; r.splits = t.splits; r.splits2 = 1;
    e = launch_reduce_splits(r, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight_first (sum of splits)");
  }
  return SK_OK;
}

}  // namespace

extern "C" {

const char* sk_status_string(sk_status status) {
  switch (status) {
    case SK_OK: return "SK_OK";
    case SK_ERR_INVALID_ARG: return "SK_ERR_INVALID_ARG: null or misaligned pointer, or non-positive size";
    case SK_ERR_UNSUPPORTED: return "SK_ERR_UNSUPPORTED: unknown dtype/op, or in/out/l*k not a multiple of 16";
    case SK_ERR_WORKSPACE: return "SK_ERR_WORKSPACE: workspace missing or too small";
    case SK_ERR_HIP: return "SK_ERR_HIP: a HIP call failed (see sk_last_hip_error)";
  }
  return "unknown sk_status";
}

const char* sk_last_hip_error(void) { return g_hip_error.c_str(); }

int sk_set_plan(int plan) {
  if (plan < 0 || plan > 3) return -1;
  return g_plan.exchange(plan);
}

int32_t sk_set_tuning(sk_tune_knob knob, int32_t value) {
  if ((int)knob < 0 || (int)knob >= SK_TUNE_COUNT) return INT32_MIN;
  return g_tune[knob].exchange(value < 0 ? -1 : value);
}

void sk_trace_begin(void) {
  delete g_hooks;
  g_hooks = new Hooks();
  g_hooks->trace = true;
}

int64_t sk_trace_end(sk_trace_access* out, int64_t max, int32_t* launches) {
  if (g_hooks == nullptr || !g_hooks->trace) return 0;
  const int64_t n = (int64_t)g_hooks->accesses.size();
  for (int64_t i = 0; i < n && i < max && out != nullptr; ++i) out[i] = g_hooks->accesses[i];
  if (launches != nullptr) *launches = (int32_t)g_hooks->launches.size();
  delete g_hooks;
  g_hooks = nullptr;
  return n;
}

int32_t sk_trace_kernel(int32_t launch, char* name, int32_t max) {
  if (g_hooks == nullptr || !g_hooks->trace || launch < 0 || launch >= (int32_t)g_hooks->launches.size()) return -1;
  if (name != nullptr && max > 0) {
    strncpy(name, g_hooks->launches[launch].c_str(), max - 1);
    name[max - 1] = 0;
  }
  return (int32_t)g_hooks->groups[launch];
}

int32_t sk_profile_begin(int32_t max_kernels) {
  delete g_hooks;
  g_hooks = nullptr;
  if (max_kernels < 1) return -1;
  Hooks* h = new Hooks();
  h->max_kernels = max_kernels;
  h->events.resize(2 * (size_t)max_kernels);
  for (size_t i = 0; i < h->events.size(); ++i) {
    if (hipEventCreate(&h->events[i]) != hipSuccess) {
      for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(h->events[j]);
      delete h;
      return -2;
    }
  }
  g_hooks = h;
  return 0;
}

int32_t sk_profile_end(sk_kernel_time* out, int32_t max) {
  Hooks* h = g_hooks;
  if (h == nullptr || h->trace) return -1;
  g_hooks = nullptr;
  const int32_t n = (int32_t)h->names.size();
  int32_t rc = n;
  if (n > 0 && hipEventSynchronize(h->events[2 * (size_t)n - 1]) != hipSuccess) rc = -3;
  for (int32_t i = 0; rc >= 0 && i < n && i < max && out != nullptr; ++i) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, h->events[2 * (size_t)i], h->events[2 * (size_t)i + 1]) != hipSuccess) {
      rc = -4;
      break;
    }
    strncpy(out[i].name, h->names[i].c_str(), sizeof(out[i].name) - 1);
    out[i].name[sizeof(out[i].name) - 1] = 0;
    out[i].ms = ms;
    out[i].groups = (int32_t)h->groups[i];
    out[i].flops = h->work[i].flops;
    out[i].bytes = h->work[i].bytes;
  }
  for (hipEvent_t e : h->events) (void)hipEventDestroy(e);
  delete h;
  return rc;
}

size_t sk_linear_workspace_bytes(sk_op op, int64_t tokens, int64_t in, int64_t out, int32_t l,
                                 int32_t k, sk_dtype dtype) {
  Shape s;
  if (op != SK_OP_FWD && op != SK_OP_BWD_INPUT && op != SK_OP_BWD_WEIGHT &&
      op != SK_OP_BWD_WEIGHT_FIRST && op != SK_OP_BWD && op != SK_OP_BWD_TWO_SIDED)
    return (size_t)-1;
  if (check_shape(tokens, in, out, l, k, dtype, s) != SK_OK) return (size_t)-1;
  if (op == SK_OP_BWD_TWO_SIDED && s.R % 32 != 0) return (size_t)-1;
  return workspace_for(op, s);
}

sk_status sk_linear_fwd(const void* x, const void* S_cat, const void* U_cat, const void* bias,
                        void* y, int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k,
                        sk_dtype dtype, void* workspace, size_t workspace_bytes, void* stream) {
  if (!x || !S_cat || !U_cat || !y) return SK_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(S_cat) || !aligned16(U_cat) || !aligned16(y) ||
      !aligned16(bias) || !aligned16(workspace))
    return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const float scale = 1.0f / (float)l;
  g_hip_error.clear();

  const Plan plan = pick_plan(s, SK_OP_FWD, workspace && workspace_bytes >= workspace_for(SK_OP_FWD, s));
  if (plan != PLAN_FUSED && (!workspace || workspace_bytes < workspace_for(SK_OP_FWD, s)))
    return SK_ERR_WORKSPACE;
  if (plan == PLAN_FUSED || plan == PLAN_SPLIT_EXPAND) {
    ChainArgs c{};
    c.A = x; c.B1 = S_cat; c.B2 = U_cat; c.bias = bias; c.C = y;
    c.lda = in; c.ldb1 = s.R; c.ldb2 = out; c.ldc = out;
    c.M = (int)tokens; c.K1 = (int)in; c.R = s.R; c.N = (int)out; c.scale = scale;
    { const ChainShape cs = chain_shape(tokens, out, s.R, plan != PLAN_FUSED); c.n_slices = cs.slices; c.bm = cs.bm; }
    if (plan == PLAN_SPLIT_EXPAND) {
      const SketchPlan q = plan_sketch(s, in);
      GemmArgs a = dense_args(x, in, S_cat, s.R, workspace, s.R, tokens, s.R, in, 1.0f, nullptr);
      a.splits = q.splits; a.k_per_split = q.k_per_split;
      const hipError_t e1 = launch_gemm_bf16(q.splits > 1 ? GEMM_NN_F32 : GEMM_NN, q.tile, a, hs);
      if (e1 != hipSuccess) return hip_fail(e1, "sk_linear_fwd (x.S, split)");
      c.Z = workspace; c.z_splits = q.splits > 1 ? q.splits : 0; c.z_slab = (int64_t)tokens * s.R;
    }
    const hipError_t e = launch_chain_bf16(false, plan == PLAN_FUSED, c, hs);
    return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_fwd (expand)");
  }
  // Z = x . S_cat, then y = scale * Z . U_cat + bias
  hipError_t e;
  e = first_gemm(s, GEMM_NN, GEMM_NN_F32,
                 dense_args(x, in, S_cat, s.R, workspace, s.R, tokens, s.R, in, 1.0f, nullptr),
                 static_cast<unsigned char*>(workspace) + align_up((size_t)tokens * s.R * s.esize), hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_fwd (x.S)");
  e = gemm(s, GEMM_NN, dense_args(workspace, s.R, U_cat, out, y, out, tokens, out, s.R, scale, bias), hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_fwd (Z.U)");
  return SK_OK;
}

sk_status sk_linear_bwd_input(const void* dY, const void* S_cat, const void* U_cat, void* dX,
                              int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k,
                              sk_dtype dtype, void* workspace, size_t workspace_bytes,
                              void* stream) {
  if (!dY || !S_cat || !U_cat || !dX) return SK_ERR_INVALID_ARG;
  if (!aligned16(dY) || !aligned16(S_cat) || !aligned16(U_cat) || !aligned16(dX) ||
      !aligned16(workspace))
    return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const float scale = 1.0f / (float)l;
  g_hip_error.clear();

  const Plan plan = pick_plan(s, SK_OP_BWD_INPUT, workspace && workspace_bytes >= workspace_for(SK_OP_BWD_INPUT, s));
  if (plan != PLAN_FUSED && (!workspace || workspace_bytes < workspace_for(SK_OP_BWD_INPUT, s)))
    return SK_ERR_WORKSPACE;
  if (plan == PLAN_FUSED || plan == PLAN_SPLIT_EXPAND) {
    ChainArgs c{};
    c.A = dY; c.B1 = U_cat; c.B2 = S_cat; c.bias = nullptr; c.C = dX;
    c.lda = out; c.ldb1 = out; c.ldb2 = s.R; c.ldc = in;
    c.M = (int)tokens; c.K1 = (int)out; c.R = s.R; c.N = (int)in; c.scale = scale;
    { const ChainShape cs = chain_shape(tokens, in, s.R, plan != PLAN_FUSED); c.n_slices = cs.slices; c.bm = cs.bm; }
    if (plan == PLAN_SPLIT_EXPAND) {
      const SketchPlan q = plan_sketch(s, out);
      GemmArgs a = dense_args(dY, out, U_cat, out, workspace, s.R, tokens, s.R, out, 1.0f, nullptr);
      a.splits = q.splits; a.k_per_split = q.k_per_split;
      const hipError_t e1 = launch_gemm_bf16(q.splits > 1 ? GEMM_NT_F32 : GEMM_NT, q.tile, a, hs);
      if (e1 != hipSuccess) return hip_fail(e1, "sk_linear_bwd_input (dY.U^T, split)");
      c.Z = workspace; c.z_splits = q.splits > 1 ? q.splits : 0; c.z_slab = (int64_t)tokens * s.R;
    }
    const hipError_t e = launch_chain_bf16(true, plan == PLAN_FUSED, c, hs);
    return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_bwd_input (expand)");
  }
  // G = dY . U_cat^T (U_cat read as [N = R, K = out]), then dX = scale * G . S_cat^T
  hipError_t e = first_gemm(s, GEMM_NT, GEMM_NT_F32,
                            dense_args(dY, out, U_cat, out, workspace, s.R, tokens, s.R, out, 1.0f, nullptr),
                            static_cast<unsigned char*>(workspace) + align_up((size_t)tokens * s.R * s.esize), hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_input (dY.U^T)");
  e = gemm(s, GEMM_NT, dense_args(workspace, s.R, S_cat, s.R, dX, in, tokens, in, s.R, scale, nullptr), hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_input (G.S^T)");
  return SK_OK;
}

sk_status sk_linear_bwd_weight(const void* x, const void* S_cat, const void* dY, float* dU_cat,
                               float* dbias, int64_t tokens, int64_t in, int64_t out, int32_t l,
                               int32_t k, sk_dtype dtype, void* workspace,
                               size_t workspace_bytes, void* stream) {
  if (!x || !S_cat || !dY || !dU_cat) return SK_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(S_cat) || !aligned16(dY) || !aligned16(dU_cat) ||
      !aligned16(dbias) || !aligned16(workspace))
    return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  const WeightPlan w = plan_weight(s);
  if (!workspace || workspace_bytes < workspace_for(SK_OP_BWD_WEIGHT, s)) return SK_ERR_WORKSPACE;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const float scale = 1.0f / (float)l;
  g_hip_error.clear();

  unsigned char* ws = static_cast<unsigned char*>(workspace);
  void* Z = ws;
  float* part = reinterpret_cast<float*>(ws + w.z_bytes);
  float* cpart = reinterpret_cast<float*>(ws + w.z_bytes + w.part_bytes);

  // Z = x . S_cat is recomputed here rather than kept from the forward pass.  In bf16
  // it is produced transposed (Z^T = S_cat^T . x^T, [R, ldz] with zero-filled row
  // padding) so that the token contraction below reads it k-contiguous.
  GemmArgs a{};
  hipError_t e;
  if (s.dtype == SK_BF16) {
    GemmArgs z = dense_args(S_cat, s.R, x, in, Z, w.ldz, s.R, tokens, in, 1.0f, nullptr);
    z.n_store = (int)w.ldz;
    if (w.z_splits > 1) {
      float* zpart = reinterpret_cast<float*>(ws + w.zpart_at());
      z.C = zpart; z.splits = w.z_splits; z.k_per_split = w.z_k_per_split;
      e = launch_gemm_bf16(GEMM_TT_F32, w.z_tile, z, hs);
      if (e == hipSuccess) e = launch_reduce_to_bf16(zpart, Z, (int64_t)s.R * w.ldz, w.z_splits, hs);
    } else {
      e = launch_gemm_bf16(GEMM_TT, w.z_tile, z, hs);
    }
    a.A = Z; a.lda = w.ldz;
  } else {
    e = first_gemm(s, GEMM_NN, GEMM_NN_F32, dense_args(x, in, S_cat, s.R, Z, s.R, tokens, s.R, in, 1.0f, nullptr),
                   ws + w.zpart_at(), hs, slab_room(w.z_bytes));
    a.A = Z; a.lda = s.R;
  }
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight (x.S)");

  // dU = scale * Z^T . dY and db = column sums of dY, the token axis split in order
  a.B = dY; a.ldb = out; a.ldc = out;
  a.M = s.R; a.N = (int)out; a.K = (int)tokens;
  a.splits = w.splits; a.k_per_split = w.k_per_split;
  a.bias = nullptr;
  if (w.splits == 1) {
    a.C = dU_cat; a.colsum = dbias; a.scale = scale;
  } else {
    a.C = part; a.colsum = dbias ? cpart : nullptr; a.scale = 1.0f;
  }
  if (s.dtype == SK_BF16 && w.own_colsum) {
    // the bias gradient from its own kernel -- or, with the uneven split, inside the launch of
    // the second, shorter round, whose GEMM leaves CUs free
    GemmArgs tail = a;
    tail.N = (int)out - w.head_cols;
    const bool ride = dbias && w.head_cols > 0 && gemm256_supported(GEMM_NN_F32, tail);
    if (dbias && !ride) {
      e = launch_colsum_bf16(dY, w.colsum_splits == 1 ? dbias : cpart, (int)tokens, (int)out,
                             w.colsum_splits, w.colsum_rows, hs);
      if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight (column sums)");
    }
    if (w.head_cols > 0) {
      // first round: whole-token tiles of the first head_cols columns, straight into dU
      GemmArgs hd = a;
      hd.N = w.head_cols; hd.C = dU_cat; hd.colsum = nullptr; hd.scale = scale;
      hd.splits = 1; hd.k_per_split = (int)((tokens + 63) / 64 * 64);
      e = launch_gemm_bf16(GEMM_NN_F32, w.tile, hd, hs);
      if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight (Z^T.dY, first columns)");
      // second, shorter round: the remaining columns, split over the tokens into slabs
      a.B = static_cast<const unsigned char*>(dY) + (size_t)w.head_cols * s.esize;
      a.N = (int)out - w.head_cols; a.ldc = a.N; a.C = part; a.colsum = nullptr; a.scale = 1.0f;
    }
    a.colsum = nullptr;   // (the big tiles have no column-sum epilogue: that is what the kernel above is for)
    if (ride)
      e = launch_gemm256_with_colsum(a, dY, w.colsum_splits == 1 ? dbias : cpart, (int)tokens,
                                           (int)out, w.colsum_splits, w.colsum_rows, hs);
    else
      e = launch_gemm_bf16(GEMM_NN_F32, w.tile, a, hs);
  } else {
    e = s.dtype == SK_BF16 ? launch_gemm_bf16(GEMM_NN_F32_COLSUM, w.tile, a, hs)
                           : launch_gemm_f32(GEMM_TN_F32, w.tile, a, hs);
  }
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight (Z^T.dY)");
  if (w.head_cols > 0) {
    e = launch_reduce_splits_2d(part, dU_cat + w.head_cols, s.R, (int)out - w.head_cols, out, w.splits,
                                scale, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight (sum of the split columns)");
  }
  const bool sum_dU = w.splits > 1 && w.head_cols == 0;
  const bool sum_db = dbias && w.colsum_splits > 1;
  if (sum_dU || sum_db) {
    ReduceArgs r{};
    r.part = part; r.out = dU_cat; r.n = sum_dU ? (int64_t)s.R * out : 0; r.scale = scale;
    r.part2 = cpart; r.out2 = dbias; r.n2 = sum_db ? out : 0; r.scale2 = 1.0f;
    r.splits = w.splits; r.splits2 = w.colsum_splits;
    e = launch_reduce_splits(r, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight (sum of splits)");
  }
  return SK_OK;
}

sk_status sk_linear_bwd_weight_noalloc(const void* x, const void* S_cat, const void* dY,
                                       float* dU_cat, float* dbias, int64_t tokens, int64_t in,
                                       int64_t out, int32_t l, int32_t k, sk_dtype dtype,
                                       void* stream) {
  // everything sk_linear_bwd_weight would reject is rejected here first, before any HIP call
  if (!x || !S_cat || !dY || !dU_cat) return SK_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(S_cat) || !aligned16(dY) || !aligned16(dU_cat) || !aligned16(dbias))
    return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  if (workspace_for(SK_OP_BWD_WEIGHT, s) > SK_NOALLOC_SCRATCH_BYTES) return SK_ERR_WORKSPACE;
  // the address of this GPU's copy of the array, looked up once per device
  constexpr int MAX_DEVICES = 64;
  static std::atomic<void*> device_scratch[MAX_DEVICES];
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight_noalloc (hipGetDevice)");
  if (dev < 0 || dev >= MAX_DEVICES) return SK_ERR_UNSUPPORTED;
  void* ptr = device_scratch[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr)
      return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol,
                      "sk_linear_bwd_weight_noalloc (hipGetSymbolAddress)");
    device_scratch[dev].store(ptr, std::memory_order_release);
  }
  // Every region of the workspace is written by the call before it is read (Z^T with its
  // zero-filled row padding, the split slabs, the column-sum partials), so what an earlier
  // call left in the array needs no clearing.
  return sk_linear_bwd_weight(x, S_cat, dY, dU_cat, dbias, tokens, in, out, l, k, dtype, ptr,
                              SK_NOALLOC_SCRATCH_BYTES, stream);
}

static sk_status bwd_both(const void* x, const void* dY, const void* S_cat, const void* U_cat, void* dX, float* dU_cat,
                          float* dbias, int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k, sk_dtype dtype,
                          void* workspace, size_t workspace_bytes, void* stream, GColumns* want, Unrounded* later) {
  if (!x || !dY || !S_cat || !U_cat || !dX || !dU_cat) return SK_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(dY) || !aligned16(S_cat) || !aligned16(U_cat) || !aligned16(dX) ||
      !aligned16(dU_cat) || !aligned16(dbias) || !aligned16(workspace))
    return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  const size_t in_bytes = workspace_for(SK_OP_BWD_INPUT, s);
  const size_t w_bytes = workspace_for(SK_OP_BWD_WEIGHT, s);
  if (!workspace || workspace_bytes < workspace_for(SK_OP_BWD, s)) return SK_ERR_WORKSPACE;
  unsigned char* ws_in = static_cast<unsigned char*>(workspace);
  unsigned char* ws_w = ws_in + in_bytes;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const float scale = 1.0f / (float)l;

  // --- fp32: dY.U^T beside x.S | sums of their slabs | Z^T.dY beside G.S^T | sums of the token splits ---
  // A partner by itself leaves the chip idle ([4096 x 768] . U^T, R = 128, is 128 work-groups of 24
  // chunks: 17 us) or is over in a launch's own time (64 tokens, 256 -> 256, R = 16: six launches of one
  // to four work-groups).  The same tiles and ranges as the separate calls, so the same results.
  // Backward pass, us, apart : shared: 60 tokens, 112 -> 176, R = 64, 18.8 : 11.0; 811, 1888 -> 1840, R = 32,
  // 34.5 : 25.9; 4096, 3072 -> 768, R = 128, 95 : 84; 1475, 1312 -> 288, R = 304, 51.7 : 45.0.
  if (s.dtype == SK_F32) return bwd_f32(s, x, dY, S_cat, U_cat, dX, dU_cat, dbias, ws_in, ws_w, want, hs);

  // Shared-launch schedules exist for the shapes the automatic plans produce on the
  // benchmark configurations (bf16; the dual kernel is built for a few tile pairs only);
  // everything else runs the two gradients one after the other.
  const WeightPlan w = plan_weight(s);
  const bool bf16_any_z = s.dtype == SK_BF16 && g_plan.load(std::memory_order_relaxed) == PLAN_AUTO && !w.own_colsum;
  // (Z^T recomputed in ranges over a long input: a schedule of its own, for narrow sketches)
  const bool bf16_auto = bf16_any_z && w.z_splits == 1;
  const Plan in_plan = pick_plan(s, SK_OP_BWD_INPUT, true);
  int z_tile = bf16_auto ? choose_tile(s.R, tokens, in, 1) : -1;
  const GemmKind du_kind = GEMM_NN_F32_COLSUM;

  void* Z = ws_w;
  float* part = reinterpret_cast<float*>(ws_w + w.z_bytes);
  float* cpart = reinterpret_cast<float*>(ws_w + w.z_bytes + w.part_bytes);
  // Z^T = S_cat^T . x^T (zero-filled row padding)
  GemmArgs z = dense_args(S_cat, s.R, x, in, Z, w.ldz, s.R, tokens, in, 1.0f, nullptr);
  z.n_store = (int)w.ldz;
  // dU (or its slabs) = Z^T . dY with the column sums of dY, the token axis split in order
  GemmArgs du{};
  du.A = Z; du.lda = w.ldz;
  du.B = dY; du.ldb = out; du.ldc = out;
  du.M = s.R; du.N = (int)out; du.K = (int)tokens;
  du.splits = w.splits; du.k_per_split = w.k_per_split;
  if (w.splits == 1) { du.C = dU_cat; du.colsum = dbias; du.scale = scale; }
  else { du.C = part; du.colsum = dbias ? cpart : nullptr; du.scale = 1.0f; }
  ReduceArgs red{};
  red.part = part; red.out = dU_cat; red.n = w.splits > 1 ? (int64_t)s.R * out : 0; red.scale = scale;
  red.part2 = cpart; red.out2 = dbias; red.n2 = (dbias && w.colsum_splits > 1) ? out : 0; red.scale2 = 1.0f;
  red.splits = w.splits; red.splits2 = w.colsum_splits;
  // the sums behind everything else: in a launch of their own, or left to the one that rounds them
  auto last_sums = [&]() -> hipError_t {
    if (!later) return launch_reduce_splits(red, hs);
    if (red.n > 0) later->du = {red.part, red.n, red.splits, red.scale};
    if (red.n2 > 0) later->db = {red.part2, red.n2, red.splits2, red.scale2};
    return hipSuccess;
  };

  // --- narrow sketch: split-K slabs of G beside Z^T | Z^T.dY beside the expansion of dX | sums, or, where the expansion's
  // runs are long, Z^T.dY | expand dX, carrying the sums ---
  // (Z^T in ranges: their slabs, and one more launch that sums them, four launches instead of six: 4096 tokens, 8192 -> 8192, R = 16
  // 68.1 : 62.5 us, 1024 41.5 : 30.8; 2048, 4096 -> 4096, R = 64 39.2 : 33.3; 3000, 6000 -> 7008, R = 96 78.8 : 65.7)
  // Not where dX by itself is one fused launch that nearly fills the chip while the slabs of G are large: from 9600 tokens on, R > 64
  // (13476 tokens, 2400 -> 336, R = 112 75.4 us here, one after the other 63.2; 15303, 5600 -> 416, R = 128 158.8 : 128.8; 30 layers of
  // 9934 to 15489 tokens 0.98 to 1.23 times the time, below that 0.84 to 1.11, and 0.97 at the median).
  const SketchPlan q = plan_sketch(s, out);
  const bool z_ranges = bf16_any_z && w.z_splits > 1 && !(in_plan == PLAN_FUSED && s.R > 64 && tokens > 9600);
  ChainArgs c{};
  c.A = dY; c.B1 = U_cat; c.B2 = S_cat; c.bias = nullptr; c.C = dX;
  c.lda = out; c.ldb1 = out; c.ldb2 = s.R; c.ldc = in;
  c.M = (int)tokens; c.K1 = (int)out; c.R = s.R; c.N = (int)in; c.scale = scale;
  { const ChainShape cs = chain_shape(tokens, in, s.R, z_ranges); c.n_slices = cs.slices; c.bm = cs.bm; }
  c.Z = ws_in; c.z_splits = q.splits; c.z_slab = (int64_t)tokens * s.R;
  // Z^T.dY shares a launch with the expansion where that is over soon (launch_factor_beside_expand), also in one range
  // of tokens: two launches, where one after the other the gradients take three or four (62 of 150 layers of 100 to 600 tokens,
  // 64 to 4096 wide, take it, in 0.61 of the time; 570 tokens, 320 -> 1808, R = 32 19.7 : 10.3 us; 164 of 250 layers of 1 to 99 tokens, 0.72 (0.57 to 0.98),
  // 60, 512 -> 1696, R = 48 17.0 : 9.8 against the few-rows kernel; x.S in ranges, 418, 3616 -> 272, R = 80 21.0 : 15.7, 80 layers of 9 to 320
  // tokens 0.80 to 0.84, 34, 3696 -> 1248, R = 112 20.1 : 16.2).
  bool beside = bf16_any_z && factor_beside_expand_supported(w.tile, du, c);
  if (!beside && z_ranges && (in <= 2 * out || tokens <= 2048)) {
    // An expansion of two work-groups a CU with one instead, to leave room: not where dX is most of what moves (5505 tokens, 3600 -> 272, R = 48
    // 38.6 : 41.3 us, 9664, 3024 -> 320, R = 32 48.6 : 51.8, 6520, 2432 -> 976, R = 16 37.3 : 38.0; 1198, 3248 -> 752, R = 64 21.5 : 19.8).
    ChainArgs fewer = c;
    fewer.n_slices = chain_shape(tokens, in, s.R, false).slices;
    if (factor_beside_expand_supported(w.tile, du, fewer)) { beside = true; c = fewer; }
  }
  // --- narrow sketch, short input: one pass over x and dY | sum of the token tiles' slabs ---
  // Not, by itself, where the two gradients share launches (below) up to 4095 tokens.  One pass : shared, backward call, us: 255 tokens,
  // 304 -> 752, R = 16 14.0 : 8.4; 1024, 768 -> 768, R = 32 15.7 : 13.3; 2411, 768 -> 992, R = 16 18.7 : 15.9.  Of 200 layers (200 to 16384 tokens, 64 to
  // 1024 outputs) 115 can share: 0.60 to 0.97 of the time up to 4095 tokens (mean 0.81).
  // Beyond, the ranges of tokens are much longer than the one pass's 32 or 64 and db's sums further from 64 bits: 1.15 times its 4.7e-8 from 4096 to 8191, 1.26 times its 6.1e-8 up to
  // 16384 (1.00 to 1.05 below; dU and dX 1.00 everywhere; 90 layers), so the one pass stays there, though of 160 layers that can share 126 with more outputs than inputs would take 0.80 to
  // 1.01 of the time (mean 0.92, one at 1.05), 34 others 0.91 to 1.09 (mean 1.01); none of the other 85 (outputs up to 240) is faster without this pass (1.08 to 1.41).
  const bool shares = beside && !z_ranges && tokens < 4096 && tune(SK_TUNE_NARROW_BWD) < 0 && q.splits > 1 &&
                      dual_gemm_supported(GEMM_NT_F32, q.tile, GEMM_TT, z_tile);
  if (const NarrowPlan n = plan_narrow(s); n.ok && !shares) {
    g_hip_error.clear();
    NarrowBwdArgs b{};
    b.x = x; b.S = S_cat; b.dY = dY; b.U = U_cat; b.dX = dX;
    b.du_slabs = reinterpret_cast<float*>(ws_in);
    b.db_slabs = dbias ? reinterpret_cast<float*>(ws_in + n.du_bytes) : nullptr;
    b.M = (int)tokens; b.K1 = (int)in; b.R = s.R; b.N = (int)out; b.scale = scale; b.tm = n.tm;
    hipError_t e = launch_bwd_narrow_bf16(b, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (one pass over x and dY)");
    ReduceArgs t{};
    t.part = b.du_slabs; t.out = dU_cat; t.n = (int64_t)s.R * out; t.splits = n.tiles_m; t.scale = scale;
    t.part2 = b.db_slabs; t.out2 = dbias; t.n2 = dbias ? out : 0; t.splits2 = n.tiles_m; t.scale2 = 1.0f;
    e = launch_reduce_tiles(t, hs);
    return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_bwd (sum of the token tiles)");
  }

  if (bf16_any_z && chain_supported(s.R) && s.R <= 128 && q.splits > 1 && (z_ranges || (w.z_splits == 1 && (w.splits > 1 || beside))) &&
      (z_ranges ? dual_gemm_supported(GEMM_NT_F32, q.tile, GEMM_TT_F32, w.z_tile) : dual_gemm_supported(GEMM_NT_F32, q.tile, GEMM_TT, z_tile))) {
    g_hip_error.clear();
    GemmArgs g = dense_args(dY, out, U_cat, out, ws_in, s.R, tokens, s.R, out, 1.0f, nullptr);
    g.splits = q.splits; g.k_per_split = q.k_per_split;
    float* const zpart = reinterpret_cast<float*>(ws_w + w.zpart_at());
    if (z_ranges) { z.C = zpart; z.splits = w.z_splits; z.k_per_split = w.z_k_per_split; }
    hipError_t e = z_ranges ? launch_dual_gemm_bf16(GEMM_NT_F32, q.tile, g, GEMM_TT_F32, w.z_tile, z, hs)
                            : launch_dual_gemm_bf16(GEMM_NT_F32, q.tile, g, GEMM_TT, z_tile, z, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (dY.U^T beside x.S)");
    if (z_ranges) {
      e = launch_reduce_to_bf16(zpart, Z, (int64_t)s.R * w.ldz, w.z_splits, hs);
      if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (sum of x.S)");
    }
    if (want) {
      c.z_out = want->room; c.z_first = (int)want->first;
      want->at = want->room; want->ld = s.R - want->first;
    }
    if (beside) {
      e = launch_factor_beside_expand(w.tile, du, c, hs);
      if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (Z^T.dY beside the expansion)");
      e = last_sums();
      return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_bwd (sum of splits)");
    }
    // Z^T.dY, then the expansion of dX carrying the sum of the token splits
    e = launch_gemm_bf16(du_kind, w.tile, du, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (Z^T.dY)");
    c.tail = red;
    e = launch_chain_bf16(true, false, c, hs);
    return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_bwd (expand + sum of splits)");
  }

  // --- wide sketch (two GEMMs per gradient): dY.U^T beside Z^T | sums of their ranges | Z^T.dY beside G.S^T | sums ---
  int g_tile = bf16_auto ? choose_tile(tokens, s.R, out, 1) : -1;
  // Nor do the first two share a launch on that tile: where it is faster by itself they go beside each
  // other on 128 x 128 tiles unless the two launches are modelled 3 us ahead, which sorts all of 20 shapes
  // measured ([12288 x 768 -> 768], R = 768, 89 us shared : 103; [33222 x 208 -> 48], R = 544, 71 : 82;
  // [12288 x 4096 -> 1024], R = 1024, 306 : 266; [32768 x 1024 -> 1024], R = 512, 187 : 171, R = 384, 147 : 150).
  auto square = [](int t) { return t == TILE_256x256 || t == TILE_128x128; };
  if (square(g_tile) && square(z_tile) && g_tile + z_tile != 2 * TILE_128x128) {
    auto alone = [&](int t, int64_t M, int64_t N, double k) {
      return t == TILE_256x256 ? big_tiles_us(M, N, k, 1) : small_tiles_us(small_tiles(M, N), k);
    };
    const double apart = alone(g_tile, tokens, s.R, (double)out) + alone(z_tile, s.R, tokens, (double)in);
    if (apart + 3.0 > small_tiles_us(2 * small_tiles(tokens, s.R), 0.5 * (double)(in + out)))
      g_tile = z_tile = TILE_128x128;
  }
  int dx_tile = bf16_auto ? choose_tile(tokens, in, s.R, 1) : -1;
  // beside Z^T.dY the expansion of dX runs on 128 x 128 tiles even where it would take the
  // 256 x 256 tile on its own: that one takes all of a CU's LDS and leaves no room to share.  Shared
  // against one after the other, us per backward call: [8192 x 3072 -> 4096], R = 768, 218 : 235;
  // [16384 x 1024 -> 4096], R = 144, 103 : 112; [16384 x 4096 -> 4096], R = 512, level; the
  // best the separate launches did was 2 % ahead ([8192 x 4096 -> 8192], R = 1024, 478 : 468)
  if (dx_tile == TILE_256x256) dx_tile = TILE_128x128;
  WidePlan pair{-1, 1, 0, 0, 0};
  const FirstPlan first = plan_first(GEMM_NT, tokens, s.R, out);
  if (bf16_any_z && in_plan == PLAN_TWO_GEMM && !first.few) {
    pair = plan_wide(s, w, first);
    if (pair.tile < 0 && w.z_splits == 1 && first.splits == 1 && g_tile == z_tile && dual_gemm_supported(GEMM_NT, g_tile, GEMM_TT, z_tile) &&
        dual_gemm_supported(du_kind, w.tile, GEMM_NT, dx_tile))
      pair = WidePlan{g_tile, 1, 0, w.tile, dx_tile};
  }
  if (pair.tile >= 0) {
    g_hip_error.clear();
    // (slabs behind G, and where a split Z has them)
    void* const g_slabs = ws_in + align_up((size_t)tokens * s.R * s.esize);
    float* const z_slabs = reinterpret_cast<float*>(ws_w + w.zpart_at());
    GemmArgs g = dense_args(dY, out, U_cat, out, ws_in, s.R, tokens, s.R, out, 1.0f, nullptr);
    RoundedSum g_sum{}, z_sum{};
    if (pair.g_splits > 1) {
      g.C = g_slabs; g.splits = pair.g_splits; g.k_per_split = pair.g_k_per_split;
      g_sum = RoundedSum{static_cast<const float*>(g_slabs), ws_in, (int64_t)tokens * s.R, g.splits};
    }
    if (w.z_splits > 1) {
      z.C = z_slabs; z.splits = w.z_splits; z.k_per_split = w.z_k_per_split;
      z_sum = RoundedSum{z_slabs, Z, (int64_t)s.R * w.ldz, z.splits};
    }
    hipError_t e = launch_dual_gemm_bf16(g.splits > 1 ? GEMM_NT_F32 : GEMM_NT, pair.tile, g, z.splits > 1 ? GEMM_TT_F32 : GEMM_TT, pair.tile, z, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (dY.U^T beside x.S)");
    e = launch_reduce_to_bf16(g_sum, z_sum, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (sums of dY.U^T and x.S)");
    if (want) want->take(ws_in, s);
    const GemmArgs dx = dense_args(ws_in, s.R, S_cat, s.R, dX, in, tokens, in, s.R, scale, nullptr);
    e = launch_dual_gemm_bf16(du_kind, pair.du_tile, du, GEMM_NT, pair.dx_tile, dx, hs);
    if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd (Z^T.dY beside G.S^T)");
    e = last_sums();
    return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_bwd (sum of splits)");
  }

  const sk_status a = sk_linear_bwd_input(dY, S_cat, U_cat, dX, tokens, in, out, l, k, dtype, ws_in,
                                          in_bytes, stream);
  if (a != SK_OK) return a;
  if (want && in_plan == PLAN_TWO_GEMM) want->take(ws_in, s);
  return sk_linear_bwd_weight(x, S_cat, dY, dU_cat, dbias, tokens, in, out, l, k, dtype, ws_w, w_bytes,
                              stream);
}

sk_status sk_linear_bwd(const void* x, const void* dY, const void* S_cat, const void* U_cat,
                        void* dX, float* dU_cat, float* dbias, int64_t tokens, int64_t in,
                        int64_t out, int32_t l, int32_t k, sk_dtype dtype, void* workspace,
                        size_t workspace_bytes, void* stream) {
  return bwd_both(x, dY, S_cat, U_cat, dX, dU_cat, dbias, tokens, in, out, l, k, dtype, workspace, workspace_bytes, stream, nullptr, nullptr);
}

sk_status sk_linear_bwd_weight_first(const void* x, const void* U_cat, const void* dY, float* dA,
                                     int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k,
                                     int64_t col_begin, int64_t col_count, sk_dtype dtype,
                                     void* workspace, size_t workspace_bytes, void* stream) {
  if (!x || !U_cat || !dY || !dA) return SK_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(U_cat) || !aligned16(dY) || !aligned16(dA) || !aligned16(workspace))
    return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  if (col_begin < 0 || col_count < 16 || col_begin % 16 != 0 || col_count % 16 != 0 ||
      col_begin + col_count > s.R)
    return SK_ERR_INVALID_ARG;
  const int64_t nc = col_count;
  if (!workspace || workspace_bytes < first_stage_bytes(s, nc)) return SK_ERR_WORKSPACE;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const float scale = 1.0f / (float)l;
  g_hip_error.clear();

  unsigned char* ws = static_cast<unsigned char*>(workspace);
  void* G = ws;
  float* part = reinterpret_cast<float*>(ws + align_up((size_t)s.T * nc * s.esize));
  const unsigned char* U_sub = static_cast<const unsigned char*>(U_cat) + (size_t)col_begin * out * s.esize;

  // G = dY . U_sub^T, rounded to the storage type like the input gradient's intermediate
  hipError_t e = first_gemm(s, GEMM_NT, GEMM_NT_F32,
                            dense_args(dY, out, U_sub, out, G, nc, tokens, nc, out, 1.0f, nullptr), part, hs);
  if (e != hipSuccess) return hip_fail(e, "sk_linear_bwd_weight_first (dY.U^T)");

  return first_stage_gradient(s, x, G, nc, nc, dA, part, hs);
}

static sk_status bwd_two_sided(const void* x, const void* dY, const void* S_cat, const void* U_cat, void* dX, float* dU_cat, float* dbias, float* dA,
                               int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k, sk_dtype dtype, void* workspace, size_t workspace_bytes,
                               void* stream, Unrounded* later) {
  if (!dA || !aligned16(dA) || !workspace || !aligned16(workspace)) return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  if (s.R % 32 != 0) return SK_ERR_UNSUPPORTED;   // (halves of a multiple of 16 columns)
  if (workspace_bytes < workspace_for(SK_OP_BWD_TWO_SIDED, s)) return SK_ERR_WORKSPACE;
  const int64_t half = s.R / 2;
  unsigned char* const ws = static_cast<unsigned char*>(workspace);
  const size_t both = workspace_for(SK_OP_BWD, s), room = align_up((size_t)s.T * half * s.esize);
  GColumns want{half, ws + both, nullptr, 0};
  const sk_status a = bwd_both(x, dY, S_cat, U_cat, dX, dU_cat, dbias, tokens, in, out, l, k, dtype, workspace, both, stream, &want, later);
  if (a != SK_OK) return a;
  if (want.at == nullptr)
    return sk_linear_bwd_weight_first(x, U_cat, dY, dA, tokens, in, out, l, k, half, half, dtype, ws + both, workspace_bytes - both, stream);
  return first_stage_gradient(s, x, want.at, want.ld, half, dA, reinterpret_cast<float*>(ws + both + room), static_cast<hipStream_t>(stream), later);
}

sk_status sk_linear_bwd_two_sided(const void* x, const void* dY, const void* S_cat, const void* U_cat, void* dX, float* dU_cat, float* dbias,
                                  float* dA, int64_t tokens, int64_t in, int64_t out, int32_t l, int32_t k, sk_dtype dtype,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  return bwd_two_sided(x, dY, S_cat, U_cat, dX, dU_cat, dbias, dA, tokens, in, out, l, k, dtype, workspace, workspace_bytes, stream, nullptr);
}

sk_status sk_linear_bwd_rounded(const void* x, const void* dY, const void* S_cat, const void* U_cat, void* dX, float* dU_cat, float* dbias, float* dA,
                                void* dU_bf16, int64_t dU_rows, void* dbias_bf16, void* dA_bf16, int64_t tokens, int64_t in, int64_t out, int32_t l,
                                int32_t k, sk_dtype dtype, void* workspace, size_t workspace_bytes, void* stream) {
  if ((!dU_bf16 && !dbias_bf16 && !dA_bf16) || !aligned16(dU_bf16) || !aligned16(dbias_bf16) || !aligned16(dA_bf16)) return SK_ERR_INVALID_ARG;
  if ((dbias_bf16 && !dbias) || (dA_bf16 != nullptr) != (dA != nullptr)) return SK_ERR_INVALID_ARG;
  Shape s;
  const sk_status st = check_shape(tokens, in, out, l, k, dtype, s);
  if (st != SK_OK) return st;
  if (dtype != SK_BF16) return SK_ERR_UNSUPPORTED;
  if (dU_bf16 && (dU_rows < 1 || dU_rows > s.R)) return SK_ERR_INVALID_ARG;
  Unrounded u{{dU_cat, 0, 1, 1.0f}, {dbias, 0, 1, 1.0f}, {dA, 0, 1, 1.0f}};
  const sk_status a = dA ? bwd_two_sided(x, dY, S_cat, U_cat, dX, dU_cat, dbias, dA, tokens, in, out, l, k, dtype, workspace, workspace_bytes, stream, &u)
                         : bwd_both(x, dY, S_cat, U_cat, dX, dU_cat, dbias, tokens, in, out, l, k, dtype, workspace, workspace_bytes, stream, nullptr, &u);
  if (a != SK_OK) return a;
  RoundArgs r{};
  int count = 0;
  auto add = [&](const Unrounded::Part& part, void* to, int64_t n) {
    if (!to) return;
    r.from[count] = part.at; r.to[count] = static_cast<unsigned short*>(to); r.n[count] = n;
    r.stride[count] = part.splits > 1 ? part.stride : n; r.splits[count] = part.splits; r.scale[count] = part.scale;
    ++count;
  };
  add(u.du, dU_bf16, dU_rows * out);
  add(u.db, dbias_bf16, out);
  add(u.da, dA_bf16, in * (s.R / 2));
  const hipError_t e = launch_round_gradients(r, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? SK_OK : hip_fail(e, "sk_linear_bwd_rounded (sums and rounding)");
}

sk_status sk_round_gradients(const float* const* from, void* const* to, const int64_t* n, int32_t count, void* stream) {
  if (!from || !to || !n || count < 1 || count > RoundArgs::MAX) return SK_ERR_INVALID_ARG;
  RoundArgs a{};
  for (int i = 0; i < count; ++i) {
    if (!from[i] || !to[i] || !aligned16(from[i]) || !aligned16(to[i]) || n[i] < 1) return SK_ERR_INVALID_ARG;
    a.from[i] = from[i]; a.to[i] = static_cast<unsigned short*>(to[i]); a.n[i] = a.stride[i] = n[i];
    a.splits[i] = 1; a.scale[i] = 1.0f;
  }
  g_hip_error.clear();
  const hipError_t e = launch_round_gradients(a, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? SK_OK : hip_fail(e, "sk_round_gradients");
}

}  // extern "C"
