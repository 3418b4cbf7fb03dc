// Launch plan and launchers of the integer GEMM (kernel in igemm_kernel.h) and the code
// unpacker used by the parity views.
#include <atomic>
#include <chrono>

#include "hot_host.h"
#include "igemm_kernel.h"

namespace hot {

__global__ void unpack_kernel(const uint8_t* __restrict__ codes, int64_t rows, int64_t K,
                              int64_t pitch, int bits, int transpose, int8_t* __restrict__ out) {
  const int64_t total = rows * K;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = i / K, k = i - row * K;
    if (bits == 16) {   // two-byte elements (bfloat16 patterns) in, two-byte elements out
      reinterpret_cast<uint16_t*>(out)[transpose ? k * rows + row : i] =
          *reinterpret_cast<const uint16_t*>(codes + row * pitch + 2 * k);
      continue;
    }
    int c;
    if (bits == 4) {
      const int byte = codes[row * pitch + (k >> 1)];
      const int nib = (k & 1) ? (byte >> 4) : (byte & 0xF);
      c = (nib ^ 8) - 8;  // sign-extend 4 bits
    } else {
      c = (int8_t)codes[row * pitch + k];
    }
    out[transpose ? k * rows + row : i] = (int8_t)c;
  }
}

hipError_t launch_unpack(const uint8_t* codes, int64_t rows, int64_t K, int64_t pitch, int bits,
                         int transpose, int8_t* out, hipStream_t s) {
  if (rows <= 0 || K <= 0) return hipSuccess;
  int64_t blocks = ceil_div(rows * K, 256);
  if (blocks > 65536) blocks = 65536;
  unpack_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(codes, rows, K, pitch, bits, transpose, out);
  return hipGetLastError();
}

// Tile configurations.  Four workgroup tiles exist for INT4 operands: 128x128 (64x64 per
// wave, three workgroups per compute unit: prologue, matrix loop and epilogue of different
// workgroups overlap, but the INT4 widening costs 6 vector instructions per matrix
// instruction), 128x256 (64x128 per wave, two workgroups per unit), 192x256 and 256x256 (96x128
// / 128x128 per wave, one workgroup per unit: half the widening and LDS traffic per matrix
// instruction, but prologue (3 us) and epilogue (3 us of instructions, or the tile's bytes at
// the unit's share of the memory bandwidth when every unit stores at once) are exposed, and a
// partial last round idles units).  INT8 and bfloat16 operands (twice and four times the
// bytes per operation) take 128x128, whose LDS traffic (1 KB per matrix instruction) is its
// limit, or 256x256 with eight waves (64x128 per wave), and 128-byte K stages.  The choice
// minimises the cost model in plan_gemm.  A GEMM with a small output and a long K (the g_w
// path of ViT-sized layers) leaves most units idle with one workgroup per tile: its K range
// is split over several workgroups per tile, which hand their partial sums to the last one
// through the workspace.
namespace {
std::atomic<int> g_gemm_mode{0};   // 0: cost model, 1: never split K, s >= 2: s slices where possible
std::atomic<int> g_gemm_wait_us{200};

// Compute units the launch plans are made for: those of the MI355X.  A constant rather than
// a device query, so that workspace sizes are a function of the configuration and the shape
// alone; on a part with fewer units the plans stay correct (every wait for another workgroup is
// bounded), only less well fitted.
constexpr int kPlanComputeUnits = 256;
int compute_units() { return kPlanComputeUnits; }

// Most slices a 128x128-tile GEMM may be cut into: at least 4 K stages per slice, and no more
// image slots than the workspace has flags for.
int64_t max_split(int64_t tiles, int64_t nk) {
  int64_t s = nk / 4;
  if (s > 8) s = 8;
  while (s > 1 && tiles * (s - 1) > kMaxSplitSlots) --s;
  return s < 1 ? 1 : s;
}
// K split of the 256x256 INT8 tile (eight waves, one workgroup per compute unit) for an output
// of at most one such tile per unit: as many slices as there are units per tile, and only when
// a slice keeps at least 16 KB of K, so that the 256 KB accumulator images the owner collects
// are a small part of the work.  0: does not apply.  Chosen against 128x128 tiles by cost (plan_gemm).
int64_t large_tile_split(int64_t M, int64_t N, int64_t k_bytes, int bits, int cus) {
  if (bits != 8) return 0;
  const int64_t tiles = ceil_div(M, 256) * ceil_div(N, 256);
  if (tiles > cus) return 0;
  int64_t s = cus / tiles;
  if (s > 8) s = 8;
  while (s > 1 && (k_bytes / s < 16384 || tiles * (s - 1) > kMaxSplitSlots)) --s;
  return s >= 2 ? s : 0;
}
// Time of a hand-over split of 128x128 tiles in us but for what does not depend on the split: the
// stages of a slice, at another rate while no unit has two workgroups, and the hand-over (the flags, the
// images an owner adds, and the images' traffic when all units write and read them).  Fitted to g_w and
// g_x GEMMs of 1200 layers, every split from 1 to 8 timed on each (512 to 200000 tokens, 43 to 512
// tiles, 8 to 800 stages); the split chosen by it takes 0.7-1.3 % longer than the best one on average.  As many
// slices as keep all workgroups resident, the rule before, took 17-31 % longer: 9840 tokens 832 x 1184 (70
// tiles, 39 stages) 34 us in 3 slices, 38 in 7; g_x of 1005 tokens 1024 x 2544 in INT8 12 us whole, 21 in 2;
// 64 tiles x 96 stages 28 us in 3, 44 in 8.
struct SplitCost { double stage, stage_two, split, slice, resident; };
constexpr SplitCost kSplit4{0.48, 0.69, 3.0, 0.84, 6.5};
constexpr SplitCost kSplit8{0.54, 0.92, 2.3, 1.0, 5.0};
double split_us(const SplitCost& c, int64_t tiles, int64_t stages, int64_t s, int cus) {
  const int64_t wgs = tiles * s;
  const double t = (double)ceil_div(stages, s) * (wgs <= cus ? c.stage : c.stage_two);
  return s == 1 ? t : t + c.split + c.slice * (double)(s - 1) + c.resident * (double)wgs / (2.0 * cus);
}
int64_t best_split(const SplitCost& c, int64_t tiles, int64_t stages, int64_t most, int cus) {
  int64_t best = 1;
  for (int64_t s = 2; s <= most && tiles * s <= 2 * (int64_t)cus; ++s)
    if (split_us(c, tiles, stages, s, cus) < split_us(c, tiles, stages, best, cus)) best = s;
  return best;
}
// The same for 256x256 INT8 tiles in `s` slices (260 layers): 110224 tokens 512 x 4416 (140 tiles of
// 128x128) 198 us in 3 slices on the large tile, 164 in 3 on the small one (205 in 4, beyond the resident
// count); 112928 x 1536 x 1952 204 in 3 slices and 237.
double large_split_us(int64_t stages, int64_t s) { return 1.25 * (double)ceil_div(stages, s) + 6.75 * (double)(s - 1) - 8.1; }
// Cost of a tile shape, fitted to measurements on MI355X: a compute unit works through its share of
// the tiles, each costing its operations at the rate the tile sustains plus its output bytes
// at the rate its stores drain, plus a constant per launch.  The share is a whole number of
// tiles while the resident workgroups (wgs per unit) take them in a few rounds, the last of
// which idles units, and averages out over many rounds.
struct Cand { int bm, bn, wgs; double us_per_mop, us_per_kb, us_launch; };
// The INT4 constants are fitted to 414 layers of 512 to 200000 tokens and 64 to 11008 outputs and inputs, all four
// tiles timed on each: the choice takes 0.9 % longer than the best tile on average (2.6 % with constants
// from ten layers, 36 % at worst: 35372 tokens 1152 x 576 35.1 us, 39.0 on 128x256 tiles).
constexpr Cand kCands4[] = {{128, 128, 3, 0.0978, 0.0289, 4.6}, {128, 256, 2, 0.0882, 0.0291, 3.3},
                            {192, 256, 1, 0.0910, 0.0405, 3.8}, {256, 256, 1, 0.0827, 0.0431, 2.3}};
constexpr Cand kCands8[] = {{128, 128, 2, 0.2560, 0.0, 0.0}, {256, 256, 1, 0.1004, 0.0476, 0.0}};
double tile_mops(const Cand& c, double K) { return 2.0 * c.bm * c.bn * K * 1e-6; }
double tile_shape_us(const Cand& c, int64_t M, int64_t N, double K, int cus) {
  const int64_t tiles = ceil_div(M, c.bm) * ceil_div(N, c.bn);
  const bool few_rounds = tiles <= 4 * (int64_t)cus * c.wgs;
  const double per_cu = few_rounds ? (double)ceil_div(tiles, cus) : (double)tiles / cus;
  const double kb = 4.0 * c.bm * c.bn / 1024.0;
  return per_cu * (tile_mops(c, K) * c.us_per_mop + kb * c.us_per_kb) + c.us_launch;
}
// Slices of a GEMM on 128x128 tiles whose partial sums a second kernel adds (kImages); 0 = does
// not apply.  A slice costs about 0.5 us per 128-byte K stage, an image 0.03 us to write and
// read back, so the sum of both is least at sqrt(16 stages / tiles) slices, with about two
// workgroups per compute unit and four stages a slice at most; counts above 8 are rounded to a
// multiple of 8, which lets an XCD keep whole slices and may pass those two by a little (16 slices
// of three stages for 4 tiles x 49, 576 workgroups for 36 x 788; 8 slices took 12.0 and 101.2).  Measured,
// best of 1-24 slices against this rule's: 4 tiles x 49 stages 12.0 / 12.4 us (the hand-over 22.8),
// 16 x 32 13.5 / 14.3 (21.6), 32 x 49 16.3 / 16.9 (25.8), 36 x 788 97.1 / 99.9 (the hand-over on
// 256x256 tiles 197), bfloat16 36 x 99 24.4 / 24.5 (unsplit 52.8), 144 x 99 52.8 / 52.8 (56.9).
// INT8 GEMMs of more than 42 tiles stay with the hand-over, which hides the images under the last
// slices' work: 56 tiles x 12 stages 16.0 against 15.9 us, 144 x 50 31.1 against 36.4, 108 x 197
// 71 against 76.  bfloat16 has no hand-over: any output with no more tiles than units, and three
// slices or more (two: 36 tiles x 16 stages 17.1 us against 14.3 unsplit).
int64_t image_slices(int64_t M, int64_t N, int64_t k_bytes, int bits, int cus) {
  if (bits == 4 || M <= 0 || N <= 0) return 0;
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128), nk = k_bytes / 128;
  if (tiles > (bits == 16 ? cus : cus / 6)) return 0;
  int64_t s = 1;
  while ((s + 1) * (s + 1) * tiles <= 16 * nk) ++s;
  if (s > 2 * cus / tiles) s = 2 * cus / tiles;
  if (s > nk / 4) s = nk / 4;
  if (s > 64) s = 64;
  if (s > 8) s = s < 12 ? 8 : (s + 4) / 8 * 8;
  return s >= (bits == 16 ? 3 : 4) ? s : 0;
}
}  // namespace

void set_gemm_mode(int mode) { g_gemm_mode.store(mode); }
void set_gemm_wait_us(int us) { g_gemm_wait_us.store(us); }

GemmPlan plan_gemm(int64_t M, int64_t N, int64_t k_bytes, int bits, bool scratch, bool images) {
  const Cand* cands = bits == 4 ? kCands4 : kCands8;
  const int ncand = bits == 4 ? 4 : 2;
  const double K = (double)k_bytes * (bits == 4 ? 2 : 1);
  const int cus = compute_units();
  GemmPlan p;
  p.split = 1;
  p.images = false;
  p.partial_bytes = 0;
  double best = 1e30;
  for (int c = 0; c < ncand; ++c) {
    const double t = tile_shape_us(cands[c], M, N, K, cus);
    if (t < best) {
      best = t;
      p.bm = cands[c].bm;
      p.bn = cands[c].bn;
      p.tiles = ceil_div(M, p.bm) * ceil_div(N, p.bn);
    }
  }
  p.bkb = bits == 4 ? 64 : 128;
  const int mode = g_gemm_mode.load();
  // fp32 sums: the slices of a bfloat16 GEMM follow from its shape alone, whatever the scratch and
  // the mode, so that its bits do too; without images one workgroup sums them in their order
  if (bits == 16) images = images && mode == 0;
  if ((images && mode == 0) || bits == 16) {
    const int64_t s = image_slices(M, N, k_bytes, bits, cus);
    if (s) {
      p.bm = p.bn = 128;
      p.tiles = ceil_div(M, 128) * ceil_div(N, 128);
      p.split = (int)s;
      p.images = images;
      if (images) p.partial_bytes = image_scratch_bytes(M, N, k_bytes, bits);
      return p;
    }
  }
  if (mode >= 10) {   // a tile forced for measurement: 10 = 128x128, 11 = 192x256 (INT4 only), 12 = 256x256
    const int bm = mode == 10 ? 128 : (mode == 11 && bits == 4 ? 192 : 256);
    p.bm = bm;
    p.bn = bm == 128 ? 128 : 256;
    if (mode == 13 && bits == 4) { p.bm = 128; p.bn = 256; }
    p.tiles = ceil_div(M, p.bm) * ceil_div(N, p.bn);
    return p;
  }
  if (bits == 16 || !scratch) return p;
  const SplitCost& cost = bits == 4 ? kSplit4 : kSplit8;
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128), nk = k_bytes / p.bkb, most = max_split(tiles, nk);
  if (mode == 0) {
    const int64_t l = large_tile_split(M, N, k_bytes, bits, cus);
    if (l) {
      p.bm = p.bn = 256;
      if (split_us(cost, tiles, nk, best_split(cost, tiles, nk, most, cus), cus) <= large_split_us(nk, l))
        p.bm = p.bn = 128;   // at most 512 tiles, of which every large one is four
      p.tiles = ceil_div(M, p.bm) * ceil_div(N, p.bn);
      if (p.bm == 256) {
        p.split = (int)l;
        p.partial_bytes = (size_t)p.tiles * (l - 1) * 256 * 256 * 4;
        return p;
      }
    }
  }
  if (p.bm == 128 && p.bn == 128 && mode != 1) {
    const int64_t s = mode >= 2 ? (mode < most ? mode : most) : best_split(cost, tiles, nk, most, cus);
    if (s >= 2) {
      p.split = (int)s;
      p.partial_bytes = (size_t)tiles * (s - 1) * 128 * 128 * 4;
    }
  }
  return p;
}

size_t image_scratch_bytes(int64_t M, int64_t N, int64_t k_bytes, int bits) {
  if (M <= 0 || N <= 0) return 0;
  return (size_t)(ceil_div(M, 128) * ceil_div(N, 128) * image_slices(M, N, k_bytes, bits, compute_units())) *
         128 * 128 * 4;
}

size_t gemm_scratch_bytes(int64_t M, int64_t N, int64_t k_bytes, int bits) {
  if (bits == 16 || M <= 0 || N <= 0) return 0;
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128);
  const int64_t s = max_split(tiles, k_bytes / (bits == 4 ? 64 : 128));
  const size_t small = (size_t)tiles * (s - 1) * 128 * 128 * 4;
  const int64_t sl = large_tile_split(M, N, k_bytes, bits, compute_units());
  const size_t large = sl ? (size_t)(ceil_div(M, 256) * ceil_div(N, 256)) * (sl - 1) * 256 * 256 * 4 : 0;
  return small > large ? small : large;
}

// Whether output stores carry the streaming hint.  Measured on MI355X: it wins for INT8 / bfloat16 operands and for
// INT4 GEMMs of up to 3072 codes of K (ViT-B fc2 at 50432 tokens 167 -> 134 us, ViT-B fc1 at 12608 tokens
// 44.5 -> 39.6 us), and loses 3 % at 4096 codes and a wide output (LLM down-projection).
// Where output rows are not whole 64-byte sectors, a sector that two stores share goes out in parts with the hint, and
// those saturate memory when many outputs follow on few K stages (11744 tokens 256 x 3079 75.8 us with it,
// 30.9 without; 4544 x 128 x 8862 70.1 and 33.2).  It pays there too
//  - for an output of the L2s' size, at any K (608 x 992 x 6570 15.5 us with it, 16.2 without); below 6 MB both
//    are the same within 1 %;
//  - where the other gradient's workgroups keep the units busy between the stores, by K and a width whose tiles
//    are under way together (16848 x 1152 x 2344 240 us a layer pass with it, 251 without; 12096 x 1088 x 4492 272 and
//    290; 5536 x 576 x 5434 too short and wide, 134 and 125);
//  - alone, where K is long and the tiles of a unit are many, so that their stores spread out (178000 x 896 x 5828 1728
//    us with it, 1493 without: too short; 26595 x 1376 x 1332 124 and 134; 9062 x 1280 x 6163 too few, 112 and 96).
// Mean loss against the better of both over such layers: 405 calls of g_x alone 0.57 % by this rule, 1.1 never,
// 8.2 always; 242 in a launch of both 0.30, 1.3, 0.63.
bool streams_out(const GemmCall& c, int64_t tiles, bool in_pair) {
  const int64_t k = c.k_bytes * (c.bits == 4 ? 2 : 1);
  if (c.bits == 4 && k > 3072) return false;
  if (c.N % 16 == 0) return true;
  const double mb = 4e-6 * (double)c.M * (double)c.N;
  if (mb <= 22.0) return mb > 6.0;
  return in_pair ? k >= 800 || (k >= 448 && c.N <= 2048) : k >= 1300 && tiles >= 6 * (int64_t)compute_units();
}

namespace {

// Waves per workgroup: 2x2, except 4x2 for the 256x256 INT8 and bfloat16 tiles.  Four waves,
// alone on their SIMDs, cannot hide the LDS traffic of those operands (two and four times the
// bytes per matrix instruction of packed INT4); eight waves of 64x128 each, two per SIMD, keep
// the whole accumulator tile in the 512 registers per lane all the same.  Measured on the
// LLM-sized g_w GEMM: INT8 320 us against 364 us (4x4 waves: 351 us), bfloat16 640 against
// 688 us; the INT4 tile and the 128x128 tiles do not gain from more waves.
template <int BM, bool INT4, bool BF16>
constexpr int gemm_waves_m() { return (BM == 256 && !INT4) ? 4 : 2; }

template <int BM, int BN, int BKB, bool INT4, bool BF16, int SPLIT>
hipError_t launch_kernel(const GemmArgs& g, unsigned grid, hipStream_t s, int gemm_stage) {
  const size_t lds = 2 * (size_t)(BM + BN) * BKB;
  constexpr int WM = gemm_waves_m<BM, INT4, BF16>();
  auto kern = igemm_kernel<BM, BN, WM, 2, BKB, INT4, BF16, SPLIT>;
  static std::atomic<bool> attr_set{false};  // per instantiation; setting it twice is harmless
  if (!attr_set.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set.store(true, std::memory_order_release);
  }
  if (gemm_stage >= 0) stage_begin(gemm_stage, s);
  kern<<<dim3(grid), dim3(64 * WM * 2), lds, s>>>(g);
  if (gemm_stage >= 0) stage_end(gemm_stage, s);
  return hipGetLastError();
}

// GemmArgs::xcd_cols of a split launch: one rectangle of the tile grid per XCD where the grid
// divides evenly, the split that fetches the fewest operand bytes (A row bands once per XCD
// column, B bands once per XCD row).
template <int BM>
int slice_placement(const GemmArgs& g, int64_t tiles) {
  if (BM == 128 && 8 % g.split == 0 && g.tiles_m % (8 / g.split) == 0) {
    // a slice per group of XCDs: the fewest operand bytes of all (ViT-B proj g_w, 36 tiles in
    // 8 slices: 50.5 -> 45 us; the 256x256 split measured slower this way, 385 against 360 us
    // on the ViT-L g_w GEMM, and keeps the rectangles)
    return -1;
  }
  if (tiles % 8 != 0) return 0;
  int cols = 0;
  double best = 0.0;
  for (int rx = 1; rx <= 8; rx *= 2) {
    const int ry = 8 / rx;
    if (g.tiles_m % ry != 0 || g.tiles_n % rx != 0) continue;
    const double fetch = (double)g.M * rx + (double)g.N * ry;
    if (cols == 0 || fetch < best) {
      best = fetch;
      cols = rx;
    }
  }
  return cols;
}

// GemmArgs' split of nk_total stages into `split` slices.
void set_slices(GemmArgs& g, int split) {
  g.split = split;
  g.slice_stages = g.nk_total / split;
  g.slice_rest = g.nk_total % split;
  g.slice_inverse = (1u << 20) / (unsigned)split + 1;   // exact for split <= 64
}

// What a hand-over launch needs beyond the tile grid: its tag, placement and bounded wait.
template <int BM>
hipError_t prepare_hand_over(GemmArgs& g, int64_t k_bytes, bool int4) {
  const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
  if (!g.partial || !g.flags || tiles * (g.split - 1) > kMaxSplitSlots) return hipErrorInvalidValue;
  g.tag = next_exchange_tag();   // the process-wide launch tag sequence
  g.xcd_cols = slice_placement<BM>(g, tiles);
  // an image normally arrives before its owner has finished its own slice; the bound only
  // has to cover workgroups that start late: never less than the whole GEMM takes at 200 TOP/s
  int64_t wait_us = g_gemm_wait_us.load();
  const int64_t gemm_us = (int64_t)(2.0 * g.M * g.N * (double)k_bytes * (int4 ? 2 : 1) / 200e6);
  if (wait_us > 0 && wait_us < gemm_us) wait_us = gemm_us;
  g.wait_ticks = wait_us < 0 ? 0 : wait_us * 100;
  return hipSuccess;
}

template <int BM, int BN, int BKB, bool INT4, bool BF16 = false>
hipError_t launch_tile(GemmArgs g, int64_t k_bytes, const GemmPlan& plan, hipStream_t s, int gemm_stage) {
  const int split = plan.split;
  g.nk_total = (int)(k_bytes / BKB);
  g.tiles_m = (int)ceil_div(g.M, BM);
  g.tiles_n = (int)ceil_div(g.N, BN);
  set_slices(g, split);
  const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
  if (split <= 1) return launch_kernel<BM, BN, BKB, INT4, BF16, kWholeK>(g, (unsigned)tiles, s, gemm_stage);
  if constexpr (BM == 128 && BN == 128 && !INT4) {
    if (plan.images) {
      if (!g.partial) return hipErrorInvalidValue;
      g.xcd_cols = split % 8 == 0 ? -2 : slice_placement<BM>(g, tiles);
      const bool timed = gemm_stage >= 0;
      if (timed) stage_begin(gemm_stage, s);
      hipError_t e = launch_kernel<BM, BN, BKB, INT4, BF16, kImages>(g, (unsigned)(tiles * split), s, -1);
      if (e == hipSuccess) {
        combine_images_kernel<BF16><<<dim3((unsigned)(tiles * 64)), dim3(256), 0, s>>>(g);
        e = hipGetLastError();
      }
      if (timed) stage_end(gemm_stage, s);
      return e;
    }
  }
  if (plan.images) return hipErrorInvalidValue;
  if constexpr (BF16 && BM == 128) {
    return launch_kernel<BM, BN, BKB, INT4, BF16, kSliceSums>(g, (unsigned)tiles, s, gemm_stage);
  } else if constexpr (BF16 || BM == 192 || BM != BN || (INT4 && BM != 128)) {
    return hipErrorInvalidValue;   // splits exist for the 128x128 tiles and the 256x256 INT8 tile
  } else {
    const hipError_t e = prepare_hand_over<BM>(g, k_bytes, INT4);
    if (e != hipSuccess) return e;
    return launch_kernel<BM, BN, BKB, INT4, false, kHandOver>(g, (unsigned)(tiles * split), s, gemm_stage);
  }
}

GemmArgs gemm_args(const GemmCall& c, int64_t tiles, bool in_pair) {
  GemmArgs g;
  g.A = c.A;
  g.B = c.B;
  g.M = (int)c.M;
  g.N = (int)c.N;
  g.pitch = c.k_bytes;
  g.out_i32 = c.out_i32;
  g.out_f32 = c.out_i32 ? nullptr : c.out_f32;  // int32 wins; callers ask one at a time
  g.partial = c.partial;
  g.flags = c.flags;
  g.tag = 0;
  g.epoch = c.epoch;
  g.wait_ticks = 0;
  g.row_scale = c.row_scale;
  g.row_stride = c.row_stride;
  g.col_scale = c.col_scale;
  g.inv_n = 1.0f / (float)c.n;
  g.xcd_cols = 0;
  g.stream_out = streams_out(c, tiles, in_pair) ? 1 : 0;
  return g;
}

// The g_w GEMM's workgroups (first: each runs longer, and a hand-over's owners wait for the others)
// and the g_x GEMM's in one launch.  Each alone leaves most units idle behind its prologue, its
// few K stages and its epilogue, and a launch behind another costs 5 us however little it does:
// layer passes of 512 tokens 768 x 768 31.2 -> 25.7 us, 3136 x 448 x 1792 56.3 -> 48.4, 3330 x 1008 x
// 771 70.2 -> 56.3.
template <int BN, bool INT4, bool BF16, int SPLIT>
__global__ __launch_bounds__(256, 2) void gemm_pair_kernel(const GemmArgs gw, const GemmArgs gx, const int gw_wgs) {
  if ((int)blockIdx.x < gw_wgs) igemm_body<128, 128, 2, 2, 128, false, BF16, SPLIT>(gw, (int)blockIdx.x);
  else igemm_body<128, BN, 2, 2, INT4 ? 64 : 128, INT4, false, kWholeK>(gx, (int)blockIdx.x - gw_wgs);
}

template <int BN, bool INT4, bool BF16, int SPLIT>
hipError_t launch_pair_kernel(const GemmArgs& gw, const GemmArgs& gx, int gw_wgs, int gx_wgs, hipStream_t s) {
  constexpr size_t lds_w = 2 * (128 + 128) * 128, lds_x = 2 * (128 + BN) * (INT4 ? 64 : 128);
  constexpr size_t lds = lds_w > lds_x ? lds_w : lds_x;
  auto kern = gemm_pair_kernel<BN, INT4, BF16, SPLIT>;
  static std::atomic<bool> attr_set{false};
  if (!attr_set.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set.store(true, std::memory_order_release);
  }
  kern<<<dim3((unsigned)(gw_wgs + gx_wgs)), dim3(256), lds, s>>>(gw, gx, gw_wgs);
  return hipGetLastError();
}

template <int BN, bool INT4>
hipError_t launch_pair_tile(const GemmArgs& gw, const GemmArgs& gx, int gw_wgs, int gx_wgs, int bits, int split, bool images,
                            hipStream_t s) {
  hipError_t e;
  if (bits == 16)
    e = images ? launch_pair_kernel<BN, INT4, true, kImages>(gw, gx, gw_wgs, gx_wgs, s)
               : launch_pair_kernel<BN, INT4, true, kWholeK>(gw, gx, gw_wgs, gx_wgs, s);
  else if (images) e = launch_pair_kernel<BN, INT4, false, kImages>(gw, gx, gw_wgs, gx_wgs, s);
  else if (split > 1) e = launch_pair_kernel<BN, INT4, false, kHandOver>(gw, gx, gw_wgs, gx_wgs, s);
  else e = launch_pair_kernel<BN, INT4, false, kWholeK>(gw, gx, gw_wgs, gx_wgs, s);
  if (e != hipSuccess || !images) return e;
  const unsigned grid = (unsigned)((int64_t)gw.tiles_m * gw.tiles_n * 64);
  if (bits == 16) combine_images_kernel<true><<<dim3(grid), dim3(256), 0, s>>>(gw);
  else combine_images_kernel<false><<<dim3(grid), dim3(256), 0, s>>>(gw);
  return hipGetLastError();
}

}  // namespace

namespace {

// us a workgroup of 128-row tiles takes for a K stage while it has its unit to itself, shares it with another
// workgroup, and in a launch that fills every place several times over; and for what is not a stage
// (first loads, epilogue).
struct StageTimes { double one, two, full, each; };
constexpr StageTimes kTimesW{0.67, 1.86, 1.29, 2.6};      // g_w, 128-byte stages
constexpr StageTimes kTimesX4{0.48, 0.65, 0.80, 3.8};     // g_x, INT4 on 128x128 tiles, 64-byte stages
constexpr StageTimes kTimesX4Wide{0.56, 1.16, 1.20, 6.5};  // the same on 128x256
constexpr StageTimes kTimesX8{0.60, 1.16, 1.44, 3.4};     // g_x, INT8, 128-byte stages
// An unsplit GEMM on 256x256 INT8 or bfloat16 tiles as a launch between a step's other kernels.
constexpr Cand kLargeAlone{256, 256, 1, 0.097, 0.125, 4.4};
// A GEMM's part of a launch (wgs = 0: the launch has none).
struct Part {
  int64_t wgs, stages;   // workgroups, K stages of each
  StageTimes t;
  int64_t slices;        // of K
  bool images;           // added by a second kernel
  double store_kb;       // output bytes of a workgroup
};
constexpr Part kNoPart{0, 0, kTimesW, 1, false, 0.0};
// us of a launch of `w`'s workgroups with `x`'s behind them on the chip's places, two to a unit: the longest of
// g_w with its hand-over, of g_x from when its last workgroups find a place, and of all the work over all
// places.
double launch_us(const Part& w, const Part& x) {
  const double cus = compute_units(), places = 2 * cus, W = (double)w.wgs, X = (double)x.wgs;
  const double x_each = x.t.each + 0.0095 * x.store_kb;
  const double x1 = X > 0 ? (double)x.stages * x.t.one + x_each : 0.0;
  const double x2 = X > 0 ? (double)x.stages * x.t.two + x_each : 0.0;
  const double x3 = X > 0 ? (double)x.stages * x.t.full + x_each : 0.0;
  const double w1 = W > 0 ? (double)w.stages * w.t.one + w.t.each : 0.0;
  const double w2 = W > 0 ? (double)w.stages * w.t.two + w.t.each : 0.0;
  const double w3 = W > 0 ? (double)w.stages * w.t.full + w.t.each : 0.0;
  const bool resident = W + X <= places, shared = W + X > cus;   // all at once; some unit has two
  double wt = w1, xt = x1;
  if (shared) {
    // what is left of the longer GEMM goes on at its own rate once the other one has ended
    const double beside = resident ? x2 : X * x2 / (places - W > 64 ? places - W : 64.0);
    const double alone = W <= cus ? w1 : w2;
    wt = w2 <= beside ? w2 : beside + (1.0 - beside / w2) * alone;
    xt = x2 <= w2 ? x2 : w2 + (1.0 - w2 / x2) * (resident && X <= cus ? x1 : x2);
  }
  const bool hands = w.slices > 1 && !w.images;
  const double load = W / places;
  const double hand = hands ? 3.6 + 1.07 * (double)(w.slices - 1) + 7.3 * (load < 2.0 ? load : 2.0) : 0.0;
  if (W > places) wt = w3 * (load + 0.66);
  const double waits = (W + (X < places ? X : places) - places) / places * w3;
  double t = wt + hand;
  if (xt + (waits > 0.0 ? waits : 0.0) > t) t = xt + (waits > 0.0 ? waits : 0.0);
  const double all = (W * w3 + X * x3) / places + 0.66 * x3 + 0.54 * hand;
  if (!resident && all > t) t = all;
  return t + (w.images ? 2.9 + 0.019 * W : 0.0) + 0.7;
}
const StageTimes& x_times(int bits, bool wide) { return bits != 4 ? kTimesX8 : wide ? kTimesX4Wide : kTimesX4; }
// us of a GEMM in a launch of its own.
double alone_us(const GemmCall& c, const GemmPlan& p, bool g_w) {
  const int64_t stages = c.k_bytes / p.bkb;
  if (p.bm == 128 && p.bn == 128) {
    const StageTimes& t = g_w ? kTimesW : x_times(c.bits, false);
    const double store_kb = 4.0 * (double)c.M * (double)c.N / (double)p.tiles / 1024.0;
    if (!g_w && p.split == 1) return launch_us(kNoPart, Part{p.tiles, stages, t, 1, false, store_kb});
    return launch_us(Part{p.tiles * p.split, ceil_div(stages, p.split), t, p.split, p.images, 0.0}, kNoPart);
  }
  if (p.split > 1) return large_split_us(stages, p.split) + 8.0;
  const double K = (double)c.k_bytes * (c.bits == 4 ? 2 : 1);
  if (c.bits != 4) return tile_shape_us(kLargeAlone, c.M, c.N, K, compute_units());
  int i = 0;
  while (kCands4[i].bm != p.bm || kCands4[i].bn != p.bn) ++i;
  return tile_shape_us(kCands4[i], c.M, c.N, K, compute_units());
}

}  // namespace

// Whether the two GEMMs of a layer share a launch, g_w's plan in it and the tile of g_x, whose workgroups then do
// the whole of K.  g_w's slices and g_x's tile follow from the time of the whole launch (launch_us), whose constants
// are fitted to layer passes of 3600 layers (128 to 201728 tokens, 64 to 11008 outputs and inputs), every
// split, both tiles and two launches timed on each in the same buffers: what is chosen takes 0.4 % longer than the best
// of them on average, more than 5 % on 44.  Slices chosen without a look at g_x's
// workgroups, and sizes of g_x for which a launch is shared, took 2.2 %: 20736 tokens 832 x 2816 with g_w unsplit
// 257 us a layer pass, 239 in two slices; 7880 x 1664 x 2757 in INT8 with bfloat16 g_w apart 214 us a call, 149 together; 128 x 40960
// x 512 in INT8 together 266 us a pass, 138 apart, where g_x splits K in eight.
// Two launches are looked at only where g_x has more than 28 stages (up to there they were the faster by 2 % on 19
// of 7400 layers) or g_w a 256x256 tile of its own.  There a shared launch has to be 10 % faster by these figures, whose
// error grows with the layer: of 996 such layers it is taken on 732 and 6.5 % faster on average over all (13653
// x 3600 x 1060 in INT8 368 us and 306, 6784 x 5824 x 768 207 and 181), more than 2 % slower on six; without that
// margin on twenty (15360 x 7712 x 3840 981 us apart, 1027 together).
// 128x128 g_x tiles in more workgroups than are resident have to be 3 % faster than 128x256.
GemmPairPlan plan_gemm_pair(const GemmCall& cw, bool images, const GemmCall& cx, bool may_share) {
  GemmPairPlan apart, plan;
  apart.together = plan.together = false;
  apart.w = plan_gemm(cw.M, cw.N, cw.k_bytes, cw.bits, true, images);
  apart.x = plan_gemm(cx.M, cx.N, cx.k_bytes, cx.bits, true, false);
  if (!may_share || g_gemm_mode.load() != 0 || cw.M <= 0 || cw.N <= 0 || cx.M <= 0 || cx.N <= 0) return apart;
  const int64_t places = 2 * (int64_t)compute_units(), most = 8 * places;
  const int64_t stages = cw.k_bytes / 128, x_stages = cx.k_bytes / (cx.bits == 4 ? 64 : 128);
  GemmPlan w = apart.w;
  w.bm = w.bn = 128;
  w.tiles = ceil_div(cw.M, 128) * ceil_div(cw.N, 128);
  int64_t image_split = 0, max_slices = 1;
  if (cw.bits == 16) {   // the slices, and so the bits, that the shape alone gives
    if (apart.w.split > 1 && !apart.w.images) return apart;   // one workgroup per tile adds them
    if (apart.w.images) image_split = apart.w.split, max_slices = 0;
  } else {
    if (images) image_split = image_slices(cw.M, cw.N, cw.k_bytes, cw.bits, compute_units());
    max_slices = max_split(w.tiles, stages);
  }
  double best_us = 1e30;
  for (int wide = 0; wide <= (cx.bits == 4 ? 1 : 0); ++wide) {
    const int64_t tiles = ceil_div(cx.M, 128) * ceil_div(cx.N, wide ? 256 : 128);
    if (w.tiles + tiles > most) continue;
    const Part px{tiles, x_stages, x_times(cx.bits, wide != 0), 1, false,
                  4.0 * (double)cx.M * (double)cx.N / (double)tiles / 1024.0};
    for (int64_t s = image_split ? 0 : 1; s <= max_slices; ++s) {   // 0: images
      const int64_t slices = s ? s : image_split, wgs = w.tiles * slices;
      if (s > 1 && wgs > places) break;
      double us = launch_us(Part{wgs, ceil_div(stages, slices), kTimesW, slices, s == 0, 0.0}, px);
      if (cx.bits == 4 && !wide && wgs + tiles > places) us *= 1.03;
      if (us >= best_us) continue;
      best_us = us;
      plan.together = true;
      plan.w = w;
      plan.w.split = (int)slices;
      plan.w.images = s == 0;
      plan.w.partial_bytes = s == 0 ? image_scratch_bytes(cw.M, cw.N, cw.k_bytes, cw.bits)
                                    : (size_t)w.tiles * (slices - 1) * 128 * 128 * 4;
      plan.x = GemmPlan{128, wide ? 256 : 128, cx.bits == 4 ? 64 : 128, 1, tiles, false, 0};
    }
  }
  if (!plan.together) return apart;
  if (x_stages <= 28 && apart.w.bm == 128) return plan;
  const double us = alone_us(cx, apart.x, false) + alone_us(cw, apart.w, true) - 0.5;
  return us * (apart.w.bm == 128 ? 1.0 : 0.9) < best_us ? apart : plan;
}

hipError_t launch_gemm_pair(const GemmCall& cw, const GemmCall& cx, const GemmPairPlan& plan, hipStream_t s, int stage) {
  const GemmPlan& p = plan.w;
  const bool int4 = cx.bits == 4, narrow = plan.x.bn == 128;
  const int64_t rows = ceil_div(cx.M, 128), w = p.tiles * p.split, x = plan.x.tiles;
  GemmArgs gw = gemm_args(cw, p.tiles, true), gx = gemm_args(cx, x, true);
  gw.nk_total = (int)(cw.k_bytes / 128);
  gw.tiles_m = (int)ceil_div(cw.M, 128);
  gw.tiles_n = (int)ceil_div(cw.N, 128);
  set_slices(gw, p.split);
  if (p.images) {
    if (!gw.partial) return hipErrorInvalidValue;
    gw.xcd_cols = p.split % 8 == 0 ? -2 : slice_placement<128>(gw, p.tiles);
  } else if (p.split > 1) {
    const hipError_t e = prepare_hand_over<128>(gw, cw.k_bytes, false);
    if (e != hipSuccess) return e;
  }
  gx.nk_total = (int)(cx.k_bytes / (int4 ? 64 : 128));
  gx.tiles_m = (int)rows;
  gx.tiles_n = (int)ceil_div(cx.N, narrow ? 128 : 256);
  set_slices(gx, 1);
  stage_begin(stage, s);
  const hipError_t e = !narrow ? launch_pair_tile<256, true>(gw, gx, (int)w, (int)x, cw.bits, p.split, p.images, s)
                       : int4  ? launch_pair_tile<128, true>(gw, gx, (int)w, (int)x, cw.bits, p.split, p.images, s)
                               : launch_pair_tile<128, false>(gw, gx, (int)w, (int)x, cw.bits, p.split, p.images, s);
  stage_end(stage, s);
  return e;
}

hipError_t launch_igemm(const GemmCall& c, const GemmPlan& plan, hipStream_t s, int gemm_stage) {
  if (c.M <= 0 || c.N <= 0) return hipSuccess;
  const GemmArgs g = gemm_args(c, plan.tiles, false);
  const int64_t k_bytes = c.k_bytes;
  const int bits = c.bits;
  const int gs = gemm_stage;
  if (bits == 16) {
    if (plan.bm == 256) return launch_tile<256, 256, 128, false, true>(g, k_bytes, plan, s, gs);
    if (plan.bm == 128) return launch_tile<128, 128, 128, false, true>(g, k_bytes, plan, s, gs);
    return hipErrorInvalidValue;
  }
  if (plan.bm == 256)
    return bits == 4 ? launch_tile<256, 256, 64, true>(g, k_bytes, plan, s, gs)
                     : launch_tile<256, 256, 128, false>(g, k_bytes, plan, s, gs);
  if (plan.bm == 192 && bits == 4) return launch_tile<192, 256, 64, true>(g, k_bytes, plan, s, gs);
  if (plan.bm == 128 && plan.bn == 256 && bits == 4) return launch_tile<128, 256, 64, true>(g, k_bytes, plan, s, gs);
  if (plan.bm == 128)
    return bits == 4 ? launch_tile<128, 128, 64, true>(g, k_bytes, plan, s, gs)
                     : launch_tile<128, 128, 128, false>(g, k_bytes, plan, s, gs);
  return hipErrorInvalidValue;
}

}  // namespace hot
