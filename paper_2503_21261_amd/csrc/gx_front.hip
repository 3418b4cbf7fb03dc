// Operands made by shared launches.  First launch of the g_x path (Sec. 5.1) when both of its
// operands are produced in one kernel (and below, those of both GEMMs of a small layer): the leading workgroups transform and quantise the weights (H.w, one scale, the
// single-pass column kernel with its abs-max exchange), the rest rotate and quantise the
// rows of g_y per token.  The two jobs are independent; sharing a launch lets the rows
// stream from HBM while the few weight workgroups sit in the latencies of their exchange,
// which as a kernel of its own is 13 us of a mostly idle chip for the ViT-B weights.
#include <mutex>

#include "col_quant_kernel.h"
#include "row_quant_kernel.h"

namespace hot {

namespace {

template <int N, int KB, int ITER, int TPR>
__global__ __launch_bounds__(256, 2) void w_and_rows_kernel(const OnepassArgs wa, const int w_tiles,
                                                            const RowQuantArgs ra) {
  // workgroups are dispatched in index order: the weight tiles, which must all be resident
  // for their exchange to complete without the fallback, come first
  if ((int)blockIdx.x < w_tiles)
    onepass_body<N, onepass_vec(N), kKeepAll4, KB>(wa, (int)blockIdx.x, w_tiles);
  else
    row_quant_body<N, ITER, TPR>(ra, (int64_t)blockIdx.x - w_tiles, (int64_t)gridDim.x - w_tiles);
}

struct FrontArgs {
  OnepassArgs wa;
  RowQuantArgs ra;
  int64_t nrb;   // row workgroups
};

template <int N, int KB, int ITER, int TPR>
hipError_t try_front(const FrontArgs& f, hipStream_t s, int stage, bool* done) {
  constexpr int VEC = onepass_vec(N);
  if (*done || f.wa.C % VEC != 0) return hipSuccess;
  const int64_t tiles = ceil_div(f.wa.C, 64 * VEC) * ceil_div(f.wa.rt.nblk, 4 * KB);
  size_t lds = (size_t)(64 * VEC) * (4 * KB * (N / 2) + 4);
  if (lds < onepass_stage_bytes<N, VEC, kKeepAll4>()) lds = onepass_stage_bytes<N, VEC, kKeepAll4>();
  auto kern = w_and_rows_kernel<N, KB, ITER, TPR>;
  static std::mutex mu;
  static int per_cu = -1, cus = 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (per_cu < 0) {
      int dev = 0, nb = 0;
      hipError_t e = hipGetDevice(&dev);
      if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
      if (e == hipSuccess && lds > 48 * 1024)
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, 256, lds);
      if (e != hipSuccess) return e;
      per_cu = nb;
    }
  }
  if (tiles > (int64_t)per_cu * cus || tiles > kMaxExchange) return hipSuccess;
  stage_begin(stage, s);
  kern<<<dim3((unsigned)(tiles + f.nrb)), dim3(256), lds, s>>>(f.wa, (int)tiles, f.ra);
  stage_end(stage, s);
  *done = true;
  return hipGetLastError();
}

template <int N, int ITER, int TPR>
hipError_t front_kb(const FrontArgs& f, hipStream_t s, int stage, bool* done) {
  hipError_t e = try_front<N, 1, ITER, TPR>(f, s, stage, done);
  if (e == hipSuccess && !*done) e = try_front<N, 2, ITER, TPR>(f, s, stage, done);
  return e;
}

template <int N>
hipError_t front_n(FrontArgs& f, hipStream_t s, int stage, bool* done) {
  const int cols = f.ra.cols;
  const int v64 = (int)ceil_div(cols, 256), v256 = (int)ceil_div(cols, 1024);
  // the row kernel's own choice of threads per row and values per thread (row_quant.hip)
  if (v64 <= 1) return hipSuccess;
  if (v64 <= 4) f.nrb = ceil_div(f.ra.rows, 4);
  else f.nrb = f.ra.rows;
  if (f.nrb > (1 << 20)) return hipSuccess;
  if (v64 == 2) return front_kb<N, 2, 64>(f, s, stage, done);
  if (v64 == 3) return front_kb<N, 3, 64>(f, s, stage, done);
  if (v64 == 4) return front_kb<N, 4, 64>(f, s, stage, done);
  if (v256 == 2) return front_kb<N, 2, 256>(f, s, stage, done);
  if (v256 == 3) return front_kb<N, 3, 256>(f, s, stage, done);
  if (v256 == 4) return front_kb<N, 4, 256>(f, s, stage, done);
  return hipSuccess;
}

// Rows of g_y (per token) and the abs-max pass of its token-direction view, for tensors far beyond the
// caches.  HBM-bound: both jobs read all of g_y, so the workgroups of an XCD (every eighth) go through
// slabs of 64 rows together, first a row each, then the slab's column tiles, whose lines the XCD's L2 then
// holds or has under way: one read of HBM instead of two.  us, rows and abs-max pass apart and together:
// 16384 tokens 11008 outputs 156 + 127 and 200, 16384 x 4096 57 + 49 and 77 (64-row blocks); 32736 x 5120
// 151 + 120 and 172, 12800 x 8192 89 + 78 and 105 (32-row blocks).  Fetched: 1.01 times g_y at 4096 columns,
// 1.78 times at 11008, whose slab is 2.8 of the L2's 4 MB; fewer workgroups under way do not help there
// (three per unit 198 us, two 244).
constexpr int kSlabRows = 64;
// Columns per lane of its column tiles: one for 64-row blocks, whose two would set the registers of the
// rows as well (16384 x 4096 92 us with two, 77 with one; 32768 x 4096 174 and 147).
__host__ __device__ constexpr int slab_vec(int n) { return n == 64 ? 1 : 2; }
template <int N, int KIND, int ITER>
__global__ __launch_bounds__(256) void rows_and_absmax_kernel(const RowQuantArgs ra, const RowTiling rt, const KeepMap map,
                                                              const int slabs, const int col_wgs, float* partials) {
  constexpr int VEC = slab_vec(N), KBW = kSlabRows / N;
  const int per_slab = kSlabRows + col_wgs, j = (int)blockIdx.x >> 3;
  const int slab = 8 * (j / per_slab) + ((int)blockIdx.x & 7), k = j % per_slab;
  if (slab >= slabs) return;
  if (k < kSlabRows) {
    const int64_t row = (int64_t)slab * kSlabRows + k;
    if (row < ra.rows) row_quant_body<N, ITER, 256>(ra, row, ra.rows);
    return;
  }
  const int64_t C = ra.cols, tiles_x = (C + 256 * VEC - 1) / (256 * VEC);
  float m = 0.0f;
  for (int64_t tx = k - kSlabRows; tx < tiles_x; tx += col_wgs)
    m = fmaxf(m, absmax_tile<N, VEC, KIND>(ra.t, rt, C, map, KBW, tx, slab));
  m = workgroup_max(m);
  if (threadIdx.x == 0) partials[slab * col_wgs + k - kSlabRows] = m;
}

template <int N, int KIND>
hipError_t rows_and_absmax_n(const RowQuantArgs& ra, const RowTiling& rt, const KeepMap& map, int slabs, int col_wgs,
                             float* partials, hipStream_t s) {
  const dim3 grid((unsigned)(ceil_div(slabs, 8) * 8 * (kSlabRows + col_wgs)));
#define HOT_ITER(ITER)                                                                                              \
  if (ra.cols <= 1024 * ITER) {                                                                                     \
    rows_and_absmax_kernel<N, KIND, ITER><<<grid, dim3(256), 0, s>>>(ra, rt, map, slabs, col_wgs, partials);        \
    return hipGetLastError();                                                                                       \
  }
  HOT_ITER(3) HOT_ITER(4) HOT_ITER(6) HOT_ITER(8) HOT_ITER(11)
#undef HOT_ITER
  return hipErrorInvalidValue;
}

// All operands of a small layer's two GEMMs in one launch: the weight tiles and the tiles of g_y's
// token-direction view (each set exchanging its own maxima, all resident at once), then the rows of
// g_y (per token, or the abs-max pass of one scale per tensor).  Three launches otherwise, each far
// from filling the chip; bound by one tile's chain of load, exchange, quantise, store.  The settings
// are branches, not instantiations: registers are those of the widest (KB blocks per wave on both
// sides), which with KB = 1 leaves five workgroups per unit (three for 64-row
// blocks).  Layer passes: 512 tokens 768 x 768 25.7 -> 21.9 us, 3136 x 448 x 1792 48.4 -> 43.0, 3330 x 1008 x
// 771 with one g_y scale 56.3 -> 48.4.
template <int N, int KB>
__global__ __launch_bounds__(256, 2) void operands_kernel(const OnepassArgs wa, const int w_tiles, const OnepassArgs ga,
                                                          const int g_tiles, const int g_kind, const RowQuantArgs ra,
                                                          const int layout) {
  constexpr int VEC = onepass_vec(N);
  int bid = (int)blockIdx.x;
  if (bid < w_tiles) {
    const bool wide = wa.C % VEC == 0;
    if (ra.bits == 4) {
      if (wide) onepass_body<N, VEC, kKeepAll4, KB>(wa, bid, w_tiles);
      else onepass_body<N, 1, kKeepAll4, KB>(wa, bid, w_tiles);
    } else {
      if (wide) onepass_body<N, VEC, kKeepAll8, KB>(wa, bid, w_tiles);
      else onepass_body<N, 1, kKeepAll8, KB>(wa, bid, w_tiles);
    }
    return;
  }
  bid -= w_tiles;
  if (bid < g_tiles) {
    if (g_kind == kKeepLowHalf) onepass_body<N, VEC, kKeepLowHalf, KB>(ga, bid, g_tiles);
    else if (g_kind == kKeepLpL1) onepass_body<N, VEC, kKeepLpL1, KB>(ga, bid, g_tiles);
    else onepass_body<N, VEC, kKeepGeneric, KB>(ga, bid, g_tiles);
    return;
  }
  bid -= g_tiles;
  const int nbid = (int)gridDim.x - w_tiles - g_tiles;
  switch (layout) {
#define HOT_LAYOUT(ITER, TPR) \
  case ITER * 1000 + TPR: row_quant_body<N, ITER, TPR>(ra, bid, nbid); break;
    HOT_LAYOUT(1, 16) HOT_LAYOUT(1, 32) HOT_LAYOUT(1, 64) HOT_LAYOUT(2, 64) HOT_LAYOUT(3, 64) HOT_LAYOUT(4, 64)
    HOT_LAYOUT(2, 256) HOT_LAYOUT(3, 256) HOT_LAYOUT(4, 256)
#undef HOT_LAYOUT
  }
}

struct OperandArgs {
  OnepassArgs wa, ga;
  int g_kind;
  RowQuantArgs ra;
  int layout;
  int64_t nrb;
  bool with_g;   // the token-direction view is part of the launch
};

template <int N, int KB>
hipError_t try_operands(const OperandArgs& f, hipStream_t s, int stage, OperandsMade* made) {
  constexpr int VEC = onepass_vec(N);
  if (*made) return hipSuccess;
  const int wv = f.wa.C % VEC == 0 ? VEC : 1;
  const int64_t wt = ceil_div(f.wa.C, 64 * wv) * ceil_div(f.wa.rt.nblk, 4 * KB);
  const int64_t gt = f.with_g ? ceil_div(f.ga.C, 64 * VEC) * ceil_div(f.ga.rt.nblk, 4 * KB) : 0;
  if (wt > kMaxExchange || gt > kMaxExchange) return hipSuccess;
  // code bytes per block and column, of either side at most
  const int bpb_w = f.ra.bits == 4 ? N / 2 : N, bpb = f.with_g && f.ga.r > bpb_w ? f.ga.r : bpb_w;
  size_t lds = (size_t)(64 * VEC) * (4 * KB * bpb + 4);
  if (lds < onepass_stage_bytes<N, VEC, kKeepGeneric>()) lds = onepass_stage_bytes<N, VEC, kKeepGeneric>();
  constexpr size_t lds_max = (size_t)(64 * VEC) * (4 * KB * N + 4);   // never below the staging bytes
  auto kern = operands_kernel<N, KB>;
  int64_t resident;
  {
    static std::mutex mu;
    static int per_cu = -1, cus = 0;
    static size_t lds_seen = 0;
    std::lock_guard<std::mutex> lock(mu);
    if (per_cu < 0 || lds != lds_seen) {
      int dev = 0, nb = 0;
      hipError_t e = hipGetDevice(&dev);
      if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
      if (e == hipSuccess && per_cu < 0 && lds_max > 48 * 1024)
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
      if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, 256, lds);
      if (e != hipSuccess) return e;
      per_cu = nb;
      lds_seen = lds;
    }
    resident = (int64_t)per_cu * cus;
  }
  if (wt + gt > resident) return hipSuccess;
  stage_begin(stage, s);
  kern<<<dim3((unsigned)(wt + gt + f.nrb)), dim3(256), lds, s>>>(f.wa, (int)wt, f.ga, (int)gt, f.g_kind, f.ra, f.layout);
  stage_end(stage, s);
  *made = f.with_g ? kOperandsAll : kOperandsOfGx;
  return hipGetLastError();
}

template <int N>
hipError_t operands_n(OperandArgs f, bool all, bool of_gx, hipStream_t s, int stage, OperandsMade* made) {
  // one block per wave: the most workgroups, the shortest chain; two where one leaves more than
  // 512 workgroups (the exchange's slots) on a side
  hipError_t e = hipSuccess;
  f.with_g = true;
  if (all) e = try_operands<N, 1>(f, s, stage, made);
  if (all && e == hipSuccess) e = try_operands<N, 2>(f, s, stage, made);
  f.with_g = false;
  if (of_gx && e == hipSuccess) e = try_operands<N, 1>(f, s, stage, made);
  if (of_gx && e == hipSuccess) e = try_operands<N, 2>(f, s, stage, made);
  return e;
}

// Whether the rows of g_y may share a launch with the column jobs: they then run at the registers
// of the widest of them (two waves per SIMD for 64-row blocks, three or four below), which a few
// megabytes of rows do not notice and long streams do; wide weights, two blocks per wave, take their
// share of the places on top.  The largest g_y that gained, in elements, and the next size timed, over
// 1450 layers (us a backward call apart and together):
//   per token   16-row blocks   any size up to where the shared passes begin; with wide weights 8.4 M
//                               (4096 tokens 2048 x 4096 104 and 106, 2048 tokens 68 and 66)
//               32              19 M (25216 x 768 x 768 103 and 100; 50432 x 2048 x 512 384 and 404);
//                               wide weights 8.4 M (8192 x 2048 x 4096 174 and 176)
//               64              9.7 M (12608 x 768 x 768 63 and 57; 12608 x 2048 x 512 117 and 128)
//   one scale   any size, where a lane has more than one 16-byte load in flight; 64-row blocks of 256 columns
//                               and fewer 26 M (201728 x 256 x 256 233 and 241)
// Weights of 64-row blocks that need all the exchange's slots lose at every size (1024 tokens
// 4096 x 4096 87 and 90).
bool rows_join(const Config& cfg, int64_t L, int64_t O, int64_t I, bool per_token) {
  const int lanes = cfg.n == 16 && I % 2 == 0 ? 2 : 1;
  auto weight_tiles = [&](int kb) { return ceil_div(I, 64 * lanes) * ceil_div(O / cfg.n, 4 * kb); };
  const bool wide = weight_tiles(1) > kMaxExchange;
  if (cfg.n == 64 && weight_tiles(2) >= kMaxExchange) return false;
  const int64_t elements = L * O, million = 1000000;
  if (!per_token) return cfg.n != 64 || O > 256 || elements <= 26 * million;
  if (cfg.n == 16) return !wide || elements <= 8 * million;
  if (cfg.n == 32) return elements <= (wide ? 12 : 20) * million;
  return elements <= 10 * million;
}

// Bounded wait (100 MHz ticks) of the single-pass workgroups over `bytes` of input.
long long wait_ticks(int64_t wait_us, int64_t bytes) {
  const int64_t stream_us = bytes / 1000000;   // as in the column kernel's own launcher
  return (wait_us > 0 && wait_us < stream_us ? stream_us : wait_us) * 100;
}

}  // namespace

// From 48 M elements on no form of the single-pass column kernel holds the kept values (42 M at most: 512
// workgroups, 160 registers), so that the abs-max pass is there to be saved; 16-row blocks have the shared
// passes.  From 2048 columns on (layer passes with 512 inputs, apart and together: 64-row blocks 23872 x 2048 218 and
// 196 us, 32000 x 2112 309 and 278, 23424 x 3072 285 and 248, 28544 x 4032 430 and 367; 32-row blocks 30464 x 2048 242 and
// 220): below, the LP_L1 list, whose column tiles are the slower ones, loses what the default list gains (32-row
// blocks 31200 x 1568 213 and 221, 64-row blocks 32704 x 1536 258 and 261 with it, 31872 x 1536 246 and 225 with the default).
// Above 11264 a slab no longer fits an XCD's L2.  At least four column workgroups per slab within kMaxPartials.
bool rows_and_absmax_applies(const Config& cfg, int64_t L, int64_t O) {
  return cfg.n >= 32 && cfg.gw_bits == 8 && cfg.sample_tokens == 0 && O >= 2048 && O <= 11264 &&
         L * O >= 48ll * 1000 * 1000 && ceil_div(L, kSlabRows) <= kMaxPartials / 4;
}

hipError_t launch_rows_and_absmax(const float* g_y, int64_t L, int64_t O, const Config& cfg, uint8_t* qg, int64_t pitch,
                                  float* s_g, float* partials, int* npartials, hipStream_t s, int stage) {
  const int64_t slabs = ceil_div(L, kSlabRows);
  const int64_t tiles_x = ceil_div(O, 256 * slab_vec(cfg.n));
  const int64_t col_wgs = tiles_x * slabs <= kMaxPartials ? tiles_x : kMaxPartials / slabs;
  const RowTiling rt = row_tiling(cfg, L);
  const RowQuantArgs ra{g_y, L, (int)O, cfg.gx_bits, cfg.rounding, 0, qg, pitch, s_g, nullptr, 0};
  const bool low = cfg.lowpass_default && cfg.r * 2 == cfg.n;
  stage_begin(stage, s);
  hipError_t e;
  if (cfg.n == 32) e = low ? rows_and_absmax_n<32, kKeepLowHalf>(ra, rt, cfg.map, (int)slabs, (int)col_wgs, partials, s)
                           : rows_and_absmax_n<32, kKeepGeneric>(ra, rt, cfg.map, (int)slabs, (int)col_wgs, partials, s);
  else e = low ? rows_and_absmax_n<64, kKeepLowHalf>(ra, rt, cfg.map, (int)slabs, (int)col_wgs, partials, s)
               : rows_and_absmax_n<64, kKeepGeneric>(ra, rt, cfg.map, (int)slabs, (int)col_wgs, partials, s);
  stage_end(stage, s);
  *npartials = (int)(slabs * col_wgs);
  return e;
}

hipError_t launch_operands(const float* w, int64_t O, int64_t I, const Config& cfg, uint8_t* qw, int64_t pitch, float* s_w,
                           float* slots_w, const float* g_y, int64_t L, bool per_token, uint8_t* qg, float* s_g,
                           float* row_partials, int* npartials, uint8_t* qgh, int64_t pitch_h, float* s_gh,
                           float* slots_g, hipStream_t s, int stage, OperandsMade* made) {
  *made = kOperandsNone;
  const int64_t wait_us = exchange_wait_us();
  if (wait_us < 0 || O > 4096 || !rows_join(cfg, L, O, I, per_token)) return hipSuccess;
  // INT4 with a scale per token has w_and_rows_kernel, whose rows keep more waves (INT8, 6304 tokens
  // 3072 x 768: 118 -> 114 us a layer pass)
  const bool all = cfg.gw_bits == 8, of_gx = cfg.gx_bits == 8 || !per_token;
  KeepMap id;
  for (int k = 0; k < 64; ++k) id.pos[k] = (int8_t)(k < cfg.n ? k : -1);
  const RowTiling rt = row_tiling(cfg, L);
  OperandArgs f;
  f.wa = OnepassArgs{w, RowTiling{O / cfg.n, 0, 1}, I, id, cfg.n, cfg.rounding,
                     reinterpret_cast<unsigned long long*>(slots_w), next_exchange_tag(), cfg.epoch,
                     wait_ticks(wait_us, O * I * 4), qw, pitch, s_w};
  f.ga = OnepassArgs{g_y, rt, O, cfg.map, cfg.r, cfg.rounding, reinterpret_cast<unsigned long long*>(slots_g),
                     next_exchange_tag(), cfg.epoch, wait_ticks(wait_us, rt.nblk * cfg.n * O * 4), qgh, pitch_h, s_gh};
  f.g_kind = cfg.lowpass_default && cfg.r * 2 == cfg.n ? kKeepLowHalf : (cfg.lp_l1 ? kKeepLpL1 : kKeepGeneric);
  f.layout = 0;
  f.nrb = 0;
  with_row_layout(O, [&](auto iter_c, auto tpr_c) {
    constexpr int ITER = decltype(iter_c)::value, TPR = decltype(tpr_c)::value;
    f.layout = ITER * 1000 + TPR;
    f.nrb = ceil_div(L, 256 / TPR);
  });
  if (!per_token && f.nrb > kMaxPartials) f.nrb = kMaxPartials;
  if (f.nrb > (1 << 20)) return hipSuccess;
  f.ra = RowQuantArgs{g_y, L, (int)O, cfg.gx_bits, cfg.rounding, per_token ? 0 : 1, qg, pitch, s_g, row_partials, 0};
  *npartials = (int)f.nrb;
  switch (cfg.n) {
    case 16: return operands_n<16>(f, all, of_gx, s, stage, made);
    case 32: return operands_n<32>(f, all, of_gx, s, stage, made);
    case 64: return operands_n<64>(f, all, of_gx, s, stage, made);
  }
  return hipSuccess;
}

hipError_t launch_w_and_rows(const float* w, int64_t O, int64_t I, const Config& cfg, uint8_t* qw,
                             int64_t pitch, float* s_w, float* slots, const float* g_y, int64_t L,
                             uint8_t* qg, float* s_g, hipStream_t s, int stage, bool* done) {
  *done = false;
  int64_t wait_us = exchange_wait_us();
  if (wait_us < 0 || cfg.gx_bits != 4 || O % cfg.n != 0 || L <= 0 || I <= 0) return hipSuccess;
  const int64_t stream_us = O * I * 4 / 1000000;   // as in the column kernel's own launcher
  if (wait_us > 0 && wait_us < stream_us) wait_us = stream_us;
  KeepMap id;
  for (int k = 0; k < 64; ++k) id.pos[k] = (int8_t)(k < cfg.n ? k : -1);
  FrontArgs f;
  f.wa = OnepassArgs{w, RowTiling{O / cfg.n, 0, 1}, I, id, cfg.n, cfg.rounding,
                     reinterpret_cast<unsigned long long*>(slots), next_exchange_tag(), cfg.epoch,
                     (long long)(wait_us * 100), qw, pitch, s_w};
  f.ra = RowQuantArgs{g_y, L, (int)O, 4, cfg.rounding, 0, qg, pitch, s_g, nullptr, 0};
  f.nrb = 0;
  switch (cfg.n) {
    case 16: return front_n<16>(f, s, stage, done);
    case 32: return front_n<32>(f, s, stage, done);
    case 64: return front_n<64>(f, s, stage, done);
  }
  return hipSuccess;
}

}  // namespace hot
