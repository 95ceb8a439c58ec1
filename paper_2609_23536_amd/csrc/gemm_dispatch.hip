// Tile choice of the FP8 GEMM.
#include "gemm_util.h"

#include <atomic>

namespace qe {

// What a product costs with each tile shape, in microseconds, fitted to a
// sweep on MI355X (M 64 to 14336, N 152 to 28672, K 128 to 19456, BF16 / FP32 /
// accumulate outputs).  Over 34 such products the shape it picks is 2% slower
// than the best one on average and never slower than 256 x 256; it is furthest
// off where several small tiles come close: 2730 x 1365 x 1000 FP32 13.7
// against 11.6 with 128 x 64 tiles, 320 x 19456 x 1373 19.1 against 16.2 with
// 128 x 128, 64 x 28672 x 4096 21.4 against 19.8 with 64 x 64
// (profiles/gemm_tile_choice_34_products.txt has every shape on each).
//
// Large tiles run one workgroup per compute unit, round after round: a round
// of 256 x 256 tiles costs F + T * s, with T = K tiles of 128, s = 1.0 on a
// chip at most a quarter full and 1.2 beyond (measured: K = 14336 on 32 tiles
// 118, on 128 tiles 136), and F the prologue and the epilogue's burst of output
// traffic, by output type (FP32: 4096 x 4096 x 256, 18 in all; an accumulation
// moves twice the bytes, and more than one round of it also waits for the
// write-back of the one before).  The narrower tiles' rounds, relative to
// 256 x 256 (K = 4096, one round of each, BF16 out): 256 x 192 0.89,
// 192 x 256 0.86 (0.75 of the MFMA work at a lower efficiency per FLOP),
// 256 x 224 0.978.
constexpr double kLargeF[3] = {14.0, 9.0, 25.0};  // by GemmParams::out: FP32, BF16, accumulate
constexpr double kLargeF2 = 28.0;                 // accumulate, more than one round
// added to F where rows are not vector-aligned: the checked epilogue (8191 x
// 8191 x 2049, four rounds: FP32 181, accumulate 260)
constexpr double kLargeScalar[3] = {11.0, 8.0, 17.0};
constexpr double kCost256x192 = 0.89;
constexpr double kCost192x256 = 0.86;
constexpr double kCost224 = 0.98;

// Small tiles cost F + c * (T * s + E), c being the tiles of the busiest
// compute unit: their K loops are bound by the LDS-bound loads (about 84 bytes
// per ns and compute unit), so s does not depend on how many workgroups share
// the unit, and E is the epilogue's traffic that the other workgroup's K loop
// does not hide.  s grows with K as the operands outgrow the caches (128 x 128,
// two tiles per unit: K = 8192 57, K = 14336 127).  `scalar` is added to E where
// rows are not vector-aligned.
struct SmallTile {
  int tile, deep;  // deep: the variant for grids of one workgroup per unit (0: none)
  int64_t bm, bn;
  double f, s, s_k, s_deep, e[3], scalar;  // s + s_k * T per K tile
};
constexpr SmallTile kSmall[] = {
    {kTile64x64, 0, 64, 64, 3.0, 0.19, 0.0, 0.0, {0.6, 0.3, 1.2}, 0.2},
    {kTile128x64, kTile128x64Deep, 128, 64, 3.5, 0.30, 0.0, 0.295, {1.2, 0.5, 2.4}, 0.4},
    {kTile64x128, kTile64x128Deep, 64, 128, 3.5, 0.30, 0.0, 0.295, {1.2, 0.5, 2.4}, 0.4},
    {kTile128x128, kTile128x128Deep, 128, 128, 4.0, 0.46, 0.0008, 0.52, {2.2, 0.6, 5.6}, 0.8},
};

// Small tiles in many rounds.  The model above was fitted where the busiest unit
// has a few small tiles; beyond, it took them for products whose output traffic
// they cannot keep up with: 4096 x 28672 x 1024 BF16 221 us with 128 x 128 tiles,
// 118 with 256 x 256; 8192 x 28672 x 512 FP32 399 and 213.  Rows whose pitch is a
// multiple of 4 KB fall on few memory channels, which costs the short runs of
// small tiles most (over short K loops, FP32, 128 x 128 tiles take 0.9 of the large
// tiles' time at other pitches and 1.1 to 1.2 of it there).  So where it
// picks a small tile for more than kFewTiles per unit, a second model chooses:
//   t = f + rounds (T (s + k T) + e + [wide pitch] p) + load T q
// with `load` the tiles per unit and `rounds` that number rounded up; fitted to
// 1986 such products on MI355X, then adjusted so that the choice costs least.
// On 410 others it is 3.1% slower than the best shape on average (the first
// model 9%; profiles/gemm_tile_choice_many_rounds.txt has every shape on a
// grid of them).  The first model's choice stays for odd rows and, at other
// pitches, for K up to kShortK, where it is the better one.  Of 900 random
// products (M, N, K up to 28672) 91 are more than 3% faster so than with the first
// model alone and 46 slower, and 9 instead of 29 are slower than with large
// tiles only.
struct ManyRounds {
  int tile;
  int64_t bm, bn;
  double f, s, q, k;
  double e[3], p[3];  // by GemmParams::out: FP32, BF16, accumulate
};
constexpr int64_t kFewTiles = 2, kShortK = 192, kWidePitch = 4096;  // bytes
constexpr ManyRounds kManyRounds[] = {
    {kTile256x256, 256, 256, 1.21, 0.863, 0.437, 0.00293, {10.9, 9.18, 14}, {0.0241, 0.25, 0.954}},
    {kTile256x224, 256, 224, 3.91, 0.826, 0.783, 0.000663, {6.25, 11.4, 23.8}, {0.514, 0.406, 0.453}},
    {kTile256x192, 256, 192, 1.62, 0.588, 0.4, 0.00323, {9.93, 9.4, 22.7}, {0.11, 0, 0.281}},
    {kTile192x256, 192, 256, 2.64, 0.743, 0.475, 0.000228, {7.77, 7.53, 9.06}, {0.0508, 0.401, 0.0188}},
    {kTile64x64, 64, 64, 1.74, 0.064, 0.0487, 0.00104, {1.16, 1.86, 1.43}, {0.3, 0.0529, 0.369}},
    {kTile128x64, 128, 64, 1.99, 0.118, 0.0831, 0.00175, {1.7, 2.61, 1.81}, {0.459, 0.465, 0.235}},
    {kTile64x128, 64, 128, 1.51, 0.126, 0.118, 0.00261, {1.44, 1.83, 1.49}, {0.423, 0.00483, 0.144}},
    {kTile128x128, 128, 128, 5.01, 0.00963, 0.508, 0.000325, {1.68, 2.28, 7.87}, {0.176, 0.058, 0.671}},
};

static std::atomic<int> g_tile_override{0};

// Compute units of the current device, read once per device from its properties; 256 on MI355X.
static int cu_count() {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> cache[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  int n = cache[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
  cache[dev].store(n, std::memory_order_relaxed);
  return n;
}

hipError_t launch_gemm(const GemmParams &g, hipStream_t s, const UpdateParams *fused) {
  UpdateParams none;
  memset(&none, 0, sizeof(none));
  const UpdateParams &u = fused != nullptr ? *fused : none;
  if (g.m <= 0 || g.n <= 0) return u.n > 0 ? launch_scale_update(u, s) : hipSuccess;
  // The kernel addresses each operand with 32-bit offsets: split any operand
  // of 2 GiB or more into row blocks (independent GEMMs on disjoint outputs),
  // whole 256-row tiles per block where a tile's rows fit in 2 GiB, else as
  // many rows as fit (at least one: its offsets are then 0 plus the K offset,
  // which stays below 2^31 because K does).
  constexpr int64_t kLim = int64_t(1) << 31;
  if (g.k >= kLim) return hipErrorInvalidValue;
  auto block_rows = [](int64_t ld) -> int64_t {
    const int64_t r = (kLim - 1) / ld;
    return r >= 256 ? r / 256 * 256 : (r > 0 ? r : 1);
  };
  const int64_t cbytes = g.out == 1 ? 2 : 4;
  if (g.m * g.lda >= kLim) {
    const int64_t rows = block_rows(g.lda);
    for (int64_t r = 0; r < g.m; r += rows) {
      GemmParams sub = g;
      sub.a = g.a + r * g.lda;
      sub.m = g.m - r < rows ? g.m - r : rows;
      sub.c = static_cast<char *>(g.c) + r * g.ldc * cbytes;
      const hipError_t e = launch_gemm(sub, s, r + rows >= g.m ? fused : nullptr);  // the update rides on the last
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (g.n * g.ldb >= kLim) {
    const int64_t cols = block_rows(g.ldb);
    for (int64_t c0 = 0; c0 < g.n; c0 += cols) {
      GemmParams sub = g;
      sub.b = g.b + c0 * g.ldb;
      sub.n = g.n - c0 < cols ? g.n - c0 : cols;
      sub.c = static_cast<char *>(g.c) + c0 * cbytes;
      const hipError_t e = launch_gemm(sub, s, c0 + cols >= g.n ? fused : nullptr);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const int force = g_tile_override.load(std::memory_order_relaxed);
  if (force == kTile256x128) return launch_gemm_ring(force, g, s, u);
  if (force > 0) return launch_gemm_large(force, g, s, u);
  const int64_t cus = cu_count();
  const double T = double((g.k + 127) / 128);
  auto tiles = [&](int64_t bm, int64_t bn) { return ((g.m + bm - 1) / bm) * ((g.n + bn - 1) / bn); };
  const bool scalar = !gemm_vec_ok(g);
  double best = 0.0;
  int pick = 0;
  int64_t per_unit = 0;  // of a small pick
  auto offer = [&](int tile, double cost) {
    if (pick == 0 || cost < best) {
      best = cost;
      pick = tile;
    }
  };
  // Large tiles: the narrower ones win where the 256 x 256 grid leaves its
  // last round mostly empty (N = 6144: 384 tiles = 1.5 rounds, against 512
  // tiles of 256 x 192 = 2 rounds of 0.89; N = 14336: 896 tiles = 3.5 rounds,
  // against 1024 of 256 x 224 = 4 of 0.98).
  auto large = [&](int tile, int64_t bm, int64_t bn, double rel) {
    const int64_t n = tiles(bm, bn), rounds = (n + cus - 1) / cus;
    const double f = (g.out == 2 && rounds > 1 ? kLargeF2 : kLargeF[g.out]) + (scalar ? kLargeScalar[g.out] : 0.0);
    offer(tile, rel * double(rounds) * (f + T * (4 * n <= cus ? 1.0 : 1.2)));
  };
  large(kTile256x256, 256, 256, 1.0);
  large(kTile256x224, 256, 224, kCost224);
  large(kTile256x192, 256, 192, kCost256x192);
  large(kTile192x256, 192, 256, kCost192x256);
  for (const SmallTile &t : kSmall) {
    const int64_t c = (tiles(t.bm, t.bn) + cus - 1) / cus;
    const bool deep = t.deep != 0 && c == 1;
    const int tile = deep ? t.deep : t.tile;
    offer(tile, t.f + double(c) * (T * (deep ? t.s_deep : t.s + t.s_k * T) + t.e[g.out] + (scalar ? t.scalar : 0.0)));
    if (pick == tile) per_unit = c;
  }
  const bool wide_pitch = g.ldc * cbytes % kWidePitch == 0;
  if (pick >= kTile64x64 && per_unit > kFewTiles && !scalar && (wide_pitch || g.k > kShortK)) {
    pick = 0;
    for (const ManyRounds &t : kManyRounds) {
      const int64_t n = tiles(t.bm, t.bn);
      const double round = T * (t.s + t.k * T) + t.e[g.out] + (wide_pitch ? t.p[g.out] : 0.0);
      offer(t.tile, t.f + double((n + cus - 1) / cus) * round + double(n) / double(cus) * T * t.q);
    }
  }
  return pick >= kTile64x64 ? launch_gemm_ring(pick, g, s, u) : launch_gemm_large(pick, g, s, u);
}

void set_gemm_tile_override(int tile) { g_tile_override.store(tile, std::memory_order_relaxed); }

}  // namespace qe
