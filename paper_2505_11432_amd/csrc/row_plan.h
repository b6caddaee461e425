// Tile of the row-segmented grouped GEMMs, dealing of tiles, kernel and tile of the fp32 products (code without HIP: the choices are functions
// of sizes).
//
// The host knows the bound M on the rows and E, not the segments (any segments are correct with any tile), so the choice goes
// by the average: max(E, M / rows-of-a-tile + E / 2) row tiles.
//   FEW, up to 32 rows per expert: the launch is a stream over the weights.  64 x 128 tiles, 256 bytes of every row per
//     k-step in three stages: two stages, 64 KB of weights, in flight per CU instead of 32, four to eight times the tiles to
//     deal out, and quarter-size A tiles.
//   FULL, 256 x 256: the tile for arithmetic, 1.3 times the rate of the next on a filled chip.
//   MID, 128 x 128 in three stages of eight waves: where FULL leaves CUs idle: fewer tiles than CUs, or a second round for
//     a few.  A tile is a quarter of the work in a third of the time.  With a fused epilogue it also exists as two
//     workgroups of four waves per CU (pair): one's products run beside the other's epilogue.  Both are taken from 96 rows per
//     expert on (below, the weights bound them: 8 experts, 64 rows, FC1 of 4096 x 14336 415 alone, 427 in pairs).
// Between FULL and MID the estimated time of the rounds decides, from measured tile times: FULL 13 us + 1.5 per 128-byte
// k-step, MID 6 + 0.58 (0.66 where the weights are read across their rows and only stored; up to 12 % less in long lists of
// tiles), plus the epilogue's share; a split last round costs 18 or 9 us for writing and adding the parts.
// Measured, FC1 + SwiGLU / FC2 without split (us; FULL, MID, FEW), multinomial segments, weights from memory:
//   8 experts, 4096 x 14336:   4 rows 419/314, 299/155, 305/157;   32 rows 455/374, 333/178, 315/156;
//                             64 rows 507/386, 346/178, 372/244;  128 rows 504/371, 479/298, 556/311;  256 rows 617/333, 744/420, -
//   64 experts, 2048 x 1408:  32 rows 194/88, 151/78, 142/73;      64 rows 203/93, 162/85, 165/90;     128 rows 205/96, 209/110, -
//   24 experts, 1040 x 1424:  24 rows 66/40, 53/23, 44/19;         62 rows 70/42, 54/23, 43/31;        191 rows 80/48, 79/40, -;
//                            375 rows 110/45, 109/57, -
//   8 experts, 1024 x 2816:  250 rows 59/59, 51/28, - (35/56, 49/29 where few segments exceed 256);    500 rows 70/73, 73/55, -
// FEW does half the arithmetic per byte of MID and is bound by it once rows gather on few experts, and an average says nothing
// about that.  So it is taken only where it would not be slower than FULL either with all rows on one expert, by the time of
// the rounds again (FEW 5 us + 0.4 per k-step; cut tiles 0.45, 0.6 across weight rows, and 9 us).  Where it is not, MID costs up
// to a tenth more on even segments and keeps within a tenth of FULL on gathered ones.  Forward (FULL, MID, FEW) of
//   256 experts, 2048 x 1408, 8192 rows: even 1057, 892, 820;  Zipf 1.5 940, 865, 894;  on 8 experts 173, 206, 276
//   128 experts, 2048 x 2048, 4096 rows: even 826, 618, 573;   Zipf 1.5 714, 646, 668;  on 8 experts 123, 142, 200
//   16 experts, 4096 x 14336, 512 rows:  even 1348, 1039, 948; Zipf 1.5 1238, 1039, 1065; on 2 experts 213, 264, 329
//   64 experts, 2048 x 1408, 2056 rows (FEW by the rule): even 293, 230, 216; Zipf 1.5 263, 238, 252; on 2 experts 94, 75, 85
#pragma once

namespace moe {

enum class RowTile { FEW, MID, FULL };
// The workgroups of an XCD start in `groups` groups, each `lag` k-steps after the one before (0: all at once)
struct Stagger { int groups = 0, lag = 0; };
// split: the last round's tiles may be cut along K; pair: MID as two workgroups per CU
struct RowPlan { RowTile tile; bool split; bool pair = false; Stagger stagger = {}; };

struct RowKind {
  bool swiglu;          // pairs gate and up columns: N is f, a tile makes half its width
  bool store;           // plain store of the product (the only epilogue whose tiles may be cut)
  bool across;          // the contraction runs across the rows of the weights
};

struct TileCost { double fixed, step, cut_step, cut; };      // us: per tile, per k-step, per k-step of a cut tile, for cutting

inline double rounds_us(double tiles, const TileCost& c, int steps, bool split) {
  const double cus = 256, whole = (double)(long)(tiles / cus), rem = tiles - whole * cus;
  const double tile_us = c.fixed + c.step * steps;
  if (rem < 1) return whole * tile_us;
  double last = tile_us;
  if (split && rem <= cus / 2) {
    const double s = cus / rem < 8 ? (double)(long)(cus / rem) : 8;
    const double cut = c.fixed + c.cut_step * steps / s + c.cut;
    last = cut < last ? cut : last;
  }
  return whole * tile_us + last;
}

// Two workgroups per CU, 512 tiles to a round: us per round, per k-step of one, and the same for up to 256 tiles (one per CU).
// FC1: 16 k-steps 22 us, 24 31, 32 37, 64 68 a round; SwiGLU': 16 33, 32 51, 64 87.
struct PairCost { double fixed, step, half_fixed, half_step; };

inline double pairs_us(double tiles, const PairCost& c, int steps) {
  const double whole = (double)(long)(tiles / 512), rem = tiles - whole * 512;
  const double round_us = c.fixed + c.step * steps, half_us = c.half_fixed + c.half_step * steps;
  return whole * round_us + (rem < 1 ? 0 : rem <= 256 && half_us < round_us ? half_us : round_us);
}

// Groups of workgroups that start one after another (e4m3, see STAGGER in gemm_mfma_dma.h), so that their epilogues do not meet.  A round gains
// 2 to 5 us, from five rounds on, and the last group ends (groups - 1) * lag steps of 1.5 us late: a fixed cost, so that short launches take
// few groups and short tiles lie close.
// FC1 (us, sustained: at once, {4, 1}, {8, 1}, {8, 2}): 32 steps, 4096 x 14336 of 8 experts 512 rows 535, 524, 520, 516; 2048 rows 1769, 1697, 1657,
// 1643; 4096 rows 3380, 3273, 3241, 3229.  16 steps, of 64 experts 2048 x 1408, 2048 rows 920, 866, 836, 835; of 4, 2048 x 14336, 700 rows 229,
// 215, 212, 216.  8 steps, of 16, 1024 x 8192, 1024 rows 475, 448, 420, 426; of 8, 1024 x 14336, 2048 rows 775, 720, 696, 709.  4 steps, 512 x
// 14336, 4096 rows 1208, 1044, 1092, 1205.
inline Stagger fc1_stagger(double tiles, int steps) {
  if (tiles < 5 * 256 || steps < 4) return {};
  return steps < 8 ? Stagger{4, 1} : Stagger{8, steps < 24 ? 1 : 2};
}
// Gradients of M x N, `tiles` of 256 x 256 (us, sustained: at once, {4, 1}, {8, 1}, {8, 3}).  Narrow ones: 4 column tiles leave a group of eight
// without a common panel.  Tall ones of many steps gain nothing.
//   d_w2, 4 steps, 8 experts, 4096 x 14336 598, 503, 532, 539;  8 802, 715, 700, 698;  16 1166, 1088, 1075, 1095;  32 1880, 1804, 1806, 1797
//   d_w1 of these                          1264, 1244, 1182, 1158;  1623, 1625, 1571, 1541;  2332, 2332, 2316, 2300;  3739, 3838, 3818, 3824
//   16 steps, 8 experts, d_w2, d_w1 of 2048 x 8192 326, 316, 324, 360; 646, 636, 640, 688;  of 1024 x 14336 292, 282, 276, 275; 596, 593, 623, 647
//   16 steps, 64 experts, 2048 x 1408 486, 472, 471, 481; 985, 935, 929, 942;  4 steps 241, 226, 225, 237; 517, 487, 494, 497
//   8 steps, 16 experts, 1024 x 8192 231, 220, 222, 234; 460, 452, 485, 514;  32 experts, 1024 x 4096 235, 229, 242, 245; 489, 465, 492, 520
//   12 steps, 8 experts, 4096 x 4096 273, 262, 259, 282; 626, 523, 509, 538;  6 steps, 4 experts, 2048 x 14336 155, 145, 147, 169; 343, 350, 322, 344
inline Stagger wgrad_stagger(int M, int N, long tiles, int steps) {
  if (tiles < 5 * 256 || steps < 4 || (steps >= 28 && M > N)) return {};
  return {tiles >= 10 * 256 && N >= 2048 ? 8 : 4, 1};
}

// N: output columns (SwiGLU: f); K in elements of esz bytes
inline RowPlan plan_rows(RowKind kind, int M, int E, int N, int K, int esz) {
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  const long rows = (long)M / E;
  const int steps = (int)up((long)K * esz, 128);
  // Cutting pays from here on: the steps it takes off the last round against the parts' way through memory and a launch
  // (8 experts, 52 to 104 tiles of 256 x 256: 16 steps -2 to -4 us, 22 steps 0, 32 steps +4 to +9, 64 steps +23 to +37).
  const bool split_few = kind.store && steps >= 16, split_full = kind.store && steps >= 28, split_mid = kind.store && steps >= 40;
  const int shrink = kind.swiglu ? 2 : 1;
  auto even = [&](int bm, int bn) {
    const double mt = (double)M / bm + 0.5 * E;
    return (mt > E ? mt : E) * up(N, bn / shrink);
  };
  auto gathered = [&](int bm, int bn) { return (double)(up(M, bm) * up(N, bn / shrink)); };
  const double epi = kind.store ? 0 : kind.swiglu ? 2 : 15;        // over the plain store of a FULL tile
  // FC1 with one row tile per expert: nobody shares a weight panel and the FULL step waits for memory
  const TileCost full = {13 + epi, kind.swiglu && rows < 192 ? 1.8 : 1.5, 1.7, 18};
  const double mid_step = kind.store && kind.across ? 0.66 : 0.58;
  const TileCost mid = {6 + epi / 3, mid_step, mid_step, 9};
  const TileCost few = {5 + epi / 8, 0.4, kind.across ? 0.6 : 0.45, 9};
  if (rows <= 32 && rounds_us(gathered(64, 128), few, steps, split_few) <= rounds_us(gathered(256, 256), full, steps, split_full))
    return {RowTile::FEW, split_few};
  const double full_us = rounds_us(even(256, 256), full, steps, split_full), mid_us = rounds_us(even(128, 128), mid, steps, split_mid);
  if (!kind.store && rows >= 96 && steps <= 48) {
    const PairCost pair = kind.swiglu ? PairCost{7, 0.95, 5, 0.6} : PairCost{15.4, 1.12, 11, 0.6};
    const double pair_us = pairs_us(even(128, 128), pair, steps);
    if (pair_us < full_us && pair_us < mid_us) return {RowTile::MID, false, true};
  }
  if (mid_us < full_us) return {RowTile::MID, split_mid};
  return {RowTile::FULL, split_full, false, kind.swiglu && esz == 1 ? fc1_stagger(even(256, 256), steps) : Stagger{}};
}

// How a launch's last round is dealt.  The tile list goes to the eight XCDs in windows, one tile per CU; `left` of its `items` tiles are
// still to come, and every XCD gets so many consecutive ones.  A partly filled round as whole windows keeps some XCDs idle, and an
// XCD alone reaches 1.3 of the chip's 6 TB/s; dealt evenly, neighbouring tiles land on different XCDs and no longer share panels in an L2.
// The first counts where the last round is much of the launch, up to three rounds (of pairs four), the second in longer lists.
// Measured (us, whole windows and evenly; rounds): weight gradients of 8 experts, 250 rows, 1024 x 2816 1.4 37.1, 29.1, 2.8 55.6, 52.1; of 24
// experts, 100 rows, 3072 x 2400 11.3 152.4, 157.2, 22.5 294.7, 299.6; of 32 experts, Zipf 0.8, 2944 x 2192 13.5 185.5, 191.9; SwiGLU' of
// 12 experts, 3072 x 4096 0.75 97.1, 90.9, of 32, Zipf 1.2 3.1 143.0, 146.1; FC1 in pairs 2.3 262, 247, 3.8 179.7, 175.3.
constexpr int tiles_per_xcd(int items, int left, int window, bool pair) {
  const int even = (left + 7) / 8;
  return items < (pair ? 4 : 3) * 8 * window && even < window ? even : window;
}

// The weight gradients on 128 x 128 tiles, two workgroups per CU, instead of 256 x 256: where the large tile leaves CUs idle in
// its last (or only) round.  A segment is taken as the average one.  Measured, d_w2 / d_w1 (us, 256 x 256 and pairs):
//   8 experts, 512 rows, 512 x 512 20.2/21.4, 11.0/12.5;  250 rows, 1024 x 2816 29.6/57.4, 32.2/64.4;
//   750 rows, 1024 x 1024 28.1/33.5, 21.5/37.2;  1024 rows, 1024 x 2816 69/118, 65/130;  2048 rows, 4096 x 14336 1827/3462, 2327/5738
inline bool wgrad_in_pairs(int rows, int E, int M, int N) {
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  const int steps = (int)up(rows, 64L * E);
  const double large = (double)E * up(M, 256) * up(N, 256), small = (double)E * up(M, 128) * up(N, 128);
  const double rounds = (double)up((long)large, 256);
  return pairs_us(small, {11, 0.75, 6, 0.8}, steps) < rounds * (9.5 + 1.5 * steps) + 6.5 * large / 256;
}

// ---- fp32 expert products (gemm_f32_split.hip): the split into bf16 parts or the fp32 instruction, 64 x 64 or 128 x 128 tiles.
constexpr int kF32SplitStep = 32;        // contraction per step
struct F32Product { bool rows; int M, N, K, E; };      // rows: the segments lie along M (forward, dgrad), else along K (weight gradients)

// Tiles of 64 x 64 (three workgroups per CU) that the average segment makes
inline double f32_tiles64(const F32Product& p) {
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  return (double)up(p.N, 64) * (p.rows ? up(p.M, 64) + p.E / 2 : (double)up(p.M, 64) * p.E);
}

// Where the split is the faster way: from 192 tiles of 64 x 64 on (us, fp32 instruction and split: 216 tiles, K = 768 21.6, 18.2; 256,
// K = 512 16.8, 13.9; 160, K = 1024 19.0, 25.2; 128, K = 2816 28, 52: few tiles are one chain of steps per CU, which the 32 x 32 tiles of the
// fp32 kernel shorten), and for weight gradients of segments longer than one step (1536 tiles of 50 rows 15.8, 16.0; 11264 of 250
// 231, 192; 11264 of 25 58, 67).
inline bool f32_split_pays(const F32Product& p) { return f32_tiles64(p) >= 192 && (p.rows || p.K > (long)kF32SplitStep * p.E); }

// 128 x 128 tiles (four waves, two workgroups per CU, an element split half as often) instead of 64 x 64 (three per CU): where they give
// most CUs both, by the estimated time.  64 x 64 0.9 us + 0.5 per step for every tile of a CU; 128 x 128, up to 512 at a time, 6 us + 1.7 to
// 3.3 per step, by how many of them there are.
inline double f32_us64(double tiles, int steps) {
  const double per_cu = (double)(((long)tiles + 255) / 256), step = 0.5 * per_cu;
  return 0.9 * per_cu + (step > 0.7 ? step : 0.7) * steps;
}
inline double f32_us128(double tiles, int steps) {
  const long whole = (long)tiles / 512;
  const double rest = tiles - whole * 512.0;
  const double rate = rest <= 256 ? 1.7 + 0.3 * rest / 256 : 2.45 + 0.9 * (rest - 256) / 256;
  return whole * (6 + 3.35 * steps) + (rest < 1 ? 0 : 6 + rate * steps);
}
inline double f32_tiles128(const F32Product& p) {
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  const double mt = p.rows ? p.M / 128.0 + p.E / 2 : (double)up(p.M, 128) * p.E;
  return up(p.N, 128) * mt;
}
inline int f32_steps(const F32Product& p) {
  const int k = p.rows ? p.K : p.K / p.E;
  return (k + kF32SplitStep - 1) / kF32SplitStep;
}
// Tiles of b x b that row segments within a tenth of the average make.  Balanced routing leaves that much, and a last round is made or missed by it:
// 8 segments of 145 rows are 16 row tiles of 128, 13 by the half tile per segment that the other counts take.
inline double f32_tiles_near(const F32Product& p, int b) {
  const double mean = (double)p.M / p.E;
  auto sum = [&](double x) {                    // of the tiles of segments up to x rows long
    const long k = (long)(x / b);
    return b * (k * (k + 1) / 2.0) + (k + 1) * (x - (double)k * b);
  };
  return (p.N + b - 1) / b * p.E * (sum(1.1 * mean) - sum(0.9 * mean)) / (0.2 * mean);
}
// The larger tile has to be the faster one by both counts (8 experts, 1161 rows, FC1 of 528 x 2176, 444 and 544 tiles: 74.2 us, 64 x 64 56.6), and
// there have to be more than three tiles for every two CUs (d_w1 of 384: 1.04 of the time on 64 x 64, of 390 and 392: 0.85 and 0.87).
inline bool f32_split_in_128(const F32Product& p) {
  const int steps = f32_steps(p);
  const double tiles = f32_tiles128(p);
  if (tiles <= 1.5 * 256 || f32_us128(tiles, steps) >= f32_us64(f32_tiles64(p), steps)) return false;
  return !p.rows || f32_us128(f32_tiles_near(p, 128), steps) < f32_us64(f32_tiles_near(p, 64), steps);
}

// One round of 128 x 128 tiles by eight waves with two stages, 3.5 us + 1.33 per step: alone on a CU they beat four waves with one.  Weight
// gradients of 256 such tiles (us, 64 x 64, four waves, eight): 10 steps 26.1, -, 22.1; 16 steps -, 37.3, 31.4; 24 steps -, 50.5, 42.8; 4 steps 14.6, -, 13.4.
inline double f32_us_eight(int steps) { return 3.5 + 1.33 * steps; }
inline bool f32_split_in_eight(const F32Product& p) {
  const int steps = f32_steps(p);
  return steps >= 4 && f32_tiles128(p) <= 256 && f32_us_eight(steps) < f32_tiles64(p) / 256 * (0.85 + 0.445 * steps);
}

enum F32Shape { F32_64, F32_128, F32_128_EIGHT };
struct F32Plan { F32Shape tile; int parts; };      // parts along K
// With scratch for `room` results a product of row segments may be cut into up to that many parts (at most 6), which a kernel of its own adds:
// 4 us and 1 per 8 MB.  FC2 and dgrad1 have few tiles and long contractions.  Measured (us with the addition, whole on 64 x 64 and cut): 8
// experts, 1024 x 2816, 2000 rows FC2 138, 113 (128 x 128 in 3), dgrad1 288, 196 (in 3; in 2 247, in 5 223); 512 rows 62, 53 (64 x 64 in 4), 139, 104.
// Parts fill a round or just miss it, and then a cut costs as much as it gains elsewhere: 16 experts, 2008 rows, 784 x 1424 FC2 1.62 of the time
// whole, dgrad1 1.34.  So the tiles of a cut are counted by the half tile per segment and by f32_tiles_near, and the higher count goes, with 3 % more of
// the small and 6 % more of the large ones (XCDs fill unevenly), against the whole product by f32_tiles_near.  Over 680 shapes (300 to 4500 rows, 1 to
// 32 experts, even and skewed, widths of 384 to 2816) FC2 then takes 0.976 and dgrad1 0.907 of the time whole on 64 x 64 or eight waves, 11 of 1360 more
// than 1.03 and the worst 1.15; by the first count alone 0.978 and 0.898, but 50 more than 1.03 and the worst 1.62.
inline F32Plan f32_plan(const F32Product& p, long room) {
  const F32Plan whole = {f32_split_in_128(p) ? F32_128 : f32_split_in_eight(p) ? F32_128_EIGHT : F32_64, 1};
  if (!p.rows || room < 2) return whole;
  const int steps = f32_steps(p);
  const double t64 = f32_tiles64(p), t128 = f32_tiles128(p), near64 = f32_tiles_near(p, 64), near128 = f32_tiles_near(p, 128);
  const double whole_us = whole.tile == F32_128 ? f32_us128(t128, steps) : whole.tile == F32_128_EIGHT ? f32_us_eight(steps) : f32_us64(near64, steps);
  const double cut64 = 1.03 * (near64 > t64 ? near64 : t64), cut128 = 1.06 * (near128 > t128 ? near128 : t128);
  F32Plan best = whole;
  double best_us = 0.95 * whole_us;
  for (int n = 2; n <= (room < 6 ? room : 6) && steps / n >= 8; ++n) {
    const int each = (steps + n - 1) / n;
    const double add = 4 + (n + 1.0) * p.M * p.N * 4 / 8e6;
    const double us64 = f32_us64(cut64 * n, each) + add, us128 = f32_us128(cut128 * n, each) + add;
    const double us = us128 < us64 ? us128 : us64;
    if (us < best_us) {
      best_us = us;
      best = {us128 < us64 ? F32_128 : F32_64, n};
    }
  }
  return best;
}

}  // namespace moe
