// Tile of the row-segmented grouped GEMMs (host code without HIP: the choice is a function of sizes).
//
// The host knows the bound M on the rows and E, not the segments (any segments are correct with any tile), so the choice goes
// by the average: max(E, M / rows-of-a-tile + E / 2) row tiles.
//   FEW, up to 32 rows per expert: the launch is a stream over the weights.  64 x 128 tiles, 256 bytes of every row per
//     k-step in three stages: two stages, 64 KB of weights, in flight per CU instead of 32, four to eight times the tiles to
//     deal out, and quarter-size A tiles.
//   FULL, 256 x 256: the tile for arithmetic, 1.3 times the rate of the next on a filled chip.
//   MID, 128 x 128 in three stages of eight waves: where FULL leaves CUs idle: fewer tiles than CUs, or a second round for
//     a few.  A tile is a quarter of the work in a third of the time.
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
struct RowPlan { RowTile tile; bool split; };        // split: the last round's tiles may be cut along K

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
  return rounds_us(even(128, 128), mid, steps, split_mid) < rounds_us(even(256, 256), full, steps, split_full)
             ? RowPlan{RowTile::MID, split_mid} : RowPlan{RowTile::FULL, split_full};
}

}  // namespace moe
