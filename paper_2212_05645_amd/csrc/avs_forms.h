// Which form the target and the interface stage of a step take: a lane per
// cell or face (k_target_lanes, k_face_lanes), its leaves in one or more
// shares, or a workgroup per cell (k_target) or per four faces (k_face_eq).
// Functions of the sizes alone, so that a case takes the same form, and the
// same order of summation, alone and in a batch.  Plain C++.
#pragma once

#include <cstddef>
#include <cstdint>

namespace avs {

constexpr int LANE_WAVES = 16;              // waves of a 64-lane workgroup
constexpr size_t LANE_LDS = 144 * 1024;     // its tables' room, of 160 KiB per CU
constexpr int LANE_SHARES = 16;             // most leaf shares

template <int D, typename R>
constexpr size_t lane_tab_bytes(int numax) { return (size_t)D * numax * 64 * sizeof(R); }

// True when the 64-lane form's tables fit (numax up to 144 in FP64 2-D, 288
// in FP32 2-D, 192 in FP32 3-D).
template <int D, typename R>
inline bool lane_form(int numax) { return lane_tab_bytes<D, R>(numax) <= LANE_LDS; }

// Dynamic LDS: the tables, later the waves' partial sums (nacc doubles per
// lane from half of the waves).
template <int D, typename R>
inline size_t lane_lds(int numax, int nacc) {
  const size_t t = lane_tab_bytes<D, R>(numax), r = (size_t)(LANE_WAVES / 2) * nacc * 64 * sizeof(double);
  return t > r ? t : r;
}

// What a stage costs, us on a chip of 256 CUs; the costs of a leaf and of a
// table entry are per 1000 of them.
struct StageCost {
  int per;                          // cells or faces of a workgroup of the workgroup form
  double base, round, leaf, lat;    // workgroup form: launches and serial part, a workgroup in its CU's
                                    // turn, a leaf of one of its cells or faces, a leaf of the longest chain
  double lround, lleaf;             // 64-lane form: a workgroup in its CU's turn, a leaf
};
constexpr StageCost TARGET_COST[2] = {{1, 10.5, 0.90, 0.35, 0.45, 4.2, 22.0},     // 2-D
                                      {1, 13.0, 1.20, 0.48, 0.10, 5.0, 24.4}};    // 3-D
constexpr StageCost FACE_COST[2] = {{4, 3.8, 2.40, 0.26, 0.45, 3.8, 16.8},        // FP64
                                    {4, 5.0, 1.85, 0.21, 0.60, 4.2, 13.8}};       // FP32
template <int D>
constexpr const StageCost& target_cost() { return TARGET_COST[D - 2]; }
template <typename R>
constexpr const StageCost& face_cost() { return FACE_COST[sizeof(R) == 4]; }
constexpr double GROUP_TAB = 3.7, LANE_TAB = 16.5;       // a workgroup's exponential tables
constexpr double CLOSE_BASE = 3.3, CLOSE_SHARE = 0.4;    // the launch that adds several shares
constexpr double SHARED_WORK = 3.0;                      // weight of the work beside the time alone
constexpr double LANE_MARGIN = 3.0;                      // what the lanes have to gain

// Cost of a stage of `count` cells or faces in the 64-lane form with `shares`
// leaf shares, in the workgroup form for 0: its time alone, whole turns of the
// CUs, and its work, the same turns without rounding up.
inline double stage_cost(const StageCost& c, int D, int count, int nleaf, int numax, int shares) {
  if (shares == 0) {
    const int64_t n = ((int64_t)count + c.per - 1) / c.per;
    const double one = c.round + c.leaf * c.per * nleaf / 1000;
    return c.base + (double)((n + 255) / 256) * one + (c.lat * nleaf + GROUP_TAB * D * numax) / 1000 +
           SHARED_WORK * one * (double)n / 256;
  }
  const int64_t n = ((int64_t)count + 63) / 64 * shares;
  const double one = c.lround + (c.lleaf * nleaf / shares + LANE_TAB * D * numax) / 1000;
  return LANE_MARGIN + ((double)((n + 255) / 256) + SHARED_WORK * (double)n / 256) * one +
         (shares > 1 ? CLOSE_BASE + CLOSE_SHARE * shares : 0.0);
}

// Leaf shares of the 64-lane form for `count` cells or faces, 0 where the
// workgroup form is taken: the one of least cost.  The lanes do less work per
// leaf, but a launch has only ceil(count / 64) groups of them: with few groups
// most CUs idle and each wave walks a sixteenth of the leaves, so the leaves are
// split over `shares` workgroups per group, each with tables of its own, whose
// sums another launch adds.
// The constants are a least-squares fit to a sweep of whole steps, 508 sizes x
// 9 forms of either stage (32 to 36 864 cells, 76 to 19 972 leaves, 20 to 288
// table entries, 2-D and 3-D, FP64 and FP32), and to the stages' own times at 85
// of the larger sizes x 4 forms.  Whole steps, us, workgroup form / lanes with 1,
// 2, 4 and 8 shares:
//   target     600 cells x 1498 leaves, 256 entries, FP32     66 /  95  83  76  73
//             3584 x 1498, 256, FP32                         161 / 174 162 157 170
//             7000 x 1498, 256, FP32                         286 / 283 272 286 309
//            16384 x 256, 32, FP64                           362 / 295 303 315 337
//   interface 1836 faces x 1498, 256, FP32                    73 /  93  87  83  82
//             7232 x 1498, 256, FP32                         161 / 166 162 175 201
//            14100 x 1498, 256, FP32                         285 / 273 287 313 349
//            33024 x 256, 32, FP64                           361 / 301 314 330 369
// A case takes the same form in a batch, where other cases use what it leaves
// idle and only its work counts, which is mostly the lanes' smaller one: so the
// work counts beside the time.  The weight is a compromise.  Steps of 147 single
// cases and of 19 FP32 batches (400 to 7000 cells, 300 to 16 000 leaves, sizes
// drawn at random) against a rule for full chips, the lanes wherever their
// tables fit and the shares' tables stay within twice the leaves' work: with
// weight 0 the single cases are 4.3 % faster and the batches 10.5 % slower on
// average, with 1 4.1 and 7.7 %, with 3 3.0 and 6.0 %, with 6 1.4 and 3.9 %.
// With 3 none of the single cases is more than 5 % slower than by that rule, and
// those it had made up to half as slow again (75 to 900 cells x 1500 leaves) are
// back at the workgroup form; the largest cases take the faster form as by it.
// At most `most` shares (the partial sums' room; one share needs none).
template <int D, typename R>
inline int lane_shares(const StageCost& c, int count, int nleaf, int numax, int64_t most) {
  int best = 0;
  if (!lane_form<D, R>(numax)) return best;
  double least = stage_cost(c, D, count, nleaf, numax, 0);
  for (int s = 1; s <= LANE_SHARES && (s == 1 || s <= most); ++s) {
    const double t = stage_cost(c, D, count, nleaf, numax, s);
    if (t < least) { least = t; best = s; }
  }
  return best;
}

// Exponential tables of a cell in pass C: one per face and the cell's own, of
// at most MAXF = 2 D faces.
template <int D, typename T>
constexpr size_t passC_tab(int numax) { return (size_t)(2 * D + 1) * D * numax * sizeof(T); }
constexpr size_t PASSC_WAVE_TAB = 12 * 1024;

// One wave per cell in pass C instead of four, where the leaves are few, the
// tables small enough for many such workgroups in a CU's LDS, and the cells
// many: a cell's leaves then take four times as long (11 us per 1000 of them),
// which costs more than the set-ups of four cells at once save unless every CU
// has several cells to turn to.  What is saved per turn of 256 cells shrinks
// with the leaves and the tables; least-squares fit to 790 steps in both forms
// (64 to 12 000 cells, 64 to 1536 leaves, 1.3 to 12 KiB of tables), whose
// better form the rule misses by 0.2 % of a step on average.  Whole steps, us,
// four waves / one:
//   FP32 2-D, 798 leaves, 5 KiB    144 cells 47 / 54   1500 73 /  79   3584 112 / 110    12 000 268 / 253
//   FP64 2-D, 298 leaves, 5 KiB    144       41 / 44   1500 66 /  64   3584  99 /  88    12 000 244 / 208
//   FP32 3-D, 1492 leaves, 5 KiB    75       64 / 85   1080 105 / 126  5760 306 / 320
//   FP64 3-D, 148 leaves, 3 KiB     75       42 / 45   1080  62 /  63  5760 177 / 164
template <int D, typename T>
inline bool passC_wave_form(int nc, int nleaf, int numax) {
  const size_t tab = passC_tab<D, T>(numax);
  if (tab > PASSC_WAVE_TAB || nleaf > 1536) return false;
  const double l = nleaf / 1000.0, t = tab / 10240.0, turns = nc / 256.0;
  return sizeof(T) == 4 ? turns * (0.62 + 0.20 * l - 0.46 * t - 0.30 * l * t) > 0.6 + 11.0 * l
                        : turns * (0.94 - 0.25 * l - 0.36 * l * t) > 0.6 + 13.2 * l;
}

// What a step of a case with nleaf leaves takes: leaf shares of the target and
// of the interface stage, one wave per cell in pass C.
struct StepForms {
  int nleaf = -1;
  int target = 0, face = 0;
  bool wave = false;
};

}  // namespace avs
