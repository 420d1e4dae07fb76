// How massv_linear cuts a call into workgroups: which tile, and over how many ranges of K.  Plain host code, the one plan that the size of the
// workspace and the call itself go by.
#pragma once
#include <cstddef>
#include <cstdint>

namespace massv {

constexpr int kLinTile = 256;            // features and rows of the largest tile

// The tiles of massv_linear, by the number that stands for each in a plan and in a kernel's name, and the coefficients of linear_best's estimate: microseconds
// a 32-wide stage of one, its share of the chip's power, and its two ends.
struct LinShape { int features, rows; double stage, busy, ends; };
constexpr LinShape kLinShapes[5] = {{}, {128, 128, 0.18, 0.203, 1.92}, {256, 128, 0.27, 0.353, 1.75}, {128, 192, 0.261, 0.235, 1.66}, {256, 256, 0.54, 0.625, 1.4}};
constexpr int kLinSquare = 1, kLinFlat = 2, kLinLow = 3, kLinTall = 4;
constexpr int lin_tiles_m(int tile, int M) { return (M + kLinShapes[tile].rows - 1) / kLinShapes[tile].rows; }
constexpr int lin_tiles_n(int tile, int N) { return (N + kLinShapes[tile].features - 1) / kLinShapes[tile].features; }

// One call: its tile and the number of ranges of K.  big: 0, or that many of the tallest tiles followed by halves (linear_mixed_kernel).
struct LinPlan { int tile, parts, big; };

inline int mixed_tiles_m(int M) { return M / kLinTile + (M % kLinTile > kLinTile / 2); }
inline int mixed_halves(int M, int N, int big) {         // (of at most 128 tiles that are left)
    const int tiles_n = (N + 255) / 256, r = M % kLinTile;
    return 2 * (mixed_tiles_m(M) * tiles_n - big) + (r && r <= kLinTile / 2 ? tiles_n : 0);
}
// Whole rounds of the chip by tiles of 256 rows, and the rest, where it is at most half a round, in halves: the last round then takes half as
// long.  1.025 to 1.14 times as fast as the better of the two heights on all of 36 drawn shapes that take it (1 to 10 rounds, 1536 to
// 18944 wide, weights from memory; 1111 x 3584 -> 18944 158 -> 145 us, 16384 x 18944 -> 3584 1755 -> 1673, 6021 x 18944 -> 3584
// 768 -> 673, 10251 x 3840 -> 15360 981 -> 955); with 1.01 to 1.17 rounds of halves left 0.95 to 1.007 times.
// Over 260 shapes drawn since (31 widths, up to 16384 rows) 1.08 times as fast in the median (0.97 to 1.19; 1945 and 2027 x 1536 -> 8960 are the two below 1.0).
// (The estimate, which has the 128-feature tiles besides, is not asked here: against it, over 147 drawn shapes, 0.89 to 1.14 times as fast, 1.06 in the median.)
inline int mixed_big(int M, int N) {
    const int64_t tiles = (int64_t)mixed_tiles_m(M) * ((N + 255) / 256);
    const int big = (int)(tiles / 256 * 256);
    if (!big || tiles - big > 128) return 0;
    const int halves = mixed_halves(M, N, big);
    return halves > 0 && halves <= 256 ? big : 0;
}

// The plan comes from an estimate whose coefficients were fitted to 3000 measured (shape, plan) pairs: 14 widths from 1152 x
// 1152 to 18944 x 3584, 30 to 8000 rows; over those shapes its choice is 1.1 % slower than the best plan in the mean, at worst
// 1.22 times.  It is the larger of three terms:
//   rounds of workgroups x (stages x 0.54 or 0.27 + 1.4 or 1.75 us for the ends of a 256- or 128-row tile);
//   the share of the chip's tile slots that is used x (stages x 0.625 or 0.353 + the ends): the power limit favours the larger
//   tile.  These two are coefficients, not the time of a stage on a full chip, which is 0.80 (8192^3) to 0.90 us (4096 x 3584 ->
//   18944) of a 256-row tile: the fit is over all sizes and is there to order the plans of one size;
//   W at 8.5 TB/s, more than HBM gives (calls of the fit repeat, and the last-level cache holds a part of W);
// and a split adds its finishing launch (3 us) and its partial sums, written and read back at 2.6 TB/s.  The bound of 560
// workgroups ends the search; no plan of those shapes has more.
// What it is for, measured against one 256-row tile per workgroup at full K: 1225 x 5120 -> 5120 100 -> 64 us
// (128-row tiles: 200 workgroups instead of 100), 1111 x 18944 -> 3584 326 -> 148 us (128-row tiles, K in two: 252
// instead of 70), 60 x 18944 -> 3584 330 -> 36 us (K in twelve).
// The square tile came later: its three coefficients are fitted alone, to the choice among all plans of 6756 shapes (17 widths, 30 to 3640
// rows, weights from memory) whose taller plans stayed as they were.  It takes 71 % of them, 1.17 times as fast in the mean there (1 to 64
// workgroups 1.27, 193 to 256 1.13).  1111 x 3584 -> 3584 43.6 -> 32.6 us, 128 x 1536 -> 8960 18.1 -> 13.5, 300 x 3584 -> 3584 23.7 -> 21.0.
// The one of 192 rows in the same way, over 3861 shapes: 16 % take it, 1.07 times as fast in the mean there.  1225 x 5120 -> 3584 62.9 -> 52.2 us,
// 1111 x 3584 -> 4608 48.9 -> 40.7.
// Over 2500 shapes drawn since (31 widths, 17 to 3700 rows, weights from memory) whose plan is another than among the 256-feature tiles: 1.12 times as fast as by those in the median
// (0.86 to 1.46), 0.9 and 1.7 % of them on two cards more than 2 % slower; nearly all of these have up to 64 rows and K in several ranges, where the same shape is faster on one card
// and slower on another (30 x 3840 -> 15360 0.87, the median over such calls 1.03).
// Kinds that lost to the plans of before on the cards they were timed on are estimated higher, and so go back to those (weights from memory, each call 16 times in turn).
//   Many unsplit squares over a long K, by 10 %: 500 calls of 8 widths that this takes from the squares run 0.97 to 1.20 times as fast, 1.07 in the median
//   (1144 x 18944 -> 3584 1.18, 385 to 512 x 5120 -> 5120 1.10, 769 to 1024 x 11008 -> 4096 1.03).
//   Unsplit squares whose last row tile is more than half full, over a long K or fewer than the chip has units, by 25 %.  Rows past the last one cost a tile
//   next to nothing, and the squares' time grows faster with the rows that are there: 4096 -> 6144, three row tiles, by squares and by 256 x 128 with K in three 31.5 and
//   32.4 us with 262 rows, 33.8 and 34.0 with 300, 40.0 and 36.6 with 378; 8192 -> 3072, nine row tiles, K in two 64.7 and 67.0 us with 1065 rows, 76.0 and 70.5 with 1145.
//   Over 700 such calls of 20 widths on three cards 0.97 to 1.25 times as fast as by the squares, 1.05 in the median.
//   192-row tiles in two rounds whose last row tile is so, or over a long K, by 3 % (by the estimate a tie with one round of the tallest): 1900 such calls on four cards run 0.92 to 1.20
//   times as fast by the tallest, 1.05, 0.99, 0.99 and 1.00 in the medians of the cards (2046 x 5120 -> 5120 113 us and by the tallest 105 on the first).
//   192-row tiles with K in two, by 2 %: 270 calls that this gives to 256 x 128 with K in three run 0.97 to 1.10 times as fast, 1.04 in the median; those that are ahead of K in two by
//   256 x 128 (1.02 to 1.16) stay.
inline LinPlan linear_best(int M, int N, int K, size_t room, bool square) {
    const int big = mixed_big(M, N);
    if (big) return {kLinTall, 1, big};
    LinPlan best = {kLinTall, 1, 0};
    double best_t = 1e300;
    for (int tile = kLinTall; tile >= kLinSquare; --tile) {
        const LinShape& s = kLinShapes[tile];
        if (s.features == 128 && !square) continue;
        const int64_t tiles = (int64_t)lin_tiles_m(tile, M) * lin_tiles_n(tile, N);
        if (tile != kLinTall && tiles > (1 << 20)) break;
        for (int parts = 1; parts <= 32 && parts <= K / 64; ++parts) {
            const double bytes = (double)parts * M * N * 4.0;
            if (parts > 1 && (tiles * parts > 560 || bytes > (double)room)) break;
            const int64_t wgs = tiles * parts;
            const double stages = 2.0 * ((K / 64 + parts - 1) / parts);
            double t = (double)((wgs + 255) / 256) * (stages * s.stage + s.ends);
            const double all = (double)wgs / 256.0 * (stages * s.busy + s.ends), stream = (double)N * K * 2.0 / 8.5e6;
            if (all > t) t = all;
            if (stream > t) t = stream;
            const bool full = (M - 1) % s.rows >= s.rows / 2;
            if (tile == kLinSquare && parts == 1 && wgs > 128 && (K > 10000 || (K >= 5120 && wgs <= 160))) t *= 1.1;
            if (tile == kLinSquare && parts == 1 && full && (K > 8000 || (wgs <= (K >= 5120 ? 160 : 152) && M > 128 && K >= 2048 && K >= 24 * wgs))) t *= 1.25;
            if (tile == kLinLow && parts == 1 && wgs <= 512 && (K > 8000 || (full && wgs > 256))) t *= 1.03;
            if (parts > 1) t += 3.0 + bytes / 2.6e6;
            if (tile == kLinLow && parts == 2) t *= 1.02;
            if (t < best_t) { best_t = t; best = {tile, parts, 0}; }
        }
    }
    return best;
}

constexpr size_t kLinAnyRoom = ~(size_t)0;

inline size_t linear_part_bytes(const LinPlan& p, int M, int N) {
    return p.parts > 1 ? ((size_t)p.parts * M * N * sizeof(float) + 255) / 256 * 256 : 0;
}

// Room for partial sums that massv_linear_workspace asks for: what the best plan of the 256-feature tiles takes.  A call uses no more than this,
// however much it is given, so that its plan, and with it every bit of its result, does not go by what the caller's buffer happens to be.
// With all the room they like, the 128-feature tiles of 129 to 192 rows would split K further (18944 -> 3584 in 9 ranges instead of 7) by an estimate that
// flatters them: 0.85 to 1.04 times as fast on 18 drawn shapes of 6 widths, 0.93 in the mean (158 x 10752 -> 4096 34.3 and 40.2 us).
inline size_t linear_asked_room(int M, int N, int K) { return linear_part_bytes(linear_best(M, N, K, kLinAnyRoom, false), M, N); }

// The plan of a call.  (The best one of more room is the best one of less if it fits.)
inline LinPlan linear_plan(int M, int N, int K, size_t room) {
    const LinPlan p = linear_best(M, N, K, room, true);
    if (p.parts == 1) return p;
    const size_t asked = linear_asked_room(M, N, K);
    return linear_part_bytes(p, M, N) <= asked ? p : linear_best(M, N, K, room < asked ? room : asked, true);
}

}  // namespace massv
