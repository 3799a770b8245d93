// Large or small tiles for a contraction, and how a launch of tiles is cut: sizes alone decide, so this runs on any host.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace spo {

constexpr int kChipCUs = 256;
constexpr int kLargeEdge = 256, kSmallEdge = 128;  // tiles; a compute unit holds one large or two small ones
constexpr int kStep = 64;                          // contraction elements per step
static inline int64_t tile_edge(bool small) { return small ? kSmallEdge : kLargeEdge; }
static inline int tile_slots(bool small) { return small ? 2 * kChipCUs : kChipCUs; }
static inline int64_t tiles_over(int64_t n, bool small) { return (n + tile_edge(small) - 1) / tile_edge(small); }

// A launch ends in a partly filled round of tiles when its tile count is no multiple of the chip's
// compute units.  A short last round (at most half of the units busy) is cut off: the tiles
// before it run as they are, in whole rounds, and the `rem` tiles after them are each cut along the
// contraction into `parts` runs whose partial results are added in a fixed order afterwards.  Host
// and device code ask the same function, so the number of tiles may be known on the device only.
// Tiles count in the order in which they are launched (TileOrder): the tiles that run are then whole rounds.  (Counted
// row by row, the tiles left out were spread over the last patches, and where a band of patches is no divisor of a
// round the rest took a round more: dHidden of 5000 x 3648 x 151936, 256 + 44 tiles, 6667 us, half of that now.)
// k_steps: the contraction's length before it is limited on the device.  The steps that a cut saves have to be worth its
// two launches and the parts' way through memory, 19 us together (a step of small tiles takes about half as long).
constexpr int kCutSteps = 12;
struct TailCut {
    int64_t whole;  // tiles that run in whole rounds (all of them when nothing is cut)
    int rem, parts;
    __host__ __device__ __forceinline__ TailCut(int64_t tiles, int64_t k_steps, int slots) : whole(tiles), rem(0), parts(1) {
        const int r = static_cast<int>(tiles % slots);
        const int most = r > 0 ? (slots / r < 8 ? slots / r : 8) : 1;
        if (most > 1 && (k_steps - k_steps / most) * kChipCUs >= kCutSteps * slots) {
            whole = tiles - r;
            rem = r;
            parts = most;
        }
    }
};

// Parts that the contraction of dHidden over the vocabulary is cut into, for a chunk of Tc tokens: its
// (Tc / 256) * ceil(H / 256) tiles leave more than a quarter of the chip idle.  A part takes some 1.4 us per
// step of 64 entries and adds its tile to what reduce_split_kernel reads (64 MB for a chip full of parts,
// 15 us): up to eight parts in any case, more while a part keeps kPartSteps steps.  (Loss then gradients
// of 17 tokens at 896 x 151936, 4 tiles, 2374 steps: 948 us in 8 parts, 642 in 64; of 85 tokens at
// 3264 x 15635, 13 tiles, 245 steps: 19 parts gain what 8 leave of the chip idle.)
constexpr int64_t kPartSteps = 16;
static inline int dhidden_parts(int64_t Tc, int64_t H, int64_t V_pad, bool small) {
    const int64_t tiles = tiles_over(Tc, small) * tiles_over(H, small), slots = tile_slots(small);
    if (tiles * 4 >= slots * 3) return 1;
    return static_cast<int>(std::min<int64_t>(slots / tiles, std::max<int64_t>(8, V_pad / kStep / kPartSteps)));
}

// Small or large tiles?  A launch takes about
//   rounds of workgroups on the chip x (steps of a tile x time of a step + time of a tile's ends) + the rest, in us.
// Up to kChipCUs small tiles have a compute unit each, above two share one.  Two that share one read twice the bytes per
// product of a large tile, so what a step of theirs takes depends on where the operands come from:
//   the sweep  0.85 us with the head in the L2s, 0.90 from beyond;
//   dHidden    0.6 to 0.7 with both operands in the Infinity Cache (256 MB), 0.95 to 1.2 from memory;
//   dW         0.75 up to 96 MB of operands, 0.95 to 1.1 beyond; 1.5 (large tiles 1.8) where all are cut into 3, 5, 6 or 7 parts: the
//              parts of a tile then fall on every XCD and each L2 fetches all of both operands.
// Measured both ways on 214 shapes of 300 to 60000 tokens, H = 128 to 2112, V = 1000 to 151936.  What this chooses is behind the
// better of the two by 0.5 % on average (large tiles always: 18 % for dW), and slower than large tiles by 8 % at most.  With
// the head's bytes alone to go by, and steps fitted up to 8000 tokens, it was 2.1 and 1.3 % behind (dW, dHidden)
// and up to 47 % slower than large tiles: dW of 20000 tokens at 896 x 3000 128 us on large tiles, 189 on small, of 25000 at
// 640 x 9000 323 and 437; dHidden of 9000 at 640 x 17592 229 and 311.  (Loss and gradients of 512 fp32 tokens at 128 x 1000:
// 97 us on large tiles, 68 on small; 31 bf16 tokens at 1024 x 151936 438 and 381; 4000 at 4096 x 30000 2406 and 2875.)
struct TileTimes {
    double step, ends;             // large tiles
    double lone, near, far;        // a step of small ones: with a compute unit to itself, two on it with operands of up to near_bytes, beyond
    double ends_s;
    double rest, rest_s, cut;      // of a launch, large and small; a cut tail
    double odd, odd_s;             // a step, large and small, where all tiles are cut into a number of parts that is no divisor of eight (0: the same)
    int64_t near_bytes;
    double ahead;                  // see small_is_faster
};
constexpr TileTimes kSweepTimes{1.30, 8.3, 0.57, 0.85, 0.90, 4.4, 4.6, 5.1, 0.0, 0.0, 0.0, int64_t(32) << 20, 0.875};
constexpr TileTimes kDHiddenTimes{1.60, 4.6, 0.34, 0.70, 1.10, 0.0, 17.0, 15.4, 4.1, 0.0, 0.0, int64_t(256) << 20, 0.875};
constexpr TileTimes kDWTimes{1.52, 10.7, 0.60, 0.75, 0.95, 7.0, 3.2, 2.1, 19.0, 1.8, 1.5, int64_t(96) << 20, 0.92};

static inline double launch_time(const TileTimes &t, bool small, double rounds, int64_t wgs, int64_t steps, int64_t bytes, bool odd = false) {
    const double cut = odd ? (small ? t.odd_s : t.odd) : 0.0;
    const double step = cut > 0.0 ? cut : !small ? t.step : wgs <= kChipCUs ? t.lone : bytes <= t.near_bytes ? t.near : t.far;
    return rounds * (static_cast<double>(steps) * step + (small ? t.ends_s : t.ends)) + (small ? t.rest_s : t.rest);
}
// the same of contractions whose short last round may be cut
static inline double launch_time_cut(const TileTimes &t, bool small, int64_t tiles, int64_t steps, bool may_cut, int64_t bytes) {
    const int slots = tile_slots(small);
    const TailCut cut(may_cut ? tiles : 0, steps, slots);
    if (!cut.rem) return launch_time(t, small, static_cast<double>((tiles + slots - 1) / slots), tiles, steps, bytes);
    return launch_time(t, small, static_cast<double>(cut.whole / slots) + 1.0 / cut.parts, cut.whole ? tiles : cut.rem * cut.parts, steps,
                       bytes, !cut.whole && 8 % cut.parts != 0) + t.cut;
}
// Long launches run at the power cap, where the smaller tiles' extra traffic costs more than fitted: they have to be well
// ahead there (dW of 40485 tokens at 512 x 86540: the whole call 11.38 ms on large tiles, 11.97 on small).
static inline bool small_is_faster(const TileTimes &t, const double (&time)[2]) {
    return time[1] < time[0] * (time[0] > 500.0 ? t.ahead : 1.0);
}

static inline bool small_dhidden(int64_t T, int64_t H, int64_t V_pad) {
    // large tiles that fill the chip by themselves: long steps of a vocabulary, where they are faster than fitted (16000
    // tokens at 256 x 40000 343 and 432 us, 17497 at 640 x 35002 767 and 816, 11238 at 192 x 151936 743 and 1098)
    if (dhidden_parts(T, H, V_pad, false) == 1) return false;
    double time[2];
    for (int small = 0; small < 2; ++small) {
        const int64_t parts = dhidden_parts(T, H, V_pad, small), steps = V_pad / kStep;
        time[small] = launch_time_cut(kDHiddenTimes, small, tiles_over(T, small) * tiles_over(H, small) * parts, (steps + parts - 1) / parts,
                                      parts == 1, (T + H) * V_pad * 2);
    }
    return small_is_faster(kDHiddenTimes, time);
}
static inline bool small_dW(int64_t T, int64_t H, int64_t V) {
    double time[2];
    for (int small = 0; small < 2; ++small)
        time[small] = launch_time_cut(kDWTimes, small, tiles_over(V, small) * tiles_over(H, small), (T + kStep - 1) / kStep, true, T * (V + H) * 2);
    return small_is_faster(kDWTimes, time);
}

}  // namespace spo
