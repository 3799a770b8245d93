// Large or small tiles (csrc/tile_choice.hpp): shapes on which both were measured and one is well ahead get that one.
#define __host__
#define __device__
#define __forceinline__ inline

#include "tile_choice.hpp"

#include <cstdio>

struct Shape {
    int64_t T, H, V;
    double large, small;  // us
};

static const Shape dW[] = {
    {20000, 896, 3000, 128.2, 188.8}, {12000, 896, 3000, 83.7, 117.1},    {25000, 640, 9000, 323.2, 436.6},  // operands from memory,
    {32223, 640, 9000, 408.8, 542.3}, {8192, 896, 3000, 66.1, 86.4},      {12000, 192, 86540, 500.9, 612.2},  // parts on every XCD
    {12000, 1664, 9000, 301.9, 365.1}, {32223, 1152, 3000, 220.3, 264.3}, {32223, 896, 17592, 873.9, 961.5},
    {32223, 320, 17592, 691.6, 479.1}, {8192, 640, 3000, 61.2, 45.2},     {713, 896, 40000, 89.6, 78.7},      // large tiles are few,
    {40000, 384, 17592, 871.6, 600.0}, {8192, 1664, 1000, 46.8, 41.6},    {5000, 1664, 3000, 77.1, 66.1}};    // or mostly padding
static const Shape dHidden[] = {
    {9000, 640, 17592, 228.7, 279.4}, {8192, 896, 17592, 242.4, 275.8},  {12000, 320, 40000, 477.4, 581.2},
    {12000, 384, 17592, 230.3, 281.4}, {5000, 384, 86540, 377.7, 426.0}, {713, 896, 151936, 202.6, 235.2},
    {20000, 256, 40000, 411.6, 738.7}, {32223, 256, 1000, 45.3, 22.4},   {300, 640, 9000, 37.2, 22.4},
    {8192, 896, 3000, 63.6, 44.4},    {32223, 192, 3000, 60.9, 43.3},    {12000, 384, 9000, 121.7, 101.3}};

int main() {
    int bad = 0;
    auto look = [&](const char *what, const Shape &s, bool small) {
        if (small == s.small < s.large) return;
        std::fprintf(stderr, "%s of %lld tokens at %lld x %lld on %s tiles: large %.1f us, small %.1f\n", what, (long long)s.T, (long long)s.H,
                     (long long)s.V, small ? "small" : "large", s.large, s.small);
        ++bad;
    };
    for (const Shape &s : dW) look("dW", s, spo::small_dW(s.T, s.H, s.V));
    for (const Shape &s : dHidden) look("dHidden", s, spo::small_dhidden(s.T, s.H, (s.V + 63) / 64 * 64));
    if (bad) return 1;
    std::printf("tiles are the faster ones\n");
    return 0;
}
