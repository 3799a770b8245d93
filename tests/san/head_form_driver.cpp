// Which form of the head is read (csrc/head_form.hpp): the byte offsets that the main loop forms inside a tile, here in 64
// bits, fit its 32 for every head that is read as it was given.
#include "head_form.hpp"

#include <cstdio>
#include <cstdlib>
#include <initializer_list>

int main() {
    const int64_t limit = (int64_t(1) << 32) - 1;
    int64_t taken = 0, copied = 0;
    auto look = [&](int64_t T, int64_t H, int64_t V) {
        if (!spo::direct_head(true, true, T, H, V)) {
            ++copied;
            return false;
        }
        ++taken;
        const int64_t rows = H < 256 ? H : 256;
        const int64_t along = (rows - 1) * 2 * V + 128 - 16;               // dHidden: last piece of a stage, last row
        const int64_t across = 63 * 2 * V + (V < 256 ? V : 256) * 2 - 16;  // the sweep: last piece of the last contraction step
        if (V % 8 || along > limit || across > limit) {
            std::fprintf(stderr, "T %lld H %lld V %lld read as given: offsets %lld and %lld\n", (long long)T, (long long)H, (long long)V,
                         (long long)along, (long long)across);
            std::exit(1);
        }
        return true;
    };
    for (int64_t T : {int64_t(1), int64_t(31), int64_t(256), int64_t(8192)})
        for (int64_t H = 64; H <= 65536; H *= 2)
            for (int64_t half = 8; half < int64_t(1) << 31; half *= 2)
                for (int64_t V : {half, half + 8, half + half / 2, 2 * half - 8})
                    if (V < int64_t(1) << 31) look(T, H, V);
    for (int64_t V = 8000000; V < 9000000; V += 8) look(256, 256, V);
    // the bound does not take the form from heads that fit
    const bool kept = look(256, 256, 8388600) && !look(256, 256, 8500000) && look(31, 64, 33554424) && look(713, 256, 3000);
    if (!kept || spo::direct_head(true, true, 31, 1024, 151937) || spo::direct_head(false, true, 31, 1024, 151936) ||
        !spo::direct_head(true, false, 8192, 1024, 151936) || spo::direct_head(true, false, 8193, 1024, 151936)) {
        std::fprintf(stderr, "forms of the head are not those of the rule\n");
        return 1;
    }
    std::printf("heads read as given fit the offsets (%lld taken, %lld copied)\n", (long long)taken, (long long)copied);
    return 0;
}
