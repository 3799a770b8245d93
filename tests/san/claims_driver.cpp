// The claims that settle a draw without replacement (csrc/sampler_claims.hpp), run on the host with few bits for
// the attempt, against the sequential rule: every slot in turn takes its first attempt that no slot before it holds.
// Slots are settled in a random order, and by threads that give way to each other between a draw and its claim.
#define __host__
#define __device__
#define __forceinline__ inline

#include "sampler_claims.hpp"

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <thread>
#include <vector>

using spo::kNoOwner;

struct Trial {
    uint32_t N, B, max_attempts;
    std::vector<int32_t> table;  // candidate of attempt n of slot k at k * max_attempts + n
    int32_t draw(uint32_t k, uint32_t n) const {
        if (n >= max_attempts) {  // a slot never stands on an attempt that it may not make
            std::fprintf(stderr, "attempt %u of slot %u drawn, bound %u\n", n, k, max_attempts);
            std::abort();
        }
        return table[size_t(k) * max_attempts + n];
    }
};

template <int Bits>
static uint64_t run(std::mt19937 &rng, bool threads) {
    typedef spo::Claims<Bits> C;
    auto upto = [&](uint32_t n) { return rng() % n + 1; };
    Trial t;
    t.N = upto(24);
    t.B = upto(std::min<uint32_t>(t.N, C::kMaxSlots));
    t.max_attempts = upto(60);
    t.table.resize(size_t(t.B) * t.max_attempts);
    const uint32_t skew = upto(4);  // some prompts much more likely than others
    for (auto &c : t.table) {
        c = static_cast<int32_t>(rng() % t.N);
        for (uint32_t i = 1; i < skew; ++i) c = std::min<int32_t>(c, static_cast<int32_t>(rng() % t.N));
    }
    // the rule
    std::vector<int32_t> want(t.B, -1), holder(t.N, -1);
    uint32_t want_most = 0;
    uint64_t saturated = 0;
    for (uint32_t k = 0; k < t.B; ++k) {
        uint32_t n = 0;
        while (n < t.max_attempts && holder[t.draw(k, n)] >= 0) ++n;
        if (n < t.max_attempts) {
            want[k] = t.draw(k, n);
            holder[want[k]] = static_cast<int32_t>(k);
        }
        want_most = std::max(want_most, n);
        saturated += n > C::kMost;
    }
    // the claims
    std::unique_ptr<std::atomic<int32_t>[]> owner(new std::atomic<int32_t>[t.N]);
    for (uint32_t c = 0; c < t.N; ++c) owner[c] = kNoOwner;
    std::vector<std::atomic<int32_t>> failed(t.B);
    for (auto &f : failed) f = 0;
    std::atomic<uint32_t> most{0};
    // claims of a prompt as they were, for looks that see the past
    std::vector<std::unique_ptr<std::atomic<int32_t>[]>> past(2);
    for (auto &p : past) {
        p.reset(new std::atomic<int32_t>[t.N]);
        for (uint32_t c = 0; c < t.N; ++c) p[c] = kNoOwner;
    }
    const bool current = rng() % 2;  // looks see the claims as they are, or some as they were
    std::atomic<uint32_t> wasted{0};  // late claims that a look would have spared
    auto settle = [&](uint32_t k) {
        const uint32_t m = C::settle(
            k, t.max_attempts, [&](uint32_t s, uint32_t n) { return t.draw(s, n); },
            [&](int32_t c) {
                if (threads) std::this_thread::yield();
                const uint32_t how = (k + c) % 3;
                return !current && how ? past[how - 1][c].load() : owner[c].load();
            },
            [&](int32_t c, int32_t v) {
                if (threads) std::this_thread::yield();
                int32_t was = owner[c].load();
                wasted += was < v && (static_cast<uint32_t>(v) & ((1u << Bits) - 1)) >= C::kLookFirst;
                past[1][c] = past[0][c].load();
                past[0][c] = was;
                while (!owner[c].compare_exchange_weak(was, std::min(was, v))) {}
                return was;
            },
            [&](uint32_t s) { failed[s] += 1; });
        uint32_t was = most.load();
        while (was < m && !most.compare_exchange_weak(was, m)) {}
    };
    std::vector<uint32_t> order(t.B);
    for (uint32_t k = 0; k < t.B; ++k) order[k] = k;
    std::shuffle(order.begin(), order.end(), rng);
    if (threads) {
        std::vector<std::thread> th;
        for (uint32_t k : order) th.emplace_back(settle, k);
        for (auto &x : th) x.join();
    } else {
        for (uint32_t k : order) settle(k);
    }
    std::vector<int32_t> got(t.B, -1);
    for (uint32_t c = 0; c < t.N; ++c)
        if (owner[c] != kNoOwner) got[C::slot(owner[c])] = static_cast<int32_t>(c);
    for (uint32_t k = 0; k < t.B; ++k)
        if (got[k] != want[k] || failed[k] != (want[k] < 0 ? 1 : 0)) {
            std::fprintf(stderr, "bits %d N %u B %u attempts %u threads %d: slot %u got %d, rule %d, failed %d\n", Bits, t.N, t.B,
                         t.max_attempts, threads, k, got[k], want[k], failed[k].load());
            std::exit(1);
        }
    if (most != want_most) {
        std::fprintf(stderr, "bits %d: highest attempt %u, rule %u\n", Bits, most.load(), want_most);
        std::exit(1);
    }
    if (current && !threads && wasted) {
        std::fprintf(stderr, "bits %d: %u claims from attempt %u on where a lower one stands\n", Bits, wasted.load(), C::kLookFirst);
        std::exit(1);
    }
    return saturated;
}

int main() {
    std::mt19937 rng(20250913);
    uint64_t saturated = 0;
    for (int i = 0; i < 20000; ++i) saturated += run<2>(rng, false) + run<3>(rng, false) + run<17>(rng, false);
    for (int i = 0; i < 200; ++i) saturated += run<2>(rng, true) + run<3>(rng, true) + run<17>(rng, true);
    if (saturated < 1000) {
        std::fprintf(stderr, "only %llu slots went past the attempts that a claim can say\n", static_cast<unsigned long long>(saturated));
        return 1;
    }
    std::printf("claims follow the sequential rule (%llu slots past the attempts a claim can say)\n",
                static_cast<unsigned long long>(saturated));
    return 0;
}
