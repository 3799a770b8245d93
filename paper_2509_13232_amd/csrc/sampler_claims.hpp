// Successive sampling without replacement as claims on prompts: the part that decides, apart from where the
// draws and the claims live (memory, LDS, or a test on the host).
#pragma once

#include <stdint.h>

namespace spo {

constexpr int32_t kNoOwner = 0x7fffffff;  // no slot has claimed the prompt

// A claim is slot << Bits | attempt, so the one word that decides who holds a candidate also
// says where a displaced slot goes on.  Attempts beyond its bits are filed as the largest; such a slot
// finds its attempt again by repeating its draws from there (it stands on the first of them that gives
// this candidate: it was never turned away here before, or a lower slot would hold it).
template <int Bits>
struct Claims {
    static constexpr uint32_t kMost = (1u << Bits) - 2;           // every claim is below kNoOwner
    static constexpr uint32_t kMaxSlots = 1u << (31 - Bits);

    __host__ __device__ static int32_t filed(uint32_t slot, uint32_t attempt) {
        return static_cast<int32_t>(slot << Bits | (attempt < kMost ? attempt : kMost));
    }
    __host__ __device__ static uint32_t slot(int32_t claim) { return static_cast<uint32_t>(claim) >> Bits; }

    // Settles slot k and the slots displaced on the way; returns the highest attempt reached.
    //   draw(k, n)    candidate of attempt n of slot k
    //   peek(c)       what the claim on c is, or was at any time before
    //   claim(c, v)   atomic minimum of the claim on c and v, returning what was there
    //   fail(k)       slot k has run out of attempts
    // Claims only fall, so a slot that finds a lower one where it looks is turned away for good, without an atomic.
    // From attempt kLookFirst on it looks before it claims: few slots come so far while prompts are free, and where
    // nearly all are taken the atomics of all slots would meet at the same addresses.
    static constexpr uint32_t kLookFirst = 4;
    template <typename Draw, typename Peek, typename Claim, typename Fail>
    __host__ __device__ __forceinline__ static uint32_t settle(uint32_t k, uint32_t max_attempts, Draw draw, Peek peek, Claim claim, Fail fail) {
        uint32_t attempt = 0, most = 0;
        for (;;) {
            most = attempt > most ? attempt : most;
            if (attempt >= max_attempts) {
                fail(k);
                return most;
            }
            const int32_t c = draw(k, attempt), mine = filed(k, attempt);
            if (attempt >= kLookFirst && peek(c) < mine) {
                ++attempt;
                continue;
            }
            const int32_t was = claim(c, mine);
            if (was == kNoOwner) return most;
            if (was > mine) {  // displaced (a slot never meets a claim of its own)
                k = slot(was);
                attempt = static_cast<uint32_t>(was) & ((1u << Bits) - 1);
                if (attempt == kMost)
                    while (draw(k, attempt) != c) ++attempt;
            }
            ++attempt;
        }
    }
};

}  // namespace spo
