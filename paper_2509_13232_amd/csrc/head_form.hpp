// Which form of the LM head the contractions read, and what the 32-bit offsets inside a tile bound: sizes alone decide, so
// this runs on any host.
#pragma once

#include <stdint.h>

namespace spo {

constexpr int64_t kHeadInL2 = int64_t(32) << 20;  // bytes of a head that stays in the L2s
constexpr int64_t kDirectTokens = 8192;

// The main loop forms byte offsets inside a tile in 32 bits.  A head [H,V] read as it was given has rows of 2 V bytes: the
// sweep takes 64 of them per stage (columns along the contraction), dHidden up to kTileRows per tile (rows along it).
// The last piece of the last row has to be below 2^32 bytes.  (Copies have rows of at most 2 H bytes, or of 128.)
constexpr int64_t kTileRows = 256;
static inline bool rows_fit_offsets(int64_t H, int64_t V) {
    const int64_t rows = H < kTileRows ? H : kTileRows;  // H is a multiple of 64
    return rows * 2 * V < int64_t(1) << 32;
}

// The logit gradients of a chunk of tokens lie in blocks of 64 vocabulary entries, 128 bytes per token; d_W reads kTileRows / 64
// blocks side by side, 64 tokens at a time.  Chunks are no longer than those offsets allow (11.2 million tokens; only
// vocabularies of a few hundred entries would otherwise have longer ones by default).
constexpr int64_t kMostChunkTokens = ((int64_t(1) << 32) - 64 * 128) / ((kTileRows / 64 - 1) * 128) / 256 * 256;

// Is a bf16 head read as it was given, or copied into the forms that the main loop reads fastest?  Columns along k
// (dHidden of a head [V,H], the logits of one [H,V]) and rows that are not blocked cost 2 to 5 % of a contraction, and
// the target logits of a head [H,V] then come out of its columns, a line of memory per value; the copies take the
// time of reading the head and writing it once or twice.
//   [V,H]: only dHidden's form is spared.  8192 tokens at 1024 x 151936 6440 us with the copy, 6374 without; 522 at 2112 x
//   151936 2058 and 1843; the gain has vanished at 14000 tokens by these figures.
//   [H,V]: both forms are spared, and a launch: 271 tokens at 3136 x 151936 2035 us with the copies, 1579 without; 4000 at
//   2048 x 151936 6553 and 6414; 4000 at 4096 x 30000 2614 and 2795; 1100 at 768 x 1000 66 and 65, 4000 of them 82 and 87.
//   Values out of columns: 14 us per million where the head comes from memory, 4 out of the L2s.
static inline bool direct_head(bool bf16, bool hv, int64_t tokens, int64_t H, int64_t V) {
    if (!bf16) return false;
    if (!hv) return tokens <= kDirectTokens;
    if (V % 8 != 0) return false;  // rows of [H,V] on 16-byte boundaries
    if (!rows_fit_offsets(H, V)) return false;
    const double T = static_cast<double>(tokens), head = static_cast<double>(H) * static_cast<double>(V);
    const double columns = T * static_cast<double>(H) * (head * 2 <= static_cast<double>(kHeadInL2 / 4) ? 4e-6 : 14e-6);
    return columns + T * head * 7e-11 < 8.0 + head * 1.07e-6;
}

}  // namespace spo
