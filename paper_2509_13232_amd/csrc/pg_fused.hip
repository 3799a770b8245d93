// Fused LM-head + clipped policy-gradient loss, forward and backward, on bf16
// MFMA (Method, PPO-Clip objective over the full vocabulary).  The [T x V] logits
// never exist in memory:
//   forward   sweeps vocabulary tiles, keeping a running (max, sum-exp) per token;
//             the sampled token's logit is one dot product per token beside it;
//   backward  recomputes the logits tile by tile, turns them into bf16 logit
//             gradients dZ for one chunk of tokens at a time, and contracts that
//             chunk twice (dHidden = dZ W, dW += dZ^T X);
//   forward and backward in one call (when d(total)/d(loss) is known up front)
//             walks the batch in pieces: the sweep of a piece also stores, at two
//             bytes per logit, what the two contractions of that piece then
//             read, so the logits are formed once.
// The main loop of gemm_core.hpp takes every operand with the contraction index either contiguous or
// as its row index.  dW contracts over tokens, the row index of both dZ and the hidden states, so
// neither is copied.  The head is read as it was given by short bf16 batches (direct_head); otherwise a
// preparation kernel provides it with one row per vocabulary entry for the logits and in
// blocks along the vocabulary for dHidden.
//
// fp32 inputs use the same bf16 main loop: every value is split into three bf16
// parts (x = x0 + x1 + x2) and the six leading cross products are laid side by
// side along the contraction index, which recovers fp32-grade logits.
#include <algorithm>

#include "gemm_core.hpp"
#include "head_form.hpp"
#include "pg_common.hpp"
#include "tile_choice.hpp"
#include "timing.hpp"

namespace spo {

// 8 wavefronts, each a 128 x 64 part of the tile, on 16x16x32 MFMAs (measured 4-6 % faster
// than the same tile on 32x32x16 on the same chip: the instruction draws less power).
typedef Tile<256, 256, 2, 4> TL;
// 4 wavefronts, each a 64 x 64 part, two workgroups per compute unit: for shapes whose large tiles leave compute units
// idle or are mostly padding (see small_tiles).
typedef Tile<128, 128, 2, 2> TS;
constexpr int kSplitTerms = 6;    // cross products kept by the fp32 split
constexpr int kSweepSplits = 16;  // vocabulary splits of the forward sweep on large problems (a multiple of 8)
// Default size of a backward chunk: as many tokens as keep the chunk's bf16 logit gradients
// (2 * V bytes per token) within this budget, in whole rounds of dHidden tiles on the chip's
// 256 compute units.  dW is read and rewritten once per chunk and every launch ends in a
// partly filled round of tiles, so larger chunks (the caller's choice) are a little faster:
// at H = 4096, V = 151936 the step takes about 1 % longer with 8 GiB than with 40 GB.
constexpr int64_t kDzBudgetBytes = int64_t(8) << 30;
template <typename T> constexpr int kSlots = kChipCUs * 512 / T::NT;  // workgroups that the chip holds at a time
static_assert(TS::BM == kSmallEdge && TL::BM == kLargeEdge && kSlots<TS> == 2 * kChipCUs && kSlots<TL> == kChipCUs && kBK == kStep,
              "what tile_choice.hpp counts");
constexpr int kTailTiles = kChipCUs;  // fp32 tiles of room for the parts of cut contractions (see launch_gemm)

static int64_t gcd64(int64_t a, int64_t b) { return b ? gcd64(b, a % b) : a; }

// tokens per chunk when the caller leaves the choice to the library (a multiple of the tile)
static int64_t default_chunk_tokens(int64_t H, int64_t V_blk) {
    const int64_t fit = kDzBudgetBytes / (2 * V_blk) / TL::BN * TL::BN;  // tokens within the budget
    const int64_t nHt = (H + TL::BM - 1) / TL::BM;                        // dHidden tiles per token tile
    const int64_t round = TL::BN * (kChipCUs / gcd64(kChipCUs, nHt));     // tokens per full round of tiles
    if (fit >= round) return fit / round * round;
    return fit > TL::BN ? fit : TL::BN;
}

// ----------------------------------------------------------------------------
// operand preparation
// ----------------------------------------------------------------------------

// The three-part bf16 split of eight values, laid out along the contraction index: part j of value k at
// o[j*K + k] is part_{sel(j)} with sel = {0,0,1,0,2,1} (Side 0) or {0,1,0,2,0,1} (Side 1), so that
// sum_j side0[jK+k] * side1[jK+k] keeps the products x0y0, x0y1, x1y0, x0y2, x2y0, x1y1.
template <int Side>
__device__ __forceinline__ void store_split(bf16_t *o, int64_t K, const float (&x)[8]) {
    uint32_t part[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t two[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float v = x[2 * i + h];
            const bf16_t p0 = f32_to_bf16(v);
            const float r1 = v - bf16_to_f32(p0);
            const bf16_t p1 = f32_to_bf16(r1);
            two[h][0] = p0;
            two[h][1] = p1;
            two[h][2] = f32_to_bf16(r1 - bf16_to_f32(p1));
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) part[j][i] = two[0][j] | two[1][j] << 16;
    }
    constexpr int sel[2][kSplitTerms] = {{0, 0, 1, 0, 2, 1}, {0, 1, 0, 2, 0, 1}};
#pragma unroll
    for (int j = 0; j < kSplitTerms; ++j) {
        const uint32_t(&q)[4] = part[sel[Side][j]];
        *reinterpret_cast<uint4 *>(o + j * K) = make_uint4(q[0], q[1], q[2], q[3]);
    }
}

__device__ __forceinline__ void load8(const float *p, float (&x)[8]) {
    const float4 a = reinterpret_cast<const float4 *>(p)[0], b = reinterpret_cast<const float4 *>(p)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

__device__ __forceinline__ uint4 round8(const float (&x)[8]) {
    return make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
}

// Everything that the loss's and the gradients' kernels need beforehand and that depends on the inputs
// alone, in one launch: jobs of different kinds share a grid (small batches are bound by the number of
// launches: an fp32 step of 512 tokens went through 17, then 10: 152 -> 137 us; with smaller tiles it is 9 and 64 us).
//   head     the head W [V,H] or [H,V], read once, in every form that is asked for (NULL: not):
//            Wvh  [V][H] as it is (for a head given as [H,V]),
//            Ws   [V][6H] three-part split (fp32),
//            WT   bf16 in blocks of kBlockK vocabulary entries, [V_blk / 64][H][64], zero past V;
//   rows     the three-part split Xs [T][6H] of fp32 hidden states;
//   target   z_target[t] and, with ref2, the reference of every token (see probs_reference);
//   mask     count[0] = number of unmasked tokens, by one workgroup;
//   grad     the gradient factors g of the batch and the list of its active tokens, by one workgroup (up
//            to kPrepGradTokens tokens; above, grad_scale_kernel and compact_active_kernel).
// `head` and `target` may not be in one launch where the head is given as [H,V] (target reads Wvh).
struct PrepJobs {
    int64_t H, V, T;
    const void *W;
    void *Wvh;
    bf16_t *Ws, *WT;
    int64_t head_blocks;          // tiles of 64 x 64
    const void *X;
    bf16_t *Xs;
    int64_t rows, row_blocks;     // rows of Xs; 256 groups of eight values per workgroup
    const void *Wrows;            // the head with one row per vocabulary entry
    const int32_t *target;
    const float *old_logp;
    float *z_target, *ref2;
    int64_t T_ref;                // entries of ref2
    uint32_t *done;
    int64_t target_blocks;        // four wavefronts of target_run (1 or kTargetRun) tokens each
    int target_run, target_cols;  // target_cols: Wrows is the head as [H,V], one token per wavefront
    const uint8_t *mask;
    double *count;                // NULL: not counted
    float *g;                     // NULL: no gradient factors
    const float *logp;
    TokenInputs in;
    float grad_loss;
    int32_t *act_idx, *n_act;
    int64_t blocks() const { return head_blocks + row_blocks + target_blocks + (count ? 1 : 0) + (g ? 1 : 0); }
};

// One workgroup takes 1024 tokens per round; four rounds save two launches and pass beside the head's tiles (512
// tokens: the whole launch 6 us).
constexpr int64_t kPrepGradTokens = 4096;

// Tokens whose target logits one wavefront forms at a time.  Four, their loads together, where there are more tokens
// than the chip has wavefronts and a row is so short that a wavefront waits for it more than it reads (bf16, 200000
// tokens of 64 values 55 -> 26 us, 180000 of 1024 93 -> 68; 170000 of 2048 130 -> 162).
constexpr int kTargetRun = 4;
constexpr int64_t kTargetRunTokens = 16384, kTargetRunBytes = 2048;

constexpr int kPrepTile = 64;
template <typename T_> constexpr int kPrepPitch = sizeof(T_) == 2 ? 66 : 65;

// One 64 x 64 tile of the head.  Bound by memory: sixteen bytes per lane in and out, rows of 128 bytes
// in, whole 8 KiB pieces of WT out (151936 x 4096: 952 -> 443 us = 5.6 TB/s;
// one element per lane was 2.6).
template <typename T_, bool HV>
__device__ __forceinline__ void prep_head_tile(const PrepJobs &j, int64_t tile_id, T_ *tile) {
    constexpr int P = kPrepPitch<T_>, N = 16 / sizeof(T_);  // N values per 16-byte load
    const int64_t nh = j.H / kPrepTile;
    const int64_t v0 = tile_id / nh * kPrepTile, h0 = tile_id % nh * kPrepTile;
    const T_ *W = static_cast<const T_ *>(j.W);
    const int nv = static_cast<int>(j.V - v0 < kPrepTile ? j.V - v0 : kPrepTile);  // may be <= 0: only padding of WT
    const int tid = threadIdx.x;
    // tile[r][c], r the source's row: v (h of an [H,V] head), c its contiguous index
    constexpr int per_row = kPrepTile / N, rows_at_once = 256 / per_row;
    const bool whole = HV ? nv == kPrepTile && j.V % N == 0 : true;
    if (whole) {
#pragma unroll
        for (int r = tid / per_row; r < kPrepTile; r += rows_at_once) {
            const int c = tid % per_row * N;
            uint4 u = make_uint4(0u, 0u, 0u, 0u);
            if (HV) u = *reinterpret_cast<const uint4 *>(W + (h0 + r) * j.V + v0 + c);
            else if (r < nv) u = *reinterpret_cast<const uint4 *>(W + (v0 + r) * j.H + h0 + c);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if constexpr (sizeof(T_) == 2) *reinterpret_cast<uint32_t *>(tile + r * P + c + 2 * i) = w[i];
                else tile[r * P + c + i] = __uint_as_float(w[i]);
        }
    } else {  // an [H,V] head whose rows end or start off 16-byte boundaries
        for (int i = tid; i < kPrepTile * kPrepTile; i += 256) {
            const int r = i / kPrepTile, c = i % kPrepTile;
            tile[r * P + c] = c < nv ? W[(h0 + r) * j.V + v0 + c] : T_(0);
        }
    }
    __syncthreads();
    auto at = [&](int v, int h) { return HV ? tile[h * P + v] : tile[v * P + h]; };
    constexpr int G = kPrepTile / 8;  // groups of eight values per row
#pragma unroll
    for (int i = tid; i < kPrepTile * G; i += 256) {
        const int r = i / G, c = i % G * 8;
        if (j.WT) {  // r: hidden unit, c: vocabulary
            uint4 u;
            if constexpr (sizeof(T_) == 2) {
                uint32_t w[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) w[k] = at(c + 2 * k, r) | static_cast<uint32_t>(at(c + 2 * k + 1, r)) << 16;
                u = make_uint4(w[0], w[1], w[2], w[3]);
            } else {
                float x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) x[k] = at(c + k, r);
                u = round8(x);
            }
            *reinterpret_cast<uint4 *>(j.WT + (v0 * j.H + (h0 + r) * kBlockK + c)) = u;
        }
        if (r < nv && (j.Wvh || j.Ws)) {  // r: vocabulary, c: hidden unit
            T_ x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = at(r, c + k);
            if (j.Wvh) {
                T_ *o = static_cast<T_ *>(j.Wvh) + (v0 + r) * j.H + h0 + c;
                if constexpr (sizeof(T_) == 2) {
                    uint32_t w[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[k] = x[2 * k] | static_cast<uint32_t>(x[2 * k + 1]) << 16;
                    *reinterpret_cast<uint4 *>(o) = make_uint4(w[0], w[1], w[2], w[3]);
                } else {
                    reinterpret_cast<float4 *>(o)[0] = make_float4(x[0], x[1], x[2], x[3]);
                    reinterpret_cast<float4 *>(o)[1] = make_float4(x[4], x[5], x[6], x[7]);
                }
            }
            if constexpr (sizeof(T_) == 4)
                if (j.Ws) store_split<0>(j.Ws + (v0 + r) * (kSplitTerms * j.H) + h0 + c, j.H, x);
        }
    }
}

// n a multiple of 64; both arrays on 16-byte boundaries
__global__ void __launch_bounds__(256)
f32_to_bf16_kernel(const float *__restrict__ src, bf16_t *__restrict__ dst, int64_t n) {
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    float x[8];
    load8(src + i, x);
    *reinterpret_cast<uint4 *>(dst + i) = round8(x);
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint32_t *__restrict__ p, int64_t n_words) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n_words) p[i] = 0u;
}

// ----------------------------------------------------------------------------
// backward: compaction of the tokens that carry a gradient
// ----------------------------------------------------------------------------
// Masked tokens, tokens on the clipped branch and tokens of a response with zero
// advantage have g = 0: their rows of dZ vanish, so the backward contractions run
// over the remaining ("active") tokens only, in their original order.

// act_idx[j] = index of the j-th token t < T with g_at(t) != 0 (called once per token); n_act[0] = their
// number.  One workgroup of NT threads walks the tokens 4 * NT at a time (order-preserving, deterministic).
template <int NT, typename G>
__device__ __forceinline__ void compact_tokens(int64_t T, G g_at, int32_t *__restrict__ act_idx, int32_t *__restrict__ n_act,
                                               int *wave_cnt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int base = 0;
    for (int64_t t0 = 0; t0 < T; t0 += 4 * NT) {
        const int64_t t = t0 + threadIdx.x * 4;
        bool on[4];
        int mine = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            on[i] = t + i < T && g_at(t + i) != 0.0f;
            mine += on[i] ? 1 : 0;
        }
        // exclusive prefix of `mine` over the wavefront, then over the wavefronts
        int incl = mine;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int up = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += up;
        }
        if (lane == kWave - 1) wave_cnt[wave] = incl;
        __syncthreads();
        int off = 0, tot = 0;
#pragma unroll
        for (int w = 0; w < NT / kWave; ++w) {
            const int c = wave_cnt[w];
            off += w < wave ? c : 0;
            tot += c;
        }
        int pos = base + off + incl - mine;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (on[i]) act_idx[pos++] = static_cast<int32_t>(t + i);
        base += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) n_act[0] = base;
}

__global__ void __launch_bounds__(1024)
compact_active_kernel(const float *__restrict__ g, int64_t T, int32_t *__restrict__ act_idx,
                      int32_t *__restrict__ n_act) {
    __shared__ int wave_cnt[1024 / kWave];
    compact_tokens<1024>(T, [&](int64_t t) { return g[t]; }, act_idx, n_act, wave_cnt);
}

// Number of active tokens that fall into rows [row_base, row_base + cap) of the compact order.
__device__ __forceinline__ int64_t active_rows(const int32_t *n_act, int64_t row_base, int64_t cap) {
    const int64_t n = static_cast<int64_t>(*n_act) - row_base;
    return n < 0 ? 0 : (n > cap ? cap : n);
}

// Rows [row_base, row_base + rows) of the compact order: their hidden states X[act_idx[row_base + r]] as
// bf16 rows Xc (NULL: not) and, of fp32 ones, as the three-part split Xs (NULL: not); and, packed into
// one 16-byte record per row, the
// per-token scalars the recompute needs: tok[r] = (|g|, log2|g| - lse * log2(e), target with the
// sign of g in the top bit (set: g > 0), 0): the gradient's softmax part -g * p is then
// -sign(g) * exp2(z * log2(e) + tok.y), one multiply-add and one exponential per logit.
// Rows past the last active token are filled with zeros and (0, -inf, no target): every
// exponential underflows to an exact zero.  A wavefront per row.  The first zero_rows rows of `zero`, of
// zero_bytes each, are cleared on the way (d_hidden: rows of tokens without a gradient stay zero).
template <typename T_>
__global__ void __launch_bounds__(256)
gather_chunk_kernel(const T_ *__restrict__ X, int64_t H, const int32_t *__restrict__ act_idx,
                    const int32_t *__restrict__ n_act, int64_t row_base, int64_t rows,
                    const int32_t *__restrict__ target, const float *__restrict__ lse, const float *__restrict__ g,
                    bf16_t *__restrict__ Xc, bf16_t *__restrict__ Xs, float4 *__restrict__ tok, char *__restrict__ zero,
                    int64_t zero_rows, int64_t zero_bytes) {
    const int64_t r = flat_block() * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r < zero_rows) {
        uint4 *z = reinterpret_cast<uint4 *>(zero + r * zero_bytes);  // a multiple of 128 bytes
        for (int i = lane; i < zero_bytes / 16; i += kWave) z[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (r >= rows) return;
    const bool live = r < active_rows(n_act, row_base, rows);
    const int64_t src = live ? act_idx[row_base + r] : 0;
    for (int i = lane; i < H / 8; i += kWave) {  // H is a multiple of 64
        if constexpr (sizeof(T_) == 2) {
            reinterpret_cast<uint4 *>(Xc + r * H)[i] =
                live ? reinterpret_cast<const uint4 *>(X + src * H)[i] : make_uint4(0u, 0u, 0u, 0u);
        } else {
            float x[8] = {};
            if (live) load8(X + src * H + i * 8, x);
            if (Xc) reinterpret_cast<uint4 *>(Xc + r * H)[i] = round8(x);
            if (Xs) store_split<1>(Xs + r * (kSplitTerms * H) + i * 8, H, x);
        }
    }
    if (lane == 0) {
        const float gs = live ? g[src] : 0.0f;
        const uint32_t ts = live ? (static_cast<uint32_t>(target[src]) & 0x7fffffffu) | (gs > 0.0f ? 0x80000000u : 0u)
                                 : 0x7fffffffu;
        tok[r] = make_float4(fabsf(gs), live ? log2f(fabsf(gs)) - lse[src] * kLog2e : -INFINITY, __uint_as_float(ts), 0.0f);
    }
}

// ----------------------------------------------------------------------------
// forward: logit of the sampled token
// ----------------------------------------------------------------------------
// z_target[t] = h_t . W[target[t]] (W with one row per vocabulary entry), by one wavefront,
// products and sum in fp32.  The sweep below does not have to watch for this one
// entry of every row.  An id outside [0, V) gives NaN (the token's log-prob, and with it the
// loss, then say so instead of carrying an arbitrary number).
__device__ __forceinline__ float dot8(const uint4 a, const uint4 b) {
    const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s = fmaf(__uint_as_float(x[i] << 16), __uint_as_float(y[i] << 16), s);
        s = fmaf(__uint_as_float(x[i] & 0xffff0000u), __uint_as_float(y[i] & 0xffff0000u), s);
    }
    return s;
}

// The target logits of K consecutive tokens from t on (NaN past T) by one wavefront, the loads of all in flight together.
template <int K, typename T_>
__device__ __forceinline__ void target_logits(const T_ *__restrict__ X, const T_ *__restrict__ Wvh, int64_t H, int64_t V, int64_t T,
                                              const int32_t *__restrict__ target, int64_t t, int lane, float (&z)[K]) {
    constexpr int N = 16 / sizeof(T_);  // values per 16-byte load
    const uint4 *x[K], *w[K];
    bool ok[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t y = t + k < T ? target[t + k] : -1;
        ok[k] = y >= 0 && y < V;
        x[k] = reinterpret_cast<const uint4 *>(X + (ok[k] ? t + k : 0) * H);  // (of the others: the first row, not used)
        w[k] = reinterpret_cast<const uint4 *>(Wvh + (ok[k] ? y : 0) * H);
        z[k] = 0.0f;
    }
#pragma unroll 4 / K
    for (int i = lane; i < H / N; i += kWave) {  // H is a multiple of 64
        uint4 a[K], b[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            a[k] = x[k][i];
            b[k] = w[k][i];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (sizeof(T_) == 2) {
                z[k] += dot8(a[k], b[k]);
            } else {
                z[k] = fmaf(__uint_as_float(a[k].x), __uint_as_float(b[k].x), z[k]);
                z[k] = fmaf(__uint_as_float(a[k].y), __uint_as_float(b[k].y), z[k]);
                z[k] = fmaf(__uint_as_float(a[k].z), __uint_as_float(b[k].z), z[k]);
                z[k] = fmaf(__uint_as_float(a[k].w), __uint_as_float(b[k].w), z[k]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float s = wave_sum(z[k]);
        z[k] = ok[k] ? s : __builtin_nanf("");
    }
}

// The same of one token where the head is [H,V]: the entries of a column lie 2 V bytes apart, eight of them in flight
// per lane (the sum in the order of target_logits).
__device__ __forceinline__ float target_logit_cols(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W, int64_t H, int64_t V,
                                                   int64_t T, const int32_t *__restrict__ target, int64_t t, int lane) {
    const int64_t y = t < T ? target[t] : -1;
    const bool ok = y >= 0 && y < V;
    const uint4 *x = reinterpret_cast<const uint4 *>(X + (ok ? t : 0) * H);
    const bf16_t *w = W + (ok ? y : 0);
    float z = 0.0f;
    for (int i = lane; i < H / 8; i += kWave) {
        const uint4 a = x[i];
        uint32_t b[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) b[k] = w[(i * 8 + k) * V];
        z += dot8(a, make_uint4(b[0] | b[1] << 16, b[2] | b[3] << 16, b[4] | b[5] << 16, b[6] | b[7] << 16));
    }
    z = wave_sum(z);
    return ok ? z : __builtin_nanf("");
}

// The reference of a token whose logits are stored as scaled probabilities (see below, one-call form without
// a loss mask), times log2(e); 0 where the token has no valid target logit or old_logp is not finite (its
// stored row stays finite and is multiplied by 0).
__device__ __forceinline__ float probs_reference(float z_target, float old_logp) {
    const float r = (z_target - old_logp) * kLog2e;
    return fabsf(r) < 3.0e38f ? r : 0.0f;  // not NaN, not infinite
}

// Target logits and references of 4 * K tokens by one workgroup.
template <int K, typename T_>
__device__ __forceinline__ void prep_targets(const PrepJobs &j, int64_t block) {
    const int64_t t = (block * 4 + (threadIdx.x >> 6)) * K;
    const int lane = threadIdx.x & 63;
    float z[K];
    bool done = false;
    if constexpr (K == 1 && sizeof(T_) == 2)
        if (j.target_cols) {
            z[0] = target_logit_cols(static_cast<const bf16_t *>(j.X), static_cast<const bf16_t *>(j.Wrows), j.H, j.V, j.T, j.target, t, lane);
            done = true;
        }
    if (!done) target_logits<K>(static_cast<const T_ *>(j.X), static_cast<const T_ *>(j.Wrows), j.H, j.V, j.T, j.target, t, lane, z);
    float mine = z[0];  // lane k: token t + k
#pragma unroll
    for (int k = 1; k < K; ++k) mine = lane == k ? z[k] : mine;
    if (lane >= K) return;
    if (t + lane < j.T) j.z_target[t + lane] = mine;
    if (j.ref2 && t + lane < j.T_ref) j.ref2[t + lane] = t + lane < j.T ? probs_reference(mine, j.old_logp[t + lane]) : 0.0f;
}

template <typename T_, bool HV>
__global__ void __launch_bounds__(256) prep_kernel(PrepJobs j) {
    __shared__ __attribute__((aligned(16))) T_ tile[kPrepTile * kPrepPitch<T_>];
    __shared__ int scratch[256 / kWave];
    int64_t b = flat_block();
    if (b == 0 && threadIdx.x == 0 && j.done) *j.done = 0u;  // counts the token kernel's finished blocks
    if (b < j.head_blocks) return prep_head_tile<T_, HV>(j, b, tile);
    b -= j.head_blocks;
    if (b < j.row_blocks) {
        if constexpr (sizeof(T_) == 4) {
            const int64_t i = (b * 256 + threadIdx.x) * 8, r = i / j.H, k = i % j.H;  // H is a multiple of 64
            if (r >= j.rows) return;
            float x[8];
            load8(static_cast<const float *>(j.X) + i, x);
            store_split<1>(j.Xs + r * (kSplitTerms * j.H) + k, j.H, x);
        }
        return;
    }
    b -= j.row_blocks;
    if (b < j.target_blocks) {
        if (j.target_run > 1) prep_targets<kTargetRun, T_>(j, b);
        else prep_targets<1, T_>(j, b);
        return;
    }
    b -= j.target_blocks;
    if (b == 0 && j.count) {
        const int64_t c = j.mask ? count_mask(j.mask, j.T, scratch) : j.T;
        if (threadIdx.x == 0) j.count[0] = static_cast<double>(c);
        return;
    }
    if (b == (j.count ? 1 : 0) && j.g) {
        __shared__ int32_t cu_lds[kCuStaged];
        const int32_t *cu = stage_offsets(j.in.cu, j.in.B, cu_lds);
        const double M = static_cast<double>(j.in.mask ? count_mask(j.in.mask, j.in.T, scratch) : j.in.T);
        __syncthreads();
        compact_tokens<256>(j.in.T, [&](int64_t t) { return j.g[t] = token_grad(j.logp, j.in, cu, M, j.grad_loss, t); }, j.act_idx,
                            j.n_act, scratch);
    }
}

// The jobs that make the head's forms; those of the hidden rows X[0..rows) where they are fp32.
static PrepJobs prep_head_jobs(const spo_pg_desc *d, void *Wvh, bf16_t *Ws, bf16_t *WT) {
    PrepJobs j{};
    j.H = d->H;
    j.V = d->V;
    j.T = d->T;
    j.W = d->W;
    j.Wvh = Wvh;
    j.Ws = Ws;
    j.WT = WT;
    if (Wvh || Ws || WT) j.head_blocks = ceil_div(d->V, WT ? TL::BM : kPrepTile) * (WT ? TL::BM / kPrepTile : 1) * (d->H / kPrepTile);
    return j;
}
static void prep_rows(PrepJobs &j, const spo_pg_desc *d, const void *X, int64_t rows, bf16_t *Xs) {
    if (d->dtype != SPO_FP32) return;
    j.X = X;
    j.Xs = Xs;
    j.rows = rows;
    j.row_blocks = ceil_div(rows * (d->H / 8), 256);
}
static void launch_prep(const spo_pg_desc *d, const PrepJobs &j, hipStream_t s) {
    if (j.blocks() == 0) return;
    const bool hv = d->w_layout == SPO_W_HV;
    auto *kernel = d->dtype == SPO_FP32 ? (hv ? prep_kernel<float, true> : prep_kernel<float, false>)
                                        : (hv ? prep_kernel<bf16_t, true> : prep_kernel<bf16_t, false>);
    kernel<<<fold_grid(j.blocks()), 256, 0, s>>>(j);
}
// The jobs of `j` and the target logits: in one launch, unless the latter read a form of the head that the former make.
static void launch_prep_with_targets(const spo_pg_desc *d, PrepJobs j, float *z_target, float *ref2, int64_t T_ref,
                                     uint32_t *done, hipStream_t s) {
    if (j.Wvh) {
        launch_prep(d, j, s);
        const void *Wvh = j.Wvh;
        j = prep_head_jobs(d, nullptr, nullptr, nullptr);
        j.Wrows = Wvh;
    } else {
        j.Wrows = d->W;
    }
    j.X = d->hidden;
    j.target = d->target;
    j.old_logp = d->old_logp;
    j.z_target = z_target;
    j.ref2 = ref2;
    j.T_ref = T_ref;
    j.done = done;
    const int64_t tokens = ref2 ? T_ref : d->T;
    j.target_cols = d->w_layout == SPO_W_HV && j.Wrows == d->W;
    j.target_run = !j.target_cols && tokens > kTargetRunTokens && d->H * (d->dtype == SPO_FP32 ? 4 : 2) <= kTargetRunBytes ? kTargetRun : 1;
    j.target_blocks = ceil_div(tokens, 4 * j.target_run);
    launch_prep(d, j, s);
}

// ----------------------------------------------------------------------------
// forward: vocabulary sweep with online log-sum-exp
// ----------------------------------------------------------------------------
// Tile rows (m) are vocabulary entries, tile columns (n) are tokens, so that each
// lane owns FN tokens and reduces over the vocabulary inside its own registers.

// Vocabulary splits of the two kernels that form logits (the forward sweep and the backward's
// recompute).  A launch lasts about (rounds of workgroups on the chip) x (vocabulary tiles of the
// longest workgroup), so among the multiples of 8 the count with the smallest product is taken (the
// smallest such count: longer workgroups).  67 token tiles x 594 vocabulary tiles in 16 splits are
// 5 rounds x 38 tiles = 190, in 40 splits 11 x 15 = 165, of 155.5 that the work divided by 256 units
// comes to.  Fewer tiles than units: a workgroup each.
// slots: workgroups that the chip holds at a time.
template <typename U>
__host__ __device__ static inline U sweep_cost(U nTt, U nVt, U ns, U slots) {
    return (nTt * ns + slots - 1) / slots * ((nVt + ns - 1) / ns);
}
// Candidates: the multiples of 8 in [sweep_splits_lo, sweep_splits_hi].  From 16 token tiles on at least
// 16 splits (workgroups that share lines drift apart on longer runs), at most about 4096 workgroups
// (more gain nothing in balance and grow the partial results).
__host__ __device__ static inline uint32_t sweep_splits_lo(uint32_t nTt) { return nTt >= 16 ? kSweepSplits : 8; }
__host__ __device__ static inline uint32_t sweep_splits_hi(uint32_t nTt, uint32_t nVt, uint32_t cap) {
    uint32_t hi = 4096 / nTt;
    hi = hi < static_cast<uint32_t>(kSweepSplits) ? kSweepSplits : (hi > 512 ? 512 : hi);
    hi = hi < nVt ? hi : nVt;
    return hi < cap ? hi : cap;
}
constexpr uint32_t kNoSplitCap = 512;
// cap: the most splits the caller has room for (at least kSweepSplits)
static int sweep_splits(int64_t token_tiles, int64_t vocab_tiles, int slots, uint32_t cap = kNoSplitCap) {
    const uint64_t nTt = token_tiles > 0 ? token_tiles : 1, nVt = vocab_tiles;
    const uint64_t chip = slots;
    if (nTt * nVt <= chip && nVt <= cap) return static_cast<int>(nVt);
    const uint64_t hi = sweep_splits_hi(static_cast<uint32_t>(nTt), static_cast<uint32_t>(nVt), cap);
    uint64_t best = 0;
    for (uint64_t ns = sweep_splits_lo(static_cast<uint32_t>(nTt)); ns <= hi; ns += 8)
        if (!best || sweep_cost(nTt, nVt, ns, chip) < sweep_cost(nTt, nVt, best, chip)) best = ns;
    return static_cast<int>(best ? best : hi);
}
// The same choice by a wavefront, one candidate per lane, where the number of token tiles is known on the
// device only (the tiles of a chunk's gradients fit the memory: costs stay far below 2^22).
__device__ __forceinline__ int sweep_splits_wave(uint32_t nTt, uint32_t nVt, uint32_t slots) {
    if (nTt * nVt <= slots) return static_cast<int>(nVt);
    const uint32_t hi = sweep_splits_hi(nTt, nVt, kNoSplitCap), ns = sweep_splits_lo(nTt) + 8 * (threadIdx.x & 63);
    uint32_t key = ns <= hi ? sweep_cost(nTt, nVt, ns, slots) << 10 | ns : 0xffffffffu;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t k = __shfl_xor(key, o, kWave);
        key = k < key ? k : key;
    }
    return __builtin_amdgcn_readfirstlane(static_cast<int>(key == 0xffffffffu ? hi : key & 1023u));
}
// The most (token tile, split) pairs that any number of token tiles up to nTt can ask for.  The number of splits
// jumps with that of the token tiles; this grows with both sizes, so room sized by it for the longest batch serves
// every shorter one.
static int64_t sweep_pairs_max(int64_t nTt, int64_t nVt) {
    return std::min(nTt * std::min<int64_t>(nVt, kNoSplitCap), std::max<int64_t>(4096, nTt * kSweepSplits));
}
// Entries of room for the partial results of every token and split; roomy: also those of small tiles.
static int64_t sweep_room(int64_t T, int64_t V, bool roomy) {
    const int64_t large = sweep_pairs_max(ceil_div(T, TL::BN), ceil_div(V, TL::BM)) * TL::BN;
    return roomy ? std::max(large, sweep_pairs_max(ceil_div(T, TS::BN), ceil_div(V, TS::BM)) * TS::BN) : large;
}
// The most workgroups (ids of SweepMap) for them: what is left over by eight XCDs is rounded up.
static int64_t sweep_blocks_max(int64_t nTt, int64_t nVt) { return sweep_pairs_max(nTt, nVt) + 8; }

// Workgroup -> (token tile, vocabulary split): a workgroup keeps its token tile and walks the vocabulary
// tiles of its split.  Ids equal mod 8 run on the same XCD and share its L2: there, 32
// consecutive workgroups are a patch of 4 token tiles x 8 splits (each hidden-state panel feeds
// 8 of them, each head tile 4), and the eight XCDs work on the same splits of different token
// tiles at about the same time, so a head tile fetched from memory serves 32 token tiles out of
// the Infinity Cache.  (A 4 x 8 patch of tiles walked along the vocabulary, every head tile used by
// one XCD only, made the recompute 3.6 % slower.)  More than 8 splits shorten a workgroup's
// sweep: workgroups that share lines then have less time to drift apart.
// Token tiles left over when their number is no multiple of 8 would give some XCDs a tile more than
// others (5 tiles: three XCDs idle): those few are divided by splits instead, each XCD an eighth of the
// vocabulary of all of them (1191 tokens at H = 4096, V = 151936: 1960 us -> 1196 us with the choice of splits).
struct SweepMap {
    uint32_t ns;
    int64_t nTt, nVt, main_tt;  // tiles; token tiles that belong to one XCD each
    __host__ __device__ SweepMap(int64_t token_tiles, int64_t vocab_tiles, int splits)
        : ns(static_cast<uint32_t>(splits)), nTt(token_tiles), nVt(vocab_tiles), main_tt(token_tiles / 8 * 8) {}
    __host__ __device__ int64_t blocks() const { return main_tt * ns + ((nTt - main_tt) * ns + 7) / 8 * 8; }
    // token tile jt and split of workgroup bid; false for ids without work
    __device__ bool tile(uint32_t bid, int &split, int64_t &jt) const {
        const uint32_t xcd = bid & 7, q = bid >> 3, x = static_cast<uint32_t>(main_tt / 8);
        if (q >= x * ns) {
            const uint32_t r = static_cast<uint32_t>(nTt - main_tt), i = q - x * ns;
            if (ns % 8 == 0) {  // token tiles side by side share the head tiles of a split
                if (i >= r * (ns / 8)) return false;
                split = static_cast<int>(xcd * (ns / 8) + i / r);
                jt = main_tt + i % r;
                return true;
            }
            const uint32_t j = i * 8 + xcd;
            if (j >= r * ns) return false;
            split = static_cast<int>(j % ns);
            jt = main_tt + j / ns;
            return true;
        }
        if (ns % 8 == 0) {  // rows of patches of 4 token tiles (the last row: what is left) x 8 splits
            const uint32_t row = q / (4 * ns), i = q - row * 4 * ns, h = x - 4 * row < 4 ? x - 4 * row : 4;
            const uint32_t g = i / (8 * h), w = i - g * 8 * h;
            split = static_cast<int>(g * 8 + (w & 7));
            jt = static_cast<int64_t>(row * 4 + (w >> 3)) * 8 + xcd;
        } else {  // small vocabularies: all splits of a token tile side by side
            split = static_cast<int>(q % ns);
            jt = static_cast<int64_t>(q / ns) * 8 + xcd;
        }
        return true;
    }
    __host__ __device__ int64_t first_tile(int split) const { return split * nVt / ns; }
};

constexpr int kEmitNone = 0, kEmitLogits = 1, kEmitProbs = 2;  // see fwd_sweep_kernel
// operand stages + the per-thread running state (+ the per-token references)
template <typename T> constexpr int kSweepLds(int emit) { return T::LDS_BYTES + T::NT * (emit == kEmitProbs ? 48 : 32); }

// Exchange between neighbouring groups of 16 lanes: v_permlane16_swap(a, b) swaps the odd groups
// of a with the even groups of b.  With a, b the values a lane holds for two consecutive MFMA
// blocks q, q+1, lane group g ends up with (in a, b) the values of block q + (g & 1) from lane
// groups (g & 2) and (g & 2) + 1.
__device__ __forceinline__ void swap_lane_groups(uint32_t &a, uint32_t &b) {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u t = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = t.x;
    b = t.y;
}

// two floats as a pair of IEEE halves, round to nearest even
__device__ __forceinline__ uint32_t pack_f16x2_rn(float lo, float hi) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const h2 v = {static_cast<_Float16>(lo), static_cast<_Float16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}

// Emit = kEmitNone: the forward proper; the logits exist in registers only.
// The other two forms serve the one-call forward + backward: every finished tile is also
// written out, in the blocked layout of the logit gradients (token n of this launch, vocabulary
// entry v at Z + (v / 64) * z_blk + n * 64 + v % 64).
// Emit = kEmitLogits: fp16 of (logit - offset).  The offset is the running maximum of the token
// over the TT::WM vocabulary rows per tile (128 of large tiles, 64 of small ones) that the wavefront has seen so far in its
// sweep, this tile included: one value per (vocabulary tile, part of WM rows, token), written to
// offs[(tile * WGM + part) * T_pad + n].  Stored values are <= 0, and an entry within d of the
// row's largest logit is stored within d of zero, where fp16 resolves 2^-11 * d: the entries
// that carry the softmax are the most exact ones.  Rows past the vocabulary are stored as -inf.
// Emit = kEmitProbs: bf16 of exp(logit - r_n), with r_n a per-token reference known before the
// sweep (offs[n] = r_n * log2(e) on entry; see the host code for the choice that makes these
// the softmax probabilities divided by the token's importance ratio).  The exponentials are the
// ones the running sum needs anyway, times one factor per token and lane; exponents are capped
// at 126 so that nothing stored is infinite.  Rows past the vocabulary are stored as zeros.
// WCols: W is the head as [H,V], read as it is.
template <int Emit, typename TT, bool WCols>
__global__ void __launch_bounds__(TT::NT, 2)
fwd_sweep_kernel(const char *__restrict__ W, int64_t ldw_bytes, int64_t V, const char *__restrict__ X,
                 int64_t ldx_bytes, int64_t T, int KT, int nsplit, int64_t nTt, int64_t nVt, int64_t T_pad,
                 float *__restrict__ part_max, float *__restrict__ part_sum, uint16_t *__restrict__ Z, int64_t z_blk,
                 float *__restrict__ offs) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const SweepMap map(nTt, nVt, nsplit);  // the host sized the partial results with the same map
    int split;
    int64_t jt;
    if (!map.tile(blockIdx.x, split, jt)) return;
    const int64_t n0 = jt * TT::BN;
    const int64_t vt0 = map.first_tile(split), vt1 = map.first_tile(split + 1);
    const int lane = threadIdx.x & 63;

    // Running (maximum, sum of exponentials) of this lane's FN tokens.  Between tiles they wait in
    // the LDS the operand stages leave free (a slot per thread): the main loop needs every register.
    static_assert(TT::FN == 4, "one 16-byte slot each for the maxima and the sums");
    auto state = [&] {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // not to be traced: the address is formed anew at every use
        return reinterpret_cast<float4 *>(lds + TT::LDS_BYTES) + (Emit == kEmitProbs ? 3 : 2) * tid;
    };
    state()[0] = make_float4(kNegBig, kNegBig, kNegBig, kNegBig);
    state()[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (Emit == kEmitProbs) {  // the references of this lane's four tokens: the workgroup keeps its token tile
        const float *r = offs + n0 + TT::wave_n0() + (lane & 15);
        state()[2] = make_float4(r[0], r[TT::MI], r[2 * TT::MI], r[3 * TT::MI]);
    }
    // One finished tile.  Online log-sum-exp over its rows: three operations per logit (multiply-add
    // into the exponent, exponential, add) plus its share of the maximum.  With Emit, the tile's
    // values also leave for memory, token column by token column as each is done, so that the stores
    // of one column are on their way while the next is being worked on.  A lane holds runs of four
    // consecutive vocabulary entries of one token; after an exchange between neighbouring lane
    // groups it holds 16 contiguous bytes of two 64-entry blocks out of four (the scheme of the
    // recompute's epilogue below).
    auto finish_tile = [&](typename TT::Acc &acc, int64_t vt) {
        const int64_t m0 = vt * TT::BM;
        if (m0 + TT::BM > V) {  // ragged last tile: rows past the vocabulary do not count
#pragma unroll
            for (int fm = 0; fm < TT::FM; ++fm)
#pragma unroll
                for (int r = 0; r < TT::ACC_R; ++r)
                    if (m0 + TT::acc_row(fm, r) >= V)
#pragma unroll
                        for (int fn = 0; fn < TT::FN; ++fn) acc[fm][fn][r] = -INFINITY;
        }
        int l = threadIdx.x & 63;
        asm volatile("" : "+v"(l));  // not to be traced: nothing derived from it lives through the main loop
        const int grp = l >> 4, col = l & 15;
        const int64_t wave_blk = vt * (TT::BM / kBlockK) + TT::wave_m0() / kBlockK;
        const int piece = (grp & 1) * 16 + (grp & 2) * 4;  // elements: byte offset 32 * (g & 1) + 8 * (g & 2)
        float4 *st = state();
        const float4 m4 = st[0], s4 = st[1];
        float m_run[TT::FN] = {m4.x, m4.y, m4.z, m4.w}, s_run[TT::FN] = {s4.x, s4.y, s4.z, s4.w};
        float ref[TT::FN] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (Emit == kEmitProbs) {
            const float4 r4 = st[2];
            ref[0] = r4.x; ref[1] = r4.y; ref[2] = r4.z; ref[3] = r4.w;
        }
#pragma unroll
        for (int fn = 0; fn < TT::FN; ++fn) {
            float mx = -INFINITY;
#pragma unroll
            for (int fm = 0; fm < TT::FM; ++fm)
#pragma unroll
                for (int r = 0; r < TT::ACC_R; ++r) mx = fmaxf(mx, acc[fm][fn][r]);
            // the running maximum starts at a finite sentinel, so nm is finite even when every
            // row of the tile is masked (their logits are -inf and add exact zeros)
            const float nm = fmaxf(m_run[fn], mx);
            const float c = -nm * kLog2e;
            // what is stored of an entry: a * value + b, with value the exponential (kEmitProbs: times
            // exp(nm - r), capped) or the logit itself (kEmitLogits: minus the offset, the largest logit the
            // wavefront's WM rows have shown for this token so far)
            float a = 0.0f, off = 0.0f;
            if (Emit == kEmitProbs) a = __builtin_amdgcn_exp2f(fminf(fmaf(nm, kLog2e, -ref[fn]), 126.0f));
            if (Emit == kEmitLogits) {
                off = fmaxf(nm, __shfl_xor(nm, 16, kWave));
                off = fmaxf(off, __shfl_xor(off, 32, kWave));
                if (grp == 0)
                    offs[(vt * TT::WGM + TT::wave_m0() / TT::WM) * T_pad + n0 + TT::wave_n0() + fn * TT::MI + col] = off;
            }
            float s = 0.0f;
            uint16_t *row = Emit ? Z + (n0 + TT::wave_n0() + fn * TT::MI + col) * kBlockK + piece : nullptr;
#pragma unroll
            for (int b = 0; b < TT::FM / 4; ++b) {
                uint32_t lo[4], hi[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float e[4], v[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        e[r] = __builtin_amdgcn_exp2f(fmaf(acc[4 * b + q][fn][r], kLog2e, c));
                        s += e[r];
                        v[r] = Emit == kEmitProbs ? e[r] * a : acc[4 * b + q][fn][r] - off;
                    }
                    if (Emit == kEmitProbs) {
                        lo[q] = pack_bf16x2_rn(v[0], v[1]);
                        hi[q] = pack_bf16x2_rn(v[2], v[3]);
                    }
                    if (Emit == kEmitLogits) {
                        lo[q] = pack_f16x2_rn(v[0], v[1]);
                        hi[q] = pack_f16x2_rn(v[2], v[3]);
                    }
                }
                if (Emit) {
                    swap_lane_groups(lo[0], lo[1]);
                    swap_lane_groups(hi[0], hi[1]);
                    swap_lane_groups(lo[2], lo[3]);
                    swap_lane_groups(hi[2], hi[3]);
                    uint16_t *out = row + (wave_blk + b) * z_blk;
                    *reinterpret_cast<uint4 *>(out) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
                    *reinterpret_cast<uint4 *>(out + kBlockK / 2) = make_uint4(lo[2], hi[2], lo[3], hi[3]);
                }
            }
            s_run[fn] = s_run[fn] * __builtin_amdgcn_exp2f((m_run[fn] - nm) * kLog2e) + s;
            m_run[fn] = nm;
        }
        st[0] = make_float4(m_run[0], m_run[1], m_run[2], m_run[3]);
        st[1] = make_float4(s_run[0], s_run[1], s_run[2], s_run[3]);
    };
    // Where tiles are stored they are a run: the first stages of the next tile are requested in the last step of this one,
    // and this one's stores (at least kStores per wavefront) are not waited for before its first step: 8192 tokens at 1024 x
    // 151936 6420 -> 6345 us, 11238 masked ones at 192 x 151936 4101 -> 4022, 20000 at 2048 x 60000 the same.  (Without stores
    // it is 2 % slower, and so no gain for the recompute, whose records would have to wait in LDS.)  Large tiles then have more
    // values between two tiles than registers: scaled probabilities spill 4 of them (a head [H,V] read as it is 20, its logits
    // 13; without stores 8, the recompute 3), which come back in up to 10 four-byte loads per tile, none inside the loop over the
    // steps.
    constexpr bool kRun = Emit != kEmitNone;
    constexpr int kStores = kRun ? TT::FN * (TT::FM / 4) * 2 : 0;
    typedef typename TT::template Loop<WCols, false> Tiles;
    auto tile = [&](int64_t vt) {
        const int tid = TT::fresh_thread();
        return Tiles({W, ldw_bytes, vt * TT::BM, V, 0}, {X, ldx_bytes, n0, T, 0}, lds, tid, kRun ? TT::fresh_thread() : tid);
    };
    for (int64_t vt = vt0; vt < vt1; ++vt) {
        typename TT::Acc acc;
        TT::zero(acc);
        Tiles loop = tile(vt);
        if (!kRun) __syncthreads();  // every wave is done with the previous contents of lds
        if (!kRun || vt == vt0) loop.start(KT);
        loop.template run<kStores, kRun>(KT, acc, vt == vt0, vt + 1 < vt1, [&](auto real) {
            if constexpr (decltype(real)::value) return tile(vt + 1 < vt1 ? vt + 1 : vt);
            else return 0;
        });
        finish_tile(acc, vt);
    }
    // merge the lane groups that hold different rows of the same token, then the WGM
    // wavefronts that share a token column
    float *red_m = reinterpret_cast<float *>(lds);
    float *red_s = red_m + TT::WGM * TT::BN;
    const float4 m4 = state()[0], s4 = state()[1];
    const float m_run[TT::FN] = {m4.x, m4.y, m4.z, m4.w}, s_run[TT::FN] = {s4.x, s4.y, s4.z, s4.w};
    __syncthreads();  // operand stages are no longer read
#pragma unroll
    for (int fn = 0; fn < TT::FN; ++fn) {
        float m = m_run[fn], sum = s_run[fn];
#pragma unroll
        for (int o = TT::MI; o < kWave; o <<= 1) {
            const float om = __shfl_xor(m, o, kWave), os = __shfl_xor(sum, o, kWave);
            const float nm = fmaxf(m, om);
            sum = sum * __builtin_amdgcn_exp2f((m - nm) * kLog2e) + os * __builtin_amdgcn_exp2f((om - nm) * kLog2e);
            m = nm;
        }
        if (lane < TT::MI) {
            const int slot = (TT::wave_id() % TT::WGM) * TT::BN + TT::acc_col(fn);
            red_m[slot] = m;
            red_s[slot] = sum;
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < TT::BN; c += TT::NT) {
        float nm = kNegBig;
#pragma unroll
        for (int w = 0; w < TT::WGM; ++w) nm = fmaxf(nm, red_m[w * TT::BN + c]);
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < TT::WGM; ++w)
            s += red_s[w * TT::BN + c] * __builtin_amdgcn_exp2f((red_m[w * TT::BN + c] - nm) * kLog2e);
        part_max[split * T_pad + n0 + c] = nm;
        part_sum[split * T_pad + n0 + c] = s;
    }
}

// ----------------------------------------------------------------------------
// backward, step 1: recompute the logits tile by tile and emit their bf16 gradient
// ----------------------------------------------------------------------------
// dz[t][v] = g[t] * ([v == target[t]] - exp(z[t][v] - lse[t])), written once, in blocks
// of kBlockK = 64 vocabulary entries: dz[t][v] at dZ + (v / 64) * dz_blk + t * 64 + v % 64
// (dz_blk elements per block = rows of the chunk * 64).  dHidden reads the blocks as a
// k-blocked operand (contraction over v: one block per k-step), dW reads the BM / 64
// blocks of a tile as a matrix with the tokens as rows (contraction over t).  Entries with v >= V and
// tokens past the active rows of their tile are written as zeros.  Token tiles that start at
// or after the number of active rows of this chunk (device value n_act[0] - row_base) are
// skipped altogether.
//
// Workgroups map to (token tile, vocabulary split) as in the forward sweep (SweepMap).  The
// gradients go from the accumulators to memory without a detour through LDS.

template <typename TT, bool WCols>
__global__ void __launch_bounds__(TT::NT, 2)
recompute_dz_kernel(const char *__restrict__ W, int64_t ldw_bytes, int64_t V,
                    const char *__restrict__ X, int64_t ldx_bytes, int64_t T_valid, int KT,
                    const float4 *__restrict__ tok, int64_t nVt, bf16_t *__restrict__ dZ,
                    int64_t dz_blk, const int32_t *__restrict__ n_act, int64_t row_base) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    static_assert(TT::BM % kBlockK == 0 && kBlockK == 4 * TT::MI && TT::FM % 4 == 0,
                  "a block of dZ is four MFMA blocks of vocabulary rows");
    const int act = static_cast<int>(active_rows(n_act, row_base, T_valid));
    if (act == 0) return;
    const uint32_t act_tt = static_cast<uint32_t>((act + TT::BN - 1) / TT::BN);
    const SweepMap map(act_tt, nVt, sweep_splits_wave(act_tt, static_cast<uint32_t>(nVt), kSlots<TT>));
    int split;
    int64_t jt;
    if (!map.tile(blockIdx.x, split, jt)) return;
    const int tn = static_cast<int>(jt);
    const int vt0 = static_cast<int>(map.first_tile(split)), vt1 = static_cast<int>(map.first_tile(split + 1));
    // gradients of one finished tile
    auto emit = [&](typename TT::Acc &acc, int tile_m, int tile_n) {
        const int m0 = tile_m * TT::BM, n0 = tile_n * TT::BN;
        if (m0 + TT::BM > V) {  // ragged last tile: rows past the vocabulary get probability zero
#pragma unroll
            for (int fm = 0; fm < TT::FM; ++fm)
#pragma unroll
                for (int r = 0; r < TT::ACC_R; ++r)
                    if (m0 + TT::acc_row(fm, r) >= V)
#pragma unroll
                        for (int fn = 0; fn < TT::FN; ++fn) acc[fm][fn][r] = -INFINITY;
        }
        // A lane holds runs of four consecutive vocabulary entries (8 bytes of bf16) of ONE token,
        // at offset 32 * (fm % 4) + 8 * group inside that token's 128-byte row of a block of dZ.
        // After an exchange between neighbouring lane groups a lane holds 16 contiguous bytes of
        // two blocks out of four: per store instruction every token gets a contiguous 64-byte half
        // of its row.  (Everything that depends on the lane is derived here from a value the
        // compiler cannot trace, so that none of it is kept in registers across the main loop.)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int grp = lane >> 4, col = lane & 15;
        const int wave_blk = tile_m * (TT::BM / kBlockK) + TT::wave_m0() / kBlockK;
        const int piece = (grp & 1) * 16 + (grp & 2) * 4;  // elements: byte offset 32 * (g & 1) + 8 * (g & 2)
        // the records of this wavefront's 64 tokens, one per lane (handed round with lane shuffles below)
        const float4 rec = tok[static_cast<int64_t>(n0) + TT::wave_n0() + lane];
#pragma unroll
        for (int fn = 0; fn < TT::FN; ++fn) {
            const int src = fn * TT::MI + col;
            const float ag = __shfl(rec.x, src, kWave), nl = __shfl(rec.y, src, kWave);
            const uint32_t ts = __float_as_uint(__shfl(rec.z, src, kWave));
            // the values are formed as |g| * p >= 0; the sign of -g is put on afterwards, two at a time
            const uint32_t sgn = (ts & 0x80000000u) ? 0x80008000u : 0u;
            // where the target's vocabulary row sits among this wave's rows, if it does
            const int dy = static_cast<int>(ts & 0x7fffffffu) - (m0 + TT::wave_m0());
            int fq = 0, rq = 0, gq = 0;
            const bool in_wave = static_cast<unsigned>(dy) < static_cast<unsigned>(TT::WM);
            if (in_wave) TT::locate(dy, fq, rq, gq);
            const bool mine = in_wave && gq == grp;
            bf16_t *row = dZ + static_cast<int64_t>(n0 + TT::wave_n0() + fn * TT::MI + col) * kBlockK + piece;
#pragma unroll
            for (int b = 0; b < TT::FM / 4; ++b) {
                uint32_t lo[4], hi[4];  // bf16 pairs: lo = rows +0,+1, hi = rows +2,+3 of the run of block 4b+q
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float e[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) e[i] = __builtin_amdgcn_exp2f(fmaf(acc[4 * b + q][fn][i], kLog2e, nl));
                    lo[q] = pack_bf16x2_rn(e[0], e[1]);
                    hi[q] = pack_bf16x2_rn(e[2], e[3]);
                }
                if (mine && (fq >> 2) == b) {  // rare: the one-hot term, |g| * (p - 1) before the sign goes on
                    float x = 0.0f;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if ((fq & 3) == q && rq == i) x = acc[4 * b + q][fn][i];
                    const uint32_t v = f32_to_bf16(__builtin_amdgcn_exp2f(fmaf(x, kLog2e, nl)) - ag);
                    const uint32_t keep = (rq & 1) ? 0x0000ffffu : 0xffff0000u, put = (rq & 1) ? v << 16 : v;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if ((fq & 3) == q) {
                            if (rq & 2) hi[q] = (hi[q] & keep) | put;
                            else lo[q] = (lo[q] & keep) | put;
                        }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    lo[q] ^= sgn;
                    hi[q] ^= sgn;
                }
                swap_lane_groups(lo[0], lo[1]);
                swap_lane_groups(hi[0], hi[1]);
                swap_lane_groups(lo[2], lo[3]);
                swap_lane_groups(hi[2], hi[3]);
                bf16_t *out = row + (wave_blk + b) * dz_blk;
                *reinterpret_cast<uint4 *>(out) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
                *reinterpret_cast<uint4 *>(out + kBlockK / 2) = make_uint4(lo[2], hi[2], lo[3], hi[3]);
            }
        }
    };
    for (int tm = vt0; tm < vt1; ++tm) {
        typename TT::Acc acc;
        TT::zero(acc);
        TT::template mainloop<WCols, false>({W, ldw_bytes, static_cast<int64_t>(tm) * TT::BM, V, 0},
                                            {X, ldx_bytes, static_cast<int64_t>(tn) * TT::BN, T_valid, 0}, KT, lds, acc);
        emit(acc, tm, tn);
    }
}

// Host and device ask TailCut (tile_choice.hpp) what is cut off a launch's end.
constexpr int kTailNone = 0, kTailWhole = 1, kTailCut = 2;  // what a launch does about a short last round

// ----------------------------------------------------------------------------
// backward, steps 2 and 3: plain contraction with a store / accumulate epilogue
// ----------------------------------------------------------------------------
// out[row(m)*ldo + n] (=|+=) sum_k A(m,k) B(n,k).  ACols, BCols: the operand has the contraction index as its row index
// (rows then readable up to the next multiple of 8 elements past M or N), otherwise contiguous.  An operand with
// a_blk / b_blk != 0 is stored in blocks of kBlockK = 64 elements of its contiguous index, blk bytes apart, rows
// 128 bytes apart inside a block: that index is k, or (Cols) m or n, of which a tile takes BM / 64 blocks (see
// Tile::Operand).
// With n_act != NULL the extent that holds active tokens is read on the device
// (rows = active_rows(n_act, row_base, .)): limit == kLimitRows keeps only the first
// `rows` rows of A and stores row m at out row row_map[m] (dHidden: scatter back to the
// tokens' own rows); limit == kLimitK contracts only over the first `rows` values of
// the contraction index, rounded up to whole tiles of tokens (dW).  row_scale != NULL (stores that
// do not add to the output): row m of the product is multiplied by row_scale[m] on its way out.
constexpr int kLimitRows = 1, kLimitK = 2;

// With nsplit > 1 (k contiguous in A only) the contraction is cut into nsplit equal runs of k-steps;
// workgroup (tile, part) writes its fp32 partial tile to partials[part][m][n] (leading
// dimension N) and reduce_split_kernel adds the parts in a fixed order: shapes with fewer
// tiles than the chip has compute units still fill it, and the result does not depend on timing.
//
// The instruction gets its operands exchanged (Across), so that a lane holds runs of four consecutive columns of one
// output row.
//
// Epilogue: straight from the accumulators, 16 bytes per lane, 64 contiguous bytes of 16 rows per instruction, and
// nothing that waits between the stores.  (Through LDS, a half tile at a time with a look at the row's place and scale
// per row, every store waited for the one before: 12.6 us per tile in a launch of 16 workgroups, where a compute unit
// stores 256 KB in 2.)  Added to fp32 rows: the old values of the next 16 rows are requested before those of this 16
// are rewritten.
struct GemmOut {
    void *out;
    int64_t ldo, m0, m_end;          // rows m0.. below m_end
    int n0, N;                       // columns n0.. below N
    int dtype, accumulate;
    const int32_t *row_map;          // NULL: rows in place
    const float *row_scale;          // NULL: unscaled
};

// values that may only be aligned to their elements (the hardware takes it)
typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u_t __attribute__((ext_vector_type(4), aligned(2)));

// Adds: sums are added to and rows are in place (dW); otherwise neither is added to.
template <bool Adds, typename TT>
__device__ __forceinline__ void store_tile(const typename TT::Acc &acc, const GemmOut &o) {
    constexpr int R = TT::FM, C = TT::FN;  // 16 x 16 blocks down and across
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // not to be traced: nothing derived from it is to live through the main loop
    const int grp = lane >> 4, col = lane & 15;
    const int n_first = o.n0 + TT::wave_n0();
    const int rows = static_cast<int>(o.m_end), m_wave = static_cast<int>(o.m0) + TT::wave_m0();
    int at[R], place[R];
    float scale[R];
    bool live[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int m = m_wave + i * TT::MI + col;
        live[i] = m < rows;
        place[i] = at[i] = live[i] ? m : rows - 1;  // always a load, none of them behind a branch
        scale[i] = 1.0f;
    }
    if (!Adds && o.row_map)
#pragma unroll
        for (int i = 0; i < R; ++i) place[i] = o.row_map[at[i]];
    if (!Adds && o.row_scale)
#pragma unroll
        for (int i = 0; i < R; ++i) scale[i] = o.row_scale[at[i]];
    auto row = [&](int i) { return place[i] * o.ldo; };  // where this lane's rows begin, in elements
    if (o.dtype == SPO_FP32) {
        float *out = static_cast<float *>(o.out) + n_first + 4 * grp;
        const int n = n_first + 4 * grp;
        if (Adds && o.accumulate) {
            constexpr int G = 2;  // blocks down that are requested at a time
            const bool whole = m_wave + TT::WM <= rows && n_first + TT::WN <= o.N;
            f32x4u_t old[2][G][C];
            if (whole) {  // (a condition on every store would have the next values wait for the stores)
                auto request = [&](int i) {
#pragma unroll
                    for (int j = 0; j < G * C; ++j)
                        old[i / G & 1][j / C][j % C] = *reinterpret_cast<const f32x4u_t *>(out + row(i + j / C) + j % C * TT::MI);
                };
                request(0);
#pragma unroll
                for (int i = 0; i < R; i += G) {
                    if (i + G < R) request(i + G);
#pragma unroll
                    for (int j = 0; j < G * C; ++j)
                        *reinterpret_cast<f32x4u_t *>(out + row(i + j / C) + j % C * TT::MI) =
                            old[i / G & 1][j / C][j % C] + acc[i + j / C][j % C];
                }
            } else {
#pragma unroll
                for (int i = 0; i < R; i += G) {
#pragma unroll
                    for (int j = 0; j < G * C; ++j)
                        if (live[i + j / C] && n + j % C * TT::MI + 3 < o.N)
                            old[0][j / C][j % C] = *reinterpret_cast<const f32x4u_t *>(out + row(i + j / C) + j % C * TT::MI);
                    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): here, or every store below waits for the one before
#pragma unroll
                    for (int j = 0; j < G * C; ++j)
                        if (live[i + j / C] && n + j % C * TT::MI + 3 < o.N)
                            *reinterpret_cast<f32x4u_t *>(out + row(i + j / C) + j % C * TT::MI) =
                                old[0][j / C][j % C] + acc[i + j / C][j % C];
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < C; ++j)
                    if (live[i] && n + j * TT::MI + 3 < o.N)
                        *reinterpret_cast<f32x4u_t *>(out + row(i) + j * TT::MI) = acc[i][j] * scale[i];
        }
        if (n_first + TT::WN > o.N && o.N % 4 != 0) {  // the last columns, where they are no whole run
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    const int c = n + j * TT::MI;
                    if (!live[i] || c + 3 < o.N) continue;
#pragma unroll
                    for (int r = 0; r < 3; ++r)  // (c + 3 is past them)
                        if (c + r < o.N) {
                            float *p = out + row(i) + j * TT::MI + r;
                            *p = Adds && o.accumulate ? *p + acc[i][j][r] : acc[i][j][r] * scale[i];
                        }
                }
        }
        return;
    }
    // bf16, never added to: after an exchange between neighbouring lane groups a lane holds eight consecutive columns
    uint16_t *out = static_cast<uint16_t *>(o.out);
    const int n = n_first + (grp & 1) * TT::MI + (grp & 2) * 4;
    auto eight = [&](int i, int j) {
        uint32_t lo[2], hi[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const auto v = acc[i][j + q] * scale[i];
            lo[q] = pack_bf16x2_rn(v[0], v[1]);
            hi[q] = pack_bf16x2_rn(v[2], v[3]);
        }
        swap_lane_groups(lo[0], lo[1]);
        swap_lane_groups(hi[0], hi[1]);
        return u32x4u_t{lo[0], hi[0], lo[1], hi[1]};
    };
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < C; j += 2) {
            const u32x4u_t w = eight(i, j);
            if (live[i] && n + j * TT::MI + 7 < o.N) *reinterpret_cast<u32x4u_t *>(out + row(i) + n + j * TT::MI) = w;
        }
    if (n_first + TT::WN > o.N && o.N % 8 != 0) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < C; j += 2) {
                const u32x4u_t w = eight(i, j);
                const int c = n + j * TT::MI;
                if (!live[i] || c + 7 < o.N) continue;
#pragma unroll
                for (int r = 0; r < 7; ++r)
                    if (c + r < o.N) out[row(i) + c + r] = static_cast<uint16_t>(w[r / 2] >> (16 * (r & 1)));
            }
    }
}

template <typename TT, bool ACols, bool BCols, bool Clamp>
__global__ void __launch_bounds__(TT::NT, 2)
gemm_store_kernel(const char *__restrict__ A, int64_t lda_bytes, int64_t M, const char *__restrict__ B,
                  int64_t ldb_bytes, int64_t N, int KT, void *__restrict__ out, int64_t ldo, int out_dtype,
                  int accumulate, const int32_t *__restrict__ n_act, int64_t row_base, int limit, int limit_edge,
                  const int32_t *__restrict__ row_map, int64_t a_blk, int64_t b_blk, int nsplit,
                  float *__restrict__ partials, int tail, const float *__restrict__ row_scale, int k_valid) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    static_assert(TT::BM % kBlockK == 0 && TT::BN == TT::BM, "a tile of a blocked operand is a whole number of blocks");
    int64_t m_end = M;
    if (n_act && limit == kLimitRows) m_end = active_rows(n_act, row_base, M);
    // (rows that are not there, known on the device only, leave the ids at the end without a tile)
    const TileOrder ord(ceil_div(m_end, TT::BM), ceil_div(N, TT::BN));
    // kTailWhole: the launch of the whole rounds; kTailCut: the launch of the cut tiles (workgroup
    // i * parts + p takes part p of tile whole + i of the order); both see the same cut
    const TailCut cut(tail == kTailNone ? 0 : ord.tiles(), KT, kSlots<TT>);
    uint32_t i;
    int part;
    if (tail == kTailCut) {
        if (blockIdx.x >= static_cast<unsigned>(cut.rem * cut.parts)) return;
        part = static_cast<int>(blockIdx.x % static_cast<unsigned>(cut.parts));
        i = static_cast<uint32_t>(cut.whole) + blockIdx.x / static_cast<unsigned>(cut.parts);
    } else {
        const uint32_t tiles = static_cast<uint32_t>(tail == kTailWhole ? cut.whole : ord.tiles());
        if (!TileOrder::item(blockIdx.x, tiles * nsplit, i)) return;
        part = static_cast<int>(i / tiles);
        i -= part * tiles;
    }
    int64_t tm, tn;
    ord.at(i, tm, tn);
    const int64_t m0 = tm * TT::BM, n0 = tn * TT::BN;
    if (n_act && limit == kLimitK) {
        const int64_t k_rows = active_rows(n_act, row_base, static_cast<int64_t>(KT) * kBK);
        KT = __builtin_amdgcn_readfirstlane(static_cast<int>(ceil_div(k_rows, limit_edge) * (limit_edge / kBK)));
        if (KT == 0 && accumulate && tail != kTailCut) return;  // nothing to add
    }
    const int KT_all = KT;
    int kt0 = 0;
    const int parts = tail == kTailCut ? cut.parts : nsplit;
    if (parts > 1) {  // this part's run of k-steps
        const int per = (KT + parts - 1) / parts;
        kt0 = part * per;
        KT = KT - kt0 < per ? KT - kt0 : per;
    }
    typename TT::Acc acc;
    TT::zero(acc);
    if (KT > 0) {
        // a k-step starts kBK rows (Cols), blk bytes (blocked) or one stage of 128 bytes further on; the last part's last
        // may not be whole
        const int64_t sa = ACols ? kBK * lda_bytes : a_blk ? a_blk : kBK * 2, sb = BCols ? kBK * ldb_bytes : b_blk ? b_blk : kBK * 2;
        const int64_t Mr = ACols ? (a_blk ? m0 + TT::BM : (M + 7) & ~int64_t(7)) : M;
        const int64_t Nr = BCols ? (b_blk ? n0 + TT::BN : (N + 7) & ~int64_t(7)) : N;
        TT::template mainloop<ACols, BCols, true, Clamp>({A + kt0 * sa, lda_bytes, m0, Mr, a_blk}, {B + kt0 * sb, ldb_bytes, n0, Nr, b_blk}, KT, lds,
                                                         acc, Clamp && kt0 + KT == KT_all ? k_valid : 0);
    }
    GemmOut o{out, ldo, m0, m_end, static_cast<int>(n0), static_cast<int>(N), out_dtype, accumulate, row_map, row_scale};
    if (nsplit > 1 || tail == kTailCut) {  // a part: fp32, in place, unscaled (parts are scaled when they are added)
        const bool tile = tail == kTailCut;  // [part][tile - whole][BM][BN], otherwise [part][M][N]
        const int64_t at = tile ? (static_cast<int64_t>(part) * cut.rem + (i - cut.whole)) * (TT::BM * TT::BN) : static_cast<int64_t>(part) * M * N;
        o = GemmOut{partials + at, tile ? TT::BN : N, tile ? 0 : m0, tile ? TT::BM : m_end, tile ? 0 : static_cast<int>(n0),
                    tile ? TT::BN : static_cast<int>(N), SPO_FP32, 0, nullptr, nullptr};
    }
    store_tile<ACols, TT>(acc, o);
}

// out[row_map[m]][n] = row_scale[m] * sum over the parts (in order) of partials[part][m][n] for m
// below the number of active rows (n_act, row_map, row_scale may each be NULL: all M rows, in
// place, unscaled); four values per thread (N is a multiple of 4 here).
__global__ void __launch_bounds__(256)
reduce_split_kernel(const float *__restrict__ partials, int nsplit, int64_t M, int64_t N,
                    const int32_t *__restrict__ n_act, int64_t row_base, const int32_t *__restrict__ row_map,
                    void *__restrict__ out, int64_t ldo, int out_dtype, const float *__restrict__ row_scale) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t per_row = N / 4, m = i / per_row, n = (i % per_row) * 4;
    if (m >= (n_act ? active_rows(n_act, row_base, M) : M)) return;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    constexpr int U = 8;  // parts requested at a time
    for (int p0 = 0; p0 < nsplit; p0 += U) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u < nsplit ? p0 + u : nsplit - 1;  // always a load, none of them behind a branch
            v[u] = *reinterpret_cast<const float4 *>(partials + (static_cast<int64_t>(p) * M + m) * N + n);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (p0 + u < nsplit) s = make_float4(s.x + v[u].x, s.y + v[u].y, s.z + v[u].z, s.w + v[u].w);
    }
    if (row_scale) {
        const float sc = row_scale[m];
        s = make_float4(s.x * sc, s.y * sc, s.z * sc, s.w * sc);
    }
    const int64_t mo = row_map ? row_map[m] : m;
    if (out_dtype == SPO_FP32) {
        *reinterpret_cast<float4 *>(static_cast<float *>(out) + mo * ldo + n) = s;
    } else {
        *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(out) + mo * ldo + n) =
            make_uint2(pack_bf16x2_rn(s.x, s.y), pack_bf16x2_rn(s.z, s.w));
    }
}

// The cut tiles of a launch's short last round (TailCut): out[row_map[m]][n] (=|+=) row_scale[m] times
// the sum, in order, of partials[part][tile - whole][m % BM][n % BN] over the parts.  The launch is
// sized for the most tiles a cut can have; n_act (with limit == kLimitRows), row_map and row_scale
// may be NULL.  Four values per thread.
template <typename TT>
__global__ void __launch_bounds__(256)
reduce_tail_kernel(const float *__restrict__ partials, int64_t M, int64_t N, int64_t KT, const int32_t *__restrict__ n_act,
                   int64_t row_base, int limit, const int32_t *__restrict__ row_map, void *__restrict__ out, int64_t ldo,
                   int out_dtype, int accumulate, const float *__restrict__ row_scale) {
    constexpr int64_t per_tile = TT::BM * TT::BN / 4;
    const int64_t m_end = n_act && limit == kLimitRows ? active_rows(n_act, row_base, M) : M;
    const TileOrder ord(ceil_div(m_end, TT::BM), ceil_div(N, TT::BN));
    const TailCut cut(ord.tiles(), KT, kSlots<TT>);
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t tl = i / per_tile, r = (i % per_tile) / (TT::BN / 4), c = (i % (TT::BN / 4)) * 4;
    if (tl >= cut.rem) return;
    int64_t tm, tn;
    ord.at(static_cast<uint32_t>(cut.whole + tl), tm, tn);
    const int64_t m = tm * TT::BM + r, n = tn * TT::BN + c;
    if (m >= m_end || n >= N) return;
    float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int p = 0; p < cut.parts; ++p) {
        const float4 v = *reinterpret_cast<const float4 *>(
            partials + ((static_cast<int64_t>(p) * cut.rem + tl) * TT::BM + r) * TT::BN + c);
        sum = make_float4(sum.x + v.x, sum.y + v.y, sum.z + v.z, sum.w + v.w);
    }
    if (row_scale) {
        const float sc = row_scale[m];
        sum = make_float4(sum.x * sc, sum.y * sc, sum.z * sc, sum.w * sc);
    }
    const int64_t mo = row_map ? row_map[m] : m;
    const float e[4] = {sum.x, sum.y, sum.z, sum.w};
    const bool vec = ldo % 4 == 0 && n + 3 < N && reinterpret_cast<uintptr_t>(out) % 16 == 0;
    if (out_dtype == SPO_FP32) {
        float *o = static_cast<float *>(out) + mo * ldo + n;
        if (vec) {
            float4 w = sum;
            if (accumulate) {
                const float4 old = *reinterpret_cast<const float4 *>(o);
                w = make_float4(old.x + sum.x, old.y + sum.y, old.z + sum.z, old.w + sum.w);
            }
            *reinterpret_cast<float4 *>(o) = w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (n + j < N) o[j] = accumulate ? o[j] + e[j] : e[j];
        }
    } else {  // bf16 outputs are never added to
        bf16_t *o = static_cast<bf16_t *>(out) + mo * ldo + n;
        if (vec) {
            *reinterpret_cast<uint2 *>(o) = make_uint2(pack_bf16x2_rn(e[0], e[1]), pack_bf16x2_rn(e[2], e[3]));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (n + j < N) o[j] = f32_to_bf16(e[j]);
        }
    }
}

// ----------------------------------------------------------------------------
// one-call forward + backward: logit gradients from the logits the forward stored
// ----------------------------------------------------------------------------
// dZ[j][v] = g * ([v == target] - exp(z[v] - lse)) for the active tokens j of a piece of the
// batch, from the fp16 offsets written by fwd_sweep_kernel<kEmitLogits> (z = stored value + offset of
// the entry's part of a tile, bph blocks of 64), into the blocked bf16 layout the two contractions read.
// Row j of the output is token act_idx[j] of the piece; tok[j] is its record (see
// gather_chunk_kernel); rows from the number of active tokens up to the next multiple of `edge`
// (a tile's tokens) are written as zeros, rows beyond are left alone (no contraction reads them).  A wavefront
// moves 8 rows x 128 bytes of one 64-entry block per step (16 bytes per lane), a workgroup 32
// rows, over `per_wg` consecutive blocks.
__global__ void __launch_bounds__(256)
dz_from_logits_kernel(const uint16_t *__restrict__ Z, int64_t z_blk, const float *__restrict__ offs, int64_t off_stride,
                      const int32_t *__restrict__ act_idx,
                      const int32_t *__restrict__ n_act, int64_t rows_cap, const float4 *__restrict__ tok,
                      bf16_t *__restrict__ dZ, int64_t dz_blk, int64_t n_blk, int per_wg, int bph, int edge) {
    const int64_t act = active_rows(n_act, 0, rows_cap);
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 32 + (threadIdx.x >> 3);
    if (static_cast<int64_t>(blockIdx.x) * 32 >= (act + edge - 1) / edge * edge) return;
    const int part = threadIdx.x & 7;  // which 8 of the block's 64 entries
    const bool live = j < act;
    const int64_t src = live ? act_idx[j] : 0;
    const float4 rec = live ? tok[j] : make_float4(0.0f, -INFINITY, __uint_as_float(0x7fffffffu), 0.0f);
    const uint32_t ts = __float_as_uint(rec.z);
    const uint32_t sgn = (ts & 0x80000000u) ? 0x80008000u : 0u;  // the values are formed as |g| * p; the sign of -g goes on in pairs
    const int64_t y = ts & 0x7fffffffu;
    const int64_t b0 = static_cast<int64_t>(blockIdx.y) * per_wg;
    for (int64_t b = b0; b < b0 + per_wg && b < n_blk; ++b) {
        uint4 o = make_uint4(0u, 0u, 0u, 0u);
        if (live) {
            const float off = offs[(b / bph) * off_stride + src];
            const float c = fmaf(off, kLog2e, rec.y);  // log2|g| + (offset - lse) * log2(e)
            const uint4 zz = *reinterpret_cast<const uint4 *>(Z + b * z_blk + src * kBlockK + part * 8);
            const uint32_t w[4] = {zz.x, zz.y, zz.z, zz.w};
            float e[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                typedef _Float16 h2 __attribute__((ext_vector_type(2)));
                const h2 h = __builtin_bit_cast(h2, w[i]);
                e[2 * i] = __builtin_amdgcn_exp2f(fmaf(static_cast<float>(h.x), kLog2e, c));
                e[2 * i + 1] = __builtin_amdgcn_exp2f(fmaf(static_cast<float>(h.y), kLog2e, c));
            }
            const int64_t dy = y - (b * kBlockK + part * 8);
            if (dy >= 0 && dy < 8) {  // the one-hot term: |g| * (p - 1) before the sign goes on
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (dy == i) e[i] -= rec.x;
            }
            o = make_uint4(pack_bf16x2_rn(e[0], e[1]) ^ sgn, pack_bf16x2_rn(e[2], e[3]) ^ sgn,
                           pack_bf16x2_rn(e[4], e[5]) ^ sgn, pack_bf16x2_rn(e[6], e[7]) ^ sgn);
        }
        *reinterpret_cast<uint4 *>(dZ + b * dz_blk + j * kBlockK + part * 8) = o;
    }
}

// ----------------------------------------------------------------------------
// one-call forward + backward without a loss mask: the sweep stores what the contractions read
// ----------------------------------------------------------------------------
// The reference of token t is r_t = z_t[y_t] - old_logp_t: the log-sum-exp the token would have if
// the policy had not moved since the behaviour policy sampled it.  Both terms are known before
// the sweep (the logit of the sampled token costs one dot product).  Then
//   Q[t][v] = exp(z[t][v] - r_t) = softmax(z_t)[v] / ratio_t,   ratio_t = exp(logp_t - old_logp_t),
// lies near the probabilities whatever the logits' scale (bf16 keeps 8 bits of each entry), and
//   dZ[t][v] = g_t ([v == y_t] - softmax[v]) = c_t (Q[t][v] - [v == y_t] / ratio_t),  c_t = -g_t ratio_t.
// So once a piece's log-probs are known, one entry per token is rewritten (Q[t][y_t] = exp(old_logp_t)
// by construction, so the new value is formed afresh in fp32 and rounded once) and the contractions
// run on Q itself: dHidden_t = c_t (Q_t W), dW = Q^T (c X).  No pass over the stored tile is needed;
// the price is that rows of tokens without a gradient (c_t = 0) are multiplied like the others,
// which is why this form serves batches without a loss mask.

// dst[t][:] = bf16(c[t] * src[t][:]) for t < rows_pad (c is 0 from the last valid row on: zeros).
// One workgroup per row; H is a multiple of 64.
template <typename T_>
__global__ void __launch_bounds__(256)
scale_rows_kernel(const T_ *__restrict__ src, const float *__restrict__ c, int64_t rows, int64_t H,
                  bf16_t *__restrict__ dst) {
    const int64_t t = blockIdx.x;
    const float ct = c[t];
    const bool live = t < rows && ct != 0.0f;
    uint2 *out = reinterpret_cast<uint2 *>(dst + t * H);
    for (int i = threadIdx.x; i < H / 4; i += 256) {
        float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (live) {
            if constexpr (sizeof(T_) == 2) {
                const uint2 v = reinterpret_cast<const uint2 *>(src + t * H)[i];
                x[0] = __uint_as_float(v.x << 16); x[1] = __uint_as_float(v.x & 0xffff0000u);
                x[2] = __uint_as_float(v.y << 16); x[3] = __uint_as_float(v.y & 0xffff0000u);
            } else {
                const float4 v = reinterpret_cast<const float4 *>(src + t * H)[i];
                x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
            }
        }
        out[i] = make_uint2(pack_bf16x2_rn(x[0] * ct, x[1] * ct), pack_bf16x2_rn(x[2] * ct, x[3] * ct));
    }
}

// ----------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------
// The kernels use more dynamic LDS than the default limit allows.  The attribute belongs
// to the current device's copy of the kernel, so it is set on every call (a host-side
// table lookup) rather than remembered in a process-wide flag.
template <typename K>
static int allow_lds(K kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess
               ? SPO_OK : SPO_EHIP;
}

static inline int64_t round_up(int64_t x, int64_t a) { return ceil_div(x, a) * a; }
static inline unsigned grid1(int64_t n, int per = 256) { return static_cast<unsigned>(ceil_div(n, per)); }

// the logits of T tokens, Kc values long each (forward sweep, recompute)
static bool small_sweep(int64_t T, int64_t V, int64_t Kc) {
    double time[2];
    for (int small = 0; small < 2; ++small) {
        const int64_t nTt = std::max<int64_t>(ceil_div(T, tile_edge(small)), 1), nVt = ceil_div(V, tile_edge(small));
        const int64_t ns = sweep_splits(nTt, nVt, tile_slots(small)), rounds = ceil_div(nTt * ns, tile_slots(small)) * ceil_div(nVt, ns);
        time[small] = launch_time(kSweepTimes, small, static_cast<double>(rounds), nTt * ns, Kc / kBK, V * Kc * 2);
    }
    return small_is_faster(kSweepTimes, time);
}
static_assert(TL::BN <= kTileRows && TS::BN <= kTileRows && kBK <= 64 && kBlockK == 64 && kMostChunkTokens % TL::BN == 0, "what head_form.hpp counts");
static bool direct_head(const spo_pg_desc *d) {
    return direct_head(d->dtype == SPO_BF16, d->w_layout == SPO_W_HV, d->T, d->H, d->V);
}

struct FwdPlan {
    bool small;
    int64_t nTt, nVt, T_pad, Kc;  // Kc: contraction length seen by the main loop
    int nsplit;
    int64_t nblk_tok;
    // workspace
    float *part_max, *part_sum, *z_target;
    FwdPartial *partials;
    uint32_t *done;
    bf16_t *Xs, *Ws;  // split-expanded operands (fp32)
    void *Wvh;        // [V,H] copy of a head given as [H,V]
    size_t bytes;
};

// room for the [V,H] copy of a head given as [H,V]
static void *take_head_copy(Arena &a, const spo_pg_desc *d) {
    if (d->w_layout != SPO_W_HV) return nullptr;
    char *p = a.take<char>(static_cast<size_t>(d->V) * d->H * (d->dtype == SPO_FP32 ? 4 : 2));
    return p;
}

// roomy: with room for the partial results of small tiles, without which they are not taken (workspaces of the size that
// large tiles need are accepted as well).
static FwdPlan plan_fwd(const spo_pg_desc *d, void *ws, bool roomy) {
    FwdPlan p;
    p.Kc = d->dtype == SPO_FP32 ? kSplitTerms * d->H : d->H;
    p.small = roomy && small_sweep(d->T, d->V, p.Kc);
    const int64_t edge = tile_edge(p.small);
    p.nTt = ceil_div(d->T, edge);
    p.nVt = ceil_div(d->V, edge);
    p.T_pad = p.nTt * edge;
    p.nsplit = sweep_splits(p.nTt, p.nVt, tile_slots(p.small));
    p.nblk_tok = ceil_div(std::max<int64_t>(d->T, 1), kTokThreads);
    Arena a(ws);
    const size_t room = static_cast<size_t>(sweep_room(d->T, d->V, roomy));  // [nsplit][T_pad] and more
    p.part_max = a.take<float>(room);
    p.part_sum = a.take<float>(room);
    p.z_target = a.take<float>(round_up(d->T, TL::BN));
    p.partials = a.take<FwdPartial>(p.nblk_tok);
    p.done = a.take<uint32_t>(1);
    p.Xs = p.Ws = nullptr;
    if (d->dtype == SPO_FP32) {
        p.Xs = a.take<bf16_t>(static_cast<size_t>(std::max<int64_t>(d->T, 1)) * p.Kc);
        p.Ws = a.take<bf16_t>(static_cast<size_t>(d->V) * p.Kc);
    }
    p.Wvh = take_head_copy(a, d);
    p.bytes = a.used;
    return p;
}

static int check_fused(const spo_pg_desc *d) {
    if (reinterpret_cast<uintptr_t>(d->hidden) % 16 || reinterpret_cast<uintptr_t>(d->W) % 16) return SPO_EINVAL;
    return SPO_OK;
}

int fused_fwd_workspace(const spo_pg_desc *d, size_t *bytes) {
    *bytes = plan_fwd(d, nullptr, true).bytes;
    return SPO_OK;
}

// The sweep of one piece of T tokens on tiles TT; W: the head as the sweep reads it (cols: [H,V]).
struct Sweep {
    const void *W;
    int64_t V, Kc;
    bool cols;
    const void *X;
    int64_t T;
    float *part_max, *part_sum;
    uint16_t *Z;
    int64_t z_blk;
    float *offs;
};
template <int Emit, typename TT, bool WCols>
static int launch_sweep(const Sweep &w, const SweepMap &map, hipStream_t s) {
    auto *kernel = fwd_sweep_kernel<Emit, TT, WCols>;
    constexpr int lds = kSweepLds<TT>(Emit);
    if (int rc = allow_lds(kernel, lds)) return rc;
    ScopedKernelTimer timer(kTimeFwdSweep, s);
    kernel<<<static_cast<unsigned>(map.blocks()), TT::NT, lds, s>>>(
        static_cast<const char *>(w.W), (WCols ? w.V : w.Kc) * 2, w.V, static_cast<const char *>(w.X), w.Kc * 2, w.T,
        static_cast<int>(w.Kc / kBK), map.ns, map.nTt, map.nVt, map.nTt * TT::BN, w.part_max, w.part_sum, w.Z, w.z_blk, w.offs);
    return SPO_OK;
}
template <int Emit>
static int launch_sweep(const Sweep &w, bool small, const SweepMap &map, hipStream_t s) {
    if (small) return w.cols ? launch_sweep<Emit, TS, true>(w, map, s) : launch_sweep<Emit, TS, false>(w, map, s);
    return w.cols ? launch_sweep<Emit, TL, true>(w, map, s) : launch_sweep<Emit, TL, false>(w, map, s);
}

int fused_fwd(const spo_pg_desc *d, float *loss, float *logp, float *lse, float *stats, void *ws,
              size_t ws_bytes, hipStream_t s) {
    int rc = check_fused(d);
    if (rc) return rc;
    FwdPlan p = plan_fwd(d, ws, true);
    if (ws_bytes < p.bytes) p = plan_fwd(d, ws, false);
    if (ws_bytes < p.bytes) return SPO_EWORKSPACE;
    if (d->T > 0) {
        const bool fp32 = d->dtype == SPO_FP32, direct = direct_head(d), hv = d->w_layout == SPO_W_HV;
        PrepJobs jobs = prep_head_jobs(d, direct ? nullptr : p.Wvh, p.Ws, nullptr);
        prep_rows(jobs, d, d->hidden, d->T, p.Xs);
        launch_prep_with_targets(d, jobs, p.z_target, nullptr, 0, p.done, s);
        Sweep w{};
        w.W = fp32 ? p.Ws : direct || !p.Wvh ? d->W : p.Wvh;
        w.V = d->V;
        w.Kc = p.Kc;
        w.cols = direct && hv;
        w.X = fp32 ? static_cast<const void *>(p.Xs) : d->hidden;
        w.T = d->T;
        w.part_max = p.part_max;
        w.part_sum = p.part_sum;
        if ((rc = launch_sweep<kEmitNone>(w, p.small, SweepMap(p.nTt, p.nVt, p.nsplit), s))) return rc;
    }
    const TokenShape tok = token_shape(p.nsplit, p.nblk_tok);
    token_loss_kernel<<<tok.blocks, tok.threads, 0, s>>>(
        p.part_max, p.part_sum, p.nsplit, tok.ways, p.T_pad, p.z_target, token_inputs(d, 0, d->T), logp, lse, p.partials,
        TokenGrad{}, p.nblk_tok, p.nblk_tok, p.done, loss, stats);
    return launch_status();
}

struct BwdPlan {
    int64_t Tc, V_pad, V_blk, Kc, T_pad;  // V rounded up to a k-step (64) and to whole tiles (256)
    double *count;
    float *g, *dW_acc;
    bf16_t *WT, *Xc, *dZ, *Xs, *Ws;  // Xc: the gathered rows in bf16
    void *Wvh;                 // [V,H] copy of a head given as [H,V]
    int32_t *act_idx, *n_act;  // active-token list, its length
    float4 *tok;               // per-chunk records (g, -lse*log2e, target) of the gathered rows
    float *part_tiles;         // room for kTailTiles fp32 tiles: partial results of a cut contraction (see launch_gemm)
    size_t bytes;
};

static BwdPlan plan_bwd(const spo_pg_desc *d, int64_t chunk_tokens, void *ws, bool need_dw_acc) {
    BwdPlan p;
    const int64_t Tmax = round_up(std::max<int64_t>(d->T, 1), TL::BN);
    p.T_pad = Tmax;
    p.V_pad = round_up(d->V, kBK);
    p.V_blk = round_up(d->V, TL::BM);
    const int64_t tc = chunk_tokens > 0 ? round_up(chunk_tokens, TL::BN) : default_chunk_tokens(d->H, p.V_blk);
    p.Tc = std::min({tc, Tmax, kMostChunkTokens});
    p.Kc = d->dtype == SPO_FP32 ? kSplitTerms * d->H : d->H;
    Arena a(ws);
    p.count = a.take<double>(1);
    p.g = a.take<float>(p.T_pad);
    p.act_idx = a.take<int32_t>(p.T_pad);
    p.n_act = a.take<int32_t>(1);
    p.tok = a.take<float4>(p.Tc);
    p.Xc = a.take<bf16_t>(static_cast<size_t>(p.Tc) * d->H);
    p.WT = a.take<bf16_t>(static_cast<size_t>(d->H) * p.V_blk);   // [V_blk / 64][H][64]
    p.dZ = a.take<bf16_t>(static_cast<size_t>(p.Tc) * p.V_blk);  // [V_blk / 64][rows of the chunk][64]
    p.Xs = p.Ws = nullptr;
    p.dW_acc = nullptr;
    if (d->dtype == SPO_FP32) {
        p.Xs = a.take<bf16_t>(static_cast<size_t>(p.Tc) * p.Kc);
        p.Ws = a.take<bf16_t>(static_cast<size_t>(d->V) * p.Kc);
    }
    // the logits of a bf16 head are formed from rows per vocabulary entry; an fp32 head is split from any layout
    p.Wvh = d->dtype == SPO_BF16 ? take_head_copy(a, d) : nullptr;
    if (need_dw_acc && d->T > p.Tc) p.dW_acc = a.take<float>(static_cast<size_t>(d->V) * d->H);
    p.part_tiles = a.take<float>(static_cast<size_t>(kTailTiles) * TL::BM * TL::BN);
    p.bytes = a.used;
    return p;
}

// What a query adds where its chunk holds all tokens and the fp32 sum of a bf16 d_W is left out: a call with
// shorter chunks needs the sum, and a workspace that serves long chunks serves short ones.  (Up to a tile of tokens
// every choice is one chunk.)
static size_t room_for_shorter_chunks(const spo_pg_desc *d, int64_t chunk) {
    return d->T > TL::BN && d->T <= chunk ? align_up(static_cast<size_t>(d->V) * d->H * sizeof(float), 256) : 0;
}

int fused_bwd_workspace(const spo_pg_desc *d, int64_t chunk_tokens, size_t *bytes) {
    // sized for the larger case (bf16 d_W needs an fp32 accumulator)
    const BwdPlan p = plan_bwd(d, chunk_tokens, nullptr, true);
    *bytes = p.bytes + room_for_shorter_chunks(d, p.Tc);
    return SPO_OK;
}

// `partials`: room for kTailTiles fp32 tiles: the parts of a contraction cut nsplit times (at most as many part
// tiles as the chip has units), or those of a short last round of tiles, which is cut along the
// contraction (TailCut): 9504 tiles of dW on 256 units take 37 rounds and an eighth instead of 38,
// and a dHidden launch whose number of active rows leaves a round nearly empty loses a fifth of a
// round instead of a whole one.  Where the tile count depends on n_act the two extra launches
// are made in any case and find out on the device that there is nothing to cut.
struct Gemm {
    const bf16_t *A;
    int64_t lda, M;
    const bf16_t *B;
    int64_t ldb, N, K;                  // K: whole steps; with k_valid the last has that many elements
    void *out;
    int64_t ldo;
    int out_dtype, accumulate;
    const int32_t *n_act;
    int64_t row_base;
    int limit, limit_edge;
    const int32_t *row_map;
    int64_t a_blk, b_blk;               // elements
    const float *row_scale;
    int k_valid;
};
template <typename TT, bool ACols, bool BCols, bool Clamp>
static int launch_gemm(const Gemm &g, hipStream_t s, int nsplit, float *partials) {
    auto *kernel = gemm_store_kernel<TT, ACols, BCols, Clamp>;
    if (int rc = allow_lds(kernel, TT::LDS_BYTES)) return rc;
    constexpr int slots = kSlots<TT>;
    const int64_t tiles = ceil_div(g.M, TT::BM) * ceil_div(g.N, TT::BN), steps = ceil_div(g.K, kBK);
    const bool rows_on_device = g.n_act && g.limit == kLimitRows;
    const TailCut host_cut(tiles, steps, slots);
    const bool cut = nsplit == 1 && (rows_on_device ? tiles > slots : host_cut.rem > 0);
    auto launch = [&](int64_t blocks, int splits, int tail, const float *row_scale) {
        kernel<<<static_cast<unsigned>(blocks), TT::NT, TT::LDS_BYTES, s>>>(
            reinterpret_cast<const char *>(g.A), g.lda * 2, g.M, reinterpret_cast<const char *>(g.B), g.ldb * 2, g.N,
            static_cast<int>(steps), g.out, g.ldo, g.out_dtype, g.accumulate, g.n_act, g.row_base, g.limit, g.limit_edge, g.row_map,
            g.a_blk * 2, g.b_blk * 2, splits, partials, tail, row_scale, g.k_valid);
    };
    if (!cut || rows_on_device || host_cut.whole > 0)
        launch(TileOrder::blocks(tiles * nsplit), nsplit, cut ? kTailWhole : kTailNone, g.row_scale);
    if (nsplit > 1)
        reduce_split_kernel<<<grid1(g.M * (g.N / 4)), 256, 0, s>>>(partials, nsplit, g.M, g.N, g.n_act, g.row_base, g.row_map, g.out,
                                                                   g.ldo, g.out_dtype, g.row_scale);
    if (cut) {
        // (on the device: sized for the most a cut can be, half of the slots' worth of tiles, as many part-tiles as slots)
        launch(rows_on_device ? slots : host_cut.rem * host_cut.parts, 1, kTailCut, nullptr);
        const int rem_most = rows_on_device ? slots / 2 : host_cut.rem;
        reduce_tail_kernel<TT><<<grid1(rem_most * (TT::BM * TT::BN / 4)), 256, 0, s>>>(
            partials, g.M, g.N, steps, g.n_act, g.row_base, g.limit, g.row_map, g.out, g.ldo, g.out_dtype, g.accumulate,
            g.row_scale);
    }
    return SPO_OK;
}

// The gathered rows of a chunk (see gather_chunk_kernel), and d_hidden[0..zero_rows) (NULL: not) cleared.
static void launch_gather(const spo_pg_desc *d, const void *X, const int32_t *act_idx, const int32_t *n_act, int64_t row_base,
                          int64_t rows, const int32_t *target, const float *lse, const float *g, bf16_t *Xc, bf16_t *Xs,
                          float4 *tok, void *d_hidden, int d_hidden_dtype, int64_t zero_rows, hipStream_t s) {
    if (!d_hidden) zero_rows = 0;
    const dim3 grid = fold_grid(ceil_div(std::max(rows, zero_rows), 4));
    const int64_t zero_bytes = d->H * (d_hidden_dtype == SPO_FP32 ? 4 : 2);
    if (d->dtype == SPO_FP32)
        gather_chunk_kernel<float><<<grid, 256, 0, s>>>(static_cast<const float *>(X), d->H, act_idx, n_act, row_base, rows,
                                                        target, lse, g, Xc, Xs, tok, static_cast<char *>(d_hidden), zero_rows,
                                                        zero_bytes);
    else
        gather_chunk_kernel<bf16_t><<<grid, 256, 0, s>>>(static_cast<const bf16_t *>(X), d->H, act_idx, n_act, row_base, rows,
                                                         target, lse, g, Xc, Xs, tok, static_cast<char *>(d_hidden), zero_rows,
                                                         zero_bytes);
}

// The logit gradients of the active ones of Tcp gathered rows X; W: the head as it reads it (cols: [H,V]).
template <typename TT, bool WCols>
static int launch_recompute(const spo_pg_desc *d, const void *W, const bf16_t *X, int64_t Kc, int64_t Tcp, const float4 *tok, bf16_t *dZ,
                            const int32_t *n_act, int64_t row_base, hipStream_t s) {
    auto *kernel = recompute_dz_kernel<TT, WCols>;
    if (int rc = allow_lds(kernel, TT::LDS_BYTES)) return rc;
    const int64_t nVt = ceil_div(d->V, TT::BM), wgs = sweep_blocks_max(Tcp / TT::BN, nVt);
    ScopedKernelTimer timer(kTimeRecompute, s);
    kernel<<<static_cast<unsigned>(wgs), TT::NT, TT::LDS_BYTES, s>>>(
        static_cast<const char *>(W), (WCols ? d->V : Kc) * 2, d->V, reinterpret_cast<const char *>(X), Kc * 2, Tcp,
        static_cast<int>(Kc / kBK), tok, nVt, dZ, Tcp * kBlockK, n_act, row_base);
    return SPO_OK;
}
static int launch_recompute(const spo_pg_desc *d, const void *W, bool cols, const bf16_t *X, int64_t Kc, int64_t Tcp, bool small,
                            const float4 *tok, bf16_t *dZ, const int32_t *n_act, int64_t row_base, hipStream_t s) {
    if (small) return cols ? launch_recompute<TS, true>(d, W, X, Kc, Tcp, tok, dZ, n_act, row_base, s)
                           : launch_recompute<TS, false>(d, W, X, Kc, Tcp, tok, dZ, n_act, row_base, s);
    return cols ? launch_recompute<TL, true>(d, W, X, Kc, Tcp, tok, dZ, n_act, row_base, s)
                : launch_recompute<TL, false>(d, W, X, Kc, Tcp, tok, dZ, n_act, row_base, s);
}

// dHidden of M rows (of Tcp in the blocks of dZ): every part of the vocabulary, the head as WT, or as it was given (NULL).
static int launch_dhidden(const spo_pg_desc *d, const bf16_t *dZ, int64_t M, int64_t Tcp, const bf16_t *WT, int64_t V_pad, void *out,
                          int out_dtype, const int32_t *n_act, int64_t row_base, const int32_t *row_map, const float *row_scale,
                          float *partials, hipStream_t s) {
    const int64_t H = d->H, V = d->V;
    const bool small = small_dhidden(M, H, V_pad), hv = d->w_layout == SPO_W_HV;
    const int parts = dhidden_parts(M, H, V_pad, small);
    Gemm g{};
    g.A = dZ;
    g.lda = kBlockK;
    g.M = M;
    g.a_blk = Tcp * kBlockK;
    g.N = H;
    g.K = V_pad;
    g.out = out;
    g.ldo = H;
    g.out_dtype = out_dtype;
    g.n_act = n_act;
    g.row_base = row_base;
    g.limit = kLimitRows;
    g.row_map = row_map;
    g.row_scale = row_scale;
    ScopedKernelTimer timer(kTimeDHidden, s);
    if (WT) {  // both operands k-blocked over the vocabulary: a stage of a tile is 32 KiB contiguous
        g.B = WT;
        g.ldb = kBlockK;
        g.b_blk = H * kBlockK;
        return small ? launch_gemm<TS, false, false, false>(g, s, parts, partials) : launch_gemm<TL, false, false, false>(g, s, parts, partials);
    }
    g.B = static_cast<const bf16_t *>(d->W);
    g.ldb = hv ? V : H;
    g.k_valid = static_cast<int>(V % kBK);
    if (hv) return small ? launch_gemm<TS, false, false, true>(g, s, parts, partials) : launch_gemm<TL, false, false, true>(g, s, parts, partials);
    return small ? launch_gemm<TS, false, true, true>(g, s, parts, partials) : launch_gemm<TL, false, true, true>(g, s, parts, partials);
}

// dW (=|+=) dZ^T X over Tcp tokens, or the first of them that are active, rounded up to edge.
static int launch_dW(const spo_pg_desc *d, const bf16_t *dZ, const bf16_t *X, int64_t Tcp, int64_t edge, void *out, int out_dtype,
                     int accumulate, const int32_t *n_act, int64_t row_base, float *partials, hipStream_t s) {
    const bool hv = d->w_layout == SPO_W_HV;
    Gemm g{};
    g.A = hv ? X : dZ;
    g.B = hv ? dZ : X;
    g.lda = hv ? d->H : kBlockK;
    g.ldb = hv ? kBlockK : d->H;
    g.M = hv ? d->H : d->V;
    g.N = hv ? d->V : d->H;
    (hv ? g.b_blk : g.a_blk) = Tcp * kBlockK;
    g.K = Tcp;
    g.out = out;
    g.ldo = g.N;
    g.out_dtype = out_dtype;
    g.accumulate = accumulate;
    g.n_act = n_act;
    g.row_base = row_base;
    g.limit = kLimitK;
    g.limit_edge = static_cast<int>(edge);
    ScopedKernelTimer timer(kTimeDW, s);
    return small_dW(Tcp, d->H, d->V) ? launch_gemm<TS, true, true, false>(g, s, 1, partials) : launch_gemm<TL, true, true, false>(g, s, 1, partials);
}

int fused_bwd(const spo_pg_desc *d, const float *logp, const float *lse, float grad_loss, void *d_hidden,
              int d_hidden_dtype, void *d_W, int d_W_dtype, int accumulate_dW, int64_t chunk_tokens, void *ws,
              size_t ws_bytes, hipStream_t s) {
    int rc = check_fused(d);
    if (rc) return rc;
    if (accumulate_dW && d_W && d_W_dtype != SPO_FP32) return SPO_EINVAL;
    const BwdPlan p = plan_bwd(d, chunk_tokens, ws, d_W && d_W_dtype == SPO_BF16);
    // a bf16 d_W is summed in fp32 beside it, unless one chunk holds all tokens: its tiles are rounded as they are stored
    // (an fp32 d_W of 151936 x 4096 written, read and rounded again: 2 ms)
    const bool need_acc = p.dW_acc != nullptr;
    if (ws_bytes < p.bytes) return SPO_EWORKSPACE;
    const int64_t H = d->H, V = d->V, T = d->T;
    void *dW_sum = need_acc ? p.dW_acc : d_W;
    const int dW_sum_dtype = need_acc ? SPO_FP32 : d_W_dtype;
    if (T == 0) {
        if (d_W && !accumulate_dW) {
            const int64_t words = d_W_dtype == SPO_FP32 ? V * H : V * H / 2;
            fill_zero_kernel<<<grid1(words), 256, 0, s>>>(static_cast<uint32_t *>(d_W), words);
        }
        return launch_status();
    }
    // vocabulary-major head for the recompute, hidden-major head for dHidden; the gradient factors and the
    // tokens that carry one, in order: the chunks below run over this list
    const bool direct = direct_head(d), hv = d->w_layout == SPO_W_HV;
    PrepJobs jobs = prep_head_jobs(d, direct ? nullptr : p.Wvh, p.Ws, d_hidden && !direct ? p.WT : nullptr);
    const bool grad_inside = T <= kPrepGradTokens;
    if (grad_inside) {
        jobs.g = p.g;
        jobs.logp = logp;
        jobs.in = token_inputs(d, 0, T);
        jobs.grad_loss = grad_loss;
        jobs.act_idx = p.act_idx;
        jobs.n_act = p.n_act;
    }
    launch_prep(d, jobs, s);
    if (!grad_inside) {
        launch_grad_scale(d, logp, p.T_pad, grad_loss, p.count, p.g, s);
        compact_active_kernel<<<1, 1024, 0, s>>>(p.g, T, p.act_idx, p.n_act);
    }
    const void *Wk = d->dtype == SPO_FP32 ? p.Ws : direct || !p.Wvh ? d->W : p.Wvh;
    for (int64_t t0 = 0, c = 0; t0 < T; t0 += p.Tc, ++c) {
        // rows [t0, t0 + Tcp) of the compact order; how many of them exist is known on the
        // device only, so every launch is sized for the most there can be and trims itself
        const int64_t Tv = std::min(p.Tc, T - t0);
        const bool small = small_sweep(Tv, V, p.Kc);
        const int64_t edge = tile_edge(small), Tcp = round_up(Tv, edge);
        // (the first chunk's launch also clears d_hidden: later ones would clear what earlier ones wrote)
        launch_gather(d, d->hidden, p.act_idx, p.n_act, t0, Tcp, d->target, lse, p.g, d->dtype == SPO_BF16 || d_W ? p.Xc : nullptr,
                      p.Xs, p.tok, c == 0 ? d_hidden : nullptr, d_hidden_dtype, T, s);
        const bf16_t *Xk = d->dtype == SPO_FP32 ? p.Xs : p.Xc, *Xrows = p.Xc;  // operands of the recompute and of dW
        if ((rc = launch_recompute(d, Wk, direct && hv, Xk, p.Kc, Tcp, small, p.tok, p.dZ, p.n_act, t0, s))) return rc;
        if (d_hidden && (rc = launch_dhidden(d, p.dZ, Tcp, Tcp, direct ? nullptr : p.WT, p.V_pad, d_hidden, d_hidden_dtype, p.n_act, t0,
                                             p.act_idx + t0, nullptr, p.part_tiles, s)))
            return rc;
        // contraction over the chunk's tokens, the row index of both dZ and the gathered hidden rows
        if (d_W && (rc = launch_dW(d, p.dZ, Xrows, Tcp, edge, dW_sum, dW_sum_dtype, (c > 0 || accumulate_dW) ? 1 : 0, p.n_act, t0,
                                   p.part_tiles, s)))
            return rc;
    }
    if (need_acc) f32_to_bf16_kernel<<<grid1(V * H / 8), 256, 0, s>>>(p.dW_acc, static_cast<bf16_t *>(d_W), V * H);
    return launch_status();
}

// ----------------------------------------------------------------------------
// forward and backward in one call
// ----------------------------------------------------------------------------
// With the gradient of the total w.r.t. the loss known up front, nothing has to be formed
// twice: the batch is walked in pieces of Tz tokens; the forward sweep of a piece also stores
// its logits (fp16 offsets, 2 * V bytes per token), the piece's log-probs give the gradient
// factors, one pass turns the stored logits of the piece's active tokens into bf16 logit
// gradients, and the two contractions follow: three products of size T x V x H instead of four.
// By default a piece's stored logits stay within kDzBudgetBytes, and so do its gradients.
// Without a loss mask the pass over the stored logits is left out as well: the sweep stores
// bf16 scaled probabilities that the contractions read as they are (probs_reference).
//
// A batch with a mask stores its logits and turns them into gradients in a pass over them: 2 V bytes written, read and
// written again per token.  Where a logit is few steps of the contraction, forming it again for the active tokens is
// cheaper: 11238 tokens (a fifth masked) at V = 151936 with H = 192 3936 -> 3366 us, 384 5728 -> 5488, but 512 6210 -> 6261
// and 1024 10096 -> 11151; short batches gain more (300 at H = 256 247 -> 192 us) and small vocabularies nothing
// (8000 at 256 x 3000 120.1 and 119.5).  fp32 heads are three times the steps and gain nothing down to H = 64 (189 -> 201).
constexpr int64_t kAgainSteps = 6;
static bool form_again(const spo_pg_desc *d) { return d->mask && d->dtype == SPO_BF16 && ceil_div(d->H, kBK) <= kAgainSteps; }

struct FbPlan {
    bool small;
    int64_t Tz, T_pad, V_pad, V_blk, Kc, nVt, nblk_tok, room;  // room: entries of part_max, part_sum
    double *count;
    float *g, *z_target, *part_max, *part_sum, *offs, *dW_acc, *part_tiles, *cscale;
    bool dense;  // no loss mask: the sweep stores what the contractions read; offs: the references of all tokens
    FwdPartial *partials;
    uint32_t *done;
    int32_t *act_idx, *n_act;
    float4 *tok;
    uint16_t *Z;  // (and offs: none where the logits of a masked batch are formed again)
    bf16_t *dZ, *WT, *Xc, *Xs, *Ws;
    void *Wvh;
    size_t bytes;
};

static FbPlan plan_fb(const spo_pg_desc *d, int64_t chunk_tokens, void *ws, bool need_dw_acc, bool want_dx, bool roomy) {
    FbPlan p;
    p.T_pad = round_up(std::max<int64_t>(d->T, 1), TL::BN);
    p.V_pad = round_up(d->V, kBK);
    p.V_blk = round_up(d->V, TL::BM);
    p.nVt = p.V_blk / TL::BM;
    p.Kc = d->dtype == SPO_FP32 ? kSplitTerms * d->H : d->H;
    // tokens per piece: a multiple of 4096 (16 splits x 16 token tiles = one round of workgroups
    // of the sweep on 256 compute units) that keeps the stored logits within the budget, and the
    // logit gradients likewise
    int64_t tz = chunk_tokens > 0 ? round_up(chunk_tokens, TL::BN) : kDzBudgetBytes / (2 * p.V_blk) / 4096 * 4096;
    if (tz < TL::BN) tz = TL::BN;
    p.Tz = std::min({tz, p.T_pad, kMostChunkTokens});
    p.small = roomy && small_sweep(std::min(p.Tz, d->T), d->V, p.Kc);
    p.room = sweep_splits(p.Tz / TL::BN, p.nVt, kSlots<TL>) * p.Tz;
    if (roomy) p.room = std::max(p.room, sweep_room(p.Tz, d->V, true));
    p.nblk_tok = p.T_pad / kTokThreads;
    static_assert(TL::BN % kTokThreads == 0, "pieces start at a block of the per-token kernels");
    Arena a(ws);
    p.count = a.take<double>(1);
    p.g = a.take<float>(p.T_pad);
    p.z_target = a.take<float>(p.T_pad);
    p.partials = a.take<FwdPartial>(p.nblk_tok);
    p.done = a.take<uint32_t>(1);
    p.part_max = a.take<float>(static_cast<size_t>(p.room));
    p.part_sum = a.take<float>(static_cast<size_t>(p.room));
    p.dense = d->mask == nullptr;
    const bool stored = !form_again(d);
    p.offs = p.dense ? a.take<float>(p.T_pad) : stored ? a.take<float>(static_cast<size_t>(p.V_blk / (roomy ? TS::WM : TL::WM)) * p.Tz) : nullptr;
    p.cscale = p.dense ? a.take<float>(p.Tz) : nullptr;
    p.act_idx = a.take<int32_t>(p.Tz);
    p.n_act = a.take<int32_t>(1);
    p.tok = a.take<float4>(p.Tz);
    p.Xc = a.take<bf16_t>(static_cast<size_t>(p.Tz) * d->H);
    p.WT = want_dx ? a.take<bf16_t>(static_cast<size_t>(d->H) * p.V_blk) : nullptr;
    p.Z = stored ? a.take<uint16_t>(static_cast<size_t>(p.Tz) * p.V_blk) : nullptr;
    p.dZ = p.dense ? nullptr : a.take<bf16_t>(static_cast<size_t>(p.Tz) * p.V_blk);
    p.Xs = p.Ws = nullptr;
    p.dW_acc = nullptr;
    if (d->dtype == SPO_FP32) {
        p.Xs = a.take<bf16_t>(static_cast<size_t>(p.Tz) * p.Kc);
        p.Ws = a.take<bf16_t>(static_cast<size_t>(d->V) * p.Kc);
    }
    p.Wvh = take_head_copy(a, d);
    if (need_dw_acc && d->T > p.Tz) p.dW_acc = a.take<float>(static_cast<size_t>(d->V) * d->H);
    p.part_tiles = a.take<float>(static_cast<size_t>(kTailTiles) * TL::BM * TL::BN);
    p.bytes = a.used;
    return p;
}

int fused_fwd_bwd_workspace(const spo_pg_desc *d, int64_t chunk_tokens, size_t *bytes) {
    const FbPlan p = plan_fb(d, chunk_tokens, nullptr, true, true, true);  // sized for the larger case
    *bytes = p.bytes;
    if (d->mask) {  // enough for a batch without one as well: a program that masks some of its batches keeps one workspace
        spo_pg_desc all = *d;
        all.mask = nullptr;
        *bytes = std::max(*bytes, plan_fb(&all, chunk_tokens, nullptr, true, true, true).bytes);
    }
    *bytes += room_for_shorter_chunks(d, p.Tz);
    return SPO_OK;
}

int fused_fwd_bwd(const spo_pg_desc *d, float grad_loss, float *loss, float *logp, float *lse, float *stats,
                  void *d_hidden, int d_hidden_dtype, void *d_W, int d_W_dtype, int accumulate_dW,
                  int64_t chunk_tokens, void *ws, size_t ws_bytes, hipStream_t s) {
    int rc = check_fused(d);
    if (rc) return rc;
    if (accumulate_dW && d_W && d_W_dtype != SPO_FP32) return SPO_EINVAL;
    FbPlan p = plan_fb(d, chunk_tokens, ws, d_W && d_W_dtype == SPO_BF16, d_hidden != nullptr, true);
    if (ws_bytes < p.bytes) p = plan_fb(d, chunk_tokens, ws, d_W && d_W_dtype == SPO_BF16, d_hidden != nullptr, false);
    const bool need_acc = p.dW_acc != nullptr;  // a bf16 d_W of several pieces (see fused_bwd)
    if (ws_bytes < p.bytes) return SPO_EWORKSPACE;
    const int64_t H = d->H, V = d->V, T = d->T;
    void *dW_sum = need_acc ? p.dW_acc : d_W;
    const int dW_sum_dtype = need_acc ? SPO_FP32 : d_W_dtype;
    if (T == 0) {
        if (d_W && !accumulate_dW) {
            const int64_t words = d_W_dtype == SPO_FP32 ? V * H : V * H / 2;
            fill_zero_kernel<<<grid1(words), 256, 0, s>>>(static_cast<uint32_t *>(d_W), words);
        }
        token_loss_kernel<<<1, kTokThreads, 0, s>>>(nullptr, nullptr, 0, 1, 0, nullptr, token_inputs(d, 0, 0), logp, lse,
                                                    p.partials, TokenGrad{}, 1, 1, p.done, loss, stats);
        return launch_status();
    }
    // the head as the kernels read it: one row per vocabulary entry for the logits, one row per
    // hidden unit (blocked over the vocabulary) for dHidden; the first piece's rows; the target logits
    const bool direct = direct_head(d), hv = d->w_layout == SPO_W_HV;
    PrepJobs jobs = prep_head_jobs(d, direct ? nullptr : p.Wvh, p.Ws, d_hidden && !direct ? p.WT : nullptr);
    prep_rows(jobs, d, d->hidden, std::min(p.Tz, T), p.Xs);
    jobs.mask = d->mask;
    jobs.count = p.count;
    launch_prep_with_targets(d, jobs, p.z_target, p.dense ? p.offs : nullptr, p.T_pad, p.done, s);
    const void *Wk = d->dtype == SPO_FP32 ? p.Ws : direct || !p.Wvh ? d->W : p.Wvh;
    const bf16_t *WT = direct ? nullptr : p.WT;
    const int64_t edge = tile_edge(p.small);
    const int64_t T_end = (T - 1) / p.Tz * p.Tz + round_up((T - 1) % p.Tz + 1, edge);  // rows of all pieces
    const size_t x_elt = d->dtype == SPO_FP32 ? 4 : 2, dx_elt = d_hidden_dtype == SPO_FP32 ? 4 : 2;
    for (int64_t t0 = 0, c = 0; t0 < T; t0 += p.Tz, ++c) {
        const int64_t Tv = std::min(p.Tz, T - t0), Tzp = round_up(Tv, edge);
        const char *Xpiece = static_cast<const char *>(d->hidden) + t0 * H * x_elt;
        const char *Xk = Xpiece;
        if (d->dtype == SPO_FP32) {
            if (c > 0) {
                jobs = prep_head_jobs(d, nullptr, nullptr, nullptr);
                prep_rows(jobs, d, Xpiece, Tv, p.Xs);
                launch_prep(d, jobs, s);
            }
            Xk = reinterpret_cast<const char *>(p.Xs);
        }
        // a piece's own choice of splits (the last may be shorter), within the room for partial results
        const int64_t nTt = Tzp / edge, nVt = ceil_div(V, edge);
        const SweepMap map(nTt, nVt, sweep_splits(nTt, nVt, tile_slots(p.small),
                                                  static_cast<uint32_t>(std::min<int64_t>(p.room / Tzp, kNoSplitCap))));
        const Sweep w{Wk, V, p.Kc, direct && hv, Xk, Tv, p.part_max, p.part_sum, p.Z, Tzp * kBlockK, p.dense ? p.offs + t0 : p.offs};
        const bool back = d_hidden || d_W, again = form_again(d);
        if ((rc = p.dense  ? launch_sweep<kEmitProbs>(w, p.small, map, s)
                  : again ? launch_sweep<kEmitNone>(w, p.small, map, s)
                          : launch_sweep<kEmitLogits>(w, p.small, map, s)))
            return rc;
        TokenGrad gr{};
        if (back) gr = TokenGrad{p.g + t0, Tzp, p.count, grad_loss, nullptr, nullptr, 0, V, d->target + t0};
        if (back && p.dense) {
            gr.c = p.cscale;
            gr.Q = p.Z;
            gr.q_blk = Tzp * kBlockK;
        }
        const int64_t n_blocks = ceil_div(back ? Tzp : Tv, kTokThreads);
        const TokenShape tok = token_shape(static_cast<int>(map.ns), n_blocks);
        token_loss_kernel<<<tok.blocks, tok.threads, 0, s>>>(
            p.part_max, p.part_sum, map.ns, tok.ways, Tzp, p.z_target + t0, token_inputs(d, t0, Tv), logp + t0, lse + t0,
            p.partials, gr, n_blocks, back ? T_end / kTokThreads : ceil_div(T, kTokThreads), p.done, loss, stats);
        if (!back) continue;
        if (p.dense) {
            // the contractions run on what the sweep stored: every row of the piece, scaled by c_t
            const bf16_t *Q = p.Z;
            if (d_hidden && (rc = launch_dhidden(d, Q, Tv, Tzp, WT, p.V_pad, static_cast<char *>(d_hidden) + t0 * H * dx_elt,
                                                 d_hidden_dtype, nullptr, 0, nullptr, p.cscale, p.part_tiles, s)))
                return rc;
            if (d_W) {
                bf16_t *Xc = p.Xc;  // c_t x_t, the rows past the piece zero
                if (d->dtype == SPO_FP32)
                    scale_rows_kernel<float><<<static_cast<unsigned>(Tzp), 256, 0, s>>>(
                        reinterpret_cast<const float *>(Xpiece), p.cscale, Tv, H, Xc);
                else
                    scale_rows_kernel<bf16_t><<<static_cast<unsigned>(Tzp), 256, 0, s>>>(
                        reinterpret_cast<const bf16_t *>(Xpiece), p.cscale, Tv, H, Xc);
                if ((rc = launch_dW(d, Q, Xc, Tzp, edge, dW_sum, dW_sum_dtype, (c > 0 || accumulate_dW) ? 1 : 0, nullptr, 0,
                                    p.part_tiles, s)))
                    return rc;
            }
            continue;
        }
        compact_active_kernel<<<1, 1024, 0, s>>>(p.g + t0, Tv, p.act_idx, p.n_act);
        launch_gather(d, Xpiece, p.act_idx, p.n_act, 0, Tzp, d->target + t0, lse + t0, p.g + t0,
                      d->dtype == SPO_BF16 || d_W ? p.Xc : nullptr, nullptr, p.tok,
                      d_hidden ? static_cast<char *>(d_hidden) + t0 * H * dx_elt : nullptr, d_hidden_dtype, Tv, s);
        const bf16_t *Xrows = p.Xc;
        if (again) {
            if ((rc = launch_recompute(d, Wk, direct && hv, Xrows, p.Kc, Tzp, p.small, p.tok, p.dZ, p.n_act, 0, s))) return rc;
        } else {
            constexpr int per_wg = 8;
            const int64_t n_blk = p.V_blk / kBlockK;
            ScopedKernelTimer timer(kTimeLogitsToDz, s);
            dz_from_logits_kernel<<<dim3(static_cast<unsigned>(Tzp / 32), grid1(n_blk, per_wg)), 256, 0, s>>>(
                p.Z, Tzp * kBlockK, p.offs, Tzp, p.act_idx, p.n_act, Tzp, p.tok, p.dZ,
                Tzp * kBlockK, n_blk, per_wg, (p.small ? TS::WM : TL::WM) / kBlockK, static_cast<int>(edge));
        }
        if (d_hidden && (rc = launch_dhidden(d, p.dZ, Tzp, Tzp, WT, p.V_pad, static_cast<char *>(d_hidden) + t0 * H * dx_elt,
                                             d_hidden_dtype, p.n_act, 0, p.act_idx, nullptr, p.part_tiles, s)))
            return rc;
        if (d_W && (rc = launch_dW(d, p.dZ, Xrows, Tzp, edge, dW_sum, dW_sum_dtype, (c > 0 || accumulate_dW) ? 1 : 0, p.n_act, 0,
                                   p.part_tiles, s)))
            return rc;
    }
    if (need_acc) f32_to_bf16_kernel<<<grid1(V * H / 8), 256, 0, s>>>(p.dW_acc, static_cast<bf16_t *>(d_W), V * H);
    return launch_status();
}

}  // namespace spo
