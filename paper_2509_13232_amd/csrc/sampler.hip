// Prioritized prompt sampling: weights -> exact integer CDFs -> Philox draws.
// Method, "Prioritized Prompt Sampling" (sampling-weight equation and the batch
// draw of the training loop).  The O(N) part (weights + scans of blocks) streams the tracker
// once; the draw itself is B searches, of the blocks' sums and of a block's CDF.  Tables of one scan block are
// handled by a single launch that keeps the CDF in LDS (a step of 16 prompts: 7 launches -> 3,
// 52 us -> 35 us, what was left being the host's: 16 us with the plain calls in an extension).
//
// Everything that decides an index is integer arithmetic or a single correctly
// rounded IEEE fp64 operation (add, divide, subtract, multiply, sqrt: no fused
// multiply-add can form because no product feeds an addition), so the indices do
// not depend on the machine, the launch shape or the order of summation.
#include <algorithm>
#include <mutex>

#include "common.hpp"
#include "sampler_claims.hpp"

namespace spo {

constexpr int kScanThreads = 1024;
constexpr int kScanRows = 4;                                // rows of kScanThreads items per block
constexpr int kScanItems = kScanThreads * kScanRows;        // 4096 items per block
constexpr int kInlineBlocks = 1024;                         // block sums that every workgroup of a draw adds up by itself
constexpr int kMaxSlotsNoReplace = 16384;

__device__ __forceinline__ uint64_t weight_code(float alpha, float beta, double eps) {
    const double a = static_cast<double>(alpha), b = static_cast<double>(beta);
    const double s = a + b;
    double w = eps;
    if (s > 0.0) {
        const double v = a / s;
        const double q = 1.0 - v;
        const double p = v * q;
        w = sqrt(p) + eps;
    }
    return static_cast<uint64_t>(floor(w * 4294967296.0));
}

// Inclusive scan over kScanRows rows of blockDim.x values (row r before row r + 1), by up to 16
// wavefronts; lds holds 65 values.  The rows are scanned side by side and meet in one exchange.
__device__ __forceinline__ void block_scan_rows(uint64_t (&x)[kScanRows], uint64_t *lds, uint64_t &total) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, nwave = blockDim.x / kWave;
    static_assert(kScanRows * kScanThreads / kWave <= kWave, "one wavefront scans the wavefronts' totals");
    auto wave_scan = [&](uint64_t v) {
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint64_t y = __shfl_up(v, o, kWave);
            if (lane >= o) v += y;
        }
        return v;
    };
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) x[r] = wave_scan(x[r]);
    __syncthreads();  // lds may still be read
    if (lane == kWave - 1)
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) lds[r * nwave + wave] = x[r];
    __syncthreads();
    if (wave == 0) {
        const uint64_t v = lane < kScanRows * nwave ? lds[lane] : 0, inc = wave_scan(v);
        lds[lane] = inc - v;
        if (lane == kWave - 1) lds[kWave] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) x[r] += lds[r * nwave + wave];
    total = lds[kWave];
}

// Weight codes of kScanRows rows of blockDim.x prompts from `base` on (0 past the last prompt).
__device__ __forceinline__ void weight_rows(const float *__restrict__ alpha, const float *__restrict__ beta, int64_t N,
                                            double eps, int64_t base, uint64_t (&x)[kScanRows]) {
    float a[kScanRows], b[kScanRows];
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        const int64_t i = base + r * blockDim.x + threadIdx.x;
        a[r] = i < N ? alpha[i] : 0.0f;
        b[r] = i < N ? beta[i] : 0.0f;
    }
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        const int64_t i = base + r * blockDim.x + threadIdx.x;
        x[r] = i < N ? weight_code(a[r], b[r], eps) : 0;
    }
}

// Phase 1: the inclusive CDF of the codes inside every block of kScanItems prompts and the blocks' sums, the claims
// cleared (owner != NULL) with info.  One pass over the tracker; what lies before a block is added up by the draws (the
// sums first and the CDF over the whole table in a second pass took 21 us at 2^20 prompts).  A thread takes four
// prompts in a row, so that one scan over the threads is left (rows of 1024 prompts, four scans side by side: 13.0 us, this
// 11.4; 7.5 and 5.0 for five blocks).
template <typename V4>
__device__ __forceinline__ V4 load4(const void *p) {
    typedef V4 U __attribute__((aligned(4)));
    return *static_cast<const U *>(p);
}
__global__ void __launch_bounds__(kScanThreads)
weight_scan_kernel(const float *__restrict__ alpha, const float *__restrict__ beta, int64_t N, double eps,
                   uint64_t *__restrict__ cdf, uint64_t *__restrict__ block_sums, int32_t *__restrict__ owner,
                   int32_t *__restrict__ info) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    static_assert(kScanRows == 4, "four prompts per thread");
    constexpr int NW = kScanThreads / kWave;
    __shared__ uint64_t wave_sums[NW];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kScanItems + threadIdx.x * 4;
    f4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = a;
    if (i + 3 < N) {
        a = load4<f4>(alpha + i);
        b = load4<f4>(beta + i);
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
            if (i + r < N) {
                a[r] = alpha[i + r];
                b[r] = beta[i + r];
            }
    }
    uint64_t x[4], run = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = run += i + r < N ? weight_code(a[r], b[r], eps) : 0;
    uint64_t upto = run;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint64_t y = __shfl_up(upto, o, kWave);
        if (lane >= o) upto += y;
    }
    if (lane == kWave - 1) wave_sums[wave] = upto;
    __syncthreads();
    uint64_t before = upto - run, tot = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint64_t v = wave_sums[w];
        before += w < wave ? v : 0;
        tot += v;
    }
    typedef uint64_t u2 __attribute__((ext_vector_type(2)));
    typedef int32_t i4 __attribute__((ext_vector_type(4)));
    if (i + 3 < N) {  // (the tables begin on 256-byte boundaries)
        *reinterpret_cast<u2 *>(cdf + i) = u2{before + x[0], before + x[1]};
        *reinterpret_cast<u2 *>(cdf + i + 2) = u2{before + x[2], before + x[3]};
        if (owner) *reinterpret_cast<i4 *>(owner + i) = i4{kNoOwner, kNoOwner, kNoOwner, kNoOwner};
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
            if (i + r < N) {
                cdf[i + r] = before + x[r];
                if (owner) owner[i + r] = kNoOwner;
            }
    }
    if (threadIdx.x == 0) {
        block_sums[blockIdx.x] = tot;
        if (blockIdx.x == 0 && owner && info) info[0] = info[1] = 0;
    }
}

// Phase 2, only where there are more than kInlineBlocks blocks: inclusive scan of the block sums
// (one workgroup, carried in chunks).
__global__ void __launch_bounds__(kScanThreads)
scan_block_sums_kernel(uint64_t *__restrict__ block_sums, int64_t nblocks) {
    __shared__ uint64_t lds[kWave + 1];
    uint64_t carry = 0;
    for (int64_t base = 0; base < nblocks; base += kScanItems) {
        uint64_t x[kScanRows], tot;
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int64_t i = base + r * kScanThreads + threadIdx.x;
            x[r] = i < nblocks ? block_sums[i] : 0;
        }
        block_scan_rows(x, lds, tot);
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int64_t i = base + r * kScanThreads + threadIdx.x;
            if (i < nblocks) block_sums[i] = carry + x[r];
        }
        carry += tot;
    }
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds, each two 32x32->64 products
// whose halves are crossed with the other counter words and the round key; the
// key grows by the two Weyl constants after every round.
__device__ __forceinline__ uint64_t philox_bits(uint64_t seed, uint64_t iteration, uint32_t slot, uint32_t attempt) {
    uint32_t c0 = slot, c1 = attempt, c2 = static_cast<uint32_t>(iteration), c3 = static_cast<uint32_t>(iteration >> 32);
    uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return static_cast<uint64_t>(c0) | (static_cast<uint64_t>(c1) << 32);
}

// First index in [lo, hi) whose entry of v[] is above t (hi: none; entries do not fall).  Each round asks 15 entries at
// once, a sixteenth of the range apart: three dependent loads for a block of 4096.
__device__ __forceinline__ uint32_t first_above(const uint64_t *__restrict__ v, uint32_t lo, uint32_t hi, uint64_t t) {
    while (lo < hi) {
        const uint32_t step = (hi - lo + 15) / 16;
        uint32_t c = 0;
#pragma unroll
        for (uint32_t j = 1; j < 16; ++j) {
            const uint32_t p = lo + j * step - 1;
            const uint64_t x = v[p < hi ? p : hi - 1];  // always a load, none of them behind a branch
            c += static_cast<uint32_t>(x <= t) & static_cast<uint32_t>(p < hi);
        }
        lo += c * step;
        const uint32_t end = lo + step - 1;  // the first probe above t, if one was
        hi = c < 15 && end < hi ? end : hi;
    }
    return lo;
}

// The tables of a draw: the CDF inside every block, and the inclusive sums over the blocks, in LDS (`sums`, kInlineBlocks
// entries) or, where there are more, in memory as scan_block_sums_kernel left them.
struct DrawTables {
    const uint64_t *cdf, *sums;
    uint32_t N, nblocks;
    uint64_t total;

    // All threads of the workgroup (whole wavefronts) call this; `sums` holds kInlineBlocks values.
    __device__ __forceinline__ DrawTables(const uint64_t *cdf_, const uint64_t *block_sums, int64_t N_, int64_t nb, uint64_t *lds)
        : cdf(cdf_), sums(block_sums), N(static_cast<uint32_t>(N_)), nblocks(static_cast<uint32_t>(nb)) {
        if (nblocks <= kInlineBlocks) {
            if (threadIdx.x < kWave) {  // one wavefront scans them, a run of consecutive ones per lane
                constexpr int RUN = kInlineBlocks / kWave;
                const uint32_t per = (nblocks + kWave - 1) / kWave, first = threadIdx.x * per;
                uint64_t x[RUN], run = 0;
#pragma unroll
                for (uint32_t j = 0; j < RUN; ++j) x[j] = j < per && first + j < nblocks ? block_sums[first + j] : 0;
#pragma unroll
                for (uint32_t j = 0; j < RUN; ++j) run += x[j];
                uint64_t before = run;
#pragma unroll
                for (int o = 1; o < kWave; o <<= 1) {
                    const uint64_t y = __shfl_up(before, o, kWave);
                    if (static_cast<int>(threadIdx.x) >= o) before += y;
                }
                before -= run;
#pragma unroll
                for (uint32_t j = 0; j < RUN; ++j) {
                    before += x[j];
                    if (j < per && first + j < nblocks) lds[first + j] = before;
                }
            }
            sums = lds;
            __syncthreads();
        }
        total = sums[nblocks - 1];
    }
    // index of draw (slot, attempt): first i whose entry of the CDF over the table is above floor(bits * total / 2^64)
    __device__ __forceinline__ int32_t index(uint64_t seed, uint64_t iteration, uint32_t slot, uint32_t attempt) const {
        const uint64_t t = __umul64hi(philox_bits(seed, iteration, slot, attempt), total);
        uint32_t b = 0, hi = nblocks - 1;  // t < total: the last block's sum is above t
        if (nblocks <= kInlineBlocks) {  // LDS answers fast: a plain binary search
            while (b < hi) {
                const uint32_t mid = (b + hi) >> 1;
                if (sums[mid] > t) hi = mid; else b = mid + 1;
            }
        } else {
            b = first_above(sums, 0, hi, t);
        }
        const uint64_t rest = t - (b ? sums[b - 1] : 0);
        const uint32_t lo = b * kScanItems, end = N - lo < kScanItems ? N : lo + kScanItems;
        return static_cast<int32_t>(first_above(cdf, lo, end, rest));
    }
    // The same by a whole wavefront for one draw (slot and attempt the same in every lane): 64 entries at once, two
    // dependent loads of a block, one each per lane.
    __device__ __forceinline__ int32_t index_wave(uint64_t seed, uint64_t iteration, uint32_t slot, uint32_t attempt) const {
        const uint32_t lane = threadIdx.x & (kWave - 1);
        const uint64_t t = __umul64hi(philox_bits(seed, iteration, slot, attempt), total);
        auto first = [&](const uint64_t *v, uint32_t lo, uint32_t hi, uint32_t step, uint64_t x) {  // the first of 64 probes above x
            const uint32_t p = lo + (lane + 1) * step - 1;
            return static_cast<uint32_t>(__builtin_ctzll(__ballot(v[p < hi ? p : hi - 1] > x)));  // (the last entry is)
        };
        uint32_t b;
        if (nblocks <= kInlineBlocks) {
            constexpr uint32_t RUN = kInlineBlocks / kWave;
            b = RUN * first(sums, 0, nblocks, RUN, t);
            b += first(sums, b, nblocks - b < RUN ? nblocks : b + RUN, 1, t);
        } else {
            b = first_above(sums, 0, nblocks - 1, t);
        }
        const uint64_t rest = t - (b ? sums[b - 1] : 0);
        uint32_t lo = b * kScanItems;
        const uint32_t end = N - lo < kScanItems ? N : lo + kScanItems;
        lo += kWave * first(cdf, lo, end, kWave, rest);
        return static_cast<int32_t>(lo + first(cdf, lo, end, 1, rest));
    }
};
static_assert(kScanItems == kWave * kWave, "two rounds of 64 probes find an entry of a block");

__global__ void __launch_bounds__(256)
draw_with_replacement_kernel(const uint64_t *__restrict__ cdf, int64_t N, const uint64_t *__restrict__ block_sums, int64_t nblocks,
                             uint64_t seed, uint64_t iteration, int B, int32_t *__restrict__ idx_out,
                             int32_t *__restrict__ info) {
    __shared__ uint64_t lds[kInlineBlocks];
    const DrawTables tab(cdf, block_sums, N, nblocks, lds);
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    // a total of zero: every weight is zero, nothing can be drawn
    if (k < B) idx_out[k] = tab.total ? tab.index(seed, iteration, k, 0) : -1;
    if (info && k == 0) { info[0] = tab.total ? 0 : 1; info[1] = 0; }
}

// Successive sampling without replacement: slot k takes its first attempt that no slot before it has
// taken.  Found by deferred acceptance: a slot claims the candidate of its attempt with an atomic
// minimum; where a lower slot is found it goes on to its next attempt, where a higher one is found
// that one is displaced and the same thread takes it on from the attempt it was at.  A slot leaves a
// candidate only for a lower one, so the lowest slot that ever claimed a candidate holds it at the
// end, whatever the order of the claims: the result is the sequential one on every run, no slot waits
// for another, and no barrier is needed.  (One workgroup in sweeps over all slots: 121 us for 4096 of
// 2^20 prompts, this: 12 us, and 4 us for the indices.)  Attempts only grow and stop at max_attempts.
typedef Claims<17> SlotClaims;
static_assert(SlotClaims::kMaxSlots >= kMaxSlotsNoReplace, "claims fit 31 bits");

// The claims over many workgroups, a wavefront per slot; the one place they meet is the atomics on owner[].  Bound by the
// latency of an attempt, twice that where a slot is turned away: a lane per slot asks for 15 entries of a block three times
// in a row (4096 of 2^20 prompts: 10.7 us), a wavefront for 64 twice (7.6).  Where nearly all prompts are taken the atomics of
// all slots meet at the same addresses, 11 ns each, one wavefront's lanes together but wavefronts apart: late attempts look
// before they claim, past the caches (4096 slots on 100 prompts, an attempt: 4.5 us by lanes, 12.1 by wavefronts, 1.4 with
// the look; 16384 on one 186, 186 and 9).
__global__ void __launch_bounds__(256)
draw_claim_kernel(const uint64_t *__restrict__ cdf, int64_t N, const uint64_t *__restrict__ block_sums, int64_t nblocks,
                  uint64_t seed, uint64_t iteration, int B, uint32_t max_attempts, int32_t *__restrict__ idx_out,
                  int32_t *__restrict__ info, int32_t *__restrict__ owner) {
    __shared__ uint64_t lds[kInlineBlocks];
    const DrawTables tab(cdf, block_sums, N, nblocks, lds);
    const uint32_t k = __builtin_amdgcn_readfirstlane(blockIdx.x * (256 / kWave) + threadIdx.x / kWave);
    const bool lead = (threadIdx.x & (kWave - 1)) == 0;
    if (k >= static_cast<uint32_t>(B)) return;
    if (tab.total == 0) {  // every weight is zero: nothing can be drawn
        if (lead) {
            idx_out[k] = -1;
            if (info && k == 0) info[0] = 1;
        }
        return;
    }
    const uint32_t most = SlotClaims::settle(
        k, max_attempts,
        [&](uint32_t s, uint32_t n) { return static_cast<int32_t>(__builtin_amdgcn_readfirstlane(tab.index_wave(seed, iteration, s, n))); },
        [&](int32_t c) {
            return static_cast<int32_t>(__builtin_amdgcn_readfirstlane(__hip_atomic_load(&owner[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
        },
        [&](int32_t c, int32_t v) {
            int32_t was = 0;
            if (lead) was = atomicMin(&owner[c], v);
            return static_cast<int32_t>(__builtin_amdgcn_readfirstlane(was));
        },
        [&](uint32_t s) {
            if (!lead) return;
            idx_out[s] = -1;
            if (info) atomicOr(&info[0], 1);
        });
    if (lead && info && most) atomicMax(&info[1], static_cast<int32_t>(most));
}

// The other slots' indices, from the prompts they hold.
__global__ void __launch_bounds__(256)
place_slots_kernel(const int32_t *__restrict__ owner, int64_t N, int32_t *__restrict__ idx_out) {
    constexpr int PER = 4;
    int32_t o[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int64_t i = static_cast<int64_t>(blockIdx.x) * (256 * PER) + j * 256 + threadIdx.x;
        o[j] = i < N ? owner[i] : kNoOwner;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (o[j] != kNoOwner)
            idx_out[SlotClaims::slot(o[j])] = static_cast<int32_t>(static_cast<int64_t>(blockIdx.x) * (256 * PER) + j * 256 + threadIdx.x);
}

// Everything in one workgroup, for tables of at most kScanItems prompts: the CDF and the
// claims stay in LDS.  Launched with enough threads for the table (kScanRows prompts each).
__global__ void __launch_bounds__(kScanThreads)
sample_small_kernel(const float *__restrict__ alpha, const float *__restrict__ beta, int N, double eps, uint64_t seed,
                    uint64_t iteration, int replace, int B, uint32_t max_attempts, int32_t *__restrict__ idx_out,
                    int32_t *__restrict__ info) {
    __shared__ uint64_t cdf[kScanItems];
    __shared__ int32_t owner[kScanItems];
    __shared__ uint64_t lds[kWave + 1];
    __shared__ int failed, most_sh;
    const int tid = threadIdx.x, NT = blockDim.x;
    uint64_t x[kScanRows], total;
    weight_rows(alpha, beta, N, eps, 0, x);
    block_scan_rows(x, lds, total);
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        const int i = r * NT + tid;
        if (i < N) {
            cdf[i] = x[r];
            owner[i] = kNoOwner;
        }
    }
    if (tid == 0) failed = most_sh = 0;
    __syncthreads();
    if (total == 0) {  // every weight is zero: nothing can be drawn
        for (int k = tid; k < B; k += NT) idx_out[k] = -1;
        if (info && tid == 0) { info[0] = 1; info[1] = 0; }
        return;
    }
    auto draw = [&](uint32_t k, uint32_t n) {  // LDS answers fast: a plain binary search
        const uint64_t t = __umul64hi(philox_bits(seed, iteration, k, n), total);
        int lo = 0, hi = N;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cdf[mid] > t) hi = mid; else lo = mid + 1;
        }
        return static_cast<int32_t>(lo);
    };
    if (replace) {
        for (int k = tid; k < B; k += NT) idx_out[k] = draw(k, 0);
        if (info && tid == 0) info[0] = info[1] = 0;
        return;
    }
    uint32_t most = 0;
    for (int k = tid; k < B; k += NT) {
        const uint32_t m = SlotClaims::settle(
            k, max_attempts, draw, [](int32_t) { return kNoOwner; }, [&](int32_t c, int32_t v) { return atomicMin(&owner[c], v); },
            [&](uint32_t s) {
                idx_out[s] = -1;
                failed = 1;
            });
        most = m > most ? m : most;
    }
    if (most) atomicMax(&most_sh, static_cast<int>(most));
    __syncthreads();
    for (int c = tid; c < N; c += NT)
        if (owner[c] != kNoOwner) idx_out[SlotClaims::slot(owner[c])] = c;
    if (info && tid == 0) {
        info[0] = failed;
        info[1] = most_sh;
    }
}

struct SamplerWorkspace {
    uint64_t *cdf, *block_sums;
    int32_t *owner;
    size_t bytes;
};

static SamplerWorkspace sampler_layout(void *ws, int64_t N) {
    Arena a(ws);
    SamplerWorkspace w;
    w.cdf = a.take<uint64_t>(static_cast<size_t>(N));
    w.block_sums = a.take<uint64_t>(static_cast<size_t>(ceil_div(N, kScanItems)));
    a.take<uint64_t>(1);  // (a size that programs may have kept)
    w.owner = a.take<int32_t>(static_cast<size_t>(N));
    w.bytes = a.used;
    return w;
}

}  // namespace spo

using namespace spo;

extern "C" size_t spo_sample_prompts_workspace_bytes(int64_t N, int32_t B) {
    (void)B;
    if (N < 1) return 0;
    return sampler_layout(nullptr, N).bytes;
}

// Checks and launches shared by the two entry points; ws holds sampler_layout(ws, N).
static int sample_launch(const float *alpha, const float *beta, int64_t N, int32_t B, double eps_explore,
                         uint64_t seed, uint64_t iteration, int replace, uint32_t max_attempts,
                         int32_t *idx_out, int32_t *info, void *ws, hipStream_t s) {
    const SamplerWorkspace w = sampler_layout(ws, N);
    // The bound on a hopeless draw: 0.1 s for 4096 slots on 100 prompts of a large table (1.4 us per attempt), 0.6 s where
    // 16384 slots want the same prompt (9 us).
    if (max_attempts == 0) max_attempts = 1u << 16;
    if (N <= kScanItems && B <= kScanItems) {
        unsigned threads = kWave;
        while (threads < kScanThreads && static_cast<int64_t>(threads) * kScanRows < std::max<int64_t>(N, B)) threads *= 2;
        sample_small_kernel<<<1, threads, 0, s>>>(alpha, beta, static_cast<int>(N), eps_explore, seed, iteration, replace, B,
                                                  max_attempts, idx_out, info);
        return launch_status();
    }
    const int64_t nblocks = ceil_div(N, kScanItems);
    weight_scan_kernel<<<static_cast<unsigned>(nblocks), kScanThreads, 0, s>>>(alpha, beta, N, eps_explore, w.cdf, w.block_sums,
                                                                               replace ? nullptr : w.owner, info);
    if (nblocks > kInlineBlocks) scan_block_sums_kernel<<<1, kScanThreads, 0, s>>>(w.block_sums, nblocks);
    if (replace) {
        draw_with_replacement_kernel<<<(B + 255) / 256, 256, 0, s>>>(w.cdf, N, w.block_sums, nblocks, seed, iteration, B, idx_out, info);
    } else {
        draw_claim_kernel<<<static_cast<unsigned>(ceil_div(B, 256 / kWave)), 256, 0, s>>>(
            w.cdf, N, w.block_sums, nblocks, seed, iteration, B, max_attempts, idx_out, info, w.owner);
        place_slots_kernel<<<static_cast<unsigned>(ceil_div(N, 1024)), 256, 0, s>>>(w.owner, N, idx_out);
    }
    return launch_status();
}

static int sample_check(const float *alpha, const float *beta, int64_t N, int32_t B, double eps_explore,
                        int replace, const int32_t *idx_out) {
    if (!alpha || !beta || !idx_out) return SPO_ENULL;
    if (N < 1 || N >= (int64_t(1) << 31) || B < 1 || !(eps_explore >= 0.0) || !(eps_explore <= 1.0))
        return SPO_EINVAL;
    if (!replace && B > N) return SPO_EINVAL;
    if (!replace && B > kMaxSlotsNoReplace) return SPO_ERANGE;
    return SPO_OK;
}

extern "C" int spo_sample_prompts(const float *alpha, const float *beta, int64_t N, int32_t B,
                                  double eps_explore, uint64_t seed, uint64_t iteration, int replace,
                                  uint32_t max_attempts, int32_t *idx_out, int32_t *info, void *ws,
                                  size_t ws_bytes, spo_stream_t stream) {
    const int rc = sample_check(alpha, beta, N, B, eps_explore, replace, idx_out);
    if (rc) return rc;
    if (!ws) return SPO_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return SPO_EINVAL;
    if (ws_bytes < sampler_layout(nullptr, N).bytes) return SPO_EWORKSPACE;
    return sample_launch(alpha, beta, N, B, eps_explore, seed, iteration, replace, max_attempts, idx_out, info, ws,
                         as_stream(stream));
}

// ----------------------------------------------------------------------------
// The same draw for callers that cannot allocate: the CDF, the block sums and the
// owner table live in a fixed array in device memory that belongs to the library
// (one copy per GPU, held until the process ends).
// ----------------------------------------------------------------------------
namespace spo {

constexpr int64_t kStaticMaxN = SPO_SAMPLE_STATIC_MAX_N;
// what sampler_layout takes for kStaticMaxN prompts: 8 B (CDF) + 4 B (owner) per prompt,
// one 8-byte sum per 4096 prompts, the total, each block rounded up to 256 bytes
constexpr size_t kStaticBytes = static_cast<size_t>(kStaticMaxN) * 12 + (kStaticMaxN / kScanItems + 1) * 8 + 4 * 256;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

// Device address of `scratch` on the current device.  In host code the array's name is only a
// handle for hipGetSymbolAddress; every GPU has its own copy at its own address, looked up
// once per device with that device current.
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];

static int static_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SPO_EHIP;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SPO_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SPO_OK;
}

}  // namespace spo

extern "C" int spo_sample_prompts_static(const float *alpha, const float *beta, int64_t N, int32_t B,
                                         double eps_explore, uint64_t seed, uint64_t iteration, int replace,
                                         uint32_t max_attempts, int32_t *idx_out, int32_t *info,
                                         spo_stream_t stream) {
    int rc = sample_check(alpha, beta, N, B, eps_explore, replace, idx_out);
    if (rc) return rc;
    if (N > kStaticMaxN) return SPO_ERANGE;  // the fixed array holds the tables of at most this many prompts
    if (sampler_layout(nullptr, N).bytes > kStaticBytes) return SPO_ERANGE;
    void *ws = nullptr;
    if ((rc = static_scratch(&ws))) return rc;
    return sample_launch(alpha, beta, N, B, eps_explore, seed, iteration, replace, max_attempts, idx_out, info, ws,
                         as_stream(stream));
}
