// Prioritized prompt sampling: weights -> exact integer CDF -> Philox draws.
// Method, "Prioritized Prompt Sampling" (sampling-weight equation and the batch
// draw of the training loop).  The O(N) part (weights + scan) streams the tracker
// once per phase; the draw itself is B searches of the CDF.  Tables of one scan block are
// handled by a single launch that keeps the CDF in LDS (a step of 16 prompts: 7 launches -> 3,
// 52 us -> 35 us, what is left being the host's).
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
constexpr int kInlineBlocks = kScanThreads;                 // block sums that every block adds up by itself
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

// Phase 1: per-block sum of the weight codes.
__global__ void __launch_bounds__(kScanThreads)
weight_block_sums_kernel(const float *__restrict__ alpha, const float *__restrict__ beta, int64_t N,
                         double eps, uint64_t *__restrict__ block_sums) {
    __shared__ uint64_t scratch[kScanThreads / kWave];
    uint64_t x[kScanRows];
    weight_rows(alpha, beta, N, eps, static_cast<int64_t>(blockIdx.x) * kScanItems, x);
    uint64_t s = 0;
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) s += x[r];
    s = block_sum(s, scratch);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = s;
}

// Phase 2, only where there are more than kInlineBlocks blocks: exclusive scan of the block sums
// (one workgroup, carried in chunks).
__global__ void __launch_bounds__(kScanThreads)
scan_block_sums_kernel(uint64_t *__restrict__ block_sums, int64_t nblocks) {
    __shared__ uint64_t lds[kWave + 1];
    uint64_t carry = 0;
    for (int64_t base = 0; base < nblocks; base += kScanItems) {
        uint64_t v[kScanRows], x[kScanRows], tot;
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int64_t i = base + r * kScanThreads + threadIdx.x;
            v[r] = x[r] = i < nblocks ? block_sums[i] : 0;
        }
        block_scan_rows(x, lds, tot);
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int64_t i = base + r * kScanThreads + threadIdx.x;
            if (i < nblocks) block_sums[i] = carry + x[r] - v[r];
        }
        carry += tot;
    }
}

// Phase 3: inclusive CDF of the codes, its last value as *total, and (owner != NULL) the claims
// cleared, with info.  summed: block_sums holds what scan_block_sums_kernel made of it; otherwise
// (at most kInlineBlocks blocks) every block adds up the sums before its own.
__global__ void __launch_bounds__(kScanThreads)
weight_cdf_kernel(const float *__restrict__ alpha, const float *__restrict__ beta, int64_t N, double eps,
                  const uint64_t *__restrict__ block_sums, int summed, uint64_t *__restrict__ cdf,
                  uint64_t *__restrict__ total, int32_t *__restrict__ owner, int32_t *__restrict__ info) {
    __shared__ uint64_t lds[kWave + 1];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanItems;
    uint64_t before;
    if (summed) before = block_sums[blockIdx.x];
    else before = block_sum(threadIdx.x < blockIdx.x ? block_sums[threadIdx.x] : uint64_t(0), lds);
    uint64_t x[kScanRows], tot;
    weight_rows(alpha, beta, N, eps, base, x);
    block_scan_rows(x, lds, tot);
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        const int64_t i = base + r * kScanThreads + threadIdx.x;
        if (i < N) {
            cdf[i] = before + x[r];
            if (owner) owner[i] = kNoOwner;
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        *total = before + tot;
        if (owner && info) info[0] = info[1] = 0;
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

// index of draw (slot, attempt): first i with cdf[i] > floor(bits * total / 2^64).  Each round asks 15
// entries at once, a sixteenth of the range apart: five dependent loads for 2^20 prompts instead of
// twenty.
__device__ __forceinline__ int32_t draw_index(const uint64_t *__restrict__ cdf, int64_t N, uint64_t total,
                                              uint64_t seed, uint64_t iteration, uint32_t slot, uint32_t attempt) {
    const uint64_t t = __umul64hi(philox_bits(seed, iteration, slot, attempt), total);
    uint32_t lo = 0, hi = static_cast<uint32_t>(N);  // N < 2^31; cdf[i] <= t below lo, > t from hi on
    while (lo < hi) {
        const uint32_t step = (hi - lo + 15) / 16;
        uint32_t c = 0;
#pragma unroll
        for (uint32_t j = 1; j < 16; ++j) {
            const uint32_t p = lo + j * step - 1;
            const uint64_t v = cdf[p < hi ? p : hi - 1];  // always a load, none of them behind a branch
            c += static_cast<uint32_t>(v <= t) & static_cast<uint32_t>(p < hi);
        }
        lo += c * step;
        const uint32_t end = lo + step - 1;  // the first probe above t, if one was
        hi = c < 15 && end < hi ? end : hi;
    }
    return static_cast<int32_t>(lo);
}

__global__ void __launch_bounds__(256)
draw_with_replacement_kernel(const uint64_t *__restrict__ cdf, int64_t N, const uint64_t *__restrict__ total,
                             uint64_t seed, uint64_t iteration, int B, int32_t *__restrict__ idx_out,
                             int32_t *__restrict__ info) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t tot = *total;  // zero: every weight is zero, nothing can be drawn
    if (k < B) idx_out[k] = tot ? draw_index(cdf, N, tot, seed, iteration, k, 0) : -1;
    if (info && k == 0) { info[0] = tot ? 0 : 1; info[1] = 0; }
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

// The claims over many workgroups; the one place they meet is the atomics on owner[].
__global__ void __launch_bounds__(kWave)
draw_claim_kernel(const uint64_t *__restrict__ cdf, int64_t N, const uint64_t *__restrict__ total_p, uint64_t seed,
                  uint64_t iteration, int B, uint32_t max_attempts, int32_t *__restrict__ idx_out,
                  int32_t *__restrict__ info, int32_t *__restrict__ owner) {
    const uint32_t k = blockIdx.x * kWave + threadIdx.x;
    const uint64_t total = *total_p;
    if (k >= static_cast<uint32_t>(B)) return;
    if (total == 0) {  // every weight is zero: nothing can be drawn
        idx_out[k] = -1;
        if (info && k == 0) info[0] = 1;
        return;
    }
    const uint32_t most = SlotClaims::settle(
        k, max_attempts, [&](uint32_t s, uint32_t n) { return draw_index(cdf, N, total, seed, iteration, s, n); },
        [&](int32_t c, int32_t v) { return atomicMin(&owner[c], v); },
        [&](uint32_t s) {
            idx_out[s] = -1;
            if (info) atomicOr(&info[0], 1);
        });
    if (info && most) atomicMax(&info[1], static_cast<int32_t>(most));
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
        const uint32_t m = SlotClaims::settle(k, max_attempts, draw, [&](int32_t c, int32_t v) { return atomicMin(&owner[c], v); },
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
    uint64_t *cdf, *block_sums, *total;
    int32_t *owner;
    size_t bytes;
};

static SamplerWorkspace sampler_layout(void *ws, int64_t N) {
    Arena a(ws);
    SamplerWorkspace w;
    w.cdf = a.take<uint64_t>(static_cast<size_t>(N));
    w.block_sums = a.take<uint64_t>(static_cast<size_t>(ceil_div(N, kScanItems)));
    w.total = a.take<uint64_t>(1);
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
    // The bound on a hopeless draw: 0.3 s for 4096 slots on 100 prompts of a large table (4 to 8 us per attempt), up to
    // 12 s where 16384 slots want the same prompt (190 us: their claims meet at one address).
    if (max_attempts == 0) max_attempts = 1u << 16;
    if (N <= kScanItems && B <= kScanItems) {
        unsigned threads = kWave;
        while (threads < kScanThreads && static_cast<int64_t>(threads) * kScanRows < std::max<int64_t>(N, B)) threads *= 2;
        sample_small_kernel<<<1, threads, 0, s>>>(alpha, beta, static_cast<int>(N), eps_explore, seed, iteration, replace, B,
                                                  max_attempts, idx_out, info);
        return launch_status();
    }
    const int64_t nblocks = ceil_div(N, kScanItems);
    const bool summed = nblocks > kInlineBlocks;
    if (nblocks > 1)
        weight_block_sums_kernel<<<static_cast<unsigned>(nblocks), kScanThreads, 0, s>>>(alpha, beta, N, eps_explore, w.block_sums);
    if (summed) scan_block_sums_kernel<<<1, kScanThreads, 0, s>>>(w.block_sums, nblocks);
    weight_cdf_kernel<<<static_cast<unsigned>(nblocks), kScanThreads, 0, s>>>(
        alpha, beta, N, eps_explore, w.block_sums, summed, w.cdf, w.total, replace ? nullptr : w.owner, info);
    if (replace) {
        draw_with_replacement_kernel<<<(B + 255) / 256, 256, 0, s>>>(w.cdf, N, w.total, seed, iteration, B, idx_out, info);
    } else {
        draw_claim_kernel<<<static_cast<unsigned>(ceil_div(B, kWave)), kWave, 0, s>>>(w.cdf, N, w.total, seed, iteration, B,
                                                                                      max_attempts, idx_out, info, w.owner);
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
