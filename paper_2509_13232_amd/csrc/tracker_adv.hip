// Beta value tracker (update, initialisation) and single-stream advantages.
// Method, "A KL-Adaptive Value Tracker" and "Advantage Estimation and Policy
// Optimization".  Plain ALU work on scattered entries, a few thousand as a rule: chains of cache misses and the
// latency of launches.
#include <algorithm>

#include "common.hpp"

namespace spo {

// rho = 2^(-D/D_half) kept inside [rho_min, rho_max]; fp64 so that the fp32
// result of rho*alpha + r carries a single rounding.
__device__ __forceinline__ double discount(float kl, double d_half, double rho_min, double rho_max) {
    const double d = kl > 0.0f ? static_cast<double>(kl) : 0.0;
    double rho = exp2(-d / d_half);
    rho = rho < rho_min ? rho_min : rho;
    rho = rho > rho_max ? rho_max : rho;
    return rho;
}

__device__ __forceinline__ void observe(float &a, float &b, float r, double rho) {
    const double rd = static_cast<double>(r);
    a = static_cast<float>(rho * static_cast<double>(a) + rd);
    b = static_cast<float>(rho * static_cast<double>(b) + (1.0 - rd));
}

// Moving-average form: v <- v + (r - v)/(rho n + 1), n <- rho n + 1.
__device__ __forceinline__ void observe_ema(float &v, float &n, float r, double rho) {
    const double vd = static_cast<double>(v), nd = static_cast<double>(n);
    const double eta = 1.0 / (rho * nd + 1.0);
    v = static_cast<float>(vd + eta * (static_cast<double>(r) - vd));
    n = static_cast<float>(rho * nd + 1.0);
}

// Both forms of the tracker share the update kernels: Ema = false keeps
// (alpha, beta), Ema = true keeps (v_hat, n_eff) in the same two arrays.
template <bool Ema>
__device__ __forceinline__ float mean_of(float a, float b) {
    if constexpr (Ema) return a;
    return static_cast<float>(static_cast<double>(a) / (static_cast<double>(a) + static_cast<double>(b)));
}

template <bool Ema>
__device__ __forceinline__ void apply(float &a, float &b, float r, double rho) {
    if constexpr (Ema) observe_ema(a, b, r, rho);
    else observe(a, b, r, rho);
}

constexpr int32_t kNoOwner = 0x7fffffff;
constexpr int kInfoRange = 1, kInfoRepeat = 2;  // bits of info[0]

__global__ void __launch_bounds__(256) fill_slots_kernel(int32_t *__restrict__ slot, int64_t N) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < N) slot[i] = kNoOwner;
}

__global__ void clear_info_kernel(int32_t *__restrict__ info) { info[0] = 0; }

// One thread per observation; ids are unique, so every thread owns its entry.  An id outside
// [0, N) is skipped and flagged.  With a slot table (all kNoOwner) a repeated id is flagged too:
// every observation files its number under its id and the ones that find another there raise
// the flag (the entries are left filed; the table is refilled before its next use).
template <bool Ema>
__global__ void __launch_bounds__(256)
tracker_update_unique_kernel(float *__restrict__ alpha, float *__restrict__ beta, int64_t N,
                             const int32_t *__restrict__ idx, const float *__restrict__ reward,
                             const float *__restrict__ kl, int B, double d_half, double rho_min,
                             double rho_max, uint32_t *__restrict__ n_obs,
                             float *__restrict__ v_prev, int32_t *__restrict__ info,
                             int32_t *__restrict__ slot) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= B) return;
    const int64_t i = idx[k];
    if (i < 0 || i >= N) {
        if (info) atomicOr(&info[0], kInfoRange);
        if (v_prev) v_prev[k] = __builtin_nanf("");
        return;
    }
    if (slot && info && atomicExch(&slot[i], k) != kNoOwner) atomicOr(&info[0], kInfoRepeat);
    float a = alpha[i], b = beta[i];
    if (v_prev) v_prev[k] = mean_of<Ema>(a, b);
    apply<Ema>(a, b, reward[k], discount(kl[k], d_half, rho_min, rho_max));
    alpha[i] = a;
    beta[i] = b;
    if (n_obs) n_obs[i] += 1u;
}

// Repeated ids, applied one after the other in batch order.  Every id belongs to one workgroup (a hash of
// the id), which reads the whole list of ids, keeps its own observations in LDS, sorts them by (id,
// place in the batch) and lets one thread per id walk that id's run: the state passes through
// registers from one observation to the next, and neither a table over the prompts nor an atomic
// on memory is needed.  (One workgroup filing claims in a table and applying the earliest pending
// observation of every id per round: 952 us for a prompt step of 40000 responses to 20000 prompts,
// 84 us now, 30 of them here before the lists were sorted by ranks.)  A list that might overflow is applied and restarted: the ids are read in
// batch order, so what is applied earlier is earlier in the batch.
// What is left is latency: the ids come a chunk of Vecs vectors per thread at a time, all of a thread's in flight together, and are
// counted before they are filed, so that a list which cannot overflow takes three barriers per chunk (4096 ids
// requested at a time and a barrier or two per 1024 of them: 26 us for that step, 18.5 now).  Up to kOwnCap ids need no
// count, and a chunk is no longer than the list: with one length of chunk for all, 16 ids took 5.4 us, 1000 9.5 and
// 5000 8.2, against 3.1, 6.3 and 7.1.
constexpr int kOwnThreads = 512, kOwnCap = 4096, kOwnVec = 4 * kOwnThreads;
static_assert(kOwnVec <= kOwnCap, "the ids of one vector per thread fit an empty list");
typedef int32_t i32x4u_t __attribute__((ext_vector_type(4), aligned(4)));  // (the list may start anywhere)
constexpr int kOwnSpan = 2048;          // sorted observations whose rewards and discounts are in LDS at a time
constexpr int kOwnGroups = 256;         // most workgroups: one per compute unit
constexpr int kOwnPerGroup = 128;       // observations per workgroup below that
// Up to here a list is sorted by ranks, n broadcast reads per thread and two barriers, instead of the 36 rounds
// with a barrier each that a bitonic sort of 256 keys takes (that step, with the diagnostics' shorter reductions:
// 88 -> 84 us).  The reads grow with n * n: longer lists keep the bitonic sort.
constexpr int kOwnRank = 256;

template <bool Ema, int Vecs>
__global__ void __launch_bounds__(kOwnThreads)
tracker_update_owned_kernel(float *__restrict__ alpha, float *__restrict__ beta, int64_t N,
                            const int32_t *__restrict__ idx, const float *__restrict__ reward,
                            const float *__restrict__ kl, int B, double d_half, double rho_min,
                            double rho_max, uint32_t *__restrict__ n_obs, float *__restrict__ v_prev,
                            int32_t *__restrict__ info, int shift) {
    __shared__ uint64_t key[kOwnCap];  // id << 32 | place in the batch
    __shared__ double rho[kOwnSpan];
    __shared__ float rew[kOwnSpan];
    __shared__ int count, coming;
    constexpr int kOwnVecs = Vecs, kOwnChunk = Vecs * kOwnVec;
    constexpr bool kOnce = kOwnChunk <= kOwnCap;  // launched for one chunk at most, which the list holds
    const int tid = threadIdx.x;
    auto mine = [&](int32_t i) {
        return static_cast<uint32_t>(i) < static_cast<uint32_t>(N) &&
               static_cast<uint64_t>(static_cast<uint32_t>(i) * 0x9E3779B1u) >> shift == blockIdx.x;
    };
    auto out_of_range = [&](int64_t k) {
        if (info) atomicOr(&info[0], kInfoRange);
        if (v_prev) v_prev[k] = __builtin_nanf("");
    };
    // applies the n observations in key[] (n is the same in every thread)
    auto apply_list = [&](int n) {
        if (n <= kOwnRank) {  // every key counts the smaller ones (keys are distinct)
            __syncthreads();
            const uint64_t mine = tid < n ? key[tid] : 0;
            int rank = 0;
            if (tid < n)
#pragma unroll 8
                for (int i = 0; i < n; ++i) rank += key[i] < mine;
            __syncthreads();
            if (tid < n) key[rank] = mine;
            __syncthreads();
        } else {
            int P = 1;
            while (P < n) P <<= 1;
            for (int i = n + tid; i < P; i += kOwnThreads) key[i] = ~0ull;
            __syncthreads();
            for (int k = 2; k <= P; k <<= 1)
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int t = tid; t < P / 2; t += kOwnThreads) {
                        const int i = 2 * t - (t & (j - 1));
                        const uint64_t x = key[i], y = key[i + j];
                        if ((x > y) == ((i & k) == 0)) {
                            key[i] = y;
                            key[i + j] = x;
                        }
                    }
                    __syncthreads();
                }
        }
        for (int w0 = 0; w0 < n; w0 += kOwnSpan) {
            const int w1 = n - w0 < kOwnSpan ? n : w0 + kOwnSpan;
            for (int i = w0 + tid; i < w1; i += kOwnThreads) {
                const int k = static_cast<int>(static_cast<uint32_t>(key[i]));
                rew[i - w0] = reward[k];
                rho[i - w0] = discount(kl[k], d_half, rho_min, rho_max);
            }
            __syncthreads();
            for (int i = w0 + tid; i < w1; i += kOwnThreads) {
                const uint32_t id = static_cast<uint32_t>(key[i] >> 32);
                if (i > w0 && static_cast<uint32_t>(key[i - 1] >> 32) == id) continue;  // not the first of its run
                float a = alpha[id], b = beta[id];
                int j = i;
                do {
                    if (v_prev) v_prev[static_cast<uint32_t>(key[j])] = mean_of<Ema>(a, b);
                    apply<Ema>(a, b, rew[j - w0], rho[j - w0]);
                    ++j;
                } while (j < w1 && static_cast<uint32_t>(key[j] >> 32) == id);
                alpha[id] = a;
                beta[id] = b;
                if (n_obs) n_obs[id] += static_cast<uint32_t>(j - i);
            }
            __syncthreads();  // the state is written, rew / rho / key may be overwritten
        }
    };
    if (tid == 0) count = 0;
    if constexpr (kOnce) {
        int32_t id[4 * Vecs];
#pragma unroll
        for (int j = 0; j < 4 * Vecs; ++j) id[j] = j * kOwnThreads + tid < B ? idx[j * kOwnThreads + tid] : 0;
        __syncthreads();  // the count is set
#pragma unroll
        for (int j = 0; j < 4 * Vecs; ++j) {
            const int k = j * kOwnThreads + tid;
            if (k >= B) continue;
            if (mine(id[j])) key[atomicAdd(&count, 1)] = static_cast<uint64_t>(id[j]) << 32 | static_cast<uint32_t>(k);
            else if (blockIdx.x == 0 && static_cast<uint32_t>(id[j]) >= static_cast<uint32_t>(N)) out_of_range(k);
        }
        __syncthreads();
        return apply_list(count);
    }
    for (int64_t base = 0; base < B; base += kOwnChunk) {
        i32x4u_t id[kOwnVecs];
        if (tid == 0) coming = 0;
        auto request = [&](int64_t k, i32x4u_t &v) {
            if (k + 3 < B) {
                v = *reinterpret_cast<const i32x4u_t *>(idx + k);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = k + e < B ? idx[k + e] : 0;
            }
        };
        auto file = [&](int64_t k) { key[atomicAdd(&count, 1)] = static_cast<uint64_t>(idx[k]) << 32 | static_cast<uint32_t>(k); };
#pragma unroll
        for (int c = 0; c < kOwnVecs; ++c) request(base + c * kOwnVec + tid * 4, id[c]);
        uint32_t own = 0;  // bit 4 c + e: id[c][e] is this workgroup's
        bool bad = false;
#pragma unroll
        for (int c = 0; c < kOwnVecs; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                own |= mine(id[c][e]) ? 1u << (4 * c + e) : 0u;
                bad |= static_cast<uint32_t>(id[c][e]) >= static_cast<uint32_t>(N);
            }
        if (base + kOwnChunk > B)  // ids past the end of the list are nobody's
#pragma unroll
            for (int c = 0; c < kOwnVecs; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (base + c * kOwnVec + tid * 4 + e >= B) own &= ~(1u << (4 * c + e));
        if (blockIdx.x == 0 && bad)
#pragma unroll 1
            for (int j = 0; j < 4 * kOwnVecs; ++j) {
                const int64_t k = base + (j >> 2) * kOwnVec + tid * 4 + (j & 3);
                if (k < B && static_cast<uint32_t>(idx[k]) >= static_cast<uint32_t>(N)) out_of_range(k);
            }
        __syncthreads();  // coming is cleared, the list of the chunk before is complete
        if (own) atomicAdd(&coming, __popc(own));
        __syncthreads();
        const int seen = count, more = coming;
        __syncthreads();  // everyone has seen them
        if (seen + more <= kOwnCap) {
            while (own) {
                const int j = __ffs(own) - 1;
                own &= own - 1;
                file(base + (j >> 2) * kOwnVec + tid * 4 + (j & 3));
            }
        } else {  // a vector per thread at a time, the list applied where the next might not fit
            int bound = seen;
#pragma unroll 1
            for (int c = 0; c < kOwnVecs; ++c) {
                if (bound + kOwnVec > kOwnCap) {
                    __syncthreads();
                    bound = count;
                    __syncthreads();
                    if (bound + kOwnVec > kOwnCap) {
                        apply_list(bound);
                        if (tid == 0) count = 0;
                        bound = 0;
                    }
                }
                __syncthreads();  // the count is set
                bound += kOwnVec;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (own >> (4 * c + e) & 1) file(base + c * kOwnVec + tid * 4 + e);
            }
        }
        __syncthreads();  // count and coming have been read
    }
    __syncthreads();
    apply_list(count);
}

__global__ void __launch_bounds__(256)
tracker_init_kernel(const float *__restrict__ v0, int64_t N, double n0, float *__restrict__ alpha,
                    float *__restrict__ beta) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const double v = static_cast<double>(v0[i]);
    alpha[i] = static_cast<float>(n0 * v);
    beta[i] = static_cast<float>(n0 * (1.0 - v));
}

// Raw advantage of response k in fp64.  An id outside [0, N) reads nothing: its baseline is NaN
// (so are the batch statistics) and it is flagged.
__device__ __forceinline__ double raw_advantage(const float *__restrict__ alpha, const float *__restrict__ beta,
                                                const int32_t *__restrict__ idx, const float *__restrict__ reward,
                                                int use_baseline, int64_t N, int32_t *__restrict__ info, int k) {
    double v = 0.0;
    if (use_baseline) {
        const int64_t i = idx[k];
        if (i < 0 || i >= N) {
            if (info) info[0] = kInfoRange;
            return __builtin_nan("");
        }
        const double a = alpha[i];
        v = beta ? a / (a + static_cast<double>(beta[i])) : a;
    }
    return static_cast<double>(reward[k]) - v;
}

// The same for responses k0, k0 + stride, ... below n (PER of them), the loads of all in flight together.
template <int PER>
__device__ __forceinline__ void raw_advantages(const float *__restrict__ alpha, const float *__restrict__ beta,
                                               const int32_t *__restrict__ idx, const float *__restrict__ reward,
                                               int use_baseline, int64_t N, int32_t *__restrict__ info, int k0, int stride,
                                               int n, double (&out)[PER]) {
    int32_t id[PER];
    float a[PER], b[PER], r[PER];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int k = k0 + i * stride;
        id[i] = use_baseline && k < n ? idx[k] : 0;
        r[i] = k < n ? reward[k] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const bool in = use_baseline && id[i] >= 0 && id[i] < N;  // (use_baseline: N >= 1, so id 0 may be read)
        a[i] = in ? alpha[id[i]] : 0.0f;
        b[i] = in && beta ? beta[id[i]] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        double v = 0.0;
        if (use_baseline) {
            v = beta ? static_cast<double>(a[i]) / (static_cast<double>(a[i]) + static_cast<double>(b[i])) : static_cast<double>(a[i]);
            if (id[i] < 0 || id[i] >= N) {
                v = __builtin_nan("");
                ok = false;
            }
        }
        out[i] = static_cast<double>(r[i]) - v;
    }
    if (info && !ok) info[0] = kInfoRange;
}

// One workgroup: raw advantages, then mean and standard deviation in fp64 with a
// fixed reduction order, then the normalised values.  The centred second pass
// avoids the cancellation of the sum-of-squares shortcut.
//
// Bound by the latency of id -> (alpha, beta): each of the three passes waited for both loads, one
// response per thread after the other.  Up to PER responses per thread stay in registers for all passes, their
// loads requested kAdvBatch at a time (a step of 4096 responses to 2^20 prompts: 57 -> 48 us; 8192 of them
// 31 -> 15 us, 16383 120 -> 47; all sixteen at once do not fit the registers of 1024 threads: 21 and 51).
// PER = 0 is the form without a limit.
constexpr int kAdvThreads = 1024;
constexpr int kAdvBatch = 8;

template <int PER>
__global__ void __launch_bounds__(kAdvThreads)
advantages_kernel(const float *__restrict__ alpha, const float *__restrict__ beta,
                  const int32_t *__restrict__ idx, const float *__restrict__ reward, int B, int ddof,
                  double eps_norm, int use_baseline, float *__restrict__ adv_raw,
                  float *__restrict__ adv_norm, float *__restrict__ stats, int64_t N, int32_t *__restrict__ info) {
    __shared__ double scratch[kAdvThreads / kWave];
    const int tid = threadIdx.x, NT = PER ? blockDim.x : kAdvThreads;
    auto raw = [&](int k) { return raw_advantage(alpha, beta, idx, reward, use_baseline, N, info, k); };
    if (info) {
        if (tid == 0) info[0] = 0;
        __syncthreads();
    }
    double kept[PER ? PER : 1];
    if constexpr (PER > kAdvBatch) {
#pragma unroll
        for (int h = 0; h < PER; h += kAdvBatch) {
            double part[kAdvBatch] = {};
            if (h * NT < B) raw_advantages<kAdvBatch>(alpha, beta, idx, reward, use_baseline, N, info, tid + h * NT, NT, B, part);
#pragma unroll
            for (int i = 0; i < kAdvBatch; ++i) kept[h + i] = part[i];
        }
    } else if constexpr (PER > 0) {
        raw_advantages<PER>(alpha, beta, idx, reward, use_baseline, N, info, tid, NT, B, kept);
    }
    auto each = [&](auto f) {  // f(k, raw advantage) for this thread's responses, in order
        if constexpr (PER > 0) {
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (tid + i * NT < B) f(tid + i * NT, kept[i]);
        } else {
            for (int64_t k = tid; k < B; k += NT) f(static_cast<int>(k), raw(static_cast<int>(k)));
        }
    };
    double s = 0.0;
    each([&](int k, double a) {
        if (adv_raw) adv_raw[k] = static_cast<float>(a);
        s += a;
    });
    const double mu = block_sum(s, scratch) / static_cast<double>(B);
    double ss = 0.0;
    each([&](int, double a) { ss += (a - mu) * (a - mu); });
    ss = block_sum(ss, scratch);
    const double dn = static_cast<double>(B - ddof);
    const double sigma = dn > 0.0 ? sqrt(ss / dn) : 0.0;
    const double den = sigma + eps_norm;
    // den is >= 0, or NaN and says so
    each([&](int k, double a) { adv_norm[k] = den == 0.0 ? 0.0f : static_cast<float>((a - mu) / den); });
    if (stats && tid == 0) {
        stats[0] = static_cast<float>(mu);
        stats[1] = static_cast<float>(sigma);
    }
}

// The same over many workgroups: two launches, each workgroup over `span` responses.  One compute unit fetches a line of
// memory per response and counter, 8192 of them for 4096 responses, in 10 us; spread over 16 units that is one latency.
// part[0..nb) are the workgroups' sums of the raw advantages, part[nb..2nb) the sums of
// squares about each workgroup's own mean; every workgroup of the second launch joins them
// (squares about the common mean = own squares + n (own mean - common mean)^2) in the same fixed
// order, so all of them hold the same mean and deviation, bit for bit, in every run.  (The order
// differs from the one-workgroup kernel's: the two agree to fp64 rounding, not bitwise.)
// Threads of a workgroup: kAdvNarrow with one response each, or kAdvThreads with kAdvPer.
constexpr int kAdvNarrow = 256, kAdvPer = 4, kAdvSpan = kAdvThreads * kAdvPer;

// phase 0: raw advantages and their partial sums; phase 1: normalised values and the statistics
template <int Phase, int NT, int PER>
__global__ void __launch_bounds__(NT)
advantages_wide_kernel(const float *__restrict__ alpha, const float *__restrict__ beta,
                       const int32_t *__restrict__ idx, const float *__restrict__ reward, int B, int ddof,
                       double eps_norm, int use_baseline, float *__restrict__ adv_raw, float *__restrict__ adv_norm,
                       float *__restrict__ stats, int64_t N, int32_t *__restrict__ info, double *__restrict__ part) {
    __shared__ double scratch[2 * NT / kWave];
    constexpr int span = NT * PER;
    const int nb = gridDim.x, tid = threadIdx.x;
    const int k0 = blockIdx.x * span, n = B - k0 < span ? B - k0 : span;  // n >= 1
    double kept[PER];
    raw_advantages<PER>(alpha, beta, use_baseline ? idx + k0 : idx, reward + k0, use_baseline, N, info, tid, NT, n, kept);
    if (Phase == 0) {
        double s = 0.0, ss = 0.0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int k = tid + i * NT;
            if (k >= n) continue;
            if (adv_raw) adv_raw[k0 + k] = static_cast<float>(kept[i]);
            s += kept[i];
        }
        s = block_sum(s, scratch);
        const double mu = s / static_cast<double>(n);
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (tid + i * NT < n) ss += (kept[i] - mu) * (kept[i] - mu);
        ss = block_sum(ss, scratch);
        if (tid == 0) {
            part[blockIdx.x] = s;
            part[nb + blockIdx.x] = ss;
        }
        return;
    }
    double s = 0.0, ss = 0.0;
    for (int i = tid; i < nb; i += NT) s += part[i];
    const double mu = block_sum(s, scratch) / static_cast<double>(B);
    for (int i = tid; i < nb; i += NT) {
        const double ni = static_cast<double>(i == nb - 1 ? B - i * span : span), d = part[i] / ni - mu;
        ss += part[nb + i] + ni * d * d;
    }
    ss = block_sum(ss, scratch);
    const double dn = static_cast<double>(B - ddof);
    const double sigma = dn > 0.0 ? sqrt(ss / dn) : 0.0;
    const double den = sigma + eps_norm;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int k = tid + i * NT;
        // den is >= 0, or NaN and says so
        if (k < n) adv_norm[k0 + k] = den == 0.0 ? 0.0f : static_cast<float>((kept[i] - mu) / den);
    }
    if (stats && blockIdx.x == 0 && tid == 0) {
        stats[0] = static_cast<float>(mu);
        stats[1] = static_cast<float>(sigma);
    }
}

// Diagnostics of the unnormalised advantages (one workgroup, fp64, fixed order).  Bound by the latency
// of a thread's loads and by its fp64 instructions: up to PER responses per thread stay in registers for both passes, all
// loads in flight together, a thread adds up its own in two chains (40000 responses: 14.5 us with eight
// requested at a time and a second pass over memory, 11.9 now; 8 and
// 8193 of them 6.4 and 7.7 us then, 6.6 and 7.9 by the kernels of 8 and 24 per thread, 6.3 and 7.4 by those of 1 and 12).  PER = 0 is the form without a limit: kDiagAhead responses
// requested at a time, and only a thread's last group asks which of its responses exist (10^6 responses: 275 us if every
// group does, 194).
constexpr int kDiagAhead = 8;

template <int PER>
__global__ void __launch_bounds__(kAdvThreads)
advantage_diagnostics_kernel(const float *__restrict__ adv_raw, const float *__restrict__ reward, int B,
                             float tau_tight, float tau_loose, float *__restrict__ diag) {
    __shared__ double scratch[4 * kAdvThreads / kWave];
    float a_kept[PER ? PER : 1], r_kept[PER ? PER : 1];
    if constexpr (PER > 0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const float *a_row = adv_raw + i * kAdvThreads, *r_row = reward + i * kAdvThreads;  // one place in a register for all
            const bool in = static_cast<int>(threadIdx.x) < B - i * kAdvThreads;
            a_kept[i] = in ? a_row[threadIdx.x] : 0.0f;
            r_kept[i] = in ? r_row[threadIdx.x] : 0.0f;
        }
    }
    auto each = [&](auto f) {  // f(advantage, reward) for this thread's responses, in order
        if constexpr (PER > 0) {
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (static_cast<int>(threadIdx.x) < B - i * kAdvThreads) f(a_kept[i], r_kept[i]);
            return;
        }
        int64_t k0 = threadIdx.x;
        for (; k0 + (kDiagAhead - 1) * kAdvThreads < B; k0 += kDiagAhead * kAdvThreads) {
            float a[kDiagAhead], r[kDiagAhead];
#pragma unroll
            for (int i = 0; i < kDiagAhead; ++i) {
                a[i] = adv_raw[k0 + i * kAdvThreads];
                r[i] = reward[k0 + i * kAdvThreads];
            }
#pragma unroll
            for (int i = 0; i < kDiagAhead; ++i) f(a[i], r[i]);
        }
        if (k0 < B) {  // this thread's last ones
            float a[kDiagAhead], r[kDiagAhead];
#pragma unroll
            for (int i = 0; i < kDiagAhead; ++i) {
                const int64_t k = k0 + i * kAdvThreads, kk = k < B ? k : B - 1;  // always a load, none behind a branch
                a[i] = adv_raw[kk];
                r[i] = reward[kk];
            }
#pragma unroll
            for (int i = 0; i < kDiagAhead; ++i)
                if (k0 + i * kAdvThreads < B) f(a[i], r[i]);
        }
    };
    int tight = 0, loose = 0;
    double sa = 0.0, sr = 0.0;
    each([&](float a, float r) {
        tight += fabsf(a) <= tau_tight ? 1 : 0;
        loose += fabsf(a) <= tau_loose ? 1 : 0;
        sa += static_cast<double>(a);
        sr += static_cast<double>(r);
    });
    double s[4] = {static_cast<double>(tight), static_cast<double>(loose), sa, sr};  // within tau_tight, tau_loose, advantages, rewards
    block_sums(s, scratch);
    const double ma = s[2] / B, mr = s[3] / B;
    if constexpr (PER > 0)  // not to be traced: their fp64 values, kept from the first pass, would not fit the registers
#pragma unroll
        for (int i = 0; i < PER; ++i) asm volatile("" : "+v"(a_kept[i]), "+v"(r_kept[i]));
    double v[2] = {};
    each([&](float a, float r) {
        const double da = static_cast<double>(a) - ma, dr = static_cast<double>(r) - mr;
        v[0] += da * da;
        v[1] += dr * dr;
    });
    block_sums(v, scratch);
    if (threadIdx.x == 0) {
        diag[0] = static_cast<float>(s[0] / B);
        diag[1] = static_cast<float>(s[1] / B);
        diag[2] = static_cast<float>(v[0] / B);
        diag[3] = static_cast<float>(v[1] / B);
    }
}

}  // namespace spo

using namespace spo;

extern "C" int spo_advantage_diagnostics(const float *adv_raw, const float *reward, int32_t B, float tau_tight,
                                         float tau_loose, float *diag, spo_stream_t stream) {
    if (!adv_raw || !reward || !diag) return SPO_ENULL;
    if (B < 1 || !(tau_tight >= 0.0f) || !(tau_loose >= tau_tight)) return SPO_EINVAL;
    auto *kernel = B <= kAdvThreads        ? advantage_diagnostics_kernel<1>
                   : B <= 8 * kAdvThreads  ? advantage_diagnostics_kernel<8>
                   : B <= 12 * kAdvThreads ? advantage_diagnostics_kernel<12>
                   : B <= 24 * kAdvThreads ? advantage_diagnostics_kernel<24>
                   : B <= 40 * kAdvThreads ? advantage_diagnostics_kernel<40>
                                           : advantage_diagnostics_kernel<0>;
    kernel<<<1, kAdvThreads, 0, as_stream(stream)>>>(adv_raw, reward, B, tau_tight, tau_loose, diag);
    return launch_status();
}

static size_t slot_table_bytes(int64_t N) { return align_up(static_cast<size_t>(N) * sizeof(int32_t), 256); }

template <bool Ema>
static int tracker_update_launch(float *alpha, float *beta, int64_t N, const int32_t *idx,
                                 const float *reward, const float *kl, int32_t B, float d_half,
                                 float rho_min, float rho_max, int ids_unique, uint32_t *n_obs,
                                 float *v_prev_out, int32_t *info, void *ws, size_t ws_bytes,
                                 spo_stream_t stream) {
    if (!alpha || !beta || !idx || !reward || !kl) return SPO_ENULL;
    if (N < 1 || N >= (int64_t(1) << 31) || B < 1) return SPO_EINVAL;
    if (!(d_half > 0.0f) || !(rho_min >= 0.0f) || !(rho_max <= 1.0f) || !(rho_min <= rho_max))
        return SPO_EINVAL;
    if (ws && (reinterpret_cast<uintptr_t>(ws) % 256 != 0)) return SPO_EINVAL;
    if ((ws || !ids_unique) && (!ws || ws_bytes < slot_table_bytes(N))) return SPO_EWORKSPACE;
    hipStream_t s = as_stream(stream);
    int32_t *slot = static_cast<int32_t *>(ws);
    if (info) clear_info_kernel<<<1, 1, 0, s>>>(info);
    if (ids_unique) {
        if (slot) fill_slots_kernel<<<static_cast<unsigned>(ceil_div(N, 256)), 256, 0, s>>>(slot, N);
        const int threads = 256, blocks = (B + threads - 1) / threads;
        tracker_update_unique_kernel<Ema><<<blocks, threads, 0, s>>>(alpha, beta, N, idx, reward, kl, B, d_half, rho_min,
                                                                      rho_max, n_obs, v_prev_out, info, slot);
    } else {
        int bits = 0;
        while (1 << bits < kOwnGroups && (static_cast<int64_t>(kOwnPerGroup) << bits) < B) ++bits;
        auto *kernel = B <= kOwnVec       ? tracker_update_owned_kernel<Ema, 1>
                       : B <= 2 * kOwnVec ? tracker_update_owned_kernel<Ema, 2>
                       : B <= 4 * kOwnVec ? tracker_update_owned_kernel<Ema, 4>
                                          : tracker_update_owned_kernel<Ema, 8>;
        kernel<<<1u << bits, kOwnThreads, 0, s>>>(alpha, beta, N, idx, reward, kl, B, d_half, rho_min, rho_max, n_obs, v_prev_out, info, 32 - bits);
    }
    return launch_status();
}

extern "C" size_t spo_tracker_update_workspace_bytes(int64_t N) { return N < 1 ? 0 : slot_table_bytes(N); }

extern "C" int spo_tracker_update(float *alpha, float *beta, int64_t N, const int32_t *idx,
                                  const float *reward, const float *kl, int32_t B, float d_half,
                                  float rho_min, float rho_max, int ids_unique, uint32_t *n_obs,
                                  float *v_prev_out, int32_t *info, void *ws, size_t ws_bytes,
                                  spo_stream_t stream) {
    return tracker_update_launch<false>(alpha, beta, N, idx, reward, kl, B, d_half, rho_min, rho_max,
                                        ids_unique, n_obs, v_prev_out, info, ws, ws_bytes, stream);
}

extern "C" int spo_tracker_update_ema(float *v_hat, float *n_eff, int64_t N, const int32_t *idx,
                                      const float *reward, const float *kl, int32_t B, float d_half,
                                      float rho_min, float rho_max, int ids_unique, uint32_t *n_obs,
                                      float *v_prev_out, int32_t *info, void *ws, size_t ws_bytes,
                                      spo_stream_t stream) {
    return tracker_update_launch<true>(v_hat, n_eff, N, idx, reward, kl, B, d_half, rho_min, rho_max,
                                       ids_unique, n_obs, v_prev_out, info, ws, ws_bytes, stream);
}

extern "C" int spo_tracker_init(const float *v0, int64_t N, float rho_min, float *alpha,
                                float *beta, spo_stream_t stream) {
    if (!v0 || !alpha || !beta) return SPO_ENULL;
    if (N < 1 || !(rho_min >= 0.0f) || !(rho_min < 1.0f)) return SPO_EINVAL;
    const int threads = 256;
    const int64_t blocks = ceil_div(N, threads);
    if (blocks >= (int64_t(1) << 31)) return SPO_ERANGE;
    tracker_init_kernel<<<static_cast<unsigned>(blocks), threads, 0, as_stream(stream)>>>(
        v0, N, 1.0 / (1.0 - static_cast<double>(rho_min)), alpha, beta);
    return launch_status();
}

// Responses that one workgroup takes although there is a workspace: what two launches cost is gained back where a compute unit
// waits for lines of memory, later where they come from the L2, latest where the table is a few lines per response or there is
// none.  (us in one workgroup and in two launches: 1025 responses to 2^20 prompts 7.8 and 6.6, 4096 15.1 and 7.6; 2048 to 2^18
// prompts 6.9 and 6.6, 1300 6.05 and 6.1; 2500 to 20000 6.6 and 6.6, 1025 5.8 and 6.3; 3000 to 1000 6.4 and 6.6.)
static int adv_one_workgroup(int64_t N) { return (N > int64_t(1) << 18 ? 1 : N > int64_t(1) << 15 ? 2 : 3) * kAdvThreads; }
// Above, up to kAdvNarrowMost workgroups of kAdvNarrow responses, then ones of kAdvSpan.
constexpr int kAdvNarrowMost = 256;
static size_t adv_parts_bytes(int B, int span) { return static_cast<size_t>(2 * ceil_div(B, span)) * sizeof(double); }

// (never smaller for a larger batch)
extern "C" size_t spo_advantages_workspace_bytes(int32_t B) {
    if (B < 1) return 0;
    const int narrow = B < kAdvNarrowMost * kAdvNarrow ? B : kAdvNarrowMost * kAdvNarrow;
    return std::max(adv_parts_bytes(narrow, kAdvNarrow), adv_parts_bytes(B, kAdvSpan));
}

extern "C" int spo_advantages(const float *alpha, const float *beta, int64_t N, const int32_t *idx,
                              const float *reward, int32_t B, int ddof, float eps_norm,
                              int use_baseline, float *adv_raw, float *adv_norm, float *stats,
                              int32_t *info, void *ws, size_t ws_bytes, spo_stream_t stream) {
    if (!reward || !adv_norm) return SPO_ENULL;
    if (use_baseline && (!alpha || !idx)) return SPO_ENULL;
    if (B < 1 || (use_baseline && N < 1) || ddof < 0 || ddof > 1 || !(eps_norm >= 0.0f))
        return SPO_EINVAL;
    if (ws && reinterpret_cast<uintptr_t>(ws) % 256 != 0) return SPO_EINVAL;
    if (ws && ws_bytes < adv_parts_bytes(B, kAdvSpan)) return SPO_EWORKSPACE;  // (enough for workgroups of kAdvSpan responses)
    hipStream_t s = as_stream(stream);
    double *part = static_cast<double *>(ws);
    auto two = [&](auto *first, auto *second, int span, int threads) {
        const unsigned nb = static_cast<unsigned>(ceil_div(B, span));
        if (info) clear_info_kernel<<<1, 1, 0, s>>>(info);
        first<<<nb, threads, 0, s>>>(alpha, beta, idx, reward, B, ddof, eps_norm, use_baseline, adv_raw, adv_norm, stats, N, info, part);
        second<<<nb, threads, 0, s>>>(alpha, beta, idx, reward, B, ddof, eps_norm, use_baseline, adv_raw, adv_norm, stats, N, info, part);
        return launch_status();
    };
    if (ws && B > adv_one_workgroup(use_baseline ? N : 0) && B <= kAdvNarrowMost * kAdvNarrow && ws_bytes >= adv_parts_bytes(B, kAdvNarrow))
        return two(advantages_wide_kernel<0, kAdvNarrow, 1>, advantages_wide_kernel<1, kAdvNarrow, 1>, kAdvNarrow, kAdvNarrow);
    if (ws && B >= 4 * kAdvSpan)
        return two(advantages_wide_kernel<0, kAdvThreads, kAdvPer>, advantages_wide_kernel<1, kAdvThreads, kAdvPer>, kAdvSpan, kAdvThreads);
    const int threads = B <= kWave ? kWave : kAdvThreads;
    auto *kernel = B <= kAdvThreads         ? advantages_kernel<1>
                   : B <= 4 * kAdvThreads   ? advantages_kernel<4>
                   : B <= 16 * kAdvThreads  ? advantages_kernel<16>
                                            : advantages_kernel<0>;
    kernel<<<1, threads, 0, s>>>(alpha, beta, idx, reward, B, ddof, eps_norm, use_baseline, adv_raw, adv_norm, stats, N, info);
    return launch_status();
}
