// Pieces shared by the fused and the logits-in forms of the clipped
// policy-gradient loss: the per-token surrogate, the masked reduction and the
// per-token gradient scale (Method, PPO-Clip objective with the normalised
// advantage of a response applied to each of its tokens).
#pragma once

#include "common.hpp"

namespace spo {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;  // finite stand-in for -inf in running maxima

struct Surrogate {
    float ratio, obj;
    bool active;  // the unclipped branch is the minimum: gradient flows
};

__device__ __forceinline__ Surrogate surrogate(float logp, float old_logp, float adv, float eps_low, float eps_high) {
    Surrogate r;
    r.ratio = expf(logp - old_logp);
    const float s1 = r.ratio * adv;
    const float c = fminf(fmaxf(r.ratio, 1.0f - eps_low), 1.0f + eps_high);
    const float s2 = c * adv;
    r.active = s1 <= s2;
    r.obj = r.active ? s1 : s2;
    return r;
}

// Per-block partial sums of the forward, added in block order by the last workgroup to finish.
struct FwdPartial {
    double sum_obj, count, clipped, sum_ratio;
};

// Response offsets a token workgroup keeps in LDS (a binary search through global memory is seven
// dependent loads for 128 responses).
constexpr int kCuStaged = 1024;

// cu - or, where B + 1 offsets fit, a copy of it in LDS - for response_of_token.  A barrier follows before it is read.
__device__ __forceinline__ const int32_t *stage_offsets(const int32_t *cu, int B, int32_t *lds) {
    if (B >= kCuStaged) return cu;
    for (int i = threadIdx.x; i <= B; i += blockDim.x) lds[i] = cu[i];
    return lds;
}

// What the per-token kernels of a call read; every per-token array starts at token t_base of the batch.
struct TokenInputs {
    const float *old_logp;
    const uint8_t *mask;      // NULL: all ones
    const float *adv_norm;
    const int32_t *cu;
    int B;
    float eps_low, eps_high;
    int64_t T, t_base;
};

static inline TokenInputs token_inputs(const spo_pg_desc *d, int64_t t0, int64_t T) {
    return TokenInputs{d->old_logp + t0, d->mask ? d->mask + t0 : nullptr, d->adv_norm, d->cu_seqlens, d->B,
                       d->eps_low, d->eps_high, T, t0};
}

// What a piece of the batch needs for its backward, where the weight of the loss is known beforehand:
// g[t] (see grad_factor; zero for T <= t < T_pad), and for batches without a mask what turns stored
// scaled probabilities into operands of the contractions (see the one-call form): c[t] and one entry
// of Q per token.
struct TokenGrad {
    float *g;                // NULL: forward only
    int64_t T_pad;
    const double *count;     // number of unmasked tokens
    float grad_loss;
    float *c;                // NULL: no scaled probabilities
    uint16_t *Q;
    int64_t q_blk, V;
    const int32_t *target;
};

// -(mask / M) * A * ratio * [unclipped branch is the minimum] * grad_loss
__device__ __forceinline__ float grad_factor(const Surrogate &r, float adv, double M, float grad_loss) {
    return r.active ? -(adv * r.ratio * grad_loss) / static_cast<float>(M) : 0.0f;
}

// One lane per token, a block of 64 tokens per `ways` wavefronts.  These merge the (running max, sum of
// exponentials) pairs of the vocabulary splits together (1191 tokens x 408 splits by one thread per token, a load
// at a time: 312 us); their first one forms lse, logp, the surrogate and, where asked for, the gradient factors.
// z_target[t] is the logit of the sampled token.  The workgroup that finishes last (counted in *done in blocks,
// zero beforehand, over all launches of the call: total_blocks) adds the partial sums in order and writes the loss.
constexpr int kTokThreads = kWave;  // tokens per block
constexpr int kTokWaves = 16;       // most wavefronts per workgroup

// How a launch over n_blocks blocks is cut: four splits for each of `ways` wavefronts while the blocks alone do not
// fill the chip (kTokChipWaves), and from kTokFewBlocks on several blocks per workgroup, more where there would be
// more than kTokChipGroups workgroups: their counts meet at one address.  (200000 tokens of two splits: 19 us, 27 with four
// blocks per workgroup and 71 with one, of 16 wavefronts.  Fitted while a count still wrote caches back, 11 ns each, and
// not again since it does not: it may be cheaper now.)
constexpr int kTokChipWaves = 2048, kTokChipGroups = 512, kTokFewBlocks = 64;
struct TokenShape {
    unsigned blocks, threads;
    int ways;
};
static inline TokenShape token_shape(int nsplit, int64_t n_blocks) {
    int ways = 1;
    while (ways < kTokWaves && ways * 4 < nsplit && ways * n_blocks < kTokChipWaves) ways *= 2;
    int waves = ways;
    while (waves < 4 ? n_blocks >= kTokFewBlocks : waves < kTokWaves && n_blocks * ways / waves > kTokChipGroups) waves *= 2;
    return TokenShape{static_cast<unsigned>(ceil_div(n_blocks, waves / ways)), static_cast<unsigned>(waves * kWave), ways};
}

static __global__ void __launch_bounds__(kTokWaves * kWave)
token_loss_kernel(const float *__restrict__ part_max, const float *__restrict__ part_sum, int nsplit, int ways,
                  int64_t split_stride, const float *__restrict__ z_target, TokenInputs in, float *__restrict__ logp_out,
                  float *__restrict__ lse_out, FwdPartial *__restrict__ partials, TokenGrad gr, int64_t n_blocks,
                  int64_t total_blocks, uint32_t *__restrict__ done, float *__restrict__ loss, float *__restrict__ stats) {
    __shared__ float sm[kTokWaves][kWave], ss[kTokWaves][kWave];
    __shared__ int32_t cu_lds[kCuStaged];
    __shared__ double scratch[4 * kTokWaves];
    __shared__ FwdPartial block_part[kTokWaves];
    __shared__ int last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, way = wave % ways;
    const int per_wg = static_cast<int>(blockDim.x >> 6) / ways;  // blocks per workgroup
    const int64_t first = static_cast<int64_t>(blockIdx.x) * per_wg, t = (first + wave / ways) * kTokThreads + lane;
    // What the end needs of this lane's token is requested first, and its advantage as soon as its response is known:
    // on their way while the splits are merged instead of one after the other behind them.
    const bool mine_t = way == 0 && t < in.T;
    float z = 0.0f, old = 0.0f, adv = 0.0f;
    double unmasked = 1.0;
    int64_t y = -1;
    bool live = false;
    if (mine_t) {
        z = z_target[t];
        old = in.old_logp[t];
        if (gr.g) unmasked = *gr.count;
        if (gr.c) y = gr.target[t];
        live = !in.mask || in.mask[t];
    }
    stage_offsets(in.cu, in.B, cu_lds);
    __syncthreads();
    if (live) {  // (apart: through one pointer to either memory every step of the search waits for all loads before it)
        const int r = in.B < kCuStaged ? response_of_token(cu_lds, in.B, in.t_base + t) : response_of_token(in.cu, in.B, in.t_base + t);
        adv = in.adv_norm[r];
    }
    float m = kNegBig, s = 0.0f;
    if (t < in.T) {
        constexpr int U = 8;  // pairs requested at a time
        for (int i0 = way; i0 < nsplit; i0 += U * ways) {
            float pm[U], ps[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * ways;
                pm[u] = i < nsplit ? part_max[i * split_stride + t] : kNegBig;
                ps[u] = i < nsplit ? part_sum[i * split_stride + t] : 0.0f;
            }
            float nm = m;
#pragma unroll
            for (int u = 0; u < U; ++u) nm = fmaxf(nm, pm[u]);
            s *= expf(m - nm);
#pragma unroll
            for (int u = 0; u < U; ++u) s += ps[u] * expf(pm[u] - nm);
            m = nm;
        }
    }
    sm[wave][lane] = m;
    ss[wave][lane] = s;
    __syncthreads();
    double so = 0.0, cnt = 0.0, clp = 0.0, sr = 0.0;
    if (way == 0) {
        float g = 0.0f, c = 0.0f;
        if (mine_t) {
            for (int w = 1; w < ways; ++w) m = fmaxf(m, sm[wave + w][lane]);
            s = 0.0f;
            for (int w = 0; w < ways; ++w) s += ss[wave + w][lane] * expf(sm[wave + w][lane] - m);
            const float lse = m + logf(s);
            const float logp = z - lse;
            lse_out[t] = lse;
            logp_out[t] = logp;
            if (live) {
                const Surrogate r = surrogate(logp, old, adv, in.eps_low, in.eps_high);
                so = logp == logp ? r.obj : logp;  // a NaN log-prob (target id outside the vocabulary) reaches the loss
                cnt = 1.0;
                clp = r.active ? 0.0 : 1.0;
                sr = r.ratio;
                if (gr.g) g = grad_factor(r, adv, unmasked, gr.grad_loss);
                if (gr.c && g != 0.0f) {
                    c = -g * r.ratio;  // the ratio is finite and positive where g != 0
                    if (y >= 0 && y < gr.V)
                        gr.Q[(y / 64) * gr.q_blk + t * 64 + y % 64] = f32_to_bf16(expf(old) - 1.0f / r.ratio);
                }
            }
        }
        if (gr.g && t < gr.T_pad) {
            gr.g[t] = g;
            if (gr.c) gr.c[t] = c;
        }
        so = wave_sum(so);
        cnt = wave_sum(cnt);
        clp = wave_sum(clp);
        sr = wave_sum(sr);
        if (lane == 0) block_part[wave / ways] = FwdPartial{so, cnt, clp, sr};
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int mine = static_cast<int>(n_blocks - first < per_wg ? n_blocks - first : per_wg);
        // Stores and loads that every XCD sees, and a wait for them before the count: a count that releases and acquires
        // would write back and invalidate whole caches for these 32 bytes.  That the sums are seen where the count is seen
        // is a property of gfx950, not of the language's memory model: relaxed stores and loads at agent scope go past the
        // caches of the XCD, and a store counts as done (vmcnt) when it is there.  (With what is requested first above: forward,
        // 100000 tokens at 64 x 128 39.1 -> 35.2 us, 8192 at 128 x 3000 29.1 -> 27.5, 25 at 384 x 30471 21.0 -> 20.3.)
        for (int b = 0; b < mine; ++b) {
            FwdPartial *p = partials + (in.t_base / kTokThreads + first + b);
            __hip_atomic_store(&p->sum_obj, block_part[b].sum_obj, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&p->count, block_part[b].count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&p->clipped, block_part[b].clipped, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&p->sum_ratio, block_part[b].sum_ratio, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = total_blocks == mine ||
               __hip_atomic_fetch_add(done, static_cast<uint32_t>(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   static_cast<uint32_t>(total_blocks - mine);
    }
    __syncthreads();
    if (!last) return;
    double v[4] = {};  // objective, unmasked, clipped, ratios
    constexpr int A = 4;  // partial sums requested at a time
    for (int64_t i0 = threadIdx.x; i0 < total_blocks; i0 += A * blockDim.x) {
        FwdPartial p[A];
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int64_t i = i0 + a * static_cast<int64_t>(blockDim.x);
            FwdPartial *q = partials + (i < total_blocks ? i : total_blocks - 1);  // always a load, none of them behind a branch
            p[a].sum_obj = __hip_atomic_load(&q->sum_obj, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            p[a].count = __hip_atomic_load(&q->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            p[a].clipped = __hip_atomic_load(&q->clipped, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            p[a].sum_ratio = __hip_atomic_load(&q->sum_ratio, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int a = 0; a < A; ++a) {
            if (i0 + a * static_cast<int64_t>(blockDim.x) >= total_blocks) break;
            v[0] += p[a].sum_obj;
            v[1] += p[a].count;
            v[2] += p[a].clipped;
            v[3] += p[a].sum_ratio;
        }
    }
    block_sums(v, scratch);
    if (threadIdx.x == 0) {
        cnt = v[1];
        loss[0] = cnt > 0.0 ? static_cast<float>(-v[0] / cnt) : 0.0f;
        if (stats) {
            stats[0] = static_cast<float>(cnt);
            stats[1] = cnt > 0.0 ? static_cast<float>(v[2] / cnt) : 0.0f;
            stats[2] = cnt > 0.0 ? static_cast<float>(v[3] / cnt) : 0.0f;
            stats[3] = static_cast<float>(v[0]);
        }
    }
}

// Number of set entries of mask[0..T), by one workgroup of up to 1024 threads; every thread receives it.
__device__ __forceinline__ int64_t count_mask(const uint8_t *__restrict__ mask, int64_t T, int *scratch) {
    auto set_bytes = [](uint32_t x) {  // bytes that are not zero
        x |= x >> 4;
        x |= x >> 2;
        x |= x >> 1;
        return __popc(x & 0x01010101u);
    };
    const int64_t off = (16 - reinterpret_cast<uintptr_t>(mask) % 16) % 16, head = off < T ? off : T;
    const int64_t nvec = (T - head) / 16, tail0 = head + nvec * 16;
    const uint4 *v = reinterpret_cast<const uint4 *>(mask + head);
    int c = 0;
    if (threadIdx.x < head) c += mask[threadIdx.x] != 0;
    if (tail0 + threadIdx.x < T) c += mask[tail0 + threadIdx.x] != 0;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < nvec; i += blockDim.x) {
        const uint4 u = v[i];
        c += set_bytes(u.x) + set_bytes(u.y) + set_bytes(u.z) + set_bytes(u.w);
    }
    return block_sum(c, scratch);  // T < 2^31
}

// Gradient factor of token t from the forward's log-prob; cu: see stage_offsets, M: number of unmasked tokens.
__device__ __forceinline__ float token_grad(const float *__restrict__ logp, const TokenInputs &in, const int32_t *cu, double M,
                                            float grad_loss, int64_t t) {
    if (in.mask && !in.mask[t]) return 0.0f;
    const float adv = in.adv_norm[response_of_token(cu, in.B, in.t_base + t)];
    return grad_factor(surrogate(logp[t], in.old_logp[t], adv, in.eps_low, in.eps_high), adv, M, grad_loss);
}

// count[0] = number of unmasked tokens.  One workgroup.
static __global__ void __launch_bounds__(1024)
mask_count_kernel(const uint8_t *__restrict__ mask, int64_t T, double *__restrict__ count) {
    __shared__ int scratch[1024 / kWave];
    const int64_t c = count_mask(mask, T, scratch);
    if (threadIdx.x == 0) count[0] = static_cast<double>(c);
}

// g[t] (see grad_factor) from the forward's log-probs; entries T <= t < T_pad are zero so that padded
// tokens contribute nothing.  count == NULL: every workgroup counts the mask itself (kCountInline).
constexpr int kGradThreads = 256;
constexpr int64_t kCountInline = 32768;  // tokens: 8 loads per thread; above, one workgroup counts for all

static __global__ void __launch_bounds__(kGradThreads)
grad_scale_kernel(const float *__restrict__ logp, TokenInputs in, int64_t T_pad, float grad_loss,
                  const double *__restrict__ count, float *__restrict__ g) {
    __shared__ int32_t cu_lds[kCuStaged];
    __shared__ int scratch[kGradThreads / kWave];
    const int64_t t = static_cast<int64_t>(blockIdx.x) * kGradThreads + threadIdx.x;
    const int32_t *cu = stage_offsets(in.cu, in.B, cu_lds);
    const double M = count ? count[0] : static_cast<double>(in.mask ? count_mask(in.mask, in.T, scratch) : in.T);
    __syncthreads();
    if (t >= T_pad) return;
    g[t] = t < in.T ? token_grad(logp, in, cu, M, grad_loss, t) : 0.0f;
}

// The gradient factors of a whole batch; `count` is scratch for batches with a long mask.
static inline void launch_grad_scale(const spo_pg_desc *d, const float *logp, int64_t T_pad, float grad_loss,
                                     double *count, float *g, hipStream_t s) {
    const bool apart = d->mask && d->T > kCountInline;
    if (apart) mask_count_kernel<<<1, 1024, 0, s>>>(d->mask, d->T, count);
    grad_scale_kernel<<<static_cast<unsigned>(ceil_div(T_pad, kGradThreads)), kGradThreads, 0, s>>>(
        logp, token_inputs(d, 0, d->T), T_pad, grad_loss, apart ? count : nullptr, g);
}

// Host-side checks common to forward and backward.
static inline int validate_pg_desc(const spo_pg_desc *d) {
    if (!d) return SPO_ENULL;
    if (d->struct_size != sizeof(spo_pg_desc)) return SPO_EINVAL;
    if (d->dtype != SPO_BF16 && d->dtype != SPO_FP32) return SPO_EINVAL;
    if (d->T < 0 || d->V < 1 || d->B < 1) return SPO_EINVAL;
    if (d->T >= (int64_t(1) << 31) || d->V >= (int64_t(1) << 31)) return SPO_ERANGE;
    if (!(d->eps_low >= 0.0f) || !(d->eps_high >= 0.0f)) return SPO_EINVAL;
    if (!d->adv_norm || !d->cu_seqlens) return SPO_ENULL;
    if (d->T > 0 && (!d->target || !d->old_logp)) return SPO_ENULL;
    if (!d->logits) {
        if (d->w_layout != SPO_W_VH && d->w_layout != SPO_W_HV) return SPO_EINVAL;
        if (!d->W || (d->T > 0 && !d->hidden)) return SPO_ENULL;
        if (d->H < 1) return SPO_EINVAL;
        if (d->H % 64 != 0) return SPO_EUNSUPPORTED;
        if (d->H > 65536) return SPO_ERANGE;
    }
    return SPO_OK;
}

}  // namespace spo
