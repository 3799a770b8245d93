// Logits-in form of the clipped policy-gradient loss: the [T x V] logits already
// exist and are streamed once (forward) or read once and written once
// (backward).  Pure HBM streaming, 16 bytes per lane and access.
#include <algorithm>

#include "pg_common.hpp"
#include "timing.hpp"

namespace spo {

// What bounds both kernels is memory, and how many separate streams of addresses are open at once:
// a workgroup per row of 304 KB keeps 2048 rows open (8192 x 151936 bf16: forward 451 us, backward
// 968 us = 5.5 and 5.1 TB/s).  So a row is cut into short segments, neighbouring workgroups work on
// neighbouring segments, and the chip sweeps the array nearly in order (350 us = 7.1 TB/s and
// 772 us = 6.4 TB/s).  The forward takes two rounds of kLseGroup 16-byte loads per thread (a third of
// the partial results of one round; with four 368 us), the second on its way while the first is worked
// on; the backward has nothing to carry along and takes one round of kGradGroup (four per thread:
// 806 us, two rounds of four 842 us).
// Arrays that no cache can hold are read and written with the non-temporal hint: the forward of the
// next pass then finds no modified lines of the gradients to drain first (forward 437 -> 350 us).
// Rows of a few thousand entries are bound by instructions as well: a thread works on two or three vectors per
// row.  There vectors that a segment does not have are not worked on, a segment of one round has no second one to
// request, and a wavefront's pairs are merged with one exponential (60000 rows of 4104 in bf16: 138 -> 81 us;
// a workgroup per row without segments took 96).
constexpr int kRowThreads = 256;
// Largest magnitude of a maximum at which the exponents are formed in one multiply-add.  What is lost with the
// maximum's product is half of its last place: a factor common to all, as small as the log-sum-exp's own rounding up to
// here, but past the range of exponents in rows that are masked with -1e30 throughout.
constexpr float kFarLogit = 65536.0f;
constexpr int kLseGroup = 4, kLseRounds = 2, kGradGroup = 2;
constexpr int64_t kStreamBytes = int64_t(256) << 20;  // the Infinity Cache

// 16 bytes of a row as floats and back
template <typename T> struct Vec;
template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    __device__ static __forceinline__ void unpack(const uint4 &u, float (&x)[8]) {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = __uint_as_float(w[i] << 16);
            x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ static __forceinline__ uint4 pack(const float (&x)[8]) {
        return make_uint4(pack_bf16x2_rn(x[0], x[1]), pack_bf16x2_rn(x[2], x[3]), pack_bf16x2_rn(x[4], x[5]),
                          pack_bf16x2_rn(x[6], x[7]));
    }
    __device__ static __forceinline__ float get(const bf16_t *p) { return bf16_to_f32(*p); }
    __device__ static __forceinline__ void put(bf16_t *p, float v) { *p = f32_to_bf16(v); }
};
template <> struct Vec<float> {
    static constexpr int N = 4;
    __device__ static __forceinline__ void unpack(const uint4 &u, float (&x)[4]) {
        x[0] = __uint_as_float(u.x); x[1] = __uint_as_float(u.y); x[2] = __uint_as_float(u.z); x[3] = __uint_as_float(u.w);
    }
    __device__ static __forceinline__ uint4 pack(const float (&x)[4]) {
        return make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
    }
    __device__ static __forceinline__ float get(const float *p) { return *p; }
    __device__ static __forceinline__ void put(float *p, float v) { *p = v; }
};

// 16 bytes from an address that may only be aligned to the element (the hardware takes it), and to a
// 16-byte boundary; Stream: with the non-temporal hint
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <typename T> struct Unaligned16;
template <> struct Unaligned16<bf16_t> { typedef u32x4_t V __attribute__((aligned(2))); };
template <> struct Unaligned16<float> { typedef u32x4_t V __attribute__((aligned(4))); };

template <bool Stream, typename T>
__device__ __forceinline__ uint4 load16(const T *p) {
    const auto *q = reinterpret_cast<const typename Unaligned16<T>::V *>(p);
    const u32x4_t v = Stream ? __builtin_nontemporal_load(q) : *q;
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool Stream>
__device__ __forceinline__ void store16(uint4 *p, const uint4 &u) {
    const u32x4_t v = {u.x, u.y, u.z, u.w};
    if (Stream) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(p));
    else *reinterpret_cast<u32x4_t *>(p) = v;
}

// Elements [0, n) of a row segment as: a head of single elements up to the first 16-byte boundary,
// whole vectors, a tail of single elements.
struct Span {
    int head, nvec, tail;  // a segment has fewer than 2^31 elements
    template <typename T>
    __device__ __forceinline__ Span(const T *p, int n) {
        const int off = static_cast<int>((16 - reinterpret_cast<uintptr_t>(p) % 16) % 16 / sizeof(T));
        head = off < n ? off : n;
        nvec = (n - head) / Vec<T>::N;
        tail = n - head - nvec * Vec<T>::N;
    }
};

// Which part of which row a group of threads works on: `unit` counts (row, segment) pairs, the
// segments of a row next to each other.
struct RowGrid {
    int64_t rows, seg_len;  // elements per segment
    int nseg, per_wg;       // segments per row, (row, segment) pairs per workgroup
    __host__ __device__ uint32_t units() const { return static_cast<uint32_t>(rows * nseg); }  // < 2^32: of 4 KB segments, 16 TB
    __host__ dim3 blocks() const { return fold_grid(ceil_div(rows * nseg, per_wg)); }
};

// The unit of a group of TR threads, a value the compiler knows to be the same in a whole wavefront: its place and
// extent are then scalar arithmetic (30000 rows of 4104 in bf16: 66 -> 62 us).
template <int TR>
__device__ __forceinline__ int64_t group_unit() {
    if constexpr (TR == kRowThreads) return flat_block();
    else return flat_block() * (kRowThreads / TR) + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / TR);
}

// running (max, sum of exp(x - max)) merged with another pair
__device__ __forceinline__ void lse_merge(float &m, float &s, float om, float os) {
    const float nm = fmaxf(m, om);
    s = s * __builtin_amdgcn_exp2f((m - nm) * kLog2e) + os * __builtin_amdgcn_exp2f((om - nm) * kLog2e);
    m = nm;
}

// (max, sum-exp) of one segment of a row, by TR threads (a workgroup or one wavefront of it), and the
// target's logit.  part_max / part_sum [segment][row].  Also clears *done.
template <typename T, int TR, int Rounds, bool Stream>
__global__ void __launch_bounds__(kRowThreads)
logits_row_lse_kernel(const T *__restrict__ logits, int64_t V, RowGrid grid, const int32_t *__restrict__ target,
                      float *__restrict__ part_max, float *__restrict__ part_sum, float *__restrict__ z_target,
                      uint32_t *__restrict__ done) {
    constexpr int N = Vec<T>::N, U = kLseGroup;
    const int64_t unit = group_unit<TR>();
    const int tid = threadIdx.x % TR;
    if (unit == 0 && threadIdx.x == 0) *done = 0u;  // for the kernel that follows
    if (unit >= grid.units()) return;  // TR < kRowThreads only: no barrier below in that case
    const uint32_t seg = static_cast<uint32_t>(unit) % static_cast<uint32_t>(grid.nseg);
    const int64_t t = static_cast<uint32_t>(unit) / static_cast<uint32_t>(grid.nseg), e0 = seg * grid.seg_len;
    const T *p = logits + t * V + e0;
    const Span sp(p, static_cast<int>(V - e0 < grid.seg_len ? V - e0 : grid.seg_len));
    float zt = 0.0f;
    if (seg == 0 && tid == 0) {
        const int64_t y = target[t];  // an id outside [0, V) gives NaN instead of a read out of bounds
        zt = (y >= 0 && y < V) ? Vec<T>::get(logits + t * V + y) : __builtin_nanf("");
    }
    // the few elements outside the whole vectors, one per thread
    float m = kNegBig, s = 0.0f;
    if (tid < sp.head + sp.tail) {
        const float x = Vec<T>::get(p + (tid < sp.head ? tid : tid + sp.nvec * N));
        m = fmaxf(m, x);
        s = __builtin_amdgcn_exp2f((x - m) * kLog2e);
    }
    const T *body = p + sp.head;
    auto request = [&](uint4 (&v)[U], int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * TR < sp.nvec) v[u] = load16<Stream>(body + (i0 + u * TR) * N);
    };
    auto take = [&](const uint4 (&v)[U], int i0) {
        // one new maximum and one rescaling of the running sum for the whole group; vectors past the end are left out
        // (rows of 4104: one in two of the group's)
        float x[U][N], mx = m;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * TR >= sp.nvec) break;
            Vec<T>::unpack(v[u], x[u]);
#pragma unroll
            for (int i = 0; i < N; ++i) mx = fmaxf(mx, x[u][i]);
        }
        const float nm2 = -mx * kLog2e;
        float a[U] = {};
        auto add = [&](auto exponent) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u * TR >= sp.nvec) break;
#pragma unroll
                for (int i = 0; i < N; ++i) a[u] += __builtin_amdgcn_exp2f(exponent(x[u][i]));
            }
        };
        if (__any(i0 < sp.nvec && fabsf(mx) > kFarLogit)) add([&](float v) { return (v - mx) * kLog2e; });
        else add([&](float v) { return fmaf(v, kLog2e, nm2); });
        s = s * __builtin_amdgcn_exp2f((m - mx) * kLog2e) + ((a[0] + a[1]) + (a[2] + a[3]));
        m = mx;
    };
    uint4 cur[U];
    request(cur, tid);
    if constexpr (Rounds > 1) {
        uint4 nxt[U];
        for (int i0 = tid; i0 < sp.nvec; i0 += U * TR) {
            request(nxt, i0 + U * TR);
            take(cur, i0);
#pragma unroll
            for (int u = 0; u < U; ++u) cur[u] = nxt[u];
        }
    } else {
        take(cur, tid);
    }
    // one maximum for the wavefront, then one rescaling and the sum (merging pairs takes two exponentials per step)
    float top = m;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, kWave));
    s = wave_sum(s * __builtin_amdgcn_exp2f((m - top) * kLog2e));
    m = top;
    if constexpr (TR > kWave) {
        __shared__ float sm[TR / kWave], ss[TR / kWave];
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) { sm[wave] = m; ss[wave] = s; }
        __syncthreads();
        m = sm[0];
        s = ss[0];
        for (int w = 1; w < TR / kWave; ++w) lse_merge(m, s, sm[w], ss[w]);
    }
    if (tid == 0) {
        part_max[seg * grid.rows + t] = m;
        part_sum[seg * grid.rows + t] = s;
        if (seg == 0) z_target[t] = zt;
    }
}

// d_logits[t][v] = g[t] * ([v == target[t]] - exp(z[t][v] - lse[t])) of one segment of a row (at most
// kGradGroup vectors per thread); rows whose scale is zero are written as zeros without being read.
// Vectors are aligned on the output side; the input's (the same boundaries unless the two arrays are
// offset against each other) may be unaligned.
template <typename T, int TR, bool Stream>
__global__ void __launch_bounds__(kRowThreads)
logits_row_grad_kernel(const T *__restrict__ logits, int64_t V, RowGrid grid, const int32_t *__restrict__ target,
                       const float *__restrict__ lse, const float *__restrict__ g, T *__restrict__ d_logits) {
    constexpr int N = Vec<T>::N, U = kGradGroup;
    const int64_t unit = group_unit<TR>();
    const int tid = threadIdx.x % TR;
    if (unit >= grid.units()) return;
    const uint32_t nseg = static_cast<uint32_t>(grid.nseg);
    const int64_t t = static_cast<uint32_t>(unit) / nseg, e0 = (static_cast<uint32_t>(unit) % nseg) * grid.seg_len;
    const T *p = logits + t * V + e0;
    T *out = d_logits + t * V + e0;
    const Span sp(out, static_cast<int>(V - e0 < grid.seg_len ? V - e0 : grid.seg_len));
    const float gt = g[t], ng = -gt, nl = -lse[t] * kLog2e;
    const int64_t yl = static_cast<int64_t>(target[t]) - e0;  // target's place in the segment
    const int y = yl >= 0 && yl < grid.seg_len ? static_cast<int>(yl) : -1;
    auto grad = [&](float x) { return ng * __builtin_amdgcn_exp2f(fmaf(x, kLog2e, nl)); };
    if (tid < sp.head + sp.tail) {
        const int e = tid < sp.head ? tid : tid + sp.nvec * N;
        Vec<T>::put(out + e, gt != 0.0f ? grad(Vec<T>::get(p + e)) + (e == y ? gt : 0.0f) : 0.0f);
    }
    const T *body = p + sp.head;
    uint4 *dst = reinterpret_cast<uint4 *>(out + sp.head);
    if (gt == 0.0f) {
        for (int i = tid; i < sp.nvec; i += TR) store16<Stream>(dst + i, make_uint4(0u, 0u, 0u, 0u));
        return;
    }
    const int yv = y >= sp.head ? (y - sp.head) / N : -1, yr = y >= sp.head ? (y - sp.head) % N : 0;
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (tid + u * TR < sp.nvec) v[u] = load16<Stream>(body + (tid + u * TR) * N);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int iv = tid + u * TR;
        if (iv >= sp.nvec) break;
        float x[N];
        Vec<T>::unpack(v[u], x);
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = grad(x[i]);
        if (iv == yv) {
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (i == yr) x[i] += gt;
        }
        store16<Stream>(dst + iv, Vec<T>::pack(x));
    }
}

// How the rows are cut: into segments of `rounds` rounds of `group` vectors per thread, of which a short rest is one
// more.  Where that would be one of few, all are made equal (8000 rows of 16392 in bf16 in segments of 16384 and 8:
// 68 us, in halves 50); where it is one of many, whole rounds are the better cut (8192 rows of 151936, loss and
// gradient in turn: 1200 us, in equal segments 1216).  Rows that give a workgroup little work go
// to single wavefronts, four to a workgroup: up to narrow_eighths eighths of a round (60000 rows of 4104 in bf16:
// a workgroup each 116 us, two wavefronts each 96; of 8192, a whole round, 84 against 97).
constexpr int kLseNarrow = 5, kGradNarrow = 4, kFewSegments = 8;
static RowGrid row_grid(const spo_pg_desc *d, int group, int rounds, int narrow_eighths) {
    const int64_t n = d->dtype == SPO_FP32 ? 4 : 8;  // elements per vector
    RowGrid g;
    g.rows = d->T;
    const bool narrow = d->V * 8 <= kRowThreads * group * n * narrow_eighths;
    g.per_wg = narrow ? kRowThreads / kWave : 1;
    g.seg_len = (narrow ? kWave : kRowThreads) * group * n * rounds;
    g.nseg = static_cast<int>(ceil_div(d->V, g.seg_len));
    // of few segments, equal ones: at most as long as they were, so as many of them, none empty
    constexpr int64_t kLine = 64;  // elements: they start on cache lines when the row does
    if (g.nseg <= kFewSegments) g.seg_len = ceil_div(ceil_div(d->V, g.nseg), kLine) * kLine;
    return g;
}

// the forward goes down to one round per segment where two would leave compute units without their
// eight workgroups (256 x 151936 bf16: 17.4 against 18.0 us)
static RowGrid lse_grid(const spo_pg_desc *d) {
    const RowGrid g = row_grid(d, kLseGroup, kLseRounds, kLseNarrow);
    return g.units() >= 2048 ? g : row_grid(d, kLseGroup, 1, kLseNarrow);
}

static bool streams(const spo_pg_desc *d) {
    return d->T * d->V * (d->dtype == SPO_FP32 ? 4 : 2) > kStreamBytes;
}

struct LogitsFwdPlan {
    RowGrid grid;
    float *row_max, *row_sum, *z_target;
    FwdPartial *partials;
    uint32_t *done;
    int64_t nblk_tok;
    size_t bytes;
};

static LogitsFwdPlan plan_logits_fwd(const spo_pg_desc *d, void *ws) {
    LogitsFwdPlan p;
    const int64_t Tn = std::max<int64_t>(d->T, 1);
    p.nblk_tok = ceil_div(Tn, kTokThreads);
    p.grid = lse_grid(d);
    Arena a(ws);
    // room for rows of T and V cut into the shortest segments of either type (0.4 % of the logits' bytes): the segments
    // in use get longer with T and V, and room sized for the largest batch is to serve every smaller one
    const size_t room = static_cast<size_t>(Tn * ceil_div(d->V, kWave * kLseGroup * Vec<float>::N));
    p.row_max = a.take<float>(room);
    p.row_sum = a.take<float>(room);
    p.z_target = a.take<float>(Tn);
    p.partials = a.take<FwdPartial>(p.nblk_tok);
    p.done = a.take<uint32_t>(1);
    p.bytes = a.used;
    return p;
}

template <typename T, int TR, bool Stream>
static void launch_row_lse(const spo_pg_desc *d, const LogitsFwdPlan &p, hipStream_t s) {
    auto *kernel = p.grid.seg_len <= TR * kLseGroup * Vec<T>::N ? logits_row_lse_kernel<T, TR, 1, Stream>
                                                               : logits_row_lse_kernel<T, TR, kLseRounds, Stream>;
    kernel<<<p.grid.blocks(), kRowThreads, 0, s>>>(
        static_cast<const T *>(d->logits), d->V, p.grid, d->target, p.row_max, p.row_sum, p.z_target,
        p.done);
}
template <typename T>
static void launch_row_lse(const spo_pg_desc *d, const LogitsFwdPlan &p, hipStream_t s) {
    if (p.grid.per_wg > 1) streams(d) ? launch_row_lse<T, kWave, true>(d, p, s) : launch_row_lse<T, kWave, false>(d, p, s);
    else if (streams(d)) launch_row_lse<T, kRowThreads, true>(d, p, s);
    else launch_row_lse<T, kRowThreads, false>(d, p, s);
}

template <typename T, int TR, bool Stream>
static void launch_row_grad(const spo_pg_desc *d, const RowGrid &grid, const float *lse, const float *g, void *d_logits,
                            hipStream_t s) {
    logits_row_grad_kernel<T, TR, Stream><<<grid.blocks(), kRowThreads, 0, s>>>(
        static_cast<const T *>(d->logits), d->V, grid, d->target, lse, g, static_cast<T *>(d_logits));
}
template <typename T>
static void launch_row_grad(const spo_pg_desc *d, const float *lse, const float *g, void *d_logits, hipStream_t s) {
    const RowGrid grid = row_grid(d, kGradGroup, 1, kGradNarrow);
    if (grid.per_wg > 1) launch_row_grad<T, kWave, false>(d, grid, lse, g, d_logits, s);
    else if (streams(d)) launch_row_grad<T, kRowThreads, true>(d, grid, lse, g, d_logits, s);
    else launch_row_grad<T, kRowThreads, false>(d, grid, lse, g, d_logits, s);
}

int logits_fwd_workspace(const spo_pg_desc *d, size_t *bytes) {
    *bytes = plan_logits_fwd(d, nullptr).bytes;
    return SPO_OK;
}

int logits_fwd(const spo_pg_desc *d, float *loss, float *logp, float *lse, float *stats, void *ws,
               size_t ws_bytes, hipStream_t s) {
    const LogitsFwdPlan p = plan_logits_fwd(d, ws);
    if (ws_bytes < p.bytes) return SPO_EWORKSPACE;
    if (d->T > 0) {
        ScopedKernelTimer timer(kTimeLogitsFwd, s);
        if (d->dtype == SPO_BF16) launch_row_lse<bf16_t>(d, p, s);
        else launch_row_lse<float>(d, p, s);
    }
    const TokenShape tok = token_shape(p.grid.nseg, p.nblk_tok);
    token_loss_kernel<<<tok.blocks, tok.threads, 0, s>>>(
        p.row_max, p.row_sum, p.grid.nseg, tok.ways, d->T, p.z_target, token_inputs(d, 0, d->T), logp, lse, p.partials,
        TokenGrad{}, p.nblk_tok, p.nblk_tok, p.done, loss, stats);
    return launch_status();
}

struct LogitsBwdPlan {
    double *count;
    float *g;
    size_t bytes;
};

static LogitsBwdPlan plan_logits_bwd(const spo_pg_desc *d, void *ws) {
    LogitsBwdPlan p;
    Arena a(ws);
    p.count = a.take<double>(1);
    p.g = a.take<float>(std::max<int64_t>(d->T, 1));
    p.bytes = a.used;
    return p;
}

int logits_bwd_workspace(const spo_pg_desc *d, size_t *bytes) {
    *bytes = plan_logits_bwd(d, nullptr).bytes;
    return SPO_OK;
}

int logits_bwd(const spo_pg_desc *d, const float *logp, const float *lse, float grad_loss, void *d_logits,
               void *ws, size_t ws_bytes, hipStream_t s) {
    if (!d_logits) return SPO_ENULL;
    const LogitsBwdPlan p = plan_logits_bwd(d, ws);
    if (ws_bytes < p.bytes) return SPO_EWORKSPACE;
    if (d->T == 0) return SPO_OK;
    launch_grad_scale(d, logp, d->T, grad_loss, p.count, p.g, s);
    ScopedKernelTimer timer(kTimeLogitsBwd, s);
    if (d->dtype == SPO_BF16) launch_row_grad<bf16_t>(d, lse, p.g, d_logits, s);
    else launch_row_grad<float>(d, lse, p.g, d_logits, s);
    return launch_status();
}

}  // namespace spo
