// bf16 MFMA contraction core for gfx950 (CDNA4, 64-wide wavefronts).
//
// Computes a BM x BN tile of  D[m][n] = sum_k A(m,k) B(n,k)  where each operand is stored
// either with the contraction index contiguous (rows along k: hidden states and a head
// [V,H] for the logits, dZ for dHidden) or with the contraction index as the row index
// (columns along k: dZ and hidden states for dW, which contracts over tokens; a head as it
// was given, for the contraction that runs across its rows).  All forms share the tile shape, the
// schedule and the accumulator layout.
//
// Data path per stage of 64 contraction elements (128 bytes = one cache line per
// operand row; half-line rows were measured to halve the L2->LDS rate):
//   HBM/L2 --global_load_lds_dwordx4--> LDS (two stages)  --ds_read_b128-->
//   VGPR fragments --v_mfma_f32_16x16x32_bf16--> fp32 accumulators.
// Global loads go straight to LDS without passing through registers.  A tile
// row is 8 chunks of 16 bytes; chunk c of row r is stored at chunk position
// c ^ swz(r), which makes both the 64 lanes x 16 B fragment reads and the
// linear DMA writes free of bank conflicts.  The swizzle is applied on the
// global side (each lane fetches the chunk that belongs at its LDS slot),
// because the DMA writes lane i at base + 16*i.
//
// Accumulator layout of one 16x16 block (v_mfma_f32_16x16x32_bf16): lane l
// holds column n = l % 16 and, in register r, row m = 4*(l/16) + r.
// Callers put the index they reduce over or scale by per row of the tile
// (vocabulary entries) on m and the index with per-lane constants (tokens) on n.
// With Across the instruction gets its operands exchanged: lane l holds row m = l % 16
// and, in register r, column n = 4*(l/16) + r, four consecutive values of an output row.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace spo {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;      // contraction elements per stage
constexpr int kStages = 2;   // LDS stages
constexpr int kRowBytes = kBK * 2;
constexpr int kChunks = kRowBytes / 16;
constexpr int kBlockK = kBK;  // contraction elements per block of a k-blocked operand: one stage

// chunk swizzle of a tile row (3 bits): a bijection on 0..7 both over rows 0..7
// and over the rows of equal parity in 0..15, i.e. 16 consecutive rows reading
// the same chunk touch 16 different 16-byte slots of any 256-byte window, and 8
// consecutive rows 8 different slots of any 128-byte window
__device__ __forceinline__ int swz(int row) {
    return ((row >> 1) & 3) | (((row ^ (row >> 3)) & 1) << 2);
}

// MI is the edge of the MFMA block: 16 for v_mfma_f32_16x16x32_bf16, the instruction the
// main loop is written for.  (The same tile on v_mfma_f32_32x32x16_bf16, with two
// phase-shifted groups of wavefronts, was 4-6 % slower on the same chip.)
template <int BM_, int BN_, int WGM_, int WGN_, int MI_ = 16>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, MI = MI_;
    static_assert(MI == 16, "the main loop issues 16x16x32 MFMAs");
    static constexpr int NWAVE = WGM * WGN, NT = NWAVE * kWave;
    static constexpr int WM = BM / WGM, WN = BN / WGN;     // wave tile
    static constexpr int FM = WM / MI, FN = WN / MI;       // MI x MI blocks per wave
    static constexpr int KK = kBK / (512 / MI);            // MFMA k-slices per stage (16 or 32 elements deep)
    static constexpr int ACC_R = MI * MI / kWave;          // accumulator registers per block and lane
    static constexpr int A_BYTES = BM * kRowBytes, B_BYTES = BN * kRowBytes;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int LDS_BYTES = kStages * STAGE_BYTES;
    static constexpr int A_LOADS = BM * kChunks / NT, B_LOADS = BN * kChunks / NT;
    static constexpr int STAGE_LOADS = A_LOADS + B_LOADS;  // DMA instructions per thread and stage
    static_assert(BM * kChunks % NT == 0 && BN * kChunks % NT == 0, "tile rows must split evenly over the threads");
    static_assert((NT / kChunks) % 16 == 0, "swizzle must be the same for every load of a thread");
    static_assert(WM % MI == 0 && WN % MI == 0, "wave tile is made of MI x MI blocks");

    typedef float AccBlock __attribute__((ext_vector_type(ACC_R)));
    typedef AccBlock Acc[FM][FN];

    __device__ static __forceinline__ int wave_id() {
        return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
    }
    __device__ static __forceinline__ int wave_m0() { return (wave_id() % WGM) * WM; }
    __device__ static __forceinline__ int wave_n0() { return (wave_id() / WGM) * WN; }
    // Accumulator layout of a 16x16 block: lane l holds column l % 16 and, in register r, row
    // 4*(l/16) + r: a lane owns a run of four consecutive rows, a quad of lanes four consecutive
    // columns, and the four groups of 16 lanes hold different rows of the same columns.
    // tile row of accumulator register r of block fm
    __device__ static __forceinline__ int acc_row(int fm, int r) {
        return wave_m0() + fm * MI + 4 * ((threadIdx.x & 63) / MI) + r;
    }
    // tile column of block fn
    __device__ static __forceinline__ int acc_col(int fn) {
        return wave_n0() + fn * MI + (threadIdx.x & (MI - 1));
    }
    static constexpr int GROUPS = kWave / MI;  // lane groups that hold different rows of the same column
    // Row d of the wavefront's part of the tile (0 <= d < WM) lives in block fm, register r of
    // the lanes of group g.
    __device__ static __forceinline__ void locate(int d, int &fm, int &r, int &g) {
        fm = d / MI;
        g = (d >> 2) & (GROUPS - 1);
        r = d & 3;
    }

    // One operand of a tile as it lies in memory.
    // Rows along k (Cols = false): element k of row r at base + r * ld + k * 2 bytes, `count` rows in all (rows of the
    // tile beyond them are fetched from the last one; the caller masks them).  It may be stored in blocks of
    // kBlockK contraction elements: element k of row r at base + (k / kBlockK) * blk + r * ld + (k % kBlockK) * 2
    // bytes (blk = 0: plain row-major).  With ld = 128 bytes a stage of a tile is then one contiguous
    // 32 KiB piece instead of 256 lines a whole matrix row apart: the 256 rows stay within a few
    // pages of the address translation and spread evenly over the memory channels.
    // Columns along k (Cols = true): element k of column c at base + k * ld + c * 2 bytes; `count` is the readable
    // length of a row (a multiple of 8 elements; pieces past it are fetched from the last readable one, the caller
    // masks those columns), blk != 0: the columns are stored in blocks of kBlockK, column c at
    // base + (c / kBlockK) * blk + k * ld + (c % kBlockK) * 2 bytes, all columns of the tile readable.
    // first: the tile's first row / column, a whole number of blocks where blk != 0 and Cols.
    // Elements of the last stage past the contraction's end are fetched like the others - the other operand is zero
    // there - unless the second operand ends inside it (see mainloop).
    struct Operand {
        const char *base;
        int64_t ld, first, count, blk;
    };

    // the same in every lane; say so, the DMA wants it in SGPRs
    __device__ static __forceinline__ const char *uniform(const char *p) {
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32));
        return reinterpret_cast<const char *>((static_cast<uint64_t>(hi) << 32) | lo);
    }
    __device__ static __forceinline__ uint32_t lds_address(const char *p) {
        return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char *)p));
    }

    // The DMA is issued from inline assembly.  Issued through the compiler it would
    // make every later LDS read wait for ALL outstanding DMA (the wait-count pass
    // cannot tell the stages apart); here every vmcnt wait for these loads is
    // explicit instead.  M0 holds the LDS base of the 64 lanes x 16 bytes written.  (M0 cannot
    // be named as a clobber: the compiler reserves the register and keeps no value of its
    // own in it across an asm statement; these kernels use nothing else that goes through M0.)
    __device__ static __forceinline__ void dma(const char *base, uint32_t off, uint32_t lds_addr) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds_addr), "v"(off), "s"(base)
                     : "memory");
    }

    // The same where `go` (wave-uniform) is not zero.  The branch is inside the assembly: seen by the compiler, a way round the
    // requests would split the step they are spread over, and its registers would spill.
    // (`go` comes in a vector register: the compiler may hold it in one although it is the same in every lane.)
    __device__ static __forceinline__ void dma_if(int go, const char *base, uint32_t off, uint32_t lds_addr) {
        int t;
        asm volatile("v_readfirstlane_b32 %0, %4\n\ts_cmp_eq_u32 %0, 0\n\ts_cbranch_scc1 1f\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %3\n1:"
                     : "=&s"(t)
                     : "s"(lds_addr), "v"(off), "s"(base), "v"(go)
                     : "memory", "scc");
    }
    // Waits until at most N vector memory operations are outstanding where `some` is not zero, otherwise for all, and for
    // all LDS reads.
    template <int N>
    __device__ static __forceinline__ void wait_for(int some) {
        int t;
        asm volatile("v_readfirstlane_b32 %0, %1\n\ts_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 1f\n\ts_waitcnt vmcnt(0)\n1:\n\t"
                     "s_waitcnt vmcnt(%2) lgkmcnt(0)"
                     : "=&s"(t)
                     : "v"(some), "n"(N)
                     : "memory", "scc");
    }

    // LDS stage of an operand whose columns run along k: kBK rows of EDGE elements, chunk c of row r at position
    // c ^ ksw(r).  ksw moves bits 1-2 of the position with the row inside a group of four and the bits from 3 on with
    // the group of eight rows, so the 8-byte pieces a transposing read collects (4 rows x 32 bytes per group of 16
    // lanes, the groups 8 rows apart) fall on distinct banks, and so do the linear DMA writes.
    template <int EDGE>
    __device__ static __forceinline__ int ksw(int r) { return ((r & 3) << 1) | (((r >> 3) & (EDGE == 256 ? 3 : 1)) << 3); }

    // The thread index through an empty asm, so that the compiler cannot trace what is derived from it: hoisted out of a
    // loop over tiles these few cheap values would sit in registers across the main loop, where every register counts.
    __device__ static __forceinline__ int fresh_thread() {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        return tid;
    }

    // One operand's side of the main loop: EDGE rows (columns) of the tile, F blocks of 16 of them per wavefront.
    // Global -> LDS: slot q = i*NT + tid of a stage <-> (row q / chunks per row, position q % chunks per row).
    // LDS -> fragments: READS reads per k-slice of 32.
    template <int EDGE, int F, bool Cols>
    struct Side {
        static_assert(EDGE == 256 || EDGE == 128, "swizzle of columns along k");
        static constexpr int CHUNKS = Cols ? EDGE * 2 / 16 : kChunks;  // 16-byte chunks per row of a stage
        static constexpr int ROWB = CHUNKS * 16;
        static constexpr int LOADS = EDGE * kChunks / NT;              // DMA instructions per thread and stage
        static constexpr int READS = Cols ? 2 * F : F;
        typedef short v4s __attribute__((ext_vector_type(4)));
        typedef short v8s __attribute__((ext_vector_type(8)));
        const char *base;            // first row / column of the panel (wave-uniform)
        int64_t step;                // bytes from one stage to the next
        uint32_t off[LOADS];         // this lane's byte offsets inside the panel
        uint32_t lds_wave;           // LDS address of this wave's 1 KiB slice of stage 0
        uint32_t src[Cols ? F : KK];  // Cols: LDS address of this lane's piece of each block, slice 0, of the stage in use;
                                     // otherwise its offset inside 16 rows, per k-slice
        const char *rows;            // the wavefront's rows in stage 0
        bf16x8_t whole[Cols ? 1 : 2][Cols ? 1 : F];
        v4s half[Cols ? 2 : 1][Cols ? F : 1][2];  // two halves of the 8 contraction values

        // region: where this operand lies inside a stage; row0: the wavefront's first row / column of the tile
        // tid: fresh_thread()
        __device__ __forceinline__ Side(const Operand &o, char *lds, int region, int row0, int tid) {
            const int lane = tid & 63;
            lds_wave = lds_address(lds) + region + wave_id() * (kWave * 16);
            aim(o, tid);
            if constexpr (Cols) {
                // within 16 lanes a transposing read gives lane i element i%4 of the source lanes i/4 + 4e: source lane s
                // points at row k0 + s/4, columns 4*(s%4).. of a 16-column block, so lane i ends up with rows
                // k0..k0+3 of column i; the lane group sets k0 = 8*(l/16) and a second read 4 rows down
                // completes the 8 values per lane that the MFMA wants
#pragma unroll
                for (int b = 0; b < F; ++b) {
                    const int row = 8 * (lane >> 4) + ((lane & 15) >> 2), col = row0 + b * MI + 4 * (lane & 3);
                    src[b] = lds_address(lds) + region + row * ROWB + (((col >> 3) ^ ksw<EDGE>(row)) << 4) + ((col >> 2) & 1) * 8;
                }
                static_assert((32 + 4) * ROWB < 65536, "slice and half offsets fit the read's offset field");
            } else {
                // lane reads row (l%16) of a 16-row block, chunk 4*kk + l/16
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) src[kk] = (lane & 15) * kRowBytes + (((4 * kk + (lane >> 4)) ^ swz(lane & 15)) * 16);
                rows = lds + region + row0 * kRowBytes;
            }
        }
        // where the transfers of the tile at o.first come from
        __device__ __forceinline__ void aim(const Operand &o, int tid) {
            // 32-bit byte offsets from the tile's first row (a tile spans < 4 GiB)
            const uint32_t ld = static_cast<uint32_t>(o.ld);
            if constexpr (Cols) {
                base = uniform(o.blk ? o.base + o.first / kBlockK * o.blk : o.base + o.first * 2);
                step = kBK * o.ld;
                const int c_last = (o.count - o.first >= EDGE ? CHUNKS : static_cast<int>(o.count - o.first) / 8) - 1;
#pragma unroll
                for (int i = 0; i < LOADS; ++i) {
                    const int q = i * NT + tid, row = q / CHUNKS, c = (q % CHUNKS) ^ ksw<EDGE>(row);
                    constexpr int cpb = kBlockK / 8;  // 16-byte chunks per block of columns
                    off[i] = o.blk ? static_cast<uint32_t>((c / cpb) * o.blk + row * o.ld + (c % cpb) * 16)
                                   : static_cast<uint32_t>(row) * ld + static_cast<uint32_t>((c < c_last ? c : c_last) * 16);
                }
            } else {
                base = uniform(o.base + o.first * o.ld);
                step = o.blk ? o.blk : kRowBytes;
                const int ld_row = tid / kChunks;
                const uint32_t chunk16 = static_cast<uint32_t>(((tid % kChunks) ^ swz(ld_row & 15)) * 16);
                const uint32_t r_last = static_cast<uint32_t>(o.count - o.first >= EDGE ? EDGE - 1 : o.count - 1 - o.first);
#pragma unroll
                for (int i = 0; i < LOADS; ++i) {
                    const uint32_t r = static_cast<uint32_t>(i * (NT / kChunks) + ld_row);
                    off[i] = (r < r_last ? r : r_last) * ld + chunk16;
                }
            }
        }
        // DMA instruction i of this thread's share of stage kt, into LDS stage buf
        __device__ __forceinline__ void one(int kt, int buf, int i) const {
            dma(base + kt * step, off[i], lds_wave + buf * STAGE_BYTES + i * (NT * 16));
        }
        __device__ __forceinline__ void one_if(int go, int kt, int buf, int i) const {
            dma_if(go, base + kt * step, off[i], lds_wave + buf * STAGE_BYTES + i * (NT * 16));
        }
        // A last stage of `end` elements (rows along k: a multiple of 8): does piece i of this thread lie past them?
        __device__ static __forceinline__ bool past(int i, int tid, int end) {
            return (Cols ? (i * NT + tid) / CHUNKS : ((tid % kChunks) ^ swz(tid / kChunks & 15)) * 8) >= end;
        }
        // from the next stage on, pieces past its end are fetched from its first one
        __device__ __forceinline__ void clamp(int end) {
            const int tid = fresh_thread();
#pragma unroll
            for (int i = 0; i < LOADS; ++i) off[i] = past(i, tid, end) ? 0u : off[i];
        }
        // ... and cleared in LDS stage buf.  This thread's transfers have landed.
        __device__ __forceinline__ void clear(int buf, int end) const {
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
            const int tid = fresh_thread();
            const uint32_t at = lds_wave + buf * STAGE_BYTES + (tid & 63) * 16;
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                if (past(i, tid, end)) *(u4 __attribute__((address_space(3))) *)(uintptr_t)(at + i * (NT * 16)) = u4{0, 0, 0, 0};
        }
        // read r (0 .. READS-1) of k-slice kk into register set buf: of stage kt, or (Cols) of the stage that src points at
        __device__ __forceinline__ void read(int kt, int kk, int buf, int r) {
            if constexpr (Cols)
                half[buf][r >> 1][r & 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (v4s __attribute__((address_space(3))) *)(uintptr_t)(src[r >> 1] + (32 * kk + 4 * (r & 1)) * ROWB));
            else
                whole[buf][r] = *reinterpret_cast<const bf16x8_t *>(rows + (kt % kStages) * STAGE_BYTES + r * (16 * kRowBytes) + src[kk]);
        }
        __device__ __forceinline__ void turn(int to_other) {  // src to the other stage
            if constexpr (Cols)
#pragma unroll
                for (int b = 0; b < F; ++b) src[b] += to_other;
        }
        __device__ __forceinline__ bf16x8_t frag(int buf, int f) const {
            if constexpr (Cols) {
                const v8s v = __builtin_shufflevector(half[buf][f][0], half[buf][f][1], 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(bf16x8_t, v);
            } else {
                return whole[buf][f];
            }
        }
    };

    __device__ static __forceinline__ void fence_barrier() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    }

    // Column of the j-th block of a slice: along a row of blocks and back along the next, so that every instruction
    // shares an operand with the one before.  What changes hands costs power, which is what bounds large batches
    // (register-only loops 1985 -> 1995 TFLOP/s; 17043 tokens at 4096 x 151936 62.05 -> 61.84 ms, 46511 with a mask
    // 108.07 -> 107.57, of which two runs of one side differ by half).
    __device__ static constexpr int snake(int j) { return (j / FN) & 1 ? FN - 1 - j % FN : j % FN; }

    template <bool Across>
    __device__ static __forceinline__ AccBlock mfma(const bf16x8_t &a, const bf16x8_t &b, const AccBlock &c) {
        return Across ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }

    // The main loop over one tile or a run of tiles.  lds: LDS_BYTES bytes, 16-byte aligned.  All threads of the
    // block must call everything here together.
    // ACols, BCols: how the operands lie (see Operand); Clamp: B's last stage has `end` elements (0: all).
    //
    // Schedule of a step: both wavefronts of a SIMD multiply at the same time and each hides its
    // own fragment reads between its MFMAs (one read per two MFMAs, or per one where there are more, into a second
    // register set for the next k-slice of 32); whenever one of them waits, at the barrier or for its
    // operands, the other keeps the MFMA pipe fed.  One barrier per step, between the two
    // k-slices: before it a wavefront has all its reads of stage s in registers and its share of
    // stage s+1 landed; after it stage s+1 may be read and the buffer of stage s is refilled with
    // stage s+2 (its DMA instructions spread over the MFMAs).
    template <bool ACols, bool BCols, bool Across = false, bool Clamp = false>
    struct Loop {  // (a run of tiles is not clamped)
        Side<BM, FM, ACols> a;
        Side<BN, FN, BCols> b;
        static constexpr int NR = Side<BM, FM, ACols>::READS + Side<BN, FN, BCols>::READS, READ_EVERY = NR * 2 <= FM * FN ? 2 : 1;
        static constexpr int DMA_EVERY = FM * FN / STAGE_LOADS, NEXT_EVERY = FM * FN / (2 * STAGE_LOADS);
        static_assert(KK == 2 && kStages == 2, "two k-slices per stage, two stages");
        static_assert(NR * READ_EVERY <= FM * FN && DMA_EVERY >= 2 && NEXT_EVERY >= 1, "reads and DMA fit between the MFMAs of a slice");

        // (what both sides derive from one fresh thread index is formed once; a run has no registers to keep it in)
        __device__ __forceinline__ Loop(const Operand &oa, const Operand &ob, char *lds, int tid) : Loop(oa, ob, lds, tid, tid) {}
        __device__ __forceinline__ Loop(const Operand &oa, const Operand &ob, char *lds, int tid_a, int tid_b)
            : a(oa, lds, 0, wave_m0(), tid_a), b(ob, lds, A_BYTES, wave_n0(), tid_b) {}

        __device__ __forceinline__ void feed(int kt, int i) {
            if (i < A_LOADS) a.one(kt, kt % kStages, i);
            else b.one(kt, kt % kStages, i - A_LOADS);
        }
        __device__ __forceinline__ void feed_if(int go, int kt, int i) {
            if (i < A_LOADS) a.one_if(go, kt, kt % kStages, i);
            else b.one_if(go, kt, kt % kStages, i - A_LOADS);
        }
        // What B has past its end is not to be read, and what is fetched in its place must not count: zeros of A times an
        // infinite weight are NaN (a head that bans a token).  Before the requests of the last stage, and before the barrier that
        // opens it.
        __device__ __forceinline__ void clamp_if(bool last, int end) {
            if (Clamp && last && end) b.clamp(end);
        }
        __device__ __forceinline__ void clear_if(int buf, int end) {
            if (!Clamp || !end) return;
            b.clear(buf, end);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        // Requests the first stages of the tile.  Every wavefront is done with the previous contents of lds.
        __device__ __forceinline__ void start(int KT, int end = 0) {
            clamp_if(KT == 1, end);
#pragma unroll
            for (int i = 0; i < STAGE_LOADS; ++i) feed(0, i);
            clamp_if(KT == 2, end);
            if (KT > 1)
#pragma unroll
                for (int i = 0; i < STAGE_LOADS; ++i) feed(1, i);
        }
        // acc += sum over k < kBK * KT of A(m, k) B(n, k) for the tile whose first stages are on their way.
        // Younger: vector memory operations that the wavefront has surely issued since they were requested, unless
        // `fresh` (none); they may be outstanding while the stages are waited for (loads and stores leave in order).
        // more: there is a next tile (next() gives some tile in any case), whose first stages are requested in the last half step, when both LDS stages and one set
        // of fragments are free; next(true_type) is its loop, which is made anew when its turn comes (kept across the
        // work between two tiles, its addresses would not fit the registers).
        template <int Younger, bool Run, typename Next>
        __device__ __forceinline__ void run(int KT, Acc &acc, bool fresh, bool more, Next next, int end = 0) {
            auto read = [&](int kt, int kk, int buf, int r) {
                if (r < a.READS) a.read(kt, kk, buf, r);
                else b.read(kt, kk, buf, r - a.READS);
            };
            // loads return in order: stage 0 has landed
            if (Run) {  // (of a tile that follows another; both stages of the first one)
                const int after = fresh ? 0 : 1;
                if (KT > 1) wait_for<STAGE_LOADS + Younger>(after);
                else wait_for<Younger>(after);
            } else if (KT > 1) {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STAGE_LOADS) : "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                clear_if(0, end);
            }
            fence_barrier();
#pragma unroll
            for (int r = 0; r < NR; ++r) read(0, 0, 0, r);
            int go = 0, go_on = 0;       // there is a next tile, it has a second stage
            int to_other = STAGE_BYTES;  // distance to the stage that column addresses do not point at
            // One step; MORE: a stage kt+1 exists, FEED: a stage kt+2 exists, NEXT: the next tile's first stages are
            // requested.  Compile-time flags: a
            // branch around every read and every DMA instruction costs the wavefront more issue time
            // than the instruction it guards, so the last two steps are peeled off the loop instead.
            auto step = [&](int kt, auto more_t, auto feed_t, auto next_t) {
                constexpr bool MORE = decltype(more_t)::value, FEED = decltype(feed_t)::value, NEXT = decltype(next_t)::value;
                // ---- slice 0 of stage kt, reading its slice 1 between the MFMAs
#pragma unroll
                for (int j = 0; j < FM * FN; ++j) {
                    const int fm = j / FN, fn = snake(j);
                    if (j % READ_EVERY == 0 && j / READ_EVERY < NR) {
                        read(kt, 1, 1, j / READ_EVERY);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    acc[fm][fn] = mfma<Across>(a.frag(0, fm), b.frag(0, fn), acc[fm][fn]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (Run && Younger > 0) wait_for<Younger>(kt == 0 && !fresh ? 1 : 0);
                else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                if (MORE && !FEED) clear_if((kt + 1) % kStages, end);
                fence_barrier();
                a.turn(to_other);
                b.turn(to_other);
                to_other = -to_other;
                // ---- slice 1, reading slice 0 of stage kt+1 and feeding the DMA of stage kt+2
                auto following = next(std::integral_constant<bool, NEXT>{});
#pragma unroll
                for (int j = 0; j < FM * FN; ++j) {
                    const int fm = j / FN, fn = snake(j);
                    if (j % READ_EVERY == 0 && j / READ_EVERY < NR) {
                        if (MORE) read(kt + 1, 0, 0, j / READ_EVERY);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (FEED && j % DMA_EVERY == 1 && j / DMA_EVERY < STAGE_LOADS) {
                        feed(kt + 2, j / DMA_EVERY);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (NEXT) if (j % NEXT_EVERY == 0) {
                        const int i = j / NEXT_EVERY;
                        if (i < STAGE_LOADS) following.feed_if(go, 0, i);
                        else following.feed_if(go_on, 1, i - STAGE_LOADS);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    acc[fm][fn] = mfma<Across>(a.frag(1, fm), b.frag(1, fn), acc[fm][fn]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            using std::true_type, std::false_type;
            go = more ? 1 : 0;
            go_on = more && KT > 1 ? 1 : 0;
            int kt = 0;
            if constexpr (Clamp) {  // the step that requests the last stage apart: a condition in the loop spilled 36 registers
                for (; kt + 3 < KT; ++kt) step(kt, true_type{}, true_type{}, false_type{});
                if (kt + 2 < KT) {
                    clamp_if(true, end);
                    step(kt++, true_type{}, true_type{}, false_type{});
                }
            } else {
                for (; kt + 2 < KT; ++kt) step(kt, true_type{}, true_type{}, false_type{});
            }
            if (kt + 1 < KT) step(kt++, true_type{}, false_type{}, false_type{});
            step(kt, false_type{}, false_type{}, std::integral_constant<bool, Run>{});
        }
    };

    // acc += sum over k < kBK * KT of A(m, k) B(n, k) for ONE tile.  end (Clamp): B's last stage has that many elements, a
    // multiple of 8 where its rows are along k; past them A is zero.  0: all kBK may be read.
    template <bool ACols, bool BCols, bool Across = false, bool Clamp = false>
    __device__ static __forceinline__ void mainloop(const Operand &oa, const Operand &ob, int KT, char *lds, Acc &acc, int end = 0) {
        Loop<ACols, BCols, Across, Clamp> loop(oa, ob, lds, fresh_thread());
        __syncthreads();  // every wave is done with the previous contents of lds
        loop.start(KT, end);
        loop.template run<0, false>(KT, acc, true, false, [](auto) { return 0; }, end);
    }

    __device__ static __forceinline__ void zero(Acc &acc) {
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
#pragma unroll
                for (int r = 0; r < ACC_R; ++r) acc[fm][fn][r] = 0.0f;
    }
};

// Maps a linear workgroup id to a tile of an nM x nN tile grid so that the 32
// workgroups that run together on one XCD (ids equal mod 8 are dispatched to the
// same XCD and share its L2) form a 4 x 8 patch: 12 operand panels feed 32 tiles.
// Patches are walked along N first: with N the short dimension (the 16 tiles of a
// hidden size of 4096 are two patches) the eight XCDs then work on few M panels and
// all N panels at the same time, so an M panel (rows of the logit gradients, the
// large operand of both backward contractions) is fetched from memory once instead
// of once per N patch (measured against walking M first: dHidden -1.6 %, dW -2.4 %).
// Every id is a tile but for the last few: a patch at the grid's edge takes as many ids as it has
// tiles, and what does not fill the chip is divided by XCDs.  (A workgroup without a tile is not free: it
// waits for 128 KB of LDS.  2048 of them for 16 parts of tiles: 45 us.)
struct TileOrder {
    static constexpr int kPatchM = 4, kPatchN = 8, kRun = kPatchM * kPatchN, kXcds = 8;
    int64_t nM, nN;
    __host__ __device__ TileOrder(int64_t nm, int64_t nn) : nM(nm), nN(nn) {}
    __host__ __device__ int64_t tiles() const { return nM * nN; }
    // number of ids for `total` items in order
    __host__ __device__ static int64_t blocks(int64_t total) {
        return total / (kRun * kXcds) * (kRun * kXcds) + (total % (kRun * kXcds) + kXcds - 1) / kXcds * kXcds;
    }
    // item of workgroup bid: runs of 32 to each XCD in turn, the rest in eight equal runs; false past the last
    __device__ static __forceinline__ bool item(uint32_t bid, uint32_t total, uint32_t &i) {
        constexpr uint32_t round = kRun * kXcds;
        const uint32_t whole = total / round * round;
        uint32_t j = bid, run = kRun, base = bid / round * round;
        if (bid >= whole) {
            run = (total - whole + kXcds - 1) / kXcds;
            base = whole;
        }
        j -= base;
        if (j / kXcds >= run) return false;
        i = base + j % kXcds * run + j / kXcds;
        return i < total;
    }
    // the i-th tile: bands of four tile rows, patch after patch along N
    __device__ __forceinline__ void at(uint32_t i, int64_t &tm, int64_t &tn) const {
        const uint32_t m = static_cast<uint32_t>(nM), n = static_cast<uint32_t>(nN);
        const uint32_t band = i / (kPatchM * n), j = i - band * kPatchM * n;
        const uint32_t h = m - kPatchM * band < kPatchM ? m - kPatchM * band : kPatchM;
        const uint32_t g = j / (kPatchN * h), k = j - g * kPatchN * h;
        const uint32_t w = n - kPatchN * g < kPatchN ? n - kPatchN * g : kPatchN;
        tm = band * kPatchM + k / w;
        tn = g * kPatchN + k % w;
    }
};

}  // namespace spo
