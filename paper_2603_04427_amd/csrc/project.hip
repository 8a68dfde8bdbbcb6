// Thin projections for factored keys (Sec. 2.3, Eq. 6-7): Y = X W for one
// projection of a layer, written head-major for the attention kernels.
//
// After a pretrained key projection is factored per KV head (W_K ~= A B) and B
// is absorbed into the query projection (W_Q' = W_Q B^T), the layer computes
// r-wide queries q' = x W_Q' and keys k' = x W_K' = x A for every token, and
// its full-width values v = x W_V. Each is a dense product of the token rows
// X [tokens, d_model] with a weight matrix whose columns are grouped by head.
// This kernel computes one such product on the bf16 matrix cores with fp32
// accumulation and stores the result straight into the [batch, head, token,
// width] layout that tk_attn_prefill and tk_cache_append read, so no separate
// transpose pass follows.
//
// The weight is passed transposed, Wt [n_heads * width, d_model] (one row per
// output column), so both operands of the product are contiguous along
// d_model, which must be a multiple of 32 (one k-tile). The tile computes C^T = Wt X^T: a lane of each accumulator
// then holds four consecutive output columns of one token, which become one
// 8-byte store into the head-major output row.
#include "tk_device.hpp"
#include "tk_internal.hpp"

#include <type_traits>

namespace tk {

namespace {

constexpr int kXcdCount = kXcds;
constexpr int kPBK = 32;   // d_model per k-tile: 4 chunks of 8 bf16 per row
constexpr int kStages = 3; // k-tiles in LDS: the one multiplied and two in flight

// A workgroup tile of BN output columns (weight rows) x BM tokens. Its waves are
// laid out (BN / 64) x 2: each owns 64 columns x BM / 2 tokens.
template <int BN, int BM>
struct ProjTile {
    static constexpr int kWaves = (BN / 64) * 2;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kMB = BM / 64;                         // 32-token blocks per wave
    static constexpr int kWCopies = BN * kPBK / 8 / kThreads;  // copies per lane and k-tile
    static constexpr int kXCopies = BM * kPBK / 8 / kThreads;
    static constexpr int kCopies = kWCopies + kXCopies;        // a lane's copies in flight per k-tile
    static_assert(kWCopies * kThreads * 8 == BN * kPBK && kXCopies * kThreads * 8 == BM * kPBK, "tiling");
    uint16_t w[kStages][BN * kPBK];  // weight rows of the tile (swizzled 16-byte chunks)
    uint16_t x[kStages][BM * kPBK];  // token rows of the tile (same swizzle)
};

// Chunk kc (0..3) of tile row r sits in slot 4 r + (kc ^ ((r / 4) % 4)). Rows are
// 64 bytes, so four rows share one 256-byte line of the 64 LDS banks; the
// rotation gives the same chunk of the rows r, r + 4, r + 8, r + 12 four
// different 16-byte bank groups, so the 16 consecutive rows one quarter-wave
// reads cover all 64 banks once. The map is its own inverse: slot 4 r + q
// holds chunk q ^ ((r / 4) % 4).
__device__ __forceinline__ int sw(int r, int kc) { return r * kPBK + ((kc ^ ((r >> 2) & 3)) << 3); }

template <int N>
__device__ __forceinline__ void wait_copies(bool next_in_flight) {
    if (next_in_flight)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
    else
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Each wave multiplies a 64-column x BM / 2-token block. Tiles come from HBM by
// global->LDS copies (no staging registers), issued two k-tiles ahead into a
// three-stage ring. The 256 x 256 tiles run 16x16x32 products in a ping-pong
// between the two waves of each SIMD; the smaller ones run 32x32x16 products,
// each wave reading the next 16-wide k-step's operands during the current one's
// products.
//
// With KG > 1, KG groups of those waves take the k-tiles of one output tile in
// turn (group g the k-tiles g, g + KG, ...), each through a ring of its own, and
// group 0 adds up the partial tiles in LDS in group order: for calls whose tiles
// are too few to fill the CUs with waves.
template <int BN, int KG>
constexpr int proj_threads() { return 64 * (BN / 64) * 2 * KG; }

template <int BN, int BM, int KG>
union ProjSmem {
    ProjTile<BN, BM> tile[KG];
    float4 part[KG - 1 + (KG == 1)][ProjTile<BN, BM>::kWaves][KG == 1 ? 1 : 8 * (BM / 64)][64];  // accumulators as they lie
};

template <int BN, int BM, int KG>
__global__ __launch_bounds__((proj_threads<BN, KG>()), 1) void project_kernel(const ProjectParams p) {
    using T = ProjTile<BN, BM>;
    constexpr int kPThreads = T::kThreads, kWCopies = T::kWCopies, kXCopies = T::kXCopies;
    constexpr int kPBN = BN, kPBM = BM;
    static_assert(KG == 1 || BM < 256, "the ping-pong tiles take all k-tiles");
    __shared__ ProjSmem<BN, BM, KG> smem;
    const int lane = threadIdx.x & 63;
    const int all_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = KG == 1 ? all_wave : all_wave % T::kWaves;  // wave of its k group
    const int kgrp = KG == 1 ? 0 : all_wave / T::kWaves;
    const int tid = wave * 64 + lane;
    T& sm = smem.tile[kgrp];
    const int wn = wave >> 1, wm = wave & 1;  // (BN / 64) x 2 waves over the tile's columns x tokens
    // XCD-aware order: workgroups are dealt to the 8 XCDs round-robin; each XCD
    // takes a contiguous range of tiles, column tiles fastest, so the column
    // tiles of one token tile run on one XCD and share its rows through its L2
    const int per_xcd = (p.tiles + kXcdCount - 1) / kXcdCount;
    const int logical = (int)(blockIdx.x % kXcdCount) * per_xcd + (int)(blockIdx.x / kXcdCount);
    if (logical >= p.tiles) return;
    const int n_tiles = (p.N + kPBN - 1) / kPBN;
    const int n_base = (logical % n_tiles) * kPBN, m_base = (logical / n_tiles) * kPBM;

    // Copy i of this lane fills LDS slot i * 256 + tid of the tile: row slot / 4,
    // chunk (slot % 4) ^ ((row / 4) % 4) of that row in the matrix. Rows past the
    // matrix re-read its last row (finite values whose outputs are not stored).
    const int wlast = (p.N - n_base < kPBN ? p.N - n_base : kPBN) - 1;
    const int xlast = (p.M - m_base < kPBM ? p.M - m_base : kPBM) - 1;
    uint32_t woff[kWCopies], xoff[kXCopies];
#pragma unroll
    for (int i = 0; i < kWCopies; ++i) {
        const int slot = i * kPThreads + tid, r = slot >> 2, kc = (slot & 3) ^ ((r >> 2) & 3);
        woff[i] = (uint32_t)(((r < wlast ? r : wlast) * p.K + kc * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < kXCopies; ++i) {
        const int slot = i * kPThreads + tid, r = slot >> 2, kc = (slot & 3) ^ ((r >> 2) & 3);
        xoff[i] = (uint32_t)(((r < xlast ? r : xlast) * p.K + kc * 8) * 2);
    }
    const char* wg = (const char*)((const uint16_t*)p.wt + (size_t)n_base * p.K);
    const char* xg = (const char*)((const uint16_t*)p.x + (size_t)m_base * p.K);
    auto issue = [&](int kt, int stage) {
        const char* wk = wg + (size_t)kt * kPBK * 2;
        const char* xk = xg + (size_t)kt * kPBK * 2;
#pragma unroll
        for (int i = 0; i < kWCopies; ++i) copy16_to_lds(wk, woff[i], sm.w[stage] + (i * kPThreads + wave * 64) * 8);
#pragma unroll
        for (int i = 0; i < kXCopies; ++i) copy16_to_lds(xk, xoff[i], sm.x[stage] + (i * kPThreads + wave * 64) * 8);
    };

    if constexpr (BM == 256) {
        // ---- 256 x 256 tiles: ping-pong over the two waves of each SIMD ----
        // The eight waves form two groups of four, one wave of each on every SIMD;
        // the second group runs one barrier behind the first. A wave reads a whole
        // k-tile's operands while the other wave of its SIMD runs its products, then
        // runs its own products (32 of 16x16x32) while the other reads: the two
        // phases alternate at every barrier. Each lane's 16-byte operand read is row
        // r16 of a 16-row block at chunk q4, the whole 32-wide k-tile over the four
        // lane groups, and an accumulator lane ends with four consecutive output
        // columns of one token. Both groups pass 2 nk + 2 barriers: the late group's
        // extra one comes first, the early group's last.
        constexpr int kNB = BM / 32;
        const int r16 = lane & 15, q4 = lane >> 4;
        f32x4 acc[4][kNB];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < kNB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
        const int nk = p.K / kPBK;
        issue(0, 0);
        if (nk > 1) issue(1, 1);
        wait_copies<T::kCopies>(nk > 1);
        __syncthreads();
        const bool late = wave >= 4;
        if (late) {
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 a[4], b[kNB];
        int stage = 0;
        for (int kt = 0; kt < nk; ++kt) {
            // the stage k-tile kt + 2 goes to held k-tile kt - 1, which both groups
            // have read before the barrier that opened this wave's read phase
            const bool ahead = kt + 2 < nk;
            if (ahead) issue(kt + 2, stage == 0 ? 2 : stage - 1);
            const uint16_t* ws = sm.w[stage];
            const uint16_t* xs = sm.x[stage];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = *(const bf16x8*)(ws + sw(wn * 64 + i * 16 + r16, q4));
#pragma unroll
            for (int j = 0; j < kNB; ++j) b[j] = *(const bf16x8*)(xs + sw(wm * (BM / 2) + j * 16 + r16, q4));
            wait_copies<T::kCopies>(ahead);  // k-tile kt + 1 has landed before the next barrier
            // the schedule barriers keep the reads and products in their phases
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < kNB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            stage = stage == kStages - 1 ? 0 : stage + 1;
        }
        if (!late) {
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < kNB; ++j) {
            const int m = m_base + wm * (BM / 2) + j * 16 + r16;
            if (m >= p.M) continue;
            const int bb = m / p.S, s = m - bb * p.S;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = n_base + wn * 64 + i * 16 + 4 * q4;
                if (n >= p.N) continue;
                const int h = n / p.width, w = n - h * p.width;
                uint2 v;
                v.x = pack_bf16(acc[i][j][0], acc[i][j][1]);
                v.y = pack_bf16(acc[i][j][2], acc[i][j][3]);
                *(uint2*)((uint16_t*)p.y + (((size_t)bb * p.heads + h) * p.S + s) * p.width + w) = v;
            }
        }
    } else {
        // ---- smaller tiles: 32x32x16 products, software-pipelined over k-steps ----
        const int col = lane & 31, half = lane >> 5;
        f32x16 acc[2][T::kMB];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < T::kMB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

        const int nk = p.K / kPBK;
        const int nsteps = (nk + KG - 1) / KG;  // every group passes the same barriers; only its last step can be missing
        auto has = [&](int t) { return t * KG + kgrp < nk; };
        // operand reads of k-step ks of the k-tile in `st`, and the products of one k-step
        auto read_ops = [&](int st, int ks, bf16x8 (&a)[2], bf16x8 (&b)[T::kMB]) {
            const uint16_t* ws = sm.w[st];
            const uint16_t* xs = sm.x[st];
            const int kc = 2 * ks + half;
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = *(const bf16x8*)(ws + sw(wn * 64 + i * 32 + col, kc));
#pragma unroll
            for (int j = 0; j < T::kMB; ++j) b[j] = *(const bf16x8*)(xs + sw(wm * (BM / 2) + j * 32 + col, kc));
        };
        auto products = [&](const bf16x8 (&a)[2], const bf16x8 (&b)[T::kMB]) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < T::kMB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        };
        if (has(0)) issue(kgrp, 0);
        if (has(1)) issue(KG + kgrp, 1);
        wait_copies<T::kCopies>(has(1));  // this lane's copies of k-tile 0 have landed
        __syncthreads();      // ... and everyone's
        static_assert(kPBK == 32, "the pipeline below takes two 16-wide k-steps per k-tile");
        // Software pipeline over the k-steps: the operands of the next k-step are
        // read while the current one's products run, and the barrier that publishes
        // k-tile kt + 1 sits between the two k-steps of k-tile kt, so that its first
        // operand reads overlap the second k-step's products.
        bf16x8 a0[2], b0[T::kMB], a1[2], b1[T::kMB];
        read_ops(0, 0, a0, b0);
        int stage = 0;
        for (int kt = 0; kt + 1 < nsteps; ++kt) {
            // the stage k-tile kt + 2 goes to was last read before the barrier that
            // ended iteration kt - 1
            const bool ahead = has(kt + 2);
            if (ahead) issue((kt + 2) * KG + kgrp, stage == 0 ? 2 : stage - 1);
            read_ops(stage, 1, a1, b1);
            products(a0, b0);
            const int next = stage == kStages - 1 ? 0 : stage + 1;
            wait_copies<T::kCopies>(ahead);  // k-tile kt + 1 has landed (kt + 2 may still fly)
            __syncthreads();
            read_ops(next, 0, a0, b0);
            products(a1, b1);
            stage = next;
        }
        // the last k-tile
        if (KG == 1 || has(nsteps - 1)) {
            read_ops(stage, 1, a1, b1);
            products(a0, b0);
            products(a1, b1);
        }

        // ---- k groups: group 0 adds up the partial tiles
        if constexpr (KG > 1) {
            __syncthreads();  // every ring is drained
            if (kgrp > 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < T::kMB; ++j)
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            smem.part[kgrp - 1][wave][(i * T::kMB + j) * 4 + g][lane] =
                                make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
            }
            __syncthreads();
            if (kgrp > 0) return;
#pragma unroll 1
            for (int k = 1; k < KG; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < T::kMB; ++j)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const float4 w = smem.part[k - 1][wave][(i * T::kMB + j) * 4 + g][lane];
                            acc[i][j][4 * g] += w.x;
                            acc[i][j][4 * g + 1] += w.y;
                            acc[i][j][4 * g + 2] += w.z;
                            acc[i][j][4 * g + 3] += w.w;
                        }
        }

        // ---- epilogue: lane (col, half) of block (i, j) holds output columns
        // n0 + 8 g + 4 half + 0..3 (g = 0..3) of token m0 + col, rounded to bf16 and
        // stored as 8 bytes into Y[b, h, s, w .. w + 3]
#pragma unroll
        for (int j = 0; j < T::kMB; ++j) {
            const int m = m_base + wm * (BM / 2) + j * 32 + col;
            if (m >= p.M) continue;
            const int bb = m / p.S, s = m - bb * p.S;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = n_base + wn * 64 + i * 32 + 8 * g + 4 * half;
                    if (n >= p.N) continue;
                    const int h = n / p.width, w = n - h * p.width;
                    uint2 v;
                    v.x = pack_bf16(acc[i][j][4 * g], acc[i][j][4 * g + 1]);
                    v.y = pack_bf16(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
                    *(uint2*)((uint16_t*)p.y + (((size_t)bb * p.heads + h) * p.S + s) * p.width + w) = v;
                }
            }
        }
    }
}

// The fewest output tiles (decode steps, short prompts). The tiled kernel above
// walks d_model k-tile after k-tile with a barrier each, so with few workgroups
// its time is as many memory round trips whatever the token count. Here the
// output tile is small and the NW waves of a workgroup split d_model instead: a
// wave takes every NW-th granule of two 32-wide k-steps (128 bytes of each row,
// a cache line), copies them into a ring of D slots of its own (global->LDS, no
// barriers: only this wave reads them) and multiplies them with 16x16x32
// products; the waves' partial tiles are added up in LDS in wave order. The
// copies go through LDS, although no other wave shares them, because the lanes
// of a matrix operand hold 16 different rows side by side: loaded directly, four
// neighbouring lanes touch four cache lines, a quarter of the L1's rate.
template <int BN, int BM, int NW, int D>
struct SplitTile {
    static constexpr int kNA = BN / 16, kNB = BM / 16;  // 16-row blocks (one copy each) of weights and of tokens
    static constexpr int kCopies = kNA + kNB;           // a lane's copies per k-step
    static constexpr int kSlot = (BN + BM) * kPBK;      // bf16 per ring slot: weight rows, then token rows
    static constexpr int kRow = BN + 4;                 // floats per token of a partial tile (16-byte pad)
    static_assert((D & (D - 1)) == 0 && (D - 1) * kCopies <= 63, "ring depth");
    union {
        uint16_t ring[NW][D][kSlot];
        float part[NW][BM * kRow];
    };
};

template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int BN, int BM, int NW, int D>
__global__ __launch_bounds__(64 * NW, 1) void project_split_kernel(const ProjectParams p) {
    using T = SplitTile<BN, BM, NW, D>;
    constexpr int NA = T::kNA, NB = T::kNB;
    __shared__ __align__(16) T sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q4 = lane >> 4;
    const int per_xcd = (p.tiles + kXcdCount - 1) / kXcdCount;
    const int logical = (int)(blockIdx.x % kXcdCount) * per_xcd + (int)(blockIdx.x / kXcdCount);
    if (logical >= p.tiles) return;
    const int n_tiles = (p.N + BN - 1) / BN;
    const int n_base = (logical % n_tiles) * BN, m_base = (logical / n_tiles) * BM;

    // Copy i of a k-step moves 16 rows of 64 bytes, four neighbouring lanes a row,
    // into the rotated order of sw(). Weight rows past the matrix re-read its last
    // row; token rows past it are not copied, except that lane 0 re-reads the last
    // row, so that every copy is issued (the waits below count them). What lies in
    // those rows feeds only outputs that are not stored.
    const int wlast = (p.N - n_base < BN ? p.N - n_base : BN) - 1;
    const int xrows = p.M - m_base < BM ? p.M - m_base : BM;
    const int crow = lane >> 2, cchunk = (lane & 3) ^ ((lane >> 4) & 3);
    const char* wg = (const char*)p.wt + (size_t)n_base * p.K * 2;
    const char* xg = (const char*)p.x + (size_t)m_base * p.K * 2;
    uint32_t woff[NA], xoff[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = i * 16 + crow;
        woff[i] = (uint32_t)(r < wlast ? r : wlast) * (uint32_t)p.K * 2u + cchunk * 16;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int r = j * 16 + crow;
        xoff[j] = (uint32_t)(r < xrows ? r : xrows - 1) * (uint32_t)p.K * 2u + cchunk * 16;
    }

    // this wave's k-steps: granules wave, wave + NW, ... of two steps each
    const int ksteps = p.K / kPBK, granules = (ksteps + 1) / 2;
    const int mine = wave < granules ? (granules - wave + NW - 1) / NW : 0;
    const int cnt = 2 * mine - ((ksteps & 1) && mine > 0 && wave + (mine - 1) * NW == granules - 1 ? 1 : 0);
    auto issue = [&](int t) {
        const int k = 2 * (wave + NW * (t >> 1)) + (t & 1);
        const char* wk = wg + (size_t)k * (kPBK * 2);
        const char* xk = xg + (size_t)k * (kPBK * 2);
        uint16_t* slot = sm.ring[wave][t & (D - 1)];
#pragma unroll
        for (int i = 0; i < NA; ++i) copy16_to_lds(wk, woff[i], slot + i * 16 * kPBK);
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (j * 16 + crow < xrows || lane == 0) copy16_to_lds(xk, xoff[j], slot + (BN + j * 16) * kPBK);
    };
    f32x4 acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int t) {
        const uint16_t* slot = sm.ring[wave][t & (D - 1)];
        bf16x8 a[NA], b[NB];
#pragma unroll
        for (int i = 0; i < NA; ++i) a[i] = *(const bf16x8*)(slot + sw(i * 16 + r16, q4));
#pragma unroll
        for (int j = 0; j < NB; ++j) b[j] = *(const bf16x8*)(slot + BN * kPBK + sw(j * 16 + r16, q4));
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int t = 0; t < D; ++t)
        if (t < cnt) issue(t);
    int t = 0;
    for (; t + D < cnt; ++t) {
        wait_vm<(D - 1) * T::kCopies>();
        step(t);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot is read before it is filled again
        issue(t + D);
    }
    auto drain = [&](auto self, auto d_c) {
        constexpr int d = decltype(d_c)::value;
        if (t + d < cnt) {
            wait_vm<d * T::kCopies>();
            step(t++);
        }
        if constexpr (d > 0) self(self, std::integral_constant<int, d - 1>{});
    };
    drain(drain, std::integral_constant<int, D - 1>{});
    __syncthreads();  // every ring is drained: the LDS becomes the partial tiles

    // accumulator lane (r16, q4) of block (i, j): columns 16 i + 4 q4 .. + 3 of token 16 j + r16
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < NA; ++i)
            *(f32x4*)&sm.part[wave][(j * 16 + r16) * T::kRow + i * 16 + 4 * q4] = acc[i][j];
    __syncthreads();
    constexpr int GROUPS = BM * BN / 4;  // groups of four columns of one token
    for (int e = tid; e < GROUPS; e += 64 * NW) {
        const int ml = e / (BN / 4), nl = (e % (BN / 4)) * 4;
        const int m = m_base + ml, n = n_base + nl;
        f32x4 sum = *(const f32x4*)&sm.part[0][ml * T::kRow + nl];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += *(const f32x4*)&sm.part[w][ml * T::kRow + nl];
        if (m >= p.M || n >= p.N) continue;
        const int bb = m / p.S, s = m - bb * p.S;
        const int h = n / p.width, w = n - h * p.width;
        uint2 v;
        v.x = pack_bf16(sum[0], sum[1]);
        v.y = pack_bf16(sum[2], sum[3]);
        *(uint2*)((uint16_t*)p.y + (((size_t)bb * p.heads + h) * p.S + s) * p.width + w) = v;
    }
}

}  // namespace

template <int BN, int BM, int NW, int D>
static void run_split(const ProjectParams& p, dim3 grid, hipStream_t st) {
    hipLaunchKernelGGL((project_split_kernel<BN, BM, NW, D>), grid, dim3(64 * NW), 0, st, p);
}
template <int BN, int BM, int KG>
static void run_tiles(const ProjectParams& p, dim3 grid, hipStream_t st) {
    hipLaunchKernelGGL((project_kernel<BN, BM, KG>), grid, dim3((proj_threads<BN, KG>())), 0, st, p);
}

tk_status launch_project(const ProjectParams& p, hipStream_t st) {
    // whole tiles per XCD: tail workgroups of the last XCDs exit at once
    const dim3 grid((unsigned)((p.tiles + kXcdCount - 1) / kXcdCount * kXcdCount));
    switch (project_shape(p.M, p.N, p.K)) {
        case ProjShape::k16x16: run_split<16, 16, 8, 4>(p, grid, st); break;
        case ProjShape::k16x32: run_split<16, 32, 8, 4>(p, grid, st); break;
        case ProjShape::k32x32: run_split<32, 32, 8, 4>(p, grid, st); break;
        case ProjShape::k32x64: run_split<32, 64, 8, 2>(p, grid, st); break;
        case ProjShape::k64x64: run_tiles<64, 64, 4>(p, grid, st); break;
        case ProjShape::k64x128: run_tiles<64, 128, 4>(p, grid, st); break;
        case ProjShape::k128x64: run_tiles<128, 64, 2>(p, grid, st); break;
        case ProjShape::k128x128: run_tiles<128, 128, 2>(p, grid, st); break;
        case ProjShape::k128x128whole: run_tiles<128, 128, 1>(p, grid, st); break;
        case ProjShape::k256x128: run_tiles<256, 128, 1>(p, grid, st); break;
        case ProjShape::k256x256: run_tiles<256, 256, 1>(p, grid, st); break;
    }
    return hipGetLastError() == hipSuccess ? TK_OK : TK_ERR_HIP;
}

}  // namespace tk
