// Base GEMM y = x W (bf16 MFMA, fp32 accumulate), optionally with the adapter
// delta folded in: y = x W + v B_a per token, v = s_a (x A_a) from the shrink.
//
// This is the base-model product that unmerged inference shares across all
// requests of the batch, with the adapter branches added on top (paper
// sections 1-2); adding the delta to the fp32 accumulators before y is rounded
// makes unmerged inference cost close to merged inference (section 4.4).
//
// Both kernels walk the tokens in the plan's row order, in which neighbouring rows share an adapter.
//   gemm_ring_kernel: after the K loop every wavefront adds the deltas of its own 64 tokens to its accumulators,
//     adapter by adapter and 32 ranks at a time, with Bt_a[its features, ranks] and the tokens' v (split into two
//     bf16 terms v_hi + v_lo) straight from memory as MFMA operands (see the kernel).
//   gemm_tiled_kernel: the delta enters as extra k-stages of the same pipeline; for each adapter a present in a
//     row tile it runs ceil(2 r_a / 64) more stages whose "W tile" is Bt_a[features, ranks] and whose "x tile" is the
//     matching columns of [v_hi | v_lo] (rows of other adapters zero; Bt_a is simply addressed twice).  Their loads
//     are prefetched like any other stage's.
//
// x [T,K] and Wt [N,K] are both contraction-index-fastest, so tiles arrive in LDS
// as 16-byte chunks and come back out of it as ready-made MFMA operands (8
// consecutive k per lane).  Two kernels:
//
//   gemm_ring_kernel (further down): 256 x 256 tiles of large problems.  8 wavefronts, 16x16x32 MFMA,
//     loads HBM -> LDS directly into a ring of quarter stages of 64 k.
//   gemm_tiled_kernel: what neither that nor the kernels of smaller batches (kernels_gemm_small.hip,
//     kernels_gemm_mid.hip; gemm_route chooses) take.  Loads HBM -> registers -> LDS, double buffered (dynamic LDS,
//     2 x (BM + BT) x 128 bytes); workgroup tile = 4 wavefronts (2 x 2), each WB x WB MFMA blocks of 32 x 32:
//     WB = 4: 256 features x 256 tokens x 64 k (large problems with adapters and K of at most 128, or past 32-bit offsets)
//     WB = 2: 128 x 128 x 64 (products of few stages without adapters, and operands past 32-bit offsets)
//
// Lane roles in v_mfma_f32_32x32x16_bf16 (D = A*B + C, A 32x16, B 16x32):
//   lane l supplies A[row l%32][k 8*(l/32) .. +7], B[k 8*(l/32) .. +7][col l%32],
//   receives D[row 8*(i/4) + 4*(l/32) + i%4][col l%32], i = 0..15.
// MFMA rows carry output features, columns carry tokens.  MFMA row 8q+4h+p of a
// block stands for feature 16h + 4q + p, so a lane (h = l/32) ends up with the
// 16 consecutive features 16h .. 16h+15 of its token: 32-byte stores of y.
#include <atomic>
#include "kernels.h"
#include "launch.h"
#include "mfma_tile.h"

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

namespace {

constexpr int BK = 64;    // k per stage; a tile row is 128 bytes = 8 chunks of 16 bytes

// LDS tile: rows x 8 chunks of 16 bytes; chunk c of row r lives at chunk slot c ^ f(r).  A ds_read_b128 of a
// wavefront is served 8 lanes at a time, so f must take 8 different values over the 8 rows those lanes read.
// x tile: lanes read consecutive rows -> f = r & 7.  W tile: lanes 8g..8g+7 read rows 4g..4g+3 and
// 16+4g..16+4g+3 (the feature permutation of the MFMA rows) -> f = (r & 3) | bit 4 of r << 2.
__device__ __forceinline__ int lds_slot(int row, int chunk) { return row * 8 + (chunk ^ ((row >> 1) & 7)); }
__device__ __forceinline__ int lds_slot_w(int row, int chunk) { return row * 8 + (chunk ^ (((row >> 1) & 3) | ((row >> 2) & 4))); }

// 16-byte load from a wavefront-uniform base plus a 32-bit byte offset per lane (one address register per lane for any
// number of loads that share the offset); the base comes out of a table: the address space is stated, as in ld16
__device__ __forceinline__ uint4 ldg16_off(const void* uniform_base, uint32_t byte_off)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const __attribute__((address_space(1))) char* b = (const __attribute__((address_space(1))) char*)(uintptr_t)uniform_base;
    const u32x4 r = *(const __attribute__((address_space(1))) u32x4*)(b + byte_off);
    return uint4{r[0], r[1], r[2], r[3]};
#else
    return *reinterpret_cast<const uint4*>(static_cast<const char*>(uniform_base) + byte_off);
#endif
}

extern __shared__ uint4 gemm_lds[];
constexpr int META_MAX = 256;      // adapter stages of a tile whose metadata is cached in LDS (more are read from memory)

struct gemm_delta_args {
    const int32_t* order;          // [T] tokens in the plan's row order; nullptr = identity
    const int32_t* row_key;        // [T] in the order above: the token's adapter (bits 0..22; all ones: none) | removal bit
    const int32_t* rank;
    const int32_t* extra_ptr;      // [token tiles + 1]
    const int32_t* extra;          // stage id (adapter, | removal bit) | rank block << 24
    const bf16_t* vb;              // [T][2][R]: v_hi, v_lo
    int R;
    const bf16_t* const* Bt_ptrs;
    const bf16_t* zeros;           // 16 zero bytes: the source of chunks that are masked out
    const bf16_t* vb2;             // mixture mode: [T][2][R2] split of the removal's v (read by the marked stages)
    int R2;
    int merged;                    // mixture mode: the merged adapter, else -1
};

// Stage ids and row keys.  An ordinary stage (id = adapter) concerns the rows of that adapter.  A stage whose id
// carries the removal bit (mixture mode: the merged adapter's update is taken off again) concerns every row whose key
// carries it: the rows of all other adapters and of none.  Rows beyond T have the key "none" without the bit.
constexpr int STAGE_REMOVAL = LORA_UNMERGE_BIT, KEY_NONE = LORA_UNMERGE_BIT - 1;
__device__ __forceinline__ bool stage_hits(int row_key, int stage_id)
{
    return (stage_id & STAGE_REMOVAL) ? (row_key & STAGE_REMOVAL) != 0 : (row_key & KEY_NONE) == stage_id;
}
// columns [part * r + j, + 8) of the token's [v_hi | v_lo] that the stage reads
__device__ __forceinline__ const bf16_t* stage_v(const gemm_delta_args& da, int stage_id, int token, int part, int j)
{
    return (stage_id & STAGE_REMOVAL) ? da.vb2 + ((int64_t)token * 2 + part) * da.R2 + j
                                      : da.vb + ((int64_t)token * 2 + part) * da.R + j;
}

// KTAIL: K is not a multiple of 64, the last K stage's chunks beyond K are zero-filled
template <int WB, bool DELTA, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_tiled_kernel(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, gemm_delta_args da)
{
    constexpr int BM = 64 * WB;            // features per workgroup tile
    constexpr int BT = 64 * WB;            // tokens per workgroup tile
    constexpr int NLD = (BM * 8) / 256;    // 16-byte chunks of W (and of x) per thread and stage
    uint4* lds_w0 = gemm_lds;                       // [2][BM * 8]
    uint4* lds_x0 = gemm_lds + 2 * BM * 8;          // [2][BT * 8]
    // DELTA: the tile's adapter stages {adapter, rank, Bt pointer} are fetched once, up front, into LDS
    uint4* lds_meta = gemm_lds + 4 * BM * 8;        // [META_MAX]
    // DELTA: token and adapter of the rows this thread stages, parked in LDS so that they hold no
    // registers during the K stages: [NLD][256] int2
    int2* lds_rows = reinterpret_cast<int2*>(lds_meta + META_MAX);

    int tile_n, tile_t;
    tile_of_workgroup(blockIdx.x, tiles_n, tiles_t, tile_n, tile_t);
    const int n0 = tile_n * BM, t0 = tile_t * BT;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wn = (wave & 1) * (32 * WB), wt = (wave >> 1) * (32 * WB);   // wavefront tile origin
    const int c_lane8 = (tid & 7) * 8;                           // this thread's k offset inside a stage

    // global -> register staging: the rows this thread fetches in every stage
    const bf16_t* gw[NLD];
    const bf16_t* gx[NLD];
    int slot[NLD], slot_w[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int q = tid + i * 256, row = q >> 3, c = q & 7;
        int nr = n0 + row; if (nr >= N) nr = N - 1;
        int pos = t0 + row;
        const bool pos_ok = pos < T;
        if (!pos_ok) pos = T - 1;
        const int tok = DELTA ? da.order[pos] : pos;
        gw[i] = Wt + (int64_t)nr * ldw + c * 8;
        gx[i] = x + (int64_t)tok * ldx + c * 8;
        slot[i] = lds_slot(row, c);
        slot_w[i] = lds_slot_w(row, c);
        if constexpr (DELTA) lds_rows[i * 256 + tid] = make_int2(tok, pos_ok ? da.row_key[pos] : KEY_NONE);
    }

    floatx16 acc[WB][WB];
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    // LDS rows this lane reads as MFMA operands
    const int l32 = lane & 31, h = lane >> 5;
    // feature of MFMA row l32 = 8q + 4hh + p  ->  16 hh + 4 q + p
    const int frow = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);

    const int stages_k = (K + BK - 1) / BK;
    int extra_base = 0, n_extra = 0, stages = stages_k;
    if constexpr (DELTA) {
        extra_base = da.extra_ptr[tile_t];
        n_extra = da.extra_ptr[tile_t + 1] - extra_base;
        stages += n_extra;
        for (int e = tid; e < n_extra && e < META_MAX; e += 256) {
            const int packed = da.extra[extra_base + e];
            const int a_id = packed & KEY_NONE;
            const uint64_t bt = reinterpret_cast<uint64_t>(da.Bt_ptrs[a_id]);
            lds_meta[e] = uint4{(uint32_t)packed, (uint32_t)da.rank[a_id], (uint32_t)bt, (uint32_t)(bt >> 32)};
        }
    }
    bool skip[WB];                                               // column blocks without a token of the stage's adapter
#pragma unroll
    for (int b = 0; b < WB; ++b) skip[b] = false;
    uint4 rw[NLD], rx[NLD];
    auto load_k_stage = [&](int s) {
        const int k = s * BK;
        const bool in = !KTAIL || k + c_lane8 < K;               // K % 8 == 0: chunk is whole or absent
        // same issue order as in the steady loop: all W chunks, then all x chunks
#pragma unroll
        for (int i = 0; i < NLD; ++i) rw[i] = in ? *reinterpret_cast<const uint4*>(gw[i] + k) : uint4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < NLD; ++i) rx[i] = in ? *reinterpret_cast<const uint4*>(gx[i] + k) : uint4{0, 0, 0, 0};
    };
    auto load_stage = [&](int s) {
        if (!DELTA || s < stages_k) {
            load_k_stage(s);
        } else {
            // adapter stage: Bt_a[feature rows, ranks] against 64 columns of [v_hi | v_lo] of the adapter's tokens
            const int e = s - stages_k;
            int packed, r;
            const bf16_t* Bt;
            if (e < META_MAX) {
                const uint4 m = lds_meta[e];
                packed = (int)m.x;
                r = (int)m.y;
                Bt = reinterpret_cast<const bf16_t*>((uint64_t)m.z | ((uint64_t)m.w << 32));
            } else {
                packed = da.extra[extra_base + e];
                r = da.rank[packed & KEY_NONE];
                Bt = da.Bt_ptrs[packed & KEY_NONE];
            }
            const int a_id = packed & 0xffffff;
            // column of the adapter's [v_hi | v_lo] concatenation; r % 8 == 0, so a chunk lies in one half
            const int col = (packed >> 24) * 64 + c_lane8;
            const bool in = col < 2 * r;
            const int part = col >= r ? 1 : 0;
            const int j = col - part * r;
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                int nr = n0 + ((tid + i * 256) >> 3);
                if (nr >= N) nr = N - 1;
                const int2 ta = lds_rows[i * 256 + tid];         // (token, its adapter)
                rw[i] = in ? *reinterpret_cast<const uint4*>(Bt + (int64_t)nr * r + j) : uint4{0, 0, 0, 0};
                rx[i] = (in && stage_hits(ta.y, a_id))
                            ? *reinterpret_cast<const uint4*>(stage_v(da, a_id, ta.x, part, j))
                            : uint4{0, 0, 0, 0};
            }
        }
    };
    auto store_stage = [&](int buf) {
        uint4* lw = lds_w0 + buf * BM * 8;
        uint4* lx = lds_x0 + buf * BT * 8;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            lw[slot_w[i]] = rw[i];
            lx[slot[i]] = rx[i];
        }
    };
    auto read_ops = [&](const uint4* lw, const uint4* lx, int ks, op16 (&wa)[WB], op16 (&xb)[WB]) {
        const int c = ks * 2 + h;
#pragma unroll
        for (int a = 0; a < WB; ++a) wa[a].u = lw[lds_slot_w(wn + a * 32 + frow, c)];
#pragma unroll
        for (int b = 0; b < WB; ++b) xb[b].u = lx[lds_slot(wt + b * 32 + l32, c)];
    };
    auto mma = [&](const op16 (&wa)[WB], const op16 (&xb)[WB]) {
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            if (DELTA && skip[b]) continue;                      // wavefront-uniform
#pragma unroll
            for (int a = 0; a < WB; ++a)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[a].v, xb[b].v, acc[a][b], 0, 0, 0);
        }
    };
    // an adapter stage only concerns the column blocks that hold one of the adapter's tokens
    auto set_skip = [&](int stage) {
        if constexpr (DELTA) {
            if (stage < stages_k) return;
            const int e = stage - stages_k;
            const int a_id = (e < META_MAX ? (int)lds_meta[e].x : da.extra[extra_base + e]) & 0xffffff;
#pragma unroll
            for (int b = 0; b < WB; ++b) {
                // row wt + 32 b + l32 of the tile is staged by thread (row * 8) & 255 as its chunk slot (row * 8) >> 8
                const int q = (wt + b * 32 + (lane & 31)) * 8;
                skip[b] = __ballot(stage_hits(lds_rows[(q >> 8) * 256 + (q & 255)].y, a_id)) == 0;
            }
        }
    };

    // Software pipeline.  Global loads run two stages ahead (registers), LDS is double
    // buffered, MFMA operands are double buffered in registers: while the matrix cores
    // work on k-step ks the LDS reads of ks+1 are in flight, and the barrier between
    // stages sits before the last k-step so that its MFMAs cover the first reads of the
    // next stage.
    op16 waA[WB], xbA[WB], waB[WB], xbB[WB];
    int s = 0;
    const bool steady = WB == 4 && !KTAIL && stages_k >= 3 && n_extra <= META_MAX;
    if (!steady) {
        // (the adapter stages' descriptors in LDS are read by every thread: with a single K stage the load of
        // stage 1 below is already an adapter stage's)
        if constexpr (DELTA) __syncthreads();
        load_stage(0);
        store_stage(0);
        if (stages > 1) load_stage(1);
        __syncthreads();
        read_ops(lds_w0, lds_x0, 0, waA, xbA);
    }
    if constexpr (WB == 4 && !KTAIL) if (steady) {
        // (its own straight-line prologue: were the steady loop reachable through the branchy general
        // loader, the compiler would wait for all outstanding loads at the top of every iteration)
        // Running source pointers of the stage to fetch next.  A K stage advances them by 64 elements; an
        // adapter stage sets them afresh: W chunks to Bt_a[feature row, ranks], x chunks to the token's
        // [v_hi | v_lo] columns, and every chunk that is masked out (beyond the rank, or a token of another
        // adapter) to a block of zeros -- so all stages issue the same 16 unconditional loads.
        const bf16_t* pw[NLD];
        const bf16_t* px[NLD];
#pragma unroll
        for (int i = 0; i < NLD; ++i) { pw[i] = gw[i]; px[i] = gx[i]; }
        auto advance = [&](int next) {
            if (!DELTA || next < stages_k) {
#pragma unroll
                for (int i = 0; i < NLD; ++i) { pw[i] += BK; px[i] += BK; }
            } else if (next < stages) {
                const uint4 m = lds_meta[next - stages_k];
                const int a_id = (int)m.x & 0xffffff, r = (int)m.y;
                const bf16_t* Bt = reinterpret_cast<const bf16_t*>((uint64_t)m.z | ((uint64_t)m.w << 32));
                const int col = ((int)m.x >> 24) * 64 + c_lane8;
                const bool in = col < 2 * r;
                const int part = col >= r ? 1 : 0;
                const int j = col - part * r;
#pragma unroll
                for (int i = 0; i < NLD; ++i) {
                    int nr = n0 + ((tid + i * 256) >> 3);
                    if (nr >= N) nr = N - 1;
                    const int2 ta = lds_rows[i * 256 + tid];
                    pw[i] = in ? Bt + (int64_t)nr * r + j : da.zeros;
                    px[i] = (in && stage_hits(ta.y, a_id)) ? stage_v(da, a_id, ta.x, part, j) : da.zeros;
                }
            }
        };
        auto load_ptrs = [&]() {
#pragma unroll
            for (int i = 0; i < NLD; ++i) rw[i] = *reinterpret_cast<const uint4*>(pw[i]);
#pragma unroll
            for (int i = 0; i < NLD; ++i) rx[i] = *reinterpret_cast<const uint4*>(px[i]);
        };
        __syncthreads();                                 // lds_meta / lds_rows are complete
        // stages 0, 1 and 2 are K stages (stages_k >= 3): straight-line code up to the first loop (were it
        // reachable through a branch with loads in flight, the compiler would wait for all of them at the
        // top of every iteration instead of the oldest one)
        load_ptrs();
        store_stage(0);
#pragma unroll
        for (int i = 0; i < NLD; ++i) { pw[i] += BK; px[i] += BK; }
        load_ptrs();
#pragma unroll
        for (int i = 0; i < NLD; ++i) { pw[i] += BK; px[i] += BK; }
        __syncthreads();
        read_ops(lds_w0, lds_x0, 0, waA, xbA);
        // Steady state over all stages but the last two, written out so that every MFMA is followed by exactly
        // one memory operation (the scheduler is pinned to that order): the 64 MFMAs of a stage
        // carry its 32 LDS operand reads, the 16 LDS writes of the next stage and the 16 global
        // loads of the stage after that, and the matrix cores never wait for a block of them.
        auto one_read = [&](const uint4* lw, const uint4* lx, int ks, int i, op16 (&wa)[WB], op16 (&xb)[WB]) {
            const int c = ks * 2 + h;
            if (i < 4) wa[i].u = lw[lds_slot_w(wn + i * 32 + frow, c)];
            else xb[i - 4].u = lx[lds_slot(wt + (i - 4) * 32 + l32, c)];
        };
#define MMA1(WA, XB, IDX) \
        acc[(IDX) >> 2][(IDX) & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(WA[(IDX) >> 2].v, XB[(IDX) & 3].v, acc[(IDX) >> 2][(IDX) & 3], 0, 0, 0)
#define PIN(MASK) do { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(MASK, 1, 0); } while (0)
        // the body of one stage; ADV_GENERAL: the pointer update after it may set up an adapter stage
#define STAGE_BODY(ADV_GENERAL)                                                                                        \
        {                                                                                                              \
            const int buf = s & 1;                                                                                     \
            const uint4* lw = lds_w0 + buf * BM * 8;                                                                   \
            const uint4* lx = lds_x0 + buf * BT * 8;                                                                   \
            uint4* lw_n = lds_w0 + (buf ^ 1) * BM * 8;                                                                 \
            uint4* lx_n = lds_x0 + (buf ^ 1) * BT * 8;                                                                 \
            /* k-step 0: reads of k-step 1, W chunks of stage s+1 into LDS */                                          \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waA, xbA, i); one_read(lw, lx, 1, i, waB, xbB); PIN(0x100); }       \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waA, xbA, 8 + i); lw_n[slot_w[i]] = rw[i]; PIN(0x200); }           \
            /* k-step 1: reads of k-step 2, x chunks of stage s+1 into LDS */                                          \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waB, xbB, i); one_read(lw, lx, 2, i, waA, xbA); PIN(0x100); }       \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waB, xbB, 8 + i); lx_n[slot[i]] = rx[i]; PIN(0x200); }             \
            /* k-step 2: reads of k-step 3, W chunks of stage s+2 from memory */                                       \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waA, xbA, i); one_read(lw, lx, 3, i, waB, xbB); PIN(0x100); }       \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waA, xbA, 8 + i); rw[i] = *reinterpret_cast<const uint4*>(pw[i]); PIN(0x020); } \
            __syncthreads(); /* stage s+1 is in LDS; nobody reads stage s any more */                                  \
            /* k-step 3: reads of k-step 0 of stage s+1, x chunks of stage s+2 from memory */                          \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waB, xbB, i); one_read(lw_n, lx_n, 0, i, waA, xbA); PIN(0x100); }   \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) { MMA1(waB, xbB, 8 + i); rx[i] = *reinterpret_cast<const uint4*>(px[i]); PIN(0x020); } \
            if (ADV_GENERAL) advance(s + 3);                                                                           \
            else { _Pragma("unroll") for (int i = 0; i < NLD; ++i) { pw[i] += BK; px[i] += BK; } }                     \
        }
        // K stages whose successors are K stages too: a loop without any branch in its body (a branch
        // makes the compiler wait for all outstanding loads instead of the oldest one)
        for (; s + 3 < stages_k; ++s) STAGE_BODY(false)
        // the stages around and inside the adapter part
        for (; s + 2 < stages; ++s) STAGE_BODY(true)
#undef STAGE_BODY
#undef MMA1
#undef PIN
    }
    // the last two stages (and everything, for the small tile / K tail builds)
    for (; s < stages; ++s) {
        set_skip(s);
        const int buf = s & 1;
        const uint4* lw = lds_w0 + buf * BM * 8;
        const uint4* lx = lds_x0 + buf * BT * 8;
        const uint4* lw_n = lds_w0 + (buf ^ 1) * BM * 8;
        const uint4* lx_n = lds_x0 + (buf ^ 1) * BT * 8;
        read_ops(lw, lx, 1, waB, xbB);
        mma(waA, xbA);
        read_ops(lw, lx, 2, waA, xbA);
        if (s + 1 < stages) store_stage(buf ^ 1);        // stage s+1: fetched one stage ago
        if (s + 2 < stages) load_stage(s + 2);
        mma(waB, xbB);
        read_ops(lw, lx, 3, waB, xbB);
        mma(waA, xbA);
        __syncthreads();                                 // stage s+1 is in LDS; nobody reads stage s any more
        if (s + 1 < stages) read_ops(lw_n, lx_n, 0, waA, xbA);
        mma(waB, xbB);
    }

    // ---- epilogue: one rounding, store (rows go back to their tokens) ------
#pragma unroll
    for (int b = 0; b < WB; ++b) {
        const int pos = t0 + wt + b * 32 + l32;                  // this lane's row of the order in column block b
        if (pos >= T) continue;
        const int t = DELTA ? da.order[pos] : pos;
#pragma unroll
        for (int a = 0; a < WB; ++a) {
            const int n = n0 + wn + a * 32 + 16 * h;             // first of this lane's 16 features
            bf16_t* yp = y + (int64_t)t * ldy + n;
            // acc index i = 4q + p  <->  feature offset 4q + p
            if (n + 16 <= N) {
                uint32_t o[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    o[q] = (uint32_t)f32_to_bf16(acc[a][b][2 * q]) | ((uint32_t)f32_to_bf16(acc[a][b][2 * q + 1]) << 16);
                *reinterpret_cast<uint4*>(yp) = uint4{o[0], o[1], o[2], o[3]};
                *reinterpret_cast<uint4*>(yp + 8) = uint4{o[4], o[5], o[6], o[7]};
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (n + i < N) yp[i] = f32_to_bf16(acc[a][b][i]);
            }
        }
    }
}


// ---------------------------------------------------------------------------------------------------------
// 256 x 256 tiles of large problems.  Tiles go HBM -> LDS directly (global_load_lds_dwordx4: no staging registers, no
// LDS write instructions) into a ring of ten granules of 16 KB, two stages of 64 k ahead of their use.
//
// What bounds a compute unit's loads is the number of cache lines its requests touch, not their bytes: L2-resident rows
// arrive at 100 - 108 GB/s per compute unit as 8 rows x 128 bytes (whole lines) per instruction, at 59 - 65 GB/s as 16 rows x
// 64 bytes whose other halves are asked for when they have left the 32 KB L1 (with eight loads in flight per wavefront).  A
// 256 x 256 tile at 1.45 PFLOP/s of the chip takes 44 GB/s per compute unit next to its LDS reads and barriers, so stages
// of 32 k (64 bytes of a row) came near their end; hence stages of 64 k.
//
// Eight wavefronts, two per SIMD, each 128 features x 64 tokens (8 x 4 blocks of v_mfma_f32_16x16x32_bf16, 128
// accumulator registers).  A stage is four phases of 16 MFMAs, one per quadrant of the wavefront's tile:
//   phase 0: W low x x low    1: W low x x high    2: W high x x high    3: W high x x low
// and its operands are four granules (of all wavefronts together): WL, XL, XH, WH = rows of W blocks 0..3, x blocks
// 0..1, x blocks 2..3, W blocks 4..7, 128 rows x 64 k each.  Granule g (4 per stage, in that order) is read into
// registers one phase before its first use, in phase g - 1, and fetched in phase g - 9.
// A phase is a memory part (LDS reads of one granule, this wavefront's two loads of another) and a matrix part, each
// closed by a barrier.  Wavefronts 4..7 run one part behind wavefronts 0..3, with which they share the SIMDs: while
// one of the two wavefronts of a SIMD issues its 16 MFMAs back to back, the other does its memory part.
//   RAW: granule k + 2 is read in memory part k + 1; every wavefront has waited for its own loads of it (vmcnt; loads
//        return in order) at the end of its memory part k, one barrier earlier at least.
//   WAR: granule g, read in memory part g - 1, is overwritten by loads issued in memory part g + 1, when the trailing
//        wavefronts are in matrix part g; every wavefront's LDS reads of it have returned at the end of its matrix part
//        g - 1, one barrier earlier: its MFMAs use XL, XH and WH in that part; WL, first used in the part after it, is
//        waited for (by then its reads are a matrix part old and long back: the wait costs nothing).
// The loads are issued from inline assembly, so the compiler does not count them: the waits are written out.
//
// Measured against the version with stages of 32 k (same process, cold operands, bf16, T x K x N): 16384 x 5120 x 5120
// 709 -> 594 us (1.45 PFLOP/s), 16384 x 5120 x 13824 1968 -> 1623 us, 8192 x 4096 x 11008 609 -> 534 us, 4096^3 109 ->
// 99 us.  With all-zero operands it runs at 1.75 - 2.0 PFLOP/s: what is left is the clock the chip holds under the
// switching of random operands.  (v_mfma_f32_32x32x16_bf16 in the same schedule: 10 % slower.)
constexpr int RK = 64;                  // k per stage; a row of a granule is 128 bytes = 8 chunks of 16 bytes
constexpr int GRANULES = 10;            // ring slots
constexpr int GRANULE = 16384;          // bytes: 128 rows x 128 bytes

// Chunk c of granule row r lives at slot 8 r + (c ^ f(r)).  An operand read (ds_read_b128) has lane l take chunk
// 4 ks + l / 16 of one of 16 rows: x rows r0 + l % 16, W rows r0 + 16 (l % 16 / 4) + l % 4 (the MFMA row
// permutation); each f takes eight different values over the rows that eight consecutive lanes read (SQ_LDS_BANK_CONFLICT: 0).
__device__ __forceinline__ int ring_f_x(int row) { return row & 7; }
__device__ __forceinline__ int ring_f_w(int row) { return (row & 3) | ((row >> 2) & 4); }

// KTAIL: K is no multiple of 64.  The last stage's chunks past K are fetched from the row's first chunk of that stage
// (in bounds) and zeroed in the registers.
template <bool DELTA, bool KTAIL>
__global__ __launch_bounds__(512) void gemm_ring_kernel(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, gemm_delta_args da)
{
    // DELTA: the rows of the tile are tokens in the plan's row order, and after the K loop every wavefront adds the
    // adapter deltas of its own 64 tokens to its accumulators by itself: for each adapter among them (one or two,
    // mostly) and each block of 32 ranks, Bt_a[its 128 features, 32 ranks] as the MFMA row operand straight from
    // memory, and the tokens' v (its two bf16 terms) as the column operands, masked to the adapter's tokens.  No LDS,
    // no workgroup barrier, no work for the rows of other wavefronts: a wavefront pays for the adapters of its own 64
    // tokens only, where a shared adapter stage would cost all eight of them a whole 256 x 256 step per adapter and
    // block of ranks.
    constexpr int BM = 256, BT = 256, WA = 8, WX = 4;

    int tile_n, tile_t;
    tile_of_workgroup(blockIdx.x, tiles_n, tiles_t, tile_n, tile_t);
    const int n0 = tile_n * BM, t0 = tile_t * BT;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = (wave & 1) * 128, wt = (wave >> 1) * 64;         // wavefront tile origin
    // Lane roles in v_mfma_f32_16x16x32_bf16 (D = A*B + C, A 16x32, B 32x16): lane l supplies A[row l%16][k 8(l/16) ..
    // +7] and B[k 8(l/16) .. +7][col l%16], and receives D[row 4(l/16) + i][col l%16], i = 0..3.  MFMA rows carry
    // features, columns carry tokens.  The 128 features of a wavefront are two groups of 64; block q of a group
    // holds the features 16 g + 4 q + i (MFMA row 4 g + i), so that over its four blocks a lane (g = l/16) ends up
    // with the 16 consecutive features 16 g .. 16 g + 15 of its token.
    const int l16 = lane & 15, kg = lane >> 4;
    const int frow = 16 * (l16 >> 2) + (l16 & 3);                   // feature (block 0 of a group) of MFMA row l16

    // Staging role: load j of this wavefront fills rows (2 wave + j) 8 .. +7 of a granule; this lane brings the chunk
    // that belongs in slot lane & 7 of row .. + lane / 8.  Granule rows: WL / WH rows r are the tile's features
    // 128 (r / 64) + r % 64 (+ 64), XL / XH rows r its tokens 64 (r / 32) + r % 32 (+ 32): every wavefront's low / high
    // half.  (The launcher keeps N ldw and T ldx below 2^31 elements, so 32-bit byte offsets do.)
    uint32_t off_w[2][2], off_x[2][2];                               // [high half][load]
    int cut_w = 0, cut_x = 0;                                        // KTAIL: what takes an offset back to its row's first chunk
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = (wave * 2 + j) * 8 + (lane >> 3);
        const int cw = (lane & 7) ^ ring_f_w(row), cx = (lane & 7) ^ ring_f_x(row);     // (the same for both j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int nr = n0 + (row >> 6) * 128 + (row & 63) + 64 * h; if (nr >= N) nr = N - 1;
            int pos = t0 + (row >> 5) * 64 + (row & 31) + 32 * h; if (pos >= T) pos = T - 1;
            const int tok = DELTA ? da.order[pos] : pos;
            off_w[h][j] = (uint32_t)(nr * ldw * 2) + cw * 16;
            off_x[h][j] = (uint32_t)(tok * ldx * 2) + cx * 16;
        }
        if (KTAIL) {
            const int last = (K - 1) / RK * RK;
            cut_w = last + cw * 8 >= K ? cw * 16 : 0;
            cut_x = last + cx * 8 >= K ? cx * 16 : 0;
        }
    }
    // DELTA: token and key of row wt + lane of the tile (this wavefront's 64 tokens, one per lane)
    int my_tok = 0, my_key = KEY_NONE;
    if constexpr (DELTA) {
        const int pos = t0 + wt + lane;
        my_tok = da.order[pos < T ? pos : T - 1];
        my_key = pos < T ? da.row_key[pos] : KEY_NONE;
    }

    const int stages = (K + RK - 1) / RK;                            // at least 3 (checked by the launcher)

    floatx4 acc[WA][WX];
#pragma unroll
    for (int a = 0; a < WA; ++a)
#pragma unroll
        for (int b = 0; b < WX; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    // granule loads: kind 0 WL, 1 XL, 2 XH, 3 WH of stage st into ring slot `slot` (bytes)
    const char* const xb = reinterpret_cast<const char*>(x);
    const char* const wb = reinterpret_cast<const char*>(Wt);
    const uint32_t lds0 = lds_address(gemm_lds), lds_load = lds0 + wave * 2048;
    auto issue = [&](int kind, int st, uint32_t slot) {
        const bool is_w = kind == 0 || kind == 3;
        const int h = kind >= 2;
        const char* base = (is_w ? wb : xb) + (int64_t)st * (RK * 2);
        const uint32_t cut = KTAIL && st == stages - 1 ? (uint32_t)(is_w ? cut_w : cut_x) : 0u;
#pragma unroll
        for (int j = 0; j < 2; ++j) load16_to_lds(base, (is_w ? off_w[h][j] : off_x[h][j]) - cut, lds_load + slot + j * 1024);
    };

    // operand reads: lane addresses inside a granule for k-step 0; k-step 1 is 64 bytes apart by XOR
    const uint32_t rw0 = ((wave & 1) * 64 + frow) * 128 + (kg ^ ring_f_w(frow)) * 16;
    const uint32_t rx0 = ((wave >> 1) * 32 + l16) * 128 + (kg ^ ring_f_x(l16)) * 16;
    const char* const lds_c = reinterpret_cast<const char*>(gemm_lds);
    op16 wl[2][4], wh[2][4], xl[2][2], xh[2][2];                     // [k-step][block]
    auto read_w = [&](op16 (&w)[2][4], uint32_t slot) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int a = 0; a < 4; ++a) w[ks][a].u = *reinterpret_cast<const uint4*>(lds_c + (slot + (rw0 ^ (ks * 64))) + a * 512);
    };
    auto read_x = [&](op16 (&xo)[2][2], uint32_t slot) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int b = 0; b < 2; ++b) xo[ks][b].u = *reinterpret_cast<const uint4*>(lds_c + (slot + (rx0 ^ (ks * 64))) + b * 2048);
    };
    auto cut_tail = [&](op16& o, int ks) {                           // KTAIL, last stage: chunks past K are zero
        if ((stages - 1) * RK + (ks * 4 + kg) * 8 >= K) o.u = uint4{0, 0, 0, 0};
    };
    auto mma = [&](const op16 (&w)[2][4], const op16 (&xo)[2][2], int a0, int b0) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a0 + a][b0 + b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][a].v, xo[ks][b].v, acc[a0 + a][b0 + b], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
    };
#define RING_BARRIER() do { __builtin_amdgcn_sched_barrier(0); asm volatile("s_barrier" ::: "memory"); __builtin_amdgcn_sched_barrier(0); } while (0)
#define RING_WAIT_(N_) asm volatile("s_waitcnt vmcnt(" #N_ ")" ::: "memory")
#define RING_WAIT(N_) RING_WAIT_(N_)
#define RING_READS_RETURNED() asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory")

    // prologue: granules 0..8 on their way, granule 0 (WL of stage 0) into registers, granule 1 landed
#pragma unroll
    for (int gr = 0; gr < 9; ++gr) issue(gr & 3, gr >> 2, gr * GRANULE);
    RING_WAIT(16);
    RING_BARRIER();
    read_w(wl, 0);
    RING_WAIT(14);
    RING_READS_RETURNED();
    RING_BARRIER();
    if (wave >= 4) RING_BARRIER();                                   // the trailing wavefronts: one part behind

    // one stage; q: slot of granule 4 s (bytes).  NI: how many of its phases issue loads; W0..W3: loads that may be
    // outstanding at the end of the memory parts
    auto wrap = [](uint32_t v) { return v >= GRANULES * GRANULE ? v - GRANULES * GRANULE : v; };
    uint32_t q = 0;
    int s = 0;
#define RING_STAGE(NI, W0, W1, W2, W3, LAST)                                                                           \
    {                                                                                                                  \
        const uint32_t q2 = wrap(q + 2 * GRANULE), q4 = wrap(q + 4 * GRANULE), q9 = wrap(q + 8 * GRANULE) + GRANULE;   \
        read_x(xl, q + GRANULE);                                                                                       \
        if (NI > 0) issue(1, s + 2, q9);                                                                               \
        if (KTAIL && LAST) { _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) { _Pragma("unroll") for (int a = 0; a < 4; ++a) cut_tail(wl[ks][a], ks); _Pragma("unroll") for (int b = 0; b < 2; ++b) cut_tail(xl[ks][b], ks); } } \
        RING_WAIT(W0);                                                                                                 \
        RING_BARRIER();                                                                                                \
        mma(wl, xl, 0, 0);                                                                                             \
        RING_BARRIER();                                                                                                \
        read_x(xh, q2);                                                                                                \
        if (NI > 1) issue(2, s + 2, q);                                                                                \
        if (KTAIL && LAST) { _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) { _Pragma("unroll") for (int b = 0; b < 2; ++b) cut_tail(xh[ks][b], ks); } } \
        RING_WAIT(W1);                                                                                                 \
        RING_BARRIER();                                                                                                \
        mma(wl, xh, 0, 2);                                                                                             \
        RING_BARRIER();                                                                                                \
        read_w(wh, q2 + GRANULE);                                                                                      \
        if (NI > 2) issue(3, s + 2, q + GRANULE);                                                                      \
        if (KTAIL && LAST) { _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) { _Pragma("unroll") for (int a = 0; a < 4; ++a) cut_tail(wh[ks][a], ks); } } \
        RING_WAIT(W2);                                                                                                 \
        RING_BARRIER();                                                                                                \
        mma(wh, xh, 4, 2);                                                                                             \
        RING_BARRIER();                                                                                                \
        if (!(LAST)) read_w(wl, q4);                                                                                   \
        if (NI > 3) issue(0, s + 3, q2);                                                                               \
        RING_WAIT(W3);                                                                                                 \
        RING_BARRIER();                                                                                                \
        mma(wh, xl, 4, 0);                                                                                             \
        RING_READS_RETURNED();                                                                                         \
        RING_BARRIER();                                                                                                \
        q = q4;                                                                                                        \
        ++s;                                                                                                           \
    }
    while (s < stages - 3) RING_STAGE(4, 14, 14, 14, 14, false)
    // the last three stages: the last loads go out in the first of them
    RING_STAGE(3, 14, 14, 14, 12, false)
    RING_STAGE(0, 10, 8, 6, 4, false)
    RING_STAGE(0, 2, 0, 0, 0, true)
    if (wave < 4) RING_BARRIER();
#undef RING_STAGE
#undef RING_BARRIER
#undef RING_WAIT
#undef RING_WAIT_
#undef RING_READS_RETURNED

    // ---- adapter deltas of this wavefront's 64 tokens -----------------------
    if constexpr (DELTA) {
        // token of MFMA column l16 of token block b
        int tokb[WX];
#pragma unroll
        for (int b = 0; b < WX; ++b) tokb[b] = __shfl(my_tok, 16 * b + l16);
        // acc += Bt_a[features, ranks] x v[tokens in `members`, ranks]^T  (members: bit i = row wt + i of the tile)
        auto apply = [&](int a, uint64_t members, const bf16_t* __restrict__ vb, int R) {
            const int r = da.rank[a];
            const char* Bt = reinterpret_cast<const char*>(da.Bt_ptrs[a]);
            const int row = n0 + wn + frow;                          // feature of MFMA row l16 in block 0
            for (int j0 = 0; j0 < r; j0 += 32) {
                const int j = j0 + 8 * kg;                           // this lane's 8 ranks of the block
                const bool in = j < r;                               // r % 8 == 0: all eight or none
                const uint32_t lane_off = (uint32_t)(row * r + j) * 2u;
                // all loads of the block go out before the first is waited for (no branch between them)
                op16 wb[WA], vh[WX], vl[WX];
#pragma unroll
                for (int blk = 0; blk < WA; ++blk) {
                    const int d = (blk >> 2) * 64 + (blk & 3) * 4;   // block blk holds the features row + d
                    wb[blk].u = (in && row + d < N) ? ldg16_off(Bt + (int64_t)d * r * 2, lane_off) : uint4{0, 0, 0, 0};
                }
#pragma unroll
                for (int b = 0; b < WX; ++b) {
                    const bool mine = in && ((members >> (16 * b + l16)) & 1ull);
                    const uint32_t off = (uint32_t)(tokb[b] * 2 * R + j) * 2u;   // (the launcher keeps T R 4 below 2^32)
                    vh[b].u = mine ? ldg16_off(vb, off) : uint4{0, 0, 0, 0};
                    vl[b].u = mine ? ldg16_off(vb, off + (uint32_t)R * 2u) : uint4{0, 0, 0, 0};
                }
#pragma unroll
                for (int b = 0; b < WX; ++b) {
                    const uint64_t in16 = (members >> (16 * b)) & 0xffffull;      // wavefront-uniform
                    if (in16 == 0) continue;
                    const bool mine = (in16 >> l16) & 1ull;
#pragma unroll
                    for (int blk = 0; blk < WA; ++blk) {
                        floatx4 e = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[blk].v, vh[b].v, acc[blk][b], 0, 0, 0);
                        e = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[blk].v, vl[b].v, e, 0, 0, 0);
                        // (a product with zeros would carry the adapter's infinities over to other tokens)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[blk][b][i] = mine ? e[i] : acc[blk][b][i];
                    }
                    __builtin_amdgcn_sched_barrier(0);               // (one block of tokens at a time, or registers spill)
                }
            }
        };
        const int own = my_key & KEY_NONE;
        uint64_t todo = __ballot(own != KEY_NONE);
        while (todo) {                                               // the distinct adapters among the 64 tokens
            const int a = __builtin_amdgcn_readlane(own, __ffsll((unsigned long long)todo) - 1);
            const uint64_t members = __ballot(own == a);
            todo &= ~members;
            apply(a, members, da.vb, da.R);
        }
        const uint64_t removal = __ballot((my_key & STAGE_REMOVAL) != 0);
        if (removal) apply(da.merged, removal, da.vb2, da.R2);     // mixture mode: the merged adapter, negated, for all of them
    }

    // ---- epilogue: one rounding, store (rows go back to their tokens) ------
#pragma unroll
    for (int b = 0; b < WX; ++b) {
        const int pos = t0 + wt + b * 16 + l16;
        if (pos >= T) continue;
        const int t = DELTA ? da.order[pos] : pos;
#pragma unroll
        for (int G = 0; G < 2; ++G) {
            const int n = n0 + wn + 64 * G + 16 * kg;                // first of this lane's 16 features
            bf16_t* yp = y + (int64_t)t * ldy + n;
            // feature offset 4 q + i is element i of block 4 G + q
            if (n + 16 <= N) {
                uint32_t o[8];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[2 * q] = (uint32_t)f32_to_bf16(acc[4 * G + q][b][0]) | ((uint32_t)f32_to_bf16(acc[4 * G + q][b][1]) << 16);
                    o[2 * q + 1] = (uint32_t)f32_to_bf16(acc[4 * G + q][b][2]) | ((uint32_t)f32_to_bf16(acc[4 * G + q][b][3]) << 16);
                }
                *reinterpret_cast<uint4*>(yp) = uint4{o[0], o[1], o[2], o[3]};
                *reinterpret_cast<uint4*>(yp + 8) = uint4{o[4], o[5], o[6], o[7]};
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (n + i < N) yp[i] = f32_to_bf16(acc[4 * G + (i >> 2)][b][i & 3]);
            }
        }
    }
}

// v (sum of its K parts, fp32) -> two bf16 terms hi + lo, rows [t][0][R] and [t][1][R] of vb; one wavefront per token
__global__ __launch_bounds__(256) void v_split_kernel(
    const int32_t* __restrict__ perm, int n_active, const int32_t* __restrict__ token_adapter, const int32_t* __restrict__ rank,
    const float* __restrict__ v, lora_vspec vsp, bf16_t* __restrict__ vb)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= n_active) return;
    const int t = perm[row];
    const int r = rank[token_adapter[t]];
    for (int j = threadIdx.x & 63; j < r; j += 64) {
        float f = v[(int64_t)t * vsp.R + j];
        for (int q = 1; q < vsp.P; ++q) f += v[q * vsp.part + (int64_t)t * vsp.R + j];
        const bf16_t hi = f32_to_bf16(f);
        vb[(int64_t)t * 2 * vsp.R + j] = hi;
        vb[(int64_t)t * 2 * vsp.R + vsp.R + j] = f32_to_bf16(f - bf16_to_f32(hi));
    }
}

template <int WB, bool DELTA, bool KTAIL>
hipError_t launch_one(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                      void* y, int64_t ldy, const gemm_delta_args& da, hipStream_t stream)
{
    constexpr int BM = 64 * WB;
    const int tiles_n = (N + BM - 1) / BM, tiles_t = (T + BM - 1) / BM;
    const size_t lds_bytes = (size_t)2 * 2 * BM * 8 * sizeof(uint4) +
                             (DELTA ? META_MAX * sizeof(uint4) + (size_t)(BM * 8 / 256) * 256 * sizeof(int2) : 0);
    static std::atomic<bool> attr_set{false};                 // dynamic LDS above 64 KB has to be allowed once per kernel
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiled_kernel<WB, DELTA, KTAIL>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    LORA_LAUNCH(DELTA ? LORA_K_GEMM_TILED_DELTA : LORA_K_GEMM_TILED, (gemm_tiled_kernel<WB, DELTA, KTAIL>),
                dim3(tiles_n * tiles_t), dim3(256), lds_bytes, stream, T, K, N, (const bf16_t*)x, ldx, (const bf16_t*)Wt, ldw,
                (bf16_t*)y, ldy, tiles_n, tiles_t, da);
    return hipGetLastError();
}

template <bool DELTA, bool KTAIL>
hipError_t launch_ring(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                       void* y, int64_t ldy, const gemm_delta_args& da, hipStream_t stream)
{
    const int tiles_n = (N + 255) / 256, tiles_t = (T + 255) / 256;
    const size_t lds_bytes = (size_t)GRANULES * GRANULE;
    static std::atomic<bool> attr_set{false};                 // dynamic LDS above 64 KB has to be allowed once per kernel
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_ring_kernel<DELTA, KTAIL>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    LORA_LAUNCH(DELTA ? LORA_K_GEMM_RING_DELTA : LORA_K_GEMM_RING, (gemm_ring_kernel<DELTA, KTAIL>),
                dim3(tiles_n * tiles_t), dim3(512), lds_bytes, stream, T, K, N, (const bf16_t*)x, ldx, (const bf16_t*)Wt, ldw,
                (bf16_t*)y, ldy, tiles_n, tiles_t, da);
    return hipGetLastError();
}

}  // namespace

bool gemm_tiled_supported(int32_t T, int32_t K, int32_t N, int32_t dtype, const void* x, int64_t ldx,
                          const void* Wt, int64_t ldw, const void* y, int64_t ldy)
{
    auto mis = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) != 0; };
    if (dtype != LORA_BF16 || T < 1 || N < 1) return false;
    if (K % 8 || ldx % 8 || ldw % 8 || ldy % 8) return false;
    if (mis(x) || mis(Wt) || mis(y)) return false;
    const int64_t tiles = (int64_t)((N + 127) / 128) * ((T + 127) / 128);
    return tiles < (1ll << 31);
}

// The ring kernel: at least three stages of 64 k; rows of W and x addressed by 32-bit byte offsets
static bool ring_takes(int32_t T, int32_t K, int32_t N, int64_t ldx, int64_t ldw)
{
    return K > 2 * RK && (int64_t)N * ldw * 2 < (1ll << 32) && (int64_t)T * ldx * 2 < (1ll << 32);
}

// (the planner, which orders the rows, knows no kernels)
static bool product_by_stage_lists(const lora_plan* p)
{
    return gemm_route(p->T, p->K, p->N, p->K, p->K, true, true) == GEMM_TILED && !ring_takes(p->T, p->K, p->N, p->K, p->K);
}
namespace {
struct install_by_stage_lists { install_by_stage_lists() { lora_product_by_stage_lists = product_by_stage_lists; } } g_install_by_stage_lists;
}  // namespace

// p != nullptr: fold the adapter delta in; v holds the shrink's output and vb (room for T*2*R bf16) receives its split
// (split_done: the shrink has written it already);
// rm: likewise for the removal of the merged adapter (mixture mode)
hipError_t launch_gemm_tiled(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx,
                             const void* Wt, int64_t ldw, void* y, int64_t ldy,
                             const lora_plan* p, const lora_dev_tables* d, const float* v, void* vb, bool split_done,
                             const gemm_removal& rm, const void* const* Bt, hipStream_t stream, gemm_route_id route)
{
    const bool delta = p && (!p->perm.empty() || rm.plan);
    // (the ring kernel's delta part has 32-bit byte offsets of the split of v, too.)  The register-staged kernel takes what the
    // ring does not: 256 x 256 tiles once there are enough of them to fill the 256 compute units
    const bool ring_ok = route == GEMM_TILED && ring_takes(T, K, N, ldx, ldw) &&
                         (!delta || ((int64_t)T * p->R * 4 < (1ll << 32) && (!rm.plan || (int64_t)T * rm.plan->R * 4 < (1ll << 32))));
    const bool big = route == GEMM_TILED && (int64_t)((N + 255) / 256) * ((T + 255) / 256) >= 192;
    gemm_delta_args da{};
    if (delta) {
        // the bf16 split of v, unless the shrink has written it already
        if (!split_done && !p->perm.empty()) {
            LORA_LAUNCH(LORA_K_V_SPLIT, v_split_kernel, dim3((unsigned)(p->perm.size() + 3) / 4), dim3(256), 0, stream,
                        d->perm, (int)p->perm.size(), d->token_adapter, d->rank, v, lora_vspec_of(p), (bf16_t*)vb);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        if (!rm.split_done && rm.plan) {
            LORA_LAUNCH(LORA_K_V_SPLIT, v_split_kernel, dim3((unsigned)(rm.plan->perm.size() + 3) / 4), dim3(256), 0, stream,
                        rm.tables->perm, (int)rm.plan->perm.size(), rm.tables->token_adapter, rm.tables->rank, rm.v,
                        lora_vspec_of(rm.plan), (bf16_t*)rm.vb);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        da = gemm_delta_args{d->order, d->row_key, d->rank,
                             big ? d->extra_ptr256 : d->extra_ptr128,
                             big ? d->extra256 : d->extra128, (const bf16_t*)vb, p->R,
                             (const bf16_t* const*)Bt, (const bf16_t*)d->zeros,
                             (const bf16_t*)rm.vb, rm.plan ? rm.plan->R : 0, rm.plan ? p->merged : -1};
    }
    const bool ktail = (K % BK) != 0;
    if (ring_ok) {
#define RING_DISPATCH(D_, KT_) launch_ring<D_, KT_>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)
        if (delta) return ktail ? RING_DISPATCH(true, true) : RING_DISPATCH(true, false);
        return ktail ? RING_DISPATCH(false, true) : RING_DISPATCH(false, false);
#undef RING_DISPATCH
    }
#define GEMM_DISPATCH(WB_, D_, KT_) launch_one<WB_, D_, KT_>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)
    if (big) {
        if (delta) return ktail ? GEMM_DISPATCH(4, true, true) : GEMM_DISPATCH(4, true, false);
        return ktail ? GEMM_DISPATCH(4, false, true) : GEMM_DISPATCH(4, false, false);
    }
    if (delta) return ktail ? GEMM_DISPATCH(2, true, true) : GEMM_DISPATCH(2, true, false);
    return ktail ? GEMM_DISPATCH(2, false, true) : GEMM_DISPATCH(2, false, false);
#undef GEMM_DISPATCH
}
