// Base GEMM y = x W (+ adapter deltas) of small batches (bf16) and of every fp32 batch: the contraction is split over
// the wavefronts of a workgroup instead of over workgroups.
//
// A batch of T tokens with few of them is bound by reading W once, and the 128 x 128 tiles of the other GEMM kernels
// leave most compute units without any: 64 tokens x 4096 features are 32 workgroups, each walking the whole K alone.
// Here a workgroup (8 wavefronts) owns 16 FB features x 16 TB tokens, its wavefronts take contiguous slices of K, and
// the partial sums meet in LDS: the chip is full from N = 4096 features on (FB = 1: 256 workgroups), no partial sum
// ever goes to memory and no second launch is needed.  Nothing is shared between the wavefronts (each has its own k
// range), so the K loop needs no barrier: D units of 128 bytes per row are in flight per wavefront, through its own part
// of LDS.
//
// fp32 runs on v_mfma_f32_16x16x4_f32 the same way (fp32 products and sums); there the matrix cores bind (256
// flops/clk per compute unit) and the same tiles serve every batch size.
//
// Measured (whole lora_fused_forward): 64 single-token requests on 32 adapters, 4096 -> 4096, 104 -> 15.6 us, 22.5 where all
// of W comes from memory; fp32, 256 tokens, 4096 -> 4096: this kernel 600 -> 73 us (the matrix cores' share of that at 2.1 GHz
// is 64 us).
//
// DELTA: tokens in the plan's row order; before the partial sums are added up, the wavefronts share out the deltas of the
// tile's tokens and add v B_a of theirs to their own partial sums, so the delta is spread over the workgroup and joins the same
// fp32 sum.  Two ways to share out (deltas_in_items chooses): items (16-token block, adapter in it, rank step), or pairs
// (adapter, rank step) over all blocks.  The delta costs trips to memory: an item's operands are requested one item ahead, the
// first item's beside the K loop (32 tokens on 32 adapters, 4096 -> 11008: kernel 32.5 -> 30.0 us; 64 tokens, 5120 -> 13824:
// 52.1 -> 45.8; the product alone takes 21 and 35).  The shrink goes in the same launch where layer_small_planned says so.
// v is read as the shrink left it (fp32, K parts added in order); with bf16 it is split into two bf16 terms in registers, or,
// for ranks off the tuned kernels, multiplied as it is (fp32 products: 64 tokens on 32 adapters of ranks 4 to 100, 4096 ->
// 4096, 25.3 us, with two terms 24.1).
#include <algorithm>
#include <atomic>

#include "kernels.h"
#include "launch.h"
#include "split_k.h"

namespace {

// Hand-off of v inside a launch (layer_small_kernel).  Shrink workgroup b counts itself in slot b % 16 of `done` when its
// part of v is published, product workgroup b in slot b % 16 of `through` when it has no more use for v; neither is ever
// reset.  A product workgroup that is not through itself divides its slot of `through` by that slot's workgroups and has
// the number of launches before this one, so it knows what every slot of `done` will read when all of v is there.
// Shrink workgroups wait for nothing and start first.  The wait for them is bounded in time: after wait_ticks of the
// device's wall clock a wavefront computes the rows of v that it needs itself, from x and At.
constexpr int kSyncSlots = 16;
struct layer_sync_slot {         // a cache line of its own
    unsigned long long done, through;
    unsigned long long pad[14];
};
static_assert(sizeof(layer_sync_slot) * kSyncSlots == LORA_LAYER_SYNC_BYTES, "size of the slots in a plan's device tables");
__host__ __device__ constexpr int workgroups_of_slot(int n, int slot) { return (n + kSyncSlots - 1 - slot) / kSyncSlots; }

struct shrink_args {
    const lora_tile* tiles;      // list_parts K parts each, next to each other; here `parts` of them
    const int32_t* perm;
    const float* scale;
    const bf16_t* const* At_ptrs;
    layer_sync_slot* sync;
    int n_wg, parts, list_parts;
    long long wait_ticks;
};

__device__ __forceinline__ unsigned long long ld_agent(const void* p)
{
    return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One tile of features x tokens.  BY_ITEM: the deltas in items, otherwise in pairs (see there).  HANDOFF: v is published during
// this launch (see above)
template <typename E, int FB, int TB, int D, row_delta DELTA, bool BY_ITEM, bool KTAIL, bool HANDOFF>
__device__ __forceinline__ void gemm_small_tile_of(
    const int wg, int T, int K, int N, const E* __restrict__ x, int64_t ldx, const E* __restrict__ Wt, int64_t ldw,
    E* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, bool y_vec, const row_delta_args& da, const shrink_args& sh)
{
    constexpr int WAVES = 8;
    // workgroups are dealt round-robin to the 8 XCDs; every XCD gets an eighth of the tiles, the token tiles of one feature
    // tile next to each other, so that its W rows come from memory once and are then in that XCD's L2
    const int n_wg = tiles_n * tiles_t, xcd = wg & 7;
    const int tile = xcd * (n_wg / 8) + min(xcd, n_wg % 8) + (wg >> 3);
    const int tile_n = tile / tiles_t, tile_t = tile % tiles_t;
    const int n0 = tile_n * 16 * FB, t0 = tile_t * 16 * TB;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;

    // DELTA: row `lane` of the tile, its adapter (none: KEY_NONE), that adapter's rank and Bt: two rounds of loads that run
    // beside the K loop's first
    int my_tok = 0, my_key = KEY_NONE, my_rank = 0;
    uint64_t my_bt = 0;
    if constexpr (DELTA != NO_DELTA) {
        const int pos = t0 + lane;
        const bool row_in = lane < 16 * TB && pos < T;
        my_tok = da.order[row_in ? pos : T - 1];
        my_key = row_in ? da.row_key[pos] : KEY_NONE;
    }
    const int own = my_key & KEY_NONE;
    // (the launcher keeps N ldw and T ldx below 2^32 bytes)
    using slice = split_k<E, FB, TB, D, KTAIL>;
    constexpr int ES = slice::ES, EPC = slice::EPC, KSTEP = slice::KSTEP;
    slice part(
        K, Wt, x, wave, [&](int row) { return (int64_t)min(n0 + row, N - 1) * ldw; },
        [&](int row) {
            const int r = min(t0 + row, T - 1);
            return (int64_t)(DELTA != NO_DELTA ? da.order[r] : r) * ldx;
        });
    floatx4 (&acc)[FB][TB][1] = part.acc;
    const int u_begin = (int)(((int64_t)part.units * wave) / WAVES), u_end = (int)(((int64_t)part.units * (wave + 1)) / WAVES);
    if (DELTA != NO_DELTA && own != KEY_NONE) {
        my_rank = da.rank[own];
        my_bt = reinterpret_cast<uint64_t>(da.Bt_ptrs[own]);
    }
    part.start(u_begin, u_end);

    // v B of rows `mine` of one 16-token block onto its sums; v as f
    auto add_rows = [&](int b, bool mine, const op16 (&bt)[FB], const float (&f)[EPC]) __attribute__((always_inline)) {
        auto take = [&](auto product) __attribute__((always_inline)) {
#pragma unroll
            for (int w = 0; w < FB; ++w) {
                const floatx4 e = product(bt[w], acc[w][b][0]);
                // (a product with zeros would carry the adapter's infinities over to other tokens)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[w][b][0][i] = mine ? e[i] : acc[w][b][0][i];
            }
        };
        if constexpr (ES == 4) {
            op16 vo;
            vo.f = floatx4{f[0], f[1], f[2], f[3]};
            take([&](const op16& w, floatx4 c) { return mma(w, vo, c, E{}); });
        } else if constexpr (DELTA == PLAIN_DELTA) {
            take([&](const op16& w, floatx4 c) { return mma_plain(w, f, c); });
        } else {
            op16 vo[2];
            bf16_terms<2>(f, vo);
            take([&](const op16& w, floatx4 c) { return mma(w, vo[1], mma(w, vo[0], c, E{}), E{}); });
        }
    };
    if constexpr (DELTA == NO_DELTA) {
        part.drain(u_begin, u_end, [] {}, [] {});
    } else if constexpr (!BY_ITEM) {
        // ---- adapter deltas, in pairs (adapter, KSTEP ranks) over all blocks of the tile, in turn to the wavefronts ----
        part.drain(u_begin, u_end, [] {}, [] {});
        int tokb[TB], turn = 0;
#pragma unroll
        for (int b = 0; b < TB; ++b) tokb[b] = __shfl(my_tok, 16 * b + m);
        auto apply = [&](const E* Bt, int r, uint64_t members, const float* v, const lora_vspec& vsp) {
            for (int j0 = 0; j0 < r; j0 += KSTEP) {
                if ((turn++ & (WAVES - 1)) != wave) continue;
                const int j = j0 + EPC * g;
                op16 bt[FB];
                float vf[TB][EPC];
#pragma unroll
                for (int f = 0; f < FB; ++f) {
                    const int n = n0 + 4 * FB * (m >> 2) + 4 * f + (m & 3);
                    bt[f] = row_chunk<E>(Bt + (int64_t)(n < N ? n : N - 1) * r, j, r);
                }
#pragma unroll
                for (int b = 0; b < TB; ++b) v_values<EPC>(v, vsp, tokb[b], j, r, (members >> (16 * b + m)) & 1ull, vf[b]);
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    if ((members >> (16 * b)) & 0xffffull) add_rows(b, (members >> (16 * b + m)) & 1ull, bt, vf[b]);   // (wavefront-uniform)
            }
        };
        uint64_t todo = __ballot(own != KEY_NONE);
        while (todo) {
            const int src = __ffsll((unsigned long long)todo) - 1, a = __builtin_amdgcn_readlane(own, src);
            const uint64_t bt = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_bt, src) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_bt >> 32), src) << 32);
            const uint64_t members = __ballot(own == a);
            todo &= ~members;
            apply(reinterpret_cast<const E*>(bt), __builtin_amdgcn_readlane(my_rank, src), members, da.v, da.vsp);
        }
        const uint64_t removal = __ballot((my_key & LORA_UNMERGE_BIT) != 0);
        if (removal) apply(reinterpret_cast<const E*>(da.Bt_ptrs[da.merged]), da.rank[da.merged], removal, da.v2, da.vsp2);
    } else {
        // ---- adapter deltas, in items of (16-token block, adapter in it, KSTEP ranks), in turn to the wavefronts; an item's
        // operands are requested before the item before it is multiplied, the first item's inside the K loop ----
        int my_steps = 0, my_end = 0, items = 0, rm_rank = 0, rm_steps = 0;
        uint64_t removal = 0, rm_bt = 0;
        auto share_out = [&]() {
            // the first row of an adapter in its block leads: items [my_end - my_steps, my_end) are its
            const int before = __shfl_up(own, 1);
            const bool leads = own != KEY_NONE && (m == 0 || before != own);
            my_end = my_steps = leads ? (my_rank + KSTEP - 1) / KSTEP : 0;
#pragma unroll
            for (int q = 1; q < 64; q *= 2) {
                const int up = __shfl_up(my_end, q);
                my_end += lane >= q ? up : 0;
            }
            items = __builtin_amdgcn_readlane(my_end, 63);
            // mixture mode: the merged adapter's on every block, masked to the rows that the removal applies to
            removal = HANDOFF ? 0 : __ballot((my_key & LORA_UNMERGE_BIT) != 0);
            if (removal) {
                rm_rank = da.rank[da.merged];
                rm_steps = (rm_rank + KSTEP - 1) / KSTEP;
                rm_bt = reinterpret_cast<uint64_t>(da.Bt_ptrs[da.merged]);
            }
        };
        struct item {                                        // (wavefront-uniform)
            const E* Bt;
            int a, r, j0, block;
            uint32_t rows;                                   // of the block that are the adapter's
            bool rm;
        };
        auto find = [&](int i, item& it) {
            if (i < items) {
                const int src = __ffsll((unsigned long long)__ballot(my_end > i)) - 1, a = __builtin_amdgcn_readlane(own, src);
                it.block = src >> 4;
                it.rows = (uint32_t)(__ballot(own == a) >> (src & 48)) & 0xffffu;
                it.a = a;
                it.r = __builtin_amdgcn_readlane(my_rank, src);
                it.j0 = (i - __builtin_amdgcn_readlane(my_end, src) + __builtin_amdgcn_readlane(my_steps, src)) * KSTEP;
                it.Bt = reinterpret_cast<const E*>((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_bt, src) |
                                                   ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_bt >> 32), src) << 32));
                it.rm = false;
                return true;
            }
            i -= items;
            if (HANDOFF || i >= TB * rm_steps) return false;
            it.block = i / rm_steps;
            it.rows = (uint32_t)(removal >> (16 * it.block)) & 0xffffu;
            it.a = da.merged;
            it.r = rm_rank;
            it.j0 = (i - it.block * rm_steps) * KSTEP;
            it.Bt = reinterpret_cast<const E*>(rm_bt);
            it.rm = true;
            return true;
        };
        // K parts of v that are requested ahead (as many as registers hold; the others when they are used)
        constexpr int AHEAD = ES == 4 || (FB * TB >= 8 && !HANDOFF) ? 4 : 1;
        struct operands {
            op16 bt[FB];
            floatx4 v[AHEAD][EPC / 4];
        };
        // (past a rank's end v and Bt are read where there is something; `add` masks it)
        auto v_at = [&](const item& it) {
            const lora_vspec& vsp = !HANDOFF && it.rm ? da.vsp2 : da.vsp;
            return (!HANDOFF && it.rm ? da.v2 : da.v) + (int64_t)__shfl(my_tok, 16 * it.block + m) * vsp.R + min(it.j0 + EPC * g, vsp.R - EPC);
        };
        auto v_chunk = [&](const float* p) {
            if constexpr (HANDOFF) {
                // (past the caches of this XCD, which may hold what an earlier launch left there)
                const unsigned long long q[2] = {ld_agent(p), ld_agent(p + 2)};
                return floatx4{__uint_as_float((uint32_t)q[0]), __uint_as_float((uint32_t)(q[0] >> 32)),
                               __uint_as_float((uint32_t)q[1]), __uint_as_float((uint32_t)(q[1] >> 32))};
            } else {
                return *reinterpret_cast<const floatx4*>(p);
            }
        };
        bool published = true;                               // (wavefront-uniform)
        auto load_bt = [&](const item& it, operands& o) {
#pragma unroll
            for (int f = 0; f < FB; ++f) {
                const int n = n0 + 4 * FB * (m >> 2) + 4 * f + (m & 3);
                o.bt[f] = row_chunk<E>(it.Bt + (int64_t)(n < N ? n : N - 1) * it.r, it.j0 + EPC * g, it.r);
            }
        };
        auto load_v = [&](const item& it, operands& o) {
            if constexpr (HANDOFF) {
                if (!published) {                            // not seen in time: this lane's ranks of its token, from x and At
                    const float s_a = sh.scale[it.a];
                    const bf16_t* const xr = x + (int64_t)__shfl(my_tok, 16 * it.block + m) * ldx;
                    const bf16_t* const At = sh.At_ptrs[it.a];
#pragma unroll
                    for (int q = 0; q < EPC / 4; ++q) o.v[0][q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (int i = 0; i < EPC; ++i) {
                        const bf16_t* const ar = At + (int64_t)min(it.j0 + EPC * g + i, it.r - 1) * K;
                        float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                        for (int k = 0; k < K; k += 8) {
                            const u32x4 xa = ldg_unaligned(xr + k), aa = ldg_unaligned(ar + k);
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                sum[q] = fmaf(bf16_to_f32((bf16_t)(xa[q] & 0xffffu)), bf16_to_f32((bf16_t)(aa[q] & 0xffffu)), sum[q]);
                                sum[q] = fmaf(bf16_to_f32((bf16_t)(xa[q] >> 16)), bf16_to_f32((bf16_t)(aa[q] >> 16)), sum[q]);
                            }
                        }
                        const float f = s_a * ((sum[0] + sum[1]) + (sum[2] + sum[3]));
#pragma unroll
                        for (int q = 0; q < EPC; ++q) o.v[0][q >> 2][q & 3] = q == i ? f : o.v[0][q >> 2][q & 3];
                    }
                    return;
                }
            }
            const lora_vspec& vsp = !HANDOFF && it.rm ? da.vsp2 : da.vsp;
            const float* const p = v_at(it);
#pragma unroll
            for (int s = 0; s < AHEAD; ++s)
                if (s < vsp.P) {
#pragma unroll
                    for (int q = 0; q < EPC / 4; ++q) o.v[s][q] = v_chunk(p + s * vsp.part + 4 * q);
                }
        };
        auto load = [&](const item& it, operands& o) {
            load_bt(it, o);
            load_v(it, o);
        };
        auto add = [&](const item& it, operands& o) {
            const lora_vspec& vsp = !HANDOFF && it.rm ? da.vsp2 : da.vsp;
            if (HANDOFF && !published) {
                // (the sum itself)
            } else if constexpr (AHEAD > 1) {
#pragma unroll
                for (int s = 1; s < 4; ++s)
                    if (s < vsp.P) {
#pragma unroll
                        for (int q = 0; q < EPC / 4; ++q) o.v[0][q] += o.v[s][q];
                    }
            } else if (vsp.P > 1) {
                const float* const p = v_at(it);
                floatx4 rest[3][EPC / 4];
#pragma unroll
                for (int s = 1; s < 4; ++s)
                    if (s < vsp.P) {
#pragma unroll
                        for (int q = 0; q < EPC / 4; ++q) rest[s - 1][q] = v_chunk(p + s * vsp.part + 4 * q);
                    }
#pragma unroll
                for (int s = 1; s < 4; ++s)
                    if (s < vsp.P) {
#pragma unroll
                        for (int q = 0; q < EPC / 4; ++q) o.v[0][q] += rest[s - 1][q];
                    }
            }
            const bool mine = (it.rows >> m) & 1u;
            float f[EPC];
#pragma unroll
            for (int i = 0; i < EPC; ++i) f[i] = mine && it.j0 + EPC * g + i < it.r ? o.v[0][i >> 2][i & 3] : 0.f;
#pragma unroll
            for (int b = 0; b < TB; ++b)
                if (b == it.block) add_rows(b, mine, o.bt, f);
        };
        item i0, i1;
        operands o0, o1;
        int i = wave;
        bool more = false;
        // HANDOFF: lane l < 16 looks after slot l of `done`
        unsigned long long before = 0, seen = 0;
        const layer_sync_slot* slot = nullptr;
        const int own_slot = wg & (kSyncSlots - 1);
        const auto first = [&] {
            share_out();
            more = find(i, i0);
            if (!more) return;
            if constexpr (HANDOFF) {
                load_bt(i0, o0);
                before = ld_agent(&sh.sync[own_slot].through);
                slot = sh.sync + (lane & (kSyncSlots - 1));
            } else {
                load(i0, o0);
            }
        };
        if constexpr (HANDOFF) {
            part.drain(u_begin, u_end, first, [&] { if (more) seen = ld_agent(&slot->done); });
            if (more) {
                const unsigned long long target =
                    (before / (unsigned)workgroups_of_slot(n_wg, own_slot) + 1) * (unsigned)workgroups_of_slot(sh.n_wg, lane & (kSyncSlots - 1));
                if (sh.wait_ticks == 0) {
                    published = false;                       // (asked for: not even a look)
                } else if (__ballot(seen < target) != 0) {
                    const long long t0 = (long long)wall_clock64();
                    for (;;) {
                        seen = ld_agent(&slot->done);
                        published = __ballot(seen < target) == 0;
                        if (published || (long long)wall_clock64() - t0 >= sh.wait_ticks) break;
                        __builtin_amdgcn_s_sleep(2);
                    }
                }
                // the counts have been seen, so every store of v was acknowledged before; the fence keeps the compiler from
                // moving loads of v up
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                load_v(i0, o0);
            }
        } else if constexpr (ES == 4) part.drain(u_begin, u_end, [] {}, first);  // (a branch in its loop costs the matrix cores more than it hides)
        else part.drain(u_begin, u_end, first, [] {});
        while (more) {
            more = find(i += WAVES, i1);
            if (more) load(i1, o1);
            add(i0, o0);
            if (!more) break;
            more = find(i += WAVES, i0);
            if (more) load(i0, o0);
            add(i1, o1);
        }
    }

    // ---- partial sums meet in LDS, one rounding, store (rows go back to their tokens) ----
    part.park();
    __syncthreads();
    if (HANDOFF && tid == 0)
        __hip_atomic_fetch_add(&sh.sync[wg & (kSyncSlots - 1)].through, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // a thread finishes F4 consecutive blocks (4 F4 consecutive features) of one lane's token
    constexpr int ITEMS = FB * TB * 64, F4 = ITEMS > 512 ? ITEMS / 512 : 1;
    if (wave * F4 >= FB * TB) return;
    const int b = wave * F4 / FB, f0 = wave * F4 % FB;
    floatx4 sum[F4];
#pragma unroll
    for (int f = 0; f < F4; ++f) sum[f] = slice::total(f0 + f, b);
    const int pos = t0 + 16 * b + m;
    if (pos >= T) return;
    const int n = n0 + 4 * FB * g + 4 * f0;
    E* yp = y + (int64_t)(DELTA != NO_DELTA ? da.order[pos] : pos) * ldy + n;
#pragma unroll
    for (int f = 0; f < F4; ++f) {
        if constexpr (ES == 4) {
            if (y_vec && n + 4 * f + 4 <= N) {
                *reinterpret_cast<floatx4*>(yp + 4 * f) = sum[f];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + 4 * f + i < N) yp[4 * f + i] = sum[f][i];
            }
        } else {
            const uint32_t o0 = (uint32_t)f32_to_bf16(sum[f][0]) | ((uint32_t)f32_to_bf16(sum[f][1]) << 16);
            const uint32_t o1 = (uint32_t)f32_to_bf16(sum[f][2]) | ((uint32_t)f32_to_bf16(sum[f][3]) << 16);
            if (n + 4 * f + 4 <= N) {
                *reinterpret_cast<uint2*>(yp + 4 * f) = uint2{o0, o1};            // (ldy % 8 == 0, y 16-byte aligned)
            } else {
                const uint32_t o[2] = {o0, o1};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + 4 * f + i < N) yp[4 * f + i] = (bf16_t)(o[i >> 1] >> (16 * (i & 1)));
            }
        }
    }
}

template <typename E, int FB, int TB, int D, row_delta DELTA, bool BY_ITEM, bool KTAIL>
__global__ __launch_bounds__(512) void gemm_small_kernel(
    int T, int K, int N, const E* __restrict__ x, int64_t ldx, const E* __restrict__ Wt, int64_t ldw,
    E* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, bool y_vec, row_delta_args da)
{
    gemm_small_tile_of<E, FB, TB, D, DELTA, BY_ITEM, KTAIL, false>((int)blockIdx.x, T, K, N, x, ldx, Wt, ldw, y, ldy, tiles_n, tiles_t,
                                                                  y_vec, da, shrink_args{});
}

// A tile of the shrink (16 FB rank rows x 16 tokens x a K part) in a launch that reads v: stored past this XCD's caches,
// counted when the stores are acknowledged.
template <int FB, int D, bool KTAIL>
__device__ __forceinline__ void publish_shrink(const lora_tile& t, int wg, int K, const bf16_t* __restrict__ x, int64_t ldx, float* v,
                                               const lora_vspec& vsp, const shrink_args& sh)
{
    const uint64_t at = reinterpret_cast<uint64_t>(sh.At_ptrs[t.adapter] + (int64_t)t.c0 * K);
    const bf16_t* const At = reinterpret_cast<const bf16_t*>((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at) |
                                                            ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) << 32));
    const int32_t* rows = sh.perm + t.row0;
    const float s_a = __int_as_float(t.reserved1);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kpart = wg % sh.parts;
    using slice = split_k<bf16_t, FB, 1, D, KTAIL>;
    const int units = (K + slice::KUNIT - 1) / slice::KUNIT;
    const int p_begin = units * kpart / sh.parts, p_end = units * (kpart + 1) / sh.parts;
    const auto w_row = [&](int row) { return (int64_t)min(row, t.cn - 1) * K; };
    const auto x_row = [&](int row) { return (int64_t)rows[min(row, t.nrows - 1)] * ldx; };
    slice part(K, At, x, wave, w_row, x_row);
    const int u_begin = p_begin + (p_end - p_begin) * wave / 8, u_end = p_begin + (p_end - p_begin) * (wave + 1) / 8;
    // whole lines to LDS need 16-byte rows, and 32-bit offsets a tile of less than 4 GB
    if ((reinterpret_cast<uintptr_t>(At) & 15) == 0 && (int64_t)t.cn * K * 2 <= (1ll << 32)) part.run(u_begin, u_end);
    else part.run_anywhere(At, x, w_row, x_row, u_begin, u_end);
    part.park();
    __syncthreads();
    const int m = lane & 15, j = 4 * FB * (lane >> 4) + 4 * wave;
    if (wave < FB && m < t.nrows && j < t.cn) {              // (ranks are multiples of 8)
        const floatx4 sum = s_a * slice::total(wave, 0);
        float* const dst = v + kpart * vsp.part + (int64_t)rows[m] * vsp.R + t.c0 + j;
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            const unsigned long long two = (unsigned long long)__float_as_uint(sum[i]) | ((unsigned long long)__float_as_uint(sum[i + 1]) << 32);
            __hip_atomic_store(reinterpret_cast<unsigned long long*>(dst + i), two, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // every storing thread waits for its stores' acknowledgement, then one adds the workgroup to the count
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(&sh.sync[wg & (kSyncSlots - 1)].done, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Shrink and product of a small batch in one launch: workgroups [0, n_wg) of the shrink, then those of the product, which
// need v only behind their K loop.  The shrink alone is a launch of 4 to 7 us that leaves most of the memory rate unused;
// here it runs beside the product's first loads of W (what that gave: layer_small_planned).
template <int FB, int TB, int D, bool KTAIL>
__global__ __launch_bounds__(512) void layer_small_kernel(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, row_delta_args da, float* v, shrink_args sh)
{
    const int wg = (int)blockIdx.x;
    if (wg < sh.n_wg) {
        const lora_tile t = sh.tiles[wg / sh.parts * sh.list_parts];
        if (((t.shape >> 4) & 15) == 1) publish_shrink<1, 2, KTAIL>(t, wg, K, x, ldx, v, da.vsp, sh);
        else publish_shrink<2, 1, KTAIL>(t, wg, K, x, ldx, v, da.vsp, sh);
    } else {
        gemm_small_tile_of<bf16_t, FB, TB, D, TERMS_DELTA, true, KTAIL, true>(wg - sh.n_wg, T, K, N, x, ldx, Wt, ldw, y, ldy, tiles_n,
                                                                              tiles_t, true, da, sh);
    }
}

// dynamic LDS above 64 KB has to be allowed once per kernel
template <typename Kernel>
hipError_t allow_lds(Kernel kernel, size_t bytes, std::atomic<bool>& done)
{
    if (bytes <= 65536 || done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done = true;
    return e;
}

template <typename E, int FB, int TB, int D, row_delta DELTA, bool BY_ITEM, bool KTAIL>
hipError_t launch_one(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw, void* y, int64_t ldy,
                      const row_delta_args& da, hipStream_t stream)
{
    const int tiles_n = (N + 16 * FB - 1) / (16 * FB), tiles_t = (T + 16 * TB - 1) / (16 * TB);
    constexpr size_t lds_bytes = (size_t)8 * D * (2 * FB + 2 * TB) * 1024;
    static_assert(D * (2 * FB + 2 * TB) >= FB * TB && lds_bytes <= 163840, "a wavefront's partial sums go where its operands were");
    static std::atomic<bool> allowed{false};
    const hipError_t e = allow_lds(&gemm_small_kernel<E, FB, TB, D, DELTA, BY_ITEM, KTAIL>, lds_bytes, allowed);
    if (e != hipSuccess) return e;
    LORA_LAUNCH(DELTA != NO_DELTA ? LORA_K_GEMM_SMALL_DELTA : LORA_K_GEMM_SMALL, (gemm_small_kernel<E, FB, TB, D, DELTA, BY_ITEM, KTAIL>),
                dim3((unsigned)(tiles_n * tiles_t)), dim3(512), lds_bytes, stream, T, K, N, (const E*)x, ldx, (const E*)Wt, ldw,
                (E*)y, ldy, tiles_n, tiles_t, ldy % 4 == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0, da);
    return hipGetLastError();
}

// Tile (FB, TB) and units in flight D of a problem.  A compute unit is bound by what it loads, (16 FB + 16 TB) K
// elements per workgroup at about 100 GB/s, fp32 also by its matrix cores (256 flops/clk), and the launch by the
// compute unit with the most workgroups; the largest tile among the cheapest is taken.  Measured, bf16, N = K = 4096,
// microseconds (the tile this picks, then the nearest other): 16 tokens (1,1) 8.3, (1,2) 8.6; 32: (1,2) 9.7, (1,1) 11.4;
// 64: (2,2) 11.6, (1,4) 12.8; 128: (2,4) 15.6, (2,2) 18.5; 256: (4,4) 19.4, (2,4) 27.0.  One unit in flight is enough
// where two or more workgroups share a compute unit; (1,1) has room for more.
struct small_tile { int fb, tb; };
constexpr small_tile kSmallTiles[] = {{4, 4}, {2, 4}, {4, 2}, {2, 2}, {4, 1}, {1, 2}, {1, 1}};

double small_cost(const small_tile& t, int32_t T, int32_t K, int32_t N, int32_t dtype)
{
    const int64_t wgs = (int64_t)((N + 16 * t.fb - 1) / (16 * t.fb)) * ((T + 16 * t.tb - 1) / (16 * t.tb));
    const int64_t rounds = (wgs + 255) / 256;
    const double es = dtype == LORA_F32 ? 4.0 : 2.0;
    const double load = (t.fb + t.tb) * 16.0 * es / 100e9, math = t.fb * t.tb * 512.0 / (dtype == LORA_F32 ? 0.54e12 : 8.6e12);
    return rounds * (double)K * std::max(load, math);
}

small_tile choose_small_tile(int32_t T, int32_t K, int32_t N, int32_t dtype)
{
    small_tile best = kSmallTiles[0];
    for (const small_tile& t : kSmallTiles)
        if (small_cost(t, T, K, N, dtype) < small_cost(best, T, K, N, dtype)) best = t;
    return best;
}

// bf16 deltas in items or in pairs.  An item covers one block: its operands are requested one item ahead, the first ones beside
// the K loop, but an adapter's part of Bt is read again for every block it is in.  A pair reads it once for the whole tile, and
// nothing of it holds the K loop up.  Items where the tiles hold more than four adapters each, few of them in more than one
// block, of short ranks (up to 2.5 steps on average) -- of longer ones in 64-token tiles with more than twelve items for each
// wavefront --, and 32 features or more.  Microseconds of lora_fused_forward, pairs / items, 4096 -> 4096: 100 tokens on 100
// adapters of rank 8 38.7 / 28.2, of rank 128 76 / 60; mixture mode, 470 tokens on 128 of rank 16 86.5 / 64.5; 310 tokens on
// 16 of rank 100 67.3 / 75.3; 25 tokens on 32 of rank 128, mixture mode, 38.0 / 39.3; 1024 -> 4096, 197 tokens on 4 of rank 100
// 20.5 / 23.6, 120 on 128 of rank 256 103 / 70; 4096 -> 1024, one token of rank 4 9.7 / 10.9.
// Of 2300 calls (1 to 700 tokens, ranks 4 to 256, with and without mixture mode) items alone made 385 slower than they were with
// pairs alone by more than 3 %, up to 1.20 times; this rule 10, up to 1.09 times.
bool deltas_in_items(const lora_plan* p, const small_tile& t)
{
    if (t.fb == 1 || p->perm.empty()) return false;
    const int64_t groups = (int64_t)p->group_adapter.size(), tokens = (int64_t)p->perm.size(), rows = 16 * t.tb;
    const int64_t runs = groups + tokens / rows, block_runs = groups + tokens / 16;      // (adapter, tile) and (adapter, block), about
    const int64_t tiles = (tokens + rows - 1) / rows;
    if (2 * p->rank_steps > 5 * groups) return t.tb == 4 && runs * p->rank_steps > 96 * tiles * groups;
    return runs > 4 * tiles && 2 * block_runs <= 3 * runs;
}

template <typename E, row_delta DELTA, bool KTAIL>
hipError_t launch_tile(const small_tile& t, bool items, int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                       void* y, int64_t ldy, const row_delta_args& da, hipStream_t stream)
{
    constexpr bool MAY = DELTA != NO_DELTA, MUST = MAY && sizeof(E) == 4;                // (items; FB = 1: see deltas_in_items)
#define SMALL_TILE(FB_, TB_, D_)                                                                                                          \
    if (t.fb == FB_ && t.tb == TB_)                                                                                                       \
        return MUST || (items && MAY && FB_ > 1)                                                                                          \
                   ? launch_one<E, FB_, TB_, D_, DELTA, MUST || (MAY && FB_ > 1), KTAIL>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)    \
                   : launch_one<E, FB_, TB_, D_, DELTA, MUST, KTAIL>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream);
    SMALL_TILE(4, 4, 1) SMALL_TILE(2, 4, 1) SMALL_TILE(4, 2, 1) SMALL_TILE(2, 2, 1) SMALL_TILE(4, 1, 1) SMALL_TILE(1, 2, 1) SMALL_TILE(1, 1, 2)
#undef SMALL_TILE
    return hipErrorInvalidValue;
}

}  // namespace

bool gemm_small_supported(int32_t T, int32_t K, int32_t N, int32_t dtype, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                          const void* y, int64_t ldy)
{
    auto mis = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) != 0; };
    const int64_t es = dtype == LORA_F32 ? 4 : 2, epc = 16 / es;
    // (fp32 of less than one unit per row is the general kernel's: 1019 tokens, 4 -> 2600, 9.0 us, here 14.3; 386, 12 -> 3728
    // 5.6, here 10.0; 1487, 20 -> 1056 9.1, here 9.3)
    if (dtype == LORA_F32 && K < 32) return false;
    if (T < 1 || N < 1 || K % epc || ldx % epc || ldw % epc || mis(x) || mis(Wt)) return false;
    if (dtype == LORA_BF16 && (ldy % 8 || mis(y))) return false;
    if ((int64_t)N * ldw * es >= (1ll << 32) || (int64_t)T * ldx * es >= (1ll << 32)) return false;      // 32-bit byte offsets
    return (int64_t)((N + 15) / 16) * ((T + 15) / 16) < (1ll << 31);
}

// microseconds (measured: 1.35 times the bound, and a start for every workgroup a compute unit gets; see gemm_route)
double gemm_small_time(int32_t T, int32_t K, int32_t N)
{
    const small_tile t = choose_small_tile(T, K, N, LORA_BF16);
    const int64_t wgs = (int64_t)((N + 16 * t.fb - 1) / (16 * t.fb)) * ((T + 16 * t.tb - 1) / (16 * t.tb));
    return 1.35e6 * small_cost(t, T, K, N, LORA_BF16) + 1.0 + 0.75 * ((wgs + 255) / 256);
}

int32_t gemm_small_tile(int32_t T, int32_t K, int32_t N, int32_t dtype)
{
    const small_tile t = choose_small_tile(T, K, N, dtype);
    return t.fb << 8 | t.tb;
}

// p != nullptr: fold the adapter delta in; v holds the shrink's output.  rm: likewise for the removal of the merged
// adapter (mixture mode).  The plan has its row order (p->order) where there is any delta.
hipError_t launch_gemm_small(int32_t T, int32_t K, int32_t N, int32_t dtype, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                             void* y, int64_t ldy, const lora_plan* p, const lora_dev_tables* d, const float* v,
                             const gemm_removal& rm, const void* const* Bt, hipStream_t stream)
{
    const bool delta = p && (!p->perm.empty() || rm.plan);
    const bool ktail = K % (dtype == LORA_F32 ? 32 : 64) != 0;
    const small_tile t = choose_small_tile(T, K, N, dtype);
    const row_delta_args da = delta ? row_deltas_of(p, d, v, rm, Bt) : row_delta_args{};
    const bool items = delta && deltas_in_items(p, t);
#define SMALL_LAUNCH(E_, D_, KT_) launch_tile<E_, D_, KT_>(t, items, T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)
#define SMALL_DISPATCH(E_, D_) (ktail ? SMALL_LAUNCH(E_, D_, true) : SMALL_LAUNCH(E_, D_, false))
    if (dtype == LORA_F32) return delta ? SMALL_DISPATCH(float, PLAIN_DELTA) : SMALL_DISPATCH(float, NO_DELTA);
    if (!delta) return SMALL_DISPATCH(bf16_t, NO_DELTA);
    return p->extra_ptr256.empty() ? SMALL_DISPATCH(bf16_t, PLAIN_DELTA) : SMALL_DISPATCH(bf16_t, TERMS_DELTA);
#undef SMALL_DISPATCH
#undef SMALL_LAUNCH
}

namespace {
// Shrink and product in one launch: the shrink's tiles, and the K parts of each.  Few tiles are a long chain each, many take
// compute units from the product, and a second part is another trip to memory for each of its items.  Microseconds with 1 / 2 /
// 4 parts, 4096 -> 4096: 4 tiles (one token) 10.9 / 9.9 / 9.2, 16 (8 tokens) 12.3 / 11.8 / 12.3, 60 (32 tokens) 16.5 / 16.1 /
// 23.3; 30 tiles, 4096 -> 11008, 24.6 / 26.4 / 30.3
int layer_parts(const lora_plan* p, int64_t tiles)
{
    int parts = 1;
    while (parts < p->v_parts && 2 * parts * tiles <= 32) parts *= 2;
    return parts;
}

// Whether shrink and product of a small batch go in one launch, the shrink in so many tiles.  Microseconds of
// lora_fused_forward, two launches / one; requests of one token: 64 tokens on 32 adapters, 4096 -> 4096, 18.7 / 15.3; one
// token 12.0 / 9.2; 16 tokens, 4096 -> 11008, 28.1 / 23.6; 12 tokens, 13824 -> 5120, 44.8 / 35.9; 90 tokens on 64 adapters,
// 4096 -> 11008, 72.4 / 63.0; 160 tokens, 4096 -> 4096, 23.9 / 17.8; 256 on 256 adapters of ranks 8 to 64 50.4 / 45.8; longer
// ones: 64 tokens, rank 64, 18.4 / 12.1; 256 tokens, rank 128, 31.7 / 26.2.  Not
//  - on the 32 x 64 tiles: of those a compute unit holds one workgroup, and they come where there is one for each, so some
//    start only behind the shrink (100 tokens on 100 adapters of rank 8, 22.5 / 23.2; on 64 of rank 64 35.5 / 34.4)
//  - on tiles that a compute unit holds two of, where shrink and product together are more than that: those of the product that
//    start behind the shrink then share a compute unit with one that is under way (64 tokens on 64 adapters of rank 128, 4096 ->
//    4096, 47.2 / 66.3; 62 on 64, 2048 -> 2048, 34.2 / 45.8; 228 on 256 of rank 64, 4096 -> 1024, 38.9 / 51.4)
//  - on the 16 x 16 tiles with more than 48 tiles of the shrink: a product of 10 us ends before they do (51 tokens on 32
//    adapters of rank 64, 4096 -> 1024, 17.8 / 19.3)
// Of 4000 calls of up to 700 tokens, ranks 8 to 128, the choice takes 0.2 % longer than the better of the two on average; the
// most, 1.17 times, on the largest tiles with three times as many workgroups of the shrink as compute units, and 1.11 times
// where the product's workgroups just fill the chip and a few of them start behind the shrink.
bool layer_takes(const lora_plan* p, int64_t tiles)
{
    if (tiles == 0 || p->dtype != LORA_BF16 || p->family != LORA_VARIANT_TILED || p->unmerge || p->is_removal || p->extra_ptr256.empty() ||
        (int32_t)p->order.size() != p->T || gemm_route(p->T, p->K, p->N, p->K, p->K, true, true) != GEMM_SMALL)
        return false;
    const small_tile t = choose_small_tile(p->T, p->K, p->N, LORA_BF16);
    if (t.fb * t.tb >= 8) return !(t.fb == 2 && t.tb == 4);
    if (t.fb == 1 && t.tb == 1 && tiles > 48) return false;
    const int64_t product = (int64_t)((p->N + 16 * t.fb - 1) / (16 * t.fb)) * ((p->T + 16 * t.tb - 1) / (16 * t.tb));
    return product + tiles * layer_parts(p, tiles) <= (product + 511) / 512 * 512;
}
// (the planner, which makes the tiles, knows no kernels)
struct install_layer_takes { install_layer_takes() { lora_layer_takes = layer_takes; } } g_install_layer_takes;
}  // namespace

bool layer_small_planned(const lora_plan* p)
{
    return layer_takes(p, p->shrink_small ? (int64_t)p->shrink_tiles.size() / p->v_parts : (int64_t)p->layer_shrink_tiles.size());
}

namespace {
template <int FB, int TB, int D, bool KTAIL>
hipError_t launch_layer_one(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw, void* y, int64_t ldy,
                            const row_delta_args& da, float* v, const shrink_args& sh, hipStream_t stream)
{
    const int tiles_n = (N + 16 * FB - 1) / (16 * FB), tiles_t = (T + 16 * TB - 1) / (16 * TB);
    // (the shrink's widest: 8 KB a wavefront)
    constexpr size_t lds_bytes = std::max<size_t>((size_t)8 * D * (2 * FB + 2 * TB) * 1024, 65536);
    static std::atomic<bool> allowed{false};
    const hipError_t e = allow_lds(&layer_small_kernel<FB, TB, D, KTAIL>, lds_bytes, allowed);
    if (e != hipSuccess) return e;
    LORA_LAUNCH(LORA_K_LAYER_SMALL, (layer_small_kernel<FB, TB, D, KTAIL>), dim3((unsigned)(sh.n_wg + tiles_n * tiles_t)), dim3(512), lds_bytes,
                stream, T, K, N, (const bf16_t*)x, ldx, (const bf16_t*)Wt, ldw, (bf16_t*)y, ldy, tiles_n, tiles_t, da, v, sh);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_layer_small(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw, void* y, int64_t ldy,
                              const lora_plan* p, const lora_dev_tables* d, float* v, const void* const* At, const void* const* Bt,
                              hipStream_t stream)
{
    static std::atomic<int> wall_khz[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (wall_khz[dev] == 0) {
        int khz = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) khz = 100000;
        wall_khz[dev] = khz;
    }
    const small_tile t = choose_small_tile(T, K, N, LORA_BF16);
    const int list_parts = p->shrink_small ? p->v_parts : 1, tiles = (int)(p->shrink_small ? p->shrink_tiles : p->layer_shrink_tiles).size() / list_parts;
    const int parts = layer_parts(p, tiles);
    row_delta_args da = row_deltas_of(p, d, v, gemm_removal{}, Bt);
    da.vsp.P = parts;
    const shrink_args sh{p->shrink_small ? d->shrink_tiles : d->layer_shrink_tiles, d->perm, d->scale, (const bf16_t* const*)At,
                         (layer_sync_slot*)d->layer_sync, tiles * parts, parts, list_parts, (long long)p->fused_wait_us * wall_khz[dev] / 1000};
    const bool ktail = K % 64 != 0;
#define LAYER_TILE(FB_, TB_, D_)                                                                                                           \
    if (t.fb == FB_ && t.tb == TB_)                                                                                                        \
        return ktail ? launch_layer_one<FB_, TB_, D_, true>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, v, sh, stream)                            \
                     : launch_layer_one<FB_, TB_, D_, false>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, v, sh, stream);
    LAYER_TILE(4, 4, 1) LAYER_TILE(4, 2, 1) LAYER_TILE(2, 2, 1) LAYER_TILE(4, 1, 1) LAYER_TILE(1, 2, 1) LAYER_TILE(1, 1, 2)
#undef LAYER_TILE
    return hipErrorInvalidValue;
}
