// Base GEMM y = x W (+ adapter deltas) of batches of some hundred to a few thousand tokens (bf16): tiles of 128 tokens x
// 64, 128, 192 or 256 features, for problems that are too few 256 x 256 tiles to give every compute unit one (or that leave a
// last round nearly empty).
//
// A workgroup (8 wavefronts, two per SIMD) has the compute unit's LDS to itself: a ring of S stages of 64 k (whole
// 128-byte lines of 64 WA rows of W and 128 rows of x), filled straight from memory S - 1 stages ahead.  A stage takes 0.51 us
// for WA = 3 (0.43 for WA = 2) with few compute units at work and 0.70 (0.53) with all of them, where the matrix cores need 768
// clk (512), 0.37 us at 2.1 GHz, and the 40 KB (32 KB) of fills 0.38 us at 105 GB/s.  What binds with W from memory is how much
// of it is on its way: 120 KB a compute unit at 60 GB/s, 2 us (5120 -> 5120, 1111 tokens: 66 us, W in the infinity cache 54; a
// ninth wavefront that asks for W's lines ahead took 5 to 15 % off the former and added as much to the latter).
//
// With adapters (DELTA) a wavefront owns 16 WA features x 64 tokens (WA x 4 blocks of v_mfma_f32_16x16x32_bf16).  A phase is
// one k-step of 32: a memory part (the LDS reads of its operands; in a stage's second phase also the loads of
// stage s + S - 1) and a matrix part (4 WA MFMAs), each closed by a barrier.  Wavefronts 4..7 run one part behind
// wavefronts 0..3, with which they share the SIMDs, so one of the two reads LDS while the other issues MFMAs.
//   RAW: stage s + 1 is first read in memory part 2 s + 2; every wavefront has waited for its own loads of it (vmcnt;
//        loads return in order) at the end of its memory part 2 s + 1, one barrier earlier at least.
//   WAR: stage s - 1, last read in memory part 2 s - 1, is overwritten by loads issued in memory part 2 s + 1; the LDS
//        reads of the trailing wavefronts have returned before their MFMAs of phase 2 s - 1 issued, one barrier earlier.
// Without adapters and with more than 24 stages (APART) a wavefront multiplies 32 WA features x 64 tokens, but only one of a
// stage's two k-steps -- a third fewer bytes read from LDS (WA = 3: 29 %; cycles, by counter, with the sums' way 30 and 25) --,
// and the two sums meet in LDS at the end.  A stage is one memory and one matrix part.
//   RAW: as above, with stage s read in memory part s and its successor waited for at that part's end.
//   WAR: stage s - 1 is overwritten by loads issued in memory part s; its reads have returned before the barrier that ends
//        memory part s - 1 (lgkmcnt), the trailing wavefronts' one barrier before the leading ones' part s.
// lora_base_gemm, W in the infinity cache / from memory: 1024 tokens, 4096 -> 4096, 38.4 -> 33.8 / 42.8 -> 40.9 us; 900, 11008 ->
// 4096, 85 -> 75 / 101.  (With adapters the sums' way through LDS takes what it gives: 0.95 to 1.04 times, 40 batches.)  That way
// takes about 0.3 us (WA = 3: 0.5), which short products do not get back.  lora_base_gemm, W from memory, APART / not, mean of
// 60 to 580 drawn products: 2 stages 1.09, 3 1.04, 5 to 8 1.02, 9 to 16 1.005 (WA = 3: 1.02), 21 to 24 0.998 (1.002), 25 to 32
// 0.996 (1.000), above 50 0.99.
// Tiles of 64 features are for products of 21 stages and more that are one round of them (129 to 256 tiles), which leave the small
// kernel a second round of its own: 300 tokens, 4096 -> 4096, 34.1 -> 27.7; 11008 -> 4096 83 -> 72; 100 tokens, 5120 -> 13824,
// 51.7 -> 41.8; 7785 drawn products of 641 to 16000 tokens 0.78 times as long as what they took before, three above 1.03.
// Tiles of 256 features (a ring of three stages) are for what would be a round and a bit of the narrower ones and half a round
// of 256 x 256: 2048 tokens, 4096 -> 4096, 74.3 -> 61.9 us; 1536, 5120 -> 5120, 90.6 -> 76.3; 1428, 13824 -> 5120, 219 -> 165; 1106,
// 5120 -> 13824, 163 -> 139.  All four widths are bound by their fills: with the LDS reads and the MFMAs taken out the same
// launches take 0.95 to 0.98 of their time, without the fills 0.6 (1024 tokens, 4096 -> 4096, 39.0 / 38.4 / 24.1 us), however
// many stages are on their way (two, three or four: the same to 1 %) and whether a stage's loads go out in its memory part or
// between its MFMAs; so what a tile costs is its rows, (64 WA + 128) x 128 bytes a stage, and wider ones fetch less in all.
// The loads are issued from inline assembly, so the compiler does not count them: the waits are written out.
//
// DELTA: tokens in the plan's row order; after the K loop every wavefront adds the deltas of its own 64 tokens: per
// adapter and 32 ranks, Bt_a[its features] and v (as the shrink left it, split into two bf16 terms, or, for ranks off the
// tuned kernels, in fp32 products: 1111 tokens of ranks 100 and 20, 5120 -> 5120, 109 us, with two terms 99) as MFMA operands.
// (v read by every wavefront for itself, step by step behind Bt: lora_fused_forward of 1111 tokens in mixture mode, 5120 ->
// 5120, 113 us; as operands in LDS, Bt a step ahead: 96.  It took 134 in the register-staged 128 x 128 tiles.)
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "kernels.h"
#include "launch.h"
#include "split_k.h"

namespace {

constexpr int MID_TOKENS = 128;

template <int WA, row_delta DELTA, bool APART, bool KTAIL>
__device__ __forceinline__ void gemm_mid_tile(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, const row_delta_args& da)
{
    constexpr int BM = 64 * WA, NL = WA + 2, STAGE = (BM + MID_TOKENS) * 128, S = 163840 / STAGE, XOFF = BM * 128;
    int tile_n, tile_t;
    tile_of_workgroup(blockIdx.x, tiles_n, tiles_t, tile_n, tile_t);
    const int n0 = tile_n * BM, t0 = tile_t * MID_TOKENS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 15, g = lane >> 4;
    // APART: the wavefronts of a SIMD share a quadrant of the tile in the K loop and take one k-step of every stage each; half
    // of its features are a wavefront's own
    static_assert(!APART || DELTA == NO_DELTA, "built without adapters only");
    const int half = wave >> 2, qn = (wave & 1) * 32 * WA;
    const int wn = APART ? qn + half * 16 * WA : (wave & 3) * 16 * WA, wt = (APART ? (wave >> 1) & 1 : half) * 64;   // the wavefront's origin in the tile

    // Loads: 128 bytes of 8 rows each; lane l brings the chunk that belongs in slot l % 8 of row l / 8.  Of W's rows this
    // wavefront brings 8 WA, of x's 16.  (The launcher keeps N ldw and T ldx below 2^32 bytes; rows past the end re-read
    // the last one and are never stored.)  Chunk c of row r lies at slot c ^ f(r), f eight different values over the rows
    // that eight consecutive lanes read.
    uint32_t off[NL], cut[NL];                                       // cut (KTAIL): back from past K to the row's first chunk of the last stage
    const int stages = (K + 63) / 64, last_k = (stages - 1) * 64;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const bool is_w = i < WA;
        const int row = (is_w ? wave * WA + i : wave * 2 + i - WA) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ (is_w ? (row & 3) | (((row / (4 * WA)) & 1) << 2) : row & 7);
        const int pos = min(t0 + row, T - 1);
        const int64_t r = is_w ? min(n0 + row, N - 1) * ldw : (DELTA != NO_DELTA ? da.order[pos] : pos) * ldx;
        off[i] = (uint32_t)(r * 2) + c * 16;
        cut[i] = KTAIL && last_k + c * 8 >= K ? c * 16 : 0;
    }
    // DELTA: row wt + lane of the tile: its adapter (none: KEY_NONE), that adapter's rank and Bt, whether the removal applies;
    // and row 16 wave + m, whose v this wavefront makes operands of
    int my_own = KEY_NONE, my_rank = 0, v_tok = 0, v_rank = 0, v_removal = 0;
    uint64_t my_bt = 0, removal = 0;
    if constexpr (DELTA != NO_DELTA) {
        const int pos = t0 + wt + lane, v_pos = t0 + 16 * wave + m;
        const int key = pos < T ? da.row_key[pos] : KEY_NONE;
        v_tok = da.order[min(v_pos, T - 1)];
        const int v_key = v_pos < T ? da.row_key[v_pos] : KEY_NONE, v_own = v_key & KEY_NONE;
        my_own = key & KEY_NONE;
        removal = __ballot((key & LORA_UNMERGE_BIT) != 0);
        if (my_own != KEY_NONE) {
            my_rank = da.rank[my_own];
            my_bt = reinterpret_cast<uint64_t>(da.Bt_ptrs[my_own]);
        }
        v_rank = v_own != KEY_NONE ? da.rank[v_own] : 0;
        v_removal = (v_key & LORA_UNMERGE_BIT) ? da.rank[da.merged] : 0;
    }
    const char *const wb = reinterpret_cast<const char*>(Wt), *const xb = reinterpret_cast<const char*>(x);
    const uint32_t lds0 = lds_address(small_lds);
    auto issue = [&](int st, uint32_t slot) {
        const bool tail = KTAIL && st == stages - 1;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            load16_to_lds((i < WA ? wb : xb) + (int64_t)st * 128, tail ? off[i] - cut[i] : off[i],
                          lds0 + slot + (i < WA ? (wave * WA + i) * 1024 : XOFF + (wave * 2 + i - WA) * 1024));
    };

    // sums: the wavefront's own features and tokens; APART: then those of the other half of the quadrant, over its k-steps
    constexpr int WQ = APART ? 2 * WA : WA;
    floatx4 acc[WQ][4];
#pragma unroll
    for (int a = 0; a < WQ; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    // operand addresses of k-step 0 (k-step 1: 64 bytes away by XOR); MFMA row 4 q + i of block a is feature 4 WA q + 4 a + i
    const char* const lds_c = reinterpret_cast<const char*>(small_lds);
    const uint32_t rw = (4 * WA * (m >> 2) + (m & 3)) * 128 + (g ^ (m & 7)) * 16;
    const uint32_t rw_half[2] = {rw + wn * 128, rw + (2 * qn + 16 * WA - wn) * 128};
    const uint32_t rx = XOFF + (wt + m) * 128 + (g ^ (m & 7)) * 16;
    op16 w[WQ], xo[4];
    auto read = [&](uint32_t slot, int ks, bool last) {
#pragma unroll
        for (int a = 0; a < WQ; ++a) w[a].u = *reinterpret_cast<const u32x4*>(lds_c + (slot + (rw_half[a / WA] ^ (ks * 64))) + a % WA * 512);
#pragma unroll
        for (int b = 0; b < 4; ++b) xo[b].u = *reinterpret_cast<const u32x4*>(lds_c + (slot + (rx ^ (ks * 64))) + b * 2048);
        if (KTAIL && last && last_k + (ks * 4 + g) * 8 >= K) {
#pragma unroll
            for (int a = 0; a < WQ; ++a) w[a].u = u32x4{0, 0, 0, 0};
#pragma unroll
            for (int b = 0; b < 4; ++b) xo[b].u = u32x4{0, 0, 0, 0};
        }
    };
    auto multiply = [&]() {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int a = 0; a < WQ; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[a].v, xo[b].v, acc[a][b], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
    };
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto reads_returned = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    // waits until all but the youngest n stages' loads of this wavefront have landed
    auto landed = [&](int n) {
        if (S >= 6 && n >= 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NL) : "memory");
        else if (S >= 5 && n >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NL) : "memory");
        else if (n == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
        else if (n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    for (int st = 0; st < S - 1 && st < stages; ++st) issue(st, st * STAGE);
    landed(min(S - 1, stages) - 1);
    barrier();
    if (wave >= 4) barrier();                                        // the trailing wavefronts: one part behind
    auto next = [](uint32_t slot) { return slot + STAGE == S * STAGE ? 0u : slot + STAGE; };
    uint32_t slot = 0, fill = (S - 1) * STAGE;
    int s = 0;
    for (; s < stages - (S - 1); ++s) {
        read(slot, APART ? half : 0, false);
        if constexpr (APART) {
            issue(s + S - 1, fill);
            reads_returned();
        } else {
            barrier();
            multiply();
            barrier();
            read(slot, 1, false);
            issue(s + S - 1, fill);
        }
        landed(S - 2);
        barrier();
        multiply();
        barrier();
        fill = slot;
        slot = next(slot);
    }
    for (; s < stages; ++s) {                                        // nothing is left to be fetched
        read(slot, APART ? half : 0, s == stages - 1);
        if constexpr (APART) {
            reads_returned();
        } else {
            barrier();
            multiply();
            barrier();
            read(slot, 1, s == stages - 1);
        }
        landed(max(stages - 2 - s, 0));
        barrier();
        multiply();
        barrier();
        slot = next(slot);
    }
    if (wave < 4) barrier();
    if constexpr (APART) {
        // the sums of both k-steps meet: a wavefront hands on the half that is not its own
        __syncthreads();                                             // (the ring has been read)
#pragma unroll
        for (int a = 0; a < WA; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) small_lds[((wave * WA + a) * 4 + b) * 64 + lane] = acc[WA + a][b];
        __syncthreads();
#pragma unroll
        for (int a = 0; a < WA; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] += small_lds[(((wave ^ 4) * WA + a) * 4 + b) * 64 + lane];
    }

    // ---- adapter deltas of this wavefront's 64 tokens: v of the tile's tokens as operands in LDS (a wavefront makes those
    // of one block of 16 tokens), then (adapter, 32 ranks) by (adapter, 32 ranks), Bt one step ahead ----
    if constexpr (DELTA != NO_DELTA) {
        constexpr int VSTEPS = LORA_MAX_RANK / 32;
        op16* const vops = reinterpret_cast<op16*>(small_lds);       // [8 token blocks][VSTEPS][two bf16 terms, or two halves in fp32][64 lanes]
        auto make_operands = [&](const float* v, const lora_vspec& vsp, int r) {
            int rmax = r;
#pragma unroll
            for (int q = 1; q < 16; q *= 2) rmax = max(rmax, __shfl_xor(rmax, q));
            const int steps = (__builtin_amdgcn_readfirstlane(rmax) + 31) / 32;
            const float* const row = v + (int64_t)v_tok * vsp.R;
            auto steps_of = [&](auto parts_t, int s0, int n) {       // n <= 2 steps, all loads first
                constexpr int P = decltype(parts_t)::value;
                floatx4 part[2][P][2];
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (q < n) {
                        const float* p = row + min((s0 + q) * 32 + 8 * g, vsp.R - 8);
#pragma unroll
                        for (int i = 0; i < P; ++i)
#pragma unroll
                            for (int h = 0; h < 2; ++h) part[q][i][h] = *reinterpret_cast<const floatx4*>(p + i * vsp.part + 4 * h);
                    }
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (q < n) {
#pragma unroll
                        for (int i = 1; i < P; ++i)
#pragma unroll
                            for (int h = 0; h < 2; ++h) part[q][0][h] += part[q][i][h];
                        float f[8];
                        op16 o[2];
#pragma unroll
                        for (int i = 0; i < 8; ++i) f[i] = (s0 + q) * 32 + 8 * g + i < r ? part[q][0][i >> 2][i & 3] : 0.f;   // past the rank v holds nothing
                        if constexpr (DELTA == PLAIN_DELTA) {
                            o[0].f = floatx4{f[0], f[1], f[2], f[3]};
                            o[1].f = floatx4{f[4], f[5], f[6], f[7]};
                        } else {
                            bf16_terms<2>(f, o);
                        }
                        vops[((wave * VSTEPS + s0 + q) * 2) * 64 + lane] = o[0];
                        vops[((wave * VSTEPS + s0 + q) * 2 + 1) * 64 + lane] = o[1];
                    }
            };
            for (int s0 = 0; s0 < steps; s0 += 2) {
                const int n = min(2, steps - s0);
                if (vsp.P == 1) steps_of(std::integral_constant<int, 1>{}, s0, n);
                else if (vsp.P == 2) steps_of(std::integral_constant<int, 2>{}, s0, n);
                else steps_of(std::integral_constant<int, 4>{}, s0, n);
            }
        };
        const int row = n0 + wn + 4 * WA * (m >> 2) + (m & 3);       // feature of MFMA row m in block 0
        uint64_t todo, members;
        int r, j0;
        const bf16_t* Bt;
        auto advance = [&]() {                                       // to the next (adapter, 32 ranks); everything wavefront-uniform
            j0 += 32;
            if (j0 < r) return true;
            if (!todo) return false;
            const int src = __ffsll((unsigned long long)todo) - 1, a = __builtin_amdgcn_readlane(my_own, src);
            members = __ballot(my_own == a);
            todo &= ~members;
            r = __builtin_amdgcn_readlane(my_rank, src);
            Bt = reinterpret_cast<const bf16_t*>((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_bt, src) |
                                                 ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_bt >> 32), src) << 32));
            j0 = 0;
            return true;
        };
        auto load = [&](op16 (&bt)[WA]) {
            const int j = j0 + 8 * g;
            const bool whole = r % 8 == 0;
#pragma unroll
            for (int f = 0; f < WA; ++f) {
                const bf16_t* p = Bt + (int64_t)min(row + 4 * f, N - 1) * r;
                if (whole) bt[f].u = ldg_unaligned(p + (j < r ? j : 0));
                else bt[f] = row_chunk<bf16_t>(p, j, r);
            }
        };
        auto add = [&](op16 (&bt)[WA], uint64_t in, int j, int rank) {
            if (j + 8 * g >= rank) {
#pragma unroll
                for (int f = 0; f < WA; ++f) bt[f].u = u32x4{0, 0, 0, 0};
            }
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (((in >> (16 * b)) & 0xffffull) == 0) continue;                 // wavefront-uniform
                const op16* vp = vops + (((wt / 16 + b) * VSTEPS + j / 32) * 2) * 64 + lane;
                const op16 v0 = vp[0], v1 = vp[64];
                const bool mine = (in >> (16 * b + m)) & 1ull;       // (a product with zeros would carry the adapter's infinities over)
                auto take = [&](auto product) {
#pragma unroll
                    for (int f = 0; f < WA; ++f) {
                        const floatx4 e = product(bt[f], acc[f][b]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[f][b][i] = mine ? e[i] : acc[f][b][i];
                    }
                };
                if constexpr (DELTA == PLAIN_DELTA) {
                    const float f8[8] = {v0.f[0], v0.f[1], v0.f[2], v0.f[3], v1.f[0], v1.f[1], v1.f[2], v1.f[3]};
                    take([&](const op16& w, floatx4 c) { return mma_plain(w, f8, c); });
                } else {
                    take([&](const op16& w, floatx4 c) { return mma(w, v1, mma(w, v0, c, bf16_t{}), bf16_t{}); });
                }
            }
        };
        auto run = [&]() {
            op16 b0[WA], b1[WA];
            bool more = advance();
            if (more) load(b0);
            while (more) {
                uint64_t in = members;
                int j = j0, rank = r;
                more = advance();
                if (more) load(b1);
                add(b0, in, j, rank);
                if (!more) break;
                in = members; j = j0; rank = r;
                more = advance();
                if (more) load(b0);
                add(b1, in, j, rank);
            }
        };
        __syncthreads();
        make_operands(da.v, da.vsp, v_rank);
        __syncthreads();
        todo = __ballot(my_own != KEY_NONE);
        r = j0 = 0;
        run();
        if (da.merged >= 0) {                                        // mixture mode: the merged adapter, negated, where it applies
            __syncthreads();
            make_operands(da.v2, da.vsp2, v_removal);
            __syncthreads();
            todo = 0;
            members = removal;
            r = removal ? da.rank[da.merged] : 0;
            Bt = reinterpret_cast<const bf16_t*>(da.Bt_ptrs[da.merged]);
            j0 = -32;
            run();
        }
    }

    // ---- one rounding, store (rows go back to their tokens): a lane has 4 WA consecutive features of its tokens ----
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int pos = t0 + wt + 16 * b + m;
        if (pos >= T) continue;
        const int n = n0 + wn + 4 * WA * g;
        bf16_t* yp = y + (int64_t)(DELTA != NO_DELTA ? da.order[pos] : pos) * ldy + n;
#pragma unroll
        for (int a = 0; a < WA; ++a) {
            const floatx4 e = acc[a][b];
            const uint2 o = {(uint32_t)f32_to_bf16(e[0]) | ((uint32_t)f32_to_bf16(e[1]) << 16),
                             (uint32_t)f32_to_bf16(e[2]) | ((uint32_t)f32_to_bf16(e[3]) << 16)};
            if (n + 4 * a + 4 <= N) {
                *reinterpret_cast<uint2*>(yp + 4 * a) = o;           // (ldy % 8 == 0, y 16-byte aligned)
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + 4 * a + i < N) yp[4 * a + i] = f32_to_bf16(e[i]);
            }
        }
    }
}

template <int WA, row_delta DELTA, bool APART, bool KTAIL>
__global__ __launch_bounds__(512) void gemm_mid_kernel(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, row_delta_args da)
{
    gemm_mid_tile<WA, DELTA, APART, KTAIL>(T, K, N, x, ldx, Wt, ldw, y, ldy, tiles_n, tiles_t, da);
}

// tiles of 64 features, without adapters
template <bool KTAIL>
__global__ __launch_bounds__(512) void gemm_narrow_kernel(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, row_delta_args da)
{
    gemm_mid_tile<1, NO_DELTA, true, KTAIL>(T, K, N, x, ldx, Wt, ldw, y, ldy, tiles_n, tiles_t, da);
}

// tiles of 256 features
template <row_delta DELTA, bool APART, bool KTAIL>
__global__ __launch_bounds__(512) void gemm_wide_kernel(
    int T, int K, int N, const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ Wt, int64_t ldw,
    bf16_t* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, row_delta_args da)
{
    gemm_mid_tile<4, DELTA, APART, KTAIL>(T, K, N, x, ldx, Wt, ldw, y, ldy, tiles_n, tiles_t, da);
}

template <int WA, row_delta DELTA, bool APART, bool KTAIL>
constexpr auto mid_kernel()
{
    if constexpr (WA == 1) return &gemm_narrow_kernel<KTAIL>;
    else if constexpr (WA == 4) return &gemm_wide_kernel<DELTA, APART, KTAIL>;
    else return &gemm_mid_kernel<WA, DELTA, APART, KTAIL>;
}

template <int WA, row_delta DELTA, bool APART, bool KTAIL>
hipError_t launch_one(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw, void* y, int64_t ldy,
                      const row_delta_args& da, hipStream_t stream)
{
    const int tiles_n = (N + 64 * WA - 1) / (64 * WA), tiles_t = (T + MID_TOKENS - 1) / MID_TOKENS;
    constexpr size_t lds_bytes = 163840;
    constexpr auto kernel = mid_kernel<WA, DELTA, APART, KTAIL>();
    static std::atomic<bool> attr_set{false};                 // dynamic LDS above 64 KB has to be allowed once per kernel
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    LORA_LAUNCH(DELTA != NO_DELTA ? LORA_K_GEMM_MID_DELTA : LORA_K_GEMM_MID, kernel, dim3((unsigned)(tiles_n * tiles_t)),
                dim3(512), lds_bytes, stream, T, K, N, (const bf16_t*)x, ldx, (const bf16_t*)Wt, ldw, (bf16_t*)y, ldy, tiles_n, tiles_t, da);
    return hipGetLastError();
}

}  // namespace

// The kernel a problem takes least time on.  Each is modelled as rounds of tiles over the 256 compute units; a round
// takes a fixed part (first loads, last stores) and per stage of 64 k a time that grows from an almost idle chip to a
// full one.  Measured, cold weights, microseconds (small / 128 / 192 / 256 x 256 ring / what it was before):
//   4096 -> 4096,  256 tokens 16 / 31 / 35 / 64 / 16,  640: 42 / 33 / 36 / 63 / 45,  1280: 79 / 64 / 44 / 68 / 70,
//                  1536: - / 67 / 79 / 69 / 75,  2048: - / 68 / 80 / 72 / 77,  3072: - / 111 / 128 / 85 / 85
//   5120 -> 5120,  1024 tokens 91 / 79 / 53 / 84 / 85,  2048: - / 116 / 99 / 84 / 137
//   4096 -> 11008, 256 tokens 42 / 34 / 38 / 65 / 42,  512: 80 / 64 / 45 / - / 71,  1024: 157 / 98 / 84 / 73 / 115
//   5120 -> 13824, 320 tokens 108 / 87 / 66 / - / 86,  640: 180 / 128 / 116 / 95 / 138
// 128 / 192 / 256 features / 256 x 256 ring, where 256 features are the choice: 2048 tokens, 4096 -> 4096, 75 / 80 / 62 / 76;  1500,
// 11008 -> 4096, 189 / 201 / 151 / 200;  2607, 3288 -> 3064, 75 / 86 / 58 / 67;  and just where they are not: 2321, 5120 -> 5120,
// 118 / 140 / 115 / 100;  3000, 4096 -> 4096, 110 / 116 / 109 / 80;  991, 5120 -> 5120, 71 / 49 / 56 / 83.
// Products of few stages are the register-staged 128 x 128 tiles' (two on a compute unit, so that one's stores and first
// loads run beside the other's stages; without adapters, whose infinities they do not keep apart).  Kernel times, small /
// 128 / 192 / ring / register-staged: 2944 tokens, 32 -> 2568, 24.6 / 11.1 / 12.7 / - / 8.8;  4944, 128 -> 3496: 48.8 / 24.1 /
// 21.7 / - / 18.6;  9901, 256 -> 1568: 53.4 / 24.5 / 24.6 / 23.4 / 18.1;  1452, 1024 -> 4096: 34.6 / 25.7 / 29.3 / 24.4 / 22.9.
// Tiles of 64 features (no adapters), W from memory, before / with them: 4096 -> 4096, 300 tokens 34.1 / 27.7, 512 34.7 / 29.7;
// 5120 -> 5120, 384, 45.9 / 40.3;  4096 -> 11008, 100, 38.8 / 31.5.
// The constants of the five others are fitted to such times of 2000 problems (8 to 16384 tokens, K 8 to 13824, N 64 to 13824): with
// the kernels of that time the choice took 0.4 % longer than the best of the five on average, 1.24 times at worst.  Those of
// 128 and 192 features are 1 % faster without adapters since, from 25 stages on: a distance that the fit does not see.  Those of
// 256 features are fitted to 8 products.  Drawn calls that go to them, forced to each kernel in turn: 70 of lora_base_gemm (K from
// 1264; shorter ones mostly are the register-staged tiles') 1.16 times as fast as the best of all others, two below 0.98 (2933 tokens,
// 1704 -> 11112, 133 us, ring 125); 70 of lora_fused_forward, K from 8, 1.15, two below 0.98 (1183, 120 -> 5768, 42.2, 192 features 38.4).
gemm_route_id gemm_route(int32_t T, int32_t K, int32_t N, int64_t ldx, int64_t ldw, bool delta, bool tiled)
{
    if ((int64_t)N * ldw * 2 >= (1ll << 32) || (int64_t)T * ldx * 2 >= (1ll << 32)) return GEMM_TILED;   // 32-bit byte offsets
    const double stages = (K + 63) / 64;
    // slots: tiles the chip holds at a time
    auto rounds = [&](int32_t bm, int32_t bt, double slots, double fixed, double idle, double more, int power) {
        const int64_t tiles = (int64_t)((N + bm - 1) / bm) * ((T + bt - 1) / bt);
        const int64_t full = tiles / (int64_t)slots;
        const double left = (double)(tiles % (int64_t)slots) / slots;
        double us = full * (fixed + stages * (idle + more));
        if (left > 0) us += fixed + stages * (idle + more * (power == 2 ? left * left : left));
        return us;
    };
    const bool ring = tiled && K > 128;                       // (its fewest stages: three)
    if (tiled && !ring && delta && (int64_t)((N + 255) / 256) * ((T + 255) / 256) >= 192) return GEMM_TILED;
    gemm_route_id best = GEMM_SMALL;
    double us = gemm_small_time(T, K, N);
    auto take = [&](gemm_route_id id, double t) {
        if (t < us) { us = t; best = id; }
    };
    take(GEMM_MID_128, rounds(128, 128, 256, 2.0, 0.43, 0.10, 1));
    take(GEMM_MID_192, rounds(192, 128, 256, 3.1, 0.51, 0.19, 1));
    take(GEMM_MID_256, rounds(256, 128, 256, 4.0, 0.70, 0.20, 1));
    if (!delta) take(GEMM_MID_64, rounds(64, 128, 256, 3.5, 0.36, 0.05, 1));
    if (ring) take(GEMM_TILED, rounds(256, 256, 256, 4.4, 0.95, 0.55, 2));
    if (!delta) take(GEMM_TILED_128, 0.3 + rounds(128, 128, 512, 1.7, 0.585, 0.56, 1));
    return best;
}

// p != nullptr: fold the adapter delta in; v holds the shrink's output
hipError_t launch_gemm_mid(gemm_route_id route, int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                           void* y, int64_t ldy, const lora_plan* p, const lora_dev_tables* d, const float* v,
                           const gemm_removal& rm, const void* const* Bt, hipStream_t stream)
{
    const bool delta = p && (!p->perm.empty() || rm.plan);
    const row_delta_args da = delta ? row_deltas_of(p, d, v, rm, Bt) : row_delta_args{};
#define MID_LAUNCH(WA_, D_, A_, KT_) launch_one<WA_, D_, A_, KT_>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)
#define MID_WIDTH(D_, A_, KT_) (route == GEMM_MID_128 ? MID_LAUNCH(2, D_, A_, KT_) : route == GEMM_MID_192 ? MID_LAUNCH(3, D_, A_, KT_) : MID_LAUNCH(4, D_, A_, KT_))
#define MID_DISPATCH(D_, A_) (K % 64 ? MID_WIDTH(D_, A_, true) : MID_WIDTH(D_, A_, false))
    if (route == GEMM_MID_64) return delta ? hipErrorInvalidValue : K % 64 ? MID_LAUNCH(1, NO_DELTA, true, true) : MID_LAUNCH(1, NO_DELTA, true, false);
    if (!delta) return K > 24 * 64 ? MID_DISPATCH(NO_DELTA, true) : MID_DISPATCH(NO_DELTA, false);
    return p->extra_ptr256.empty() ? MID_DISPATCH(PLAIN_DELTA, false) : MID_DISPATCH(TERMS_DELTA, false);
#undef MID_DISPATCH
#undef MID_WIDTH
#undef MID_LAUNCH
}
