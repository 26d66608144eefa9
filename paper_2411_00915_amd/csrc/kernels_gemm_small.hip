// Base GEMM y = x W (+ adapter deltas) of small batches (bf16) and of every fp32 batch: the contraction is split over
// the wavefronts of a workgroup instead of over workgroups.
//
// A batch of T tokens with few of them is bound by reading W once, and the 128 x 128 tiles of the other GEMM kernels
// leave most compute units without any: 64 tokens x 4096 features are 32 workgroups, each walking the whole K alone.
// Here a workgroup (8 wavefronts) owns 16 FB features x 16 TB tokens, its wavefronts take contiguous slices of K, and
// the partial sums meet in LDS: the chip is full from N = 4096 features on (FB = 1: 256 workgroups), no partial sum
// ever goes to memory and no second launch is needed.  Nothing is shared between the wavefronts (each has its own k
// range), so
// the K loop needs no barrier: D units of 128 bytes per row are in flight per wavefront, through its own part of LDS.
//
// fp32 runs on v_mfma_f32_16x16x4_f32 the same way (fp32 products and sums); there the matrix cores bind (256
// flops/clk per compute unit) and the same tiles serve every batch size.
//
// Measured (whole lora_fused_forward, cold weights): 64 single-token requests on 32 adapters, 4096 -> 4096, 104 -> 21 us;
// fp32, 256 tokens, 4096 -> 4096: this kernel 600 -> 73 us (the matrix cores' share of that at 2.1 GHz is 64 us).
//
// DELTA: tokens in adapter-sorted order; before the partial sums are added up, the wavefronts share out the (adapter,
// rank step) pairs of the tile's tokens and add v B_a of theirs to their own partial sums, so the delta is spread over
// the workgroup and joins the same fp32 sum.  v is read as the shrink left it (fp32, K parts added in order); with bf16
// it is split into two bf16 terms in registers, or, for ranks off the tuned kernels, multiplied as it is (fp32 products:
// 64 tokens on 32 adapters of ranks 4 to 100, 4096 -> 4096, 25.3 us, with two terms 24.1).
#include <algorithm>
#include <atomic>

#include "kernels.h"
#include "launch.h"
#include "split_k.h"

namespace {

template <typename E, int FB, int TB, int D, row_delta DELTA, bool KTAIL>
__global__ __launch_bounds__(512) void gemm_small_kernel(
    int T, int K, int N, const E* __restrict__ x, int64_t ldx, const E* __restrict__ Wt, int64_t ldw,
    E* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, bool y_vec, row_delta_args da)
{
    constexpr int WAVES = 8;
    // workgroups are dealt round-robin to the 8 XCDs; every XCD gets an eighth of the tiles, the token tiles of one feature
    // tile next to each other, so that its W rows come from memory once and are then in that XCD's L2
    const int n_wg = tiles_n * tiles_t, xcd = (int)blockIdx.x & 7;
    const int tile = xcd * (n_wg / 8) + min(xcd, n_wg % 8) + ((int)blockIdx.x >> 3);
    const int tile_n = tile / tiles_t, tile_t = tile % tiles_t;
    const int n0 = tile_n * 16 * FB, t0 = tile_t * 16 * TB;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;

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
    part.run((int)(((int64_t)part.units * wave) / WAVES), (int)(((int64_t)part.units * (wave + 1)) / WAVES));

    // ---- adapter deltas: the (adapter, rank step) pairs of the tile's tokens in turn to the wavefronts ------
    if constexpr (DELTA != NO_DELTA) {
        const int pos = t0 + lane;
        const bool row_in = lane < 16 * TB && pos < T;
        const int my_tok = da.order[row_in ? pos : T - 1];
        const int my_key = row_in ? da.row_key[my_tok] : KEY_NONE;
        const int own = my_key & KEY_NONE;
        const int my_rank = own != KEY_NONE ? da.rank[own] : 0;
        const uint64_t my_bt = own != KEY_NONE ? reinterpret_cast<uint64_t>(da.Bt_ptrs[own]) : 0;
        int tokb[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b) tokb[b] = __shfl(my_tok, 16 * b + m);
        int turn = 0;
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
                for (int b = 0; b < TB; ++b) {
                    if (((members >> (16 * b)) & 0xffffull) == 0) continue;       // wavefront-uniform
                    const bool mine = (members >> (16 * b + m)) & 1ull;
                    auto add = [&](auto product) {
#pragma unroll
                        for (int f = 0; f < FB; ++f) {
                            const floatx4 e = product(bt[f], acc[f][b][0]);
                            // (a product with zeros would carry the adapter's infinities over to other tokens)
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc[f][b][0][i] = mine ? e[i] : acc[f][b][0][i];
                        }
                    };
                    if constexpr (ES == 4) {
                        op16 vo;
                        vo.f = floatx4{vf[b][0], vf[b][1], vf[b][2], vf[b][3]};
                        add([&](const op16& w, floatx4 c) { return mma(w, vo, c, E{}); });
                    } else if constexpr (DELTA == PLAIN_DELTA) {
                        add([&](const op16& w, floatx4 c) { return mma_plain(w, vf[b], c); });
                    } else {
                        op16 vo[2];
                        bf16_terms<2>(vf[b], vo);
                        add([&](const op16& w, floatx4 c) { return mma(w, vo[1], mma(w, vo[0], c, E{}), E{}); });
                    }
                }
            }
        };
        uint64_t todo = __ballot(own != KEY_NONE);
        while (todo) {
            const int src = __ffsll((unsigned long long)todo) - 1;
            const int a = __builtin_amdgcn_readlane(own, src), r = __builtin_amdgcn_readlane(my_rank, src);
            const uint64_t bt = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_bt, src) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_bt >> 32), src) << 32);
            const uint64_t members = __ballot(own == a);
            todo &= ~members;
            apply(reinterpret_cast<const E*>(bt), r, members, da.v, da.vsp);
        }
        const uint64_t removal = __ballot((my_key & LORA_UNMERGE_BIT) != 0);
        if (removal) apply(reinterpret_cast<const E*>(da.Bt_ptrs[da.merged]), da.rank[da.merged], removal, da.v2, da.vsp2);
    }

    // ---- partial sums meet in LDS, one rounding, store (rows go back to their tokens) ----
    part.park();
    __syncthreads();
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

template <typename E, int FB, int TB, int D, row_delta DELTA, bool KTAIL>
hipError_t launch_one(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw, void* y, int64_t ldy,
                      const row_delta_args& da, hipStream_t stream)
{
    const int tiles_n = (N + 16 * FB - 1) / (16 * FB), tiles_t = (T + 16 * TB - 1) / (16 * TB);
    constexpr size_t lds_bytes = (size_t)8 * D * (2 * FB + 2 * TB) * 1024;
    static_assert(D * (2 * FB + 2 * TB) >= FB * TB && lds_bytes <= 163840, "a wavefront's partial sums go where its operands were");
    if (lds_bytes > 65536) {                                  // dynamic LDS above 64 KB has to be allowed once per kernel
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_small_kernel<E, FB, TB, D, DELTA, KTAIL>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    LORA_LAUNCH(DELTA != NO_DELTA ? LORA_K_GEMM_SMALL_DELTA : LORA_K_GEMM_SMALL, (gemm_small_kernel<E, FB, TB, D, DELTA, KTAIL>),
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

template <typename E, row_delta DELTA, bool KTAIL>
hipError_t launch_tile(const small_tile& t, int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                       void* y, int64_t ldy, const row_delta_args& da, hipStream_t stream)
{
#define SMALL_TILE(FB_, TB_, D_) \
    if (t.fb == FB_ && t.tb == TB_) return launch_one<E, FB_, TB_, D_, DELTA, KTAIL>(T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream);
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
#define SMALL_LAUNCH(E_, D_, KT_) launch_tile<E_, D_, KT_>(t, T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)
#define SMALL_DISPATCH(E_, D_) (ktail ? SMALL_LAUNCH(E_, D_, true) : SMALL_LAUNCH(E_, D_, false))
    if (dtype == LORA_F32) return delta ? SMALL_DISPATCH(float, PLAIN_DELTA) : SMALL_DISPATCH(float, NO_DELTA);
    if (!delta) return SMALL_DISPATCH(bf16_t, NO_DELTA);
    return p->extra_ptr256.empty() ? SMALL_DISPATCH(bf16_t, PLAIN_DELTA) : SMALL_DISPATCH(bf16_t, TERMS_DELTA);
#undef SMALL_DISPATCH
#undef SMALL_LAUNCH
}
