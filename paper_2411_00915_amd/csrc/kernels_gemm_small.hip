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
// the workgroup and joins the same fp32 sum.  v is read as the shrink left it (fp32, K parts added in order) and, for
// bf16, split into two bf16 terms in registers.
#include <algorithm>
#include <atomic>

#include "device_util.h"
#include "kernels.h"
#include "launch.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

union op16 {            // 16 bytes of one row: 8 bf16 or 4 fp32 consecutive k
    u32x4 u;
    bf16x8 v;
    floatx4 f;
};

// 16-byte loads from a wavefront-uniform base plus a 32-bit byte offset per lane
__device__ __forceinline__ u32x4 ldg(const char* base, uint32_t off)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(1))) u32x4*)((const __attribute__((address_space(1))) char*)(uintptr_t)base + off);
#else
    return *reinterpret_cast<const u32x4*>(base + off);
#endif
}

typedef __attribute__((address_space(3))) void* lds_void_ptr;
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lds_void_ptr)p; }
// lane i's 16 bytes at base + off -> LDS byte address lds_base + 16 i (base and lds_base wavefront-uniform); issued
// from inline assembly, so the waits for it are written out
__device__ __forceinline__ void load16_to_lds(const char* base, uint32_t off, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_base) : "memory");
}

__device__ __forceinline__ floatx4 mma(const op16& a, const op16& b, floatx4 c, bf16_t)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mma(const op16& a, const op16& b, floatx4 c, float)
{
    // lane group g supplies k = g of each 16x16x4 product; taking element i of every lane's chunk permutes k the same
    // way on both sides
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[i], b.f[i], c, 0, 0, 0);
    return c;
}

struct small_delta_args {
    const int32_t* order;          // [T] tokens sorted by adapter, then tokens without adapter
    const int32_t* row_key;        // [T] adapter of the token (bits 0..22; all ones: none) | removal bit
    const int32_t* rank;
    const float* v;
    lora_vspec vsp;
    const void* const* Bt_ptrs;
    const float* v2;               // mixture mode: the removal's v
    lora_vspec vsp2;
    int merged;                    // the merged adapter, or -1
};

constexpr int KEY_NONE = LORA_UNMERGE_BIT - 1;

// elements [j, j + 16 / sizeof(E)) of a row of r elements; those past the row's end are zero
template <typename E>
__device__ __forceinline__ op16 row_chunk(const E* row, int j, int r)
{
    constexpr int EPC = 16 / (int)sizeof(E);
    op16 o;
    o.u = u32x4{0, 0, 0, 0};
    if (j >= r) return o;
    if (r % EPC == 0) {                                      // uniform: the chunk is whole and aligned
        o.u = ldg(reinterpret_cast<const char*>(row), (uint32_t)j * (uint32_t)sizeof(E));
    } else if constexpr (sizeof(E) == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (j + i < r) o.f[i] = row[j + i];
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (j + i < r) o.u[i >> 1] |= (uint32_t)row[j + i] << (16 * (i & 1));
    }
    return o;
}

// v[token][j ..] (sum of its K parts) as MFMA operands: bf16: two terms hi + lo; fp32: hi alone
template <typename E>
__device__ __forceinline__ void v_chunk(const float* v, const lora_vspec& vsp, int tok, int j, int r, bool mine, op16& hi, op16& lo)
{
    constexpr int EPC = 16 / (int)sizeof(E);
    float f[EPC];
#pragma unroll
    for (int i = 0; i < EPC; ++i) f[i] = 0.f;
    if (mine && j < r) {                                     // (rows are R floats apart, R % 8 == 0)
        const float* p = v + (int64_t)tok * vsp.R + j;
        floatx4 part[EPC / 4];
#pragma unroll
        for (int q = 0; q < EPC / 4; ++q) part[q] = *reinterpret_cast<const floatx4*>(p + 4 * q);
        for (int s = 1; s < vsp.P; ++s)
#pragma unroll
            for (int q = 0; q < EPC / 4; ++q) part[q] += *reinterpret_cast<const floatx4*>(p + s * vsp.part + 4 * q);
#pragma unroll
        for (int i = 0; i < EPC; ++i) f[i] = j + i < r ? part[i >> 2][i & 3] : 0.f;      // past the rank: never written
    }
    if constexpr (sizeof(E) == 4) {
        hi.f = floatx4{f[0], f[1], f[2], f[3]};
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bf16_t h0 = f32_to_bf16(f[2 * i]), h1 = f32_to_bf16(f[2 * i + 1]);
            hi.u[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            lo.u[i] = (uint32_t)f32_to_bf16(f[2 * i] - bf16_to_f32(h0)) | ((uint32_t)f32_to_bf16(f[2 * i + 1] - bf16_to_f32(h1)) << 16);
        }
    }
}

extern __shared__ floatx4 small_lds[];

// Lane roles of the 16x16 MFMAs (rows = features, columns = tokens): lane l supplies row / column m = l % 16, chunk
// g = l / 16 of a 64-byte step, and receives rows 4 g + i of column m.  Row 4 q + i of block f stands for feature
// 4 FB q + 4 f + i of the tile, so over its FB blocks a lane holds 4 FB consecutive features of its token.
template <typename E, int FB, int TB, int D, bool DELTA, bool KTAIL>
__global__ __launch_bounds__(512) void gemm_small_kernel(
    int T, int K, int N, const E* __restrict__ x, int64_t ldx, const E* __restrict__ Wt, int64_t ldw,
    E* __restrict__ y, int64_t ldy, int tiles_n, int tiles_t, bool y_vec, small_delta_args da)
{
    constexpr int WAVES = 8, ES = (int)sizeof(E), EPC = 16 / ES, KSTEP = 4 * EPC, KUNIT = 2 * KSTEP;
    // workgroups are dealt round-robin to the 8 XCDs; the token tiles of one feature tile follow each other on one
    // XCD, so that its W rows come from memory once and are then in that XCD's L2
    const int q = (int)blockIdx.x >> 3, xcd = (int)blockIdx.x & 7;
    const int tile_t = q % tiles_t, tile_n = (q / tiles_t) * 8 + xcd;
    if (tile_n >= tiles_n) return;
    const int n0 = tile_n * 16 * FB, t0 = tile_t * 16 * TB;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;

    // Loads: an instruction brings 128 bytes of 8 rows (whole cache lines: a compute unit gets 100 - 120 GB/s that way,
    // 38 GB/s as 64 bytes of 16 rows, the MFMA operand shape) straight into this wavefront's own part of LDS; lane l
    // fetches the chunk that belongs in slot l % 8 of row l / 8.  (The launcher keeps N ldw and T ldx below 2^32
    // bytes; rows past the end re-read the last one and are never stored.)
    constexpr int NW = 2 * FB, NX = 2 * TB, NL = NW + NX;                // loads of a unit
    const int lrow = lane >> 3, lslot = lane & 7;
    auto swz_w = [](int row) { return (row & 3) | (((row / (4 * FB)) & 1) << 2); };   // eight values over the rows of eight lanes
    auto swz_x = [](int row) { return row & 7; };
    uint32_t off[NL];
    uint32_t cut[NL];                                                    // KTAIL: what takes a chunk past K in the last unit back to its row's first
    const int last_k = (K - 1) / KUNIT * KUNIT;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const bool is_w = i < NW;
        const int row = (is_w ? i : i - NW) * 8 + lrow;
        const int c = lslot ^ (is_w ? swz_w(row) : swz_x(row));
        cut[i] = KTAIL && last_k + c * EPC >= K ? c * 16 : 0;
        int64_t r = is_w ? n0 + row : t0 + row;
        if (is_w) r = (r < N ? r : N - 1) * ldw;
        else { r = r < T ? r : T - 1; r = (DELTA ? da.order[r] : r) * ldx; }
        off[i] = (uint32_t)(r * ES) + c * 16;
    }

    floatx4 acc[FB][TB];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[f][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    // this wavefront's units of 128 bytes per row, D of them in LDS
    const int units = (K + KUNIT - 1) / KUNIT;
    const int u_begin = (int)(((int64_t)units * wave) / WAVES), u_end = (int)(((int64_t)units * (wave + 1)) / WAVES);
    char* const own_lds = reinterpret_cast<char*>(small_lds) + wave * (D * NL * 1024);
    const uint32_t own_addr = lds_address(small_lds) + wave * (D * NL * 1024);
    const char* const wb = reinterpret_cast<const char*>(Wt);
    const char* const xb = reinterpret_cast<const char*>(x);
    auto issue = [&](int u, int slot) {
        const bool tail = KTAIL && u == units - 1;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            load16_to_lds((i < NW ? wb : xb) + (int64_t)u * 128, tail ? off[i] - cut[i] : off[i], own_addr + slot * (NL * 1024) + i * 1024);
        }
    };
    op16 w[2][FB], xr[2][TB];
    auto read = [&](int slot) {
        const char* p = own_lds + slot * (NL * 1024);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int c = 4 * s + g;
#pragma unroll
            for (int f = 0; f < FB; ++f) {
                const int row = 4 * FB * (m >> 2) + 4 * f + (m & 3);
                w[s][f].u = *reinterpret_cast<const u32x4*>(p + row * 128 + (c ^ swz_w(row)) * 16);
            }
#pragma unroll
            for (int b = 0; b < TB; ++b) xr[s][b].u = *reinterpret_cast<const u32x4*>(p + NW * 1024 + (16 * b + m) * 128 + (c ^ swz_x(m)) * 16);
        }
    };
    auto compute = [&](int u) {
        if (KTAIL && u == units - 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
                if (last_k + s * KSTEP + g * EPC >= K) {
#pragma unroll
                    for (int f = 0; f < FB; ++f) w[s][f].u = u32x4{0, 0, 0, 0};
#pragma unroll
                    for (int b = 0; b < TB; ++b) xr[s][b].u = u32x4{0, 0, 0, 0};
                }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int f = 0; f < FB; ++f) acc[f][b] = mma(w[s][f], xr[s][b], acc[f][b], E{});
    };
    // waits until all but the youngest n units (n < D) have landed; loads return in order
    auto landed = [&](int n) {
        if (D >= 4 && n >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NL) : "memory");
        else if (D >= 3 && n == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
        else if (D >= 2 && n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (u_begin + d < u_end) issue(u_begin + d, d);
    int slot = 0, u = u_begin;
    for (; u + D < u_end; ++u) {
        landed(D - 1);
        read(slot);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                // the slot is in registers: refill it
        issue(u + D, slot);
        compute(u);
        slot = slot + 1 == D ? 0 : slot + 1;
    }
    for (; u < u_end; ++u) {
        landed(u_end - 1 - u);
        read(slot);
        compute(u);
        slot = slot + 1 == D ? 0 : slot + 1;
    }

    // ---- adapter deltas: the (adapter, rank step) pairs of the tile's tokens in turn to the wavefronts ------
    if constexpr (DELTA) {
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
                op16 bt[FB], hi[TB], lo[TB];
#pragma unroll
                for (int f = 0; f < FB; ++f) {
                    const int n = n0 + 4 * FB * (m >> 2) + 4 * f + (m & 3);
                    bt[f] = row_chunk<E>(Bt + (int64_t)(n < N ? n : N - 1) * r, j, r);
                }
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    v_chunk<E>(v, vsp, tokb[b], j, r, (members >> (16 * b + m)) & 1ull, hi[b], lo[b]);
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    if (((members >> (16 * b)) & 0xffffull) == 0) continue;       // wavefront-uniform
#pragma unroll
                    for (int f = 0; f < FB; ++f) {
                        acc[f][b] = mma(bt[f], hi[b], acc[f][b], E{});
                        if constexpr (ES == 2) acc[f][b] = mma(bt[f], lo[b], acc[f][b], E{});
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
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int f = 0; f < FB; ++f) reinterpret_cast<floatx4*>(own_lds)[(b * FB + f) * 64 + lane] = acc[f][b];
    __syncthreads();
    // a thread finishes F4 consecutive blocks (4 F4 consecutive features) of one lane's token
    constexpr int ITEMS = FB * TB * 64, F4 = ITEMS > 512 ? ITEMS / 512 : 1;
    if (wave * F4 >= FB * TB) return;
    const int b = wave * F4 / FB, f0 = wave * F4 % FB;
    floatx4 sum[F4];
#pragma unroll
    for (int f = 0; f < F4; ++f) {
        floatx4 part[WAVES];
#pragma unroll
        for (int s = 0; s < WAVES; ++s) part[s] = small_lds[s * (D * NL * 64) + (b * FB + f0 + f) * 64 + lane];
#pragma unroll
        for (int st = WAVES / 2; st > 0; st >>= 1)
#pragma unroll
            for (int s = 0; s < st; ++s) part[s] += part[s + st];
        sum[f] = part[0];
    }
    const int pos = t0 + 16 * b + m;
    if (pos >= T) return;
    const int n = n0 + 4 * FB * g + 4 * f0;
    E* yp = y + (int64_t)(DELTA ? da.order[pos] : pos) * ldy + n;
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

template <typename E, int FB, int TB, int D, bool DELTA, bool KTAIL>
hipError_t launch_one(int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw, void* y, int64_t ldy,
                      const small_delta_args& da, hipStream_t stream)
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
    LORA_LAUNCH(DELTA ? LORA_K_GEMM_SMALL_DELTA : LORA_K_GEMM_SMALL, (gemm_small_kernel<E, FB, TB, D, DELTA, KTAIL>),
                dim3((unsigned)((tiles_n + 7) / 8 * 8 * tiles_t)), dim3(512), lds_bytes, stream, T, K, N, (const E*)x, ldx, (const E*)Wt, ldw,
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

template <typename E, bool DELTA, bool KTAIL>
hipError_t launch_tile(const small_tile& t, int32_t T, int32_t K, int32_t N, const void* x, int64_t ldx, const void* Wt, int64_t ldw,
                       void* y, int64_t ldy, const small_delta_args& da, hipStream_t stream)
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
    if (T < 1 || N < 1 || K % epc || ldx % epc || ldw % epc || mis(x) || mis(Wt)) return false;
    if (dtype == LORA_BF16 && (ldy % 8 || mis(y))) return false;
    if ((int64_t)N * ldw * es >= (1ll << 32) || (int64_t)T * ldx * es >= (1ll << 32)) return false;      // 32-bit byte offsets
    return (int64_t)((N + 15) / 16 + 8) * ((T + 15) / 16) < (1ll << 31);
}

// (bf16: measured at 512 tokens, N = K = 4096: 35 us here, 104 us in 128 x 128 tiles; 1024 tokens: 69 and 100 us)
bool gemm_small_wins(int32_t T, int32_t K, int32_t N, int32_t dtype)
{
    return dtype == LORA_F32 || T <= 512;
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
    small_delta_args da{};
    if (delta)
        da = small_delta_args{d->order, d->row_key, d->rank, v, lora_vspec_of(p), Bt, rm.v, rm.plan ? lora_vspec_of(rm.plan) : lora_vspec{0, 1, 0},
                              rm.plan ? p->merged : -1};
#define SMALL_LAUNCH(E_, D_, KT_) launch_tile<E_, D_, KT_>(t, T, K, N, x, ldx, Wt, ldw, y, ldy, da, stream)
    if (dtype == LORA_F32) {
        if (delta) return ktail ? SMALL_LAUNCH(float, true, true) : SMALL_LAUNCH(float, true, false);
        return ktail ? SMALL_LAUNCH(float, false, true) : SMALL_LAUNCH(float, false, false);
    }
    if (delta) return ktail ? SMALL_LAUNCH(bf16_t, true, true) : SMALL_LAUNCH(bf16_t, true, false);
    return ktail ? SMALL_LAUNCH(bf16_t, false, true) : SMALL_LAUNCH(bf16_t, false, false);
#undef SMALL_LAUNCH
}
