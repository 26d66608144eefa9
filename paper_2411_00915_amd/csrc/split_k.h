// Pieces of the kernels that split the contraction over the wavefronts of a workgroup (gemm_small_kernel, the fp32 and
// any-rank adapter kernels): 16-byte operands of bf16 or fp32 rows, their MFMA, and split_k, one wavefront's slice of
// a tile's contraction.
#pragma once
#include "device_util.h"
#include "kernels.h"

namespace {

union op16 {            // 16 bytes of one row: 8 bf16 or 4 fp32 consecutive k
    u32x4 u;
    bf16x8 v;
    floatx4 f;
};

// 16 bytes at an address that is aligned to an element only (global loads take any address)
template <typename E>
__device__ __forceinline__ u32x4 ldg_unaligned(const E* p)
{
    typedef u32x4 unaligned_t __attribute__((aligned(2)));
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(1))) unaligned_t*)(uintptr_t)p;
#else
    return *reinterpret_cast<const unaligned_t*>(p);
#endif
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

// fp32 with a sum of its own for every element of the chunks (those of index i go to c[i % N]): a chain of additions
// is what loses digits, so it is cut in N; folded() adds the sums up as a tree
template <int N>
__device__ __forceinline__ void mma_apart(const op16& a, const op16& b, floatx4 (&c)[N], int first)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) c[(first + i) % N] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[i], b.f[i], c[(first + i) % N], 0, 0, 0);
}
template <int N>
__device__ __forceinline__ floatx4 folded(floatx4 (&c)[N])
{
#pragma unroll
    for (int st = N / 2; st > 0; st >>= 1)
#pragma unroll
        for (int i = 0; i < st; ++i) c[i] += c[i + st];
    return c[0];
}

// eight bf16 by eight fp32 values of every lane, as fp32 products
__device__ __forceinline__ floatx4 mma_plain(const op16& a, const float (&f)[8], floatx4 c)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(i & 1 ? a.u[i >> 1] & 0xffff0000u : a.u[i >> 1] << 16), f[i], c, 0, 0, 0);
    return c;
}

// elements [j, j + 16 / sizeof(E)) of a row of r elements; those past the row's end are zero
template <typename E>
__device__ __forceinline__ op16 row_chunk(const E* row, int j, int r)
{
    constexpr int EPC = 16 / (int)sizeof(E);
    op16 o;
    o.u = u32x4{0, 0, 0, 0};
    if (j >= r) return o;
    if (j + EPC <= r) {                                      // whole; aligned to an element
        o.u = ldg_unaligned(row + j);
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

// v[token][j ..] (sum of its K parts); past the rank, and for tokens that are not `mine`, zero
template <int N>
__device__ __forceinline__ void v_values(const float* v, const lora_vspec& vsp, int tok, int j, int r, bool mine, float (&f)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = 0.f;
    if (mine && j < r) {                                     // (rows are R floats apart, R % 8 == 0)
        const float* p = v + (int64_t)tok * vsp.R + j;
        floatx4 part[4][N / 4];
#pragma unroll
        for (int s = 0; s < 4; ++s)                          // all parts are requested before the first add
            if (s < vsp.P) {
#pragma unroll
                for (int q = 0; q < N / 4; ++q) part[s][q] = *reinterpret_cast<const floatx4*>(p + s * vsp.part + 4 * q);
            }
#pragma unroll
        for (int s = 1; s < 4; ++s)
            if (s < vsp.P) {
#pragma unroll
                for (int q = 0; q < N / 4; ++q) part[0][q] += part[s][q];
            }
#pragma unroll
        for (int i = 0; i < N; ++i) f[i] = j + i < r ? part[0][i >> 2][i & 3] : 0.f;     // past the rank: never written
    }
}

// f as the sum of TERMS bf16 operands, each the rounded rest of those before it: two terms keep 16 bits of the
// significand, three all 24.  Infinities, and what rounds to one, give NaN in the last term.
template <int TERMS>
__device__ __forceinline__ void bf16_terms(const float (&f)[8], op16 (&o)[TERMS])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float f0 = f[2 * i], f1 = f[2 * i + 1];
#pragma unroll
        for (int t = 0; t < TERMS; ++t) {
            const bf16_t h0 = f32_to_bf16(f0), h1 = f32_to_bf16(f1);
            o[t].u[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            f0 -= bf16_to_f32(h0);
            f1 -= bf16_to_f32(h1);
        }
    }
}

// Adapter deltas of kernels whose rows are the tokens in the plan's order: none, with v as two bf16 terms, or with v in
// fp32 products (fp32, and bf16 with ranks off the tuned kernels, whose v was always taken whole)
enum row_delta { NO_DELTA, TERMS_DELTA, PLAIN_DELTA };
struct row_delta_args {
    const int32_t* order;          // [T] tokens in the plan's row order
    const int32_t* row_key;        // [T] in that order: adapter of the token (bits 0..22; all ones: none) | removal bit
    const int32_t* rank;
    const float* v;
    lora_vspec vsp;
    const void* const* Bt_ptrs;
    const float* v2;               // mixture mode: the removal's v
    lora_vspec vsp2;
    int merged;                    // the merged adapter, or -1
};
constexpr int KEY_NONE = LORA_UNMERGE_BIT - 1;

inline row_delta_args row_deltas_of(const lora_plan* p, const lora_dev_tables* d, const float* v, const gemm_removal& rm, const void* const* Bt)
{
    return row_delta_args{d->order, d->row_key, d->rank, v, lora_vspec_of(p), Bt, rm.v, rm.plan ? lora_vspec_of(rm.plan) : lora_vspec{0, 1, 0},
                          rm.plan ? p->merged : -1};
}

extern __shared__ floatx4 small_lds[];

// One wavefront's slice of K of a tile of 16 FB rows of W (features, or rank rows of an adapter) x 16 TB tokens.
//
// Lane roles of the 16x16 MFMAs (rows = rows of W, columns = tokens): lane l supplies row / column m = l % 16, chunk
// g = l / 16 of a 64-byte step, and receives rows 4 g + i of column m.  Row 4 q + i of block f stands for row
// 4 FB q + 4 f + i of the tile, so over its FB blocks a lane holds 4 FB consecutive rows' results of its token.
//
// Loads: an instruction brings 128 bytes of 8 rows (whole cache lines: a compute unit gets 100 - 108 GB/s that way,
// 59 - 65 GB/s as 64 bytes of 16 rows, the MFMA operand shape) straight into this wavefront's own part of LDS; lane l
// fetches the chunk that belongs in slot l % 8 of row l / 8.  Nothing is shared between wavefronts, so the loop has no
// barrier: D units of 128 bytes per row are in flight per wavefront.
// SUMS (fp32): partial sums kept apart per result, see mma_apart.
template <typename E, int FB, int TB, int D, bool KTAIL, int SUMS = 1>
struct split_k {
    static constexpr int ES = (int)sizeof(E), EPC = 16 / ES, KSTEP = 4 * EPC, KUNIT = 2 * KSTEP;
    static constexpr int NW = 2 * FB, NX = 2 * TB, NL = NW + NX;         // loads of a unit
    static constexpr int LDS_BYTES = D * NL * 1024;                      // of a wavefront
    int K, last_k, units, m, g;
    uint32_t off[NL];
    uint32_t cut[NL];                                                    // KTAIL: what takes a chunk past K in the last unit back to its row's first
    char* own_lds;
    uint32_t own_addr;
    const char *wb, *xb;
    floatx4 acc[FB][TB][SUMS];
    op16 w[2][FB], xr[2][TB];

    static __device__ __forceinline__ int swz_w(int row) { return (row & 3) | (((row / (4 * FB)) & 1) << 2); }   // eight values over the rows of eight lanes
    static __device__ __forceinline__ int swz_x(int row) { return row & 7; }

    // w_row(row), x_row(row): element offsets of the tile's rows from W and x, below 2^32 bytes (rows that do not exist
    // name one that does: what is computed for them is not stored)
    template <typename RowW, typename RowX>
    __device__ __forceinline__ split_k(int K_, const E* W, const E* x, int wave, RowW w_row, RowX x_row)
        : K(K_), last_k((K_ - 1) / KUNIT * KUNIT), units((K_ + KUNIT - 1) / KUNIT), wb(reinterpret_cast<const char*>(W)), xb(reinterpret_cast<const char*>(x))
    {
        const int lane = threadIdx.x & 63;
        m = lane & 15;
        g = lane >> 4;
        const int lrow = lane >> 3, lslot = lane & 7;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const bool is_w = i < NW;
            const int row = (is_w ? i : i - NW) * 8 + lrow;
            const int c = lslot ^ (is_w ? swz_w(row) : swz_x(row));
            cut[i] = KTAIL && last_k + c * EPC >= K ? c * 16 : 0;
            const int64_t r = is_w ? w_row(row) : x_row(row);
            off[i] = (uint32_t)(r * ES) + c * 16;
        }
#pragma unroll
        for (int f = 0; f < FB; ++f)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int i = 0; i < SUMS; ++i) acc[f][b][i] = floatx4{0.f, 0.f, 0.f, 0.f};
        own_lds = reinterpret_cast<char*>(small_lds) + wave * LDS_BYTES;
        own_addr = lds_address(small_lds) + wave * LDS_BYTES;
    }
    __device__ __forceinline__ void issue(int u, int slot)
    {
        const bool tail = KTAIL && u == units - 1;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            load16_to_lds((i < NW ? wb : xb) + (int64_t)u * 128, tail ? off[i] - cut[i] : off[i], own_addr + slot * (NL * 1024) + i * 1024);
    }
    __device__ __forceinline__ void read(int slot)
    {
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
    }
    __device__ __forceinline__ void compute(int u)
    {
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
                for (int f = 0; f < FB; ++f) {
                    if constexpr (SUMS > 1) mma_apart(w[s][f], xr[s][b], acc[f][b], 4 * s);
                    else acc[f][b][0] = mma(w[s][f], xr[s][b], acc[f][b][0], E{});
                }
    }
    // waits until all but the youngest n units (n < D) have landed; loads return in order
    static __device__ __forceinline__ void landed(int n)
    {
        static_assert(D <= 4, "as many waits as units in flight");
        if (D >= 4 && n == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NL) : "memory");
        else if (D >= 3 && n == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
        else if (D >= 2 && n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    // adds units [u_begin, u_end) of 128 bytes per row: `start` requests the first D, `drain` goes through them all.  For
    // loads of the caller's that its own code after the loop needs: `early` is called when the second round of requests is
    // out, `late` before the last unit is multiplied (where there are too few units, both before the first wait).
    __device__ __forceinline__ void start(int u_begin, int u_end)
    {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (u_begin + d < u_end) issue(u_begin + d, d);
    }
    __device__ __forceinline__ void run(int u_begin, int u_end)
    {
        start(u_begin, u_end);
        drain(u_begin, u_end, [] {}, [] {});
    }
    template <typename Early, typename Late>
    __device__ __forceinline__ void drain(int u_begin, int u_end, Early early, Late late)
    {
        if (u_begin + D >= u_end) early();
        if (u_begin >= u_end) late();
        int slot = 0, u = u_begin;
        for (; u + D < u_end; ++u) {
            landed(D - 1);
            read(slot);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // the slot is in registers: refill it
            issue(u + D, slot);
            if (u == u_begin) early();
            compute(u);
            slot = slot + 1 == D ? 0 : slot + 1;
        }
        for (; u < u_end; ++u) {
            landed(u_end - 1 - u);
            read(slot);
            if (u == u_end - 1) late();
            compute(u);
            slot = slot + 1 == D ? 0 : slot + 1;
        }
    }
    // The same for rows of W at any address, 64 bits of it: 64-byte pieces straight to registers.  bf16 off a dword is
    // fetched as the dwords that hold it (what they hold beside it is shifted out): lora_shrink of 256 tokens on 64 adapters
    // of rank 2 to 256, K = 4096, 18.5 us, by loads at its own address 31.4, a wavefront per value 171; W aligned 10.
    template <typename RowW, typename RowX>
    __device__ __forceinline__ void run_anywhere(const E* W, const E* x, RowW w_row, RowX x_row, int u_begin, int u_end)
    {
        const bool odd = ES == 2 && (reinterpret_cast<uintptr_t>(W) & 3) != 0;         // every row of W (K % EPC == 0)
        const E *wr[FB], *xp[TB];
#pragma unroll
        for (int f = 0; f < FB; ++f) wr[f] = W + w_row(4 * FB * (m >> 2) + 4 * f + (m & 3)) - (odd ? 1 : 0);
#pragma unroll
        for (int b = 0; b < TB; ++b) xp[b] = x + x_row(16 * b + m);
        for (int u = u_begin; u < u_end; ++u) {
            uint32_t fifth[2][FB];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int k = min(u * KUNIT + s * KSTEP + g * EPC, K - EPC);           // (past K: zeroed by compute)
#pragma unroll
                for (int f = 0; f < FB; ++f) {
                    w[s][f].u = ldg_unaligned(wr[f] + k);
                    if (odd) fifth[s][f] = *reinterpret_cast<const uint32_t*>(wr[f] + k + EPC);
                }
#pragma unroll
                for (int b = 0; b < TB; ++b) xr[s][b].u = ldg_unaligned(xp[b] + k);
            }
            if (odd) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int f = 0; f < FB; ++f) {
                        u32x4& q = w[s][f].u;
                        q = u32x4{(q[0] >> 16) | (q[1] << 16), (q[1] >> 16) | (q[2] << 16), (q[2] >> 16) | (q[3] << 16),
                                  (q[3] >> 16) | (fifth[s][f] << 16)};
                    }
            }
            compute(u);
        }
    }
    // leaves this wavefront's partial sums where its operands were (a barrier, then the workgroup adds them up)
    __device__ __forceinline__ void park()
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int f = 0; f < FB; ++f) reinterpret_cast<floatx4*>(own_lds)[(b * FB + f) * 64 + lane] = folded(acc[f][b]);
    }
    // the sum over `waves` (8) wavefronts of block (f, b)
    static __device__ __forceinline__ floatx4 total(int f, int b)
    {
        const int lane = threadIdx.x & 63;
        floatx4 part[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) part[s] = small_lds[s * (LDS_BYTES / 16) + (b * FB + f) * 64 + lane];
#pragma unroll
        for (int st = 4; st > 0; st >>= 1)
#pragma unroll
            for (int s = 0; s < st; ++s) part[s] += part[s + st];
        return part[0];
    }
};

}  // namespace
