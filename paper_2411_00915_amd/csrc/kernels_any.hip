// Shrink and expand for fp32 (v_mfma_f32_16x16x4_f32: fp32 products and sums) and for bf16 batches whose ranks the tuned
// kernels do not take.
//
// Shrink: tiles of 16 FB rank rows x 16 TB tokens of one adapter, the contraction split over the eight wavefronts of a
// workgroup (split_k.h) and over up to four workgroups.  It is bound by reading At and x.  fp32, 256 tokens on 16 adapters
// of rank 8..64, K = 4096: 267 us (one token per workgroup, At read once per token) -> 5.  bf16, K = 4096, lora_shrink
// against 64-byte pieces of 16 rows straight into registers: 256 tokens on 64 adapters of rank 2..256 11.7 -> 10.0 us, 1024
// tokens 19.2 -> 12.4; lora_delta of 1000 single tokens on 24 adapters of rank 256 73 -> 52.
// Expand: 16 or 32 tokens x 64 features per wavefront; bound by y and Bt.
// Delta in one launch: see delta_f32_kernel.
#include "kernels.h"
#include "launch.h"
#include "split_k.h"

#include <atomic>
#include <type_traits>

namespace {

// v[kpart][token][c0 ..] = s_a * (x A_a) over one K part
template <typename E, int FB, int TB, int D, bool KTAIL, int SUMS>
__global__ __launch_bounds__(512) void shrink_rows_kernel(
    const lora_tile* __restrict__ tiles, const int32_t* __restrict__ perm, const E* __restrict__ x, int64_t ldx,
    const E* const* __restrict__ At_ptrs, int K, float* __restrict__ v, lora_vspec vsp)
{
    const lora_tile t = tiles[blockIdx.x];
    const int kpart = (t.shape >> 8) & 15, kparts = (t.shape >> 12) & 15;
    const E* At = At_ptrs[t.adapter] + (int64_t)t.c0 * K;
    const int32_t* rows = perm + t.row0;
    const float s_a = __int_as_float(t.reserved1);
    float* const vp = v + kpart * vsp.part + t.c0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    using slice = split_k<E, FB, TB, D, KTAIL, SUMS>;
    const int units = (K + slice::KUNIT - 1) / slice::KUNIT;
    const int p_begin = units * kpart / kparts, p_end = units * (kpart + 1) / kparts;
    const auto w_row = [&](int row) { return (int64_t)min(row, t.cn - 1) * K; };
    const auto x_row = [&](int row) { return (int64_t)rows[min(row, t.nrows - 1)] * ldx; };
    slice part(K, At, x, wave, w_row, x_row);
    const int u_begin = p_begin + (p_end - p_begin) * wave / 8, u_end = p_begin + (p_end - p_begin) * (wave + 1) / 8;
    // whole lines to LDS need 16-byte rows, and 32-bit offsets a tile of less than 4 GB
    if ((reinterpret_cast<uintptr_t>(At) & 15) == 0 && (int64_t)t.cn * K * (int64_t)sizeof(E) <= (1ll << 32)) part.run(u_begin, u_end);
    else part.run_anywhere(At, x, w_row, x_row, u_begin, u_end);
    part.park();
    __syncthreads();
    // a thread finishes F4 consecutive blocks (4 F4 consecutive rank rows) of one lane's token
    constexpr int ITEMS = FB * TB * 64, F4 = ITEMS > 512 ? ITEMS / 512 : 1;
    if (wave * F4 >= FB * TB) return;
    const int b = wave * F4 / FB, f0 = wave * F4 % FB, row = 16 * b + (lane & 15);
    if (row >= t.nrows) return;
    float* const dst = vp + (int64_t)rows[row] * vsp.R;
#pragma unroll
    for (int f = 0; f < F4; ++f) {
        const floatx4 sum = s_a * slice::total(f0 + f, b);
        const int j = 4 * FB * (lane >> 4) + 4 * (f0 + f);
        if (j + 4 <= t.cn) {
            *reinterpret_cast<floatx4*>(dst + j) = sum;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (j + i < t.cn) dst[j + i] = sum[i];
        }
    }
}

// Four consecutive features of one token: y = beta y + d, rounded once.
__device__ __forceinline__ void finish4(float* yp, floatx4 yin, floatx4 d, float beta, bool vec, int left)
{
    if (vec && left >= 4) {
        if (beta != 0.f)
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = fmaf(beta, yin[i], d[i]);
        *reinterpret_cast<floatx4*>(yp) = d;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < left) yp[i] = beta != 0.f ? fmaf(beta, yp[i], d[i]) : d[i];
    }
}

// Sixteen consecutive features of one token: y = beta y + d, rounded once.  `yin`: what was there, where `vec` (whole,
// aligned 16-byte pieces); the others are read here.
template <typename E>
__device__ __forceinline__ void finish16(E* yp, const u32x4 (&yin)[sizeof(E)], const floatx4 (&d)[4], float beta, bool vec, int left)
{
    if (vec && left >= 16) {
        if constexpr (sizeof(E) == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) finish4(yp + 4 * q, __builtin_bit_cast(floatx4, yin[q]), d[q], beta, true, 4);
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 out;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float e0 = d[2 * h + q / 2][q % 2 * 2], e1 = d[2 * h + q / 2][q % 2 * 2 + 1];
                    if (beta != 0.f) {
                        e0 = fmaf(beta, bf16_to_f32((bf16_t)(yin[h][q] & 0xffffu)), e0);
                        e1 = fmaf(beta, bf16_to_f32((bf16_t)(yin[h][q] >> 16)), e1);
                    }
                    out[q] = (uint32_t)f32_to_bf16(e0) | ((uint32_t)f32_to_bf16(e1) << 16);
                }
                *reinterpret_cast<u32x4*>(yp + 8 * h) = out;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (i < left) {
                const float e = d[i >> 2][i & 3];
                elem<E>::store(yp + i, beta != 0.f ? fmaf(beta, elem<E>::load(yp + i), e) : e);
            }
    }
}

// Expand, 16 TB tokens of one adapter per workgroup, chunks of 64 features per wavefront.  Bt and y come straight from
// memory as each lane needs them (rows of any length, aligned to an element); v is common to the wavefronts and lies in
// LDS as operands (bf16: three terms, all of its 24 bits; with two, lora_delta took 2 to 5 % less).  MFMA row 4 q + i of
// block f stands for feature 16 q + 4 f + i of the chunk: a lane ends with 16 consecutive features of each of its tokens.
//
// Chunks of Bt are fetched whole from where they lie, into the next row if need be and, where they would reach past the
// matrix, from before their place (N >= 8: there is a whole chunk); what is not theirs is shifted out and masked when
// they are used.
// 1000 tokens on 24 adapters of ranks 4 to 256, N = 4096: 123 us (one token per workgroup, Bt a row per thread) -> 15.
// bf16: two steps of Bt on their way, as in the tiles of 16 tokens, leave the tiles of 32 registers for three workgroups on a
// compute unit; a tile is a chain of trips (descriptor, tokens, Bt and y, v, Bt again) of 7 to 15 us, so that what shortens a
// launch is more of them side by side: lora_delta, two workgroups with four steps / three with two: 997 single tokens on 71
// adapters of rank 100, 4096 -> 4096, 52.2 / 48.5; 672 on 61 of rank 100, 5120 -> 13824, 37.6 / 34.4; 299 on 114, 80.1 / 76.4.
// Launches of 300 to 512 tiles, which had a place each before, lose nothing by the shorter reach: 16 batches of ranks 97 to 256
// 1.02 times as fast, between 0.992 and 1.072 (420 tokens on 19 of rank 256, 4096 -> 4096, 30.5 / 28.6).
template <typename E>
__device__ __forceinline__ u32x4 own_elements(u32x4 b, uint32_t drop, int keep)
{
    if constexpr (sizeof(E) == 4) {
        if (drop & 2) b = u32x4{b[2], b[3], 0, 0};
        if (drop & 1) b = u32x4{b[1], b[2], b[3], 0};
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = i < keep ? b[i] : 0u;
    } else {
        if (drop & 4) b = u32x4{b[2], b[3], 0, 0};
        if (drop & 2) b = u32x4{b[1], b[2], b[3], 0};
        if (drop & 1) b = u32x4{(b[0] >> 16) | (b[1] << 16), (b[1] >> 16) | (b[2] << 16), (b[2] >> 16) | (b[3] << 16), b[3] >> 16};
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = 2 * i + 2 <= keep ? b[i] : (2 * i < keep ? b[i] & 0xffffu : 0u);
    }
    return b;
}

// Sixteen features of one token by fp32 products, rank after rank.  The terms of an infinite v, and their products with an
// infinite Bt, add up to NaN also where v Bt is an infinity or a number: sums that came out as NaN are done again.
template <typename E>
__device__ __forceinline__ void plain_tile_row(int tok, const float* __restrict__ v, const lora_vspec& vsp, const E* __restrict__ Bt, int r,
                                               E* __restrict__ y, int64_t ldy, int n, int n_end, float beta)
{
    v += (int64_t)tok * vsp.R;
    y += (int64_t)tok * ldy;
    for (int i = n; i < min(n + 16, n_end); ++i) {
        float d = 0.f;
        for (int j = 0; j < r; ++j) {
            float vj = v[j];
            for (int p = 1; p < vsp.P; ++p) vj += v[p * vsp.part + j];
            d = fmaf(vj, elem<E>::load(Bt + (int64_t)i * r + j), d);
        }
        elem<E>::store(y + i, beta != 0.f ? fmaf(beta, elem<E>::load(y + i), d) : d);
    }
}

template <typename E, int TB>
__device__ __forceinline__ void expand_rows_tile(
    const lora_tile& t, const int32_t* __restrict__ perm, const float* __restrict__ v, const lora_vspec& vsp,
    const E* __restrict__ Bt, E* __restrict__ y, int64_t ldy, int N, float beta, bool y_vec, op16* lds)
{
    constexpr int ES = (int)sizeof(E), EPC = 16 / ES, KSTEP = 4 * EPC, TERMS = ES == 2 ? 3 : 1;
    constexpr int KS = TB == 1 || ES == 2 ? 2 : 4;           // steps of KSTEP ranks whose loads go out together (as many as registers hold)
    constexpr int SUMS = ES == 4 ? 4 / TB : 1;               // (see mma_apart)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
    const int r = t.reserved0, n_end = t.c0 + t.cn, steps = (r + KSTEP - 1) / KSTEP;
    int tok[TB];
#pragma unroll
    for (int b = 0; b < TB; ++b) tok[b] = perm[t.row0 + min(16 * b + m, t.nrows - 1)];
    int n0 = t.c0 + wave * 64;
    op16 bt[KS][4];
    u32x4 yin[TB][ES];
    const uint32_t last = (uint32_t)N * (uint32_t)r - EPC;   // where the matrix's last whole chunk is (N r < 2^31)
    const bool whole = r % EPC == 0;
    auto place = [&](int s, int f) {                         // of the chunk of step s that this lane needs for block f
        const int n = n0 + 16 * (m >> 2) + 4 * f + (m & 3);
        return (uint32_t)min(n, n_end - 1) * (uint32_t)r + (uint32_t)(s * KSTEP + EPC * g);
    };
    auto load_b = [&](int s0) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (s0 + s < steps) {
#pragma unroll
                for (int f = 0; f < 4; ++f) bt[s][f].u = ldg_unaligned(Bt + min(place(s0 + s, f), last));
            }
    };
    auto load_y = [&]() {
        if (beta != 0.f && y_vec && n0 + 16 * g + 16 <= n_end) {
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int q = 0; q < ES; ++q) yin[b][q] = *reinterpret_cast<const u32x4*>(y + (int64_t)tok[b] * ldy + n0 + 16 * g + q * EPC);
        }
    };
    if (n0 < n_end) {                                        // what does not depend on v goes out before it
        load_y();
        load_b(0);
    }
    for (int s = wave; s < steps; s += 4)
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            float f[EPC];
            op16 o[TERMS];
            v_values<EPC>(v, vsp, tok[b], s * KSTEP + EPC * g, r, true, f);
            if constexpr (ES == 4) o[0].f = floatx4{f[0], f[1], f[2], f[3]};
            else bf16_terms<TERMS>(f, o);
#pragma unroll
            for (int t = 0; t < TERMS; ++t) lds[((s * TB + b) * TERMS + t) * 64 + lane] = o[t];
        }
    __syncthreads();
    for (bool first = true; n0 < n_end; n0 += 256, first = false) {
        if (!first) load_y();
        floatx4 acc[TB][4][SUMS];
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int f = 0; f < 4; ++f)
#pragma unroll
                for (int i = 0; i < SUMS; ++i) acc[b][f][i] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < steps; s0 += KS) {
            if (!first || s0 > 0) load_b(s0);
#pragma unroll
            for (int s = 0; s < KS; ++s)
                if (s0 + s < steps) {
                    const int left = r - (s0 + s) * KSTEP - EPC * g;
#pragma unroll
                    for (int f = 0; f < 4; ++f) {
                        if (whole) {
                            if (left <= 0) bt[s][f].u = u32x4{0, 0, 0, 0};
                        } else {
                            const uint32_t at = place(s0 + s, f);
                            bt[s][f].u = own_elements<E>(bt[s][f].u, at > last ? at - last : 0u, left);
                        }
                    }
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        const op16* vp = lds + (((s0 + s) * TB + b) * TERMS) * 64 + lane;
#pragma unroll
                        for (int f = 0; f < 4; ++f) {
                            if constexpr (ES == 4) {
                                mma_apart(bt[s][f], vp[0], acc[b][f], 0);
                            } else {
#pragma unroll
                                for (int t = 0; t < TERMS; ++t) acc[b][f][0] = mma(bt[s][f], vp[t * 64], acc[b][f][0], E{});
                            }
                        }
                    }
                }
        }
        int again = 0;
#pragma unroll
        for (int b = 0; b < TB; ++b)
            if (16 * b + m < t.nrows) {
                floatx4 d[4];
#pragma unroll
                for (int f = 0; f < 4; ++f) d[f] = folded(acc[b][f]);
                bool nan = false;                            // (of features that are not there, too: their sums are a neighbour's)
                if (ES == 2) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) nan |= d[i >> 2][i & 3] != d[i >> 2][i & 3];
                }
                if (nan) again |= 1 << b;
                else finish16<E>(y + (int64_t)tok[b] * ldy + n0 + 16 * g, yin[b], d, beta, y_vec, n_end - n0 - 16 * g);
            }
        if (ES == 2 && again) {
#pragma unroll 1
            for (int b = 0; b < TB; ++b)
                if ((again >> b) & 1) plain_tile_row(perm[t.row0 + 16 * b + m], v, vsp, Bt, r, y, ldy, n0 + 16 * g, n_end, beta);
        }
    }
}

extern __shared__ op16 expand_rows_lds[];

// TBMAX: token blocks of the plan's largest tile (the kernel's register count is that of its widest case: small batches
// get more wavefronts onto a compute unit)
template <typename E, int TBMAX>
__global__ __launch_bounds__(256, TBMAX == 1 || sizeof(E) == 2 ? 3 : 2) void expand_rows_kernel(
    const lora_tile* __restrict__ tiles, const int32_t* __restrict__ perm, const float* __restrict__ v, lora_vspec vsp,
    const E* const* __restrict__ Bt_ptrs, E* __restrict__ y, int64_t ldy, int N, float beta, bool y_vec)
{
    const lora_tile t = tiles[blockIdx.x];
    const E* Bt = Bt_ptrs[t.adapter];
    if (TBMAX >= 2 && t.nrows > 16) expand_rows_tile<E, 2>(t, perm, v, vsp, Bt, y, ldy, N, beta, y_vec, expand_rows_lds);
    else expand_rows_tile<E, 1>(t, perm, v, vsp, Bt, y, ldy, N, beta, y_vec, expand_rows_lds);
}

// Problems so small that launches are what they cost: shrink and expand in one.  A workgroup owns 16 tokens of one adapter
// x 128 features and computes the v of its tokens itself (K split over its eight wavefronts, added up in LDS), once per
// 128 features instead of once.  Bt and y are requested before that.  Ranks up to 64.
// 64 tokens, 256 -> 256, rank 8: kernels of 4.0 + 3.0 us -> one of 4.1, 11.4 -> 7.9 us per call.
// Plans with such tiles run the shrink alone on the same arithmetic, so that both ways give the same bits.

// s_a (x A_a) of the tile's 16 tokens: wavefront j < JB returns ranks 16 j + 4 g + i of token m (zero past the rank)
template <int JB>
__device__ __forceinline__ floatx4 small_v(const lora_tile& t, int tok, const float* __restrict__ x, int64_t ldx,
                                           const float* __restrict__ At, int K, floatx4* lds)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), m = lane & 15, g = lane >> 4;
    const int r = t.reserved0;
    constexpr int SUMS = JB <= 2 ? 8 : 4;
    floatx4 acc[JB][SUMS];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int i = 0; i < SUMS; ++i) acc[jb][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int steps = (K + 15) / 16;
    const float* const xrow = x + (int64_t)tok * ldx;
    const int s_end = steps * (wave + 1) / 8, whole = min(s_end, K / 16);
    int s = steps * wave / 8;
    const float* arow[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) arow[jb] = At + (int64_t)min(16 * jb + m, r - 1) * K;
    auto add = [&](auto n_steps) {                           // whole steps: no chunk is cut, all their loads go out first
        constexpr int U = decltype(n_steps)::value;
        op16 xo[U], a[U][JB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 16 * (s + u) + 4 * g;
            xo[u].u = ldg_unaligned(xrow + k);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) a[u][jb].u = ldg_unaligned(arow[jb] + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) mma_apart(a[u][jb], xo[u], acc[jb], 4 * (u & 1));
        s += U;
    };
    while (s + 4 <= whole) add(std::integral_constant<int, 4>{});
    if (s + 2 <= whole) add(std::integral_constant<int, 2>{});
    if (s < whole) add(std::integral_constant<int, 1>{});
    if (s < s_end) {
        const op16 xo = row_chunk<float>(xrow, 16 * s + 4 * g, K);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) mma_apart(row_chunk<float>(arow[jb], 16 * s + 4 * g, K), xo, acc[jb], 0);
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) lds[(wave * JB + jb) * 64 + lane] = folded(acc[jb]);
    __syncthreads();
    floatx4 part[8];
    if (wave >= JB) return floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 8; ++q) part[q] = lds[(q * JB + wave) * 64 + lane];
#pragma unroll
    for (int st = 4; st > 0; st >>= 1)
#pragma unroll
        for (int q = 0; q < st; ++q) part[q] += part[q + st];
    const float s_a = __int_as_float(t.reserved1);
#pragma unroll
    for (int i = 0; i < 4; ++i) part[0][i] = 16 * wave + 4 * g + i < r ? s_a * part[0][i] : 0.f;
    return part[0];
}

// ... to the rows of v
template <int JB>
__device__ __forceinline__ void store_small_v(const lora_tile& t, int tok, floatx4 e, float* __restrict__ v, const lora_vspec& vsp)
{
    const int lane = threadIdx.x & 63, j = 16 * ((int)threadIdx.x >> 6) + 4 * (lane >> 4);
    if ((lane & 15) >= t.nrows) return;
    float* const dst = v + (int64_t)tok * vsp.R + j;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (j + i < min(t.reserved0, 16 * JB)) dst[i] = e[i];
}

template <int JB>
__device__ __forceinline__ void shrink_small_f32_tile(
    const lora_tile& t, const int32_t* __restrict__ perm, const float* __restrict__ x, int64_t ldx, const float* __restrict__ At, int K,
    float* __restrict__ v, const lora_vspec& vsp, floatx4* lds)
{
    const int tok = perm[t.row0 + min((int)threadIdx.x & 15, t.nrows - 1)];
    store_small_v<JB>(t, tok, small_v<JB>(t, tok, x, ldx, At, K, lds), v, vsp);
}

// (tiles: 16 tokens x all ranks)
__global__ __launch_bounds__(512) void shrink_small_f32_kernel(
    const lora_tile* __restrict__ tiles, const int32_t* __restrict__ perm, const float* __restrict__ x, int64_t ldx,
    const float* const* __restrict__ At_ptrs, int K, float* __restrict__ v, lora_vspec vsp)
{
    __shared__ floatx4 lds[8 * 4 * 64];
    const lora_tile t = tiles[blockIdx.x];
    const float* At = At_ptrs[t.adapter];
    if (t.reserved0 <= 16) shrink_small_f32_tile<1>(t, perm, x, ldx, At, K, v, vsp, lds);
    else if (t.reserved0 <= 32) shrink_small_f32_tile<2>(t, perm, x, ldx, At, K, v, vsp, lds);
    else shrink_small_f32_tile<4>(t, perm, x, ldx, At, K, v, vsp, lds);
}

template <int JB>
__device__ __forceinline__ void delta_f32_tile(
    const lora_tile& t, const int32_t* __restrict__ perm, const float* __restrict__ x, int64_t ldx, const float* __restrict__ At, int K,
    const float* __restrict__ Bt, float* __restrict__ v, const lora_vspec& vsp, float* __restrict__ y, int64_t ldy, float beta, bool y_vec,
    floatx4* lds)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 15, g = lane >> 4;
    const int r = t.reserved0, n_end = t.c0 + t.cn, tok = perm[t.row0 + min(m, t.nrows - 1)];
    // Bt rows and y of this wavefront's 16 features
    const int n0 = t.c0 + 16 * wave, n_lane = n0 + 4 * g;
    float* const yp = y + (int64_t)tok * ldy + n_lane;
    op16 bt[JB];
    floatx4 yin = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < JB; ++s) bt[s] = row_chunk<float>(Bt + (int64_t)min(n0 + m, n_end - 1) * r, 16 * s + 4 * g, r);
    if (beta != 0.f && y_vec && n_lane + 4 <= n_end) yin = *reinterpret_cast<const floatx4*>(yp);

    const floatx4 e = small_v<JB>(t, tok, x, ldx, At, K, lds);
    floatx4* const vt = lds + 8 * JB * 64;                   // v as operands: [JB][64 lanes]
    if (wave < JB) vt[wave * 64 + lane] = e;
    if (v && t.c0 == 0) store_small_v<JB>(t, tok, e, v, vsp);
    __syncthreads();
    floatx4 d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        op16 vo;
        vo.f = vt[j * 64 + lane];
        mma_apart(bt[j], vo, d, 0);
    }
    if (m < t.nrows) finish4(yp, yin, folded(d), beta, y_vec, n_end - n_lane);
}

__global__ __launch_bounds__(512) void delta_f32_kernel(
    const lora_tile* __restrict__ tiles, const int32_t* __restrict__ perm, const float* __restrict__ x, int64_t ldx,
    const float* const* __restrict__ At_ptrs, int K, const float* const* __restrict__ Bt_ptrs, float* __restrict__ v, lora_vspec vsp,
    float* __restrict__ y, int64_t ldy, float beta, bool y_vec)
{
    __shared__ floatx4 lds[9 * 4 * 64];
    const lora_tile t = tiles[blockIdx.x];
    const float *At = At_ptrs[t.adapter], *Bt = Bt_ptrs[t.adapter];
    if (t.reserved0 <= 16) delta_f32_tile<1>(t, perm, x, ldx, At, K, Bt, v, vsp, y, ldy, beta, y_vec, lds);
    else if (t.reserved0 <= 32) delta_f32_tile<2>(t, perm, x, ldx, At, K, Bt, v, vsp, y, ldy, beta, y_vec, lds);
    else delta_f32_tile<4>(t, perm, x, ldx, At, K, Bt, v, vsp, y, ldy, beta, y_vec, lds);
}

template <typename E, int FB, int TB, int D, int SUMS, bool KTAIL>
hipError_t launch_shrink_shape(const lora_plan* p, const lora_dev_tables& d, const void* x, int64_t ldx, const void* const* At, float* v,
                               hipStream_t stream)
{
    constexpr size_t lds_bytes = (size_t)8 * split_k<E, FB, TB, D, KTAIL, SUMS>::LDS_BYTES;
    static_assert(D * (2 * FB + 2 * TB) >= FB * TB && lds_bytes <= 163840, "a wavefront's partial sums go where its operands were");
    if (lds_bytes > 65536) {                                  // dynamic LDS above 64 KB has to be allowed once per kernel
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&shrink_rows_kernel<E, FB, TB, D, KTAIL, SUMS>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    LORA_LAUNCH(LORA_K_SHRINK_ROWS, (shrink_rows_kernel<E, FB, TB, D, KTAIL, SUMS>), dim3((unsigned)p->rows_shrink_tiles.size()), dim3(512),
                lds_bytes, stream, d.rows_shrink_tiles, d.perm, (const E*)x, ldx, (const E* const*)At, p->K, v, lora_vspec_of(p));
    return hipGetLastError();
}

bool vec_rows(const void* y, int64_t ldy, int64_t es) { return ldy * es % 16 == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0; }

}  // namespace

bool shrink_rows_supported(const lora_plan* p, const void* x, int64_t ldx)
{
    if (!p->f32_delta_tiles.empty()) return true;            // (no alignment demands)
    const int64_t es = p->dtype == LORA_F32 ? 4 : 2;
    return !p->rows_shrink_tiles.empty() && ldx * es % 16 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
           (int64_t)p->T * ldx * es < (1ll << 32);           // 32-bit byte offsets
}

hipError_t launch_shrink_rows(const lora_plan* p, const lora_dev_tables& d, const void* x, int64_t ldx, const void* const* At, float* v,
                              hipStream_t stream)
{
    if (!p->f32_delta_tiles.empty()) {
        LORA_LAUNCH(LORA_K_SHRINK_ROWS, shrink_small_f32_kernel, dim3((unsigned)p->rows_shrink_tiles.size()), dim3(512), 0, stream,
                    d.rows_shrink_tiles, d.perm, (const float*)x, ldx, (const float* const*)At, p->K, v, lora_vspec_of(p));
        return hipGetLastError();
    }
#define SHRINK_ROWS(E_, FB_, TB_, D_, SUMS_)                                                                            \
    if (p->rows_shrink_fb == FB_ && p->rows_shrink_tb == TB_ && p->rows_shrink_d == D_)                                 \
        return p->K % (128 / (int)sizeof(E_)) ? launch_shrink_shape<E_, FB_, TB_, D_, SUMS_, true>(p, d, x, ldx, At, v, stream)  \
                                              : launch_shrink_shape<E_, FB_, TB_, D_, SUMS_, false>(p, d, x, ldx, At, v, stream);
    if (p->dtype == LORA_F32) {
        SHRINK_ROWS(float, 1, 1, 2, 8) SHRINK_ROWS(float, 2, 2, 1, 4)
    } else {
        SHRINK_ROWS(bf16_t, 1, 1, 2, 1) SHRINK_ROWS(bf16_t, 2, 1, 1, 1) SHRINK_ROWS(bf16_t, 4, 1, 1, 1)
        SHRINK_ROWS(bf16_t, 2, 2, 1, 1) SHRINK_ROWS(bf16_t, 4, 2, 1, 1) SHRINK_ROWS(bf16_t, 4, 4, 1, 1)
        SHRINK_ROWS(bf16_t, 1, 1, 4, 1) SHRINK_ROWS(bf16_t, 2, 2, 2, 1)
    }
#undef SHRINK_ROWS
    return hipErrorInvalidValue;
}

hipError_t launch_expand_rows(const lora_plan* p, const lora_dev_tables& d, const float* v, const void* const* Bt, void* y, int64_t ldy,
                              float beta, hipStream_t stream)
{
#define EXPAND_ROWS(E_, TBMAX_)                                                                                              \
    LORA_LAUNCH(LORA_K_EXPAND_ROWS, (expand_rows_kernel<E_, TBMAX_>), dim3((unsigned)p->rows_expand_tiles.size()), dim3(256), \
                (size_t)p->rows_expand_lds, stream, d.rows_expand_tiles, d.perm, v, lora_vspec_of(p), (const E_* const*)Bt,   \
                (E_*)y, ldy, p->N, beta, vec_rows(y, ldy, sizeof(E_)))
    if (p->dtype == LORA_F32) {
        if (p->rows_expand_tb == 1) EXPAND_ROWS(float, 1);
        else EXPAND_ROWS(float, 2);
    } else {
        if (p->rows_expand_tb == 1) EXPAND_ROWS(bf16_t, 1);
        else EXPAND_ROWS(bf16_t, 2);
    }
#undef EXPAND_ROWS
    return hipGetLastError();
}

hipError_t launch_delta_f32(const lora_plan* p, const lora_dev_tables& d, const void* x, int64_t ldx, const void* const* At,
                            const void* const* Bt, float* v, void* y, int64_t ldy, float beta, hipStream_t stream)
{
    LORA_LAUNCH(LORA_K_DELTA_F32, delta_f32_kernel, dim3((unsigned)p->f32_delta_tiles.size()), dim3(512), 0, stream, d.f32_delta_tiles,
                d.perm, (const float*)x, ldx, (const float* const*)At, p->K, (const float* const*)Bt, v, lora_vspec_of(p), (float*)y, ldy, beta, vec_rows(y, ldy, 4));
    return hipGetLastError();
}
