// Host-side batch planner: segment table -> token/adapter maps, stable grouping
// by adapter, and the tile lists of the shrink and expand launches.
//
// Stands where ATMM consults its shape-keyed table for the tile configuration of
// the input at hand (paper section 4.3.1, adaptive tiling; section 4.3.2, the
// table built by profiling).  No HIP calls in this file: everything here runs,
// and is tested, without a GPU.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <queue>
#include <utility>
#include <vector>

#include "plan_internal.h"

namespace {
std::mutex g_tuning_mutex;                       // guards the process defaults and the shape table
constexpr lora_tuning kDefaultTuning = {
    /*shrink_waves*/ 8,
    /*shrink_tb2_min_rows*/ 64,
    /*shrink_max_jb*/ 4,
    /*expand_wave_bytes*/ 16384,
    /*expand_tb2_min_rows*/ 64,
    /*expand_tb4_min_rows*/ 1 << 30,
    /*tiled_min_tokens*/ 1,
    /*shrink_small_waves*/ 16,
    /*shrink_small_jb*/ 1,
    /*shrink_target_wgs*/ 768,
    /*fused_wait_us*/ 2001,
    /*fused_delay*/ 3,
    /*expand_wave_bytes_big*/ 131072,
    /*shrink_tb4_min_rows*/ 64,
    /*shrink_stream_min_tokens*/ 1024,
    /*shrink_stream_wgs*/ 512,
    /*expand_stream_stages*/ LORA_EXPAND_BY_ROUNDS,
};
lora_tuning g_lora_tuning = kDefaultTuning;

// The shape table the library ships with: written by the offline search (autotune.py) on MI355X.
const lora_tuning_entry kShippedTable[] = {
#include "tuning_table.inc"
};
constexpr int32_t kShippedCount = (int32_t)(sizeof(kShippedTable) / sizeof(kShippedTable[0]));
std::vector<lora_tuning_entry> g_table(kShippedTable, kShippedTable + kShippedCount);

int32_t rank_class(int32_t r)
{
    int32_t c = 8;
    while (c < r) c *= 2;
    return c;
}

void overlay(lora_tuning* t, const int32_t* values, int32_t count)
{
    int32_t* dst = reinterpret_cast<int32_t*>(t);
    for (int32_t i = 0; i < count && i < LORA_TUNING_COUNT; ++i)
        if (values[i] > 0) dst[i] = values[i];
}

// The tunables of one plan: defaults, then the table entry of the batch's shape class, then the descriptor's own.
void snapshot_tuning(lora_plan* p, const lora_batch_desc* d, int32_t active_tokens, int32_t max_rank, int32_t max_group)
{
    std::lock_guard<std::mutex> lock(g_tuning_mutex);
    p->tuning = g_lora_tuning;
    p->tuning_source = 0;
    // group class: 0 every adapter group below 64 tokens (decode-shaped); 2 groups of 512 tokens or more on average
    // (few long requests, e.g. image-sized prefill); 1 everything between
    const int32_t n_groups = (int32_t)p->group_adapter.size();
    const int32_t rc = rank_class(max_rank),
                  gc = max_group < 64 ? 0 : ((int64_t)active_tokens >= 512ll * std::max(n_groups, 1) ? 2 : 1);
    const lora_tuning_entry* best = nullptr;
    for (const lora_tuning_entry& e : g_table) {
        if (e.k != p->K || e.n != p->N || e.max_rank != rc || e.group_class != gc) continue;
        if (!best) { best = &e; continue; }
        const bool e_covers = e.tokens >= active_tokens, b_covers = best->tokens >= active_tokens;
        if (e_covers != b_covers ? e_covers : (e_covers ? e.tokens < best->tokens : e.tokens > best->tokens)) best = &e;
    }
    if (best && active_tokens > 0) {                             // (a row of zeros: the class keeps the defaults)
        bool any = false;
        for (int32_t i = 0; i < LORA_TUNING_COUNT; ++i) any = any || best->values[i] > 0;
        overlay(&p->tuning, best->values, LORA_TUNING_COUNT);
        if (any) p->tuning_source = 1;
    }
    if (d->tuning && d->tuning_count > 0) {
        bool any = false;
        for (int32_t i = 0; i < d->tuning_count && i < LORA_TUNING_COUNT; ++i) any = any || d->tuning[i] > 0;
        overlay(&p->tuning, d->tuning, d->tuning_count);
        if (any) p->tuning_source += 2;
    }
}
}  // namespace

extern "C" void lora_tuning_set(const int32_t* values, int32_t count)
{
    if (!values) return;
    std::lock_guard<std::mutex> lock(g_tuning_mutex);
    overlay(&g_lora_tuning, values, count);
}

extern "C" void lora_tuning_get(int32_t* values, int32_t count)
{
    if (!values) return;
    std::lock_guard<std::mutex> lock(g_tuning_mutex);
    const int32_t* src = reinterpret_cast<const int32_t*>(&g_lora_tuning);
    for (int32_t i = 0; i < count && i < LORA_TUNING_COUNT; ++i) values[i] = src[i];
}

extern "C" lora_status lora_tuning_table_set(const lora_tuning_entry* entries, int32_t count)
{
    if (count < 0 || (count > 0 && !entries)) return LORA_ERR_INVALID_ARG;
    for (int32_t i = 0; i < count; ++i)
        if (entries[i].tokens < 0 || entries[i].k < 1 || entries[i].n < 1 || entries[i].max_rank != rank_class(entries[i].max_rank) ||
            entries[i].max_rank > LORA_MAX_RANK || entries[i].group_class < 0 || entries[i].group_class > 2)
            return LORA_ERR_INVALID_ARG;
    try {
        std::vector<lora_tuning_entry> next = count ? std::vector<lora_tuning_entry>(entries, entries + count)
                                                    : std::vector<lora_tuning_entry>(kShippedTable, kShippedTable + kShippedCount);
        std::lock_guard<std::mutex> lock(g_tuning_mutex);
        g_table.swap(next);
    } catch (const std::bad_alloc&) {
        return LORA_ERR_NOMEM;
    }
    return LORA_OK;
}

extern "C" int32_t lora_tuning_table_get(lora_tuning_entry* entries, int32_t capacity)
{
    std::lock_guard<std::mutex> lock(g_tuning_mutex);
    if (entries)
        for (int32_t i = 0; i < capacity && i < (int32_t)g_table.size(); ++i) entries[i] = g_table[i];
    return (int32_t)g_table.size();
}

static bool validate(const lora_batch_desc* d)
{
    if (d->num_tokens < 0 || d->num_segments < 0 || d->num_adapters < 0) return false;
    if (d->k < 1 || d->n < 1) return false;
    if (d->dtype != LORA_F32 && d->dtype != LORA_BF16) return false;
    if (d->variant < LORA_VARIANT_AUTO || d->variant > LORA_VARIANT_TILED) return false;
    if (d->tuning_count < 0 || (d->tuning_count > 0 && !d->tuning)) return false;
    if (d->merged_adapter_plus1 < 0 || d->merged_adapter_plus1 > d->num_adapters) return false;
    if (!d->seg_indptr) return false;                       // even S = 0 has the single entry [0]
    if (d->num_segments > 0 && !d->seg_adapter) return false;
    if (d->num_adapters > 0 && (!d->adapter_rank || !d->adapter_scale)) return false;
    if (d->seg_indptr[0] != 0) return false;
    for (int32_t s = 0; s < d->num_segments; ++s) {
        if (d->seg_indptr[s + 1] < d->seg_indptr[s]) return false;
        const int32_t a = d->seg_adapter[s];
        if (a < -1 || a >= d->num_adapters) return false;
    }
    if (d->seg_indptr[d->num_segments] != d->num_tokens) return false;
    for (int32_t a = 0; a < d->num_adapters; ++a) {
        if (d->adapter_rank[a] < 0 || d->adapter_rank[a] > LORA_MAX_RANK) return false;
        if (!std::isfinite(d->adapter_scale[a])) return false;
    }
    return true;
}

static int32_t round_up(int32_t v, int32_t m) { return (v + m - 1) / m * m; }

// Tiles of 16 fb rank rows x 16 tb tokens of one adapter that the batch is
static int64_t rows_shrink_tiles_of(const lora_plan* p, int32_t fb, int32_t tb)
{
    int64_t tiles = 0;
    for (size_t g = 0; g < p->group_adapter.size(); ++g)
        tiles += (int64_t)((p->group_offset[g + 1] - p->group_offset[g] + 16 * tb - 1) / (16 * tb)) *
                 ((p->rank[p->group_adapter[g]] + 16 * fb - 1) / (16 * fb));
    return tiles;
}

struct rows_shape { int32_t fb, tb, d; };
static const rows_shape kRowsF32[] = {{2, 2, 1}, {1, 1, 2}}, kRowsBf16[] = {{4, 4, 1}, {4, 2, 1}, {2, 2, 1}, {4, 1, 1}, {2, 1, 1}, {1, 1, 2}};

// Whether a batch of the streaming shrink goes to the one that splits K over its wavefronts, and then its tile and K parts.  A
// streaming tile walks its K part in stages, one after the other, whatever else is idle: with few tiles the launch is that
// chain.  The other kernel's is shorter (8 wavefronts, each with `d` units of 128 bytes per row on their way), but it asks for
// more: an adapter's rows for every 16 tb tokens, x for every 16 fb ranks.  Microseconds, fitted to 70 batches with x and At from
// memory; a K part more is another read of v by whoever takes it.  lora_shrink, K = 11008, streaming / this: 128 tokens of rank
// 16 14.6 / 4.7, rank 128 20.8 / 5.6; 300 tokens on 3 adapters of rank 64 15.5 / 7.7; 535 on 5 of rank 64 15.9 / 9.6, of rank 128
// 23.6 / 16.1; not taken: 2000 on 8 of rank 64 17.5 / 19.7.  What it is chosen for is lora_delta: fewer parts are the expand's gain,
// and lora_shrink by itself loses near the line (391 drawn calls 0.83 times as long, 55 of them over 1.02: 1831 tokens of rank
// 16, K = 4096, four parts to one, 7.1 -> 8.1).  Not where the streaming shrink's own tunables were given other values
// than the defaults: whoever gives them steers, or searches, that kernel's tiles and K parts.
static bool choose_rows_shrink(lora_plan* p, int32_t max_rank)
{
    if (p->tuning.shrink_stream_min_tokens != kDefaultTuning.shrink_stream_min_tokens ||
        p->tuning.shrink_stream_wgs != kDefaultTuning.shrink_stream_wgs)
        return false;
    if (p->unmerge || p->is_removal || (int64_t)p->shrink_tiles.size() * p->v_parts > 256) return false;   // (mixture mode: one launch for both)
    static const rows_shape shapes[] = {{4, 4, 1}, {2, 2, 2}, {1, 1, 4}};
    const double part_us = 0.3 + 0.008 * max_rank;
    const int32_t own_parts = p->v_parts, stages = ((p->K + 31) / 32 / own_parts + 3) / 4, units = (p->K + 63) / 64;
    double best = 3.3 + stages * (0.3 + 0.005 * max_rank) + own_parts * part_us;
    bool rows = false;
    for (const rows_shape& s : shapes) {
        const int64_t tiles = rows_shrink_tiles_of(p, s.fb, s.tb);
        for (int32_t P = 1; P <= 4 && units / P >= 8; P *= 2) {
            // (lora_delta_static keeps v in an array of its own: parts must not be what outgrows it)
            if (P > own_parts && (size_t)P * p->T * p->R * sizeof(float) > LORA_STATIC_V_BYTES) break;
            const int64_t per_unit = 160 / (16 * s.d * (s.fb + s.tb)), rounds = (tiles * P + 256 * per_unit - 1) / (256 * per_unit);
            const double trips = std::max(1.0, units / (8.0 * P * s.d)), bytes = (s.fb + s.tb) * 32.0 * p->K * tiles;
            // (the 64 x 64 tile: eight wavefronts' sums of 16 blocks meet at its end.  Without that microsecond 87 of 700 drawn
            // lora_delta calls at the line took over 1.02 times as long, 1500 tokens of rank 64, 11008 -> 4096, 27.9 -> 29.8 us)
            const double us = 2.6 + (s.fb == 4 ? 1.0 : 0.0) + std::max(2.5 * trips * rounds, bytes / 7e6) + P * part_us;
            if (us < best) {
                best = us;
                rows = true;
                p->rows_shrink_fb = s.fb;
                p->rows_shrink_tb = s.tb;
                p->rows_shrink_d = s.d;
                p->v_parts = P;
            }
        }
    }
    return rows;
}

// When a launch ends whose tiles, `count` times `ns` each, longest first, are taken by 256 compute units as these get free
struct equal_tiles { int64_t ns, count; };
static int64_t list_schedule_end(const std::vector<equal_tiles>& longest_first)
{
    typedef std::pair<int64_t, int64_t> units;               // free from then on, how many
    std::vector<units> heap{{0, 256}};
    const std::greater<units> later;
    int64_t end = 0;
    for (const equal_tiles& t : longest_first)
        for (int64_t left = t.count; left > 0;) {
            std::pop_heap(heap.begin(), heap.end(), later);
            units& u = heap.back();
            const int64_t take = std::min(u.second, left);
            const units busy{u.first + t.ns, take};
            left -= take;
            if ((u.second -= take) == 0) heap.pop_back();
            else std::push_heap(heap.begin(), heap.end(), later);
            heap.push_back(busy);
            std::push_heap(heap.begin(), heap.end(), later);
            end = std::max(end, busy.first);
        }
    return end;
}

// Tiles of the streaming expand from its token tiles: `stages` stages of features each, or, with stages = 0, as many as end the
// launch earliest.  A compute unit has one tile at a time, and a tile takes about as long for few tokens as for many, for short
// ranks as for long (few tokens take more features a stage, and short ranks too): microseconds by time stamps in a launch of 992
// tiles, 3.3, 4.6 and 5.5 until the first stage with ranks up to 32, 64 and 128, and 1.1 to 1.4 a stage.  What a launch loses is its
// last round: that one took 114 where its tiles took 90 for each compute unit.  So the feature ranges are as long as some number of
// rounds of the 256 compute units makes them, the one that ends first with the longest tiles first, and half of the longest
// tile is counted for what tiles of one model differ by.  A launch of many rounds takes no less than memory does, y
// and each adapter's Bt once at 5 TB/s: up to there shorter tiles, whose starts then are hidden, cost nothing.
// lora_delta, 16 stages, halved down to four while there were fewer than
// 512 tiles / so: 8192 mixed tokens on 128 adapters, 4096 -> 11008, 136.6 / 132.2 us; 4671 on 3 of rank 64, 11008 -> 4096, 64.6 /
// 55.9; 1732 on 23 of rank 16, 4840 -> 4304, 22.0 / 19.4; 468 on 3, 4096 -> 4096, 13.4 / 10.7; 49608 on 412 of rank 64, 1024 -> 11008,
// 532 / 509 (604 with y uncut, 414 tiles, which end a second round with 158); 70000 on 40 of rank 128, 1024 -> 4096, 300 / 300 (uncut
// 395).  200 drawn calls of 128 to 70000 tokens 1.07 times as fast, seven below 0.95 (36287 on 2 of rank 64, 1024 -> 4096, 141 / 155:
// the estimate takes 13 stages, 8 are the best).  (Without that half, 3 % slower for the first of these.)
static void deal_expand_features(lora_plan* p, const std::vector<lora_tile>& blocks, int32_t stages)
{
    constexpr int64_t kComputeUnits = 256;
    auto features = [](const lora_tile& t) { return 64 * lora_shape_jb(t.shape); };          // of a stage
    auto all_stages = [&](const lora_tile& t) { return (p->N + features(t) - 1) / features(t); };
    // stages of a tile: an equal share
    auto share = [](int32_t all, int32_t longest) {
        const int32_t n = (all + longest - 1) / longest;
        return (all + n - 1) / n;
    };
    auto nanoseconds = [](const lora_tile& t, int32_t n) {
        return t.reserved0 <= 32 ? 3300 + 1130 * (int64_t)n : t.reserved0 <= 64 ? 4600 + 1360 * (int64_t)n : 5500 + 1330 * (int64_t)n;
    };
    int32_t longest = stages;
    if (stages == 0) {
        // token tiles of a kind have the same stages and take the same time: three lengths of rank, one to eight chunks a stage
        struct kind { const lora_tile* tile; int32_t all; int64_t count; };
        kind kinds[3][9] = {};
        std::vector<kind> in_use;
        int32_t most = 1;
        int64_t moved = 0;                                   // values of each feature: of y, read and written, and of Bt, once
        int32_t group = -1;
        for (const lora_tile& t : blocks) {
            kind& k = kinds[t.reserved0 <= 32 ? 0 : t.reserved0 <= 64 ? 1 : 2][lora_shape_jb(t.shape)];
            if (k.count++ == 0) k = kind{&t, all_stages(t), 1};
            moved += 2 * (int64_t)t.nrows + (t.reserved1 != group ? t.reserved0 : 0);
            group = t.reserved1;
        }
        for (const auto& of_rank : kinds)
            for (const kind& k : of_rank)
                if (k.count) {
                    in_use.push_back(k);
                    most = std::max(most, k.all);
                }
        const int64_t at_least = moved * 2 * p->N / 5000;
        auto tiles_of = [&](int32_t n) {
            int64_t tiles = 0;
            for (const kind& k : in_use) tiles += k.count * ((k.all + n - 1) / n);
            return tiles;
        };
        std::vector<equal_tiles> runs;
        int64_t best = 0;
        int32_t tried = 0;
        for (int64_t rounds = std::max<int64_t>(1, ((int64_t)blocks.size() + kComputeUnits - 1) / kComputeUnits); tried != 1; rounds += std::max<int64_t>(1, rounds / 4)) {
            int32_t lo = 1, hi = most;                       // the shortest ranges that make no more tiles than that
            while (lo < hi) {
                const int32_t mid = (lo + hi) / 2;
                if (tiles_of(mid) <= rounds * kComputeUnits) hi = mid;
                else lo = mid + 1;
            }
            if (lo == tried) continue;                       // (more rounds may still make shorter ones)
            tried = lo;
            runs.clear();
            int64_t sum = 0;
            for (const kind& k : in_use) {
                const int32_t per = share(k.all, lo), n = (k.all + per - 1) / per;
                if (n > 1) runs.push_back({nanoseconds(*k.tile, per), (n - 1) * k.count});
                runs.push_back({nanoseconds(*k.tile, k.all - (n - 1) * per), k.count});
                sum += k.count * ((n - 1) * nanoseconds(*k.tile, per) + runs.back().ns);
            }
            if (best != 0 && sum / kComputeUnits >= best) break;         // and more tiles are more in all
            std::sort(runs.begin(), runs.end(), [](const equal_tiles& x, const equal_tiles& y) { return x.ns > y.ns; });
            const int64_t end = std::max(list_schedule_end(runs), at_least) + runs[0].ns / 2;
            if (best != 0 && end >= best) continue;
            best = end;
            longest = lo;
        }
    }
    // (a block's tiles are all as long, the last one aside: sorted by blocks)
    struct run { int64_t ns; int32_t block, first, end, per; };
    std::vector<run> runs;
    for (int32_t i = 0; i < (int32_t)blocks.size(); ++i) {
        const int32_t all = all_stages(blocks[i]), per = stages ? stages : share(all, longest), whole = all / per * per;
        if (stages || whole == all) {
            runs.push_back({nanoseconds(blocks[i], per), i, 0, all, per});
        } else {
            if (whole > 0) runs.push_back({nanoseconds(blocks[i], per), i, 0, whole, per});
            runs.push_back({nanoseconds(blocks[i], all - whole), i, whole, all, per});
        }
    }
    if (stages == 0) std::stable_sort(runs.begin(), runs.end(), [](const run& x, const run& y) { return x.ns > y.ns; });
    for (const run& r : runs)
        for (int32_t st = r.first; st < r.end; st += r.per) {
            lora_tile t = blocks[r.block];
            t.c0 = st * features(t);
            t.cn = (int32_t)std::min<int64_t>((int64_t)r.per * features(t), p->N - t.c0);
            p->expand_tiles.push_back(t);
        }
}

// Tile lists of the tiled (MFMA) family.  A shrink tile is 16*TB tokens of one
// adapter times 16*JB of its rank indices over the whole K range (the
// workgroup's wavefronts split K).  An expand tile is 16*TB tokens times a range
// of output features that the workgroup's four wavefronts split evenly.
// shrink_only: tiles for the shrink alone (ranks the expand kernels cannot take), for the kernels that tile the rank
// axis in blocks of 16 rows -- no streaming, no single launch.
static void build_tiles(lora_plan* p, bool shrink_only = false)
{
    const lora_tuning& tu = p->tuning;
    p->shrink_max_blocks = 1;
    p->shrink_small = true;
    p->expand_small = true;
    const int G = (int)p->group_adapter.size();
    // Prefill-sized batches (ranks up to 128) take the streaming shrink; its tiles hold 128 tokens, or 64
    // when 128 would leave the launch with few workgroups even after the K split.
    // Smaller batches take it too when they cannot run as the single decode launch (a group too long or a rank
    // too high for the small tiles) and have a group of at least 64 tokens or 128 tokens in all: measured, the
    // streaming kernels then need 18-33 us where the 32- and 64-token tiles of the other family need 24-52.
    int32_t max_rank = 0, max_group = 0;
    bool small_tiles_only = true;
    for (int g = 0; g < G; ++g) {
        const int32_t r = p->rank[p->group_adapter[g]], m = p->group_offset[g + 1] - p->group_offset[g];
        max_rank = std::max(max_rank, r);
        max_group = std::max(max_group, m);
        if (m >= tu.shrink_tb2_min_rows || m >= tu.shrink_tb4_min_rows || m >= tu.expand_tb2_min_rows ||
            m >= tu.expand_tb4_min_rows || r > 64)
            small_tiles_only = false;
    }
    const int64_t active = (int64_t)p->perm.size();
    p->shrink_stream = max_rank <= 128 && p->K >= 1024 &&
                       (active >= tu.shrink_stream_min_tokens ||
                        (tu.shrink_stream_min_tokens < (1 << 30) && !small_tiles_only && (max_group >= 64 || active >= 128)));
    if (shrink_only) p->shrink_stream = false;
    p->expand_stream = p->shrink_stream && p->N >= 64 && p->N % 8 == 0;       // it stores whole 16-byte pieces of a row
    p->expand_stream_ks = 1;
    p->expand_stream_lds = 0;
    int32_t stream_tokens = 128;
    if (p->shrink_stream) {
        int64_t n128 = 0;
        for (int g = 0; g < G; ++g) n128 += (p->group_offset[g + 1] - p->group_offset[g] + 127) / 128;
        if (n128 * 4 < tu.shrink_stream_wgs) stream_tokens = 64;
    }
    // streaming expand: feature range per workgroup, in stages, where the caller or the shape table gives one; halved while the
    // launch would have fewer than two workgroups per CU (but at least 4 stages: the start-up of a tile has to pay off).
    // Otherwise deal_expand_features chooses the ranges.
    const bool expand_by_rounds = tu.expand_stream_stages >= LORA_EXPAND_BY_ROUNDS;
    int32_t expand_stages = expand_by_rounds ? 16 : std::max(1, tu.expand_stream_stages);
    // (its token tiles: 128 tokens -- every token tile of an adapter fetches Bt_a again, and the launch has feature
    // ranges to make workgroups of -- unless that leaves fewer than two rounds of tiles, counted with ranges of 16 stages
    // where they are not chosen yet)
    int32_t expand_tokens = 128;
    if (p->expand_stream) {
        auto token_tiles = [&](int32_t per) {
            int64_t n = 0;
            for (int g = 0; g < G; ++g) n += (p->group_offset[g + 1] - p->group_offset[g] + per - 1) / per;
            return n;
        };
        auto ranges = [&](int64_t features) { return (p->N + features - 1) / features; };   // (given stages may be more than 32 bits of features)
        if (token_tiles(128) * ranges((int64_t)expand_stages * 64) < 512) expand_tokens = stream_tokens;
        const int64_t n_tt = token_tiles(expand_tokens);
        while (expand_stages > 4 && n_tt * ranges((int64_t)expand_stages * 64) < 512) expand_stages /= 2;
    }
    std::vector<lora_tile> expand_blocks;                    // streaming expand: token tiles, features not yet dealt out
    for (int g = 0; g < G; ++g) {
        const int32_t a = p->group_adapter[g];
        const int32_t r = p->rank[a];
        const int32_t lo = p->group_offset[g], hi = p->group_offset[g + 1];
        const int32_t m = hi - lo;

        // ---- shrink, prefill-sized batches: streaming tiles of up to 128 (or 64) tokens over all rank rows
        if (p->shrink_stream) {
            const int jblocks = (r + 15) / 16;
            const int jbk = jblocks <= 1 ? 1 : (jblocks <= 2 ? 2 : (jblocks <= 4 ? 4 : 8));
            for (int32_t row = lo; row < hi; row += stream_tokens) {
                lora_tile t{};
                t.adapter = a; t.row0 = row; t.nrows = std::min<int32_t>(stream_tokens, hi - row);
                t.c0 = 0; t.cn = r;
                const int nblk = (t.nrows + 15) / 16;
                t.shape = lora_shape_code(nblk > 4 ? 8 : (nblk > 2 ? 4 : 2), jbk) | ((g & 0xffff) << 16);
                t.reserved0 = r;
                std::memcpy(&t.reserved1, &p->scale[a], sizeof(float));
                p->shrink_max_blocks = std::max(p->shrink_max_blocks, jbk);
                p->shrink_small = false;
                p->shrink_tiles.push_back(t);
            }
        } else
        // ---- shrink: groups with many tokens take 32- or 64-token tiles over up to 64
        // rank rows (x is the big stream, and At is re-read once per tile); groups with few tokens
        // take 16-token tiles over 16 (or 32) rank rows so that the launch has
        // many workgroups (A is the big stream, each byte is read once anyway)
        {
            const int jblocks = (r + 15) / 16;
            const bool large = m >= tu.shrink_tb2_min_rows;
            const int tb = m >= tu.shrink_tb4_min_rows ? 4 : (large ? 2 : 1);
            const int jb = std::min(jblocks, large ? std::max(1, std::min(tu.shrink_max_jb, 4))
                                                   : std::max(1, std::min(tu.shrink_small_jb, 2)));
            for (int32_t row = lo; row < hi; row += 16 * tb) {
                const int32_t nrows = std::min<int32_t>(16 * tb, hi - row);
                for (int32_t j0 = 0; j0 < r; j0 += 16 * jb) {
                    lora_tile t{};
                    t.adapter = a; t.row0 = row; t.nrows = nrows;
                    t.c0 = j0; t.cn = std::min<int32_t>(16 * jb, r - j0);
                    const int tbk = nrows > 32 ? 4 : (nrows > 16 ? 2 : 1), jbk = (t.cn + 15) / 16;
                    t.shape = lora_shape_code(tbk, jbk) | ((g & 0xffff) << 16);   // bits 16..31: adapter group
                    t.reserved0 = r;
                    std::memcpy(&t.reserved1, &p->scale[a], sizeof(float));   // s_a travels with the tile
                    p->shrink_max_blocks = std::max(p->shrink_max_blocks, tbk * jbk);
                    if (tbk != 1 || jbk > 2) p->shrink_small = false;
                    p->shrink_tiles.push_back(t);
                }
            }
        }
        // ---- expand, prefill-sized batches: streaming tiles, the same token ranges as the streaming shrink;
        // with fewer than 8 token blocks the wavefronts also spread over FW 64-feature chunks per stage
        // (as far as the slab of Bt rows, 64 FW x 32 KS ranks, stays within 32 KB)
        if (shrink_only) {
            p->expand_small = false;
        } else if (p->expand_stream) {
            const int ks = r <= 32 ? 1 : (r <= 64 ? 2 : 4);
            const int fw_max = 8 / ks;
            for (int32_t row = lo; row < hi; row += expand_tokens) {
                const int32_t nrows = std::min<int32_t>(expand_tokens, hi - row);
                const int nblk = (nrows + 15) / 16;
                const int nb = nblk > 4 ? 8 : (nblk > 2 ? 4 : (nblk > 1 ? 2 : 1));
                const int fw = std::min(8 / nb, fw_max);
                lora_tile t{};
                t.adapter = a; t.row0 = row; t.nrows = nrows;
                t.shape = lora_shape_code(nb, fw);
                t.reserved0 = r;
                t.reserved1 = g;
                p->expand_small = false;
                p->expand_stream_ks = std::max(p->expand_stream_ks, ks);
                p->expand_stream_lds = std::max(p->expand_stream_lds, fw * ks * 4 * 2048 + 8 * 16 * 68 * 4);
                expand_blocks.push_back(t);
            }
        } else
        // ---- expand ----
        {
            int tb = 1;
            if (m >= tu.expand_tb4_min_rows && r <= 64) tb = 4;
            else if (m >= tu.expand_tb2_min_rows) tb = 2;
            // output features per wavefront: a multiple of 64, sized so that the
            // wavefront streams about expand_wave_bytes of Bt and y
            const int64_t per_n = 2 * (int64_t)r + 4 * 16 * (int64_t)tb;
            // (long ranges for big groups and big batches: the wavefront loops with the next chunk in flight;
            // short ranges for decode-sized batches, where the launch is one round of memory latency)
            const int64_t wave_bytes = (tb > 1 || p->perm.size() >= 1024) ? tu.expand_wave_bytes_big : tu.expand_wave_bytes;
            int32_t nw = (int32_t)std::max<int64_t>(64, (wave_bytes / per_n) / 64 * 64);
            const int32_t n_tile = 4 * nw;
            for (int32_t row = lo; row < hi; row += 16 * tb) {
                const int32_t nrows = std::min<int32_t>(16 * tb, hi - row);
                for (int32_t n0 = 0; n0 < p->N; n0 += n_tile) {
                    lora_tile t{};
                    t.adapter = a; t.row0 = row; t.nrows = nrows;
                    t.c0 = n0; t.cn = std::min<int32_t>(n_tile, p->N - n0);
                    const int tbk = (nrows + 15) / 16;
                    t.shape = lora_shape_code(tbk == 3 ? 4 : tbk, 0);
                    t.reserved0 = r;
                    t.reserved1 = g;                                             // adapter group
                    if (tbk != 1 || r > 64) p->expand_small = false;
                    p->expand_tiles.push_back(t);
                }
            }
        }
    }
    if (p->expand_stream) deal_expand_features(p, expand_blocks, expand_by_rounds ? 0 : expand_stages);
    // wavefronts per shrink workgroup: they split K in steps of 32; the LDS
    // reduction buffer (1 KB per wavefront and 16x16 block) stays within 64 KB
    const int steps = (p->K + 31) / 32;
    // Small build: a workgroup's bandwidth is bounded (one CU), so a launch with
    // fewer workgroups than CUs leaves HBM idle.  Split K over P workgroups per
    // tile (P in 1, 2, 4); each part writes its own slice of v and every consumer
    // of v adds the parts in order, so there are no atomics and no zeroing.
    p->v_parts = 1;
    {
        int P = 1;
        // (the streaming shrink has 8 wavefronts per workgroup and long tiles: half as many workgroups do)
        const int64_t target = p->shrink_stream ? std::max(1, tu.shrink_stream_wgs / 2) : tu.shrink_target_wgs;
        while (P < 4 && (int64_t)p->shrink_tiles.size() * P < target && steps / (2 * P) >= 8) P *= 2;
        p->v_parts = P;
        if (p->shrink_stream && p->variant_req == LORA_VARIANT_AUTO) p->shrink_by_rows = choose_rows_shrink(p, max_rank);
    }
    {
        std::vector<lora_tile> split;
        split.reserve(p->shrink_tiles.size() * p->v_parts);
        for (const lora_tile& t : p->shrink_tiles)
            for (int q = 0; q < p->v_parts; ++q) {
                lora_tile u = t;
                u.shape |= (q << 8) | (p->v_parts << 12);
                split.push_back(u);
            }
        p->shrink_tiles.swap(split);
    }
    if (p->shrink_stream)
        p->shrink_waves = 8;
    else if (p->shrink_small)
        p->shrink_waves = std::max(1, std::min({tu.shrink_small_waves / p->v_parts, 16, steps / p->v_parts}));
    else
        p->shrink_waves = std::max(1, std::min({tu.shrink_waves, 8, 64 / p->shrink_max_blocks, steps / p->v_parts}));
    // Single-launch decode kernel: an expand tile carries (bits 8..31 of its shape)
    // the numbers of shrink tiles
    // (bits 8..19 of its shape) and of expand tiles (bits 20..31) of its adapter group.
    p->fused_ok = p->shrink_small && p->expand_small && G <= 4096;
    p->fused_wait_us = tu.fused_wait_us - 1;
    p->fused_delay = std::max(0, std::min(tu.fused_delay - 1, 64));
    // The single launch holds 5 workgroups per compute unit at a time (1280 on the 256 units of an MI355X).  A few
    // workgroups beyond that start only when earlier ones end, microseconds into a launch that lasts little longer,
    // and then end it late.  While the launch is over that number by less than a tenth, the expand tiles of the
    // adapter groups with the least bytes per tile (lowest rank first, then fewest tokens) are joined in pairs
    // along the features -- they are the cheapest to double.
    constexpr size_t kResidentWorkgroups = 1280;
    if (p->fused_ok && p->shrink_tiles.size() + p->expand_tiles.size() > kResidentWorkgroups &&
        (p->shrink_tiles.size() + p->expand_tiles.size()) * 10 <= kResidentWorkgroups * 11) {
        std::vector<int> groups((size_t)G);
        for (int g = 0; g < G; ++g) groups[(size_t)g] = g;
        std::stable_sort(groups.begin(), groups.end(), [&](int a, int b) {
            const int32_t ra = p->rank[p->group_adapter[a]], rb = p->rank[p->group_adapter[b]];
            if (ra != rb) return ra < rb;
            return p->group_offset[a + 1] - p->group_offset[a] < p->group_offset[b + 1] - p->group_offset[b];
        });
        std::vector<char> join((size_t)G, 0);
        size_t total = p->shrink_tiles.size() + p->expand_tiles.size();
        std::vector<size_t> tiles_of((size_t)G, 0);
        for (const lora_tile& t : p->expand_tiles) tiles_of[(size_t)t.reserved1] += 1;
        for (int g : groups) {
            if (total <= kResidentWorkgroups) break;
            join[(size_t)g] = 1;
            total -= tiles_of[(size_t)g] / 2;
        }
        std::vector<lora_tile> joined;
        joined.reserve(p->expand_tiles.size());
        for (size_t i = 0; i < p->expand_tiles.size(); ++i) {
            lora_tile t = p->expand_tiles[i];
            if (join[(size_t)t.reserved1] && i + 1 < p->expand_tiles.size()) {
                const lora_tile& n = p->expand_tiles[i + 1];
                if (n.reserved1 == t.reserved1 && n.row0 == t.row0 && n.c0 == t.c0 + t.cn) {
                    t.cn += n.cn;
                    ++i;
                }
            }
            joined.push_back(t);
        }
        p->expand_tiles.swap(joined);
    }
    if (p->fused_ok) {
        std::vector<int32_t> need((size_t)G, 0), ncons((size_t)G, 0);
        for (const lora_tile& t : p->shrink_tiles) need[(size_t)((uint32_t)t.shape >> 16)] += 1;
        for (const lora_tile& t : p->expand_tiles) ncons[(size_t)t.reserved1] += 1;
        for (int g = 0; g < G; ++g)
            if (need[g] > 4095 || ncons[g] > 4095) p->fused_ok = false;
        if (p->fused_ok)
            for (lora_tile& t : p->expand_tiles)
                t.shape |= (need[(size_t)t.reserved1] << 8) | (int32_t)((uint32_t)ncons[(size_t)t.reserved1] << 20);
    }
    // Heaviest tiles first so the tail of the launch is made of light ones;
    // stable, so equal descriptors give identical lists.
    auto weight = [&](const lora_tile& t) { return (int64_t)((t.nrows + 15) / 16) * t.cn; };
    std::stable_sort(p->shrink_tiles.begin(), p->shrink_tiles.end(),
                     [&](const lora_tile& x, const lora_tile& y) { return weight(x) > weight(y); });
    // (the streaming expand's tiles differ in size by up to 8x: the same for them)
    if (p->expand_stream && !expand_by_rounds) {
        std::stable_sort(p->expand_tiles.begin(), p->expand_tiles.end(),
                         [&](const lora_tile& x, const lora_tile& y) { return weight(x) > weight(y); });
        // Workgroups start in index order, one per compute unit at a time.  With equal tiles a launch of 3.3
        // rounds of them takes 4: so towards the end of the list the tiles shrink (guided self-scheduling): a
        // tile heavier than its share of what is left -- the remaining work over the number of compute units --
        // is cut along the features into 2 or 4, as long as a piece keeps at least 4 stages (the start-up of a
        // tile has to pay off).
        constexpr int64_t kComputeUnits = 256;
        int64_t remaining = 0;
        for (const lora_tile& t : p->expand_tiles) remaining += weight(t);
        std::vector<lora_tile> cut;
        cut.reserve(p->expand_tiles.size() + 4 * (size_t)kComputeUnits);
        for (const lora_tile& t : p->expand_tiles) {
            const int64_t w = weight(t);
            const int32_t stage = 64 * lora_shape_jb(t.shape);           // features per stage (64 FW)
            const int32_t stages = (t.cn + stage - 1) / stage;
            int32_t pieces = 1;
            while (pieces < 4 && w / pieces > std::max<int64_t>(remaining / kComputeUnits, 1) && stages / (pieces * 2) >= 4)
                pieces *= 2;
            const int32_t per = (stages + pieces - 1) / pieces * stage;
            for (int32_t c = 0; c < t.cn; c += per) {
                lora_tile q = t;
                q.c0 = t.c0 + c;
                q.cn = std::min(per, t.cn - c);
                cut.push_back(q);
            }
            remaining -= w;
        }
        // Taken only if it pays: finish time of both lists when every compute unit takes the next tile as soon as
        // it is free, a tile costing its weight plus a start-up of about two stages.
        auto finish = [&](const std::vector<lora_tile>& tiles) {
            std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> free_at;
            for (int64_t c = 0; c < kComputeUnits; ++c) free_at.push(0);
            int64_t last = 0;
            for (const lora_tile& t : tiles) {
                const int64_t at = free_at.top() + weight(t) + (int64_t)((t.nrows + 15) / 16) * 2 * 64 * lora_shape_jb(t.shape);
                free_at.pop();
                free_at.push(at);
                last = std::max(last, at);
            }
            return last;
        };
        if (finish(cut) * 100 < finish(p->expand_tiles) * 97) p->expand_tiles.swap(cut);
    }
    // Single-launch decode kernel: the 16 tokens of every tile, in tile order and padded with the tile's
    // first token, so that a workgroup can fetch them by its index alone, at the same time as its
    // tile descriptor instead of after it
    p->shrink_rows.clear();
    p->expand_rows.clear();
    if (p->fused_ok) {
        auto rows_of = [&](const std::vector<lora_tile>& tiles, std::vector<int32_t>& rows) {
            rows.resize(tiles.size() * 16);
            for (size_t i = 0; i < tiles.size(); ++i)
                for (int m = 0; m < 16; ++m)
                    rows[i * 16 + m] = p->perm[(size_t)tiles[i].row0 + (m < tiles[i].nrows ? m : 0)];
        };
        rows_of(p->shrink_tiles, p->shrink_rows);
        rows_of(p->expand_tiles, p->expand_rows);
    }
}

// Tiles of the expand that takes rows of any length: 16 tokens x 256 features; twice the tokens where that leaves more
// than two workgroups per compute unit (microseconds of lora_delta, ranks 256, 32 / 16 tokens a tile: 64 tokens 18.7 /
// 16.4, 300 tokens 29.3 / 29.6, 1000 tokens 54.8 / 76.5), more features where it leaves more than the chip holds at a
// time; the heaviest first.
// per: tokens of a tile, 0: by that rule, and no tiles at all for problems so small that a tile's chain of loads is what
// they cost: below 12 million products, y's way through a value counted as eight of them, the general kernel, which has a
// thread per value, takes less (kernel times, this / general, by products alone: 0.3 - 1 million 5.9 / 4.8 us, 2 - 4 7.0 /
// 6.0, 4 - 8 7.5 / 6.7, 8 - 16 7.8 / 8.5, 16 - 32 7.8 / 11.8; 505 tokens of rank 1, N = 13768, 7 million, 16.4 / 22.5; fp32 up
// to rank 16, whose sums are as exact either way: 0.3 - 1 million 5.1 / 4.3, 2 - 4 6.6 / 5.5, 8 - 16 9.7 / 10.0).
static void build_rows_expand_tiles(lora_plan* p, int32_t per)
{
    if (p->N < 8 || (int64_t)p->N * LORA_MAX_RANK >= (1ll << 31)) return;   // the kernel fetches whole chunks, by 32-bit offsets
    const int G = (int)p->group_adapter.size();
    int32_t max_rank = 0, min_rank = LORA_MAX_RANK;
    bool odd_above_24 = false;
    for (int g = 0; g < G; ++g) {
        const int32_t r = p->rank[p->group_adapter[g]];
        max_rank = std::max(max_rank, r);
        min_rank = std::min(min_rank, r);
        odd_above_24 = odd_above_24 || (r > 24 && r % 2);
    }
    if (per == 0 && p->variant_req == LORA_VARIANT_AUTO) {
        int64_t products = 0;
        for (int g = 0; g < G; ++g) {
            const int32_t r = p->rank[p->group_adapter[g]];
            products += (int64_t)(p->group_offset[g + 1] - p->group_offset[g]) * (r + 8) * p->N;
        }
        if (products < 12000000 && (p->dtype == LORA_BF16 || max_rank <= 16)) return;
    }
    const int32_t kstep = p->dtype == LORA_F32 ? 16 : 32, terms = p->dtype == LORA_F32 ? 1 : 3;
    auto token_tiles = [&](int32_t per) {
        int64_t n = 0;
        for (int g = 0; g < G; ++g) n += (p->group_offset[g + 1] - p->group_offset[g] + per - 1) / per;
        return n;
    };
    const int64_t blocks = (p->N + 255) / 256;
    // bf16 of one MFMA step: little of Bt to read again and little v to hold, so 16 tokens, and two or four blocks of features for
    // v and the rows' numbers once they are enough tiles all the same.  lora_delta, K = 512, 32 tokens / so: 2188 tokens of
    // rank 20 -> 11008, 41.5 / 37.3 us; 5715 of rank 12 on 64 adapters -> 5120, 52.8 / 44.2; 1114 of rank 4 -> 4096, 16.4 / 13.9;
    // 5400 batches of ranks up to 32, 100 to 6600 tokens, 1.12 times as fast.  Odd ranks above 24, whose rows' elements all have to
    // be shifted into place, only above 1024 tiles so and below 3072 tiles of 32 tokens where requests of more than 16 tokens fill
    // these (tiles of 16 are half as many again): 702 tokens of rank 31, 5120 -> 5120, 15.3 / 16.2; 1018 of ranks 31 and 9, 4096 ->
    // 4096, 15.1 / 15.9; 5379 of rank 25 -> 11008, 89.4 / 100.9; 97 of 605 such batches over 1.02 times as long, of the 1199
    // others 7.  Higher ranks lose by 16 tokens: 4708 of rank 100 -> 4096, 68.0 / 71.4.
    const bool one_step = per == 0 && p->dtype == LORA_BF16 && max_rank <= 32 &&
                          (!odd_above_24 || 2 * token_tiles(16) <= 3 * token_tiles(32) ||
                           (token_tiles(16) * blocks > 1024 && token_tiles(32) * blocks < 3072));
    const bool higher = per == 0 && p->dtype == LORA_BF16 && max_rank > 32;
    if (per == 0) per = one_step || token_tiles(16) * blocks <= 512 ? 16 : 32;
    const int64_t tiles = token_tiles(per) * blocks;
    int64_t wide = one_step ? (tiles < 1024 ? 1 : tiles < 2560 ? 2 : 4) : tiles / 1024;
    // Higher ranks, all about as long: the chip holds 768 tiles, so two blocks a tile where that makes at most one round of them (odd
    // ranks, whose elements all have to be shifted into place: two thirds of one), else four where that makes two thirds of one.
    // lora_delta, one block / so: 1329 tokens of rank 256, 5120 -> 5120 (840 tiles of one block), 54.2 / 47.2 us; 741 on 28 of rank 34,
    // 1920 -> 7720 (1209), 25.2 / 19.9; 1021 on 4 of rank 160, 4096 -> 11008 (1419), 48.5 / 41.4; 1272 on 9 of ranks 90 and 100, 4096 ->
    // 11008 (1892), 50.1 / 42.2; 100 drawn batches of 1024 to 1536 tiles 1.06 times as fast, the slowest 0.976; with ranks 255 and 200
    // 0.955, 2234 tokens, 4096 -> 4096, 82.1 / 93.6.  (With ranks of 4 to 256 in one batch the rounds are not full: 0.94 on average.)
    // With fewer than eight tokens a tile Bt alone is what it reads, and more and shorter workgroups read it the faster.
    if (higher && per == 32 && 4 * min_rank >= 3 * max_rank && (int64_t)p->perm.size() >= 8 * token_tiles(32)) {
        auto held = [&](int64_t n) { return token_tiles(32) * ((blocks + n - 1) / n); };
        if (blocks >= 2 && tiles >= 768 && held(2) <= (odd_above_24 ? 512 : 768)) wide = 2;
        else if (blocks >= 4 && tiles >= 1536 && held(4) <= 512) wide = 4;
    }
    const int32_t n_tile = 256 * (int32_t)std::max<int64_t>(1, std::min(blocks, wide));
    // Ranks of very different length in one batch: the launch then is its longest tiles, which all start first (microseconds of a
    // tile of 32 tokens, by time stamps in a launch of 640: ranks up to 48 7.1, 100 8.2 to 10.4, 256 11 to 15).  Those of ranks
    // above 128 are of 16 tokens where all tiles have a place on the chip at once then (768, and a twelfth more, which begin as the
    // first short ones end) and are a quarter more at most: each reads Bt again.  lora_delta, 32 / 16 tokens: 726 on 4 adapters of ranks 140 and 8, 11008 -> 4096, 20.5 / 18.1 us; 914 single tokens
    // on 7 of ranks 4 to 256, 26.1 / 23.9; 742 on 40, 1416 -> 4016, 22.9 / 20.9; not taken: 154 on 6 of ranks 129 and 64, 5120 -> 13824,
    // 23.3 / 27.2 (378 and 486 tiles); 999 on 2 of 256 and 100, 11008 -> 4096, 35.4 / 40.5 (512 and 800).  120 drawn batches that
    // are cut so 1.07 times as fast, three below 0.98 (219 on 7 of 129 and 64, 2136 -> 12144, 28.8 / 30.8);
    // of 769 to 832 tiles 29 drawn ones 1.03 times as fast, four below 0.98; of 833 to 960 46 1.003, 13 below 0.98.
    int32_t long_rank = LORA_MAX_RANK + 1;                   // ranks from here on: tiles of 16 tokens
    if (higher && per == 32 && max_rank > 128 && 2 * min_rank < max_rank) {
        int64_t shorter = 0;
        for (int g = 0; g < G; ++g) {
            const int32_t own = p->rank[p->group_adapter[g]] > 128 ? 16 : per;
            shorter += (p->group_offset[g + 1] - p->group_offset[g] + own - 1) / own;
        }
        if (shorter * ((p->N + n_tile - 1) / n_tile) <= 832 && 4 * shorter <= 5 * token_tiles(32)) long_rank = 129;
    }
    for (int g = 0; g < G; ++g)
        for (int32_t row = p->group_offset[g], own = p->rank[p->group_adapter[g]] >= long_rank ? 16 : per; row < p->group_offset[g + 1]; row += own)
            for (int32_t n0 = 0; n0 < p->N; n0 += n_tile) {
                lora_tile t{};
                t.adapter = p->group_adapter[g];
                t.row0 = row;
                t.nrows = std::min(own, p->group_offset[g + 1] - row);
                t.c0 = n0;
                t.cn = std::min(n_tile, p->N - n0);
                t.reserved0 = p->rank[t.adapter];
                const int32_t tb = t.nrows > 16 ? 2 : 1;
                p->rows_expand_tb = std::max(p->rows_expand_tb, tb);
                p->rows_expand_lds = std::max(p->rows_expand_lds, (t.reserved0 + kstep - 1) / kstep * tb * terms * 1024);
                p->rows_expand_tiles.push_back(t);
            }
    auto weight = [](const lora_tile& t) { return (int64_t)t.cn * (t.reserved0 + 2 * t.nrows); };   // of Bt read, of y read and written
    std::stable_sort(p->rows_expand_tiles.begin(), p->rows_expand_tiles.end(),
                     [&](const lora_tile& x, const lora_tile& y) { return weight(x) > weight(y); });
}

// Tiles of the shrink that splits K over its wavefronts, of the plan's shape and K parts
static void list_rows_shrink_tiles(lora_plan* p)
{
    const int32_t fb = p->rows_shrink_fb, tb = p->rows_shrink_tb, G = (int)p->group_adapter.size();
    for (int g = 0; g < G; ++g) {
        const int32_t a = p->group_adapter[g], r = p->rank[a];
        for (int32_t row = p->group_offset[g]; row < p->group_offset[g + 1]; row += 16 * tb)
            for (int32_t j = 0; j < r; j += 16 * fb)
                for (int32_t q = 0; q < p->v_parts; ++q) {
                    lora_tile t{};
                    t.adapter = a;
                    t.row0 = row;
                    t.nrows = std::min(16 * tb, p->group_offset[g + 1] - row);
                    t.c0 = j;
                    t.cn = std::min(16 * fb, r - j);
                    t.shape = (q << 8) | (p->v_parts << 12);
                    t.reserved0 = r;
                    std::memcpy(&t.reserved1, &p->scale[a], sizeof(float));
                    p->rows_shrink_tiles.push_back(t);
                }
    }
}

// Their shape.  A compute unit loads 16 (fb + tb) rows per workgroup at about
// 100 GB/s and multiplies at 256 (bf16: 4096) flops/clk; the launch takes as long as the unit with the most workgroups;
// a K part costs the consumers of v another read of it.  parts: K parts, 0: by the same rule
static void build_rows_shrink_tiles(lora_plan* p, int32_t parts)
{
    const bool f32 = p->dtype == LORA_F32;
    const rows_shape* shapes = f32 ? kRowsF32 : kRowsBf16;
    const int n_shapes = f32 ? 2 : 6;
    const int32_t kunit = f32 ? 32 : 64, units = (p->K + kunit - 1) / kunit;
    double best = 0;
    for (int i = 0; i < n_shapes; ++i) {
        const int32_t fb = shapes[i].fb, tb = shapes[i].tb;
        const int64_t tiles = rows_shrink_tiles_of(p, fb, tb);
        for (int32_t P = parts ? parts : 1; P <= (parts ? parts : 4); P *= 2) {
            // (lora_delta_static keeps v in an array of its own: parts must not be what outgrows it)
            if (!parts && P > 1 && (units / P < 8 || (size_t)P * p->T * p->R * sizeof(float) > LORA_STATIC_V_BYTES)) break;
            const double load = (fb + tb) * 16.0 * (f32 ? 4 : 2) / 100e9, math = fb * tb * 512.0 / (f32 ? 0.54e12 : 8.6e12);
            const double cost = (double)((tiles * P + 255) / 256) * ((double)units * kunit / P * std::max(load, math) + 0.5e-6) + (P - 1) * 0.3e-6;
            if (best == 0 || cost < best) {
                best = cost;
                p->rows_shrink_fb = fb;
                p->rows_shrink_tb = tb;
                p->rows_shrink_d = shapes[i].d;
                p->v_parts = P;
            }
        }
    }
    list_rows_shrink_tiles(p);
}

// Tiles of the fp32 matrix-core kernels.
static void build_f32_tiles(lora_plan* p)
{
    const int G = (int)p->group_adapter.size();
    if (G == 0) return;
    auto rows_of = [&](int g) { return p->group_offset[g + 1] - p->group_offset[g]; };
    auto rank_of = [&](int g) { return p->rank[p->group_adapter[g]]; };
    auto tile_of = [&](int g, int32_t row, int32_t per) {
        lora_tile t{};
        t.adapter = p->group_adapter[g];
        t.row0 = row;
        t.nrows = std::min(per, p->group_offset[g + 1] - row);
        t.reserved0 = rank_of(g);
        std::memcpy(&t.reserved1, &p->scale[t.adapter], sizeof(float));
        return t;
    };
    // ---- shrink and expand in one launch, where every 128 features read the tile's x and At again.  Microseconds per
    // call, one launch / two, 64 tokens on 8 adapters: rank 8, K = N = 1024 7.7 / 10.8, 2048 8.4 / 10.8; ranks to 64, 512
    // 8.5 / 11.1, 768 10.8 / 10.8, 1024 12.9 / 11.0.  (The two steps alone then run on tiles of the same arithmetic.)
    int64_t token_tiles16 = 0;
    int32_t max_rank = 0;
    for (int g = 0; g < G; ++g) {
        token_tiles16 += (rows_of(g) + 15) / 16;
        max_rank = std::max(max_rank, rank_of(g));
    }
    if (max_rank <= 64 && p->N >= 8 && (int64_t)(16 + max_rank) * p->K * 4 <= 192 * 1024 && token_tiles16 * ((p->N + 127) / 128) <= 512) {
        for (int g = 0; g < G; ++g)
            for (int32_t row = p->group_offset[g]; row < p->group_offset[g + 1]; row += 16) {
                lora_tile t = tile_of(g, row, 16);
                p->rows_shrink_tiles.push_back(t);
                for (int32_t n0 = 0; n0 < p->N; n0 += 128) {
                    t.c0 = n0;
                    t.cn = std::min(128, p->N - n0);
                    p->f32_delta_tiles.push_back(t);
                }
            }
        build_rows_expand_tiles(p, 16);
        return;
    }
    if (p->K % 4 == 0) build_rows_shrink_tiles(p, 0);        // (16-byte chunks of rows)
    build_rows_expand_tiles(p, 0);
}

// Rows of the fused GEMM that carry a delta, dealt to segments of 64: a wavefront of the ring and of the medium GEMM adds the
// deltas of 64 rows, adapter by adapter and 32 ranks at a time, and its tile ends with the last of them.  Sorted by adapter,
// long requests leave wavefronts one adapter each, and the short ones share the rest: up to a dozen.  Here the adapters with
// fewer than 64 rows go whole to the segment with the fewest steps that has room, and those with more fill what is left, the
// cheapest where most steps are already.  An adapter is one run of rows in a segment.
// `cheap`: rows without an adapter of their own (mixture mode's, for the removal).  Returns an empty list where that
// does not take a third off the sum over tiles of 256 rows of the longest wavefront: dealt rows put more adapters in a tile
// (6055 tokens on 240 adapters, 4096 -> 11008, sum 172 and 128: 523 -> 536 us; 6935 on 105, 96 and 77: 82 -> 84), or where
// there are eight adapters and more to a segment: uniform ones are evened out by chance, and 4000 took half a millisecond to deal
// (very uneven popularity would still gain: 825 single tokens on 201 adapters, sum 125 and 74).
// Sum over tiles of the longest wavefront's steps, sorted and dealt: 1111 tokens of mixed requests 21 and 9 (longest 18 and 3),
// 16384 tokens on 256 adapters 396 and 225.  lora_fused_forward, W from memory: 96.5 -> 89.6 us in mixture mode (4096 -> 4096),
// 1300 tokens on 64 adapters (4096 -> 4096) 67.0 -> 62.7, 2637 on 191 (11008 -> 4096) 366 -> 300.  The cost is that of the ring and
// of the medium GEMM; in the small one, whose wavefronts share the adapters of 16 to 64 rows, 5800 drawn batches that are
// dealt take 0.94 times as long, 47 of them over 1.02 (up to 1.09).
static std::vector<int32_t> deal_rows(const lora_plan* p, const std::vector<int32_t>& cheap)
{
    struct run { int32_t segment, group, first, count; };    // group -1: `cheap`
    const int32_t G = (int32_t)p->group_adapter.size(), rows = (int32_t)(p->perm.size() + cheap.size()), n = (rows + 63) / 64;
    if (n < 2 || G < 2 || G >= 8 * n) return {};
    auto steps_of = [&](int32_t g) { return g < 0 ? 0 : (p->rank[p->group_adapter[g]] + 31) / 32; };
    auto size_of = [&](int32_t g) { return g < 0 ? (int32_t)cheap.size() : p->group_offset[g + 1] - p->group_offset[g]; };
    auto cost = [&](auto steps_at) {                         // (sum over tiles, longest)
        std::pair<int64_t, int32_t> c{0, 0};
        for (int32_t i = 0; i < n; i += 4) {
            int32_t longest = 0;
            for (int32_t q = i; q < std::min(i + 4, n); ++q) longest = std::max(longest, steps_at(q));
            c.first += longest;
            c.second = std::max(c.second, longest);
        }
        return c;
    };
    // Dealing costs a plan up to 80 us, and few batches end with it: those are sent back first that cannot, because the steps
    // of whole requests, spread evenly, are too many already.  lora_plan_create of 8192 tokens on 128 adapters 192 -> 163 us.
    std::vector<int32_t> sorted_steps((size_t)n, 0);
    int64_t fewest = 0;
    for (int32_t g = 0; g < G; ++g) {
        for (int32_t i = p->group_offset[g] / 64; i <= (p->group_offset[g + 1] - 1) / 64; ++i) sorted_steps[(size_t)i] += steps_of(g);
        fewest += (int64_t)steps_of(g) * ((size_of(g) + 63) / 64);
    }
    const auto sorted = cost([&](int32_t i) { return sorted_steps[(size_t)i]; });
    if (3 * ((fewest + 3) / 4) > 2 * sorted.first) return {};
    struct group { int32_t steps, size, id; };
    std::vector<group> small, large;
    for (int32_t g = 0; g < G; ++g) (size_of(g) < 64 ? small : large).push_back(group{steps_of(g), size_of(g), g});
    if (small.empty()) return {};
    if (!cheap.empty()) large.push_back(group{0, (int32_t)cheap.size(), -1});

    std::vector<run> runs;
    runs.reserve((size_t)G + n + 1);
    std::vector<int32_t> steps((size_t)n, 0), room((size_t)n, 64);
    room[(size_t)n - 1] = rows - 64 * (n - 1);
    auto put = [&](int32_t i, const group& g, int32_t first, int32_t count) {
        runs.push_back(run{i, g.id, first, count});
        room[(size_t)i] -= count;
        steps[(size_t)i] += g.steps;
    };
    std::sort(small.begin(), small.end(), [](const group& a, const group& b) {
        return a.steps != b.steps ? a.steps > b.steps : a.size != b.size ? a.size > b.size : a.id < b.id;
    });
    typedef std::pair<int32_t, int32_t> entry;               // steps so far, segment: a heap, fewest steps first
    std::vector<entry> least((size_t)n), passed;
    for (int32_t i = 0; i < n; ++i) least[(size_t)i] = {0, i};
    const std::greater<entry> later;
    for (const group& g : small) {
        bool done = false;
        passed.clear();
        while (!done && !least.empty() && passed.size() < 4) {
            std::pop_heap(least.begin(), least.end(), later);
            const int32_t i = least.back().second;
            least.pop_back();
            if ((done = room[(size_t)i] >= g.size)) put(i, g, 0, g.size);
            if (room[(size_t)i]) passed.push_back({steps[(size_t)i], i});
        }
        if (!done) large.push_back(g);                       // in pieces, then
        for (const entry& e : passed) {
            least.push_back(e);
            std::push_heap(least.begin(), least.end(), later);
        }
    }
    std::stable_sort(large.begin(), large.end(), [](const group& a, const group& b) { return a.steps < b.steps; });
    std::vector<int32_t> order((size_t)n);
    for (int32_t i = 0; i < n; ++i) order[(size_t)i] = i;
    const std::vector<int32_t> whole = steps;
    std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return whole[(size_t)a] != whole[(size_t)b] ? whole[(size_t)a] > whole[(size_t)b] : a < b; });
    size_t at = 0;
    for (const group& g : large)
        for (int32_t first = 0; first < g.size;) {
            while (room[(size_t)order[at]] == 0) ++at;
            const int32_t count = std::min(room[(size_t)order[at]], g.size - first);
            put(order[at], g, first, count);
            first += count;
        }
    // segments of like length to the same tile; the last one, if short, stays last
    for (int32_t i = 0; i < n; ++i) order[(size_t)i] = i;
    std::sort(order.begin(), order.end() - (rows % 64 ? 1 : 0), [&](int32_t a, int32_t b) {
        return steps[(size_t)a] != steps[(size_t)b] ? steps[(size_t)a] > steps[(size_t)b] : a < b;
    });

    const auto dealt = cost([&](int32_t i) { return steps[(size_t)order[(size_t)i]]; });
    if (3 * dealt.first > 2 * sorted.first || dealt.second > sorted.second) return {};

    std::vector<int32_t> out((size_t)rows), to((size_t)n);
    for (int32_t q = 0; q < n; ++q) to[(size_t)order[(size_t)q]] = 64 * q;
    for (const run& r : runs) {
        const int32_t* from = (r.group < 0 ? cheap.data() : p->perm.data() + p->group_offset[r.group]) + r.first;
        std::copy_n(from, r.count, out.begin() + to[(size_t)r.segment]);
        to[(size_t)r.segment] += r.count;
    }
    return out;
}

// Time, in stages, of a product by the stage lists: tiles of 256 rows of `stages` stages each, in that order, times `columns` tiles
// of features, on 256 compute units; a tile's base stages, start and stores are about four.
static int64_t time_by_stage_lists(const std::vector<int32_t>& stages, int32_t columns)
{
    typedef std::pair<int64_t, int32_t> units;               // free from then on, how many
    std::vector<units> heap{{0, 256}};
    const std::greater<units> later;
    int64_t end = 0;
    for (int32_t s : stages)
        for (int32_t left = columns; left > 0;) {
            std::pop_heap(heap.begin(), heap.end(), later);
            units& u = heap.back();
            const int32_t take = std::min(u.second, left);
            const units busy{u.first + 4 + s, take};
            left -= take;
            if ((u.second -= take) == 0) heap.pop_back();
            else std::push_heap(heap.begin(), heap.end(), later);
            heap.push_back(busy);
            std::push_heap(heap.begin(), heap.end(), later);
            end = std::max(end, busy.first);
        }
    return end;
}

// Tables of the fused GEMM: it walks the tokens in adapter-sorted order (or dealt, see above), so a tile of rows holds few
// adapters, and folds each adapter's delta in (v_hi, v_lo against Bt_a; the register-staged kernels as extra
// k-stages from the lists below, the ring kernel per wavefront from the row keys).  The full
// blocks of 256 sorted rows are then put heaviest first (most adapter stages): workgroups start in
// index order, so the long tiles run early and the short ones fill the tail of the launch.
// Mixture mode: the removal of the merged adapter concerns every token of `unmerge`'s single adapter group; a tile
// that holds such a token gets the merged adapter's stages once more, marked, after its own.  Tokens without adapter
// that need the removal sort before the merged adapter's tokens, so that tiles of the latter keep no stage at all.
// stage_lists: also the lists of adapter stages (16-byte rows of Bt_a, i.e. ranks that are multiples of 8); the row
// order alone serves the kernels that find the adapters of their rows themselves.
static void build_gemm_tables(lora_plan* p, bool stage_lists)
{
    const lora_plan* u = p->unmerge;
    std::vector<int32_t> key((size_t)p->T);                   // by token
    for (int32_t t = 0; t < p->T; ++t) {
        const int32_t a = p->token_adapter[t];
        key[t] = (a < 0 ? LORA_UNMERGE_BIT - 1 : a) | (u && u->token_adapter[t] >= 0 ? LORA_UNMERGE_BIT : 0);
    }
    std::vector<int32_t> removal_only, plain;
    for (int32_t t = 0; t < p->T; ++t)
        if (p->token_adapter[t] < 0) ((key[t] & LORA_UNMERGE_BIT) ? removal_only : plain).push_back(t);
    std::vector<int32_t> sorted = p->perm, dealt = deal_rows(p, removal_only);
    sorted.insert(sorted.end(), removal_only.begin(), removal_only.end());
    sorted.insert(sorted.end(), plain.begin(), plain.end());
    if (!dealt.empty()) dealt.insert(dealt.end(), plain.begin(), plain.end());

    // adapter stages of a block of 256 rows, one per 64 columns of [v_hi | v_lo] (2 r columns) and adapter, the removal's last;
    // in lists, if there are any, those of the block and those of each half
    struct lists { std::vector<int32_t> ptr128{0}, of128, ptr256{0}, of256; };
    std::vector<int32_t> seen128((size_t)p->n_a, 0), seen256((size_t)p->n_a, 0);
    int32_t halves = 0, wholes = 0;
    auto stages_of = [&](const std::vector<int32_t>& rows, int32_t block, lists* to) {
        int32_t n = 0, last = LORA_UNMERGE_BIT - 1;
        bool removal = false;
        ++wholes;
        for (int32_t lo = 256 * block; lo < std::min(256 * block + 256, p->T); lo += 128) {
            bool half_removal = false;
            ++halves;
            last = LORA_UNMERGE_BIT - 1;
            for (int32_t q = lo; q < std::min(lo + 128, p->T); ++q) {
                const int32_t k = key[(size_t)rows[(size_t)q]];
                if (k == last) continue;                     // (of a run of rows only the first)
                last = k;
                half_removal = half_removal || (k & LORA_UNMERGE_BIT);
                const int32_t a = k & (LORA_UNMERGE_BIT - 1);
                if (a == LORA_UNMERGE_BIT - 1 || seen128[(size_t)a] == halves) continue;
                seen128[(size_t)a] = halves;
                const bool first = seen256[(size_t)a] != wholes;
                seen256[(size_t)a] = wholes;
                for (int32_t jb = 0; jb * 64 < 2 * p->rank[a]; ++jb) {
                    n += first;
                    if (to) to->of128.push_back(a | (jb << 24));
                    if (to && first) to->of256.push_back(a | (jb << 24));
                }
            }
            for (int32_t jb = 0; half_removal && to && jb * 64 < 2 * p->rank[p->merged]; ++jb) to->of128.push_back(p->merged | LORA_UNMERGE_BIT | (jb << 24));
            if (to) to->ptr128.push_back((int32_t)to->of128.size());
            removal = removal || half_removal;
        }
        for (int32_t jb = 0; removal && jb * 64 < 2 * p->rank[p->merged]; ++jb, ++n)
            if (to) to->of256.push_back(p->merged | LORA_UNMERGE_BIT | (jb << 24));
        if (to) to->ptr256.push_back((int32_t)to->of256.size());
        return n;
    };

    const int32_t full = p->T / 256, all = (p->T + 255) / 256;
    if (!dealt.empty()) {
        // The kernel that walks the stage lists has every wavefront go through all stages of its 256 rows: dealt rows even
        // these out, too, but are more in all.  Both ways are laid out on the compute units; K <= 128, 1449 drawn batches that
        // could be dealt: 0.81 times as long if all are, but one in ten longer (10764 tokens on 203 adapters, 8 -> 1272, 66 ->
        // 82 us; 2559 on 77, 40 -> 7256, 115 -> 142); so 0.82, three of them above 1.03.
        bool take = true;
        if (stage_lists && lora_product_by_stage_lists && lora_product_by_stage_lists(p)) {
            const int32_t columns = (p->N + 255) / 256;
            int64_t time[2], work[2];
            for (int i = 0; i < 2; ++i) {
                std::vector<int32_t> stages((size_t)all);
                int64_t sum = 0;
                for (int32_t b = 0; b < all; ++b) sum += stages[(size_t)b] = stages_of(i ? dealt : sorted, b, nullptr);
                std::sort(stages.begin(), stages.begin() + full, std::greater<int32_t>());
                time[i] = time_by_stage_lists(stages, columns);
                work[i] = 4 + *std::max_element(stages.begin(), stages.end()) / 2 + sum * columns / 256;
            }
            take = time[1] < time[0] && 20 * work[1] < 19 * work[0];
        }
        if (take) sorted.swap(dealt);
    }

    lists found;
    std::vector<int32_t> weight((size_t)all), blocks((size_t)all);
    for (int32_t b = 0; b < all; ++b) {
        weight[(size_t)b] = stages_of(sorted, b, stage_lists ? &found : nullptr);
        blocks[(size_t)b] = b;
    }
    std::stable_sort(blocks.begin(), blocks.begin() + full, [&](int32_t x, int32_t y) { return weight[(size_t)x] > weight[(size_t)y]; });
    p->order.reserve((size_t)p->T);
    for (int32_t b : blocks) p->order.insert(p->order.end(), sorted.begin() + (size_t)b * 256, sorted.begin() + std::min(b * 256 + 256, p->T));
    p->row_key.resize((size_t)p->T);
    for (int32_t q = 0; q < p->T; ++q) p->row_key[q] = key[p->order[q]];

    for (int32_t a : p->group_adapter) p->rank_steps += (p->rank[a] + 31) / 32;

    if (!stage_lists) return;
    auto append = [](std::vector<int32_t>& ptr, std::vector<int32_t>& lst, const std::vector<int32_t>& from_ptr, const std::vector<int32_t>& from, int32_t tile) {
        lst.insert(lst.end(), from.begin() + from_ptr[(size_t)tile], from.begin() + from_ptr[(size_t)tile + 1]);
        ptr.push_back((int32_t)lst.size());
    };
    p->extra_ptr128.assign(1, 0);
    p->extra_ptr256.assign(1, 0);
    p->extra128.reserve(found.of128.size());
    p->extra256.reserve(found.of256.size());
    for (int32_t b : blocks) {
        append(p->extra_ptr256, p->extra256, found.ptr256, found.of256, b);
        for (int32_t half = 2 * b; half < 2 * b + 2 && half * 128 < p->T; ++half) append(p->extra_ptr128, p->extra128, found.ptr128, found.of128, half);
    }
}

// Shrink tiles of 16 tokens x up to 32 rank rows for the launch that has the product of a small batch in it, where there is
// that launch and the plan's own are not of that size (requests of several tokens, ranks above 64).  Measured up to 512 tokens:
// beyond, such batches take two launches.
static void build_layer_tiles(lora_plan* p)
{
    if (p->family != LORA_VARIANT_TILED || p->shrink_small || p->T > 512 || !lora_layer_takes) return;
    int64_t tiles = 0;
    for (size_t g = 0; g < p->group_adapter.size(); ++g)
        tiles += (int64_t)((p->group_offset[g + 1] - p->group_offset[g] + 15) / 16) * ((p->rank[p->group_adapter[g]] + 31) / 32);
    if (!lora_layer_takes(p, tiles)) return;
    p->layer_shrink_tiles.reserve((size_t)tiles);
    for (size_t g = 0; g < p->group_adapter.size(); ++g) {
        const int32_t a = p->group_adapter[g], r = p->rank[a];
        for (int32_t row = p->group_offset[g]; row < p->group_offset[g + 1]; row += 16)
            for (int32_t j = 0; j < r; j += 32) {
                lora_tile t{};
                t.adapter = a;
                t.row0 = row;
                t.nrows = std::min(16, p->group_offset[g + 1] - row);
                t.c0 = j;
                t.cn = std::min(32, r - j);
                t.shape = lora_shape_code(1, t.cn > 16 ? 2 : 1);
                t.reserved0 = r;
                std::memcpy(&t.reserved1, &p->scale[a], sizeof(float));
                p->layer_shrink_tiles.push_back(t);
            }
    }
    std::stable_sort(p->layer_shrink_tiles.begin(), p->layer_shrink_tiles.end(),
                     [](const lora_tile& x, const lora_tile& y) { return x.cn > y.cn; });
}

// One plan over the descriptor's segments as they stand; `unmerge` (may be null) is the removal's plan of a batch
// in mixture mode, which the new plan takes over; is_removal: this is such a plan.
static lora_status create_plain(const lora_batch_desc* d, int32_t merged, lora_plan* unmerge, lora_plan** out, bool is_removal = false)
{
    lora_plan* p = new (std::nothrow) lora_plan();
    if (!p) {
        lora_plan_destroy(unmerge);
        return LORA_ERR_NOMEM;
    }
    p->merged = unmerge ? merged : -1;
    p->unmerge = unmerge;
    p->is_removal = is_removal;
    try {
        p->T = d->num_tokens; p->S = d->num_segments; p->n_a = d->num_adapters;
        p->K = d->k; p->N = d->n; p->dtype = d->dtype; p->variant_req = d->variant;
        p->rank.assign(d->adapter_rank, d->adapter_rank + p->n_a);
        p->scale.assign(d->adapter_scale, d->adapter_scale + p->n_a);

        // adapter of every token; adapters of rank 0 count as "none"
        p->token_adapter.assign((size_t)p->T, -1);
        std::vector<int32_t> count((size_t)p->n_a + 1, 0);
        for (int32_t s = 0; s < p->S; ++s) {
            int32_t a = d->seg_adapter[s];
            if (a >= 0 && p->rank[a] == 0) a = -1;
            for (int32_t t = d->seg_indptr[s]; t < d->seg_indptr[s + 1]; ++t) p->token_adapter[t] = a;
            if (a >= 0) count[a] += d->seg_indptr[s + 1] - d->seg_indptr[s];
        }
        // counting sort by adapter id = stable grouping
        std::vector<int32_t> start((size_t)p->n_a + 1, 0);
        int32_t max_rank = 0;
        bool ranks_mult8 = true;
        p->group_offset.push_back(0);
        for (int32_t a = 0; a < p->n_a; ++a) {
            start[a + 1] = start[a] + count[a];
            if (count[a] > 0) {
                p->group_adapter.push_back(a);
                p->group_offset.push_back(start[a + 1]);
                max_rank = std::max(max_rank, p->rank[a]);
                if (p->rank[a] % 8) ranks_mult8 = false;
            }
        }
        p->perm.resize((size_t)start[p->n_a]);
        std::vector<int32_t> cursor(start.begin(), start.end() - 1);
        for (int32_t t = 0; t < p->T; ++t) {
            const int32_t a = p->token_adapter[t];
            if (a >= 0) p->perm[cursor[a]++] = t;
        }
        int32_t table_max = 0;
        for (int32_t a = 0; a < p->n_a; ++a) table_max = std::max(table_max, p->rank[a]);
        p->R = std::max(8, round_up(table_max, 8));

        int32_t max_group = 0;
        for (size_t g = 0; g + 1 < p->group_offset.size(); ++g)
            max_group = std::max(max_group, p->group_offset[g + 1] - p->group_offset[g]);
        snapshot_tuning(p, d, (int32_t)p->perm.size(), max_rank, max_group);

        // the tiled kernels take bf16, 16-byte rows (K and ranks multiples of 8), ranks <= 128
        p->tiled_layout_ok = (p->dtype == LORA_BF16) && (p->K % 8 == 0) && ranks_mult8 && max_rank <= 128;
        const int32_t n_active = (int32_t)p->perm.size();
        if (p->variant_req == LORA_VARIANT_GENERAL || !p->tiled_layout_ok)
            p->family = LORA_VARIANT_GENERAL;
        else if (p->variant_req == LORA_VARIANT_TILED)
            p->family = LORA_VARIANT_TILED;
        else
            p->family = (n_active >= p->tuning.tiled_min_tokens) ? LORA_VARIANT_TILED : LORA_VARIANT_GENERAL;
        if (p->family == LORA_VARIANT_TILED) build_tiles(p);
        if (p->shrink_by_rows) list_rows_shrink_tiles(p);
        if (p->dtype == LORA_F32 && p->variant_req != LORA_VARIANT_GENERAL) build_f32_tiles(p);
        // Ranks that only the expand kernels cannot take (not multiples of 8: rows of Bt_a would not be 16-byte
        // aligned; above 128): the shrink still runs on the MFMA kernels, which tile the rank axis in blocks of 16
        // rows of At_a and mask what they store.  That is also the path of task heads, whose widths are arbitrary.
        p->shrink_tiled_only = false;
        if (p->family == LORA_VARIANT_GENERAL && !p->tiled_layout_ok && p->variant_req != LORA_VARIANT_GENERAL &&
            p->dtype == LORA_BF16 && p->K % 8 == 0 && max_rank <= LORA_MAX_RANK &&
            (p->variant_req == LORA_VARIANT_TILED || n_active >= p->tuning.tiled_min_tokens)) {
            build_tiles(p, true);
            p->shrink_tiled_only = !p->shrink_tiles.empty();
            if (p->shrink_tiled_only) build_rows_shrink_tiles(p, p->v_parts);
        }
        // ... and the expand on the kernel for rows of any length
        if (p->family == LORA_VARIANT_GENERAL && !p->tiled_layout_ok && p->variant_req != LORA_VARIANT_GENERAL &&
            p->dtype == LORA_BF16 && n_active > 0 && (p->variant_req == LORA_VARIANT_TILED || n_active >= p->tuning.tiled_min_tokens))
            build_rows_expand_tiles(p, 0);
        // (in mixture mode the removal's v must have the layout the GEMM's stages read, too)
        if (p->n_a < LORA_UNMERGE_BIT) build_gemm_tables(p, p->tiled_layout_ok && (!unmerge || unmerge->tiled_layout_ok));
        build_layer_tiles(p);
    } catch (const std::bad_alloc&) {
        lora_plan_destroy(p);
        return LORA_ERR_NOMEM;
    }
    *out = p;
    return LORA_OK;
}

extern "C" lora_status lora_plan_create(const lora_batch_desc* d, lora_plan** out)
{
    if (!d || !out) return LORA_ERR_INVALID_ARG;
    *out = nullptr;
    if (!validate(d)) return LORA_ERR_INVALID_ARG;
    const int32_t m = d->merged_adapter_plus1 - 1;
    if (m < 0 || d->adapter_rank[m] == 0) return create_plain(d, -1, nullptr, out);

    // Mixture mode (section 4.4.1) as two batches over the same tokens: the removal of the merged adapter
    // (every segment that is not m's uses m, scale negated) and the tokens' own branches (m's segments use none).
    lora_plan* removal = nullptr;
    try {
        std::vector<int32_t> seg((size_t)d->num_segments);
        std::vector<float> scale(d->adapter_scale, d->adapter_scale + d->num_adapters);
        scale[m] = -scale[m];
        for (int32_t s = 0; s < d->num_segments; ++s) seg[s] = d->seg_adapter[s] == m ? -1 : m;
        lora_batch_desc dr = *d;
        dr.seg_adapter = seg.data();
        dr.adapter_scale = scale.data();
        dr.merged_adapter_plus1 = 0;
        lora_status st = create_plain(&dr, -1, nullptr, &removal, true);
        if (st != LORA_OK) return st;
        for (int32_t s = 0; s < d->num_segments; ++s) seg[s] = d->seg_adapter[s] == m ? -1 : d->seg_adapter[s];
        lora_batch_desc own = *d;
        own.seg_adapter = seg.data();
        own.merged_adapter_plus1 = 0;
        return create_plain(&own, m, removal, out);
    } catch (const std::bad_alloc&) {
        lora_plan_destroy(removal);
        return LORA_ERR_NOMEM;
    }
}

void (*lora_plan_device_release)(lora_plan*) = nullptr;
bool (*lora_layer_takes)(const lora_plan*, int64_t) = nullptr;
bool (*lora_product_by_stage_lists)(const lora_plan*) = nullptr;

extern "C" void lora_plan_destroy(lora_plan* p)
{
    if (!p) return;
    if (p->d_buf && lora_plan_device_release) lora_plan_device_release(p);
    lora_plan_destroy(p->unmerge);
    delete p;
}

extern "C" lora_status lora_plan_query(const lora_plan* p, int32_t* v_row_stride, size_t* v_bytes,
                                       size_t* fused_workspace_bytes)
{
    if (!p) return LORA_ERR_INVALID_ARG;
    size_t vb = lora_own_v_bytes(p);
    size_t split = ((size_t)p->T * 2 * p->R * 2 + 255) / 256 * 256;
    if (p->unmerge) {
        vb = lora_unmerge_v_offset(p) + lora_own_v_bytes(p->unmerge);
        split += ((size_t)p->T * 2 * p->unmerge->R * 2 + 255) / 256 * 256;
    }
    if (v_row_stride) *v_row_stride = p->R;
    if (v_bytes) *v_bytes = vb;
    // workspace of the fused call: v (all parts; in mixture mode the removal's share behind it), then the bf16
    // split [T][2][R] of each
    if (fused_workspace_bytes) *fused_workspace_bytes = (vb + 255) / 256 * 256 + split;
    return LORA_OK;
}

extern "C" lora_status lora_plan_export(const lora_plan* p, lora_plan_view* v)
{
    if (!p || !v) return LORA_ERR_INVALID_ARG;
    v->num_tokens = p->T;
    v->num_active = (int32_t)p->perm.size();
    v->num_groups = (int32_t)p->group_adapter.size();
    v->v_row_stride = p->R;
    v->kernel_family = p->family;
    v->shrink_kernel_family = (p->family == LORA_VARIANT_TILED || p->shrink_tiled_only) ? LORA_VARIANT_TILED : LORA_VARIANT_GENERAL;
    v->shrink_waves = p->shrink_waves;
    v->v_parts = p->v_parts;
    v->tuning_source = p->tuning_source;
    std::memcpy(v->tuning, &p->tuning, sizeof(p->tuning));
    v->token_adapter = p->token_adapter.data();
    v->perm = p->perm.data();
    v->group_adapter = p->group_adapter.data();
    v->group_offset = p->group_offset.data();
    v->shrink_tiles = p->shrink_tiles.data();
    v->num_shrink_tiles = (int32_t)p->shrink_tiles.size();
    v->expand_tiles = p->expand_tiles.data();
    v->num_expand_tiles = (int32_t)p->expand_tiles.size();
    const bool gemm_tables = !p->extra_ptr256.empty() && (int32_t)p->order.size() == p->T;
    v->num_gemm_rows = gemm_tables ? p->T : 0;
    v->num_gemm_tiles = gemm_tables ? (int32_t)p->extra_ptr256.size() - 1 : 0;
    v->gemm_order = gemm_tables ? p->order.data() : nullptr;
    v->gemm_stage_offset = gemm_tables ? p->extra_ptr256.data() : nullptr;
    v->gemm_stage = gemm_tables ? p->extra256.data() : nullptr;
    const lora_plan* u = p->unmerge;
    v->merged_adapter = p->merged;
    v->num_unmerge = u ? (int32_t)u->perm.size() : 0;
    v->unmerge_v_row_stride = u ? u->R : 0;
    v->unmerge_v_parts = u ? u->v_parts : 0;
    v->unmerge_v_offset = u ? lora_unmerge_v_offset(p) : 0;
    v->unmerge_perm = u ? u->perm.data() : nullptr;
    v->unmerge_shrink_tiles = u ? u->shrink_tiles.data() : nullptr;
    v->num_unmerge_shrink_tiles = u ? (int32_t)u->shrink_tiles.size() : 0;
    v->unmerge_expand_tiles = u ? u->expand_tiles.data() : nullptr;
    v->num_unmerge_expand_tiles = u ? (int32_t)u->expand_tiles.size() : 0;
    return LORA_OK;
}

extern "C" const char* lora_status_str(lora_status s)
{
    switch (s) {
        case LORA_OK: return "ok";
        case LORA_ERR_INVALID_ARG: return "invalid argument";
        case LORA_ERR_UNSUPPORTED: return "unsupported";
        case LORA_ERR_NOMEM: return "out of memory";
        case LORA_ERR_WORKSPACE: return "workspace too small or misaligned";
        case LORA_ERR_DEVICE: return "device error";
    }
    return "unknown status";
}
