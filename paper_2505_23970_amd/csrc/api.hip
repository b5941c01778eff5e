// Host side of the C ABI declared in include/greencache.h: argument checks,
// work-split policy, workspace layout and kernel launches. Every check runs
// before the first HIP call, so invalid calls enqueue nothing.
#include <cmath>
#include <cstdint>
#include <mutex>

#include "gc_internal.h"
#include "greencache.h"

namespace {

struct Shape {
    int64_t total_tokens = 0;
    int group = 1;
    bool small = false;          // small-tile (decode) path
    bool wide = false;           // 8-wavefront prefill tiles
    int block_m = gc::kBlockM;   // query rows per tile
    int block_n = gc::kBlockN;   // keys per tile
    int tq = 1;                  // new tokens per query tile
};

struct Plan {
    int chunk = 0;  // key tiles per chunk, 0 = no split
    int64_t items = 0, combines = 0, partials = 0;
    int max_splits = 1;  // key chunks of the query tile with the most
    bool heaviest_decides = false;  // the heaviest work item ends the launch (see heaviest_decides)
    bool three = false;             // a third 128-row workgroup per compute unit pays (8-bit pools, d = 64)
    int group_cost = gc::kCostBuckets;  // work-list order (gc::PlanArgs)
    int buckets = gc::kCostBuckets;
    gc::WorkspaceLayout layout{};
};

gc_status check_common(const gc_geometry* geo, const gc_batch* b, Shape* sh) {
    if (geo == nullptr || b == nullptr) return GC_ERR_NULL_ARG;
    if (b->batch < 0) return GC_ERR_BAD_SHAPE;
    if (geo->num_q_heads <= 0 || geo->num_kv_heads <= 0 || geo->head_dim <= 0 ||
        geo->page_size <= 0 || geo->num_blocks < 0 || geo->max_blocks_per_seq < 0)
        return GC_ERR_BAD_SHAPE;
    if (geo->num_q_heads % geo->num_kv_heads != 0) return GC_ERR_BAD_SHAPE;
    const int group = geo->num_q_heads / geo->num_kv_heads;
    if (group > gc::kBlockM) return GC_ERR_UNSUPPORTED;
    if (geo->num_kv_heads > 65535) return GC_ERR_UNSUPPORTED;  // append grid dimension
    if (geo->head_dim != 64 && geo->head_dim != 128) return GC_ERR_UNSUPPORTED;
    if (geo->page_size != gc::kPage) return GC_ERR_UNSUPPORTED;
    sh->group = group;
    sh->tq = gc::tokens_per_tile(group, sh->block_m);
    sh->total_tokens = 0;
    if (b->batch == 0) return GC_OK;
    if (b->prefix_lens_host == nullptr || b->new_lens_host == nullptr) return GC_ERR_NULL_ARG;
    int64_t total = 0;
    for (int r = 0; r < b->batch; ++r) {
        const int64_t P = b->prefix_lens_host[r], n = b->new_lens_host[r];
        if (P < 0 || n < 0) return GC_ERR_BAD_SHAPE;
        if (P + n > (int64_t)INT32_MAX - gc::kBlockN) return GC_ERR_BAD_SHAPE;
        total += n;
    }
    if (total > (int64_t)INT32_MAX) return GC_ERR_BAD_SHAPE;
    for (int r = 0; r < b->batch; ++r) {
        const int64_t P = b->prefix_lens_host[r], n = b->new_lens_host[r];
        if (n > 0 && (P + n + gc::kPage - 1) / gc::kPage > geo->max_blocks_per_seq)
            return GC_ERR_BLOCK_TABLE;
    }
    sh->total_tokens = total;
    // the append grid: one workgroup per (page receiving new tokens, KV head), plus
    // the planner's in the combined launch
    if (gc::append_pages_host(b->prefix_lens_host, b->new_lens_host, b->batch) * geo->num_kv_heads >=
        (int64_t)INT32_MAX)
        return GC_ERR_UNSUPPORTED;
    if (total > 0) {
        if (geo->num_blocks <= 0) return GC_ERR_BAD_SHAPE;
        if (b->prefix_lens_dev == nullptr || b->cu_new_lens_dev == nullptr ||
            b->block_tables_dev == nullptr)
            return GC_ERR_NULL_ARG;
    }
    return GC_OK;
}

gc_status check_options(const gc_plan_options* o) {
    if (o == nullptr) return GC_OK;
    if (o->tiling != GC_TILES_AUTO && o->tiling != GC_TILES_PREFILL && o->tiling != GC_TILES_SMALL &&
        o->tiling != GC_TILES_WIDE)
        return GC_ERR_BAD_SHAPE;
    for (int i = 0; i < 6; ++i)
        if (o->reserved[i] != 0) return GC_ERR_BAD_SHAPE;
    return GC_OK;
}

// Tiling: small tiles (one wavefront per 16 query rows, K and V pages streamed through
// its own LDS ring) when every request's new tokens fit one such tile, which is the
// decode case. Otherwise LDS-staged prefill tiles, 128 rows (two workgroups per CU) or
// wide (256 rows, one workgroup per CU). Wide tiles copy each K/V tile once for twice the
// rows; over 8-bit pools, which share their plans with bf16 ones, they also widen it once for
// twice the rows. So at d = 128 and with wide tiles >= 85 % full they are taken, except
//   - between one and two per CU, where whole units leave the last round mostly idle (bf16,
//     128-row against wide: 965 us / 1072 at 288 wide tiles);
//   - below one per CU with fewer than kWideSplitTiles key tiles per CU: a wide launch that
//     short is one prologue, and two small workgroups cover each other's (20.2 / 23.6 at
//     1.4 tiles, 20.0 / 23.8 at 1.7; over 8-bit pools 24.9 / 25.7 and 24.2 / 25.3; at 2.5
//     22.0 / 23.9, but 26.4 / 25.4 over 8-bit pools).
// Above two per CU, 128-row tiles win over bf16 pools up to about 140 key tiles per CU (79 / 93
// at 19, 182 / 189 at 85) and lose 2 to 16 % over 8-bit pools at every size, so wide.
// Not at d = 64 (half the products for the same weights): three 128-row workgroups share a
// compute unit there (164 registers) and overlap better: 16 misses of 100 to 1500 tokens 120 us
// against 148 on wide tiles.
constexpr int kWideSplitTiles = 2;
int device_cus();

// f(key tiles) for every query tile of the batch (block_n: a power of two).
template <typename F>
inline void for_each_tile(const gc_batch* b, int tq, int block_n, F&& f) {
    const int shift = __builtin_ctz((unsigned)block_n);
    for (int r = 0; r < b->batch; ++r) {
        const uint32_t P = (uint32_t)b->prefix_lens_host[r], n = (uint32_t)b->new_lens_host[r];
        for (uint32_t q0 = 0; q0 < n; q0 += (uint32_t)tq) {
            const uint32_t end = q0 + (uint32_t)tq < n ? q0 + (uint32_t)tq : n;
            f((int)((P + end + (uint32_t)block_n - 1) >> shift));
        }
    }
}

gc_status choose_tiling(const gc_geometry* geo, const gc_batch* b, const gc_plan_options* o, Shape* sh) {
    const int want = o == nullptr ? GC_TILES_AUTO : o->tiling;
    bool small = false, wide = false;
    if (want == GC_TILES_SMALL) {
        if (sh->group > gc::kDecM) return GC_ERR_UNSUPPORTED;
        small = true;
    } else if (want == GC_TILES_WIDE) {
        wide = true;
    } else if (want == GC_TILES_AUTO) {
        if (sh->group <= gc::kDecM) {
            small = true;
            for (int r = 0; r < b->batch && small; ++r)
                small = (int64_t)b->new_lens_host[r] * sh->group <= gc::kDecM;
        }
        if (!small && geo->head_dim == 128) {
            const int tq = gc::tokens_per_tile(sh->group, gc::kWideM);
            int64_t units = 0, rows = 0;
            for (int r = 0; r < b->batch; ++r) {
                units += gc::ceil_div64(b->new_lens_host[r], tq);
                rows += (int64_t)b->new_lens_host[r] * sh->group;
            }
            const int64_t cus = device_cus();
            const int64_t grid = units * geo->num_kv_heads;
            if (rows * 100 >= units * gc::kWideM * 85) {
                wide = grid >= 2 * cus;
                if (grid <= cus) {
                    int64_t tiles = 0;
                    for_each_tile(b, tq, gc::kBlockN, [&](int kt) { tiles += kt; });
                    wide = tiles * geo->num_kv_heads >= kWideSplitTiles * cus;
                }
            }
        }
    }
    sh->small = small;
    sh->wide = wide;
    sh->block_m = small ? gc::kDecM : (wide ? gc::kWideM : gc::kBlockM);
    sh->block_n = small ? gc::kDecN : gc::kBlockN;
    sh->tq = gc::tokens_per_tile(sh->group, sh->block_m);
    return GC_OK;
}

// Compute units of the current device (cached per device id).
int device_cus() {
    static std::mutex mu;
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
    if (dev < 64) {
        std::lock_guard<std::mutex> g(mu);
        if (cache[dev] > 0) return cache[dev];
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    if (dev < 64) {
        std::lock_guard<std::mutex> g(mu);
        cache[dev] = cus;
    }
    return cus;
}

// Split policy: keep whole query tiles when there are at least as many work
// items as resident slots (per compute unit: two 128-row workgroups, one wide
// workgroup, or four small-tile wavefronts); otherwise cut the keys into chunks
// so that the launch fills those slots: the smallest chunk that makes no more items
// than slots (each query tile's chunks are rounded up, so equal shares of the key
// tiles make a few items more, which run a round of their own), unless the busiest slot
// ends 8 % sooner with equal shares; and at least 512 keys
// (384 for small tiles), below which the partial rows and a work item's fixed cost
// outweigh the shorter chunks.
// Measured on MI355X (attention and merge, 70B heads): one request of 4100 tokens
// 15.9 us with chunks of 384 keys (24.3 with 1024), four requests of 61 MB of codes
// 18.1 us (29.4 with 1024, 21.5 with 128); 32 requests of 791 MB 145 us with 1000
// items (155 with 1150, 162 with 4000). 16 requests of 4 to 64 new tokens on 4000
// cached ones: 85 us with 480 128-row items (103 with the 600 of equal shares, 97 with
// 1000); one request of 512 on 8000: 137 us with 256 wide items (165 with 288).
// Fitting against equal shares on batches of 0.4 to 1 query tile per slot (1000 of them), by the
// busiest slot of the shares over the fitting chunk, each with an item's fixed cost in key tiles.
// Below 0.92 (12/11) prefill tiles lose by fitting (wide: 114 us / 202 at 0.48, 145 / 220 at
// 0.60, 126 / 159 at 0.69, 66 / 74 at 0.77; 128-row: 230 / 287 at 0.78, 89 / 110 at 0.82), above it
// they gain (wide 45 / 38 at 1.09, 62 / 47 at 1.21; 128-row 89 / 70 at 0.97, 110 / 89 at 1.25),
// with an exception in 100 batches. Small tiles are bound by the memory, not by the slot that ends last, so
// a second item has to save much: 264 / 333 at 0.68, but 59 / 48 at 1.47 and 335 / 278 at 0.95
// (8-bit pools would gain up to 30 % between 0.8 and 1.1, and share their plans with bf16 ones).
constexpr int kSmallMinChunkKeys = 384;
constexpr int kItemTilesSmall = 64, kItemTiles = 16, kItemTilesWide = 5;
constexpr int64_t kMaxSlots = 2048;  // (of 256 compute units: 1024)
int64_t resident_slots(const Shape& sh) {
    const int64_t slots = (sh.small ? 4LL : (sh.wide ? 1LL : 2LL)) * device_cus();
    return slots < kMaxSlots ? slots : kMaxSlots;
}

// Key tiles, and `fixed` for each item, of the slot that ends last when the query tiles kts[0 .. units)
// are cut into chunks of c key tiles (every one `heads` times), more items than slots and at most
// twice as many, and run heaviest first: the items past the slots follow the lightest of the first
// round, the heaviest of the one after the lightest of the other. (Sizes in at most 512 steps.)
// partials: the chunks of the query tiles that are cut.
int busiest_slot(const int32_t* kts, int units, int c, int heads, int64_t slots, int fixed, int64_t* partials) {
    constexpr int kSizes = 512;
    int shift = 0;
    while ((c >> shift) >= kSizes) ++shift;
    const int top = c >> shift;
    int32_t count[kSizes];
    for (int s = 0; s <= top; ++s) count[s] = 0;
    int whole = 0, cut = 0;  // items of query tiles in one piece, and in several
    for (int i = 0; i < units; ++i) {
        if (kts[i] <= c) {
            count[kts[i] >> shift] += 1;
            whole += 1;
            continue;
        }
        const int ns = 1 + (int)((double)(kts[i] - 1) / (double)c);  // (exact, as in choose_chunk)
        const int lo = (int)((double)kts[i] / (double)ns), n_hi = kts[i] - lo * ns;
        count[lo >> shift] += ns - n_hi;
        if (n_hi > 0) count[(lo + 1) >> shift] += n_hi;
        cut += ns;
    }
    *partials = cut;
    int64_t past = (int64_t)(whole + cut) * heads - slots;
    // the size `a` at place slots - 1 of the list, then upwards; `b` from place slots downwards
    int a = top;
    int64_t in_a = (int64_t)count[a] * heads, first = slots;
    int alone = 0, two = 0;  // most tiles of a slot with one item, with two
    while (first > in_a && a > 0) {
        if (in_a > 0 && alone == 0) alone = a;
        first -= in_a;
        in_a = (int64_t)count[--a] * heads;
    }
    int b = a;
    int64_t in_b = in_a - first;  // those of size a past the slots
    in_a = first;
    while (past > 0) {
        while (in_a == 0 && a < top) in_a = (int64_t)count[++a] * heads;
        while (in_b == 0 && b > 0) in_b = (int64_t)count[--b] * heads;
        const int64_t m = in_a < in_b ? in_a : in_b;
        if (m <= 0) break;
        if (a + b > two) two = a + b;
        in_a -= m;
        in_b -= m;
        past -= m;
    }
    alone = (alone << shift) + fixed;
    two = (two << shift) + 2 * fixed;
    return alone > two ? alone : two;
}

int choose_chunk(const gc_geometry* geo, const gc_batch* b, const Shape& sh,
                 const gc_plan_options* o) {
    if (o != nullptr && o->kv_split_tiles != 0) return o->kv_split_tiles > 0 ? o->kv_split_tiles : 0;
    const int64_t target = resident_slots(sh), heads = geo->num_kv_heads;
    int64_t all_units = 0;
    for (int r = 0; r < b->batch; ++r) all_units += gc::ceil_div64(b->new_lens_host[r], sh.tq);
    if (all_units * heads >= target || all_units == 0) return 0;
    const int units = (int)all_units;  // fewer than slots
    int32_t kts[kMaxSlots];            // their key tiles
    int max_tiles = 1, at = 0;
    int64_t tiles = 0;
    for_each_tile(b, sh.tq, sh.block_n, [&](int kt) {
        kts[at++] = kt;
        tiles += kt;
        if (kt > max_tiles) max_tiles = kt;
    });
    const int64_t least = (tiles * heads + target - 1) / target;  // equal shares
    const int min_keys = sh.small ? kSmallMinChunkKeys : 512;
    int lo = least < min_keys / sh.block_n ? min_keys / sh.block_n : (int)least;  // (least <= max_tiles)
    if (lo >= max_tiles) return lo;  // unsplit
    // The smallest chunk whose items fit the slots, per KV head. A chunk of c makes fewer than
    // tiles / c + units items, which bounds the search from above.
    const int64_t slots = target / heads;
    auto items = [&](int c) {  // (exact: a double holds either operand, and quotients below 2^31 apart)
        int k = units;
        for (int i = 0; i < units; ++i) k += (int)((double)(kts[i] - 1) / (double)c);
        return (int64_t)k;
    };
    const int64_t shares = items(lo);
    if (shares <= slots) return lo;
    int hi = max_tiles;  // unsplit tiles: units < slots
    if (slots > units && (tiles + slots - units - 1) / (slots - units) < hi)
        hi = (int)((tiles + slots - units - 1) / (slots - units));
    // Near as many query tiles as slots, few of them can be cut: where the chunk that fits is far
    // above the load of the busiest slot with equal shares, those are better.
    // (That slot carries at least the mean load.)
    const int fixed = sh.small ? kItemTilesSmall : sh.wide ? kItemTilesWide : kItemTiles;
    auto limit = [&](int64_t load) { return load * 12 / 11 - fixed; };
    const int64_t mean = (tiles + shares * fixed) * heads / target;
    if (limit(mean) < hi && items((int)limit(mean)) <= slots) {
        hi = (int)limit(mean);
    } else if (limit(mean) < hi && shares < 2 * slots) {
        int64_t partials;
        const int64_t fits = limit(busiest_slot(kts, units, lo, (int)heads, target, fixed, &partials));
        // (partial rows within 60 MB, that the calls on the fixed scratch take the batch)
        if (fits < hi && partials * heads * sh.block_m * (geo->head_dim + 1) * 4 <= 60000000) {
            if (fits <= lo || items((int)fits) > slots) return lo;
            hi = (int)fits;
        }
    }
    lo += 1;
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (items(mid) <= slots) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// Work-list order. Items run in list order, and a list in strict cost order,
// heaviest first, ends on its lightest items (longest-processing-time order).
// Only the end needs that order, though: before it the items are sorted by the
// length of their request instead, so that a request's query tiles, which read
// nearly the same keys, run side by side and share the K/V tiles in L2. In cost
// order the tiles of a long miss (one of every cost from 1 up) are spread over the
// whole launch and each fetches the same K/V again. The lightest items, two rounds
// of the resident slots, keep the strict order: items of fewer than group_cost
// key tiles; a list no longer than that is not grouped at all.
void choose_order(const gc_geometry* geo, const gc_batch* b, const Shape& sh, Plan* pl) {
    pl->group_cost = gc::kCostBuckets;
    const int64_t tail = (2 * resident_slots(sh) + geo->num_kv_heads - 1) / geo->num_kv_heads;  // items per KV head
    if (pl->items <= tail) return;
    int64_t hist[gc::kCostBuckets] = {};  // items per cost (clamped like the planner's buckets)
    for_each_tile(b, sh.tq, sh.block_n, [&](int kt) {
        const int ns = gc::num_splits(kt, pl->chunk);
        const int lo = ns == 1 ? kt : kt / ns, n_hi = kt - lo * ns;
        hist[lo < gc::kCostBuckets - 1 ? lo : gc::kCostBuckets - 1] += ns - n_hi;
        if (n_hi > 0) hist[lo + 1 < gc::kCostBuckets - 1 ? lo + 1 : gc::kCostBuckets - 1] += n_hi;
    });
    int64_t below = 0;
    int c = 0;
    while (c < gc::kCostBuckets && below < tail) below += hist[c++];
    pl->group_cost = c;  // the items of cost < c make up the tail
}

// Which 128-row workgroups the kernel prefers (attention_kernels.h): of the two that share a
// compute unit, the first round's, which hold the heaviest items, or the second's. The
// first where the heaviest item decides the end: in launches of one round, and beyond where its
// key tiles exceed the mean load of a slot by a quarter (an item's fixed cost counted as four
// tiles; below a quarter the lighter items had better end soon and make room). Preferring the
// second round against the first, bf16 / 8-bit pools, 200 ragged batches: one round 1.00 to
// 1.13 times the time (520 items, the longest of 63 tiles on a mean load of 41: 100.0 us / 89.2,
// 126.5 / 117.1); 1.25 to 3 times the mean load 0.92 to 1.15, two in three above 1.04; below,
// 0.84 to 1.06 (chat turns of 648 items, 62 tiles on 56: 117.1 / 120.4, 151.0 / 173.1).
bool heaviest_decides(int64_t items, int64_t tiles, int heaviest, int64_t slots) {
    constexpr int kItemTiles = 4;
    return items <= slots || (heaviest + kItemTiles) * slots * 4 >= (tiles + kItemTiles * items) * 5;
}

// 8-bit pools at d = 64: 128-row tiles run three workgroups per compute unit, at the price of spilled
// registers, where there is a third one and the mean load of a slot (two per unit) is long enough
// for the spills at an item's ends (three workgroups / two: 84.2 us / 95.0 at 58 tiles, 41.1 / 46.7
// at 28, 69.2 / 74.2 at 17, 30.4 / 30.9 at 15; 24.4 / 23.1 at 11, 22.2 / 21.1 at 9).
constexpr int kThirdTiles = 13;

gc_status make_plan(const gc_geometry* geo, const gc_batch* b, const Shape& sh,
                    const gc_plan_options* o, Plan* pl) {
    pl->chunk = choose_chunk(geo, b, sh, o);
    int longest = 0;  // key tiles of the longest query tile
    const int chunk = pl->chunk;
    int64_t units = 0, combines = 0, partials = 0, tiles = 0;
    for_each_tile(b, sh.tq, sh.block_n, [&](int kt) {
        units += 1;
        tiles += kt;
        if (kt > longest) longest = kt;
        if (chunk > 0 && kt > chunk) {
            combines += 1;
            partials += (uint32_t)(kt + chunk - 1) / (uint32_t)chunk;
        }
    });
    pl->items = units - combines + partials;
    pl->combines = combines;
    pl->partials = partials;
    pl->max_splits = gc::num_splits(longest, chunk);
    if (pl->items > (int64_t)INT32_MAX / geo->num_kv_heads) return GC_ERR_BAD_SHAPE;
    const int64_t slots = resident_slots(sh);
    pl->heaviest_decides = heaviest_decides(pl->items * geo->num_kv_heads, tiles * geo->num_kv_heads,
                                            chunk > 0 && longest > chunk ? chunk : longest, slots);
    pl->three = pl->items * geo->num_kv_heads > slots && tiles * geo->num_kv_heads >= kThirdTiles * slots;
    pl->layout = gc::workspace_layout(b->batch, pl->items, pl->combines, pl->partials,
                                      geo->num_kv_heads, geo->head_dim, sh.block_m);
    choose_order(geo, b, sh, pl);
    // the largest sort key: a request's key tiles where items are grouped, an item's otherwise
    int key = pl->group_cost < gc::kCostBuckets || pl->chunk <= 0 || longest < pl->chunk ? longest : pl->chunk;
    if (key > gc::kCostBuckets - 1) key = gc::kCostBuckets - 1;
    pl->buckets = (key / gc::kPlanThreads + 1) * gc::kPlanThreads;
    return GC_OK;
}

template <typename T>
T* at(void* ws, size_t off) {
    return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

gc_status plan_checked(const gc_geometry* geo, const gc_batch* b, const gc_plan_options* o,
                       Shape* sh, Plan* pl) {
    gc_status st = check_common(geo, b, sh);
    if (st != GC_OK) return st;
    st = check_options(o);
    if (st != GC_OK) return st;
    st = choose_tiling(geo, b, o, sh);
    if (st != GC_OK) return st;
    if (sh->total_tokens == 0) return GC_OK;
    return make_plan(geo, b, *sh, o, pl);
}

gc::PlanArgs plan_args(const gc_geometry* geo, const gc_batch* b, const Shape& sh, const Plan& pl, void* ws) {
    gc::PlanArgs a{};
    a.prefix_lens = b->prefix_lens_dev;
    a.cu_new_lens = b->cu_new_lens_dev;
    a.scratch = at<int32_t>(ws, pl.layout.scratch_off);
    a.items = at<gc::WorkItem>(ws, pl.layout.items_off);
    a.combines = at<gc::CombineItem>(ws, pl.layout.combine_off);
    a.status = at<int32_t>(ws, pl.layout.status_off);
    a.queues = at<int32_t>(ws, pl.layout.queue_off);
    a.batch = b->batch;
    a.tq = sh.tq;
    a.chunk = pl.chunk;
    a.block_n = sh.block_n;
    a.expect_items = (int32_t)pl.items;
    a.expect_combines = (int32_t)pl.combines;
    a.expect_partials = (int32_t)pl.partials;
    a.total_tokens = (int32_t)sh.total_tokens;
    a.max_blocks = geo->max_blocks_per_seq;
    a.group_cost = pl.group_cost;
    a.buckets = pl.buckets;
    return a;
}

gc_status enqueue_plan(const gc_geometry* geo, const gc_batch* b, const Shape& sh, const Plan& pl,
                       void* ws, hipStream_t stream) {
    return gc::launch_plan(plan_args(geo, b, sh, pl, ws), stream) == hipSuccess ? GC_OK : GC_ERR_HIP;
}

// Wide tiles with at least two rounds of work items per compute unit run as a
// resident launch (one workgroup per CU taking items from per-XCD queues;
// attention_kernels.h): it removes the dispatch gaps between items and lets the XCDs that
// finish first take the last items of the others. A single round has nothing to
// balance. 0: the regular launch.
int resident_workgroups(const gc_geometry* geo, const Shape& sh, const Plan& pl) {
    if (!sh.wide) return 0;
    const int cus = device_cus();
    if (cus % gc::kQueues != 0) return 0;
    return pl.items * geo->num_kv_heads >= 2LL * cus ? cus : 0;
}

// Pools of bf16 elements (fp8 false, scales 1) or of E4M3 codes with one scale each.
struct PoolKind {
    bool fp8 = false;
    float k_scale = 1.f, v_scale = 1.f;
};

gc_status enqueue_run(const gc_geometry* geo, const gc_batch* b, const Shape& sh, const Plan& pl,
                      const void* q, const void* k_pool, const void* v_pool, float scale,
                      void* out, float* lse, void* ws, hipStream_t stream, const PoolKind& pk = PoolKind{}) {
    gc::AttnArgs a{};
    a.q = static_cast<const uint16_t*>(q);
    a.k_pool = static_cast<const uint16_t*>(k_pool);
    a.v_pool = static_cast<const uint16_t*>(v_pool);
    a.out = static_cast<uint16_t*>(out);
    a.lse = lse;
    a.part_o = at<float>(ws, pl.layout.part_o_off);
    a.part_lse = at<float>(ws, pl.layout.part_lse_off);
    a.block_tables = b->block_tables_dev;
    a.items = at<gc::WorkItem>(ws, pl.layout.items_off);
    a.queues = at<int32_t>(ws, pl.layout.queue_off);
    a.num_q_heads = geo->num_q_heads;
    a.num_kv_heads = geo->num_kv_heads;
    a.group = sh.group;
    a.tq = sh.tq;
    a.num_blocks = geo->num_blocks;
    a.max_blocks = geo->max_blocks_per_seq;
    a.scale_log2 = (float)((double)scale * (double)pk.k_scale * 1.4426950408889634074);
    a.v_scale = pk.v_scale;
    a.prefer_span = (uint32_t)device_cus();
    a.prefer_odd = pl.heaviest_decides ? 0 : 1;
    const hipError_t e = sh.small ? gc::launch_attention_small(a, geo->head_dim, pl.items, pk.fp8, stream)
                                  : gc::launch_attention(a, geo->head_dim, pl.items, sh.wide, pl.three, pk.fp8,
                                                         resident_workgroups(geo, sh, pl), stream);
    if (e != hipSuccess) return GC_ERR_HIP;
    if (pl.combines > 0) {
        gc::CombineArgs c{};
        c.out = a.out;
        c.lse = lse;
        c.part_o = a.part_o;
        c.part_lse = a.part_lse;
        c.cu_new_lens = b->cu_new_lens_dev;
        c.combines = at<gc::CombineItem>(ws, pl.layout.combine_off);
        c.num_q_heads = geo->num_q_heads;
        c.num_kv_heads = geo->num_kv_heads;
        c.group = sh.group;
        c.tq = sh.tq;
        c.batch = b->batch;
        c.num_partials = (int32_t)pl.partials;
        c.block_m = sh.block_m;
        if (gc::launch_combine(c, geo->head_dim, pl.combines, pl.max_splits, stream) != hipSuccess) return GC_ERR_HIP;
    }
    return GC_OK;
}

gc_status check_run_args(const void* q, const void* k_pool, const void* v_pool, float scale,
                         void* out) {
    if (q == nullptr || k_pool == nullptr || v_pool == nullptr || out == nullptr)
        return GC_ERR_NULL_ARG;
    if (!std::isfinite(scale) || !(scale > 0.f)) return GC_ERR_BAD_SHAPE;
    return GC_OK;
}

gc_status check_pool_scales(float k_scale, float v_scale) {
    if (!std::isfinite(k_scale) || !(k_scale > 0.f) || !std::isfinite(v_scale) || !(v_scale > 0.f))
        return GC_ERR_BAD_SHAPE;
    // the append multiplies by fl32(1 / scale), which must be finite as well
    if (!std::isfinite(1.f / k_scale) || !std::isfinite(1.f / v_scale)) return GC_ERR_BAD_SHAPE;
    return GC_OK;
}

gc_status check_workspace(const Plan& pl, const void* ws, size_t bytes) {
    if (ws == nullptr || bytes < pl.layout.total) return GC_ERR_WORKSPACE;
    return GC_OK;
}

gc::AppendArgs append_args(const gc_geometry* geo, const gc_batch* batch, const Shape& sh,
                           const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                           const PoolKind& pk) {
    gc::AppendArgs a{};
    a.k_new = static_cast<const uint16_t*>(k_new);
    a.v_new = static_cast<const uint16_t*>(v_new);
    a.k_pool = k_pool;
    a.v_pool = v_pool;
    a.prefix_lens = batch->prefix_lens_dev;
    a.cu_new_lens = batch->cu_new_lens_dev;
    a.block_tables = batch->block_tables_dev;
    a.batch = batch->batch;
    a.total_tokens = (int32_t)sh.total_tokens;
    a.num_kv_heads = geo->num_kv_heads;
    a.num_blocks = geo->num_blocks;
    a.max_blocks = geo->max_blocks_per_seq;
    a.total_pages = (int32_t)gc::append_pages_host(batch->prefix_lens_host, batch->new_lens_host, batch->batch);
    a.k_inv = 1.f / pk.k_scale;  // IEEE division: the same fl32(1 / scale) the definition uses
    a.v_inv = 1.f / pk.v_scale;
    return a;
}

gc_status append(const gc_geometry* geo, const gc_batch* batch, const void* k_new, const void* v_new,
                 void* k_pool, void* v_pool, const PoolKind& pk, hipStream_t stream) {
    Shape sh;
    gc_status st = check_common(geo, batch, &sh);
    if (st != GC_OK) return st;
    if (sh.total_tokens == 0) return GC_OK;
    if (k_new == nullptr || v_new == nullptr || k_pool == nullptr || v_pool == nullptr)
        return GC_ERR_NULL_ARG;
    const gc::AppendArgs a = append_args(geo, batch, sh, k_new, v_new, k_pool, v_pool, pk);
    return gc::launch_append(a, geo->head_dim, pk.fp8, stream) == hipSuccess ? GC_OK : GC_ERR_HIP;
}

// Append and plan in one launch (the plan reads only the lengths, so the two are
// independent).
gc_status prepare(const gc_geometry* geo, const gc_batch* batch, const gc_plan_options* opts,
                  const void* k_new, const void* v_new, void* k_pool, void* v_pool, void* workspace,
                  size_t workspace_bytes, hipStream_t stream, const PoolKind& pk) {
    Shape sh;
    Plan pl;
    gc_status st = plan_checked(geo, batch, opts, &sh, &pl);
    if (st != GC_OK || sh.total_tokens == 0) return st;
    if (k_new == nullptr || v_new == nullptr || k_pool == nullptr || v_pool == nullptr)
        return GC_ERR_NULL_ARG;
    if (pk.fp8) {
        st = check_pool_scales(pk.k_scale, pk.v_scale);
        if (st != GC_OK) return st;
    }
    st = check_workspace(pl, workspace, workspace_bytes);
    if (st != GC_OK) return st;
    const gc::AppendArgs aa = append_args(geo, batch, sh, k_new, v_new, k_pool, v_pool, pk);
    return gc::launch_prepare(aa, plan_args(geo, batch, sh, pl, workspace), geo->head_dim, pk.fp8, stream) ==
                   hipSuccess
               ? GC_OK
               : GC_ERR_HIP;
}

gc_status run(const gc_geometry* geo, const gc_batch* batch, const gc_plan_options* opts,
              const void* q, const void* k_pool, const void* v_pool, float scale, void* out,
              float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream,
              bool with_plan, const PoolKind& pk) {
    Shape sh;
    Plan pl;
    gc_status st = plan_checked(geo, batch, opts, &sh, &pl);
    if (st != GC_OK || sh.total_tokens == 0) return st;
    st = check_run_args(q, k_pool, v_pool, scale, out);
    if (st != GC_OK) return st;
    if (pk.fp8) {
        st = check_pool_scales(pk.k_scale, pk.v_scale);
        if (st != GC_OK) return st;
    }
    st = check_workspace(pl, workspace, workspace_bytes);
    if (st != GC_OK) return st;
    if (with_plan) {
        st = enqueue_plan(geo, batch, sh, pl, workspace, stream);
        if (st != GC_OK) return st;
    }
    return enqueue_run(geo, batch, sh, pl, q, k_pool, v_pool, scale, out, lse, workspace, stream, pk);
}

// ---------------------------------------------------------------- no-allocation variant
// Workspace of gc_prefix_prefill_attention_noalloc: one file-scope device array per
// GPU the library runs on (held until the process ends). Host code never passes the
// array's name to a kernel or a copy: in host code it is a host-side stand-in, not
// a device address. The device address comes from hipGetSymbolAddress, taken once
// per device with that device current, and is kept per device.
static __device__ __align__(256) unsigned char scratch[GC_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
struct DeviceScratch {
    std::once_flag once;
    void* ptr = nullptr;
    hipError_t err = hipSuccess;
};
DeviceScratch g_scratch[kMaxDevices];

// Device address of the current device's scratch array (nullptr and a status on failure).
void* scratch_address(gc_status* st) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
        *st = GC_ERR_HIP;
        return nullptr;
    }
    if (dev >= kMaxDevices) {
        *st = GC_ERR_UNSUPPORTED;
        return nullptr;
    }
    DeviceScratch& d = g_scratch[dev];
    std::call_once(d.once, [&d]() { d.err = hipGetSymbolAddress(&d.ptr, HIP_SYMBOL(scratch)); });
    if (d.err != hipSuccess || d.ptr == nullptr) {
        *st = GC_ERR_HIP;
        return nullptr;
    }
    *st = GC_OK;
    return d.ptr;
}

// Append and run from a plan already in the workspace, as two launches. One launch that
// read the new keys from k_new / v_new and wrote them into the pool from LDS read the new keys'
// values through registers in every tile that holds some, and could not run as a resident
// launch. One / two launches, us a pass, on the same tiles: 16 chat requests of the 70B shape 214 /
// 195, 8 of the 8B shape 147 / 128, the mixed 70B batch 2547 / 2196, 6 mixed 8B requests 205 / 174;
// only the smallest calls lose the second launch (one request of 32 tokens 11.7 / 14.1).
gc_status run_with_append(const gc_geometry* geo, const gc_batch* batch, const gc_plan_options* opts,
                          const void* q, const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                          float scale, void* out, float* lse, void* workspace, size_t workspace_bytes,
                          hipStream_t stream) {
    Shape sh;
    Plan pl;
    gc_status st = plan_checked(geo, batch, opts, &sh, &pl);
    if (st != GC_OK || sh.total_tokens == 0) return st;
    st = check_run_args(q, k_pool, v_pool, scale, out);
    if (st != GC_OK) return st;
    if (k_new == nullptr || v_new == nullptr) return GC_ERR_NULL_ARG;
    st = check_workspace(pl, workspace, workspace_bytes);
    if (st != GC_OK) return st;
    // (a limit of the interface: a request's new rows within 32-bit byte offsets)
    const int64_t row_bytes = (int64_t)geo->num_kv_heads * geo->head_dim * 2;
    for (int r = 0; r < batch->batch; ++r)
        if ((int64_t)batch->new_lens_host[r] * row_bytes > INT32_MAX) return GC_ERR_UNSUPPORTED;
    const gc::AppendArgs aa = append_args(geo, batch, sh, k_new, v_new, k_pool, v_pool, PoolKind{});
    if (gc::launch_append(aa, geo->head_dim, false, stream) != hipSuccess) return GC_ERR_HIP;
    return enqueue_run(geo, batch, sh, pl, q, k_pool, v_pool, scale, out, lse, workspace, stream);
}

}  // namespace

extern "C" {

__attribute__((visibility("default")))
gc_status gc_kv_append(const gc_geometry* geo, const gc_batch* batch, const void* k_new,
                       const void* v_new, void* k_pool, void* v_pool, hipStream_t stream) {
    return append(geo, batch, k_new, v_new, k_pool, v_pool, PoolKind{}, stream);
}

__attribute__((visibility("default")))
gc_status gc_kv_append_fp8(const gc_geometry* geo, const gc_batch* batch, const void* k_new,
                           const void* v_new, float k_scale, float v_scale, void* k_pool,
                           void* v_pool, hipStream_t stream) {
    const gc_status st = check_pool_scales(k_scale, v_scale);
    if (st != GC_OK) return st;
    return append(geo, batch, k_new, v_new, k_pool, v_pool, PoolKind{true, k_scale, v_scale}, stream);
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_workspace_size(const gc_geometry* geo, const gc_batch* batch,
                                           const gc_plan_options* opts, size_t* bytes) {
    if (bytes == nullptr) return GC_ERR_NULL_ARG;
    Shape sh;
    Plan pl;
    gc_status st = plan_checked(geo, batch, opts, &sh, &pl);
    if (st != GC_OK) return st;
    *bytes = sh.total_tokens == 0 ? 0 : pl.layout.total;
    return GC_OK;
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_plan(const gc_geometry* geo, const gc_batch* batch,
                                 const gc_plan_options* opts, void* workspace,
                                 size_t workspace_bytes, hipStream_t stream) {
    Shape sh;
    Plan pl;
    gc_status st = plan_checked(geo, batch, opts, &sh, &pl);
    if (st != GC_OK || sh.total_tokens == 0) return st;
    st = check_workspace(pl, workspace, workspace_bytes);
    if (st != GC_OK) return st;
    return enqueue_plan(geo, batch, sh, pl, workspace, stream);
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_run(const gc_geometry* geo, const gc_batch* batch,
                                const gc_plan_options* opts, const void* q, const void* k_pool,
                                const void* v_pool, float scale, void* out, float* lse,
                                void* workspace, size_t workspace_bytes, hipStream_t stream) {
    return run(geo, batch, opts, q, k_pool, v_pool, scale, out, lse, workspace, workspace_bytes,
               stream, false, PoolKind{});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_attention(const gc_geometry* geo, const gc_batch* batch,
                                      const gc_plan_options* opts, const void* q,
                                      const void* k_pool, const void* v_pool, float scale,
                                      void* out, float* lse, void* workspace,
                                      size_t workspace_bytes, hipStream_t stream) {
    return run(geo, batch, opts, q, k_pool, v_pool, scale, out, lse, workspace, workspace_bytes,
               stream, true, PoolKind{});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_attention_noalloc(const gc_geometry* geo, const gc_batch* batch,
                                              const gc_plan_options* opts, const void* q,
                                              const void* k_pool, const void* v_pool, float scale,
                                              void* out, float* lse, hipStream_t stream) {
    // every host check first (workspace size included), then the device address
    Shape sh;
    Plan pl;
    gc_status st = plan_checked(geo, batch, opts, &sh, &pl);
    if (st != GC_OK || sh.total_tokens == 0) return st;
    st = check_run_args(q, k_pool, v_pool, scale, out);
    if (st != GC_OK) return st;
    if (pl.layout.total > (size_t)GC_NOALLOC_SCRATCH_BYTES) return GC_ERR_WORKSPACE;
    void* ws = scratch_address(&st);
    if (ws == nullptr) return st;
    return run(geo, batch, opts, q, k_pool, v_pool, scale, out, lse, ws, GC_NOALLOC_SCRATCH_BYTES, stream,
               true, PoolKind{});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_run_with_append(const gc_geometry* geo, const gc_batch* batch,
                                            const gc_plan_options* opts, const void* q, const void* k_new,
                                            const void* v_new, void* k_pool, void* v_pool, float scale,
                                            void* out, float* lse, void* workspace, size_t workspace_bytes,
                                            hipStream_t stream) {
    return run_with_append(geo, batch, opts, q, k_new, v_new, k_pool, v_pool, scale, out, lse, workspace,
                           workspace_bytes, stream);
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_run_fp8(const gc_geometry* geo, const gc_batch* batch,
                                    const gc_plan_options* opts, const void* q, const void* k_pool,
                                    const void* v_pool, float k_scale, float v_scale, float scale,
                                    void* out, float* lse, void* workspace, size_t workspace_bytes,
                                    hipStream_t stream) {
    return run(geo, batch, opts, q, k_pool, v_pool, scale, out, lse, workspace, workspace_bytes,
               stream, false, PoolKind{true, k_scale, v_scale});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_attention_fp8(const gc_geometry* geo, const gc_batch* batch,
                                          const gc_plan_options* opts, const void* q,
                                          const void* k_pool, const void* v_pool, float k_scale,
                                          float v_scale, float scale, void* out, float* lse,
                                          void* workspace, size_t workspace_bytes,
                                          hipStream_t stream) {
    return run(geo, batch, opts, q, k_pool, v_pool, scale, out, lse, workspace, workspace_bytes,
               stream, true, PoolKind{true, k_scale, v_scale});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_prepare(const gc_geometry* geo, const gc_batch* batch,
                                    const gc_plan_options* opts, const void* k_new, const void* v_new,
                                    void* k_pool, void* v_pool, void* workspace, size_t workspace_bytes,
                                    hipStream_t stream) {
    return prepare(geo, batch, opts, k_new, v_new, k_pool, v_pool, workspace, workspace_bytes, stream,
                   PoolKind{});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_prepare_fp8(const gc_geometry* geo, const gc_batch* batch,
                                        const gc_plan_options* opts, const void* k_new, const void* v_new,
                                        float k_scale, float v_scale, void* k_pool8, void* v_pool8,
                                        void* workspace, size_t workspace_bytes, hipStream_t stream) {
    return prepare(geo, batch, opts, k_new, v_new, k_pool8, v_pool8, workspace, workspace_bytes, stream,
                   PoolKind{true, k_scale, v_scale});
}

__attribute__((visibility("default")))
gc_status gc_prefix_prefill_plan_status(const void* workspace, size_t workspace_bytes, hipStream_t stream) {
    if (workspace == nullptr) return GC_ERR_NULL_ARG;
    if (workspace_bytes < sizeof(int32_t)) return GC_ERR_WORKSPACE;
    static_assert(gc::kStatusOffset == 0, "the status word leads the workspace");
    int32_t word = 0;
    if (hipMemcpyAsync(&word, workspace, sizeof(word), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return GC_ERR_HIP;
    return word == 0 ? GC_OK : GC_ERR_LENGTHS;
}

__attribute__((visibility("default")))
gc_status gc_read_bandwidth_probe(const void* buf, size_t bytes, void* sink, hipStream_t stream) {
    if (buf == nullptr || sink == nullptr) return GC_ERR_NULL_ARG;
    if (bytes % 16 != 0) return GC_ERR_BAD_SHAPE;
    if (bytes == 0) return GC_OK;
    return gc::launch_read_probe(buf, bytes, static_cast<uint32_t*>(sink), stream) == hipSuccess ? GC_OK
                                                                                               : GC_ERR_HIP;
}

__attribute__((visibility("default")))
gc_status gc_mfma_peak_probe(int32_t iterations, void* sink, hipStream_t stream) {
    static_assert(GC_MFMA_PROBE_SINK_FLOATS == gc::kMfmaProbeBlocks * gc::kProbeThreads, "sink size");
    static_assert(GC_MFMA_PROBE_PRODUCTS_PER_ITERATION ==
                      gc::kMfmaProbeBlocks * (gc::kProbeThreads / 64) * gc::kMfmaProbeChains * gc::kMfmaProbePerChain,
                  "products per iteration");
    if (sink == nullptr) return GC_ERR_NULL_ARG;
    if (iterations < 0) return GC_ERR_BAD_SHAPE;
    if (iterations == 0) return GC_OK;
    return gc::launch_mfma_probe(iterations, static_cast<float*>(sink), stream) == hipSuccess ? GC_OK : GC_ERR_HIP;
}

__attribute__((visibility("default")))
const char* gc_status_string(gc_status s) {
    switch (s) {
        case GC_OK: return "GC_OK: success";
        case GC_ERR_NULL_ARG: return "GC_ERR_NULL_ARG: a required pointer is NULL";
        case GC_ERR_BAD_SHAPE: return "GC_ERR_BAD_SHAPE: invalid size, length or scale";
        case GC_ERR_UNSUPPORTED: return "GC_ERR_UNSUPPORTED: head_dim must be 64 or 128, page_size 16, Hq/Hkv <= 128 (<= 16 for small tiles)";
        case GC_ERR_BLOCK_TABLE: return "GC_ERR_BLOCK_TABLE: block table too short for a request";
        case GC_ERR_WORKSPACE: return "GC_ERR_WORKSPACE: workspace missing or too small";
        case GC_ERR_HIP: return "GC_ERR_HIP: a HIP launch failed";
        case GC_ERR_LENGTHS: return "GC_ERR_LENGTHS: the device length arrays disagree with the host's";
    }
    return "unknown gc_status";
}

}  // extern "C"
