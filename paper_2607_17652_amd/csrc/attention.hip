// W-shaped block-causal window attention (Sec. 4.1; Eq. 5 per packed row).
//
// The mask of Eq. 5 reduces, for window slot s of request b, to one key count
// kv_len = o_b + (s+1)*bl: every query of that block sees keys [0, kv_len) of
// its KV head -- the frozen prefix, the earlier live blocks and its own block.
// So the work is a set of independent "prefix attentions", one per
// (live block, KV head), each with bl*(Hq/Hkv) query rows sharing one K/V
// stream (GQA rows packed together).
//
// Work decomposition (all shapes fixed by capacity, so graph-capturable):
//   unit  = (tile, KV head, 128-row group); rows are the block's
//           (position, head-in-group) pairs flattened position-major
//   item  = a unit's key range [kb, ke), a multiple of 32 keys long except at
//           kv_len; long units are split so the grid has enough items
//   plan_kernel    one workgroup: counts key tiles, picks the split size,
//                  emits items (longest first, each with its tile's request
//                  and first row) with their partial slots, and the list of
//                  split units; for packs of at most kInlineTiles tiles the
//                  attention's own waves do this instead (plan_item)
//   attn_bf16      one workgroup (4 waves x 32 rows) per item: 32-key K and
//                  V^T tiles streamed through an LDS ring (3 stages at
//                  D = 128, K refilled a step ahead of V^T; 4 below) by
//                  direct global->LDS loads,
//                  S^T = K Q^T and O^T += V^T P^T on
//                  v_mfma_f32_32x32x16_bf16, online softmax in the exp2
//                  domain with lazy rescaling
//   combine        merges split partials with their log-sum-exp weights,
//                  walking the plan's list of split units
//   attn_f32       the same items in fp32 on v_mfma_f32_32x32x2_f32
#include <float.h>

#include <type_traits>
#include <utility>

#include "internal.h"

namespace fb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kRowsPerWg = 128;     // 4 waves x 32 query rows
constexpr int kAttnThreads = 256;
constexpr int kWgsPerCu = 3;          // attention workgroups per CU aimed at (resident at D = 128)
constexpr int kKeyTile = 32;
constexpr int kF32WgsPerCu = 2;       // the same in fp32
// keys * head_dim of the cache that one fp32 workgroup walks without a plan: a
// key tile takes it about D/32 us.  The line was drawn with a plan and a merge
// of about 16 us on the other side.  Packs of at most 64 tiles have no plan
// kernel since, and a shorter merge; against that (4 requests of 2 blocks) the
// whole unit still wins at 160 keys (d = 64: 14.7 us, split 17.1; d = 128: 24.4,
// 26.9) and loses further on (288 keys, d = 64: 24.9, 19.3; d = 32: 16.0, 14.2;
// 544 keys, d = 32: 28.4, 14.6).
constexpr long long kF32DirectWork = 32768;
constexpr int kMinChunkTiles = 4;   // never split below 128 keys
constexpr int kMaxSplits = 64;      // splits of one unit the combine can merge
constexpr int kMaxHeadDim = 128;    // largest head_dim built (32, 64, 128)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kSkippedLse = INFINITY;   // part_lse of a skipped fp32 block: no row's own is +inf
constexpr float kRescaleSlack = 8.0f;  // lazy rescale: running max may lag by 2^8

// A work item: its unit, key range and partial slot, and the request and
// first packed row of its tile (copied here so the attention workgroup's
// first dependent loads are the item and then the page table).
enum ItemField { kIUnit = 0, kIKb, kIKe, kISlot, kIB, kIRow0, kIItemInts = 8 };
enum CountField { kCItems = 0, kCSplit, kCountInts = 4 };

struct AttnWs {
    int32_t* items;    // [item_cap][kIItemInts]
    int32_t* counts;   // [kCountInts]
    int4* split;       // [split_cap]: {unit, pieces, first slot, first row} of the
                       // units with more than one piece
    float* part_o;     // [slot_cap][128][D]
    float* part_lse;   // [slot_cap][128]
};

// Capacities a plan record must respect to belong to this pack and shape.
// The attention and the combine check every record they read against them,
// so a workspace used without its plan (fb_wavefront_attention_planned
// before fb_attention_plan) is reported, never followed out of bounds.
struct PlanBounds {
    int n_req;          // requests of the pack
    int row_cap;        // packed rows
    int unit_cap;       // units
    int slot_cap;       // split partial slots
    long long max_keys; // keys the page table can address
};


// ---------------------------------------------------------------- plan ----
constexpr int kPlanThreads = 256;   // 4 waves: shorter barrier and scan rounds than 16 (measured 2-4%)
constexpr int kPlanWaves = kPlanThreads / 64;

// Workgroup sum of v[0] and maximum of v[1] (one pair of barriers): each
// wave reduces its 64 lanes, then every wave reduces the kPlanWaves wave
// results itself and broadcasts lane 0's (no serial loop on one thread).
__device__ void wg_sum_max(long long (&v)[2], long long (*lds)[kPlanWaves]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        v[0] += __shfl_xor(v[0], off, 64);
        const long long o = __shfl_xor(v[1], off, 64);
        if (o > v[1]) v[1] = o;
    }
    if (lane == 0) {
        lds[0][wave] = v[0];
        lds[1][wave] = v[1];
    }
    __syncthreads();
    long long sm = lane < kPlanWaves ? lds[0][lane] : 0;
    long long mx = lane < kPlanWaves ? lds[1][lane] : 0;
#pragma unroll
    for (int off = kPlanWaves / 2; off > 0; off >>= 1) {
        sm += __shfl_xor(sm, off, 64);
        const long long o = __shfl_xor(mx, off, 64);
        if (o > mx) mx = o;
    }
    v[0] = __shfl(sm, 0, 64);
    v[1] = __shfl(mx, 0, 64);
    __syncthreads();
}

// Exclusive scans of three ints per thread across the workgroup (one pair of
// barriers for all three): v[i] becomes its exclusive prefix, tot[i] the
// workgroup total.
__device__ void wg_excl_scan3(int (&v)[3], int (&tot)[3], int3* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x[3] = {v[0], v[1], v[2]};
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int u = __shfl_up(x[i], off, 64);
            if (lane >= off) x[i] += u;
        }
    }
    if (lane == 63) lds[wave] = make_int3(x[0], x[1], x[2]);
    __syncthreads();
    const int3 l = lane < kPlanWaves ? lds[lane] : make_int3(0, 0, 0);
    int w[3] = {l.x, l.y, l.z};
#pragma unroll
    for (int off = 1; off < kPlanWaves; off <<= 1) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int u = __shfl_up(w[i], off, 64);
            if (lane >= off) w[i] += u;
        }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int before = __shfl(w[i], wave > 0 ? wave - 1 : 0, 64);
        tot[i] = __shfl(w[i], kPlanWaves - 1, 64);
        v[i] = (wave > 0 ? before : 0) + x[i] - v[i];
    }
    __syncthreads();
}

// Exclusive scan of one int per thread across the workgroup, and the total.
__device__ int wg_excl_scan(int v, int* lds, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) lds[wave] = x;
    __syncthreads();
    // every wave scans the wave totals itself
    int w = lane < kPlanWaves ? lds[lane] : 0;
#pragma unroll
    for (int off = 1; off < kPlanWaves; off <<= 1) {
        int y = __shfl_up(w, off, 64);
        if (lane >= off) w += y;
    }
    const int before = wave > 0 ? __shfl(w, wave - 1, 64) : 0;
    *total = __shfl(w, kPlanWaves - 1, 64);
    __syncthreads();
    return before + x - v;
}

// Items are written longest first (a counting sort on their key-tile count,
// counts of kLenBuckets-1 or more sharing the top bucket): the grid then
// dispatches long items before short ones, which keeps the tail short.  The
// plan works per tile: the per_tile units of a tile (kv-heads x row groups)
// have the same key range, so they get the same split and adjacent items
// (with 8 kv-heads the round-robin dispatch then keeps each kv-head on one
// XCD).  Thread i handles tiles i, i + kPlanThreads, ...; the fields of its
// first kPlanCache tiles are read once and kept in LDS.
constexpr int kLenBuckets = kPlanThreads;
constexpr int kPlanCache = 4;
constexpr int kPlanPieces = 1024;   // pieces of one round staged in LDS

struct PlanTile {
    int kt;   // key tiles of the tile; 0 (skipped, error) past the page table
    int kr;   // sort key: key tiles of its request's last live block
    int kv;   // keys the tile attends to
    int b;    // request
    int row0; // first packed row
};

__device__ inline PlanTile plan_tile(const int32_t* tiles, int t, int n_tiles, long long max_keys) {
    PlanTile p{0, 0, 0, 0, 0};
    if (t >= n_tiles) return p;
    const int32_t* tl = tiles + (size_t)t * kTileInts;
    p.kv = tl[kTKvLen];
    p.b = tl[kTB];
    p.row0 = tl[kTRow0];
    p.kt = (long long)p.kv > max_keys ? 0 : (p.kv + kKeyTile - 1) / kKeyTile;
    // the blocks of one request read the same prefix K/V: keyed by the
    // request's longest block they land in the same buckets next to each
    // other and run together, sharing the prefix through L2
    const long long blen = tl[kTKvLen] - tl[kTPos0];
    const long long kv_last = tl[kTO] + (long long)tl[kTW] * blen;
    const long long kr = (kv_last + kKeyTile - 1) / kKeyTile;
    p.kr = kr > p.kt ? (int)kr : p.kt;
    return p;
}

// Split size in key tiles.  With chunk >= total_tiles / target_items the items
// and the partial slots always fit: a unit of kt key tiles makes
// ceil(kt/chunk) <= kt/chunk + 1 items, so all units make at most
// total_tiles/chunk + n_units <= item_cap, and a split unit's
// ceil(kt/chunk) < 2 kt/chunk slots sum to at most 2 target_items =
// slot_cap.  A chunk >= kt_max / kMaxSplits keeps every unit within the
// splits the combine merges.  A requested split size is doubled until
// both hold.  (Sizes stay below 2^30 key tiles: 32-bit math in the callers.)
__device__ inline long long split_chunk(long long total_tiles, long long kt_max,
                                        int target_items, int fixed_chunk_tiles) {
    const long long up = total_tiles + target_items - 1;
    long long need = up <= 0xffffffffLL ? (long long)((uint32_t)up / (uint32_t)target_items)
                                        : up / target_items;
    const long long need_m = (kt_max + kMaxSplits - 1) / kMaxSplits;
    if (need_m > need) need = need_m;
    if (fixed_chunk_tiles > 0) {
        long long chunk = fixed_chunk_tiles;
        while (chunk < need) chunk *= 2;
        return chunk;
    }
    return need > kMinChunkTiles ? need : kMinChunkTiles;
}

__global__ void __launch_bounds__(kPlanThreads)
plan_kernel(PackView pv, AttnWs ws, int Hkv, int RG, int item_cap, int split_cap,
            int target_items, int fixed_chunk_tiles, long long max_keys) {
    __shared__ long long sum_lds[2][kPlanWaves];
    __shared__ int scan_lds[kPlanWaves + 1];
    __shared__ int3 trio_lds[kPlanWaves];
    __shared__ int bucket[kLenBuckets];
    const int n_tiles = pv.hdr[kHdrTiles];
    const int per_tile = Hkv * RG;
    const int n_rounds = (n_tiles + kPlanThreads - 1) / kPlanThreads;

    // this thread's first kPlanCache tiles, read once; kept in LDS (a
    // register array indexed by the round would live in scratch memory)
    __shared__ PlanTile s_cache[kPlanCache * kPlanThreads];
#pragma unroll
    for (int j = 0; j < kPlanCache; ++j)
        s_cache[j * kPlanThreads + threadIdx.x] =
            plan_tile(pv.tiles, j * kPlanThreads + threadIdx.x, n_tiles, max_keys);
    // this thread's tile of round c (zeros past the end)
    auto tile_of = [&](int c) -> PlanTile {
        if (c >= kPlanCache)
            return plan_tile(pv.tiles, c * kPlanThreads + threadIdx.x, n_tiles, max_keys);
        return s_cache[c * kPlanThreads + threadIdx.x];
    };

    // key tiles summed over the tiles, and the longest tile
    long long red[2] = {0, 0};
    for (int c = 0; c < n_rounds; ++c) {
        const int kt = tile_of(c).kt;
        red[0] += kt;
        if (kt > red[1]) red[1] = kt;
    }
    wg_sum_max(red, sum_lds);
    const long long total_tiles = red[0] * per_tile;
    const long long kt_max = red[1];

    const long long chunk_ll = split_chunk(total_tiles, kt_max, target_items, fixed_chunk_tiles);
    if (chunk_ll >= (1 << 30)) {
        // beyond any real cache (over 2^30 key tiles per item): nothing is
        // planned and the first tile's request is flagged
        if (threadIdx.x == 0) {
            record_error(pv.hdr, pv.tiles[kTB], FB_DERR_PAGE);
            ws.counts[kCItems] = 0;
            ws.counts[kCSplit] = 0;
        }
        return;
    }
    const int chunk = (int)chunk_ll;

    // Histogram of item lengths, then each bucket's first position with the
    // longest bucket first.
    // A unit of at most 1.5 chunks stays whole (a piece of half a chunk or
    // less costs more in its partial result and merge than it saves in
    // balance: measured 5% on hetero64's attention); longer units are cut
    // into chunk-sized pieces and a shorter last one.  Either way a unit
    // makes at most ceil(kt / chunk) items, so the bounds above hold.
    auto nsplit = [&](int kt) -> int {
        return 2LL * kt > 3LL * chunk ? (kt + chunk - 1) / chunk : (kt > 0 ? 1 : 0);
    };
    auto len_key = [&](int kt, int k) -> int {
        const int nsk = nsplit(kt);
        int len = nsk == 1 ? kt : kt - k * chunk;
        if (nsk > 1 && len > chunk) len = chunk;
        return len >= kLenBuckets - 1 ? kLenBuckets - 1 : len;
    };
    bucket[threadIdx.x] = 0;
    __syncthreads();
    for (int c = 0; c < n_rounds; ++c) {
        const PlanTile p = tile_of(c);
        const int ns = nsplit(p.kt);
        for (int k = 0; k < ns; ++k) atomicAdd(&bucket[len_key(p.kr, k)], per_tile);
    }
    __syncthreads();
    {
        const int rev = kLenBuckets - 1 - threadIdx.x;   // descending length order
        const int cnt = bucket[rev];
        int total_items;
        const int first = wg_excl_scan(cnt, scan_lds, &total_items);
        bucket[rev] = first;
        __syncthreads();
    }

    // A round's pieces are staged in LDS, then their items (a piece's
    // per_tile items are contiguous) and the round's split units are written by
    // consecutive threads to consecutive entries, so the stores coalesce;
    // a round with more pieces than the stage holds writes its items from
    // the owning thread instead.
    __shared__ int4 s_pc[kPlanPieces];   // per piece: first item, kb, ke, slot base (or -1)
    __shared__ int4 s_pt[kPlanPieces];   // per piece: tile, splits of the tile, request, first row
    __shared__ int4 s_tl[kPlanThreads];  // per tile of the round: splits, first slot, first
                                         // split entry, first row
    // the entries a thread writes: split unit / item j of every tpi-th tile or
    // piece from my_tl on (no division per entry)
    const int tpi = per_tile <= kPlanThreads ? kPlanThreads / per_tile : 1;
    const int my_tl = per_tile <= kPlanThreads ? (int)threadIdx.x / per_tile : 0;
    const int my_j = per_tile <= kPlanThreads ? (int)threadIdx.x % per_tile : 0;
    const bool by_lane = per_tile <= kPlanThreads;
    int items_before = 0, slots_before = 0, split_before = 0;
    for (int c = 0; c < n_rounds; ++c) {
        const int t = c * kPlanThreads + threadIdx.x;
        const PlanTile p = tile_of(c);
        const int ns = nsplit(p.kt);
        if (t < n_tiles && p.kt == 0)
            record_error(pv.hdr, pv.tiles[(size_t)t * kTileInts + kTB], FB_DERR_PAGE);
        // items, partial slots and split units of this round's tiles
        int ex[3] = {ns * per_tile, ns > 1 ? ns * per_tile : 0, ns > 1 ? per_tile : 0};
        int tot[3];
        wg_excl_scan3(ex, tot, trio_lds);
        const int slot_t = slots_before + ex[1];     // unit j owns slots slot_t + j*ns ..
        const int split_t = split_before + ex[2];    // and, when split, list entry split_t + j
        const int piece0 = ex[0] / per_tile;         // this tile's first piece in the round
        const int round_pieces = tot[0] / per_tile;
        const bool staged = round_pieces <= kPlanPieces;
        s_tl[threadIdx.x] = make_int4(ns, slot_t, split_t, p.row0);
        if (t < n_tiles) {
            for (int k = 0; k < ns; ++k) {
                const int pos = atomicAdd(&bucket[len_key(p.kr, k)], per_tile);
                const long long kb = (long long)k * chunk * kKeyTile;
                long long ke = k == ns - 1 ? (long long)p.kv : kb + (long long)chunk * kKeyTile;
                if (ke > p.kv) ke = p.kv;
                const int slot_k = ns > 1 ? slot_t + k : -1;
                if (staged) {
                    s_pc[piece0 + k] = make_int4(pos, (int)kb, (int)ke, slot_k);
                    s_pt[piece0 + k] = make_int4(t, ns, p.b, p.row0);
                } else {
                    for (int j = 0; j < per_tile; ++j) {
                        if (pos + j >= item_cap) break;   // cannot happen: the caps hold
                        int4* it = reinterpret_cast<int4*>(ws.items + (size_t)(pos + j) * kIItemInts);
                        it[0] = make_int4(t * per_tile + j, (int)kb, (int)ke,
                                          slot_k < 0 ? -1 : slot_k + j * ns);
                        it[1] = make_int4(p.b, p.row0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();
        int round_tiles = n_tiles - c * kPlanThreads;
        if (round_tiles > kPlanThreads) round_tiles = kPlanThreads;
        auto write_split = [&](int tl, int j) {
            const int4 q = s_tl[tl];
            const int u = (c * kPlanThreads + tl) * per_tile + j;
            if (q.x > 1 && q.z + j < split_cap)
                ws.split[q.z + j] = make_int4(u, q.x, q.y + j * q.x, q.w);
        };
        auto write_item = [&](int pc, int j) {
            const int4 a = s_pc[pc];
            const int4 m = s_pt[pc];
            if (a.x + j >= item_cap) return;   // cannot happen: the caps hold
            int4* it = reinterpret_cast<int4*>(ws.items + (size_t)(a.x + j) * kIItemInts);
            it[0] = make_int4(m.x * per_tile + j, a.y, a.z, a.w < 0 ? -1 : a.w + j * m.y);
            it[1] = make_int4(m.z, m.w, 0, 0);
        };
        if (by_lane) {
            if (my_tl < tpi) {
                for (int tl = my_tl; tl < round_tiles; tl += tpi) write_split(tl, my_j);
                if (staged)
                    for (int pc = my_tl; pc < round_pieces; pc += tpi) write_item(pc, my_j);
            }
        } else {
            for (int e = threadIdx.x; e < round_tiles * per_tile; e += kPlanThreads)
                write_split(e / per_tile, e % per_tile);
            if (staged)
                for (int e = threadIdx.x; e < round_pieces * per_tile; e += kPlanThreads)
                    write_item(e / per_tile, e % per_tile);
        }
        __syncthreads();   // the stage is reused by the next round
        items_before += tot[0];
        slots_before += tot[1];
        split_before += tot[2];
    }
    if (threadIdx.x == 0) {
        ws.counts[kCItems] = items_before < item_cap ? items_before : item_cap;
        ws.counts[kCSplit] = split_before < split_cap ? split_before : split_cap;
    }
}

// ---- the plan of a small pack, made by the attention's own workgroups ----
// plan_kernel takes 7-9 us, nearly all of it latency (a launch, dependent
// reads, barrier rounds), and the attention waits for it.  Up to 64 tiles a
// wave holds the whole pack, one tile per lane, so every wave of the attention
// finds its own item with lane moves only: the read of the tile records takes
// the place of the read of the item record, and no barrier is needed.  Same
// split size, pieces and partial slots as plan_kernel, so outputs are
// bit-identical; the order is longest first in four classes (longer than a
// chunk, a chunk, at least half of one, shorter) instead of by exact length.
// Each workgroup also stores its item where plan_kernel would (and its split
// units, which the merge reads), so the workspace then holds this pack's plan
// as before.  One request's step (3 tiles): 50.8 -> 43.7 us; 8 fp32 requests'
// attention 86 -> 80.  With four tiles per lane (up to 256 tiles, one wave
// planning for its workgroup) it gained nothing: several workgroups in turn
// pay for it on each CU and the coarser order lengthens the tail (24 requests
// of 3 blocks of 96: 62.3 -> 64.2 us; 64 requests of 4 blocks: 127 -> 129).
constexpr int kInlineTiles = 64;

struct PlanArgs {
    int per_tile;          // units of a tile: kv-heads x row groups
    int tile_cap;
    int item_cap, split_cap, target_items, fixed_chunk_tiles;
    long long max_keys;
};

struct Item {
    int u, kb, ke, slot, b, row0;
    int kv_len;            // of the item's tile
};

// Inclusive scan over the wave's lanes by data-parallel moves (a step costs a
// few cycles where a shuffle through the LDS path costs about a hundred):
// within rows of 16, then row ends into the following rows.
template <typename F>
__device__ inline int wave_scan(int x, F f) {
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));   // row_shr:1
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));   // row_shr:2
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));   // row_shr:4
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));   // row_shr:8
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));   // row_bcast:15
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return x;
}

// The item of workgroup `item`; false past the last one.  Whole waves call it
// and get the same scalars.
__device__ inline bool plan_item(const PackView& pv, const AttnWs& ws, const PlanArgs& pa,
                                 const int item, Item& out) {
    const int lane = threadIdx.x & 63;
    // every record of the capacity is read at once with the tile count;
    // those past the count are dropped below
    PlanTile p = plan_tile(pv.tiles, lane, pa.tile_cap, pa.max_keys);
    const int n_tiles = min(pv.hdr[kHdrTiles], pa.tile_cap);
    if (lane >= n_tiles) p.kt = p.kr = 0;
    auto scalar = [](int x, int from) { return __builtin_amdgcn_readlane(x, from); };
    auto add = [](int x, int y) { return x + y; };
    // (32 bits hold the sum: the host checks the capacities)
    const long long total = (long long)scalar(wave_scan(p.kt, add), 63) * pa.per_tile;
    const int kt_max = scalar(wave_scan(p.kt, [](int x, int y) { return max(x, y); }), 63);
    const long long chunk_ll = split_chunk(total, kt_max, pa.target_items, pa.fixed_chunk_tiles);
    if (chunk_ll >= (1 << 30)) {
        if (item == 0 && threadIdx.x == 0) {
            record_error(pv.hdr, pv.tiles[kTB], FB_DERR_PAGE);
            ws.counts[kCItems] = ws.counts[kCSplit] = 0;
        }
        return false;
    }
    const int chunk = (int)chunk_ll;
    // x / chunk for x < 64 chunks (chunk >= kt_max / kMaxSplits): a float
    // quotient is at most one off
    const float rcp = 1.0f / (float)chunk;
    auto over = [&](int x) {
        int q = (int)((float)x * rcp);
        const int r = x - q * chunk;
        return r < 0 ? q - 1 : r >= chunk ? q + 1 : q;
    };

    // The tile's pieces by class: `full` of class 1 (a chunk long) and at most
    // one of another, counted in `cls`.
    //   cls: class 0 in bits 0-9, class 2 in 10-19, class 3 in 20-29
    //   in[1]: class 1 in bits 0-15 (at most 64 x 64), split tiles above
    const int whole_max = (int)(3u * (uint32_t)chunk / 2u);   // a unit up to here stays whole
    const int ns = p.kt > whole_max ? over(p.kt + chunk - 1) : (p.kt > 0 ? 1 : 0);
    int full = 0, cls = 0;
    if (ns > 0) {
        const bool whole = p.kr <= whole_max;
        full = whole ? (p.kr == chunk) : min(ns, over(p.kr));
        if (ns > full) {
            const int len = whole ? p.kr : p.kr - full * chunk;
            cls = len > chunk ? 1 : 2 * len >= chunk ? 1 << 10 : 1 << 20;
        }
    }
    const int in[3] = {cls, full + (ns > 1 ? 1 << 16 : 0), ns > 1 ? ns : 0};
    int at[3], tot[2];   // exclusive prefixes in tile order, totals
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int inc = wave_scan(in[i], add);
        at[i] = inc - in[i];
        if (i < 2) tot[i] = scalar(inc, 63);
    }
    const int n0 = tot[0] & 1023, n1 = tot[1] & 0xffff;
    const int n2 = (tot[0] >> 10) & 1023, n3 = (tot[0] >> 20) & 1023;
    const int n_items = min((n0 + n1 + n2 + n3) * pa.per_tile, pa.item_cap);
    if (item == 0) {
        if (threadIdx.x == 0) {
            ws.counts[kCItems] = n_items;
            ws.counts[kCSplit] = min((tot[1] >> 16) * pa.per_tile, pa.split_cap);
        }
        // tiles past the page table: reported, not planned
        if ((int)threadIdx.x < n_tiles && p.kt == 0) record_error(pv.hdr, p.b, FB_DERR_PAGE);
    }
    if (item >= n_items) return false;
    const int piece = item / pa.per_tile;
    const int j = item - piece * pa.per_tile;

    // the piece's class, its rank in it and the tile that owns it
    int rank = piece, sh = 0;
    bool many = false;   // class 1
    if (rank >= n0) {
        rank -= n0;
        many = rank < n1;
        if (!many) {
            rank -= n1;
            sh = 10;
            if (rank >= n2) {
                rank -= n2;
                sh = 20;
            }
        }
    }
    const int before = many ? at[1] & 0xffff : (at[0] >> sh) & 1023;
    const int have = many ? full : (cls >> sh) & 1023;
    const unsigned long long owners = __ballot(rank >= before && rank < before + have);
    if (owners == 0) return false;   // cannot happen: the ranks cover the items
    const int t = __ffsll(owners) - 1;
    const int k = many ? rank - scalar(before, t) : scalar(full, t);
    const int n = scalar(ns, t);
    const int slot0 = scalar(at[2], t) * pa.per_tile + j * n;   // the unit's first slot
    out.kv_len = scalar(p.kv, t);
    out.b = scalar(p.b, t);
    out.row0 = scalar(p.row0, t);
    out.u = t * pa.per_tile + j;
    out.kb = k * chunk * kKeyTile;
    out.ke = k == n - 1 ? out.kv_len : min(out.kv_len, out.kb + chunk * kKeyTile);
    out.slot = n > 1 ? slot0 + k : -1;
    const int e = (scalar(at[1], t) >> 16) * pa.per_tile + j;   // the unit's entry if split
    if (threadIdx.x == 0) {
        int4* it = reinterpret_cast<int4*>(ws.items + (size_t)item * kIItemInts);
        it[0] = make_int4(out.u, out.kb, out.ke, out.slot);
        it[1] = make_int4(out.b, out.row0, 0, 0);
        if (n > 1 && k == 0 && e < pa.split_cap) ws.split[e] = make_int4(out.u, n, slot0, out.row0);
    }
    return true;
}

// --------------------------------------------------------- bf16 MFMA ------
// S^T accumulator layout of v_mfma_f32_32x32x16_bf16 (32x32 fp32 result):
// lane l holds column l%32 and rows (i/4)*8 + (l/32)*4 + i%4 for i = 0..15.
// Loading K row perm(m) into A-row m, with perm swapping index bits 2 and 3,
// makes lane l's value i belong to tile key 16*(i/8) + 8*(l/32) + i%8, i.e.
// eight consecutive keys per MFMA k-step -- exactly the k-slots the PV
// product needs from P^T, so P moves from the S^T accumulator into the B
// operand of the PV MFMA without any data exchange.
__device__ inline int swap_bits23(int m) {
    return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

__device__ inline float wave_xor32_max(float x) {
    return fmaxf(x, __shfl_xor(x, 32, 64));
}

// K/V staging: a ring of Ring<D>::kStages key tiles in LDS, filled by direct
// global->LDS loads (global_load_lds_dwordx4: lane i of a wave writes 16 bytes
// at M0 + 16*i).  A stage holds the K tile [32 keys][D] followed by the V^T
// tile [D][32 keys], both in 16-byte chunks whose position inside a row is
// XOR-swizzled (K: chunk ^ (key % (D/8)); V^T: chunk ^ ((d/4) % 4)) so that
// the MFMA operand reads of 16 lanes hit 16 distinct bank groups.  The loads
// are issued from inline asm so the compiler neither sees nor waits on them;
// the kernel orders them itself with explicit vmcnt waits and raw barriers.
template <int N, typename F, int... I>
__device__ __attribute__((always_inline)) inline void static_for_impl(F& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
// f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N-1>)
template <int N, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f) {
    static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

template <int D>
struct Ring {
    // Stages of the ring: three workgroups per CU (12 waves, 3 per SIMD)
    // share its 160 KB of LDS -- 3 x 48 KB at D = 128.  The third wave per
    // SIMD hides more of the exp and DMA issue work behind other waves'
    // MFMAs than a fourth ring stage would hide load latency.
    static constexpr int kStages = D == 128 ? 3 : 4;
    static constexpr int kKCh = kKeyTile * D / 8;   // K chunks per stage
    static constexpr int kVCh = D * kKeyTile / 8;   // V^T chunks per stage
    static constexpr int kCh = kKCh + kVCh;
    static constexpr int kStageBytes = kCh * 16;
    static constexpr int kPerThread = kCh / kAttnThreads;   // D / 32
    static_assert(kCh % kAttnThreads == 0, "chunks must divide the workgroup");
};

__device__ inline void dma16(const void* src, uint32_t lds_wave_base) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds_wave_base), "v"(src) : "memory");
}

__device__ inline void barrier_raw() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Wait until at most n of this wave's vector-memory loads are outstanding.
__device__ inline void wait_vm(int n) {
    switch (n) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
        case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
        case 12: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

// FAST: pages hold whole key tiles (page_size >= 32), so a tile's loads share
// one scalar base; otherwise each lane picks its page.  INLINE: the
// workgroups plan for themselves (plan_item) instead of reading plan_kernel's
// items.  FULL: every wave of a workgroup has query rows (a unit's rows come in
// whole 128s); a template, as the test in each step costs the full shapes 1-2%.
template <int D, bool FAST, bool INLINE, bool FULL>
__global__ void __launch_bounds__(kAttnThreads, kWgsPerCu)
attn_bf16_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
                 const uint16_t* __restrict__ v_cache,
                 const int32_t* __restrict__ page_table, PackView pv, AttnWs ws,
                 uint16_t* __restrict__ out, int Hq, int Hkv, int g, int bl, int RG,
                 int ps, int ps_shift, int max_pages, int num_pages, float scale_log2,
                 PlanBounds bounds, PlanArgs pa) {
    using RG_ = Ring<D>;
    constexpr int NS = RG_::kStages;
    __shared__ __attribute__((aligned(16))) unsigned char ring[NS * RG_::kStageBytes];
    constexpr int KK = D / 16;      // k-steps of the S^T product
    constexpr int DT = D / 32;      // 32-wide d tiles of O^T
    constexpr int NCH = RG_::kPerThread;
    constexpr int CPR = D / 8;      // 16-byte chunks per K row
    // A thread's loads j < NK fetch K and the rest V^T, for every wave when
    // the K chunks fill whole loads.  Then (D = 128) K and V^T are refilled
    // separately, K one step ahead (the split ring below).
    constexpr int NK = RG_::kKCh / kAttnThreads;
    constexpr bool SPLIT_RING = NS == 3 && RG_::kKCh % kAttnThreads == 0;

    Item w;
    if constexpr (INLINE) {
        if (!plan_item(pv, ws, pa, blockIdx.x, w)) return;
    } else {
        // The item's record is read together with the item count (the grid has
        // item_cap workgroups, so the record is always inside the buffer).
        const int item = blockIdx.x;
        const int32_t* it = ws.items + (size_t)item * kIItemInts;
        w.u = it[kIUnit], w.kb = it[kIKb], w.ke = it[kIKe], w.slot = it[kISlot];
        w.b = it[kIB], w.row0 = it[kIRow0];
        const int n_items = ws.counts[kCItems];
        // (the empty asm keeps the compiler from sinking the record's loads below
        // the count check, which would serialize the two round trips)
        asm volatile("" :: "s"(w.u), "s"(w.kb), "s"(w.ke), "s"(w.slot), "s"(w.b), "s"(w.row0),
                     "s"(n_items));
        if (item >= n_items) return;
        if ((unsigned)w.u >= (unsigned)bounds.unit_cap || w.kb < 0 ||
            (w.kb & (kKeyTile - 1)) != 0 || w.ke <= w.kb || (long long)w.ke > bounds.max_keys ||
            w.slot < -1 || w.slot >= bounds.slot_cap || (unsigned)w.b >= (unsigned)bounds.n_req ||
            w.row0 < 0 || w.row0 > bounds.row_cap - bl) {
            if (threadIdx.x == 0) record_error(pv.hdr, 0, FB_DERR_PLAN);
            return;
        }
    }
    const int u = w.u, kb = w.kb, ke = w.ke, slot = w.slot, b = w.b, row0 = w.row0;
    const int rg = u % RG;
    const int c = (u / RG) % Hkv;
    const int32_t* pt = page_table + (size_t)b * max_pages;

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int n = lane & 31;
    const int h = lane >> 5;
    const int r_local = wave * 32 + n;
    const int r = rg * kRowsPerWg + r_local;
    const bool row_ok = FULL || r < bl * g;
    // A wave without query rows only loads: its MFMAs and exps would take issue
    // slots from the waves that have some (64 requests, d = 128, 32 rows per
    // unit: 214 -> 172 us; d = 64, 8 rows: 122 -> 85).
    const bool wave_ok = FULL || __builtin_amdgcn_readfirstlane(rg * kRowsPerWg + wave * 32) < bl * g;
    const int pos_local = row_ok ? r / g : 0;
    const int hg = row_ok ? r % g : 0;
    const size_t q_off = ((size_t)(row0 + pos_local) * Hq + c * g + hg) * D;

    // Q fragments, loaded right after the first ring loads are issued so
    // that both latencies overlap (the first wait covers both).
    bf16x8 qf[KK];
    auto load_q = [&]() {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            if (row_ok) qf[kk] = *reinterpret_cast<const bf16x8*>(q + q_off + kk * 16 + h * 8);
            else qf[kk] = bf16x8{};
        }
    };

    // Per-thread chunk geometry, the same for every key tile: byte offset of
    // the chunk inside its page (K: [slot][d], V^T: [d][slot]) and, where a
    // tile spans several pages, which of them holds it.  Each (load j, wave)
    // is all-K or all-V, so the global base can be a wave-uniform scalar pair.
    uint32_t ch_off[NCH];
    int ch_page[NCH];
    bool ch_isk[NCH];
    const int slot_mask = FAST ? kKeyTile - 1 : ps - 1;   // a tile key's slot in its page
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        const int s = j * kAttnThreads + tid;
        if (s < RG_::kKCh) {
            const int key = s / CPR;
            const int dchunk = (s % CPR) ^ (key % CPR);
            ch_isk[j] = true;
            ch_page[j] = FAST ? 0 : key >> ps_shift;
            ch_off[j] = (uint32_t)((key & slot_mask) * D + dchunk * 8) * 2u;
        } else {
            const int s2 = s - RG_::kKCh;
            const int d = s2 >> 2;
            const int kc = (s2 & 3) ^ ((d >> 2) & 3);
            ch_isk[j] = false;
            ch_page[j] = FAST ? 0 : (kc * 8) >> ps_shift;
            ch_off[j] = (uint32_t)(d * ps + ((kc * 8) & slot_mask)) * 2u;
        }
    }
    // Which loads fetch K is wave-uniform; make it scalar so the choice of
    // base pointer is a scalar select, not a divergent branch.
    bool ld_isk[NCH];
#pragma unroll
    for (int j = 0; j < NCH; ++j) ld_isk[j] = __builtin_amdgcn_readfirstlane((int)ch_isk[j]) != 0;
    uint32_t m0_base[NCH];
    const uint32_t ring_base = (uint32_t)(uintptr_t)&ring[0];
#pragma unroll
    for (int j = 0; j < NCH; ++j)
        m0_base[j] = __builtin_amdgcn_readfirstlane(ring_base + j * 4096 + wave * 1024);
    const size_t k_head = (size_t)c * ps * D;        // head c inside a K page
    const size_t v_head = (size_t)c * D * ps;        // head c inside a V page
    const size_t page_elems = (size_t)Hkv * ps * D;  // one page of one cache
    const uint32_t page_bytes = (uint32_t)(page_elems * 2);
    const unsigned char* kb0 = reinterpret_cast<const unsigned char*>(k_cache + k_head);
    const unsigned char* vb0 = reinterpret_cast<const unsigned char*>(v_cache + v_head);

    // Per-lane LDS byte offsets of the MFMA operand reads (stage 0).
    const int krow = swap_bits23(n);
    const int kswz = krow % CPR;
    // chunk (2kk + h) ^ kswz of row krow: the row part and the chunk part
    // occupy disjoint bits, so k-step kk is one XOR away from k-step 0
    const uint32_t kx = (uint32_t)(krow * D + ((h ^ kswz) * 8)) * 2u;
    auto koff = [&](int kk) -> uint32_t { return kx ^ (uint32_t)(kk << 5); };
    // V^T rows d = dt*32 + n share the swizzle of row n ((d/4)%4 does not
    // depend on dt), so d tile dt is a constant offset from d tile 0.
    uint32_t voff0[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
        voff0[tt] = RG_::kKCh * 16 + (uint32_t)(n * kKeyTile + (((tt * 2 + h) ^ ((n >> 2) & 3)) * 8)) * 2u;
    constexpr uint32_t kVdt = 32 * kKeyTile * 2;   // bytes between d tiles of V^T
    auto voff = [&](int dt, int tt) -> uint32_t { return voff0[tt] + dt * kVdt; };

    // Page ids of key tile kt: one where a page holds whole tiles, else those
    // of its kKeyTile / ps pages (at most four; past the item's last key the
    // last page again).  They are scalar loads made a step before the tile is
    // issued, so that their latency is off the path.
    constexpr int NP = FAST ? 1 : 4;
    struct Pages {
        int id[NP];
    };
    const int pg_last = (ke - 1) >> ps_shift;
    auto tile_page = [&](int kt) -> Pages {
        Pages p;
        const int first = (kt * kKeyTile) >> ps_shift;
        p.id[0] = pt[first];
        if constexpr (!FAST) {
#pragma unroll
            for (int i = 1; i < NP; ++i) p.id[i] = pt[min(first + i, pg_last)];
        }
        return p;
    };
    // a bad page id is read as page 0 and recorded once at the end
    bool page_err = false;
    // Issue the loads of key tile kt into stage STAGE.
    // PART 0: the tile's K loads, 1: its V^T loads, 2: both
    auto issue_part = [&](int kt, auto stage_c, Pages pg, auto part_c) __attribute__((always_inline)) {
        constexpr int STAGE = decltype(stage_c)::value;
        constexpr int PART = decltype(part_c)::value;
        constexpr int J0 = PART == 1 ? NK : 0;
        constexpr int J1 = PART == 0 ? NK : NCH;
        const int key0 = kt * kKeyTile;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const bool okp = (unsigned)pg.id[i] < (unsigned)num_pages;
            page_err |= !okp;
            pg.id[i] = okp ? pg.id[i] : 0;
        }
        if (FAST) {
            // one page per tile: uniform base + per-lane constant offsets
            const int page = pg.id[0];
            const uint32_t inpage = (uint32_t)(key0 & (ps - 1));
            const size_t poff = (size_t)(uint32_t)page * (size_t)page_bytes;
            const unsigned char* kbase = kb0 + poff + inpage * (uint32_t)(D * 2);
            const unsigned char* vbase = vb0 + poff + inpage * 2u;
#pragma unroll
            for (int j = J0; j < J1; ++j) {
                const uint32_t m0 = m0_base[j] + STAGE * RG_::kStageBytes;
                // for D >= 64 the K chunks are exactly the first kKCh/256 loads
                const bool isk = (RG_::kKCh % kAttnThreads == 0) ? (j * kAttnThreads < RG_::kKCh)
                                                                 : ld_isk[j];
                const unsigned char* base = isk ? kbase : vbase;
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                             :: "s"(m0), "v"(ch_off[j]), "s"(base) : "memory");
            }
        } else {
            // several pages per tile: the chunk's own page, picked per lane
            // (24 requests of 96-wide blocks over pages of 16, d = 64: the
            // kernel takes 47 us, was 57 with the page ids read when the tile
            // was issued and the address worked out per lane each time)
#pragma unroll
            for (int j = J0; j < J1; ++j) {
                int page = pg.id[0];
#pragma unroll
                for (int i = 1; i < NP; ++i) page = ch_page[j] == i ? pg.id[i] : page;
                const bool isk = (RG_::kKCh % kAttnThreads == 0) ? (j * kAttnThreads < RG_::kKCh)
                                                                 : ld_isk[j];
                const unsigned char* src = (isk ? kb0 : vb0) + ch_off[j] +
                                           (size_t)(uint32_t)page * (size_t)page_bytes;
                const uint32_t m0 = m0_base[j] + STAGE * RG_::kStageBytes;
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                             :: "s"(m0), "v"(src) : "memory");
            }
        }
    };
    auto issue_tile = [&](int kt, auto stage_c, const Pages& page) {
        issue_part(kt, stage_c, page, std::integral_constant<int, 2>{});
    };

    floatx16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = floatx16{};
    float m_run = -INFINITY;   // running max of scores, log2 domain
    float thr_raw = -INFINITY;  // raw score above which the running max moves
    // max over the two lane halves (rows are shared by lanes l and l+32);
    // plain v_max_f32 on values that are never NaN here
    auto half_max = [&](float mx) -> float {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx),
                                                         false, false);
        float r;
        asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(__uint_as_float(sw[0])), "v"(__uint_as_float(sw[1])));
        return r;
    };
    float l_acc[2] = {0.f, 0.f};   // this lane's share of the denominator
    bf16x8 pb[2];              // P^T of the current tile (B operand of PV)

    const int kt0 = kb / kKeyTile;
    const int nt = (ke + kKeyTile - 1) / kKeyTile - kt0;
    const int valid_last = ke - (kt0 + nt - 1) * kKeyTile;   // keys of the last tile below ke
    constexpr int kAhead = KK < 2 ? KK : 2;   // LDS operand reads kept in flight

    // S^T of one key tile (K fragments from stage kst) into acc.
    auto s_mfmas = [&](const unsigned char* kst, floatx16& acc) {
        bf16x8 fr[kAhead];
#pragma unroll
        for (int m = 0; m < kAhead; ++m) fr[m] = *reinterpret_cast<const bf16x8*>(kst + koff(m));
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const bf16x8 a = fr[kk % kAhead];
            if (kk + kAhead < KK)
                fr[kk % kAhead] = *reinterpret_cast<const bf16x8*>(kst + koff(kk + kAhead));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], acc, 0, 0, 0);
        }
    };
    // O^T += V^T P^T of one key tile (V^T fragments from stage vst).
    auto pv_mfmas = [&](const unsigned char* vst) {
        constexpr int NX = DT * 2;
        constexpr int A = NX < 2 ? NX : 2;
        bf16x8 fr[A];
        // product x: d tile x % DT, key half x / DT (consecutive products
        // accumulate into different tiles)
#pragma unroll
        for (int x = 0; x < A; ++x)
            fr[x] = *reinterpret_cast<const bf16x8*>(vst + voff(x % DT, x / DT));
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const bf16x8 a = fr[x % A];
            if (x + A < NX)
                fr[x % A] = *reinterpret_cast<const bf16x8*>(vst + voff((x + A) % DT, (x + A) / DT));
            o[x % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[x / DT], o[x % DT], 0, 0, 0);
        }
    };
    // Row max of a score tile in the log2 domain (both lane halves hold
    // different keys of the same query row).
    auto tile_max = [&](const floatx16& s) -> float {
        float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
        for (int x = 3; x < 16; x += 2) mx = fmaxf(fmaxf(mx, s[x]), x + 1 < 16 ? s[x + 1] : s[x]);
        return half_max(mx) * scale_log2;
    };
    // P^T = exp2(S^T * scale - m) rounded to bf16, and the denominator from
    // the same rounded weights the PV product uses.
    auto softmax_p = [&](const floatx16& s) {
#pragma unroll
        for (int x = 0; x < 16; ++x)
            pb[x >> 3][x & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[x], scale_log2, -m_run));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int x = 0; x < 8; x += 2) {
            const bf16x2 p0 = {pb[0][x], pb[0][x + 1]};
            const bf16x2 p1 = {pb[1][x], pb[1][x + 1]};
            l_acc[0] = __builtin_amdgcn_fdot2_f32_bf16(p0, one2, l_acc[0], false);
            l_acc[1] = __builtin_amdgcn_fdot2_f32_bf16(p1, one2, l_acc[1], false);
        }
    };
    // Scores of keys at or past ke (only in the last tile) become -inf.
    auto mask_tail = [&](floatx16& s) {
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const int key = 16 * (x >> 3) + 8 * h + (x & 7);
            if (key >= valid_last) s[x] = -INFINITY;
        }
    };
    // Lazy rescale: move the running max only when a row's tile max passes
    // it by more than the slack; O and the denominator follow.
    // mx is a raw row max (not scaled); rescale when it passes thr_raw
    auto update_max = [&](float mx) {
        const bool need = mx > thr_raw;
        if (__any(need)) {
            const float m_new = need ? mx * scale_log2 : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int x = 0; x < 16; ++x) o[dt][x] *= alpha;
            l_acc[0] *= alpha;
            l_acc[1] *= alpha;
            m_run = m_new;
            thr_raw = (m_run + kRescaleSlack) / scale_log2;
        }
    };

    // Phase 1 of a step: S^T of the next tile (K fragments from kst) on the
    // matrix core, while the VALU turns the current tile's scores into P^T.
    // Each group holds one MFMA and a share of the VALU work; scheduling
    // barriers between groups keep that interleave.
    auto phase1 = [&](const unsigned char* kst, const floatx16& sc, floatx16& acc) {
        constexpr int SPG = 16 / KK;   // scores per group
        static_assert(SPG % 2 == 0, "scores go in pairs");
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
        bf16x8 fr[kAhead];
#pragma unroll
        for (int m = 0; m < kAhead; ++m) fr[m] = *reinterpret_cast<const bf16x8*>(kst + koff(m));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const bf16x8 a = fr[kk % kAhead];
            if (kk + kAhead < KK)
                fr[kk % kAhead] = *reinterpret_cast<const bf16x8*>(kst + koff(kk + kAhead));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], acc, 0, 0, 0);
#pragma unroll
            for (int y = 0; y < SPG; y += 2) {
                const int x = kk * SPG + y;
                const __bf16 p0 = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[x], scale_log2, -m_run));
                const __bf16 p1 = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[x + 1], scale_log2, -m_run));
                pb[x >> 3][x & 7] = p0;
                pb[x >> 3][(x & 7) + 1] = p1;
                const bf16x2 pp = {p0, p1};
                l_acc[x >> 3] = __builtin_amdgcn_fdot2_f32_bf16(pp, one2, l_acc[x >> 3], false);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Phase 2: O^T += V^T P^T of the current tile (V^T fragments from vst)
    // while the VALU takes the row max of the next tile's scores.
    auto phase2 = [&](const unsigned char* vst, const floatx16& sn) -> float {
        constexpr int NX = DT * 2;
        constexpr int A = NX < 2 ? NX : 2;
        constexpr int VPG = 16 / NX;   // scores per group
        bf16x8 fr[A];
#pragma unroll
        for (int x = 0; x < A; ++x)
            fr[x] = *reinterpret_cast<const bf16x8*>(vst + voff(x % DT, x / DT));
        float mx = -INFINITY;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const bf16x8 a = fr[x % A];
            if (x + A < NX)
                fr[x % A] = *reinterpret_cast<const bf16x8*>(vst + voff((x + A) % DT, (x + A) / DT));
            o[x % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[x / DT], o[x % DT], 0, 0, 0);
#pragma unroll
            for (int y = 0; y < VPG; ++y) mx = fmaxf(mx, sn[x * VPG + y]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return half_max(mx);
    };

    // Software pipeline over key tiles, one step per tile i < nt-1:
    //   wait for tile i+1 and barrier; refill the stage of tile i-1 (read by
    //   every wave before this barrier) with tile i+NS-1 (the split ring
    //   below waits and refills per half instead);
    //   phase 1: S^T(i+1) on the matrix core while the VALU turns S^T(i)
    //            into P^T(i);
    //   phase 2: O^T += V^T(i) P^T(i) while the VALU takes the row max of
    //            S^T(i+1);
    //   then the (rare) rescale for tile i+1.
    // Stages in use: i (V), i+1 (K), i+2 .. i+NS-1 in flight.
    static_assert(NS >= 3, "the ring needs the current, next and one loading stage");
    floatx16 s_cur = floatx16{};
    Pages pg_next{};
    if (!SPLIT_RING && NS - 1 < nt) pg_next = tile_page(kt0 + NS - 1);
    // KIND 0: a step with a refill and the steady-state wait (no runtime
    // checks); 1: a step near the end; 2: the step that brings in the last
    // tile (which may be partial).
    auto step = [&](int i, auto stage_c, auto kind_c) {
        constexpr int STAGE = decltype(stage_c)::value;
        constexpr int KIND = decltype(kind_c)::value;
        constexpr int NXT = (STAGE + 1) % NS;
        constexpr int FREE = (STAGE + NS - 1) % NS;
        if constexpr (KIND == 0) {
            wait_vm((NS - 3) * NCH);
            barrier_raw();
            issue_tile(kt0 + i + NS - 1, std::integral_constant<int, FREE>{}, pg_next);
            const int nx = i + NS < nt ? i + NS : nt - 1;   // clamped: no branch
            pg_next = tile_page(kt0 + nx);
        } else {
            int behind = nt - 2 - i;            // tiles issued after tile i+1
            if (behind > NS - 3) behind = NS - 3;
            wait_vm(behind * NCH);
            barrier_raw();
            if (i + NS - 1 < nt) {
                issue_tile(kt0 + i + NS - 1, std::integral_constant<int, FREE>{}, pg_next);
                if (i + NS < nt) pg_next = tile_page(kt0 + i + NS);
            }
        }
        const unsigned char* kst = ring + NXT * RG_::kStageBytes;
        const unsigned char* vst = ring + STAGE * RG_::kStageBytes;   // V^T offsets include the K part

        if (!wave_ok) return;
        floatx16 s_nxt = floatx16{};
        phase1(kst, s_cur, s_nxt);
        if constexpr (KIND == 2) {
            if (valid_last < kKeyTile) mask_tail(s_nxt);
        }
        const float mx = phase2(vst, s_nxt);
        update_max(mx);
        s_cur = s_nxt;
    };

    // The split ring (D = 128, three stages).  K(t) and V^T(t) still share
    // stage t % 3, but the K half is free a step before the V^T half (the
    // scores of tile t are taken in step t-1, its PV product in step t), so
    // step i refills them separately: K(i+3) into the K half of tile i's
    // stage and V^T(i+2) into the V^T half of tile i-1's.  Both then arrive
    // two steps before use (one for K when a tile's halves move together),
    // and step i waits only for what it reads -- K(i+1) and V^T(i), loaded
    // in step i-2 -- while the loads of step i-1 stay in flight.
    // KIND 0: both refills, no runtime checks; 1: a step near the end
    // (K(i+3) may not exist); 2: step nt-2, which takes the last tile's
    // scores and leaves only V^T(nt-1) in flight.
    Pages pg_k{}, pg_v{};   // page ids of the next K and V^T tiles to load
    auto step_split = [&](int i, auto stage_c, auto kind_c) __attribute__((always_inline)) {
        constexpr int STAGE = decltype(stage_c)::value;
        constexpr int KIND = decltype(kind_c)::value;
        constexpr int NXT = (STAGE + 1) % NS;
        constexpr int FREE = (STAGE + NS - 1) % NS;
        using KPart = std::integral_constant<int, 0>;
        using VPart = std::integral_constant<int, 1>;
        // step i-1 loaded K(i+2) (when i+2 < nt, true but in the last step)
        // and V^T(i+1)
        wait_vm(KIND == 2 ? NCH - NK : NCH);
        barrier_raw();
        if constexpr (KIND != 2) {
            if (KIND == 0 || i + 3 < nt) issue_part(kt0 + i + 3, stage_c, pg_k, KPart{});
            issue_part(kt0 + i + 2, std::integral_constant<int, FREE>{}, pg_v, VPart{});
            pg_v = pg_k;
            const int nx = i + 4 < nt ? i + 4 : nt - 1;   // clamped: no branch
            pg_k = tile_page(kt0 + nx);
        }
        const unsigned char* kst = ring + NXT * RG_::kStageBytes;
        const unsigned char* vst = ring + STAGE * RG_::kStageBytes;
        if (!wave_ok) return;
        floatx16 s_nxt = floatx16{};
        phase1(kst, s_cur, s_nxt);
        if constexpr (KIND == 2) {
            if (valid_last < kKeyTile) mask_tail(s_nxt);
        }
        const float mx = phase2(vst, s_nxt);
        update_max(mx);
        s_cur = s_nxt;
    };

    if constexpr (SPLIT_RING) if (nt > 0) {
        using C0 = std::integral_constant<int, 0>;
        using C1 = std::integral_constant<int, 1>;
        using C2 = std::integral_constant<int, 2>;
        using KPart = std::integral_constant<int, 0>;
        using VPart = std::integral_constant<int, 1>;
        const Pages p0 = tile_page(kt0);
        const Pages p1 = nt > 1 ? tile_page(kt0 + 1) : Pages{};
        const Pages p2 = nt > 2 ? tile_page(kt0 + 2) : Pages{};
        // K(0), K(1), V^T(0), then Q.  The explicit wait is for K(0) alone
        // (it does not count on Q's loads, which a wave without valid rows
        // skips); Q is waited for where it is used, and as loads complete in
        // order that wait covers K(1) and V^T(0) too.
        issue_part(kt0, C0{}, p0, KPart{});
        if (nt > 1) issue_part(kt0 + 1, C1{}, p1, KPart{});
        issue_part(kt0, C0{}, p0, VPart{});
        load_q();
        wait_vm(nt > 1 ? NCH : NCH - NK);
        barrier_raw();
        s_mfmas(ring, s_cur);
        // the loads "step -1" makes: K(2) and V^T(1)
        if (nt > 2) issue_part(kt0 + 2, C2{}, p2, KPart{});
        if (nt > 1) issue_part(kt0 + 1, C1{}, p1, VPart{});
        pg_v = p2;
        pg_k = nt > 3 ? tile_page(kt0 + 3) : p2;
        if (nt == 1 && valid_last < kKeyTile) mask_tail(s_cur);
        m_run = tile_max(s_cur);
        thr_raw = (m_run + kRescaleSlack) / scale_log2;
        using Full = std::integral_constant<int, 0>;
        using Near = std::integral_constant<int, 1>;
        using Last = std::integral_constant<int, 2>;
        // steps 0 .. nt-4 make both refills; the tail steps check (one
        // runtime-checked kind keeps the register pressure of the loop down)
        const int n_full = nt - 3 > 0 ? nt - 3 : 0;
        int i0 = 0;
        for (; i0 + NS <= n_full; i0 += NS) {
            static_for<NS>([&](auto j) { step_split(i0 + j, j, Full{}); });
        }
        for (; i0 < nt - 2; i0 += NS) {
            static_for<NS>([&](auto j) {
                if (i0 + j < nt - 2) step_split(i0 + j, j, Near{});
            });
        }
        if (nt >= 2) {
            const int st = (nt - 2) % NS;
            static_for<NS>([&](auto j) {
                if (st == j) step_split(nt - 2, j, Last{});
            });
        }
        // V^T of the last tile
        wait_vm(0);
        barrier_raw();
    }
    if (nt > 0) {
        if constexpr (!SPLIT_RING) {
            Pages pg0[NS - 1];   // page ids of the first tiles, all requested before any load
            static_for<NS - 1>([&](auto j) { pg0[j] = j < nt ? tile_page(kt0 + j) : Pages{}; });
            static_for<NS - 1>([&](auto j) {
                if (j < nt) issue_tile(kt0 + j, j, pg0[j]);
            });
            load_q();
            wait_vm((nt - 1 < NS - 2 ? nt - 1 : NS - 2) * NCH);
            barrier_raw();
            s_mfmas(ring, s_cur);
            if (nt == 1 && valid_last < kKeyTile) mask_tail(s_cur);
            m_run = tile_max(s_cur);
            thr_raw = (m_run + kRescaleSlack) / scale_log2;
            using Full = std::integral_constant<int, 0>;
            using Near = std::integral_constant<int, 1>;
            using Last = std::integral_constant<int, 2>;
            // steps 0 .. n_full-1 refill the ring (and, as NS >= 3, are not the last)
            const int n_full = nt - NS + 1 > 0 ? nt - NS + 1 : 0;
            int i0 = 0;
            for (; i0 + NS <= n_full; i0 += NS) {
                static_for<NS>([&](auto j) { step(i0 + j, j, Full{}); });
            }
            for (; i0 < nt - 2; i0 += NS) {
                static_for<NS>([&](auto j) {
                    if (i0 + j < nt - 2) step(i0 + j, j, Near{});
                });
            }
            // the step that brings in the last tile (which may be partial)
            if (nt >= 2) {
                const int st2 = (nt - 2) % NS;
                static_for<NS>([&](auto j) {
                    if (st2 == j) step(nt - 2, j, Last{});
                });
            }
        }
        // last tile: P^T, then its PV product
        softmax_p(s_cur);
        const int last_stage = (nt - 1) % NS;
        unsigned char* slast = ring + last_stage * RG_::kStageBytes;
        if (valid_last < kKeyTile) {
            // V^T columns of keys past ke may hold anything (even NaN); zero
            // them so their 0-weight products stay 0.  One 16-byte chunk (8
            // keys of one d) per thread and pass.
            unsigned char* vlds = slast + RG_::kKCh * 16;
#pragma unroll 1
            for (int e = tid; e < D * (kKeyTile / 8); e += kAttnThreads) {
                const int d = e >> 2, kc = e & 3;
                const int first = valid_last - kc * 8;   // keys >= first are past ke
                if (first >= 8) continue;
                uint4* p = reinterpret_cast<uint4*>(vlds + (d * kKeyTile + ((kc ^ ((d >> 2) & 3)) * 8)) * 2);
                if (first <= 0) {
                    *p = make_uint4(0, 0, 0, 0);
                } else {
                    const uint4 v = *p;
                    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (k >= first) w[k >> 1] &= (k & 1) ? 0x0000ffffu : 0xffff0000u;
                    *p = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
            barrier_raw();
        }
        pv_mfmas(slast);
    }

    if (page_err && tid == 0) record_error(pv.hdr, b, FB_DERR_PAGE);
    float l_part = l_acc[0] + l_acc[1];
    const float l = l_part + __shfl_xor(l_part, 32, 64);
    const float inv_l = 1.0f / l;
    if (slot < 0) {
        if (!row_ok) return;
        uint16_t* orow = out + q_off;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const int d0 = dt * 32 + grp * 8 + h * 4;
                __bf16 v4[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) v4[x] = (__bf16)(o[dt][grp * 4 + x] * inv_l);
                *reinterpret_cast<uint2*>(orow + d0) = *reinterpret_cast<const uint2*>(v4);
            }
        }
    } else {
        if (!row_ok) return;   // the merge reads valid rows only
        float* po = ws.part_o + ((size_t)slot * kRowsPerWg + r_local) * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const int d0 = dt * 32 + grp * 8 + h * 4;
                float4 v4 = make_float4(o[dt][grp * 4 + 0] * inv_l, o[dt][grp * 4 + 1] * inv_l,
                                        o[dt][grp * 4 + 2] * inv_l, o[dt][grp * 4 + 3] * inv_l);
                *reinterpret_cast<float4*>(po + d0) = v4;
            }
        }
        if (h == 0) ws.part_lse[(size_t)slot * kRowsPerWg + r_local] = m_run + __log2f(l);
    }
}

// ------------------------------------------------------------ combine -----
// Four consecutive output elements of one row.
template <typename T>
__device__ inline void store_out4(T* p, const float4& v);
template <>
__device__ inline void store_out4<uint16_t>(uint16_t* p, const float4& v) {
    __bf16 x[4] = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
    *reinterpret_cast<uint2*>(p) = *reinterpret_cast<const uint2*>(x);
}
template <>
__device__ inline void store_out4<float>(float* p, const float4& v) {
    *reinterpret_cast<float4*>(p) = v;
}

// Each split unit's rows are merged by kRowsPerWg / R workgroups of R rows
// (workgroup b takes entry b / parts of the plan's list of split units, so the
// grid covers only units that can be split): a row's per-split log-sum-exp
// weights go to LDS once, then every thread merges 16-byte columns of its
// rows, up to IF splits' loads in flight at a time.
//
// With few units it is bound by the trips to memory that follow one another,
// so a workgroup takes few rows (one column group per thread); with many, by
// the workgroups launched (most find no split unit).  Kernel trace, R = 32 / 16
// / 8: 12 units in nine pieces 8.6 / 6.3 / 5.5 us; 128 (fp32) 9.1 / 8.5 / 10.9;
// 256 15.1 / 14.4 / 19.2; 576 with few split 6.6 / 7.3 / 15.0; 768 with hardly
// any split 5.2 / 5.2 / 8.9.  (768 with a good part split, only R = 32: 10.1.)
template <typename T, int R, int IF>
__global__ void __launch_bounds__(kAttnThreads)
combine_kernel(PackView pv, AttnWs ws, T* __restrict__ out, int Hq, int Hkv,
               int g, int bl, int RG, int D, PlanBounds bounds) {
    constexpr int kParts = kRowsPerWg / R;
    __shared__ float wgt[kMaxSplits][R];
    __shared__ float inv_den[R];
    const int su = blockIdx.x / kParts;
    const int part = blockIdx.x % kParts;
    // the plan's record of this split unit (no further lookups before the
    // loads), read together with the count: the grid stays inside the list
    const int4 rec = ws.split[su];
    const int n_split = ws.counts[kCSplit];
    asm volatile("" :: "s"(rec.x), "s"(rec.y), "s"(rec.z), "s"(rec.w), "s"(n_split));
    if (su >= n_split) return;
    const int u = rec.x;
    const int ns = rec.y;   // 2 .. kMaxSplits (plan)
    if (ns <= 1) return;
    const int slot0 = rec.z;
    const int row0 = rec.w;
    if ((unsigned)u >= (unsigned)bounds.unit_cap || ns > kMaxSplits || slot0 < 0 ||
        slot0 > bounds.slot_cap - ns || row0 < 0 || row0 > bounds.row_cap - bl) {
        if (threadIdx.x == 0) record_error(pv.hdr, 0, FB_DERR_PLAN);
        return;
    }
    const int rg = u % RG;
    const int c = (u / RG) % Hkv;
    const int rbase = part * R;
    const int nrows = min(R, bl * g - rg * kRowsPerWg - rbase);
    if (nrows <= 0) return;
    const int per_row = D / 4;
    const int n_el = nrows * per_row;
    const size_t stride = (size_t)kRowsPerWg * D;   // one split's partial O
    auto src_of = [&](int e) {
        return ws.part_o + ((size_t)slot0 * kRowsPerWg + rbase + e / per_row) * D +
               (e % per_row) * 4;
    };
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    // A row's split weights exp2(lse_k - max) and 1/sum: its log-sum-exps
    // are loaded eight at a time (one round trip for up to eight splits) and
    // kept in LDS until the maximum is known.
    auto weights = [&]() {
        if (threadIdx.x < nrows) {
            const float* lse = ws.part_lse + (size_t)slot0 * kRowsPerWg + rbase + threadIdx.x;
            float mx = -INFINITY;
            for (int k0 = 0; k0 < ns; k0 += 8) {
                float l[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) l[j] = lse[(size_t)min(k0 + j, ns - 1) * kRowsPerWg];
#pragma unroll
                for (int j = 0; j < 8; ++j) mx = fmaxf(mx, l[j]);   // repeats do not move it
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (k0 + j < ns) wgt[k0 + j][threadIdx.x] = l[j];
            }
            const bool skipped = std::is_same<T, float>::value && wgt[0][threadIdx.x] == kSkippedLse;
            float den = 0.f;
            for (int k = 0; k < ns; ++k) {
                const float w = __builtin_amdgcn_exp2f(wgt[k][threadIdx.x] - mx);
                wgt[k][threadIdx.x] = w;
                den += w;
            }
            // fp32: a skipped block's rows stay unwritten (a NaN row is written)
            inv_den[threadIdx.x] = skipped ? -1.0f : 1.0f / den;
        }
        __syncthreads();
    };
    auto store = [&](int e, const float4& acc) {
        const int rr = e / per_row;
        const int d0 = (e % per_row) * 4;
        const float id = inv_den[rr];
        if (std::is_same<T, float>::value && id < 0.f) return;
        const int r = rg * kRowsPerWg + rbase + rr;
        const int pos_local = r / g, hg = r % g;
        T* dst = out + ((size_t)(row0 + pos_local) * Hq + c * g + hg) * D + d0;
        store_out4<T>(dst, make_float4(acc.x * id, acc.y * id, acc.z * id, acc.w * id));
    };
    auto add = [](float4& acc, float w, const f32x4& v) {
        acc.x += w * v[0];
        acc.y += w * v[1];
        acc.z += w * v[2];
        acc.w += w * v[3];
    };
    // Up to kFastSplits splits (the plan's usual few pieces): every load of
    // the thread's column groups (at most kMaxGroups) is issued before the
    // weights are computed, so the workgroup waits for one round trip.
    constexpr int kFastSplits = 4;
    constexpr int kMaxGroups = (R * kMaxHeadDim / 4 + kAttnThreads - 1) / kAttnThreads;
    const int n_grp = (n_el + kAttnThreads - 1) / kAttnThreads;   // workgroup-uniform
    if (ns <= kFastSplits && n_grp <= kMaxGroups) {
        f32x4 v[kMaxGroups][kFastSplits];
#pragma unroll
        for (int m = 0; m < kMaxGroups; ++m) {
            if (m < n_grp) {
                const float* src = src_of(min((int)threadIdx.x + m * kAttnThreads, n_el - 1));
#pragma unroll
                for (int k = 0; k < kFastSplits; ++k)   // past the last split: reload it, unused
                    v[m][k] = *reinterpret_cast<const f32x4*>(src + (size_t)min(k, ns - 1) * stride);
            }
        }
        weights();
#pragma unroll
        for (int m = 0; m < kMaxGroups; ++m) {
            const int e = (int)threadIdx.x + m * kAttnThreads;
            if (m < n_grp && e < n_el) {
                const int rr = e / per_row;
                float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int k = 0; k < kFastSplits; ++k)
                    if (k < ns) add(acc, wgt[k][rr], v[m][k]);
                store(e, acc);
            }
        }
        return;
    }
    // More splits: a thread's first column group has its loads (up to IF)
    // issued before the weights are ready; then IF at a time per group.
    constexpr int kInFlight = IF;
    f32x4 first[kInFlight];
    {
        const float* src = src_of(min((int)threadIdx.x, n_el - 1));
#pragma unroll
        for (int j = 0; j < kInFlight; ++j)   // past the last split: reload it, unused
            first[j] = *reinterpret_cast<const f32x4*>(src + (size_t)min(j, ns - 1) * stride);
#pragma unroll
        for (int j = 0; j < kInFlight; ++j) asm volatile("" :: "v"(first[j]));
    }
    weights();
    for (int e = threadIdx.x; e < n_el; e += kAttnThreads) {
        const int rr = e / per_row;
        const float* src = src_of(e);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k0 = 0; k0 < ns; k0 += kInFlight) {
            f32x4 v[kInFlight];
            if (k0 == 0 && e == (int)threadIdx.x) {
#pragma unroll
                for (int j = 0; j < kInFlight; ++j) v[j] = first[j];
            } else {
#pragma unroll
                for (int j = 0; j < kInFlight; ++j)
                    v[j] = *reinterpret_cast<const f32x4*>(
                        src + (size_t)min(k0 + j, ns - 1) * stride);
            }
#pragma unroll
            for (int j = 0; j < kInFlight; ++j)
                if (k0 + j < ns) add(acc, wgt[k0 + j][rr], v[j]);
        }
        store(e, acc);
    }
}

// ---------------------------------------------------------------- fp32 ----
// The same work items in fp32 on v_mfma_f32_32x32x2_f32: 4 waves x 32 query
// rows, 32-key K and V^T tiles in two LDS buffers filled by direct
// global->LDS loads.  A tile is D MFMAs of 64 cycles per wave, so the matrix
// core is the bound by far: one tile of lead covers the loads, and two
// workgroups per CU (64 KB of LDS each at D = 128) cover the softmax.
//
// Operands.  MFMA A/B lane l carries k-slot l/32, and a dot product does not
// care which k goes into which slot: lane half h reads four consecutive d
// (chunk 2j + h) in one 16-byte LDS read and feeds them to four MFMAs.  The
// accumulator layout (rows (i/4)*8 + (l/32)*4 + i%4) then makes S^T value i
// the P^T operand of the PV MFMA whose V^T operand is key chunk 2(i/4) + h,
// element i%4: P never moves between lanes, and V^T is read the same way.
//
// DIRECT: one workgroup per unit over all its keys, no plan and no merge (for
// caches too short to be worth splitting).  INLINE as in the bf16 kernel.
//
// Measured (8 requests of 256-2048 prefix keys, 16/4 heads, d = 128: 6.4
// GFLOP, 41 us at the nominal 157 TFLOP/s): the whole call, kernel and merge,
// takes 68-96 us by the lengths, against 15-16 ms for one key per lane on the
// vector units with K rows read a lane apart.
template <int D>
struct F32Tile {
    static constexpr int kCpr = D / 4;                      // 16-byte chunks of a K row
    static constexpr int kKCh = kKeyTile * kCpr;            // chunks of a K tile
    static constexpr int kVCh = D * kKeyTile / 4;           // chunks of a V^T tile
    static constexpr int kBytes = (kKCh + kVCh) * 16;       // one buffer
    static constexpr int kLoads = kKCh / kAttnThreads;      // per thread: K, and as many V^T
    static_assert(kKCh % kAttnThreads == 0 && kVCh == kKCh, "whole loads per workgroup");
    // position of chunk c in row r: the 16 rows of one read hit 16 bank groups
    __device__ static inline int kpos(int r, int c) { return c ^ (D == 32 ? (r >> 1) & 7 : r & 15); }
    __device__ static inline int vpos(int d, int c) { return c ^ ((d >> 1) & 7); }
};

__device__ inline void dma4(const void* src, uint32_t lds_wave_base) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(lds_wave_base), "v"(src) : "memory");
}

template <int D, bool DIRECT, bool INLINE>
__global__ void __launch_bounds__(kAttnThreads, 2)
attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ k_cache,
                const float* __restrict__ v_cache, const int32_t* __restrict__ page_table,
                PackView pv, AttnWs ws, float* __restrict__ out, int Hq, int Hkv, int g, int bl,
                int RG, int ps, int ps_shift, int max_pages, int num_pages, float scale_log2,
                PlanBounds bounds, PlanArgs pa) {
    using T = F32Tile<D>;
    constexpr int NL = T::kLoads;
    constexpr int DT = D / 32;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) unsigned char buf[2 * T::kBytes];

    Item w;
    if constexpr (!DIRECT && INLINE) {
        if (!plan_item(pv, ws, pa, blockIdx.x, w)) return;
    } else {
        if (DIRECT) {
            w.u = blockIdx.x;
            if (w.u >= pv.hdr[kHdrTiles] * Hkv * RG) return;
        } else {
            const int32_t* it = ws.items + (size_t)blockIdx.x * kIItemInts;
            w.u = it[kIUnit], w.kb = it[kIKb], w.ke = it[kIKe], w.slot = it[kISlot];
            if ((int)blockIdx.x >= ws.counts[kCItems]) return;
            if ((unsigned)w.u >= (unsigned)bounds.unit_cap || w.kb < 0 ||
                (w.kb & (kKeyTile - 1)) != 0 || w.ke <= w.kb ||
                (long long)w.ke > bounds.max_keys || w.slot < -1 || w.slot >= bounds.slot_cap) {
                if (threadIdx.x == 0) record_error(pv.hdr, 0, FB_DERR_PLAN);
                return;
            }
        }
        const int32_t* tile = pv.tiles + (size_t)(w.u / (RG * Hkv)) * kTileInts;
        w.b = tile[kTB];
        w.row0 = tile[kTRow0];
        w.kv_len = tile[kTKvLen];
        if (DIRECT) w.kb = 0, w.ke = w.kv_len, w.slot = -1;
    }
    const int u = w.u, kb = w.kb, ke = w.ke, slot = w.slot, b = w.b, row0 = w.row0;
    const int kv_len = w.kv_len;
    const int rg = u % RG;
    const int c = (u / RG) % Hkv;
    const int32_t* pt = page_table + (size_t)b * max_pages;

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int n = lane & 31;
    const int h = lane >> 5;
    const int r_local = wave * 32 + n;
    const int r = rg * kRowsPerWg + r_local;
    const bool row_ok = r < bl * g;
    const bool wave_ok = rg * kRowsPerWg + wave * 32 < bl * g;   // the wave has query rows

    // Every page the block reads must be valid, else the block is skipped
    // (each of a split block's pieces scans them all and says so to the merge).
    __shared__ int bad_page;
    if (tid == 0) bad_page = 0;
    __syncthreads();
    if ((long long)kv_len > bounds.max_keys) {
        if (tid == 0) bad_page = 1;
    } else {
        const int n_pages = (kv_len + ps - 1) >> ps_shift;
        for (int p = tid; p < n_pages; p += kAttnThreads)
            if ((unsigned)pt[p] >= (unsigned)num_pages) bad_page = 1;
    }
    __syncthreads();
    if (bad_page || ke > kv_len) {
        if (tid == 0) record_error(pv.hdr, b, FB_DERR_PAGE);
        if (slot >= 0 && tid < kRowsPerWg)
            ws.part_lse[(size_t)slot * kRowsPerWg + tid] = kSkippedLse;
        return;
    }

    const size_t q_off = row_ok ? ((size_t)(row0 + r / g) * Hq + c * g + r % g) * D : 0;
    f32x4 qf[D / 8];   // chunk 2j + h of the lane's query row
#pragma unroll
    for (int j = 0; j < D / 8; ++j)
        qf[j] = row_ok ? *reinterpret_cast<const f32x4*>(q + q_off + (2 * j + h) * 4) : f32x4{};

    // Loads: thread tid's load j fills LDS chunk j*256 + tid of each half of a
    // buffer.  Keys past the item's end are read as its last key (their
    // scores are masked, their V^T zeroed below).  A V^T chunk is four keys of
    // one page; with pages of one or two keys V^T goes key by key instead.
    const int n_tiles = (ke - kb + kKeyTile - 1) / kKeyTile;
    const int vkc = T::vpos(tid >> 3, tid & 7);   // key chunk of the thread's V^T loads
    const bool small_pages = ps < 4;
    auto page_of = [&](int key) { return pt[min(key, ke - 1) >> ps_shift]; };
    int pg_k[NL], pg_v = 0;
    auto load_pages = [&](int i) {
        const int key0 = kb + i * kKeyTile;
#pragma unroll
        for (int j = 0; j < NL; ++j) pg_k[j] = page_of(key0 + (j * kAttnThreads + tid) / T::kCpr);
        pg_v = page_of(key0 + vkc * 4);
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)&buf[0];
    auto issue = [&](int i) {
        const int key0 = kb + i * kKeyTile;
        const uint32_t base = lds0 + (i & 1) * T::kBytes;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int s = j * kAttnThreads + tid;
            const int kr = s / T::kCpr;
            const int key = min(key0 + kr, ke - 1);
            const float* src = k_cache +
                (((size_t)pg_k[j] * Hkv + c) * ps + (key & (ps - 1))) * D +
                T::kpos(kr, s % T::kCpr) * 4;
            dma16(src, __builtin_amdgcn_readfirstlane(base + j * 4096 + wave * 1024));
        }
        if (!small_pages) {
            const int key = min(key0 + vkc * 4, (ke - 1) & ~3);
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int d = (j * kAttnThreads + tid) >> 3;
                const float* src = v_cache + (((size_t)pg_v * Hkv + c) * D + d) * ps +
                                   (key & (ps - 1));
                dma16(src, __builtin_amdgcn_readfirstlane(base + T::kKCh * 16 + j * 4096 +
                                                          wave * 1024));
            }
        } else {
            for (int j = 0; j < NL * 4; ++j) {
                const int s = j * kAttnThreads + tid;        // float of the V^T half
                const int d = s >> 5;
                const int key = min(key0 + T::vpos(d, (s >> 2) & 7) * 4 + (s & 3), ke - 1);
                const float* src = v_cache + (((size_t)page_of(key) * Hkv + c) * D + d) * ps +
                                   (key & (ps - 1));
                dma4(src, __builtin_amdgcn_readfirstlane(base + T::kKCh * 16 + j * 1024 +
                                                         wave * 256));
            }
        }
    };

    floatx16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = floatx16{};
    // Running max of the raw scores (may lag by the slack).  Scores are scaled
    // after it is taken off, so that none that is finite overflows; while every
    // score of a row is -inf, 0 stands in for it and the row's sums stay 0.
    float m_run = -INFINITY;
    float l = 0.f;             // this lane half's share of the denominator
    const float slack = fminf(kRescaleSlack / scale_log2, FLT_MAX);

    load_pages(0);
    issue(0);
    if (n_tiles > 1) load_pages(1);
    for (int i = 0; i < n_tiles; ++i) {
        // tile i has landed and every wave is done with tile i - 1's buffer
        wait_vm(0);
        barrier_raw();
        if (i + 1 < n_tiles) {
            issue(i + 1);
            if (i + 2 < n_tiles) load_pages(i + 2);
        }
        if (!wave_ok) continue;
        const unsigned char* kt = buf + (i & 1) * T::kBytes;
        const unsigned char* vt = kt + T::kKCh * 16;
        const int valid = ke - kb - i * kKeyTile;   // keys of the tile below ke

        floatx16 s = floatx16{};
#pragma unroll
        for (int j = 0; j < D / 8; ++j) {
            const f32x4 kf = *reinterpret_cast<const f32x4*>(
                kt + (n * T::kCpr + T::kpos(n, 2 * j + h)) * 16);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[x], qf[j][x], s, 0, 0, 0);
        }
        if (valid < kKeyTile) {
#pragma unroll
            for (int x = 0; x < 16; ++x)
                if ((x >> 2) * 8 + h * 4 + (x & 3) >= valid) s[x] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int x = 1; x < 16; ++x) mx = fmaxf(mx, s[x]);
        mx = wave_xor32_max(mx);
        // rescale only when a row's max passes the running one by the slack
        if (__any(mx > m_run + slack)) {
            const float m_new = fmaxf(mx, m_run);
            const float alpha = m_run == -INFINITY
                ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int x = 0; x < 16; ++x) o[dt][x] *= alpha;
            l *= alpha;
            m_run = m_new;
        }
        const float m_ref = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
        for (int x = 0; x < 16; ++x)
            s[x] = __builtin_amdgcn_exp2f((s[x] - m_ref) * scale_log2);
        float t[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) t[x] = s[x] + s[x + 8];
        l += ((t[0] + t[4]) + (t[1] + t[5])) + ((t[2] + t[6]) + (t[3] + t[7]));
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            f32x4 vf[DT];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const int d = dt * 32 + n;
                vf[dt] = *reinterpret_cast<const f32x4*>(
                    vt + (d * (kKeyTile / 4) + T::vpos(d, grp * 2 + h)) * 16);
            }
            if (valid < kKeyTile) {
                // slots past ke may hold anything (even NaN)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (grp * 8 + h * 4 + x >= valid)
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt) vf[dt][x] = 0.f;
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
                    o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[dt][x], s[grp * 4 + x], o[dt],
                                                                0, 0, 0);
        }
    }
    if (!wave_ok) return;

    l += __shfl_xor(l, 32, 64);
    // a piece whose scores are all -inf weighs nothing in the merge
    const float inv_l = slot >= 0 && l == 0.f ? 0.f : 1.0f / l;
    if (slot < 0 && !row_ok) return;
    float* dst = slot < 0 ? out + q_off
                          : ws.part_o + ((size_t)slot * kRowsPerWg + r_local) * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const float4 v4 = make_float4(o[dt][grp * 4 + 0] * inv_l, o[dt][grp * 4 + 1] * inv_l,
                                          o[dt][grp * 4 + 2] * inv_l, o[dt][grp * 4 + 3] * inv_l);
            *reinterpret_cast<float4*>(dst + dt * 32 + grp * 8 + h * 4) = v4;
        }
    if (slot >= 0 && h == 0) {
        float lse = fmaf(m_run, scale_log2, __log2f(l));
        if (l > 0.f) lse = fminf(fmaxf(lse, -FLT_MAX), FLT_MAX);   // kSkippedLse is not a row's
        ws.part_lse[(size_t)slot * kRowsPerWg + r_local] = lse;
    }
}

}  // namespace

// fp32 caches too short to be worth a plan and a merge: the key tiles of the
// longest block a request can reach, walked by one workgroup.
static bool f32_direct(const fb_attn_shape* sh) {
    return (long long)sh->max_pages * sh->page_size * sh->head_dim <= kF32DirectWork;
}

AttnPlanSizes attention_sizes(const fb_pack* pack, const fb_attn_shape* sh,
                              int cu_count) {
    AttnPlanSizes z{};
    const int g = sh->Hq / sh->Hkv;
    z.rows_per_unit = pack->bl * g;
    z.row_groups = (z.rows_per_unit + kRowsPerWg - 1) / kRowsPerWg;
    z.unit_cap = pack->tile_cap * sh->Hkv * z.row_groups;
    // One item per workgroup the chip holds at once at D = 128 (kWgsPerCu per
    // CU in bf16, kF32WgsPerCu in fp32): more splits cost more in partial
    // writes, the merge and per-item start-up than they win in balance
    // (measured in bf16 at D = 128: 8 per CU was 2-25% slower).  Smaller heads
    // aim at the same number, though a CU holds more of them at once (by
    // registers and LDS: bf16 four at 64 and five at 32, fp32 three and four).
    const bool f32 = sh->dtype == FB_F32;
    z.target_items = (f32 ? kF32WgsPerCu : kWgsPerCu) * (cu_count > 0 ? cu_count : 256);
    z.item_cap = z.unit_cap + z.target_items;
    z.slot_cap = 2 * z.target_items;
    z.split_cap = z.target_items;   // a split unit holds at least two of the slots
    const size_t D = sh->head_dim;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off += (bytes + 255) & ~(size_t)255;
        return at;
    };
    z.off_items = take((size_t)z.item_cap * kIItemInts * sizeof(int32_t));
    z.off_counts = take(kCountInts * sizeof(int32_t));
    z.off_split = take((size_t)z.split_cap * sizeof(int4));
    if (!f32 || !f32_direct(sh)) {
        z.off_part_o = take((size_t)z.slot_cap * kRowsPerWg * D * sizeof(float));
        z.off_part_lse = take((size_t)z.slot_cap * kRowsPerWg * sizeof(float));
    } else {
        z.off_part_o = z.off_part_lse = off;
    }
    z.total = off;
    return z;
}

namespace {

AttnWs ws_view(void* wsp, const AttnPlanSizes& z) {
    char* base = static_cast<char*>(wsp);
    return AttnWs{reinterpret_cast<int32_t*>(base + z.off_items),
                  reinterpret_cast<int32_t*>(base + z.off_counts),
                  reinterpret_cast<int4*>(base + z.off_split),
                  reinterpret_cast<float*>(base + z.off_part_o),
                  reinterpret_cast<float*>(base + z.off_part_lse)};
}

}  // namespace

static void launch_plan(const fb_pack* pack, const fb_attn_shape* sh, const AttnWs& ws,
                        const AttnPlanSizes& z, hipStream_t stream) {
    const int fixed_chunk = sh->kv_split > 0 ? sh->kv_split / kKeyTile : 0;
    const long long max_keys = (long long)sh->max_pages * sh->page_size;
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, stream, pack_view(pack), ws,
                       sh->Hkv, z.row_groups, z.item_cap, z.split_cap, z.target_items,
                       fixed_chunk, max_keys);
}

hipError_t launch_attention_plan(const fb_pack* pack, const fb_attn_shape* sh, void* wsp,
                                 const AttnPlanSizes& z, hipStream_t stream) {
    if (sh->dtype == FB_F32) return hipSuccess;   // fp32 plans inside the attention call
    launch_plan(pack, sh, ws_view(wsp, z), z, stream);
    return hipGetLastError();
}

hipError_t launch_attention(const void* q, const void* k_cache,
                            const void* v_cache, const int32_t* page_table,
                            const fb_pack* pack, const fb_attn_shape* sh,
                            void* out, void* wsp, const AttnPlanSizes& z,
                            hipStream_t stream, bool planned) {
    PackView pv = pack_view(pack);
    const int g = sh->Hq / sh->Hkv;
    const float scale = sh->sm_scale > 0.f ? sh->sm_scale
                                           : 1.0f / sqrtf((float)sh->head_dim);
    const AttnWs ws = ws_view(wsp, z);
    const PlanBounds bounds{pack->B, pack->row_cap, z.unit_cap, z.slot_cap,
                            (long long)sh->max_pages * sh->page_size};
    int shift = 0;
    while ((1 << shift) < sh->page_size) ++shift;
    const float scale_log2 = scale * kLog2e;
    // Whether the workgroups plan for themselves: a pack that one wave holds
    // and whose key tiles 32 bits can sum.
    const bool inline_plan = !planned && pack->tile_cap <= kInlineTiles &&
        pack->tile_cap * (bounds.max_keys / kKeyTile + 1) < (1LL << 31);
    const PlanArgs pa{sh->Hkv * z.row_groups, pack->tile_cap, z.item_cap, z.split_cap,
                      z.target_items, sh->kv_split > 0 ? sh->kv_split / kKeyTile : 0,
                      bounds.max_keys};
    auto combine = [&](auto elt) {
        using T = decltype(elt);
        const int units = z.split_cap < z.unit_cap ? z.split_cap : z.unit_cap;
        auto go = [&](auto kernel, int rows) {
            hipLaunchKernelGGL(kernel, dim3(units * (kRowsPerWg / rows)), dim3(kAttnThreads), 0,
                               stream, pv, ws, static_cast<T*>(out), sh->Hq, sh->Hkv, g, pack->bl,
                               z.row_groups, sh->head_dim, bounds);
        };
        // the lines lie between the sizes measured at combine_kernel
        if (units <= 64) go(combine_kernel<T, 8, 16>, 8);
        else if (units <= 256) go(combine_kernel<T, 16, 8>, 16);
        else go(combine_kernel<T, 32, 8>, 32);
    };
    if (sh->dtype == FB_F32) {
        const bool direct = f32_direct(sh);
        if (!direct && !inline_plan) launch_plan(pack, sh, ws, z, stream);
        auto launch = [&](auto kernel, int grid) {
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(kAttnThreads), 0, stream,
                               static_cast<const float*>(q), static_cast<const float*>(k_cache),
                               static_cast<const float*>(v_cache), page_table, pv, ws,
                               static_cast<float*>(out), sh->Hq, sh->Hkv, g, pack->bl,
                               z.row_groups, sh->page_size, shift, sh->max_pages, sh->num_pages,
                               scale_log2, bounds, pa);
        };
        auto of_dim = [&](auto d_c) {
            constexpr int D = decltype(d_c)::value;
            if (direct) launch(attn_f32_kernel<D, true, false>, z.unit_cap);
            else if (inline_plan) launch(attn_f32_kernel<D, false, true>, z.item_cap);
            else launch(attn_f32_kernel<D, false, false>, z.item_cap);
        };
        if (sh->head_dim == 32) of_dim(std::integral_constant<int, 32>{});
        else if (sh->head_dim == 64) of_dim(std::integral_constant<int, 64>{});
        else of_dim(std::integral_constant<int, 128>{});
        if (!direct) combine(float());
        return hipGetLastError();
    }
    if (!planned && !inline_plan) launch_plan(pack, sh, ws, z, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint16_t* qb = static_cast<const uint16_t*>(q);
    const uint16_t* kc = static_cast<const uint16_t*>(k_cache);
    const uint16_t* vc = static_cast<const uint16_t*>(v_cache);
    uint16_t* ob = static_cast<uint16_t*>(out);
    const bool fast = sh->page_size >= kKeyTile;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(z.item_cap), dim3(kAttnThreads), 0, stream, qb, kc, vc,
                           page_table, pv, ws, ob, sh->Hq, sh->Hkv, g, pack->bl, z.row_groups,
                           sh->page_size, shift, sh->max_pages, sh->num_pages, scale_log2, bounds, pa);
    };
    auto of_dim = [&](auto d_c) {
        constexpr int D = decltype(d_c)::value;
        auto of_plan = [&](auto inline_c, auto full_c) {
            constexpr bool I = decltype(inline_c)::value, F = decltype(full_c)::value;
            if (fast) launch(attn_bf16_kernel<D, true, I, F>);
            else launch(attn_bf16_kernel<D, false, I, F>);
        };
        const bool full = z.rows_per_unit % kRowsPerWg == 0;
        if (inline_plan && full) of_plan(std::true_type{}, std::true_type{});
        else if (inline_plan) of_plan(std::true_type{}, std::false_type{});
        else if (full) of_plan(std::false_type{}, std::true_type{});
        else of_plan(std::false_type{}, std::false_type{});
    };
    if (sh->head_dim == 32) of_dim(std::integral_constant<int, 32>{});
    else if (sh->head_dim == 64) of_dim(std::integral_constant<int, 64>{});
    else of_dim(std::integral_constant<int, 128>{});
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    combine(uint16_t());
    return hipGetLastError();
}

}  // namespace fb
