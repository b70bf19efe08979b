// Internal layout definitions shared by the host API and the HIP kernels.
//
// Packed tile layout.  All matrices the hot kernels stream (per-cluster slabs,
// the whole-W copy, the centroids) are stored as 1 KiB tiles of 16 "items"
// (candidate tokens, or centroids) x 32 k-values, in the operand order of
// v_mfma_f32_16x16x32_f16: lane l of a wavefront owns item (l % 16) and the 8
// consecutive k-values starting at (l / 16) * 8, stored as 16 contiguous bytes
// at byte l * 16 of the tile.  The tiles of one group of 16 items follow each
// other along k (KT = d_pad / 32 tiles), so a group is one contiguous run of
// KT KiB, and consecutive groups are contiguous too: a wavefront that streams
// a range of items reads one linear range of memory, 1 KiB per load.
#pragma once
#include <stdint.h>

#define VP_TILE_ITEMS 16
#define VP_TILE_K 32
#define VP_TILE_BYTES 1024
#define VP_KPAD 256            // d is padded (with zeros) to a multiple of this
#define VP_WG_THREADS 256      // projection kernel: 4 wavefronts per workgroup
#define VP_WG_WAVES 4
#define VP_ROWS_PER_ITEM 16    // rows one work item projects (one MFMA row tile)
#define VP_BOUND_SETS 8          // per row: sets of its candidates whose best logits bound the k-th best (GEMM-shaped kernels)
#define VP_MAX_ROWS_PER_ITEM 64  // four row tiles: the GEMM-shaped kernel of single-bucket projections
#define VP_GEMV_MAX_ROWS 4
#define VP_RAW_TILES 2           // slab items of at most this many tiles per wavefront keep raw logits, no top-k lists
#define VP_XCD_BLOCK_ITEMS 32    // clustered plans with heavy buckets: consecutive items one XCD takes at a time

// A workspace begins with the header, the rows' bounds `floors` and the rows' sets.  Where they lie matters to the atomics that hundreds
// of workgroups send there at once.  The bounds start 128 bytes behind a multiple of 256: sixteen rows are 64 bytes of one line (32 bytes
// into a line 33 rows took 45.9 us where they take 39.2: full projection, V = 98,000, d = 768, top-2), and the 64 rows of an item are not
// in one block of 256 bytes, which one L2 channel serves alone (64 rows, V = 65,000, d = 1024, top-3: 48.9 us in one, 43.5 in two).
// A row's sets are 32 bytes of one line (N * 4 bytes behind a line's start 60 rows took 68 us, not 63), from a line's start on.
#define VP_FLOORS_AT 128
static inline __host__ __device__ long long vp_rows_head_bytes(int N) { return 256 + ((4ll * N * (1 + VP_BOUND_SETS) + 255) & ~255ll); }
static inline __host__ __device__ long long vp_set_bounds_at(int N)   // bytes behind the floors
{
    return (vp_rows_head_bytes(N) - VP_FLOORS_AT - 4ll * VP_BOUND_SETS * N) & ~127ll;
}
static inline __host__ __device__ unsigned int *vp_set_bounds(unsigned int *floors, int N) { return floors + vp_set_bounds_at(N) / 4; }

// One unit of projection work: some rows of one bucket (up to 16, or 32, 48 or 64 on the kernels with that many row
// slots) against a range of candidate tiles of that bucket's slab.
struct VpItem {
    int32_t cluster;     // slab set entry (cluster id; 0 for the full-vocabulary set, -1 where it is masked)
    int32_t perm_start;  // first position in perm[] of this item's rows
    int32_t nrows;       // 1 .. row slots of the kernel that takes it
    int32_t tile0;       // first candidate tile, counted within the entry's slab
    int32_t ntiles;      // candidate tiles of this item (split among the 4 wavefronts)
    int32_t shared;      // 1 if other items (further row groups of the bucket) read the same tiles
    int32_t tile_off;    // first tile of the entry's slab within the slab set (copy of tile_off[cluster])
    int32_t ncand;       // candidates of the entry (copy of n_cand[cluster])
};

// Where the merge kernel finds everything about the row at one position of
// the bucket order: its partial results sit in row slots slot0, slot0 + slot_stride, ...
// (nit of them) of the call's partial results.
struct VpRowPlan {
    int32_t row;        // row number in the caller's batch
    int32_t cluster;
    int32_t slot0;
    int32_t slot_stride;
    int32_t nit;
    int32_t ids_off;    // first entry of the cluster's token-id list; < 0: candidate positions are token ids
    int32_t pad[2];
};

// Header the planning kernel leaves for the projection and merge kernels.
struct VpPlanHeader {
    int32_t total_items;
    int32_t tiles_per_wave;
    int32_t overflow;        // set if the item list did not fit (never expected)
    int32_t total_tiles;
    // Workgroup -> item swizzle.  > 1: a single bucket whose row groups share tiles (the
    // full-vocabulary projection, masked or not): the number of row groups, with swz_chunks candidate
    // ranges.  The kernels of 16 and 32 rows and the split-k one deal whole ranges to the XCDs; the
    // rows-in-LDS kernel takes it as a mere sign and splits the item list evenly.
    // < 0: a clustered plan with buckets of many row groups: -(items per block), blocks of
    // consecutive items are dealt to the 8 XCDs in turn and every XCD starts at another place
    // of the list (see item_of_workgroup).  0: none.
    int32_t swz_rgs;
    int32_t swz_chunks;
    int32_t rows_per_item;   // row slots per item in the partial results (16, or 32 with two row tiles)
    int32_t mode;            // 0: per-cluster slabs; 1: masked full projection; 2: some clusters by the one, the others by the other
    // modes 1 and 2: the many-row kernel's items (from masked_item0 in the item list: first those that mask the full
    // projection, then those of crowded clusters' slabs) and the first row slot of their partial results;
    // mode 1 repeats the counts above
    int32_t masked_items;
    int32_t masked_item0;
    int32_t masked_slot0;
    int32_t masked_swz;
    int32_t grouped_items;
    int32_t pad[19];
};
static_assert(sizeof(VpPlanHeader) <= VP_FLOORS_AT, "the rows' bounds lie behind the header");

// State of one batch-union projection (see union.hip).
struct VpUnionHeader {
    int32_t n_occ;     // occupied clusters
    int32_t n_union;   // |U|
    int32_t tiles;     // candidate groups of 16 in the union slab
    int32_t pad[61];
};

// A set of packed slabs: the K clusters, or the single whole-vocabulary slab.
struct VpSlabSet {
    const void *tiles;        // packed fp16 tiles of all entries back to back
    const float *bias;        // fp32 bias per candidate, padded to 16 per entry
    const int32_t *ids;       // token id per candidate (-1 in padding); NULL = identity
    const int32_t *tile_off;  // [entries + 1] cumulative candidate tiles
    const int32_t *n_cand;    // [entries] candidates per entry
    int32_t entries;
    int32_t kt;               // k-tiles per candidate group (d_pad / 32)
};

// Tiles per wavefront for a projection of total_tiles candidate tiles (counted once
// per row group): about target_items items when there is plenty of work; with little
// work, fewer and longer items (at least ~4 tiles per wavefront while that still
// leaves min_items items, one per resident workgroup slot), because a short item
// spends most of its life staging rows and waiting for its first loads.
static inline __host__ __device__ int vp_tiles_per_wave(long long total_tiles, int target_items, int min_items)
{
    long long eff = total_tiles / (4 * VP_WG_WAVES);
    if (eff < min_items) eff = min_items;
    if (eff > target_items) eff = target_items;
    if (eff < 1) eff = 1;
    const long long per = (long long)VP_WG_WAVES * eff;
    const long long tpw = (total_tiles + per - 1) / per;
    return (int)(tpw > 1 ? tpw : 1);
}

// Items of a single-bucket plan for the kernel that keeps an item's rows in LDS and runs one
// workgroup per compute unit (`slots` at a time): row groups x candidate ranges as close below a
// multiple of the slots as up to eight rounds allow, so that no round is left nearly empty (86 row
// groups on 256 slots: three ranges each would be 258 items, a second round for two of them; 23
// ranges are 7.7 rounds).  At least one range per row group.
static inline __host__ __device__ int vp_rounds_item_count(int rgs, int slots, int vtiles)
{
    if (slots < 1) slots = 1;
    int best = rgs;
    double best_fill = 0.0;
    for (int rounds = 1; rounds <= 8; ++rounds) {
        int ranges = rounds * slots / rgs;   // (slots are at most 2^20)
        if (ranges > vtiles) ranges = vtiles;
        if (ranges < 1) continue;
        const int items = rgs * ranges;
        const int full = (items + slots - 1) / slots * slots;
        const double fill = (double)items / (double)full;
        if (fill > best_fill + 1e-9) {
            best_fill = fill;
            best = items;
        }
        if (fill > 0.97) break;
    }
    return best;
}

// The same with 16 row groups and more, where it matters which items run side by side.  An XCD walks its eighth of the
// item list (vp_item_of_workgroup_even), the row groups of a range one behind the other, and its workgroups read the range
// from one L2 only while they stay within a few steps of each other.  They do where every XCD has ranges of its own
// (their number a multiple of eight); ranges that straddle XCDs cost 3 to 6 %, and over long ranges that several XCDs
// share the workgroups drift apart until most of them read W through the memory side.  Full projection, top-4, V = 250,000,
// us with the rule above -> with eight ranges or a multiple: d = 1024, N = 4,096: 2,849 -> 1,764, 8,192: 4,986 -> 3,494,
// 12,000: 7,131 -> 5,143, 16,384: 7,571 -> 6,946; d = 1536, N = 3,000: 4,398 -> 2,252, 6,000: 8,115 -> 4,438; d = 512,
// 4,096: 1,220 -> 984.  Which multiple follows from how full it leaves an XCD's last round (N = 4,096, d = 1536, 86 row
// groups: 8, 16 and 24 ranges fill 0.90 of their rounds, 3,400 to 3,547 us, 32 fill 0.98, 3,098 us) and from the 40
// candidate groups or so that another round of shorter items costs (18 row groups, d = 1024: 14 ranges, one round, 535 us,
// 56 ranges 571).  Long shared ranges weigh 1.5, the geometric mean of the ratios above.  Ranges of up to 64 MB are short enough to be shared (8,192 rows, V = 60,000: two 882 us, eight 924).
static inline __host__ __device__ int vp_swept_item_count(int rgs, int slots, int vtiles, int kt, int max_items)
{
    const int whole = vp_rounds_item_count(rgs, slots, vtiles);
    if (rgs < 16) return whole;
    const int per_xcd = slots / 8 > 0 ? slots / 8 : 1;
    int best = whole;
    float best_cost = 0.f;
    for (int m = 0; m <= 8; ++m) {
        const int ranges = m == 0 ? whole / rgs : 8 * m;
        if (m > 0 && (ranges > vtiles || (long long)rgs * ranges > max_items)) break;
        const int len = (vtiles + ranges - 1) / ranges;
        const int rounds = ((rgs * ranges + 7) / 8 + per_xcd - 1) / per_xcd;
        float cost = (float)rounds * (float)(len + 40);
        if (ranges % 8 != 0) cost *= rgs > per_xcd && ranges < 8 && (long long)len * kt > 64 * 1024 ? 1.5f : 1.03f;
        if (m == 0 || cost < best_cost) {
            best_cost = cost;
            best = rgs * ranges;
        }
    }
    return best;
}

// The same for the clustered plan, which also knows its number of (bucket, row group) units:
// every unit ends with a partly filled item, so the plan has at most total / (4 tpw) + units
// items.  When that lies between one and two times the resident workgroup slots (min_items),
// the second round of workgroups would leave most of the chip idle (measured: 63 % against
// 72 % of the HBM peak at 1.4 rounds), so the items are made just long enough for one round.
static inline __host__ __device__ int vp_tiles_per_wave_units(long long total_tiles, int units, int target_items,
                                                              int min_items)
{
    const int tpw = vp_tiles_per_wave(total_tiles, target_items, min_items);
    const long long per = (long long)VP_WG_WAVES * tpw;
    const long long items_ub = (total_tiles + per - 1) / per + units;
    if (items_ub <= min_items || items_ub > 2LL * min_items || 2 * units >= min_items) return tpw;
    const long long room = (long long)VP_WG_WAVES * (min_items - units);
    const long long one_round = (total_tiles + room - 1) / room;
    return (int)(one_round > tpw ? one_round : tpw);
}

// Candidate groups per step of the many-row kernel (project_gemm_lds.hip; eight wavefronts) for an item of ntiles groups: four; one
// or two in short items, where steps of four leave wavefronts without work, or all of them with one step, whose folds then run at
// the same time behind the last load.  Every step pays for a fold, and lists of more than one entry for their upkeep.
// One against four, time in steps of four / of one by groups per item, full projection: d = 1024, top-1, one row group: 4: 1.15, 8: 1.03,
// 15: 1.10, 20: 1.04, 28: 1.04, and four row groups alike.  Lists of a few entries, several row groups (whose workgroups wait for the
// same bytes): d = 1024, four of them, top-4: 4: 1.30, 8: 1.27, 12: 1.03, 20: 0.97, 28: 0.90; top-8: 1.46, 1.30, 1.05, 0.93, 0.83; two
// of them, top-2: 1.22, 1.11, 0.94, 0.96, 0.92; d = 256 and 512 alike (at 28, top-8: 0.85, 0.80).  One row group, top-4, 24 rows: d =
// 1024: 12: 1.03, 15: 1.04, 20: 1.05, 28: 1.05; d = 768: 1.00, 0.95, 1.03, 1.03; d = 512: 0.94, 1.01, 0.93, 0.97; d = 256: 0.94, 0.88, 0.91,
// 0.88.  d = 1280 and 1536: 8: 1.11, 1.10, 12: 0.97, 0.99, beyond 16 0.98 at top-8.
// Two, where one row group alone reads the bytes; the call, all row slots in use, us in steps of four -> two by groups per item.
// Top-1: d = 256: 32: 31.6 -> 28.2, 64: 39.4 -> 36.9; 512: 48: 50.6 -> 47.8, 64: 62.3 -> 59.7; 768: 32: 49.2 -> 47.9; 1024: 32: 62.9 -> 60.6, 48: 85.4 ->
// 81.1, 64: 102.3 -> 98.3; 1280: 16: 41.5 -> 41.6 (24 rows 5 % slower; of one 39.4), 20: 49.5 -> 48.2, 32: 67.5 -> 66.3; 1536: 16: 49.1 -> 47.5, 32: 83.9 -> 80.0.
// Top-3: d = 256: 12: 26.2 -> 24.7, 16: 27.1 -> 26.4, 24: 30.0 -> 33.8, 28: 31.2 -> 36.4, 32: 37.2 -> 40.4; 512: 12: 29.5 -> 28.5, 16: 35.2 -> 32.6, 24:
// 38.1 -> 39.4, 32: 48.7 -> 53.3; 768: 32: 53.4 -> 56.2; 1024: 32: 66.8 -> 66.7, 40: 76.0 -> 71.3, 48: 89.5 -> 83.7, 64: 106.6 -> 104.5; 1280: 16: 45.5 ->
// 44.7, 20: 52.5 -> 51.8, 24: 58.2 -> 59.3, 32: 71.7 -> 72.4; 1536: 16: 52.4 -> 50.0, 24: 66.8 -> 66.4, 32: 86.9 -> 85.1, 36: 90.5 -> 91.4; longer lists alike.
// trades: items of a kernel that trades the bests of sets (vp_trades_sets): at d = 256 and 512 two as well for 32 groups, two steps for
// every wavefront with the trade between them (top-6 43.5 -> 40.3, 55.9 -> 50.6).
static inline __host__ __device__ constexpr int vp_step_groups(int kt, int k, bool shared, int ntiles, bool trades)
{
    if (k == 1) {
        if (ntiles < (kt <= 32 ? 32 : kt == 40 && !shared ? 20 : 16)) return 1;
        return !shared && ntiles <= 64 ? 2 : 4;
    }
    if (shared) return ntiles <= (k > 2 ? 12 : 8) ? 1 : 4;
    if (ntiles <= (kt > 32 ? 15 : kt >= 24 ? 31 : 8)) return 1;
    if (trades && kt <= 16 && ntiles > 28 && ntiles <= 32) return 2;
    return ntiles <= (kt <= 16 ? 16 : kt == 24 ? 0 : kt == 32 ? 64 : kt == 40 ? 20 : 32) ? 2 : 4;
}

// Whether the items of the many-row kernel trade the bests of sets of candidates before the first list entry (project_gemm_lds.hip), for N
// rows in one bucket, `slots` to an item, cut into items of ntiles candidate groups.  Of an item: most of its row slots in use (every
// atomic waits for those of all items of the row: 17 rows, V = 128,000, top-3: 60 us, 64 with the trade) and 24 items or more
// a row (below, from 1,024 rows on, there is little to learn).
static inline __host__ __device__ constexpr bool vp_item_trades_sets(int nrows, int slots, int ntiles, int ncand)
{
    return 4 * nrows >= 3 * slots && (long long)ntiles * (VP_TILE_ITEMS * 24) <= ncand;
}
// Of a call: top-4 to top-8 (fewer entries cost few insertions, more than eight sets do not bound).  Full projection, us without -> with it:
// Several row groups (their workgroups run side by side and the trade's wait is hidden): d = 256, V = 100,000, 256 rows: top-4 43.4 -> 37.5,
// top-7 51.8 -> 43.3; V = 250,000, 384 rows: 85.4 -> 77.7, 104.3 -> 89.6; d = 512, V = 250,000, 192 rows: 80.1 -> 70.3, 93.0 -> 76.1; d = 1024, V =
// 100,000, 256 rows (items of 100 groups): 76.5 -> 73.0, 84.8 -> 76.8, 192 rows: 71.2 -> 61.8, 78.6 -> 67.1.  Two row groups at top-4 and top-5: d =
// 1024 0 to 5 % slower, masked 0 to 9 %; with few rows in the second, d = 1024, V = 212,000, top-6: 65 rows 6 % slower, 96 4 %, 112 4 % faster.  d = 1280 and 1536: top-4 0 to 4 % slower, top-7 and top-8 1 to
// 6 % faster (288 rows, V = 100,000, d = 1280, top-7: 105 -> 100) but for two row groups of 36 groups an item (4 % slower).
// One row group (HBM sets the pace, and the wait shows unless the bound is worth a step of every wavefront): top-7 and top-8 up to d_pad = 512
// and at 1024 (d = 256, top-8, 48 groups an item: 51.8 -> 46.5; 512: 62.8 -> 59.8; 1024: 91.1 -> 87.1); shorter lists only where every
// wavefront has two steps or nearly (d = 1024, 32 groups, top-4: 69.3 -> 65.0, 36: 68.6 -> 70.4; d = 512, 64 groups: 71.9 -> 67.9, 36: 50.0 ->
// 52.1; d = 256, 36: 38.4 -> 40.6); d = 1536 from there on (48 groups, top-4 115.5 -> 113.7, top-8 119.4 -> 115.3; 16 groups, top-4 5 % slower); not
// at d_pad = 768 (36 groups: top-4 58.0 -> 63.0, top-8 63.7 -> 67.1, masked 8 to 14 % slower), nor at 1280 (36 groups: 78.4 -> 82.6, 82.8 -> 85.4)
// but for top-7 and top-8 in steps of two.
static inline bool vp_trades_sets(int kt, int k, int N, int slots, int ntiles, int ncand)
{
    const int rgs = (N + slots - 1) / slots, groups = vp_step_groups(kt, k, rgs > 1, ntiles, true);
    if (k < 4 || k > VP_BOUND_SETS || groups == 1 || !vp_item_trades_sets(rgs > 1 ? slots : N, slots, ntiles, ncand)) return false;
    if (rgs > 1) return kt > 32 ? rgs > 2 && k > 6 : rgs > 2 || (k > 5 && (kt < 32 || vp_item_trades_sets(N - slots, slots, ntiles, ncand)));
    const int steps = (ntiles + groups - 1) / groups;
    if (kt == 48) return steps > 12;
    if (kt == 40) return k > 6 && groups == 2;
    return kt != 24 && (k > 6 || (steps > 12 && steps <= 16 && (kt >= 16 || groups == 2)));
}

// The workgroup -> item maps behind VpPlanHeader.swz_rgs (wg = the workgroup's index in the grid;
// workgroups are handed to the 8 XCDs in turn).  Every item in [0, total_items) is taken by exactly
// one workgroup of a grid that is large enough (total_items + 8 blocks for the first map, the chunk
// count rounded up to 8 times the row groups for the second); the others get -1.
static inline __host__ __device__ int vp_item_of_workgroup(int wg, int total_items, int swz_rgs, int swz_chunks)
{
    const int xcd = wg & 7;
    if (swz_rgs < 0) {
        const int B = -swz_rgs;          // items per block
        const int l = wg >> 3;           // this XCD's l-th workgroup
        // Every XCD starts an eighth of the list further on (and wraps round), so that the
        // workgroups in flight at any time come from eight places of the list: a heavy bucket's
        // items, served by the L2, then overlap with items that stream from HBM on the other XCDs
        // instead of forming a phase of their own on the whole chip (skewed workload: 70 -> 77 %
        // of the HBM peak; most of it from this overlap, blocks of 8 to 32 items do equally well).
        const int nbx = ((total_items + B - 1) / B + 7) >> 3;   // blocks per XCD
        int i = l / B;
        if (i >= nbx) return -1;
        i = (i + xcd * ((nbx + 7) >> 3)) % nbx;
        const int it = (i * 8 + xcd) * B + l % B;
        return it < total_items ? it : -1;
    }
    if (swz_rgs > 1) {
        const int t = wg >> 3;
        const int chl = t / swz_rgs;
        const int ch = chl * 8 + xcd;
        if (ch >= swz_chunks) return -1;
        return ch * swz_rgs + (t - chl * swz_rgs);
    }
    return wg;
}

// The same for the kernel that runs one workgroup per compute unit (rows in LDS), where a plan fills
// whole rounds of the chip: every XCD takes an eighth of the item list, one item more or less.
// Dealing whole candidate ranges instead leaves XCDs with more items than compute units whenever the
// ranges do not divide by eight - 6 row groups x 42 ranges are 252 items for 256 compute units, but 36 for
// two of the XCDs and their 32 compute units, a second round for four workgroups (333 rows of
// d = 1000, V = 150,001: 208 us in the kernel, 129 us with this map).  The row groups of
// a range still follow each other on one XCD, but for the ranges at the seven seams, which two XCDs read.
static inline __host__ __device__ int vp_item_of_workgroup_even(int wg, int total_items)
{
    const int per = (total_items + 7) / 8;
    const int l = wg >> 3;
    const int it = (wg & 7) * per + l;
    return l < per && it < total_items ? it : -1;
}

// What the masked full projection needs besides the slab set: each row's cluster
// and the per-cluster membership bit lists over the vocabulary.
struct VpMaskInfo {
    const int32_t *g;          // [N] cluster of each row (NULL: no masking)
    const uint32_t *bitmaps;   // [K][words]
    int32_t words;             // 32-bit words per cluster
};

// Machine constants of the planner's cost model (bytes per second).
struct VpCostModel {
    float bw_slab;   // slabs streamed once from HBM
    float bw_full;   // one pass over the packed W from HBM
    float bw_l2;     // further passes over tiles already in the L2 (16-row items)
    float bw_gemm;   // further passes over W by the 48- / 64-row items of the GEMM-shaped kernel (rows in LDS)
    float bw_gemm_split;   // the same for the split-k kernel (k-extents beyond d_pad = 1536, k > 32)
    float bw_gather; // batch-union form: columns of U gathered from the packed W into the union slab
    float t_gather;  // ... and the fixed time of the kernels only that gather needs (seconds)
    float t_row_slab;  // the option (seconds); in the model of a call the slabs' time per row beyond the bytes
    // what else the forms of a call cost (vp_cost_of_call; seconds)
    float t_list;      // slabs: per row and item that the row is in
    float t_slab;      // slabs
    float t_masked;    // masked full projection
    float t_masked_row, t_masked_group;   // ... per row, and per row group
    float t_second;    // a second form in one plan
    float t_mixed;     // ... and if that masks some of the rows
};

// Cost model of the planner, the same on the host, which leaves out what cannot win, and in the planning kernel.  Slabs: the
// occupied slabs are streamed once from HBM, further row groups of a bucket re-read them through the L2.  Masked full
// projection with 48- or 64-row items: one pass over W from HBM, or the matrix cores' time for all row groups, whichever
// is longer (W is then served by the L2; the rate of the matrix cores is expressed in bytes of W per second), and 1.25 %
// for every entry of the lists.  With 16-row items every row group re-reads W through the L2, and the lists cost more (every
// lane of every wavefront is busy there).  Tile counts are in candidate groups, the rates of a call in groups per second.
// What the forms cost beyond that is fitted to 2,098 calls of 2 to 1,300 clusters, lists of 10 to 40,000 tokens, 17 to 8,192
// rows, d = 256 to 1,536, top-1 to top-16, each timed on the slabs, masked and as planned.  Slabs: 0.25 ns per row and k-tile
// (staging); every item a row is in builds a list, 0.4 ns per entry (512 rows, 32 lists of 2,000, d = 512, top-4: 1,484 items 58 us, cut
// into 756 38 us), 1.2 us per entry for the chain of an item; no lists for top-1 or where raw logits are kept.  Masked: starts and
// ends 6 us later, 0.25 us per row group, 1.6 ns per row and entry, 0.6 us per entry for the chain.  A second form in one plan: 12 us
// and 1.1 us per entry, 28 us more where it masks.  With 60 ns for every row on the slabs (up to the 512th, an eighth of that beyond) and nothing else,
// and 40 us for a second form, the planner's choice took 1.084 times the fastest form's time (geometric mean, up to top-8; 2 at
// most: 817 rows, 12 short lists, d = 768: 68 us masked, 35 on the slabs), with these 1.018.
static inline __host__ __device__ VpCostModel vp_cost_of_call(VpCostModel m, int k, int kt, bool raw)
{
    const float tile_bytes = (float)kt * VP_TILE_BYTES, lists = k > 1 && !raw ? (float)k : 0.f;
    m.bw_slab /= tile_bytes;
    m.bw_full /= tile_bytes;
    m.bw_l2 /= tile_bytes;
    m.bw_gemm /= tile_bytes;
    m.bw_gemm_split /= tile_bytes;
    const float per_ns = m.t_row_slab * (1.f / 60.f);   // (the option's default is 60 ns: 1 ns)
    m.t_row_slab = 0.25f * kt * per_ns;
    m.t_list = 0.4f * lists * per_ns;
    m.t_slab = 1.2e-6f * lists;
    m.t_masked = 6e-6f + 0.6e-6f * (k > 1 ? k : 0);
    m.t_masked_row = 1.6e-9f * k;
    m.t_masked_group = 0.25e-6f;
    m.t_second = 12e-6f + 1.1e-6f * (k > 1 ? k : 0);
    m.t_mixed = 28e-6f;
    return m;
}
// the matrix cores' rate over many row groups against the rate of the few that the choice between the two whole forms turns
// on (N = 512 -> 4,096 masked rows: 14.1 -> 17.5 TB/s of W at d = 1024, 10 -> 15 at d = 512, 16.8 -> 18.9 at d = 1536)
#define VP_MIX_GEMM 1.3f
static inline __host__ __device__ float vp_lists_factor(int k) { return 1.f + k * 0.0125f; }
// list_items: every row times the items its bucket is cut into
static inline __host__ __device__ float vp_time_slabs(float occ_tiles, float total_tiles, float list_items, int N, const VpCostModel &cost)
{
    return occ_tiles / cost.bw_slab + (total_tiles - occ_tiles) / cost.bw_l2 + list_items * cost.t_list + N * cost.t_row_slab + cost.t_slab;
}
// gemm: the matrix cores' rate (48- and 64-row items); without t_masked
static inline __host__ __device__ float vp_time_masked_rows(int N, int rpi, int vtiles, int k, float gemm, const VpCostModel &cost)
{
    const float rgs = (float)((N + rpi - 1) / rpi), one_pass = vtiles / cost.bw_full;
    const float passes = rgs * (vtiles / (rpi >= 48 ? gemm : cost.bw_l2));
    return (passes > one_pass ? passes : one_pass) * (rpi >= 48 ? vp_lists_factor(k) : 1.f + k * 0.125f) +
           rgs * cost.t_masked_group + N * cost.t_masked_row;
}
// What the many-row kernel saves on crowded clusters if all rows are in one, of that many candidate groups in items of tpi.
static inline __host__ __device__ float vp_grouping_saves(int N, int rpi, float tiles, int tpi, int k, const VpCostModel &cost)
{
    return (float)((N + VP_ROWS_PER_ITEM - 1) / VP_ROWS_PER_ITEM) * tiles / cost.bw_l2 + N * ((int)(tiles / tpi) + 1) * cost.t_list -
           (float)((N + rpi - 1) / rpi) * tiles / (cost.bw_gemm * VP_MIX_GEMM) * vp_lists_factor(k);
}

#define VP_GROUP_ROUNDS 2   // grouped items of such a plan aimed at: rounds of the many-row kernel's workgroups
// What a plan that chooses the form per cluster may do and has to fit.
struct VpMixLimits {
    int32_t mask;         // some of the clusters may be masked
    int32_t group;        // crowded clusters' slabs may go to the many-row kernel
    int32_t kt;           // k-tiles of a candidate group
    int32_t slots;        // workgroups of the many-row kernel that run at a time (0: no such plan)
    int32_t grid;         // its workgroups (a multiple of 8)
    int32_t list;         // records of the item list
    int64_t row_slots;    // row slots of the partial results
};

// Eq. 2 for many rows: how many centroid tiles a wavefront takes at a time (centroid_kernel), and whether it takes two row tiles.
// A round of 256 workgroups of a form takes, d = 1024 (U = k-tiles fetched together): 1 row tile x 1 centroid tile 6.7 us, x 2 7.6,
// x 4 9.7, x 8 14.4; 2 x 4 13.7, 2 x 8 18.5 (4 x 4 22.3, never the best); more workgroups take in proportion longer, fewer no
// shorter.  So the form whose workgroups x time is least.  The kernel in a trace of calls, us, 1 x 1 throughout -> with it, 1,000
// centroids: d = 1024, 256 rows (1 x 1 either way) 7.8 -> 7.9, 512: 13.6 -> 9.4, 1,024: 21.6 -> 12.4, 2,048: 39.3 -> 17.1, 4,096: 73.9 -> 22.2;
// d = 512: 512 rows 7.8 -> 6.3, 4,096: 39.1 -> 14.4; d = 1536: 512 rows 17.2 -> 12.8, 4,096: 107.5 -> 29.6; 500 centroids, d = 1536, 4,096 rows: 56.6
// -> 21.5.  Of 220 sizes (d = 512 to 1536, 100 to 2,000 centroids, 65 to 4,096 rows) none is slower beyond what two traces of one side differ.
static inline int vp_centroid_two_row_tiles(int row_tiles, int parts, int tiles_per_wave)
{
    return tiles_per_wave >= 4 && (long long)((row_tiles + 1) / 2) * parts >= (tiles_per_wave >= 8 ? 200 : 180);
}
static inline int vp_centroid_tiles_per_wave(int row_tiles, int ctiles)
{
    int best = 1;
    float least = 0.f;
    for (int ct = 1; ct <= 8; ct *= 2) {
        const int parts = (ctiles + 4 * ct - 1) / (4 * ct);
        const bool two = vp_centroid_two_row_tiles(row_tiles, parts, ct);
        const float t = ct == 1 ? 6.7f : ct == 2 ? 7.6f : ct == 4 ? (two ? 13.7f : 9.7f) : two ? 18.5f : 14.4f;
        const float wgs = (float)((row_tiles + two) / (1 + two)) * parts;
        const float cost = t * (wgs > 256.f ? wgs * (1.f / 256.f) : 1.f);
        if (ct == 1 || cost < least) {
            least = cost;
            best = ct;
        }
    }
    return best;
}

#define VP_SMALL_ROWS 16   // batches up to this size are planned by the projection workgroups themselves

// What a workgroup of the small-batch projection needs to find its own work (project.hip).
struct VpSmallArgs {
    const int32_t *cpart;       // [N][parts][2] per-part (score bits, index) minima of Eq. 2
    int parts, N, K;
    const int32_t *tile_off;    // per cluster: first candidate tile of its slab
    const int32_t *n_cand;      // per cluster: candidates
    int target_items, min_items;
    int32_t *g;                 // [N] cluster of each row (out)
    int32_t *out_cluster;       // [N] or null
    VpRowPlan *rowplan;         // [N] the merge kernel's records, indexed by row (out)
    VpPlanHeader *hdr;          // (out)
};

// Whether an iteration adds up all members again in place of the `events` (members that came or went: two for every vector
// that moved, so their number needs all 32 bits for the 2^31 - 1 vectors of the largest call).  They have to fit a
// list of n entries, and more of them would read more vectors than there are.
static inline __host__ __device__ bool vp_sums_begin_anew(uint32_t events, int64_t n) { return (int64_t)events > n; }

// Entries that a double adds up exactly whatever their signs: binary16 values are multiples of 2^-24 below 2^16.
#define VP_KM_EXACT_ENTRIES 8192

// What one iteration of the training leaves for the next kernels.
struct VpKmState {
    int32_t changed;        // centroids that are other ones than in the pass before (later passes)
    uint32_t total_events;  // members that came or went, both counted (first pass: all vectors)
    int32_t anew;           // the entries are all members, the sums begin at zero
    int32_t unsettled, settled;   // vectors in VpKmPass.parted from its front and from its end
    int32_t split;          // the last split moved centroids of clusters with members
    int32_t pad[2];
};

// The buffers of a membership pass.
struct VpKmPass {
    int32_t first;          // every vector against every centroid, nothing known before
    int32_t apart;          // rows-in-LDS kernel: passes in which few centroids changed go to its companion
    VpKmState *state;
    void *cp;               // packed centroids, padded to whole groups
    float *cnorm;
    void *cp_changed;       // the changed ones side by side, their norms and numbers
    float *cnorm_changed;
    int32_t *which_changed;
    int32_t *flag;          // [K] centroid changed
    int32_t *assign, *counts;
    int32_t *events, *cursor;   // [K]
    int32_t *prev;          // [n] the cluster in the pass before
    int32_t *rank, *rank_old;   // [n] numbers of the counting atomics (null: not kept)
    float *best;            // [n] score of the vector's cluster: left by every pass of the GEMM-shaped kernels, read by passes over
                            //     the changed centroids only
    const int32_t *order;   // [n] vectors in the order of their first clusters
    int32_t *parted;        // [n] those whose own centroids changed in front
    int32_t *was_split;     // [K] the last split moved the centroid (null: empty clusters are left alone)
};
#define VP_KM_MAX_PIECES 512   // 16-byte pieces of the widest vector

// Size in floats of one partial result: running max, sum of exponentials, then
// k logits and k candidate positions.
static inline __host__ __device__ int vp_partial_floats(int k) { return 2 + 2 * k; }

#define VP_NEG_BIG (-3.0e38f)
#define VP_IDX_NONE 0x7fffffff
#define VP_FLOOR_NONE 0x007fffffu   // order-preserving key of -infinity (float_key in project.hip)
