// Row bucketing by cluster and work planning (one workgroup, all in LDS).
//
// The paper unions the active sets of a batch (section 2.3); here each row is
// instead projected against its own cluster's slab, so rows are first grouped
// by cluster: histogram of the cluster ids -> exclusive prefix scan -> scatter
// of the row numbers into bucket order (or all or some of the clusters are left to the
// masked full projection, where that is cheaper).  The same kernel finishes Eq. 2 (it
// reduces the per-part minima of the centroid kernel) and cuts the projection
// work into items of equal slab bytes: (bucket, group of up to 16 rows, range
// of candidate tiles).  The number of tiles per item adapts to the total work
// so that any batch, from one row to thousands, yields about `target_items`
// items.  The order of rows inside a bucket is the order in which the LDS
// atomics happen to be served; each row's result is independent of its slot.
#include <hip/hip_runtime.h>
#include "vp_kernels.h"
#include "plan_common.h"
#include "vp.h"
#include "wave_ops.h"

namespace {

constexpr int PLAN_THREADS = 1024;

// Exclusive prefix sum over the workgroup; returns this thread's prefix and the
// total to everyone.  wsum: LDS scratch of PLAN_THREADS / 64 + 1 elements.
template <typename T>
__device__ T block_exscan(T v, T *total, T *wsum)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        T up = __shfl_up(inc, off);
        if (lane >= off) inc += up;
    }
    __syncthreads();   // wsum may still be read from a previous call
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    if (wave == 0) {
        const int nw = blockDim.x >> 6;
        T w = lane < nw ? wsum[lane] : T(0);
        T winc = w;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            T up = __shfl_up(winc, off);
            if (lane >= off) winc += up;
        }
        if (lane < nw) wsum[lane] = winc - w;
        if (lane == nw - 1) wsum[nw] = winc;
    }
    __syncthreads();
    *total = wsum[blockDim.x >> 6];
    return wsum[wave] + inc - v;
}


// The same scan for ints, two barriers: every wavefront scans the wavefront totals itself.
__device__ inline int block_exscan_int(int v, int *total, int *wsum)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int inc = wave_inclusive_sum(v);
    __syncthreads();   // wsum may still be read from a previous call
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    const int w = lane < nw ? wsum[lane] : 0;
    const int winc = wave_inclusive_sum(w);
    *total = __builtin_amdgcn_readlane(winc, nw - 1);
    return __builtin_amdgcn_readlane(winc - w, wave) + inc - v;
}

// Sums of three per-thread values over the workgroup, to every thread.  wsum3: 3 x 16 ints.
__device__ inline void block_sum3(int a, int b, int c, int *ta, int *tb, int *tc, int *wsum3)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    a = wave_inclusive_sum(a);
    b = wave_inclusive_sum(b);
    c = wave_inclusive_sum(c);
    __syncthreads();
    if (lane == 63) {
        wsum3[wave] = a;
        wsum3[16 + wave] = b;
        wsum3[32 + wave] = c;
    }
    __syncthreads();
    *ta = __builtin_amdgcn_readlane(wave_inclusive_sum(lane < nw ? wsum3[lane] : 0), nw - 1);
    *tb = __builtin_amdgcn_readlane(wave_inclusive_sum(lane < nw ? wsum3[16 + lane] : 0), nw - 1);
    *tc = __builtin_amdgcn_readlane(wave_inclusive_sum(lane < nw ? wsum3[32 + lane] : 0), nw - 1);
}

// The form is chosen per cluster in large batches.  A crowded cluster's slab is read once per 16 rows by the slab kernel,
// once per 48 or 64 by the many-row kernel, which takes it from about 33 rows on ("grouped").  And where the matrix
// cores, not one pass over W, set the time of the masked projection, every row costs that the same, so a cluster is masked
// when its slab takes longer than that for its
// rows (few rows, long list) and keeps its slab otherwise.  Which price per row is the best one depends on how much of
// the pass over W the masked rows fill; the full one, its half and its quarter are tried, and masking nothing, and the cheapest
// total wins if it is 8 % cheaper than either form for the whole batch (both projection kernels then have work, in one plan).
// 4,096 Zipf(1.1) rows on 500 clusters of 2,000 to 40,000 tokens, d = 1536, top-8: slabs 2,830 us, masked 3,360, both
// 2,100, crowded clusters grouped as well 1,500; 4,096 rows spread over 40 clusters of 8,000 to 16,000, d = 1024, top-6: 624
// without groups, 322 with; 1,024 rows on lists of up to 30,000, d = 1024, top-4: 823, 521, 365;
// 400 rows of that: 267 masked, 256.
constexpr int MIX_CHOICES = 4;   // prices 1, 1/2, 1/4; nothing masked
static_assert(MIX_CHOICES * PLAN_THREADS / 64 == 64, "one lane per choice and wavefront");
constexpr int SLAB_CLUSTER = 1 << 17;   // (counts clusters on the slab kernel above the masked rows)
static_assert(VP_MAX_ROWS < SLAB_CLUSTER && (long long)VP_MAX_CLUSTERS * SLAB_CLUSTER < 0x7fffffff - VP_MAX_ROWS, "one word for both");
constexpr int GROUP_TILES = 32;      // fewest candidate tiles of a grouped item

enum { ON_SLAB = 0, GROUPED = 1, MASKED_OUT = 2 };   // a cluster's form

// one cluster on its slab, in items of 1 / inv_tpi candidate groups, and grouped (in floats: integer divisions by what is not a
// constant would take most of the time)
struct ClusterTimes {
    float inv_pass_rate, inv_slab, inv_l2, k_factor, inv_rpi, inv_tpi;
    bool group;
    __device__ float slab(int rows, int tiles, const VpCostModel &cost) const
    {
        return tiles * (inv_slab + (ceil_div(rows, VP_ROWS_PER_ITEM) - 1) * inv_l2) +
               rows * (ceilf(tiles * inv_tpi) * cost.t_list + cost.t_row_slab);
    }
    __device__ float grouped(int rows, int tiles) const
    {
        // (the many-row kernel streams a little slower than the slab kernel: 5.1 against 6.8 TB/s on W)
        return group ? tiles * fmaxf(1.33f * inv_slab, ceilf(rows * inv_rpi) * inv_pass_rate) * k_factor : __builtin_inff();
    }
};

__global__ __launch_bounds__(PLAN_THREADS) void plan_kernel(
    const int2 *__restrict__ cpart, int parts, int N, int K, const int32_t *__restrict__ n_cand,
    const int32_t *__restrict__ tile_off, int target_items, int min_items, int max_items, int32_t *__restrict__ g,
    int32_t *__restrict__ out_cluster, int32_t *__restrict__ perm, VpRowPlan *__restrict__ rowplan,
    unsigned int *__restrict__ floors, VpItem *__restrict__ items, VpPlanHeader *__restrict__ hdr,
    int64_t *__restrict__ dbg_row_off, int dispatch, VpCostModel cost, int k, int V, int vtiles,
    int full_target_items, int full_min_items, int max_items_full, VpMixLimits mix)
{
    extern __shared__ int lds[];
    int *cnt = lds;             // [K]   rows per cluster
    int *off = cnt + K;         // [K]   first perm position of each bucket
    int *ioff = off + K;        // [K+1] first item of each bucket
    int *tl = ioff + K + 1;     // [K]   candidate tiles of each cluster
    int *cur = tl + K;          // [K]   scatter cursor
    int *form = cur + K;        // [K]   ON_SLAB, GROUPED or MASKED_OUT
    int *goff = form + K;       // [K+1] first grouped item of each bucket
    __shared__ int wsum[PLAN_THREADS / 64 + 1];
    __shared__ long long wsum64[PLAN_THREADS / 64 + 1];
    __shared__ int wsum3[48];
    __shared__ float mix_t[MIX_CHOICES][PLAN_THREADS / 64];
    __shared__ int mix_n[MIX_CHOICES][PLAN_THREADS / 64];
    __shared__ float wsum_f[PLAN_THREADS / 64];
    __shared__ int max_rgs;     // most row groups any bucket has
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    if (tid == 0) max_rgs = 0;
    for (int j = tid; j < K; j += PLAN_THREADS) {
        cnt[j] = 0;
        cur[j] = 0;
        form[j] = ON_SLAB;
        tl[j] = tile_off[j + 1] - tile_off[j];
    }
    __syncthreads();

    // finish Eq. 2: minimum over the centroid parts, ties to the lowest index
    vp_finish_eq2(cpart, parts, N, K, tid, PLAN_THREADS, [&](int r, int j) {
        g[r] = j;
        if (out_cluster) out_cluster[r] = j;
        atomicAdd(&cnt[j], 1);
    });
    __threadfence_block();   // the scatter below reads g[] written by other threads of this workgroup
    __syncthreads();

    // total candidate tiles of all row groups
    int my_tiles = 0, my_occ_tiles = 0, my_units = 0;
    float my_row_tiles = 0.f;
    for (int j = tid; j < K; j += PLAN_THREADS) {
        const int c = cnt[j];
        my_tiles += ceil_div(c, VP_ROWS_PER_ITEM) * tl[j];
        my_units += ceil_div(c, VP_ROWS_PER_ITEM);
        if (c > 0) my_occ_tiles += tl[j];
        my_row_tiles += (float)c * tl[j];
    }
    my_row_tiles = wave_sum_float(my_row_tiles);
    if (lane == 0) wsum_f[wave] = my_row_tiles;   // (read behind the barriers of block_sum3)
    int total_tiles, units, occ_tiles;
    block_sum3(my_tiles, my_units, my_occ_tiles, &total_tiles, &units, &occ_tiles, wsum3);

    // all forms give the same results, so the cheapest one is taken (cost model in vp_layout.h)
    int masked_rows = 0, grouped_rows = 0;
    int m_rgs = 0, m_chunks = 0, m_tpi = 0;   // the masked projection's items, where some clusters are masked
    int g_tpi = 0;                            // candidate tiles of a grouped item
    if (dispatch) {
        const int rpi = dispatch;   // rows per item of the masked projection (16, 48 or 64)
        // candidate groups of a slab item, as vp_tiles_per_wave cuts them
        const float tpi_slab = fmaxf(ceilf(total_tiles / (VP_WG_WAVES * fminf(fmaxf(total_tiles / (4.f * VP_WG_WAVES), (float)min_items), (float)target_items))), 1.f) * VP_WG_WAVES;
        const float row_tiles = __int_as_float(__builtin_amdgcn_readlane(
            __float_as_int(row_sum_float(lane < PLAN_THREADS / 64 ? wsum_f[lane] : 0.f)), PLAN_THREADS / 64 - 1));
        const float t_slab = vp_time_slabs(occ_tiles, total_tiles, row_tiles / tpi_slab + 0.5f * N, N, cost);
        const float t_full = vp_time_masked_rows(N, rpi, vtiles, k, cost.bw_gemm, cost) + cost.t_masked;
        const float pass = vtiles / (cost.bw_gemm * VP_MIX_GEMM);   // of one row group
        const float one_pass = vtiles / cost.bw_full;
        const float k_factor = vp_lists_factor(k);
        const float gemm = cost.bw_gemm * VP_MIX_GEMM;
        const float best = 0.92f * fminf(t_slab, vp_time_masked_rows(N, rpi, vtiles, k, gemm, cost) + cost.t_masked);
        // (whatever is masked, W is streamed once)
        if (mix.slots > 0 && (mix.group || best > cost.t_second + cost.t_mixed + one_pass * k_factor)) {
            const ClusterTimes time = {1.f / gemm, 1.f / cost.bw_slab, 1.f / cost.bw_l2, k_factor, 1.f / rpi, 1.f / tpi_slab, mix.group != 0};
            const float price = pass / rpi * k_factor;
            float t[MIX_CHOICES];
            int n[MIX_CHOICES];
#pragma unroll
            for (int i = 0; i < MIX_CHOICES; ++i) {
                t[i] = 0.f;
                n[i] = 0;
            }
            for (int j = tid; j < K; j += PLAN_THREADS) {
                const int c = cnt[j];
                if (c == 0) continue;
                const float ta = time.slab(c, tl[j], cost);
                const float tj = fminf(ta, time.grouped(c, tl[j]));
#pragma unroll
                for (int i = 0; i < MIX_CHOICES; ++i) {
                    const bool masked = i < MIX_CHOICES - 1 && mix.mask && tj > c * price * (1.f / (1 << i));
                    t[i] += masked ? 0.f : tj;
                    n[i] += masked ? c : tj == ta ? SLAB_CLUSTER : 0;
                }
            }
#pragma unroll
            for (int i = 0; i < MIX_CHOICES; ++i) {
                const float ts = wave_sum_float(t[i]);
                const int ns = wave_sum(n[i]);
                if (lane == 0) {
                    mix_t[i][wave] = ts;
                    mix_n[i][wave] = ns;
                }
            }
            __syncthreads();
            // lane l adds up wavefront l % 16's share under choice l / 16
            const float ts = row_sum_float(mix_t[lane >> 4][lane & 15]);
            const int ns = row_sum(mix_n[lane >> 4][lane & 15]);
            const int rows = ns & (SLAB_CLUSTER - 1);   // masked ones
            float both = ts + cost.t_second + (ns >= SLAB_CLUSTER ? cost.t_slab : 0.f) +
                         (rows > 0 ? vp_time_masked_rows(rows, rpi, vtiles, k, gemm, cost) + cost.t_mixed : 0.f);
            if (rows == N) both = __builtin_inff();
            float chosen = -1.f, least = best;   // (the price above which a cluster is masked)
#pragma unroll
            for (int i = 0; i < MIX_CHOICES; ++i) {
                const float t_i = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(both), 16 * i + 15));
                if (t_i < least) {
                    least = t_i;
                    chosen = i < MIX_CHOICES - 1 && mix.mask ? price * (1.f / (1 << i)) : __builtin_inff();
                }
            }
            if (chosen >= 0.f) {
                int my_masked = 0, my_grouped = 0, my_gtiles = 0, my_gunits = 0;
                my_tiles = my_units = 0;
                for (int j = tid; j < K; j += PLAN_THREADS) {
                    const int c = cnt[j];
                    if (c == 0) continue;
                    const float ta = time.slab(c, tl[j], cost), tb = time.grouped(c, tl[j]);
                    if (fminf(ta, tb) > c * chosen) {
                        form[j] = MASKED_OUT;
                        my_masked += c;
                    } else if (tb < ta) {
                        form[j] = GROUPED;
                        my_grouped += c;
                        my_gtiles += ceil_div(c, rpi) * tl[j];
                        my_gunits += ceil_div(c, rpi);
                    } else {
                        my_tiles += ceil_div(c, VP_ROWS_PER_ITEM) * tl[j];
                        my_units += ceil_div(c, VP_ROWS_PER_ITEM);
                    }
                }
                int s_tiles, s_units, g_tiles, g_units;
                block_sum3(my_tiles, my_units, my_masked, &s_tiles, &s_units, &masked_rows, wsum3);
                block_sum3(my_gtiles, my_gunits, my_grouped, &g_tiles, &g_units, &grouped_rows, wsum3);
                // whole rounds of the compute units for the masked items, as in a plan of its own, and no
                // more of them than workgroups
                int m_items = 0;
                if (masked_rows > 0) {
                    m_rgs = ceil_div(masked_rows, rpi);
                    int target = vp_swept_item_count(m_rgs, mix.slots, vtiles, mix.kt, mix.grid);
                    if (target > mix.grid) target = mix.grid / m_rgs * m_rgs;
                    const int m_tpw = vp_tiles_per_wave((long long)m_rgs * vtiles, max(target, 1), max(target, 1));
                    m_tpi = m_tpw * VP_WG_WAVES;
                    m_chunks = ceil_div(vtiles, m_tpi);
                    m_items = m_rgs * m_chunks;
                }
                g_tpi = max(GROUP_TILES, (ceil_div(g_tiles, VP_GROUP_ROUNDS * mix.slots) + 3) & ~3);
                const int g_items = grouped_rows > 0 ? ceil_div(g_tiles, g_tpi) + g_units : 0;   // (at most)
                // all item lists and their partial results have to fit the workspace, which is laid out for one
                // form at a time: the slabs get fewer, longer items if need be
                const int mg_items = m_items + g_items;
                const long long room = min((long long)mix.list - mg_items,
                                           (mix.row_slots - (long long)mg_items * rpi) / VP_ROWS_PER_ITEM) - s_units;
                if (masked_rows + grouped_rows > 0 && ((m_items + 7) & ~7) + ((g_items + 7) & ~7) <= mix.grid && room >= min_items) {
                    target_items = (int)min((long long)target_items, room);
                    total_tiles = s_tiles;
                    units = s_units;
                } else {
                    masked_rows = grouped_rows = 0;
                    for (int j = tid; j < K; j += PLAN_THREADS) form[j] = ON_SLAB;
                }
            }
        }
        if (masked_rows + grouped_rows == 0 && t_full < t_slab) {
            __syncthreads();
            vp_plan_single_bucket(N, V, vtiles, rpi, full_target_items, full_min_items, max_items_full, perm,
                                  rowplan, floors, items, hdr, nullptr, tid, PLAN_THREADS, true);
            return;
        }
    }
    const int tpw = vp_tiles_per_wave_units(total_tiles, units, target_items, min_items);
    const int tpi = tpw * VP_WG_WAVES;
    const int slab_rows = N - masked_rows - grouped_rows;

    // exclusive scans: rows -> bucket offsets (the grouped clusters' rows behind the others, the masked ones' last),
    // items -> item offsets
    int carry = 0, icarry = 0, gcarry = slab_rows, gicarry = 0, mcarry = slab_rows + grouped_rows;
    for (int base = 0; base < K; base += PLAN_THREADS) {
        const int j = base + tid;
        const int c = j < K ? cnt[j] : 0;
        const int t = j < K ? tl[j] : 0;
        const int f = j < K ? form[j] : ON_SLAB;
        const int rgs = ceil_div(c, VP_ROWS_PER_ITEM);
        int tot;
        const int ex = block_exscan_int(f == ON_SLAB ? c : 0, &tot, wsum);
        if (j < K && f == ON_SLAB) off[j] = carry + ex;
        carry += tot;
        const int iex = block_exscan_int(f == ON_SLAB ? rgs * ceil_div(t, tpi) : 0, &tot, wsum);
        if (j < K) ioff[j] = icarry + iex;
        icarry += tot;
        if (grouped_rows > 0) {
            const int gex = block_exscan_int(f == GROUPED ? c : 0, &tot, wsum);
            if (j < K && f == GROUPED) off[j] = gcarry + gex;
            gcarry += tot;
            const int giex = block_exscan_int(f == GROUPED ? ceil_div(c, dispatch) * ceil_div(t, g_tpi) : 0, &tot, wsum);
            if (j < K) goff[j] = gicarry + giex;
            gicarry += tot;
        }
        if (masked_rows > 0) {
            const int mex = block_exscan_int(f == MASKED_OUT ? c : 0, &tot, wsum);
            if (j < K && f == MASKED_OUT) off[j] = mcarry + mex;
            mcarry += tot;
        }
        if (f == ON_SLAB && rgs > 4) atomicMax(&max_rgs, rgs);
    }
    if (tid == 0) {
        ioff[K] = icarry;
        goff[K] = gicarry;
    }
    __syncthreads();
    const int total_items = min(icarry, max_items);
    const int m_items = m_rgs * m_chunks * (masked_rows > 0);
    const int m_slot0 = total_items * VP_ROWS_PER_ITEM;
    const int m_row0 = slab_rows + grouped_rows;

    // scatter rows into bucket order and tell the merge kernel where the partial results of each row will be
    for (int r = tid; r < N; r += PLAN_THREADS) {
        const int j = g[r];
        const int local = atomicAdd(&cur[j], 1);
        const int p = off[j] + local;
        perm[p] = r;
        floors[r] = VP_FLOOR_NONE;   // no lower bound of the row's k-th best logit known yet
        if (form[j] != ON_SLAB)
            for (int s = 0; s < VP_BOUND_SETS; ++s) vp_set_bounds(floors, N)[(size_t)r * VP_BOUND_SETS + s] = VP_FLOOR_NONE;
        VpRowPlan rp;
        rp.row = r;
        rp.cluster = j;
        rp.ids_off = tile_off[j] * VP_TILE_ITEMS;
        if (form[j] == ON_SLAB) {
            const int rgs = ceil_div(cnt[j], VP_ROWS_PER_ITEM);
            rp.slot0 = (ioff[j] + local / VP_ROWS_PER_ITEM) * VP_ROWS_PER_ITEM + local % VP_ROWS_PER_ITEM;
            rp.slot_stride = rgs * VP_ROWS_PER_ITEM;
            rp.nit = ceil_div(tl[j], tpi);
        } else if (form[j] == GROUPED) {
            rp.slot0 = m_slot0 + (m_items + goff[j]) * dispatch + local;   // (row group, slot of it) of the first range
            rp.slot_stride = ceil_div(cnt[j], dispatch) * dispatch;
            rp.nit = ceil_div(tl[j], g_tpi);
        } else {
            rp.slot0 = m_slot0 + p - m_row0;
            rp.slot_stride = m_rgs * dispatch;
            rp.nit = m_chunks;
            rp.ids_off = -1;
        }
        rp.pad[0] = rp.pad[1] = 0;
        rowplan[p] = rp;
    }

    // the items: for each bucket, candidate ranges outermost and row groups
    // innermost, so items that re-read the same tiles sit next to each other
    auto bucket_items = [&](const int *first, int count, int rows_per_item, int tiles_per_item, VpItem *out) {
        for (int it = tid; it < count; it += PLAN_THREADS) {
            int lo = 0, hi = K;   // largest j with first[j] <= it (buckets without items have empty ranges)
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (first[mid] <= it) lo = mid; else hi = mid;
            }
            const int j = lo;
            const int rows = cnt[j];
            const int rgs = ceil_div(rows, rows_per_item);
            const int local = it - first[j];
            const int ch = local / rgs;
            const int rg = local - ch * rgs;
            VpItem v;
            v.cluster = j;
            v.perm_start = off[j] + rg * rows_per_item;
            v.nrows = min(rows_per_item, rows - rg * rows_per_item);
            v.tile0 = ch * tiles_per_item;
            v.ntiles = min(tiles_per_item, tl[j] - ch * tiles_per_item);
            v.shared = rgs > 1;
            v.tile_off = tile_off[j];
            v.ncand = n_cand[j];
            out[it] = v;
        }
    };
    bucket_items(ioff, total_items, VP_ROWS_PER_ITEM, tpi, items);
    // those of the masked clusters, as a single-bucket plan has them
    for (int it = tid; it < m_items; it += PLAN_THREADS) {
        const int ch = it / m_rgs;
        const int rg = it - ch * m_rgs;
        VpItem v;
        v.cluster = -1;
        v.perm_start = m_row0 + rg * dispatch;
        v.nrows = min(dispatch, masked_rows - rg * dispatch);
        v.tile0 = ch * m_tpi;
        v.ntiles = min(m_tpi, vtiles - ch * m_tpi);
        v.shared = m_rgs > 1;
        v.tile_off = 0;
        v.ncand = V;
        items[total_items + it] = v;
    }
    if (grouped_rows > 0) bucket_items(goff, gicarry, dispatch, g_tpi, items + total_items + m_items);
    if (tid == 0) {
        hdr->total_items = total_items;
        hdr->tiles_per_wave = tpw;
        hdr->overflow = icarry > max_items;
        hdr->total_tiles = total_tiles;
        // buckets of five row groups and more: keep the row groups of a candidate range on one XCD
        hdr->swz_rgs = max_rgs > 4 ? -VP_XCD_BLOCK_ITEMS : 0;
        hdr->swz_chunks = 0;
        hdr->rows_per_item = VP_ROWS_PER_ITEM;
        hdr->mode = masked_rows + grouped_rows > 0 ? 2 : 0;
        hdr->masked_items = m_items;
        hdr->masked_item0 = total_items;
        hdr->masked_slot0 = m_slot0;
        hdr->masked_swz = m_rgs > 1 && m_chunks >= 8 ? m_rgs : 0;
        hdr->grouped_items = grouped_rows > 0 ? gicarry : 0;
    }

    // debug entry only: where each row's candidate logits start
    if (dbg_row_off) {
        __syncthreads();
        long long carry64 = 0;
        for (int base = 0; base < N; base += PLAN_THREADS) {
            const int r = base + tid;
            const long long c = r < N ? (long long)n_cand[g[r]] : 0;
            long long tot;
            const long long ex = block_exscan<long long>(c, &tot, wsum64);
            if (r < N) dbg_row_off[r] = carry64 + ex;
            carry64 += tot;
        }
        if (tid == 0) dbg_row_off[N] = carry64;
    }
}

// Plan of the full-vocabulary projection: one bucket holding every row in
// order, one slab holding every token.  Nothing depends on device data.
__global__ __launch_bounds__(256) void plan_full_kernel(
    int N, int V, int vtiles, int rpi, int target_items, int min_items, int max_items, int32_t *__restrict__ perm,
    VpRowPlan *__restrict__ rowplan, unsigned int *__restrict__ floors, VpItem *__restrict__ items,
    VpPlanHeader *__restrict__ hdr, int64_t *__restrict__ dbg_row_off)
{
    vp_plan_single_bucket(N, V, vtiles, rpi, target_items, min_items, max_items, perm, rowplan, floors, items, hdr,
                          dbg_row_off, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

}  // namespace

size_t vpk_plan_lds_bytes(int K) { return (size_t)(7 * K + 2) * sizeof(int); }

hipError_t vpk_plan_prepare()
{
    // clusters up to VP_MAX_CLUSTERS need a little over 112 KiB of dynamic LDS; allow it explicitly
    return hipFuncSetAttribute(reinterpret_cast<const void *>(plan_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, 120 * 1024);
}

void vpk_plan(const void *cpart, int parts, int N, int K, const int32_t *n_cand, const int32_t *tile_off,
              int target_items, int min_items, int max_items, int32_t *g, int32_t *out_cluster, int32_t *perm,
              VpRowPlan *rowplan, unsigned int *floors, VpItem *items, VpPlanHeader *hdr, int64_t *dbg_row_off,
              int dispatch, const VpCostModel &cost, int k, int V, int vtiles, int full_target_items,
              int full_min_items, int max_items_full, const VpMixLimits &mix, hipStream_t st)
{
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(PLAN_THREADS), vpk_plan_lds_bytes(K), st, (const int2 *)cpart,
                       parts, N, K, n_cand, tile_off, target_items, min_items, max_items, g, out_cluster, perm, rowplan, floors,
                       items, hdr, dbg_row_off, dispatch, cost, k, V, vtiles, full_target_items, full_min_items, max_items_full,
                       mix);
}

void vpk_plan_full(int N, int V, int vtiles, int rpi, int target_items, int min_items, int max_items, int32_t *perm,
                   VpRowPlan *rowplan, unsigned int *floors, VpItem *items, VpPlanHeader *hdr,
                   int64_t *dbg_row_off, hipStream_t st)
{
    const int work = max(N, max_items);
    const int blocks = min(64, (work + 255) / 256);
    hipLaunchKernelGGL(plan_full_kernel, dim3(blocks), dim3(256), 0, st, N, V, vtiles, rpi, target_items, min_items, max_items,
                       perm, rowplan, floors, items, hdr, dbg_row_off);
}
