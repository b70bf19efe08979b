// Projection of many rows against one run of slab tiles with the rows held in LDS: the
// GEMM-shaped case of Eq. 1 (section 2.1) for single-bucket plans (the full projection, the
// masked full projection, the batch-union form) of more than 16 rows and k-extents up to
// d_pad = 1536; and, in plans that choose the form per cluster, for the masked clusters' rows and for crowded clusters
// against their own slabs.
//
// An item is 64 rows (48 at d_pad = 1280 and 1536, where 64 do not fit) x a range of candidate groups, one
// workgroup of eight wavefronts.  The rows are staged once in LDS in MFMA operand order (4 or 3
// row tiles x KT KiB) and never move again.  The range is cut into steps of four candidate groups (64 candidates; of one or two in short
// items); wavefront w takes steps w, w + 8, ...  A step streams its groups' tiles straight into registers
// (a ring of a few k-tiles ahead, crossing step boundaries, so the loads never drain), and per
// k-tile feeds each loaded 1 KiB slab tile to one v_mfma_f32_16x16x32_f16 per row tile,
// whose row operands are read from LDS (one 1 KiB read per four MFMAs: four groups per step).  There is no split of the k-extent, so
// no wavefront waits for another inside the loop and there is no barrier between the staging of the rows and the end of
// the item - but for the two behind the first step of items that trade the bests of sets (below).
//
// After the 32 x 16 MFMAs of a step a lane holds, for each of the four row tiles, the 16 logits
// of one row (its quarter of each of the four groups).  They are folded in one go: bias,
// validity and membership mask, one online log-sum-exp update per row (steps 4-5 of the
// inference list of section 2.3), and the top-k (section 2.1).  Top-1 stays in registers.  For
// k >= 2 the workgroup keeps ONE list per row in LDS, shared by all eight wavefronts: k 64-bit
// keys (the logit's bits made monotone above the complemented position, so a larger key is an
// earlier entry in (logit descending, position ascending) order), always sorted.  A candidate is
// inserted without locks or turns by a cascade of LDS atomic maxima: slot 0 takes max(slot, key)
// and hands the smaller of the two to slot 1, and so on; every step keeps the multiset of keys
// (slots plus keys on their way) and the order of the slots, slots only ever grow, and a key
// leaves the far end only if k others are ahead of it - so whatever the interleaving of the
// lanes and wavefronts, the list ends as the k best keys in order.  The last slot is at all
// times a lower bound of the row's k-th best: a lane offers only candidates that are not below
// it (nor below the bound the workgroups that hold the same rows trade through global memory),
// best first, re-reading the bound after every insertion - so even the first step, which finds
// the list empty, costs a lane one or two insertions rather than sixteen.
//
// Where a row's candidates are spread over many items (and 4 <= k <= 8) the lists' upkeep is bound by how late the items learn of each
// other: each starts with an empty list, and 64 of them insert 57 entries a row where one behind the other would need two.  So
// behind the first step's MFMAs, before anything is inserted, the workgroups trade the best logits seen of eight sets that the row's
// candidates fall into (by lane quarter and the wavefront's parity): the k-th largest of the eight cannot be above the row's k-th
// best, and 64 items know it of 32,768 candidates at once.  It costs one wait for memory per item; after steps 1, 2 and 4 the
// sets are traded again without waiting, later on the k-th bests as elsewhere.  Which calls do, vp_trades_sets says; the code
// is compiled into kernels of its own (SETS), because in every list kernel the registers it takes were lost to the calls that never trade
// (masked, d_pad = 1024: 20 vector registers spilled and 72 scalar ones, without it none and 26; 64 rows, V = 200,000, d = 768, masked
// top-2: 90 us with it, 81 without).  Not for gathered columns (the union): 40 rows 1 % slower for the registers.
// Keeping the candidates in an unsorted queue instead of the cascade: 5 to 20 % slower (registers, and the queue's overflow);
// fewer atomics and plain loads of the sets: 40 us slower (the loads wait behind every atomic on their line).
#include <hip/hip_runtime.h>
#include <type_traits>
#include "vp_kernels.h"
#include "project_common.h"
#include "wave_ops.h"

namespace {

constexpr int L_NW = 8;        // wavefronts per workgroup
// row tiles per item: four (64 rows), or three where four do not fit the LDS (48 rows: 120 KiB at d_pad = 1280,
// 144 KiB at 1536)
constexpr int lds_row_tiles(int kt) { return kt > 32 ? 3 : 4; }
// Candidate groups per step: four (one 1 KiB read of the rows from LDS per four MFMAs), one or two for short items (vp_step_groups).
// About 16 KiB per wavefront are kept in flight either way.
constexpr int lds_k_tiles_in_flight(int kt, int g) { return g == 4 ? 4 : g == 2 ? 8 : kt % 16 == 0 ? 16 : 8; }
constexpr int VP_MAX_TOPK_LANES = 32;   // the epilogue writes a row's list with one lane per entry

// The k-th largest of a row's eight keys (k = 1 .. 8; a sorting network of 19 compare-exchanges).
__device__ inline unsigned int kth_of_sets(const unsigned int *set, int k)
{
    unsigned int v[VP_BOUND_SETS];
#pragma unroll
    for (int j = 0; j < VP_BOUND_SETS; ++j) v[j] = __hip_atomic_load(set + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    constexpr int pair[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                                 {0, 4}, {1, 5}, {2, 6}, {3, 7}, {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
    for (int p = 0; p < 19; ++p) {
        const unsigned int a = v[pair[p][0]], b = v[pair[p][1]];
        v[pair[p][0]] = max(a, b);
        v[pair[p][1]] = min(a, b);
    }
    unsigned int r = v[0];
#pragma unroll
    for (int j = 1; j < VP_BOUND_SETS; ++j) r = j < k ? v[j] : r;
    return r;
}

// (logit descending, position ascending), without branches
__device__ inline bool before_entry(float v, int i, float v2, int i2) { return (v > v2) | ((v == v2) & (i < i2)); }

template <int KT, int L_G, bool MASKED, bool NT, bool TOP1, bool GATHER, bool SETS>
__device__ inline void gemm_lds_item(const VpSlabSet &set, const uint4 *__restrict__ hidden, int d,
                                     const VpItem &item, int it, int k,
                                     float *__restrict__ partials, unsigned int *__restrict__ floors,
                                     unsigned int *__restrict__ bounds, const VpMaskInfo &mask,
                                     const int32_t *__restrict__ perm)
{
    constexpr int L_RT = lds_row_tiles(KT);
    constexpr int L_ROWS = 16 * L_RT;
    constexpr int L_PF = lds_k_tiles_in_flight(KT, L_G);
    static_assert(KT % L_PF == 0 && (L_G == 4 || L_G == 2 || L_G == 1), "whole passes; the mask's words");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (uniform: step numbers and tile offsets stay in scalar registers)
    const int lane = tid & 63;
    const int n = lane & 15;
    const int q = lane >> 4;

    extern __shared__ uint4 lds[];
    uint4 *ldsB = lds;                                                          // [L_RT][KT][64]: the rows
    unsigned long long *lkey = reinterpret_cast<unsigned long long *>(lds + L_RT * KT * 64);   // [k][64]: the rows' lists
    unsigned int *wg_floor = reinterpret_cast<unsigned int *>(lkey + k * L_ROWS);               // [64]
    unsigned int *set_best = wg_floor + L_ROWS;                                                 // [64][VP_BOUND_SETS] (SETS)
    // after the loop, in place of the rows:
    float *hdr_m = reinterpret_cast<float *>(lds);                              // [L_NW][64]
    float *hdr_s = hdr_m + L_NW * L_ROWS;

    const int ncand = item.ncand;
    const bool masked = MASKED && item.cluster < 0;   // (else a crowded cluster's own slab, in the same launch)
    const int gb = item.tile0;
    const int ge = item.tile0 + item.ntiles;
    const int nsteps = (item.ntiles + L_G - 1) / L_G;
    // Where the slab operands come from.  Packed slab: group after group of KT tiles of 1 KiB, lane l
    // at piece l of a tile.  GATHER (the batch-union form without a gathered copy, as the paper's
    // gathered GEMM reads its columns): the candidate's row of the token-major copy of W, whose
    // k-tile kt holds this lane's 16 bytes at piece kt * 4 + q; the candidates' token ids are U.
    constexpr int KSTEP = GATHER ? 4 : 64;   // pieces from one k-tile to the next
    const uint4 *slab = GATHER ? reinterpret_cast<const uint4 *>(set.tiles)
                               : reinterpret_cast<const uint4 *>(set.tiles) + (size_t)item.tile_off * KT * 64 + lane;
    const float *bias = set.bias + (size_t)item.tile_off * VP_TILE_ITEMS + q * 4;
    const int32_t *tokens = GATHER ? set.ids + (size_t)item.tile_off * VP_TILE_ITEMS + n : nullptr;

    // offsets (in 16-byte pieces) of the four groups of a step; groups past the item's end repeat
    // its last group (loaded, never looked at)
    auto group_off = [&](int step, unsigned int (&off)[L_G]) {
#pragma unroll
        for (int j = 0; j < L_G; ++j) {
            const int g = min(gb + step * L_G + j, ge - 1);
            if (GATHER) {
                const int tok = tokens[(size_t)g * VP_TILE_ITEMS];   // -1 in the padding of U's last group
                off[j] = (unsigned int)max(tok, 0) * (KT * 4) + q;
            } else {
                off[j] = (unsigned int)g * (KT * 64);
            }
        }
    };

    // The rows of this item -> LDS, MFMA operand order (row slots beyond nrows: zeros).  A
    // single-bucket plan keeps the rows in their own order: slot r of the item is row perm_start + r; where only
    // some clusters are masked (perm given), it is the row at that position of the bucket order.
    // All of a thread's pieces are fetched in one batch, in front of the first slab loads (loads
    // return in order: behind them, the rows would wait for bytes from HBM they do not depend on).
    constexpr int X = KT * 4;   // 16-byte pieces per padded row
    constexpr int PER = L_ROWS * X / (L_NW * 64);   // pieces per thread
    static_assert(PER * L_NW * 64 == L_ROWS * X, "the rows' pieces divide evenly over the threads");
    uint4 piece[PER];
    auto fetch = [&](auto row_of) {
        const int pieces_per_row = d >> 3;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = tid + i * (L_NW * 64);
            const int r = e / X;
            const int x = e - r * X;
            piece[i] = make_uint4(0, 0, 0, 0);
            if (r < item.nrows && x < pieces_per_row) piece[i] = hidden[(size_t)row_of(i, r) * pieces_per_row + x];
        }
    };
    if (MASKED && perm) {
        int row[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) row[i] = perm[item.perm_start + min((tid + i * (L_NW * 64)) / X, item.nrows - 1)];
        fetch([&](int i, int) { return row[i]; });
    } else {
        fetch([&](int, int r) { return item.perm_start + r; });
    }

    uint4 ring[L_PF][L_G];
    unsigned int cur[L_G], nxt[L_G];
    int step = wave;
    const bool active = step < nsteps;
    if (active) {
        group_off(step, cur);
#pragma unroll
        for (int p = 0; p < L_PF; ++p)
#pragma unroll
            for (int j = 0; j < L_G; ++j) ring[p][j] = load_piece<NT>(slab + cur[j] + p * KSTEP);
    }

#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = tid + i * (L_NW * 64);
        const int r = e / X;
        const int x = e - r * X;
        ldsB[((r >> 4) * KT + (x >> 2)) * 64 + (x & 3) * 16 + (r & 15)] = piece[i];
    }
    for (int e = tid; e < k * L_ROWS; e += L_NW * 64) lkey[e] = 0ull;   // below the key of every logit
    // this lane's row in each row tile
    int myrow[L_RT];
    bool row_valid[L_RT];
#pragma unroll
    for (int rt = 0; rt < L_RT; ++rt) {
        const int slot = rt * 16 + n;
        row_valid[rt] = slot < item.nrows;
        myrow[rt] = row_valid[rt] ? (MASKED && perm ? perm[item.perm_start + slot] : item.perm_start + slot) : -1;
    }
    // (the bounds are kept by row number, whichever form a row's cluster takes)
    if (tid < L_ROWS)
        wg_floor[tid] = !TOP1 && tid < item.nrows ? floors[MASKED && perm ? perm[item.perm_start + tid] : item.perm_start + tid]
                                                  : VP_FLOOR_NONE;
    const bool sets = SETS && L_G != 1 && vp_item_trades_sets(item.nrows, L_ROWS, item.ntiles, ncand);
    if (sets)
        for (int e = tid; e < L_ROWS * VP_BOUND_SETS; e += L_NW * 64) set_best[e] = VP_FLOOR_NONE;
    __syncthreads();

    // per row tile: running maximum, sum of exponentials, k-th best of this wavefront's list
    float m_run[L_RT], s_run[L_RT];
    float b1v[L_RT];
    int b1i[L_RT];
    unsigned int moff[L_RT];   // first word of the row's membership list
#pragma unroll
    for (int rt = 0; rt < L_RT; ++rt) {
        m_run[rt] = VP_NEG_BIG;
        s_run[rt] = 0.f;
        b1v[rt] = -__builtin_inff();
        b1i[rt] = VP_IDX_NONE;
        moff[rt] = masked ? (unsigned int)(row_valid[rt] ? mask.g[myrow[rt]] : 0) * (unsigned int)mask.words : 0u;
    }
    constexpr bool top1 = TOP1;   // k == 1: the best entry stays in registers, no list traffic in the loop
    unsigned int pending = 0;
    int pending_rt = -1;
    int done_steps = 0;
    const int my_set = q + 4 * (wave & 1);   // (a candidate is one lane's: every candidate is in one set)
    // this thread trades set tid % 8 of row slot tid / 8; its wavefront's eight rows then get their bounds anew
    unsigned int pending_set = VP_FLOOR_NONE;
    int slot_row = -1;
    bool asked = false;
    if (sets && tid / VP_BOUND_SETS < item.nrows)
        slot_row = MASKED && perm ? perm[item.perm_start + tid / VP_BOUND_SETS] : item.perm_start + tid / VP_BOUND_SETS;
    auto take_bests = [&]() {
        if (slot_row >= 0) atomicMax(set_best + tid, pending_set);
        wave_lds_fence();
        if (lane < 8 && wave * 8 + lane < item.nrows) atomicMax(wg_floor + wave * 8 + lane, kth_of_sets(set_best + (wave * 8 + lane) * VP_BOUND_SETS, k));
    };
    // behind a wavefront's first step (those without one: at the end), once by each of the eight
    auto trade_first_bests = [&]() {
        __syncthreads();
        if (slot_row >= 0) pending_set = atomicMax(bounds + (size_t)slot_row * VP_BOUND_SETS + (tid & (VP_BOUND_SETS - 1)), set_best[tid]);
        take_bests();
        __syncthreads();
    };

    uint4 bnext[L_RT];   // the rows' operands of the k-tile to come
#pragma unroll
    for (int rt = 0; rt < L_RT; ++rt) bnext[rt] = ldsB[(rt * KT) * 64 + lane];

    while (step < nsteps) {
        const int g0 = gb + step * L_G;
        const int next_step = step + L_NW;
        group_off(next_step < nsteps ? next_step : step, nxt);
        // bias and membership words of the step, wanted only after its MFMAs
        float4 bz[L_G];
#pragma unroll
        for (int j = 0; j < L_G; ++j) bz[j] = *reinterpret_cast<const float4 *>(bias + (size_t)min(g0 + j, ge - 1) * VP_TILE_ITEMS);
        uint2 mw[L_RT];
        if (MASKED && !masked) {
#pragma unroll
            for (int rt = 0; rt < L_RT; ++rt) mw[rt] = make_uint2(~0u, ~0u);
        }
        if (masked) {
            // the step's 64 candidates start at a multiple of 64: one aligned pair of 32-bit words (the
            // lists are padded to an even number of words)
#pragma unroll
            for (int rt = 0; rt < L_RT; ++rt) {
                const uint32_t *words = mask.bitmaps + (moff[rt] + ((g0 * VP_TILE_ITEMS) >> 5));
                if (L_G == 4) mw[rt] = *reinterpret_cast<const uint2 *>(words);
                else mw[rt].x = words[0] >> ((g0 & 1) * VP_TILE_ITEMS);   // (one group: half a word; two: a whole one, items start at even groups)
            }
        }

        floatx4 acc[L_RT][L_G];
#pragma unroll
        for (int rt = 0; rt < L_RT; ++rt)
#pragma unroll
            for (int j = 0; j < L_G; ++j) acc[rt][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        // L_PF k-tiles per pass of the loop body: pass b consumes the ring and refills it with
        // k-tiles (b + 1) * L_PF ... of this step, the last pass with the first k-tiles of the
        // wavefront's next step
#pragma unroll 1
        for (int b = 0; b < KT / L_PF; ++b) {
            const bool last = b == KT / L_PF - 1;
            unsigned int src[L_G];
#pragma unroll
            for (int j = 0; j < L_G; ++j) src[j] = last ? nxt[j] : cur[j] + (b + 1) * (L_PF * KSTEP);
#pragma unroll
            for (int u = 0; u < L_PF; ++u) {
                // The rows' operands of the next k-tile are read while this one's MFMAs run (after a
                // step's last k-tile: the first one again; the rows never change), and a ring slot is
                // refilled as soon as its MFMAs have been issued: the loads then have three quarters
                // of a pass, and the other wavefront's share of the matrix cores, to come back.  The
                // scheduling barrier keeps that order (left alone, the compiler sinks all loads of a
                // pass to its end, right in front of their first use).
                Frag bf[L_RT];
                const int kt_next = (b * L_PF + u + 1) == KT ? 0 : b * L_PF + u + 1;
#pragma unroll
                for (int rt = 0; rt < L_RT; ++rt) {
                    bf[rt].u = bnext[rt];
                    bnext[rt] = ldsB[(rt * KT + kt_next) * 64 + lane];
                }
#pragma unroll
                for (int rt = 0; rt < L_RT; ++rt)
#pragma unroll
                    for (int j = 0; j < L_G; ++j) {
                        Frag a;
                        a.u = ring[u][j];
                        acc[rt][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, bf[rt].h, acc[rt][j], 0, 0, 0);
                    }
#pragma unroll
                for (int j = 0; j < L_G; ++j) ring[u][j] = load_piece<NT>(slab + src[j] + u * KSTEP);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // fold the 16 logits of each of this lane's four rows
        const int c_first = g0 * VP_TILE_ITEMS + q * 4;           // position of z[0] (j = 0, i = 0) in the slab
        const bool ragged = (g0 + L_G) * VP_TILE_ITEMS > ncand || g0 + L_G > ge;   // (wavefront-uniform)
        if (asked) take_bests();   // (asked for a step ago)
        asked = false;
        if (pending_rt >= 0) {
            // bounds read from the other workgroups a step ago
#pragma unroll
            for (int rt = 0; rt < L_RT; ++rt)
                if (rt == pending_rt && q == 0 && row_valid[rt]) atomicMax(wg_floor + rt * 16 + n, pending);
            pending_rt = -1;
        }
        // (written per row tile with the tile's number a compile-time constant: the accumulators
        // and the per-tile state must stay in registers)
        auto logits_of = [&](auto rt_const, float (&z)[L_G * 4]) {
            constexpr int rt = decltype(rt_const)::value;
#pragma unroll
            for (int j = 0; j < L_G; ++j) {
                z[j * 4 + 0] = acc[rt][j][0] + bz[j].x;
                z[j * 4 + 1] = acc[rt][j][1] + bz[j].y;
                z[j * 4 + 2] = acc[rt][j][2] + bz[j].z;
                z[j * 4 + 3] = acc[rt][j][3] + bz[j].w;
            }
            if (ragged) {
#pragma unroll
                for (int j = 0; j < L_G; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (g0 + j >= ge || c_first + j * VP_TILE_ITEMS + i >= ncand) z[j * 4 + i] = -__builtin_inff();
            }
            if (MASKED) {
                // a token outside the row's active set is at -infinity (steps 4-5 of section 2.3's list):
                // the membership bit, spread over a word, keeps the logit's bits or takes -infinity's
#pragma unroll
                for (int j = 0; j < L_G; ++j) {
                    const uint32_t w = (j >> 1) ? mw[rt].y : mw[rt].x;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)w, (j & 1) * 16 + q * 4 + i, 1);   // 0 or ~0
                        z[j * 4 + i] = __uint_as_float((__float_as_uint(z[j * 4 + i]) & keep) | (0xff800000u & ~keep));
                    }
                }
            }
        };
        if (sets && done_steps == 0) {   // (one row tile at a time: four at once spill)
            auto best_of = [&](auto rt_const) {
                constexpr int rt = decltype(rt_const)::value;
                float z[L_G * 4];
                logits_of(rt_const, z);
                float tmax = z[0];
#pragma unroll
                for (int e = 1; e < L_G * 4; ++e) tmax = fmaxf(tmax, z[e]);
                if (row_valid[rt] & (tmax > -__builtin_inff())) atomicMax(set_best + (rt * 16 + n) * VP_BOUND_SETS + my_set, float_key(tmax));
            };
            best_of(std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            best_of(std::integral_constant<int, 1>{});
            __builtin_amdgcn_sched_barrier(0);
            best_of(std::integral_constant<int, 2>{});
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (L_RT > 3) best_of(std::integral_constant<int, 3>{});
            trade_first_bests();
        }
        auto fold_row_tile = [&](auto rt_const) {
            constexpr int rt = decltype(rt_const)::value;
            float z[L_G * 4];
            logits_of(rt_const, z);
            float tmax = z[0];
#pragma unroll
            for (int e = 1; e < L_G * 4; ++e) tmax = fmaxf(tmax, z[e]);
            const float mn = fmaxf(m_run[rt], tmax);
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < L_G * 4; ++e) sum += fast_exp(z[e] - mn);
            s_run[rt] = s_run[rt] * fast_exp(m_run[rt] - mn) + sum;
            m_run[rt] = mn;

            if (top1) {
                // positions ascend along a lane's own stream: a strict comparison keeps the smaller one
#pragma unroll
                for (int e = 0; e < L_G * 4; ++e) {
                    const bool take = z[e] > b1v[rt];
                    b1v[rt] = take ? z[e] : b1v[rt];
                    b1i[rt] = take ? c_first + (e >> 2) * VP_TILE_ITEMS + (e & 3) : b1i[rt];
                }
                return;
            }
            const int slot = rt * 16 + n;
            unsigned long long *list = lkey + slot;              // + p * L_ROWS
            const float far_floor = key_float(__hip_atomic_load(wg_floor + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            auto row_floor = [&]() {
                const unsigned long long kth = __hip_atomic_load(list + (k - 1) * L_ROWS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                return fmaxf(far_floor, kth ? key_float((unsigned int)(kth >> 32)) : -__builtin_inff());
            };
            float floor = row_floor();
            const bool want = row_valid[rt] & (tmax >= floor) & (tmax > -__builtin_inff());
            if (__ballot(want) != 0) {
                if (want) {
                    // this lane's candidates, best first, until one is below the bound (the others,
                    // which are not better, then are too)
                    while (true) {
                        float v = fmaxf(z[0], -__builtin_inff());   // (NaN is no candidate, and none to measure the others by)
                        int e_best = 0;
#pragma unroll
                        for (int e = 1; e < L_G * 4; ++e) {
                            const bool take = z[e] > v;   // strict: of equal logits the smaller position
                            v = take ? z[e] : v;
                            e_best = take ? e : e_best;
                        }
                        if (!((v >= floor) & (v > -__builtin_inff()))) break;
                        const unsigned int c = (unsigned int)(c_first + (e_best >> 2) * VP_TILE_ITEMS + (e_best & 3));
                        // (-0 becomes +0: equal as logits, they must tie and be ordered by position)
                        unsigned long long carry = ((unsigned long long)float_key(v + 0.f) << 32) | (unsigned int)~c;
                        for (int p = 0; p < k && carry != 0ull; ++p) {
                            const unsigned long long old = __hip_atomic_fetch_max(list + p * L_ROWS, carry, __ATOMIC_RELAXED,
                                                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
                            carry = old < carry ? old : carry;
                        }
#pragma unroll
                        for (int e = 0; e < L_G * 4; ++e) z[e] = e == e_best ? -__builtin_inff() : z[e];
                        floor = row_floor();
                    }
                }
            }
        };
        fold_row_tile(std::integral_constant<int, 0>{});
        fold_row_tile(std::integral_constant<int, 1>{});
        fold_row_tile(std::integral_constant<int, 2>{});
        if constexpr (L_RT > 3) fold_row_tile(std::integral_constant<int, 3>{});
        // every second step of a wavefront, one row tile in turn: trade bounds with the other
        // workgroups that project the same rows onto other candidate ranges (one atomicMax
        // publishes ours and returns theirs, folded into the LDS copy a step later: no wait here)
        ++done_steps;
        if (sets) asked = done_steps == 1 || done_steps == 2 || done_steps == 4;
        if (asked) {
#pragma unroll
            for (int rt = 0; rt < L_RT; ++rt)
                if (row_valid[rt] & (m_run[rt] > VP_NEG_BIG)) atomicMax(set_best + (rt * 16 + n) * VP_BOUND_SETS + my_set, float_key(m_run[rt]));
            wave_lds_fence();
            if (slot_row >= 0) pending_set = atomicMax(bounds + (size_t)slot_row * VP_BOUND_SETS + (tid & (VP_BOUND_SETS - 1)), set_best[tid]);
        } else if (!top1 && (done_steps & 1) == 0) {
            const int rt_x = ((done_steps >> 1) + wave) % L_RT;
#pragma unroll
            for (int rt = 0; rt < L_RT; ++rt)
                if (rt == rt_x && q == 0 && row_valid[rt]) {
                    const unsigned long long kth = __hip_atomic_load(lkey + (k - 1) * L_ROWS + rt * 16 + n, __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_WORKGROUP);
                    const unsigned int mine = max((unsigned int)(kth >> 32),
                                                  __hip_atomic_load(wg_floor + rt * 16 + n, __ATOMIC_RELAXED,
                                                                    __HIP_MEMORY_SCOPE_WORKGROUP));
                    pending = atomicMax(floors + myrow[rt], max(mine, (unsigned int)VP_FLOOR_NONE));
                }
            pending_rt = rt_x;
        }
#pragma unroll
        for (int j = 0; j < L_G; ++j) cur[j] = nxt[j];
        step = next_step;
    }

    if (sets && !active) trade_first_bests();   // (the others were there behind their first steps)

    // the row's four lanes (one per quarter of every group) -> one (m, s); top-1: one entry
#pragma unroll
    for (int rt = 0; rt < L_RT; ++rt) {
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float m2 = __shfl_xor(m_run[rt], off);
            const float s2 = __shfl_xor(s_run[rt], off);
            const float mn = fmaxf(m_run[rt], m2);
            s_run[rt] = s_run[rt] * fast_exp(m_run[rt] - mn) + s2 * fast_exp(m2 - mn);
            m_run[rt] = mn;
            if (top1) {
                const float v2 = __shfl_xor(b1v[rt], off);
                const int i2 = __shfl_xor(b1i[rt], off);
                const bool take = before_entry(v2, i2, b1v[rt], b1i[rt]);
                b1v[rt] = take ? v2 : b1v[rt];
                b1i[rt] = take ? i2 : b1i[rt];
            }
        }
        if (top1 && q == 0 && row_valid[rt] && b1i[rt] != VP_IDX_NONE)
            __hip_atomic_fetch_max(lkey + rt * 16 + n,
                                   ((unsigned long long)float_key(b1v[rt] + 0.f) << 32) | (unsigned int)~(unsigned int)b1i[rt],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();   // nobody reads the rows any more: their LDS becomes the (m, s) exchange
#pragma unroll
    for (int rt = 0; rt < L_RT; ++rt) {
        if (q == 0) {
            hdr_m[wave * L_ROWS + rt * 16 + n] = m_run[rt];
            hdr_s[wave * L_ROWS + rt * 16 + n] = s_run[rt];
        }
    }
    if (!top1 && tid < item.nrows) {
        const unsigned int kth = (unsigned int)(lkey[(k - 1) * L_ROWS + tid] >> 32);
        atomicMax(floors + (MASKED && perm ? perm[item.perm_start + tid] : item.perm_start + tid), max(max(kth, wg_floor[tid]), (unsigned int)VP_FLOOR_NONE));
    }
    __syncthreads();

    // one partial result per (item, row): the row's list is in order already; wavefront w takes
    // row slots w, w + 8, ...
    const int PFL = vp_partial_floats(k);
    for (int r = wave; r < item.nrows; r += L_NW) {
        float M = hdr_m[r];
#pragma unroll
        for (int w = 1; w < L_NW; ++w) M = fmaxf(M, hdr_m[w * L_ROWS + r]);
        float S = 0.f;
#pragma unroll
        for (int w = 0; w < L_NW; ++w) S += hdr_s[w * L_ROWS + r] * fast_exp(hdr_m[w * L_ROWS + r] - M);
        float *out = partials + ((size_t)it * L_ROWS + r) * PFL;
        if (lane == 0) {
            out[0] = M;
            out[1] = S;
        }
        if (lane < k) {
            const unsigned long long key = lkey[lane * L_ROWS + r];
            out[2 + lane] = key ? key_float((unsigned int)(key >> 32)) : -__builtin_inff();
            out[2 + k + lane] = __int_as_float(key ? (int)~(unsigned int)key : VP_IDX_NONE);
        }
    }
}

// One item, in steps of as many groups as pay for it.
template <int KT, bool MASKED, bool TOP1, bool GATHER, bool SETS>
__device__ __forceinline__ void many_row_item(const VpSlabSet &set, const uint4 *__restrict__ hidden, int d, const VpItem &item, int it, int k,
                                              float *__restrict__ partials, unsigned int *__restrict__ floors,
                                              unsigned int *__restrict__ bounds, const VpMaskInfo &mask, const int32_t *__restrict__ perm)
{
    const int groups = vp_step_groups(KT, k, item.shared, item.ntiles, SETS);
    if (item.shared || GATHER) {
        if (groups == 1) gemm_lds_item<KT, 1, MASKED, false, TOP1, GATHER, false>(set, hidden, d, item, it, k, partials, floors, bounds, mask, perm);
        else gemm_lds_item<KT, 4, MASKED, false, TOP1, GATHER, SETS>(set, hidden, d, item, it, k, partials, floors, bounds, mask, perm);
    } else {
        // (plain items: the order of the code is worth 1 us to short ones; masked ones spill more in the other order)
        if (!MASKED && groups == 4) gemm_lds_item<KT, 4, MASKED, true, TOP1, false, SETS>(set, hidden, d, item, it, k, partials, floors, bounds, mask, perm);
        else if (groups == 1) gemm_lds_item<KT, 1, MASKED, true, TOP1, false, false>(set, hidden, d, item, it, k, partials, floors, bounds, mask, perm);
        else if (groups == 2) gemm_lds_item<KT, 2, MASKED, true, TOP1, false, SETS>(set, hidden, d, item, it, k, partials, floors, bounds, mask, perm);
        else if (MASKED) gemm_lds_item<KT, 4, MASKED, true, TOP1, false, SETS>(set, hidden, d, item, it, k, partials, floors, bounds, mask, perm);
    }
}

template <int KT, bool MASKED, bool TOP1, bool GATHER, bool SETS>
__global__ __launch_bounds__(L_NW * 64) void project_gemm_lds_kernel(
    VpSlabSet set, const uint4 *__restrict__ hidden, int d,
    const VpItem *__restrict__ items, const VpPlanHeader *__restrict__ hdr, int k,
    float *__restrict__ partials, unsigned int *__restrict__ floors, unsigned int *__restrict__ bounds, VpMaskInfo mask,
    const int32_t *__restrict__ perm, VpSlabSet slabs)
{
    if (MASKED ? hdr->mode == 0 : hdr->mode != 0) return;   // the planner chose the other form
    const int total_items = MASKED ? hdr->masked_items : hdr->total_items;
    // (> 1: several row groups and enough candidate ranges for the 8 XCDs)
    const int swz = MASKED ? hdr->masked_swz : hdr->swz_rgs;
    int it = swz > 1 ? vp_item_of_workgroup_even(blockIdx.x, total_items) : (int)blockIdx.x;
    const int behind = (int)blockIdx.x - ((total_items + 7) & ~7);
    if (MASKED && behind >= 0) {
        // items of crowded clusters, dealt to the XCDs by themselves (they are shorter than the masked ones)
        it = vp_item_of_workgroup_even(behind, hdr->grouped_items);
        if (it < 0) return;
        it += total_items;
    } else if (it < 0 || it >= total_items) {
        return;
    }
    const VpItem item = items[MASKED ? hdr->masked_item0 + it : it];
    if (MASKED && item.cluster >= 0) {
        set.tiles = slabs.tiles;
        set.bias = slabs.bias;
    }
    if (MASKED) {
        partials += (size_t)hdr->masked_slot0 * vp_partial_floats(k);
        if (hdr->mode == 1) perm = nullptr;   // the whole batch, in its own order
    }
    const int kk = TOP1 ? 1 : k;
    // crowded clusters' items do not trade (their rows are in few items) and do not pay for the registers: 1,200 rows on 20
    // clusters of 12,000 tokens, d = 768, top-4: 113 us, with the code that trades 123
    if (MASKED && SETS && item.cluster >= 0) many_row_item<KT, MASKED, TOP1, GATHER, false>(set, hidden, d, item, it, kk, partials, floors, bounds, mask, perm);
    else many_row_item<KT, MASKED, TOP1, GATHER, SETS>(set, hidden, d, item, it, kk, partials, floors, bounds, mask, perm);
}

template <int KT, bool MASKED, bool GATHER>
void launch_lds(const VpSlabSet &set, const void *hidden, int d, const VpItem *items,
                const VpPlanHeader *hdr, int grid_items, int k, float *partials, unsigned int *floors,
                unsigned int *bounds, bool sets, const VpMaskInfo &mask, const int32_t *perm, const VpSlabSet &slabs, hipStream_t st)
{
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid_items), dim3(L_NW * 64), vpk_project_rows_lds_bytes(k, KT, sets), st, set,
                           (const uint4 *)hidden, d, items, hdr, k, partials, floors, bounds, mask, perm, slabs);
    };
    if (k == 1) launch(project_gemm_lds_kernel<KT, MASKED, true, GATHER, false>);
    else if (sets && !GATHER) launch(project_gemm_lds_kernel<KT, MASKED, false, GATHER, !GATHER>);
    else launch(project_gemm_lds_kernel<KT, MASKED, false, GATHER, false>);
}

template <int KT>
hipError_t allow_lds_bytes()
{
    const void *fns[] = {reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, false, false, false, false>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, false, false, false, true>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, false, true, false, false>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, true, false, false, false>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, true, false, false, true>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, true, true, false, false>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, false, false, true, false>),
                         reinterpret_cast<const void *>(project_gemm_lds_kernel<KT, false, true, true, false>)};
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

size_t vpk_project_rows_lds_bytes(int k, int kt, bool sets)
{
    const int rows = 16 * lds_row_tiles(kt);
    return (size_t)rows * kt * (VP_TILE_BYTES / 16) + (size_t)k * rows * 8 + rows * 4 +
           (sets ? (size_t)rows * VP_BOUND_SETS * 4 : 0);
}

// Built for d_pad = 256 to 1536 (beyond, the rows of an item do not fit the LDS beside its lists).  The alternative at 768
// and 1280, items of 16 rows, reads W once per 16 rows through the L2; full projection, V = 150,000, top-3, us per call,
// those -> this kernel: d = 768, N = 17: 102 -> 50, 64: 119 -> 55, 256: 216 -> 82, 1,024: 660 -> 227, 8,192: 6,290 -> 1,667;
// d = 1280: 142 -> 73, 195 -> 90, 431 -> 161, 1,356 -> 502, 10,036 -> 3,596.
bool vpk_project_rows_lds_supported(int kt, int k)
{
    return kt % 8 == 0 && kt >= 8 && kt <= 48 && k >= 1 && k <= VP_MAX_TOPK_LANES;
}
// row tiles of an item of that kernel
int vpk_project_rows_lds_row_tiles(int kt) { return lds_row_tiles(kt); }

hipError_t vpk_project_rows_lds_prepare()
{
    hipError_t e = allow_lds_bytes<8>();
    if (e == hipSuccess) e = allow_lds_bytes<16>();
    if (e == hipSuccess) e = allow_lds_bytes<24>();
    if (e == hipSuccess) e = allow_lds_bytes<32>();
    if (e == hipSuccess) e = allow_lds_bytes<40>();
    if (e == hipSuccess) e = allow_lds_bytes<48>();
    return e;
}

// mask: nullptr, or the membership lists of the masked full projection.  gather: the set's tiles
// are the token-major copy of W and its ids the batch's union U (no mask then); the slab operands
// are read through U instead of from a packed copy.  perm, and slabs, the clusters' own, are read only where the planner
// chooses the form per cluster: a single-bucket plan keeps the rows in their own order.  sets: items may trade the bests of sets
// (vp_trades_sets).
void vpk_project_rows_lds(const VpSlabSet &set, const void *hidden, int d, const int32_t *perm, const VpItem *items,
                          const VpPlanHeader *hdr, int grid_items, int k, float *partials, unsigned int *floors,
                          unsigned int *bounds, bool sets, const VpMaskInfo *mask, const VpSlabSet *slabs, bool gather, hipStream_t st)
{
    const VpMaskInfo none = {nullptr, nullptr, 0};
#define VP_LDS_CASE(KT)                                                                                                   \
    case KT:                                                                                                              \
        if (mask) launch_lds<KT, true, false>(set, hidden, d, items, hdr, grid_items, k, partials, floors, bounds, sets, *mask, perm, slabs ? *slabs : set, st); \
        else if (gather) launch_lds<KT, false, true>(set, hidden, d, items, hdr, grid_items, k, partials, floors, bounds, sets, none, nullptr, set, st); \
        else launch_lds<KT, false, false>(set, hidden, d, items, hdr, grid_items, k, partials, floors, bounds, sets, none, nullptr, set, st); \
        break;
    switch (set.kt) {
        VP_LDS_CASE(8)
        VP_LDS_CASE(16)
        VP_LDS_CASE(24)
        VP_LDS_CASE(32)
        VP_LDS_CASE(40)
        VP_LDS_CASE(48)
        default: break;   // callers check vpk_project_rows_lds_supported
    }
#undef VP_LDS_CASE
}
