// Offline training of the clusters on the GPU (section 2.2 and the training
// settings of section 3.1): Lloyd k-means over recorded hidden vectors and the
// active set of each cluster as the union of its members' recorded tokens.
//
// Memberships are Eq. 2 (nearest centroid, ties to the lowest index), for many vectors as a
// GEMM.  The update is exact: every binary16 value is an integer multiple of 2^-24, so sums
// of members, kept in double precision while they stay below 2^29 in magnitude, or as 64-bit
// integers in that unit where the sums of different threads meet, are exact whatever the
// order of the additions (and of the atomics), and the mean sum / count is rounded once, in
// double precision, to binary16 (nearest, ties to even).  A cluster without members keeps its
// centroid.
//
// An iteration redoes only what the last one changed, with the same results to the bit.  The sums are
// exact, so they are carried from iteration to iteration: a vector that changes its cluster is taken
// from one sum and added to the other.  A centroid that came out as it was has the same scores as
// before, so a vector whose own centroid is one of those stays with it unless a changed centroid now
// beats it; and where no centroid changed nothing can, and the remaining kernels leave at once.
// 131,072 vectors, 1,000 clusters, d = 1024, 20 iterations of the benchmark's mixture (1,000, 567, 68, 2 and
// 0 centroids change): 7,770 -> 1,470 us; 108,433 vectors, 481 clusters, d = 768, 16 iterations: 860 us; 60,000 vectors, 64
// clusters, d = 512, where it takes 17 iterations to come to rest: 890 us.
#include <hip/hip_runtime.h>
#include <algorithm>
#include "vp_kernels.h"
#include "project_common.h"
#include "wave_ops.h"

namespace {

__device__ inline bool part_less(float s, int j, float s2, int j2) { return s < s2 || (s == s2 && j < j2); }

// What the membership kernels leave behind.  The first pass counts the members; later passes compare with the pass
// before, count the events of every cluster (a member that came or went) and keep the counts up to date.  With RANK
// they keep what the counting atomics return, each vector's number among its cluster's members or events
// (kmeans_place_kernel); without it they do not ask, because a wavefront waits for what it asks for: the split-k kernel at
// 49,200 vectors, 240 clusters, d = 1024: 87 us per call without, 96 with it; 16,400 vectors, 150 clusters, d = 1536: 59
// and 64.
template <bool RANK>
__device__ __forceinline__ void record_member(VpKmPass p, long row, int j)
{
    int *const assign = p.assign;
    if (p.first) {
        assign[row] = j;
        if (RANK) p.rank[row] = atomicAdd(&p.counts[j], 1);
        else atomicAdd(&p.counts[j], 1);
        return;
    }
    const int old = assign[row];
    p.prev[row] = old;
    if (j == old) return;
    assign[row] = j;
    atomicAdd(&p.counts[j], 1);
    atomicSub(&p.counts[old], 1);
    if (RANK) {
        p.rank[row] = atomicAdd(&p.events[j], 1);
        p.rank_old[row] = atomicAdd(&p.events[old], 1);
    } else {
        atomicAdd(&p.events[j], 1);
        atomicAdd(&p.events[old], 1);
    }
}

// Finishes Eq. 2 for a chunk of rows (minimum over the centroid ranges).
template <bool RANK>
__global__ __launch_bounds__(256) void kmeans_assign_kernel(const int2 *__restrict__ cpart, int parts, long row0, int rows,
                                                            int K, VpKmPass pass)
{
    if (!pass.first && pass.state->changed == 0) return;
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    float bs = __builtin_inff();
    int bj = VP_IDX_NONE;
    for (int p = 0; p < parts; ++p) {
        const int2 e = cpart[(size_t)r * parts + p];
        const float s = __int_as_float(e.x);
        if (part_less(s, e.y, bs, bj)) {
            bs = s;
            bj = e.y;
        }
    }
    if ((unsigned)bj >= (unsigned)K) bj = 0;   // only when every score is NaN: keep the index in range
    record_member<RANK>(pass, row0 + r, bj);
}

// The operands of Eq. 2 for a pass: 16 centroids a workgroup, one a wavefront, into the packed tiles, their squared
// norms, and from the second pass on which of them are others than in the pass before.  Changed centroids are also packed
// side by side (in no particular order; their numbers beside them), where a pass can meet them without the others.  The
// norm is summed as cnorm_kernel sums it.  `always`: centroids may change without events (VP_KMEANS_SPLIT_EMPTY).
__global__ __launch_bounds__(1024) void kmeans_prepare_kernel(const uint16_t *__restrict__ C, int K, int d, int kt_count,
                                                              int always, VpKmPass pass)
{
    if (!pass.first && !always && pass.state->total_events == 0) return;   // (changed is 0 already)
    __shared__ int is_changed[16];
    __shared__ int slot0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 16 + wave;
    const int pieces = d >> 3, X = kt_count * 4;
    uint4 *const cp = reinterpret_cast<uint4 *>(pass.cp);
    auto place = [&](int slot, int x) { return ((size_t)(slot >> 4) * kt_count + (x >> 2)) * 64 + (x & 3) * 16 + (slot & 15); };
    const uint4 *row = reinterpret_cast<const uint4 *>(C + (size_t)min(j, K - 1) * d);
    bool differs = pass.first != 0;
    float acc = 0.f;
    if (j < K) {
        for (int x = lane; x < X; x += 64) {
            const uint4 v = x < pieces ? row[x] : make_uint4(0, 0, 0, 0);
            if (!pass.first) {
                const uint4 was = cp[place(j, x)];
                differs |= (v.x != was.x) | (v.y != was.y) | (v.z != was.z) | (v.w != was.w);
            }
            if (differs) cp[place(j, x)] = v;
        }
        for (int i = lane; i < d; i += 64) {
            const float c = (float)__builtin_bit_cast(_Float16, C[(size_t)j * d + i]);
            acc += c * c;
        }
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    } else if (pass.first) {   // the last group's padding
        for (int x = lane; x < X; x += 64) cp[place(j, x)] = make_uint4(0, 0, 0, 0);
        if (lane == 0) pass.cnorm[j] = __builtin_inff();
    }
    const bool changed = j < K && __ballot(differs) != 0;
    if (lane == 0 && j < K) {
        if (pass.first) pass.counts[j] = 0;
        pass.events[j] = 0;
        pass.cursor[j] = 0;
        pass.flag[j] = changed;
        if (changed) pass.cnorm[j] = acc;
    }
    if (pass.first) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) pass.state->unsettled = pass.state->settled = 0;
    if (lane == 0) is_changed[wave] = changed;
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) before += is_changed[w];
        total += is_changed[w];
    }
    if (threadIdx.x == 0 && total > 0) slot0 = atomicAdd(&pass.state->changed, total);
    __syncthreads();
    if (!changed) return;
    const int slot = __builtin_amdgcn_readfirstlane(slot0 + before);
    if (lane == 0) {
        pass.cnorm_changed[slot] = acc;
        pass.which_changed[slot] = j;
    }
    uint4 *const cc = reinterpret_cast<uint4 *>(pass.cp_changed);
    for (int x = lane; x < X; x += 64) cc[place(slot, x)] = x < pieces ? row[x] : make_uint4(0, 0, 0, 0);
}

// rows-in-LDS membership kernel: wavefronts per workgroup, centroid groups per step, row tiles per item
constexpr int KL_NW = 8;
constexpr int KL_G = 2;
constexpr int km_lds_row_tiles(int kt) { return kt > 32 ? 3 : 4; }

// Whether a later pass is worth taking apart (below): with more centroids changed, nearly every vector meets
// nearly all of them again.
__device__ inline bool few_changed(int changed, int K) { return 5 * changed <= 2 * K; }

// Membership of many vectors at once: Eq. 2 as a GEMM.  One workgroup takes 64 vectors and
// all centroids.  As in the GEMM-shaped projection kernel the k-extent is split over the four
// wavefronts, each keeping its slice of the 64 vectors in registers in MFMA operand order and
// streaming its slice of every packed centroid tile (the centroids stay in the caches), so
// each 1 KiB load feeds four MFMAs; the partial inner products of a group of 16 centroids meet
// in LDS and wavefront w keeps the running (min, argmin) of vector tile w.
// A pass in which few centroids changed takes the vectors in another order: those whose own centroids changed in front
// (PARTED: kmeans_assign_lds_kernel has parted them), or else as the first pass placed them, members of a cluster
// side by side.  64 vectors none of whose own centroids changed meet the changed centroids only, and
// each keeps its cluster where its old score is not beaten (ties to the lowest number, as everywhere); it is then
// the vectors' bytes that take the time.  131,072 vectors, 1,000 clusters, d = 1024, us per pass: all centroids 310 (rows-in-LDS kernel),
// 68 changed ones 130, two 99.
template <int KW, bool RANK, bool PARTED>
__device__ __forceinline__ void assign_split_k(const uint4 *__restrict__ X, long n, int d, int K, int ctiles, const VpKmPass &pass)
{
    constexpr int KT = KW * 4;
    constexpr int RT = 4;
    const bool first = pass.first != 0;
    const int changed = first ? K : pass.state->changed;
    const bool few = !first && few_changed(changed, K);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int nn = lane & 15;
    const int q = lane >> 4;
    __shared__ floatx4 xbuf[2 * RT * 4 * 64];

    const long r0 = (long)blockIdx.x * (16 * RT);
    const int pieces_per_row = d >> 3;
    bool all = true;
    const uint4 *tiles = reinterpret_cast<const uint4 *>(pass.cp) + (size_t)wave * KW * 64 + lane;
    const float *cnorm = pass.cnorm;
    int nc = K, groups = ctiles;
    Frag Xb[KW], Yb[KW];
    auto issue = [&](Frag(&buf)[KW], int g) {
        const uint4 *p = tiles + (size_t)g * KT * 64;
#pragma unroll
        for (int i = 0; i < KW; ++i) buf[i].u = p[i * 64];
    };
    Frag B[RT][KW];
    auto fetch_vectors = [&](auto vector_of) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const long row = vector_of(rt * 16 + nn);
#pragma unroll
            for (int i = 0; i < KW; ++i) {
                const int piece = (wave * KW + i) * 4 + q;
                B[rt][i].u = make_uint4(0, 0, 0, 0);
                if (row >= 0 && piece < pieces_per_row) B[rt][i].u = X[(size_t)row * pieces_per_row + piece];
            }
        }
    };
    int vec = -1;   // lane l's vector of the 64, in a pass that is taken apart
    if (!few) {
        issue(Xb, 0);
        if (1 < groups) issue(Yb, 1);
        fetch_vectors([&](int slot) { return r0 + slot < n ? r0 + slot : -1l; });
    } else {
        if (r0 + lane < n) vec = (PARTED ? pass.parted : pass.order)[r0 + lane];
        fetch_vectors([&](int slot) { return (long)__shfl(vec, slot); });
        if (PARTED) all = r0 < pass.state->unsettled;
        else all = __ballot(vec >= 0 && pass.flag[pass.assign[max(vec, 0)]] != 0) != 0;   // (the same in every wavefront)
        if (!all) {
            tiles = reinterpret_cast<const uint4 *>(pass.cp_changed) + (size_t)wave * KW * 64 + lane;
            cnorm = pass.cnorm_changed;
            nc = changed;
            groups = (changed + 15) >> 4;
        }
        issue(Xb, 0);
        if (1 < groups) issue(Yb, 1);
    }

    float best_s = __builtin_inff();
    int best_j = -1;               // (a score of +infinity is never taken)
    floatx4 acc[RT];
    auto compute = [&](Frag(&buf)[KW], int gnext) {
        const bool more = gnext < groups;
        const uint4 *p = tiles + (size_t)gnext * KT * 64;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            Frag a;
            a.u = buf[i].u;
            if (more) buf[i].u = p[i * 64];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, B[rt][i].h,
                                                                 i == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[rt], 0, 0, 0);
        }
    };
    auto finish = [&](int g, int par) {
        floatx4 *xw = xbuf + (size_t)par * RT * 4 * 64;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) xw[(rt * 4 + wave) * 64 + lane] = acc[rt];
        const float4 cn = *reinterpret_cast<const float4 *>(cnorm + g * 16 + q * 4);
        int4 which = make_int4(0, 0, 0, 0);
        if (!all) which = *reinterpret_cast<const int4 *>(pass.which_changed + g * 16 + q * 4);
        __syncthreads();
        const floatx4 dot = (xw[(wave * 4 + 0) * 64 + lane] + xw[(wave * 4 + 1) * 64 + lane]) +
                            (xw[(wave * 4 + 2) * 64 + lane] + xw[(wave * 4 + 3) * 64 + lane]);
        const float cnv[4] = {cn.x, cn.y, cn.z, cn.w};
        if (all) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = g * 16 + q * 4 + i;
                const float s = cnv[i] - 2.0f * dot[i];
                if (j < K && s < best_s) {   // j ascends within a lane: strict < keeps the lowest
                    best_s = s;
                    best_j = j;
                }
            }
        } else {
            const int num[4] = {which.x, which.y, which.z, which.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // (in any order)
                const float s = cnv[i] - 2.0f * dot[i];
                const bool take = (g * 16 + q * 4 + i < nc) & ((s < best_s) | ((s == best_s) & (num[i] < best_j)));
                best_s = take ? s : best_s;
                best_j = take ? num[i] : best_j;
            }
        }
    };
    int g = 0, par = 0;
    while (g < groups) {
        compute(Xb, g + 2);
        finish(g, par);
        par ^= 1;
        ++g;
        if (g >= groups) break;
        compute(Yb, g + 2);
        finish(g, par);
        par ^= 1;
        ++g;
    }
    if (best_j < 0) best_j = VP_IDX_NONE;
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const float s2 = __shfl_xor(best_s, off);
        const int j2 = __shfl_xor(best_j, off);
        if (part_less(s2, j2, best_s, best_j)) {
            best_s = s2;
            best_j = j2;
        }
    }
    long row = r0 + wave * 16 + nn;
    if (few) row = __shfl(vec, wave * 16 + nn);
    if (q == 0 && row >= 0 && row < n) {
        if (!all) {
            const float old_s = pass.best[row];
            const int old_j = pass.assign[row];
            if (!part_less(best_s, best_j, old_s, old_j)) {
                best_s = old_s;
                best_j = old_j;
            }
        }
        if ((unsigned)best_j >= (unsigned)K) best_j = 0;   // only when every score is NaN
        pass.best[row] = best_s;
        record_member<RANK>(pass, row, best_j);
    }
}

template <int KW, bool RANK>
__global__ __launch_bounds__(256, (KW <= 8 ? 2 : 1)) void kmeans_assign_gemm_kernel(const uint4 *__restrict__ X, long n, int d,
                                                                                    int K, int ctiles, VpKmPass pass)
{
    if (!pass.first && pass.state->changed == 0) return;   // nobody moves
    assign_split_k<KW, RANK, false>(X, n, d, K, ctiles, pass);
}

// The later passes of a call whose passes over everything run on the rows-in-LDS kernel: those in which few centroids changed,
// with more vectors than that kernel takes in two rounds.  The vectors whose own centroids changed meet all centroids
// here, one group behind the other, so the kernel takes about as long as a pass over everything takes it, however few they
// are, and the rows-in-LDS kernel needs half of that for a round.  20 iterations in which five or so still change centroids, us, these
// passes here / on the rows-in-LDS kernel: d = 1024, 2,000 clusters: 8,192 vectors 1,135 / 772, 16,384 1,620 / 1,146, 32,768
// 1,366 / 1,377, 65,536 1,646 / 2,034; 260 clusters: 384 / 378 at 4,096, 517 / 531 at 32,768, 821 / 915 at 65,536; d = 1536, 1,000
// clusters: 8,192 827 / 603, 24,576 780 / 786, 32,768 789 / 822; d = 512, 1,000 clusters: 16,384 492 / 402, 65,536 652 / 673.
bool takes_passes_apart(int kt, long n) { return n > 2 * 256 * 16l * km_lds_row_tiles(kt); }

template <int KW, bool RANK>
__global__ __launch_bounds__(256, (KW <= 8 ? 2 : 1)) void kmeans_reassign_kernel(const uint4 *__restrict__ X, long n, int d,
                                                                                 int K, int ctiles, VpKmPass pass)
{
    const int changed = pass.state->changed;
    if (changed == 0 || !few_changed(changed, K)) return;
    assign_split_k<KW, RANK, true>(X, n, d, K, ctiles, pass);
}

// Parts the vectors for the kernel above: those whose own centroids changed from the front of the list, the others from
// its end (in no particular order).  Called by all workgroups of a grid of `threads` threads each; one pair of
// atomics per workgroup and chunk.
__device__ inline void part_vectors(long n, const VpKmPass &pass, int *lds, int threads)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = threads >> 6;
    for (long c0 = (long)blockIdx.x * threads; c0 < n; c0 += (long)gridDim.x * threads) {
        const long r = c0 + tid;
        const bool is = r < n;
        const bool unsettled = is && pass.flag[pass.assign[is ? r : 0]] != 0;
        const unsigned long long u = __ballot(unsettled), v = __ballot(is && !unsettled);
        if (lane == 0) {
            lds[wave] = __popcll(u);
            lds[waves + wave] = __popcll(v);
        }
        __syncthreads();
        if (tid < 2) {
            int sum = 0;
            for (int w = 0; w < waves; ++w) {   // counts -> where each wavefront's vectors start in the workgroup's share
                const int c = lds[tid * waves + w];
                lds[tid * waves + w] = sum;
                sum += c;
            }
            lds[2 * waves + tid] = sum ? atomicAdd(tid == 0 ? &pass.state->unsettled : &pass.state->settled, sum) : 0;
        }
        __syncthreads();
        const unsigned long long below = (1ull << lane) - 1;
        if (unsettled) pass.parted[lds[2 * waves] + lds[wave] + __popcll(u & below)] = (int32_t)r;
        else if (is) pass.parted[n - 1 - (lds[2 * waves + 1] + lds[waves + wave] + __popcll(v & below))] = (int32_t)r;
        __syncthreads();   // lds is written again
    }
}

// A membership pass over all vectors and centroids with the vectors held in LDS (d_pad = 512 to 1536): the split-k kernel above
// meets in LDS behind a barrier for every 16 centroids, which leaves the matrix cores idle most of the time.
// An item is 64 vectors (48 at d_pad = 1280 and 1536, where 64 do not fit) against all centroids; eight wavefronts walk
// steps of two groups of 16 centroids on their own (w, w + 8, ...), the centroid tiles streaming
// from the L2 through a ring of k-tiles that runs across steps and items, the vectors' operands
// from LDS; no barrier but the two of an item.  A workgroup owns its compute unit and walks
// items, and during an item's last step it touches the next item's vectors, so that staging them finds them in
// the L2.  Every sum is formed as the split-k kernel forms it - four quarters of the k-extent, each a chain of its own
// from zero, added as (s0 + s1) + (s2 + s3) - so the memberships are the same to the bit; two groups, not
// four, because three sets of accumulators must fit the registers.
// Ten iterations of vp_kmeans with it in every pass, us per iteration, split-k kernel -> this one: 131,072 vectors x 1,000 clusters
// d = 1024: 417 -> 405, d = 512: 312 -> 274, d = 1536: 892 -> 746; 6,000 x 1,000, d = 1024: 108 -> 77;
// 4,099 x 1,000, d = 512: 84 -> 52.  (Steps of three groups spill: 526 at the first.)
template <int KT, bool RANK>
__global__ __launch_bounds__(KL_NW * 64) void kmeans_assign_lds_kernel(const uint4 *__restrict__ X, long n, int d, int K,
                                                                       int ctiles, int nitems, VpKmPass pass)
{
    const bool first = pass.first != 0;
    extern __shared__ uint4 lds[];        // [RT][KT][64]: the vectors in MFMA operand order
    if (!first) {
        const int changed = pass.state->changed;
        if (changed == 0) return;   // nobody moves
        if (pass.apart && few_changed(changed, K)) {   // kmeans_reassign_kernel takes the pass
            part_vectors(n, pass, reinterpret_cast<int *>(lds), KL_NW * 64);
            return;
        }
    }
    const uint4 *const cp = reinterpret_cast<const uint4 *>(pass.cp);
    const float *const cnorm = pass.cnorm;
    constexpr int RT = km_lds_row_tiles(KT);
    constexpr int ROWS = 16 * RT;
    constexpr int G = KL_G;
    constexpr int KW = KT / 4;            // k-tiles per quarter
    constexpr int PF = KW % 4 == 0 ? 4 : KW / 2;   // k-tiles in flight
    constexpr int XP = KT * 4;            // 16-byte pieces per padded vector
    constexpr int THREADS = KL_NW * 64;
    constexpr int PER = ROWS * XP / THREADS;
    constexpr int TOUCH = (ROWS * XP / 8 + THREADS - 1) / THREADS;   // 128-byte lines per thread
    static_assert(PER * THREADS == ROWS * XP && KW % PF == 0, "whole pieces and passes");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int nn = lane & 15;
    const int q = lane >> 4;
    float *red_s = reinterpret_cast<float *>(lds + RT * KT * 64);   // [KL_NW][ROWS]
    int *red_j = reinterpret_cast<int *>(red_s + KL_NW * ROWS);      // [KL_NW][ROWS]

    const int nsteps = (ctiles + G - 1) / G;   // >= KL_NW: every wavefront has a step
    const int pieces_per_row = d >> 3;
    const uint4 *tiles = cp + lane;
    // groups past the last one repeat it (their centroid numbers are >= K: never looked at)
    auto group_off = [&](int step, unsigned int (&off)[G]) {
#pragma unroll
        for (int j = 0; j < G; ++j) off[j] = (unsigned int)min(step * G + j, ctiles - 1) * (KT * 64);
    };
    unsigned int cur[G], nxt[G];
    uint4 ring[PF][G];
    group_off(wave, cur);
#pragma unroll
    for (int p = 0; p < PF; ++p)
#pragma unroll
        for (int j = 0; j < G; ++j) ring[p][j] = tiles[cur[j] + p * 64];

    int before = 0, before_old = 0;   // this thread's vector of the item before: the numbers its atomics returned
    long before_row = -1;
    for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
        const long r0 = (long)item * ROWS;
        {
            int t = tid;
            asm volatile("" : "+v"(t));   // the pieces' addresses are formed here, not kept in registers across the items
            uint4 piece[PER];
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int e = t + i * THREADS;
                const int r = e / XP;
                const int x = e - r * XP;
                // (without branches; vectors past the last repeat it and are never looked at)
                const uint4 v = X[(size_t)min(r0 + r, n - 1) * pieces_per_row + min(x, pieces_per_row - 1)];
                piece[i] = x < pieces_per_row ? v : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int e = t + i * THREADS;
                const int r = e / XP;
                const int x = e - r * XP;
                lds[((r >> 4) * KT + (x >> 2)) * 64 + (x & 3) * 16 + (r & 15)] = piece[i];
            }
        }
        // (the item before: its atomics have come back with the vectors)
        if (RANK && before_row >= 0) {
            pass.rank[before_row] = before;
            if (!first) pass.rank_old[before_row] = before_old;
        }
        before_row = -1;
        int old = 0;
        if (!first && tid < ROWS && r0 + tid < n) old = pass.assign[r0 + tid];   // (fetched well before it is compared)
        __syncthreads();   // the vectors are staged; red_* of the item before has been read

        float best_s[RT];
        int best_j[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            best_s[rt] = __builtin_inff();
            best_j[rt] = VP_IDX_NONE;
        }
        uint32_t touched[TOUCH];
#pragma unroll
        for (int i = 0; i < TOUCH; ++i) touched[i] = 0;
        uint4 bnext[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) bnext[rt] = lds[(rt * KT) * 64 + lane];

#pragma unroll 1
        for (int step = wave; step < nsteps; step += KL_NW) {
            const bool last_step = step + KL_NW >= nsteps;
            group_off(last_step ? wave : step + KL_NW, nxt);
            if (last_step && item + (int)gridDim.x < nitems) {
                const long r1 = r0 + (long)gridDim.x * ROWS;
                const long lines = min((long)ROWS, n - r1) * pieces_per_row;   // in pieces; the vectors are contiguous
                const uint32_t *nx = reinterpret_cast<const uint32_t *>(X + (size_t)r1 * pieces_per_row);
#pragma unroll
                for (int i = 0; i < TOUCH; ++i) {
                    const int e = (tid + i * THREADS) * 8;
                    if (e < lines) touched[i] = __hip_atomic_load(nx + (size_t)e * 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            auto quarter = [&](floatx4 (&acc)[RT][G], int sl) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int j = 0; j < G; ++j) acc[rt][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int b = 0; b < KW / PF; ++b) {
                    const int kt0 = sl * KW + b * PF;
                    const bool last = kt0 + PF == KT;
                    unsigned int src[G];
#pragma unroll
                    for (int j = 0; j < G; ++j) src[j] = last ? nxt[j] : cur[j] + (kt0 + PF) * 64;
#pragma unroll
                    for (int u = 0; u < PF; ++u) {
                        // the operands of the next k-tile are read in front of this k-tile's MFMAs and the ring
                        // slot is refilled behind them; the scheduling barriers keep both where they are
                        Frag bf[RT];
                        const int kt_next = kt0 + u + 1 == KT ? 0 : kt0 + u + 1;
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) {
                            bf[rt].u = bnext[rt];
                            bnext[rt] = lds[(rt * KT + kt_next) * 64 + lane];
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                            for (int j = 0; j < G; ++j) {
                                Frag a;
                                a.u = ring[u][j];
                                acc[rt][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, bf[rt].h, acc[rt][j], 0, 0, 0);
                            }
#pragma unroll
                        for (int j = 0; j < G; ++j) ring[u][j] = tiles[src[j] + u * 64];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            floatx4 dot[RT][G], s1[RT][G], s2[RT][G];
            quarter(dot, 0);
            quarter(s1, 1);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int j = 0; j < G; ++j) dot[rt][j] = dot[rt][j] + s1[rt][j];
            quarter(s1, 2);
            quarter(s2, 3);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int g = step * G + j;
                const float4 cn = *reinterpret_cast<const float4 *>(cnorm + min(g, ctiles - 1) * 16 + q * 4);
                const float cnv[4] = {cn.x, cn.y, cn.z, cn.w};
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const floatx4 t = dot[rt][j] + (s1[rt][j] + s2[rt][j]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int c = g * 16 + q * 4 + i;
                        const float s = cnv[i] - 2.0f * t[i];
                        const bool take = (c < K) & (s < best_s[rt]);   // c ascends within a lane: strict < keeps the lowest
                        best_s[rt] = take ? s : best_s[rt];
                        best_j[rt] = take ? c : best_j[rt];
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < G; ++j) cur[j] = nxt[j];
        }
#pragma unroll
        for (int i = 0; i < TOUCH; ++i) asm volatile("" ::"v"(touched[i]));   // (the touching loads have a use)

#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
            for (int off = 16; off <= 32; off <<= 1) {
                const float s2 = __shfl_xor(best_s[rt], off);
                const int j2 = __shfl_xor(best_j[rt], off);
                const bool take = part_less(s2, j2, best_s[rt], best_j[rt]);
                best_s[rt] = take ? s2 : best_s[rt];
                best_j[rt] = take ? j2 : best_j[rt];
            }
            if (q == 0) {
                red_s[wave * ROWS + rt * 16 + nn] = best_s[rt];
                red_j[wave * ROWS + rt * 16 + nn] = best_j[rt];
            }
        }
        __syncthreads();   // nobody reads the vectors any more; red_* is complete
        if (tid < ROWS && r0 + tid < n) {
            float bs = red_s[tid];
            int bj = red_j[tid];
#pragma unroll
            for (int w = 1; w < KL_NW; ++w) {
                const float s2 = red_s[w * ROWS + tid];
                const int j2 = red_j[w * ROWS + tid];
                if (part_less(s2, j2, bs, bj)) {
                    bs = s2;
                    bj = j2;
                }
            }
            if ((unsigned)bj >= (unsigned)K) bj = 0;   // only when every score is NaN
            const long row = r0 + tid;
            pass.best[row] = bs;
            if (first) {
                pass.assign[row] = bj;
                if (RANK) {
                    before = atomicAdd(&pass.counts[bj], 1);
                    before_row = row;
                } else {
                    atomicAdd(&pass.counts[bj], 1);
                }
            } else {
                pass.prev[row] = old;
                if (bj != old) {
                    pass.assign[row] = bj;
                    atomicAdd(&pass.counts[bj], 1);
                    atomicSub(&pass.counts[old], 1);
                    if (RANK) {
                        before = atomicAdd(&pass.events[bj], 1);
                        before_old = atomicAdd(&pass.events[old], 1);
                        before_row = row;
                    } else {
                        atomicAdd(&pass.events[bj], 1);
                        atomicAdd(&pass.events[old], 1);
                    }
                }
            }
        }
    }
    if (RANK && before_row >= 0) {
        pass.rank[before_row] = before;
        if (!first) pass.rank_old[before_row] = before_old;
    }
}

template <int KT>
constexpr size_t km_lds_bytes()
{
    constexpr int rows = 16 * km_lds_row_tiles(KT);
    constexpr size_t bytes = (size_t)rows * KT * 64 + (size_t)KL_NW * rows * 8;
    static_assert(bytes <= 160 * 1024, "vectors and reduction fit the LDS");
    return bytes;
}

template <int KT>
hipError_t prepare_assign_lds()
{
    const int bytes = (int)km_lds_bytes<KT>();
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kmeans_assign_lds_kernel<KT, false>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kmeans_assign_lds_kernel<KT, true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <int KT>
void launch_assign_lds(const void *X, long n, int d, int K, int ctiles, const VpKmPass &pass, hipStream_t st)
{
    constexpr int rows = 16 * km_lds_row_tiles(KT);
    const int nitems = (int)((n + rows - 1) / rows);
    const auto kernel = pass.rank ? kmeans_assign_lds_kernel<KT, true> : kmeans_assign_lds_kernel<KT, false>;
    hipLaunchKernelGGL(kernel, dim3(std::min(nitems, 256)), dim3(KL_NW * 64), km_lds_bytes<KT>(), st, (const uint4 *)X, n,
                       d, K, ctiles, nitems, pass);
}

// Whether the rows-in-LDS kernel is the faster one for the membership of n vectors.  From 16 groups of centroids on each
// of its eight wavefronts has a step of two groups.  With a few groups more some wavefronts take a second step and the
// others wait, and just past whole rounds of 256 items most of the chip waits; the split-k kernel has no steps to hand
// out, and its workgroups come 512 (d_pad 1536: 256) at a time.  The kernel stays ahead of either loss but not of both.  The lines are
// where the two cross on 1,500 sizes of 241 to 1,300 clusters and 4,096 to 131,072 vectors; us per call without
// iterations, split-k kernel -> this one:
//   d_pad 1024, 288 clusters: 16,384 vectors 45 -> 39, 16,400 47 -> 50, 26,000 55 -> 53, 49,200 85 -> 94, 82,000 120 -> 135;
//     384 clusters: 49 -> 42, 49 -> 49, 59 -> 53, 94 -> 88, 136 -> 136; 1,000 clusters: 16,400 82 -> 77, 131,072 321 -> 303
//   d_pad 1536 (48 vectors an item here, 64 there), 288 clusters: 12,288 vectors 49 -> 42, 12,290 47 -> 55, 16,500 72 -> 57,
//     25,000 80 -> 83, 131,072 293 -> 280; 480 clusters: 61 -> 47, 59 -> 63, 97 -> 64, 102 -> 90, 394 -> 315
//   d_pad 512: faster everywhere (288 clusters: 16,400 36 -> 31, 131,072 140 -> 116)
//   d_pad 768 and 1280 with the lines of 1024 and 1536: nowhere slower (0.56 to 0.99 and 0.55 to 0.95 of the time)
bool rows_in_lds_faster(int kt, int ctiles, long n)
{
    if (ctiles < KL_NW * KL_G || (kt != 16 && kt != 24 && kt != 32 && kt != 40 && kt != 48)) return false;
    const long rows = 16 * km_lds_row_tiles(kt);
    const long items = (n + rows - 1) / rows;
    if (kt == 16 || items <= 256) return true;
    if (kt == 24 || kt == 32) {
        // a last round of 256 that is up to half full, where the other kernel's last round of 512 is as well
        const long last = items % 512;
        const bool uneven = ctiles > 16 && ctiles <= (items <= 512 ? 27 : 19);
        return !(uneven && last > 256 && last <= (items <= 512 ? 320 : 384));
    }
    // two rounds here and one there; three rounds and hardly two
    if (n <= 64 * 256) return ctiles > 30;
    return !(ctiles > 16 && ctiles <= 19 && items > 512 && n <= 64 * 440);
}

// Where the members (first pass) or the events of the clusters go: every workgroup adds the counts up for itself (they
// are a few kilobytes; a kernel of its own for that costs 4 us a pass), then writes its vectors' entries into cluster order
// (the order inside a cluster is arbitrary: the sums are exact).  An entry is a vector's number, its highest bit set where
// the vector left the cluster.  With the numbers of the counting atomics an entry's place is known; without, a workgroup
// counts its own vectors in LDS and takes a run of places from every cluster's cursor (131,072 vectors, first pass: 1,000
// clusters 5 us with the numbers; 200 clusters 6.5 us with the runs, 115 with an atomic for every vector).
// Where more than half of the vectors moved, the sums are begun anew from all members.
constexpr int PLACE_THREADS = 1024;
__global__ __launch_bounds__(PLACE_THREADS) void kmeans_place_kernel(long n, int K, VpKmPass pass, int32_t *__restrict__ start,
                                                                     int32_t *__restrict__ list,
                                                                     unsigned long long *__restrict__ acc, size_t acc_n)
{
    extern __shared__ int base[];   // [K + 1]
    int *const mine = base + K + 1; // [K] this workgroup's members, then the first place of their run
    __shared__ int wsum[PLACE_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool first = pass.first != 0;
    auto scan = [&](const int32_t *v) {
        uint32_t carry = 0;   // (events: up to 2 n)
        for (int j0 = 0; j0 < K; j0 += PLACE_THREADS) {
            const int j = j0 + tid;
            const int c = j < K ? v[j] : 0;
            const int inc = wave_inclusive_sum(c);
            __syncthreads();   // wsum has been read
            if (lane == 63) wsum[wave] = inc;
            __syncthreads();
            const int w = wave_inclusive_sum(lane < PLACE_THREADS / 64 ? wsum[lane] : 0);
            const int below = wave ? __builtin_amdgcn_readlane(w, wave - 1) : 0;
            if (j < K) base[j] = (int)(carry + (uint32_t)below + (uint32_t)inc - (uint32_t)c);
            carry += (uint32_t)__builtin_amdgcn_readlane(w, PLACE_THREADS / 64 - 1);
        }
        if (tid == 0) base[K] = (int)carry;
        __syncthreads();
        return carry;
    };
    const uint32_t total = scan(first ? pass.counts : pass.events);
    const bool anew = first || vp_sums_begin_anew(total, n);
    if (blockIdx.x == 0 && tid == 0) {
        pass.state->total_events = total;
        pass.state->anew = anew;
        pass.state->changed = 0;   // (read by the membership pass before, counted again by the next one's preparation)
        if (first) pass.state->split = 0;
    }
    // (without events the means of split clusters are still to be written again)
    if (total == 0 && !(pass.was_split && pass.state->split)) return;
    if (anew && !first) scan(pass.counts);
    if (blockIdx.x == 0)
        for (int j = tid; j <= K; j += PLACE_THREADS) start[j] = base[j];
    if (total == 0) return;
    if (anew && !first)
        for (size_t e = (size_t)blockIdx.x * PLACE_THREADS + tid; e < acc_n; e += (size_t)gridDim.x * PLACE_THREADS) acc[e] = 0ull;
    const long r = (long)blockIdx.x * PLACE_THREADS + tid;
    const bool is = r < n;
    const int j = is ? pass.assign[r] : 0;
    if (anew && first && pass.rank) {
        if (is) list[base[j] + pass.rank[r]] = (int32_t)r;
        return;
    }
    if (anew) {
        for (int c = tid; c < K; c += PLACE_THREADS) mine[c] = 0;
        __syncthreads();
        const int local = is ? atomicAdd(&mine[j], 1) : 0;
        __syncthreads();
        for (int c = tid; c < K; c += PLACE_THREADS)
            if (mine[c]) mine[c] = atomicAdd(&pass.cursor[c], mine[c]);
        __syncthreads();
        if (is) list[base[j] + mine[j] + local] = (int32_t)r;
        return;
    }
    if (!is) return;
    const int old = pass.prev[r];
    if (j == old) return;
    list[base[j] + (pass.rank ? pass.rank[r] : atomicAdd(&pass.cursor[j], 1))] = (int32_t)r;
    list[base[old] + (pass.rank ? pass.rank_old[r] : atomicAdd(&pass.cursor[old], 1))] = (int32_t)((uint32_t)r | 0x80000000u);
}

// Running sums of 8 coordinates.  They are kept in double precision: every binary16 value is
// a multiple of 2^-24, so while a sum stays below 2^29 in magnitude every addition is exact and
// the order of the additions does not matter.  Where sums of different threads meet they are
// added as 64-bit integers in units of 2^-24 (exact conversions), which keeps that true under
// atomics.
typedef _Float16 half2t __attribute__((ext_vector_type(2)));

// entry: a vector's number; where they are EVENTS its highest bit takes the vector away (its signs are turned)
template <bool EVENTS>
__device__ inline void add_units(double (&s)[8], const uint4 v, uint32_t entry)
{
    const uint32_t turn = EVENTS ? (entry >> 31) * 0x80008000u : 0u;
    const uint32_t w[4] = {v.x ^ turn, v.y ^ turn, v.z ^ turn, v.w ^ turn};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const half2t h = __builtin_bit_cast(half2t, w[e]);
        s[2 * e] += (double)(float)h[0];
        s[2 * e + 1] += (double)(float)h[1];
    }
}

__device__ inline unsigned long long to_units(double sum) { return (unsigned long long)(long long)(sum * 0x1p24); }

// Sum of the entries [first, last) taken every `step`-th, coordinates 8 * piece and following; returns where it ended.
// Members add up exactly by the bound on x.  EVENTS may be the members of two passes together: at most
// VP_KM_EXACT_ENTRIES of them at a time.
template <bool EVENTS>
__device__ inline int sum_entries(double (&s)[8], const uint4 *__restrict__ X, int pieces, int piece,
                                  const int32_t *__restrict__ list, int first, int last, int step)
{
    int m = first;
    if (EVENTS && last - first > VP_KM_EXACT_ENTRIES * step) last = first + VP_KM_EXACT_ENTRIES * step;
    for (; m + 7 * step < last; m += 8 * step) {
        // entries first, then all eight rows: written as one expression the loads of an entry and of its row
        // alternate and every one waits for the one before
        uint32_t r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = (uint32_t)list[m + u * step];
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = X[(size_t)(r[u] & 0x7fffffffu) * pieces + piece];
#pragma unroll
        for (int u = 0; u < 8; ++u) add_units<EVENTS>(s, v[u], r[u]);
    }
    for (; m < last; m += step) {
        const uint32_t r = (uint32_t)list[m];
        add_units<EVENTS>(s, X[(size_t)(r & 0x7fffffffu) * pieces + piece], r);
    }
    return m;
}

// Sum of the entries of cluster blockIdx.x that fall to this workgroup (every `splits`-th one
// starting at blockIdx.y), added to the sums in memory.  A thread owns one 16-byte piece (8 coordinates) of the vectors;
// when a vector has fewer than 256 pieces the workgroup's threads form several member lanes that take
// the workgroup's entries in turn.  Eight rows are in flight per thread.
__global__ __launch_bounds__(256) void kmeans_sum_kernel(const uint4 *__restrict__ X, int pieces,
                                                         const int32_t *__restrict__ list,
                                                         const int32_t *__restrict__ start, int splits,
                                                         unsigned long long *__restrict__ acc, const VpKmState *__restrict__ state)
{
    if (state->total_events == 0) return;
    const int j = blockIdx.x;
    const int m0 = start[j], m1 = start[j + 1];
    const int lanes = pieces <= 128 ? 256 / pieces : 1;       // member lanes per workgroup
    const int ml = lanes > 1 ? threadIdx.x / pieces : 0;       // this thread's member lane
    if (m0 + (int)blockIdx.y * lanes >= m1) return;            // nothing falls to this workgroup
    __shared__ unsigned long long lsum[128 * 8];
    if (lanes > 1) {
        for (int e = threadIdx.x; e < pieces * 8; e += 256) lsum[e] = 0ull;
        __syncthreads();
    }
    const int step = splits * lanes;
    const int first = m0 + blockIdx.y * lanes + ml;
    for (int piece = lanes > 1 ? threadIdx.x - ml * pieces : threadIdx.x; piece < pieces && ml < lanes; piece += 256) {
        int m = first;
        do {
            double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (state->anew) m = sum_entries<false>(s, X, pieces, piece, list, m, m1, step);
            else m = sum_entries<true>(s, X, pieces, piece, list, m, m1, step);
            if (lanes > 1) {
                // the member lanes meet in LDS; one global addition per coordinate and workgroup
                unsigned long long *slot = lsum + (size_t)piece * 8;
#pragma unroll
                for (int e = 0; e < 8; ++e) atomicAdd(slot + e, to_units(s[e]));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) atomicAdd(&acc[((size_t)j * pieces + piece) * 8 + e], to_units(s[e]));
            }
        } while (m < m1);
    }
    if (lanes > 1) {
        __syncthreads();
        for (int e = threadIdx.x; e < pieces * 8; e += 256) atomicAdd(&acc[(size_t)j * pieces * 8 + e], lsum[e]);
    }
}

// double -> binary16 bits, round to nearest, ties to even (integer arithmetic on the bits).
__host__ __device__ inline uint16_t double_to_half_bits(double v)
{
    unsigned long long b;
    __builtin_memcpy(&b, &v, sizeof(b));
    const uint16_t sign = (uint16_t)((b >> 48) & 0x8000);
    const int ex = (int)((b >> 52) & 0x7ff);
    const unsigned long long man = b & ((1ull << 52) - 1);
    if (ex == 0x7ff) return (uint16_t)(sign | (man ? 0x7e00 : 0x7c00));
    if (ex == 0) return sign;                                   // zero (and double subnormals)
    const int e = ex - 1023;
    if (e > 15) return (uint16_t)(sign | 0x7c00);
    unsigned long long q, rem, half;
    uint32_t base;
    if (e >= -14) {                                             // normal binary16 range
        q = man >> 42;
        rem = man & ((1ull << 42) - 1);
        half = 1ull << 41;
        base = (uint32_t)(e + 15) << 10;
    } else {                                                    // multiples of 2^-24
        const int shift = 28 - e;                               // >= 43
        if (shift > 63) return sign;
        const unsigned long long full = man | (1ull << 52);
        q = full >> shift;
        rem = full & ((1ull << shift) - 1);
        half = 1ull << (shift - 1);
        base = 0;
    }
    uint32_t h = base + (uint32_t)q;
    if (rem > half || (rem == half && (q & 1))) h += 1;        // a carry moves into the exponent field
    if (h >= 0x7c00) h = 0x7c00;
    return (uint16_t)(sign | h);
}

// Without events the centroids are the means already, but for those that a split moved (kmeans_split_kernel).
// (was_split: null where empty clusters are left alone)
__device__ inline bool nothing_to_update(const VpKmState *state, const int32_t *was_split)
{
    return state->total_events == 0 && !(was_split && state->split);
}

// One workgroup per cluster: brings the cluster's sum up to date with its entries and writes the new centroid at once
// (no atomics between workgroups).  Used when there are enough clusters to fill
// the chip this way; the member lanes of the workgroup (two at least) meet in LDS.
constexpr int MEAN_THREADS = 1024;
static_assert(VP_KM_MAX_PIECES <= MEAN_THREADS / 2, "two member lanes at the largest width");
__global__ __launch_bounds__(MEAN_THREADS) void kmeans_mean_kernel(const uint4 *__restrict__ X, int pieces,
                                                          const int32_t *__restrict__ list,
                                                          const int32_t *__restrict__ start,
                                                          const int32_t *__restrict__ counts,
                                                          unsigned long long *__restrict__ acc,
                                                          const VpKmState *__restrict__ state,
                                                          const int32_t *__restrict__ was_split, uint4 *__restrict__ C)
{
    if (nothing_to_update(state, was_split)) return;
    const int j = blockIdx.x;
    const int m0 = start[j], m1 = start[j + 1];
    const bool anew = state->anew != 0;
    unsigned long long *const sum = acc + (size_t)j * pieces * 8;
    if (m0 == m1 && !(was_split && state->split && was_split[j])) {         // nobody came or went: the centroid stays
        if (anew)
            for (int e = threadIdx.x; e < pieces * 8; e += MEAN_THREADS) sum[e] = 0ull;
        return;
    }
    const int lanes = MEAN_THREADS / pieces;                   // member lanes
    const int ml = threadIdx.x / pieces;
    __shared__ unsigned long long lsum[(MEAN_THREADS / 2) * 8];
    for (int e = threadIdx.x; e < pieces * 8; e += MEAN_THREADS) lsum[e] = anew ? 0ull : sum[e];
    __syncthreads();
    const int piece = threadIdx.x - ml * pieces;
    if (ml < lanes && m0 + ml < m1) {
        int m = m0 + ml;
        do {
            double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (anew) m = sum_entries<false>(s, X, pieces, piece, list, m, m1, lanes);
            else m = sum_entries<true>(s, X, pieces, piece, list, m, m1, lanes);
#pragma unroll
            for (int e = 0; e < 8; ++e) atomicAdd(lsum + (size_t)piece * 8 + e, to_units(s[e]));
        } while (m < m1);
    }
    __syncthreads();
    const int c = counts[j];
    for (int p = threadIdx.x; p < pieces; p += MEAN_THREADS) {
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned long long v = lsum[p * 8 + e];
            sum[p * 8 + e] = v;
            h[e] = double_to_half_bits((double)(long long)v * 0x1p-24 / (double)c);
        }
        // (a cluster without members keeps its centroid)
        if (c > 0)
            C[(size_t)j * pieces + p] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                                                   h[6] | (h[7] << 16));
    }
}

// New centroids from the sums in memory, of the clusters with events and of those that were split.
__global__ __launch_bounds__(256) void kmeans_update_kernel(const unsigned long long *__restrict__ acc,
                                                            const int32_t *__restrict__ start,
                                                            const int32_t *__restrict__ counts,
                                                            const VpKmState *__restrict__ state,
                                                            const int32_t *__restrict__ was_split, int K, int d,
                                                            uint16_t *__restrict__ C)
{
    if (nothing_to_update(state, was_split)) return;
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (size_t)K * d) return;
    const int j = (int)(e / d);
    const int c = counts[j];
    if (c > 0 && (start[j] != start[j + 1] || (was_split && state->split && was_split[j]))) {
        const double sum = (double)(long long)acc[e];
        C[e] = double_to_half_bits(sum * 0x1p-24 / (double)c);
    }
}

// binary16 bits -> double, exactly
__device__ inline double half_bits_to_double(uint32_t h)
{
    const _Float16 v = __builtin_bit_cast(_Float16, (unsigned short)h);
    return (double)(float)v;
}

// Optional remedy for clusters without members: in ascending order each takes the cluster that
// has the most members at that moment (ties: lowest index; at least two members), whose centroid
// c becomes c (1 - 2^-10) while c (1 + 2^-10) goes to the empty cluster; half of the members
// (rounded down) are counted for the new cluster.  One workgroup; cnt lives in LDS.
// A cluster whose members stay with it has their mean written again in the next iteration: was_split, for the kernels above.
__global__ __launch_bounds__(1024) void kmeans_split_kernel(const int32_t *__restrict__ counts, int K, int d,
                                                            VpKmState *__restrict__ state, int32_t *__restrict__ was_split,
                                                            uint16_t *__restrict__ C)
{
    extern __shared__ int cnt[];   // [K]
    __shared__ int red_c[16], red_i[16];
    __shared__ int big_s, any_empty;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) any_empty = 0;
    __syncthreads();
    for (int j = tid; j < K; j += 1024) {
        cnt[j] = counts[j];
        was_split[j] = 0;
        if (cnt[j] == 0) any_empty = 1;
    }
    __syncthreads();
    if (tid == 0) state->split = any_empty;   // (cleared here after the iteration that wrote the means again)
    if (!any_empty) return;
    const double eps = 0x1p-10;
    for (int j = 0; j < K; ++j) {
        if (cnt[j] != 0) continue;          // uniform: every thread reads the same LDS word
        int bc = -1, bi = 0x7fffffff;       // largest count, lowest index
        for (int i = tid; i < K; i += 1024) {
            if (cnt[i] > bc) {
                bc = cnt[i];
                bi = i;
            }
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int c2 = __shfl_xor(bc, off), i2 = __shfl_xor(bi, off);
            if (c2 > bc || (c2 == bc && i2 < bi)) {
                bc = c2;
                bi = i2;
            }
        }
        if (lane == 0) {
            red_c[wave] = bc;
            red_i[wave] = bi;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < 16; ++w) {
                if (red_c[w] > bc || (red_c[w] == bc && red_i[w] < bi)) {
                    bc = red_c[w];
                    bi = red_i[w];
                }
            }
            big_s = bc >= 2 ? bi : -1;
        }
        __syncthreads();
        const int big = big_s;
        if (big < 0) return;                // nothing left to split (uniform)
        for (int e = tid; e < d; e += 1024) {
            const double c = half_bits_to_double(C[(size_t)big * d + e]);
            C[(size_t)j * d + e] = double_to_half_bits(c * (1.0 + eps));
            C[(size_t)big * d + e] = double_to_half_bits(c * (1.0 - eps));
        }
        __syncthreads();
        if (tid == 0) {
            const int c = cnt[big];
            was_split[big] = 1;
            cnt[j] = c / 2;
            cnt[big] = c - c / 2;
        }
        __syncthreads();
    }
}

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, size_t n, uint32_t v)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------- active sets
// bit v of cluster assign[r]'s list is set for every recorded token v of vector r
__global__ __launch_bounds__(256) void aset_flag_kernel(const int32_t *__restrict__ top,
                                                        const int32_t *__restrict__ assign, long n, int T, int K,
                                                        int V, int words, uint32_t *__restrict__ bitmaps)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * T) return;
    const int v = top[i];
    const int j = assign[i / T];
    if (v < 0 || v >= V || j < 0 || j >= K) return;
    atomicOr(&bitmaps[(size_t)j * words + (v >> 5)], 1u << (v & 31));
}

__device__ inline int block_sum_256(int v, int *lds)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    return lds[0] + lds[1] + lds[2] + lds[3];
}

__global__ __launch_bounds__(256) void aset_count_kernel(const uint32_t *__restrict__ bitmaps, int words,
                                                         int32_t *__restrict__ sizes)
{
    __shared__ int lds[4];
    const uint32_t *bm = bitmaps + (size_t)blockIdx.x * words;
    int c = 0;
    for (int w = threadIdx.x; w < words; w += 256) c += __popc(bm[w]);
    c = block_sum_256(c, lds);
    if (threadIdx.x == 0) sizes[blockIdx.x] = c;
}

// cand_off[j] = sum of the sizes below j (64-bit); one wavefront
__global__ __launch_bounds__(64) void aset_scan_kernel(const int32_t *__restrict__ sizes, int K,
                                                       int64_t *__restrict__ cand_off)
{
    long long carry = 0;
    const int lane = threadIdx.x;
    for (int base = 0; base < K; base += 64) {
        const int j = base + lane;
        const long long v = j < K ? sizes[j] : 0;
        long long inc = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long up = __shfl_up(inc, off);
            if (lane >= off) inc += up;
        }
        if (j < K) cand_off[j] = carry + inc - v;
        carry += __shfl(inc, 63);
    }
    if (lane == 0) cand_off[K] = carry;
}

// the set bits of cluster blockIdx.x's list as ascending token ids
__global__ __launch_bounds__(256) void aset_emit_kernel(const uint32_t *__restrict__ bitmaps, int words,
                                                        const int64_t *__restrict__ cand_off,
                                                        int32_t *__restrict__ cand_ids)
{
    __shared__ int wsum[4];
    const uint32_t *bm = bitmaps + (size_t)blockIdx.x * words;
    int64_t out = cand_off[blockIdx.x];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int base = 0; base < words; base += 256) {
        const int w = base + threadIdx.x;
        uint32_t bits = w < words ? bm[w] : 0u;
        const int c = __popc(bits);
        int inc = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(inc, off);
            if (lane >= off) inc += up;
        }
        __syncthreads();   // wsum of the previous round has been read
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        int before = inc - c;
        for (int x = 0; x < wave; ++x) before += wsum[x];
        const int round_total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        int64_t pos = out + before;
        while (bits) {
            const int bit = __ffs(bits) - 1;
            bits &= bits - 1;
            cand_ids[pos++] = w * 32 + bit;
        }
        out += round_total;
    }
}

}  // namespace

uint16_t vpk_round_to_half(double v) { return double_to_half_bits(v); }

void vpk_fill_u32(void *p, size_t n, uint32_t v, hipStream_t st)
{
    if (n == 0) return;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (uint32_t *)p, n, v);
}

void vpk_kmeans_prepare(const void *C, int K, int d, int kt, int K_pad, bool always, const VpKmPass &pass, hipStream_t st)
{
    hipLaunchKernelGGL(kmeans_prepare_kernel, dim3(K_pad / 16), dim3(1024), 0, st, (const uint16_t *)C, K, d, kt, always ? 1 : 0,
                       pass);
}

void vpk_kmeans_assign(const void *cpart, int parts, long row0, int rows, int K, const VpKmPass &pass, hipStream_t st)
{
    const auto kernel = pass.rank ? kmeans_assign_kernel<true> : kmeans_assign_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((rows + 255) / 256), dim3(256), 0, st, (const int2 *)cpart, parts, row0, rows, K, pass);
}

bool vpk_kmeans_rows_in_lds(int kt, int ctiles, long n)
{
    if (!rows_in_lds_faster(kt, ctiles, n)) return false;
    hipError_t e;
    if (kt == 16) e = prepare_assign_lds<16>();
    else if (kt == 24) e = prepare_assign_lds<24>();
    else if (kt == 32) e = prepare_assign_lds<32>();
    else if (kt == 40) e = prepare_assign_lds<40>();
    else if (kt == 48) e = prepare_assign_lds<48>();
    else return false;
    if (e == hipSuccess) return true;
    (void)hipGetLastError();   // the split-k kernel serves the call: no error of its
    return false;
}

bool vpk_kmeans_takes_passes_apart(int kt, long n) { return takes_passes_apart(kt, n); }

bool vpk_kmeans_assign_gemm(const void *X, long n, int d, int K, int kt, int ctiles, bool rows_in_lds, const VpKmPass &pass,
                            hipStream_t st)
{
    const dim3 grid((unsigned)((n + 63) / 64)), block(256);
#define VP_KM_LAUNCH(kernel, KW)                                                                                     \
    hipLaunchKernelGGL((pass.rank ? kernel<KW, true> : kernel<KW, false>), grid, block, 0, st, (const uint4 *)X, n, d, K, \
                       ctiles, pass)
    if (rows_in_lds) {
#define VP_KM_CASE(KT)                                                            \
    case KT:                                                                      \
        launch_assign_lds<KT>(X, n, d, K, ctiles, pass, st);                      \
        if (!pass.first && pass.apart) VP_KM_LAUNCH(kmeans_reassign_kernel, KT / 4); \
        break;
        switch (kt) {
            VP_KM_CASE(16)
            VP_KM_CASE(24)
            VP_KM_CASE(32)
            VP_KM_CASE(40)
            VP_KM_CASE(48)
            default: break;   // callers ask vpk_kmeans_rows_in_lds
        }
#undef VP_KM_CASE
        return true;
    }
#define VP_KM_CASE(KW)                                       \
    case KW * 4:                                             \
        VP_KM_LAUNCH(kmeans_assign_gemm_kernel, KW);         \
        return true;
    switch (kt) {
        VP_KM_CASE(2)
        VP_KM_CASE(4)
        VP_KM_CASE(6)
        VP_KM_CASE(8)
        VP_KM_CASE(10)
        VP_KM_CASE(12)
        default: return false;   // other k-extents: the caller falls back to the decode-time kernel
    }
#undef VP_KM_CASE
#undef VP_KM_LAUNCH
}

void vpk_kmeans_place(long n, int K, int d, const VpKmPass &pass, int32_t *start, int32_t *list, void *acc, hipStream_t st)
{
    hipLaunchKernelGGL(kmeans_place_kernel, dim3((unsigned)((n + PLACE_THREADS - 1) / PLACE_THREADS)), dim3(PLACE_THREADS),
                       (size_t)(2 * K + 1) * sizeof(int), st, n, K, pass, start, list, (unsigned long long *)acc, (size_t)K * d);
}

bool vpk_kmeans_mean_form(int K) { return K >= 256; }

void vpk_kmeans_update(const void *X, int d, const int32_t *list, const int32_t *start, const int32_t *counts, int K,
                       int splits, void *acc, const VpKmState *state, const int32_t *was_split, void *C, hipStream_t st)
{
    if (vpk_kmeans_mean_form(K)) {
        // enough clusters to fill the chip with one workgroup each
        hipLaunchKernelGGL(kmeans_mean_kernel, dim3(K), dim3(MEAN_THREADS), 0, st, (const uint4 *)X, d / 8, list, start,
                           counts, (unsigned long long *)acc, state, was_split, (uint4 *)C);
        return;
    }
    hipLaunchKernelGGL(kmeans_sum_kernel, dim3(K, splits), dim3(256), 0, st, (const uint4 *)X, d / 8, list, start,
                       splits, (unsigned long long *)acc, state);
    const size_t e = (size_t)K * d;
    hipLaunchKernelGGL(kmeans_update_kernel, dim3((unsigned)((e + 255) / 256)), dim3(256), 0, st,
                       (const unsigned long long *)acc, start, counts, state, was_split, K, d, (uint16_t *)C);
}

void vpk_kmeans_split(const int32_t *counts, int K, int d, VpKmState *state, int32_t *was_split, void *C, hipStream_t st)
{
    hipLaunchKernelGGL(kmeans_split_kernel, dim3(1), dim3(1024), (size_t)K * sizeof(int), st, counts, K, d, state, was_split,
                       (uint16_t *)C);
}

void vpk_aset_flags(const int32_t *top, const int32_t *assign, long n, int T, int K, int V, int words,
                    uint32_t *bitmaps, int32_t *sizes, int64_t *cand_off, hipStream_t st)
{
    vpk_fill_u32(bitmaps, (size_t)K * words, 0u, st);
    const long total = n * T;
    if (total > 0)
        hipLaunchKernelGGL(aset_flag_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, top, assign, n,
                           T, K, V, words, bitmaps);
    hipLaunchKernelGGL(aset_count_kernel, dim3(K), dim3(256), 0, st, bitmaps, words, sizes);
    hipLaunchKernelGGL(aset_scan_kernel, dim3(1), dim3(64), 0, st, sizes, K, cand_off);
}

void vpk_aset_emit(const uint32_t *bitmaps, int words, int K, const int64_t *cand_off, int32_t *cand_ids,
                   hipStream_t st)
{
    hipLaunchKernelGGL(aset_emit_kernel, dim3(K), dim3(256), 0, st, bitmaps, words, cand_off, cand_ids);
}
