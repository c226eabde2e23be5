// Hub tier: dense rows of a hypergraph whose 2-paths run mostly through a
// few vertices (hubs) that lie in a large part of E_s.
//
// The overlaps of a row with a window of E_s positions are a row of the
// product H_s^T H_s. Over the hubs that product is dense: it is taken with
// matrix instructions on 0/1 values (fp4, 1.0 exactly; sums in fp32, exact
// for integers below 2^24). The remaining 2-paths, through all other
// vertices, are few per pair (the planner's rule); they are added through
// 8-bit counters in LDS that start the matrix accumulators. Nothing but
// the counts of survivors is kept between the passes: the emit pass takes
// the products again, which costs less than storing and reading the
// survivors.
//
// Layout. Every rank of E_s has 128 fp4 values, 64 bytes (`nib`), kHubs of
// them hub memberships: lane l of a matrix operand holds values
// [32 (l / 16), +32) of row l % 16, 16 bytes. The last kBiasValues are 1.0 for
// every rank; against them the operand of a row holds values that sum to
// 0.5 - s_min, so that an accumulator's sign says whether the pair survives.
// A workgroup takes kHubRows consecutive hub rows and one window of
// 2^kDenseBits positions (one slot per row), in steps of kHubStep positions;
// each of its eight wavefronts covers 64 positions x 32 rows per step: four
// position tiles x two row tiles. Positions are dealt to the tiles so that a
// lane's 16 results of a row tile are 16 consecutive positions of one row.
// Workgroups are numbered window-major (slg_grid.h), so those in flight read
// the same window's 1 MiB of `nib` from L2.
#include <limits.h>

#include "slg_device.h"
#include "slg_grid.h"
#include "slg_internal.h"

namespace slg {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kHubThreads = 512;
constexpr int kHubWaves = kHubThreads / 64;
constexpr int kHubStep = 512;                // positions per step: 64 per wavefront
constexpr int kNibWords = 16;                // 32-bit words of `nib` per rank
constexpr int kNibQuads = kNibWords / 4;
constexpr int kBiasValues = 8;
// Positions whose remainder the counting pass adds up at a time (a row of
// counters is padded by 16 bytes against bank conflicts).
constexpr int kCountRange = 2048;
constexpr int kEmitRows = 16, kEmitStep = 1024;  // the emit pass's tile
constexpr int kFlush = 4;                        // rows of 64 entries written out together
static_assert(kHubRows == 32 && kHubs + kBiasValues == 8 * kNibWords && kHubStep == 64 * kHubWaves, "tile shape");
static_assert(kHubMaxMembers <= 255, "8-bit overlaps");

// ---------------------------------------------------------------------------
// choice of the hubs
// ---------------------------------------------------------------------------
// Vertex degrees from kHubMinDegree in bins of a sixteenth of an octave.
constexpr int kHubMinBits = 6;
constexpr int kHubBins = (31 - kHubMinBits) * 16;

__device__ __forceinline__ int hub_bin(unsigned d) {
    const int e = 31 - __clz((int)d);
    return (e - kHubMinBits) * 16 + (int)((d >> (e - 4)) & 15u);
}

// The hubs are the vertices of the highest bins that hold at most kHubs of
// them. The tier is used when there are enough 2-paths to pay for its setup,
// the hubs carry most of them, and those left over are rare per pair of kept
// rows. The workgroup that finishes last decides (one launch: small plans
// pay for every one). info and hist come zeroed.
__global__ __launch_bounds__(512) void hub_select_kernel(int64_t n, const int64_t *__restrict__ vs_ptr,
                                                         const int64_t *__restrict__ kept, HubInfo *info,
                                                         unsigned long long *hist) {
    static_assert(kHubBins <= 512, "one bin per thread");
    __shared__ unsigned cnt[kHubBins];
    __shared__ unsigned long long paths[kHubBins];
    __shared__ unsigned long long ws[8], hub_paths;
    __shared__ int lowest, last;
    const int tid = threadIdx.x;
    for (int b = tid; b < kHubBins; b += 512) {
        cnt[b] = 0;
        paths[b] = 0;
    }
    if (tid == 0) {
        lowest = INT_MAX;
        hub_paths = 0;
    }
    __syncthreads();
    unsigned long long all = 0;
    for (int64_t v = (int64_t)blockIdx.x * 512 + tid; v < n; v += (int64_t)gridDim.x * 512) {
        const int64_t d64 = vs_ptr[v + 1] - vs_ptr[v];
        if (d64 < 2 || d64 > INT_MAX) continue;  // out of range: malformed, flagged by the row plan
        const unsigned long long d = (unsigned long long)d64;
        all += d * (d - 1) / 2;
        if (d >= (1u << kHubMinBits)) {
            const int b = hub_bin((unsigned)d);
            atomicAdd(&cnt[b], 1u);
            atomicAdd(&paths[b], d * (d - 1) / 2);
        }
    }
    all = wave_sum(all);
    if (lane_id() == 0 && all) atomicAdd(&info->all_paths, all);
    __syncthreads();
    for (int b = tid; b < kHubBins; b += 512)
        if (cnt[b]) {
            atomicAdd(&hist[b], (unsigned long long)cnt[b]);
            atomicAdd(&hist[kHubBins + b], paths[b]);
        }
    // this thread's atomics have been performed (device-scope ones go past the
    // L2s; a device-scope fence would write an L2 back per workgroup, 60 us)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) last = atomicAdd(&info->done, 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    auto load = [](unsigned long long *p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const int b = kHubBins - 1 - tid;  // highest bin first
    const unsigned long long c = b >= 0 ? load(&hist[b]) : 0, w = b >= 0 ? load(&hist[kHubBins + b]) : 0;
    unsigned long long tot;
    const unsigned long long cincl = block_excl_scan<512>(c, ws, tot) + c;
    const unsigned long long wincl = block_excl_scan<512>(w, ws, tot) + w;
    if (b >= 0 && c && cincl <= (unsigned long long)kHubs) {
        const int e = b / 16 + kHubMinBits;
        atomicMin(&lowest, (16 + b % 16) << (e - 4));  // the bin's lower degree bound
        atomicMax(&hub_paths, wincl);
    }
    __syncthreads();
    if (tid == 0) {
        const double every = (double)load(&info->all_paths), rest = every - (double)hub_paths;
        const double rows = (double)*kept;
        const double pairs = 0.5 * rows * rows, per_pair = rows > 0 ? rest / pairs : 1.0;
        info->min_degree = lowest;
        info->hub_paths = hub_paths;
        info->use = every >= kHubMinPaths && every >= kHubMinMean * pairs && rest <= 0.125 * every &&
                    per_pair <= kHubMaxRest;
    }
}

__global__ void hub_list_kernel(int64_t n, const int64_t *__restrict__ vs_ptr, HubInfo *info) {
    const int t = info->min_degree;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        if (vs_ptr[v + 1] - vs_ptr[v] >= t) {
            const int at = atomicAdd(&info->count, 1);
            if (at < kHubs) info->vertex[at] = (int32_t)v;
        }
    }
}

// First position in the ascending list a[lo, hi) holding a value >= key (hi if
// none), by the whole wavefront: 64 probes per round.
__device__ __forceinline__ int64_t wave_lower_bound(const int32_t *__restrict__ a, int64_t lo, int64_t hi, int key) {
    const int lane = lane_id();
    while (hi > lo) {
        const int64_t step = (hi - lo + 63) / 64, probe = lo + lane * step;
        const int below = __popcll(__ballot(probe < hi && a[probe] < key));  // a prefix of the lanes
        if (below == 0) return lo;
        hi = min(hi, lo + below * step);
        lo += (below - 1) * step + 1;
    }
    return lo;
}

// nib of kBitRanks consecutive ranks per workgroup: 1.0 (fp4: 2) for every hub
// whose list holds the rank and in the bias values, put together in LDS and
// written as whole lines (with one global atomic per list entry the build took
// 0.86 ms for 1.07e6 ranks).
constexpr int kBitRanks = 512;
__global__ __launch_bounds__(256) void hub_bits_kernel(const HubInfo *__restrict__ info,
                                                       const int64_t *__restrict__ vs_ptr,
                                                       const int32_t *__restrict__ vs_cid,
                                                       uint32_t *__restrict__ nib) {
    constexpr int kStride = kNibWords + 1;  // bank conflicts
    __shared__ uint32_t x[kBitRanks * kStride];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int c0 = (int)blockIdx.x * kBitRanks, c1 = c0 + kBitRanks;
    for (int t = threadIdx.x; t < kBitRanks * kStride; t += blockDim.x)
        x[t] = t % kStride == kNibWords - 1 ? 0x22222222u : 0u;
    __syncthreads();
    const int hubs = min(info->count, kHubs);
    for (int h = wave; h < hubs; h += 4) {
        const int v = info->vertex[h];
        const int64_t hi = vs_ptr[v + 1];
        int64_t p = wave_lower_bound(vs_cid, vs_ptr[v], hi, c0);
        while (true) {
            const int c = p + lane < hi ? vs_cid[p + lane] : INT_MAX;
            if (c >= c0 && c < c1) atomicOr(&x[(c - c0) * kStride + h / 8], 2u << (4 * (h % 8)));
            if (__ballot(c < c1) != ~0ull) break;
            p += 64;
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kBitRanks * kNibWords; t += blockDim.x)
        nib[(int64_t)c0 * kNibWords + t] = x[t / kNibWords * kStride + t % kNibWords];
}

__global__ void hub_flags_kernel(int64_t m, const uint8_t *__restrict__ rclass, uint8_t *__restrict__ flag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) flag[i] = rclass[i] == kDenseHub;
}

__global__ void hub_rows_kernel(int64_t m, const uint8_t *__restrict__ flag, const int64_t *__restrict__ pre,
                                int64_t cap, int32_t *__restrict__ rows) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m && flag[i] && pre[i] < cap) rows[pre[i]] = (int32_t)i;
}

// Edges of every threshold in hub rows (for measurement).
__global__ void hub_edges_kernel(const int32_t *__restrict__ rows, int64_t count,
                                 const int64_t *__restrict__ slot_base, const int64_t *__restrict__ slot_off,
                                 int64_t S, int32_t K, unsigned long long *__restrict__ out) {
    unsigned long long sum = 0;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = rows[t];
        for (int k = 0; k < K; ++k)
            sum += (unsigned long long)(slot_off[(int64_t)k * (S + 1) + slot_base[i + 1]] -
                                        slot_off[(int64_t)k * (S + 1) + slot_base[i]]);
    }
    sum = wave_sum(sum);
    if (lane_id() == 0 && sum) atomicAdd(out, sum);
}

// ---------------------------------------------------------------------------
// counting and emit passes
// ---------------------------------------------------------------------------
template <int ROWS>
struct HubSmem {
    // members outside the hubs (more than kMembers: all are searched again
    // for every range): next position in the vertex's list, the first one
    // past the window, and the row of the group
    static constexpr int kMembers = 32 * ROWS;
    int32_t cur[kMembers], end[kMembers];
    uint8_t mrow[kMembers];
    int32_t members;
    int32_t mpre[ROWS + 1];                       // members of the group's rows, flattened
    int32_t row[ROWS], cid[ROWS], slot[ROWS];     // slot -1: the row has none in this window
    int64_t p0[ROWS];
    int32_t lim_min, lim_max;                     // smallest and largest own place of the rows with a slot
};

// The group's rows; false (for all threads) when none has a slot in window w.
template <int ROWS>
__device__ __forceinline__ bool hub_rows(HubSmem<ROWS> &sm, const Pruned &g, const HubRows &h, int64_t first, int w) {
    const int tid = threadIdx.x;
    if (tid < 64) {
        const int64_t at = first + tid;
        int i = 0, c = -1, k = 0, slot = -1;
        int64_t p0 = 0;
        if (tid < ROWS && at < h.hi) {
            i = h.rows[at];
            c = g.cid[i];
            const int t = w - ((c + 1) >> kDenseBits);
            if (t >= 0 && t < h.nslots[i]) {
                slot = (int)(h.slot_base[i] + t);
                p0 = g.he_ptr[i];
                k = (int)(g.he_ptr[i + 1] - p0);
            }
        }
        const int incl = wave_incl_scan(k);
        const int lim = c - (w << kDenseBits);
        const int lo = -wave_max(slot >= 0 ? -lim : -INT_MAX), hi = wave_max(slot >= 0 ? lim : INT_MIN);
        if (tid < ROWS) {
            sm.row[tid] = i;
            sm.cid[tid] = c;
            sm.slot[tid] = slot;
            sm.p0[tid] = p0;
            sm.mpre[tid] = incl - k;
        }
        if (tid == ROWS - 1) sm.mpre[ROWS] = incl;
        if (tid == 0) {
            sm.lim_min = lo;
            sm.lim_max = hi;
            sm.members = 0;
        }
    }
    __syncthreads();
    return sm.lim_max != INT_MIN;
}

// Member idx of the group's rows: its row, and the part [a, end) of its list
// with positions in [from, to) (empty for hubs).
template <int ROWS>
__device__ __forceinline__ void hub_member(const HubSmem<ROWS> &sm, const Pruned &g, int min_degree, int idx, int from,
                                           int to, int &r, int &a, int &end) {
    r = 0;
#pragma unroll
    for (int step = ROWS / 2; step > 0; step >>= 1)
        if (sm.mpre[r + step] <= idx) r += step;
    const int64_t p = sm.p0[r] + (idx - sm.mpre[r]);
    const int v = g.he_idx[p];
    a = g.tail_beg[p];
    end = (int)g.vs_ptr[v + 1];
    if (end - (int)g.vs_ptr[v] >= min_degree || a >= end || g.vs_cid[end - 1] < from) {
        a = end;
        return;
    }
    a = lower_bound_i32(g.vs_cid, a, end, from);
    if (g.vs_cid[end - 1] >= to) end = lower_bound_i32(g.vs_cid, a, end, to);
}

// fp4 values (eight, four bits each) that sum to -x, x = s - 0.5 <= 43.5.
__device__ __forceinline__ uint32_t hub_bias(int s) {
    uint32_t code = 0;
    int x = 2 * s - 1;  // in halves
    for (int t = 0; t < kBiasValues && x > 0; ++t) {
        const int v = x >= 12 ? 12 : x >= 8 ? 8 : x >= 6 ? 6 : x >= 4 ? 4 : x;  // 6, 4, 3, 2, 1.5, 1, 0.5
        const uint32_t c = v == 12 ? 7u : v == 8 ? 6u : v == 6 ? 5u : v == 4 ? 4u : (uint32_t)v;
        code |= (8u | c) << (4 * t);
        x -= v;
    }
    return code;
}

__device__ __forceinline__ v8i operand(uint4 x) { return v8i{(int)x.x, (int)x.y, (int)x.z, (int)x.w, 0, 0, 0, 0}; }

// acc (the remainder) + the rows' products with the positions, less the bias.
__device__ __forceinline__ v4f hub_product(uint4 pos, uint4 row, v4f acc) {
    // formats 4: fp4; scales 0x7F: 2^0
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(operand(pos), operand(row), acc, 4, 4, 0, 0x7F7F7F7F, 0,
                                                            0x7F7F7F7F);
}

// A wavefront's operand for row tile nt of the group, and the place of this
// lane's row in the window at ja.
template <int ROWS>
__device__ __forceinline__ uint4 hub_row_operand(const HubSmem<ROWS> &sm, const uint4 *__restrict__ nib, int nt,
                                                 uint32_t bias) {
    const int lane = lane_id(), q = lane >> 4, r = (lane & 15) + 16 * nt;
    uint4 op = sm.slot[r] >= 0 ? nib[(int64_t)sm.cid[r] * kNibQuads + q] : make_uint4(0u, 0u, 0u, 0u);
    if (q == kNibQuads - 1) op.w = bias;
    return op;
}

// Cursors of the members outside the hubs for places from `from` on of the
// window at ja.
template <int ROWS>
__device__ __forceinline__ void hub_cursors(HubSmem<ROWS> &sm, const Pruned &g, int min_degree, int ja, int from) {
    const int all = sm.mpre[ROWS];
    for (int idx = threadIdx.x; idx < all; idx += kHubThreads) {
        int r, a, end;
        hub_member(sm, g, min_degree, idx, ja + from, ja + kDenseWindow, r, a, end);
        if (a < end) {
            const int at = atomicAdd(&sm.members, 1);
            if (at < HubSmem<ROWS>::kMembers) {
                sm.cur[at] = a;
                sm.end[at] = end;
                sm.mrow[at] = (uint8_t)r;
            }
        }
    }
}

// Adds up to eight places (those of list positions [a, last) in [from, to);
// lists ascend and start at `from` or later) of the aligned block at blk to
// the row's counters; returns how many.
__device__ __forceinline__ int hub_add_block(uint32_t *cnt, int row, uint4 v, unsigned blk, unsigned a, unsigned last,
                                             int from, int to) {
    const uint32_t x[4] = {v.x, v.y, v.z, v.w};
    int n = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int c = (int)(e & 1 ? x[e / 2] >> 16 : x[e / 2] & 0xFFFFu);
        if (blk + e >= a && blk + e < last && (unsigned)(c - from) < (unsigned)(to - from)) {
            const unsigned at = (unsigned)(row + (c - from));
            atomicAdd(&cnt[at >> 2], 1u << (8 * (at & 3u)));
            ++n;
        }
    }
    return n;
}

// Counts the remainder of the places [from, from + len) of the window at ja
// into cnt (cleared; `stride` bytes per row), with `threads` threads (whole
// wavefronts) of which this is the tid-th. Four lanes take a member, 16
// bytes (eight 16-bit places) each, and four members at a time are loaded
// before any is used: with one lane per member the wait for the longest
// list's chain of loads was as long as the products (1.8 of 4.2 ms on 1.2e10
// pairs).
template <int ROWS>
__device__ __forceinline__ void hub_count_rest(HubSmem<ROWS> &sm, const Pruned &g, int min_degree, uint32_t *cnt,
                                               int stride, int ja, int from, int len, int tid, int threads) {
    const int to = from + len, members = uniform(sm.members);
    if (members <= HubSmem<ROWS>::kMembers) {
        constexpr int kAhead = 4;
        const int sub = tid & 3, groups = threads / 4;
        for (int m0 = tid >> 2; m0 - (tid >> 2) < members; m0 += groups * kAhead) {
            unsigned a[kAhead], end[kAhead];  // blocks after the last may start past 2^31
            int row[kAhead];
            uint4 v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int x = m0 + u * groups;
                const bool in = x < members;
                a[u] = in ? (unsigned)sm.cur[x] : 0u;
                end[u] = in ? (unsigned)sm.end[x] : 0u;
                row[u] = in ? sm.mrow[x] * stride : 0;
                const unsigned blk = block_at(a[u], sub);
                v[u] = blk < end[u] ? *reinterpret_cast<const uint4 *>(g.vs_win + blk) : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                bool more = a[u] < end[u];
                while (__any(more)) {
                    const unsigned b0 = block_at(a[u]), blk = block_at(a[u], sub);
                    int n = more ? hub_add_block(cnt, row[u], v[u], blk, a[u], min(end[u], blk + 8u), from, to) : 0;
                    n += __builtin_amdgcn_update_dpp(0, n, 0xB1, 0xF, 0xF, false);  // the four lanes' sum
                    n += __builtin_amdgcn_update_dpp(0, n, 0x4E, 0xF, 0xF, false);
                    a[u] += (unsigned)n;
                    // all 32 places taken, and the list goes on
                    more = more && a[u] == b0 + 32u && a[u] < end[u];
                    if (more && a[u] + 8u * sub < end[u])
                        v[u] = *reinterpret_cast<const uint4 *>(g.vs_win + a[u] + 8u * sub);
                }
                if (sub == 0 && m0 + u * groups < members) sm.cur[m0 + u * groups] = (int)a[u];
            }
        }
    } else {  // more members than have cursors
        for (int idx = tid; idx < sm.mpre[ROWS]; idx += threads) {
            int r, a, end;
            hub_member(sm, g, min_degree, idx, ja + from, ja + to, r, a, end);
            while (a < end) {
                const unsigned blk = block_at((unsigned)a);
                const int n = hub_add_block(cnt, r * stride, *reinterpret_cast<const uint4 *>(g.vs_win + blk), blk,
                                            (unsigned)a, min((unsigned)end, blk + 8u), from, to);
                if (n == 0) break;  // (a list that does not ascend)
                a += n;
            }
        }
    }
}

// Inclusive sum over the wavefront's lanes with row shifts and broadcasts
// (no LDS permutes).
__device__ __forceinline__ int wave_incl_scan_dpp(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
    return x;
}

// Counting pass: every threshold's survivors per slot into slot_cnt. A pair
// costs one conversion of its remainder counter, its share of a matrix
// instruction and one bit operation per threshold (two from the second on).
// 1.2e10 pairs (1.2e11 2-paths, s = 16) take 3.7 ms: 1.6 ms of it these, the
// rest the remainder's searches and walks; the LDS walk of every 2-path took
// 39.9 ms. 4.1e9 pairs (S = {8, 16}): 1.08 ms against 12.4 ms.
// KT: 1, 2 or SLG_MAX_S thresholds held in registers.
template <int KT>
__global__ __launch_bounds__(kHubThreads) __attribute__((amdgpu_waves_per_eu(4))) void hub_count_kernel(
    Pruned g, HubRows h, EmitParams prm, int64_t number0, int64_t groups, int64_t S, int64_t *__restrict__ slot_cnt) {
    constexpr int kStride = kCountRange + 16;
    __shared__ HubSmem<kHubRows> sm;
    __shared__ uint32_t cnt[kHubRows * kStride / 4];  // remainder overlaps of the range, 8 bits each
    __shared__ uint32_t tally[KT][kHubRows];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int64_t number = number0 + blockIdx.x;
    const int w = (int)(h.first_window + number / groups);
    if (!hub_rows(sm, g, h, h.lo + number % groups * kHubRows, w)) return;
    for (int x = tid; x < kHubRows * kStride / 4; x += kHubThreads) cnt[x] = 0u;
    for (int x = tid; x < KT * kHubRows; x += kHubThreads) tally[x / kHubRows][x % kHubRows] = 0u;
    const int K = prm.k, s_min = prm.s[0];
    const int ja = w << kDenseBits;
    const int lim_max = uniform(sm.lim_max);
    // positions up to every row's own hold no partner
    const int range0 = max(0, uniform(sm.lim_min) + 1) / kCountRange * kCountRange;
    const int stop = (int)min((int64_t)kDenseWindow, h.kept - ja);  // positions of E_s in the window
    const int min_degree = h.info->min_degree;
    hub_cursors(sm, g, min_degree, ja, range0);

    const int q = lane >> 4, j = lane & 15;
    const uint4 *nib = reinterpret_cast<const uint4 *>(h.nib);
    uint4 rowop[2];
    int lim[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        rowop[nt] = hub_row_operand(sm, nib, nt, hub_bias(s_min));
        lim[nt] = sm.cid[j + 16 * nt] - ja;
    }
    // lane's ranks of position tile t in a step: see the layout above
    const uint4 *posop = nib + ((int64_t)ja + wave * 64 + (j >> 2) * 16 + (j & 3)) * kNibQuads + q;
    uint4 pos[4];
    auto load_positions = [&](int sb) {
#pragma unroll
        for (int t = 0; t < 4; ++t) pos[t] = posop[(int64_t)(sb + 4 * t) * kNibQuads];
    };
    load_positions(range0);
    float above[KT];      // thresholds less s_min
    uint32_t misses[KT];  // pairs below each threshold, 16 bits per row tile (at most 512 per lane)
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
        above[kk] = kk < K ? (float)(prm.s[kk] - s_min) : 0.0f;
        misses[kk] = 0;
    }
    __syncthreads();
    for (int range = range0; range < stop; range += kCountRange) {
        hub_count_rest(sm, g, min_degree, cnt, kStride, ja, range, kCountRange, tid, kHubThreads);
        __syncthreads();  // the range's counters are complete
        for (int sb = range; sb < min(range + kCountRange, stop); sb += kHubStep) {
            const int at = wave * 64 + q * 16;  // this lane's 16 positions of the step
            v4f acc[2][4];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                uint4 *place = reinterpret_cast<uint4 *>(&cnt[((j + 16 * nt) * kStride + (sb - range) + at) / 4]);
                const uint4 c = *place;
                *place = make_uint4(0u, 0u, 0u, 0u);
                const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[nt][t] = v4f{(float)(cw[t] & 0xFFu), (float)(cw[t] >> 8 & 0xFFu),
                                     (float)(cw[t] >> 16 & 0xFFu), (float)(cw[t] >> 24)};
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[nt][t] = hub_product(pos[t], rowop[nt], acc[nt][t]);
            if (sb + kHubStep < kDenseWindow) load_positions(sb + kHubStep);  // in flight until the next products
            if (sb <= lim_max) {  // partners come after the row's own position
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (sb + at + 4 * t + r <= lim[nt]) acc[nt][t][r] = -1.0f;
            }
            // one bit per pair, the sign of overlap - threshold + 0.5
#pragma unroll
            for (int kk = 0; kk < KT; ++kk) {
                if (KT > 2 && kk >= K) break;
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    uint32_t signs = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            signs = __builtin_amdgcn_alignbit(
                                signs, __float_as_uint(kk == 0 ? acc[nt][t][r] : acc[nt][t][r] - above[kk]), 31u);
                    misses[kk] += (uint32_t)__popc(signs) << (16 * nt);
                }
            }
        }
        __syncthreads();  // the counters are cleared before the next range adds to them
    }
    // every pair of the steps was tested: the rest are survivors
    const int steps = (stop - range0 + kHubStep - 1) / kHubStep;
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
        if (kk >= K) break;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            int x = 16 * steps - (int)(misses[kk] >> (16 * nt) & 0xFFFFu);
            x += __shfl_xor(x, 16);
            x += __shfl_xor(x, 32);
            if (q == 0 && x) atomicAdd(&tally[kk][j + 16 * nt], (unsigned)x);
        }
    }
    __syncthreads();
    for (int x = tid; x < K * kHubRows; x += kHubThreads) {
        const int slot = sm.slot[x % kHubRows];
        if (slot >= 0) slot_cnt[(int64_t)(x / kHubRows) * S + slot] = tally[x / kHubRows][x % kHubRows];
    }
}

// Writes out a row of a step: its survivors in position order (overlaps in
// cr, hyperedges of the positions in ids), at the row's next output position
// of every threshold (base[kk][r], advanced), and clears the row.
template <int KT>
__device__ __forceinline__ void hub_write_row(const EmitParams &prm, uint8_t *cr, const int32_t *ids, uint16_t *queue,
                                              int i, int slot, int r, long long (*base)[kEmitRows]) {
    const int lane = lane_id(), K = prm.k;
    uint4 *place = reinterpret_cast<uint4 *>(cr) + lane;  // 16 neighbouring positions
    if (slot >= 0) {
        // the bytes that reach s_min (at most 127), in their high bits
        const uint32_t high = 0x80808080u, less = (uint32_t)prm.s[0] * 0x01010101u;
        const uint4 c = *place;
        const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
        uint32_t m[4];
        int own = 0;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            m[x] = (((cw[x] | high) - less) | cw[x]) & high;
            own += __popc(m[x]);
        }
        const int incl = wave_incl_scan_dpp(own);
        const int n = __builtin_amdgcn_readlane(incl, 63);
        uint16_t *qp = queue + (incl - own);
#pragma unroll
        for (int x = 0; x < 16; ++x)
            if (m[x / 4] & (0x80u << (8 * (x % 4)))) *qp++ = (uint16_t)(16 * lane + x);
        wave_lds_sync();
        // four rows of 64 at a time: their LDS reads overlap
        for (int f0 = 0; f0 < n; f0 += 64 * kFlush) {
            int at[kFlush], id[kFlush], ov[kFlush];
#pragma unroll
            for (int u = 0; u < kFlush; ++u) at[u] = queue[min(f0 + 64 * u + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < kFlush; ++u) {
                id[u] = ids[at[u]];
                ov[u] = cr[at[u]];
            }
#pragma unroll
            for (int kk = 0; kk < KT; ++kk) {
                if (kk >= K) break;
                const long long b = uniform(base[kk][r]);
                const auto colp = as_global(prm.col[kk] + b);
                const auto wp = as_global(prm.w[kk] + b);
                const auto rowp = as_global(prm.row[kk] + (prm.row[kk] ? b : 0));
                int out = 0;
#pragma unroll
                for (int u = 0; u < kFlush; ++u) {
                    if (f0 + 64 * u >= n) break;  // wave-uniform
                    const bool surv = f0 + 64 * u + lane < n && (kk == 0 || ov[u] >= prm.s[kk]);
                    const unsigned long long mask = __ballot(surv);
                    const unsigned o = (unsigned)(out + (kk == 0 ? lane : bits_below(mask)));
                    if (surv) {
                        colp[o] = id[u];
                        wp[o] = ov[u];
                        if (prm.row[kk]) rowp[o] = i;
                    }
                    out += __popcll(mask);
                }
                if (out == 0) break;  // larger thresholds have none either
                wave_lds_sync();
                if (lane == 0) base[kk][r] = b + out;
            }
        }
        wave_lds_sync();  // the queue is reused by the next row
    }
    *place = make_uint4(0u, 0u, 0u, 0u);
}

// Emit pass: each threshold's edges at the slot's offsets, in position order.
// Sixteen rows and steps of 1,024 positions. Half of the wavefronts take the
// products of a step, 64 positions at a time, and leave its overlaps in LDS,
// 8 bits each; meanwhile the step before is written out. Rows differ by far in
// their survivors, so wavefronts take them from a ticket, those of the first
// kind when their products are done. Loads and stores of a wavefront share one
// counter, so its stores come after all loads of a step. Three tiles go
// round: one takes the next step's remainder, one the products, one is
// written out and cleared. 7.6e8 edges of two thresholds from 4.1e9 pairs
// take 4.6 ms, 2.1 ms of it the products (the emit from stored survivors took
// 3.9 ms, after a counting pass that is 11 ms longer for writing them).
template <int KT>
__global__ __launch_bounds__(kHubThreads) __attribute__((amdgpu_waves_per_eu(4))) void hub_emit_kernel(
    Pruned g, HubRows h, EmitParams prm, int64_t number0, int64_t groups, int64_t S,
    const int64_t *__restrict__ slot_off) {
    constexpr int kStride = kEmitStep + 16;
    constexpr int kTile = kEmitRows * kStride / 4;
    constexpr int kProducers = kHubWaves / 2;
    __shared__ HubSmem<kEmitRows> sm;
    __shared__ uint32_t cnt[3][kTile];
    __shared__ int32_t ids[2][kEmitStep];              // hyperedges of the steps' positions
    __shared__ uint16_t queue[kHubWaves][kEmitStep];   // a row's survivors in a step
    __shared__ long long base[KT][kEmitRows];          // the rows' next output positions
    __shared__ int ticket[2];                          // rows of a step taken, by parity
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int64_t number = number0 + blockIdx.x;
    const int w = (int)(h.first_window + number / groups);
    if (!hub_rows(sm, g, h, h.lo + number % groups * kEmitRows, w)) return;
    for (int x = tid; x < 3 * kTile; x += kHubThreads) (&cnt[0][0])[x] = 0u;
    const int K = prm.k, s_min = prm.s[0];
    const int ja = w << kDenseBits;
    const int lim_max = uniform(sm.lim_max);
    const int first = max(0, uniform(sm.lim_min) + 1) / kEmitStep * kEmitStep;
    const int stop = (int)min((int64_t)kDenseWindow, h.kept - ja);  // positions of E_s in the window
    const int steps = (stop - first + kEmitStep - 1) / kEmitStep;
    const int min_degree = h.info->min_degree;
    hub_cursors(sm, g, min_degree, ja, first);
    const bool producer = wave < kProducers;
    for (int x = tid; x < K * kEmitRows; x += kHubThreads) {
        const int kk = x / kEmitRows, r = x % kEmitRows;
        base[kk][r] = sm.slot[r] >= 0 ? slot_off[(int64_t)kk * (S + 1) + sm.slot[r]] - prm.out_base[kk] : 0;
    }
    if (tid < 2) ticket[tid] = 0;
    __syncthreads();
    auto write_rows = [&](int it) {  // rows of step it, while there are any
        const int tile = it % 3;
        while (true) {
            int r = 0;
            if (lane == 0) r = atomicAdd(&ticket[it & 1], 1);
            r = uniform(r);
            if (r >= kEmitRows) break;
            hub_write_row<KT>(prm, reinterpret_cast<uint8_t *>(cnt[tile]) + r * kStride, ids[it & 1], queue[wave],
                              uniform(sm.row[r]), uniform(sm.slot[r]), r, base);
        }
    };
    // a step's ticket is cleared in the next one, before the barrier that
    // opens the step that takes it again
    if (!producer) {
        for (int it = 0; it <= steps; ++it) {
            __syncthreads();  // step it - 1 is ready
            if (tid == 64 * kProducers) ticket[it & 1] = 0;
            if (it > 0) write_rows(it - 1);
        }
        return;
    }
    const int q = lane >> 4, j = lane & 15;
    const uint4 *nib = reinterpret_cast<const uint4 *>(h.nib);
    const uint4 rowop = hub_row_operand(sm, nib, 0, hub_bias(s_min));
    const int lim = sm.cid[j] - ja;
    const uint4 *posop = nib + ((int64_t)ja + wave * 64 + (j >> 2) * 16 + (j & 3)) * kNibQuads + q;
    uint4 pos[4];
    auto load_positions = [&](int sb) {
#pragma unroll
        for (int t = 0; t < 4; ++t) pos[t] = posop[(int64_t)(sb + 4 * t) * kNibQuads];
    };
    constexpr int kPart = 64 * kProducers;  // positions the producers take at a time
    const float b = (float)s_min - 0.5f;
    load_positions(first);
    hub_count_rest(sm, g, min_degree, cnt[0], kStride, ja, first, kEmitStep, tid, 64 * kProducers);
    for (int it = 0; it <= steps; ++it) {
        __syncthreads();
        if (it < steps) {
            const int sb = first + it * kEmitStep, tile = it % 3;
            for (int x = tid; x < kEmitStep; x += 64 * kProducers)
                ids[it & 1][x] = sb + x < stop ? g.cid_row[ja + sb + x] : 0;
            if (it + 1 < steps)
                hub_count_rest(sm, g, min_degree, cnt[(it + 1) % 3], kStride, ja, sb + kEmitStep, kEmitStep, tid,
                               64 * kProducers);
#pragma unroll 2
            for (int part = 0; part < kEmitStep; part += kPart) {
                const int at = part + wave * 64 + q * 16;  // this lane's 16 positions
                uint4 *place = reinterpret_cast<uint4 *>(&cnt[tile][(j * kStride + at) / 4]);
                const uint4 c = *place;
                const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
                v4f acc[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t] = v4f{(float)(cw[t] & 0xFFu), (float)(cw[t] >> 8 & 0xFFu), (float)(cw[t] >> 16 & 0xFFu),
                                 (float)(cw[t] >> 24)};
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[t] = hub_product(pos[t], rowop, acc[t]);
                if (sb + part + kPart < kDenseWindow) load_positions(sb + part + kPart);
                if (sb + part <= lim_max) {  // partners come after the row's own position
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (sb + at + 4 * t + r <= lim) acc[t][r] = -b;
                }
                uint32_t ov[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    ov[t] = 0u;
#pragma unroll
                    for (int r = 0; r < 4; ++r) ov[t] = __builtin_amdgcn_cvt_pk_u8_f32(acc[t][r] + b, r, ov[t]);
                }
                *place = make_uint4(ov[0], ov[1], ov[2], ov[3]);
            }
            // the loads above are waited for before the stores below
#pragma unroll
            for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(pos[t].x), "+v"(pos[t].y), "+v"(pos[t].z), "+v"(pos[t].w));
        }
        if (it > 0) write_rows(it - 1);
    }
}

unsigned grid_of(int64_t n, int64_t cap) {
    int64_t b = (n + 255) / 256;
    if (b > cap) b = cap;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

int64_t hub_hist_words() { return 2 * kHubBins; }

hipError_t launch_hub_select(int64_t n, const int64_t *vs_ptr, const int64_t *kept, HubInfo *info, int64_t *hist,
                             hipStream_t st) {
    // few workgroups: each adds its own histogram to the shared one
    hub_select_kernel<<<grid_of(n / 32, 256), 512, 0, st>>>(n, vs_ptr, kept, info,
                                                            reinterpret_cast<unsigned long long *>(hist));
    return hipGetLastError();
}

int64_t hub_nib_words(int64_t kept) {
    return ((kept >> kDenseBits) + 1) * (int64_t)kDenseWindow * kNibWords;
}

hipError_t launch_hub_bits(int64_t n, HubInfo *info, const int64_t *vs_ptr, const int32_t *vs_cid, int64_t kept,
                           uint32_t *nib, hipStream_t st) {
    static_assert(kDenseWindow % kBitRanks == 0 && kHubs % 8 == 0, "whole workgroups, whole words");
    hub_list_kernel<<<grid_of(n, 1024), 256, 0, st>>>(n, vs_ptr, info);
    hub_bits_kernel<<<(unsigned)(hub_nib_words(kept) / kNibWords / kBitRanks), 256, 0, st>>>(info, vs_ptr, vs_cid, nib);
    return hipGetLastError();
}

hipError_t launch_hub_rows(int64_t m, const uint8_t *rclass, uint8_t *flag, int64_t *pre, int64_t *partials,
                           int64_t cap, int32_t *rows, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    hub_flags_kernel<<<grid_of(m, INT_MAX), 256, 0, st>>>(m, rclass, flag);
    const hipError_t e = launch_exclusive_scan_u8(flag, m, pre, partials, st);
    if (e != hipSuccess) return e;
    hub_rows_kernel<<<grid_of(m, INT_MAX), 256, 0, st>>>(m, flag, pre, cap, rows);
    return hipGetLastError();
}

hipError_t launch_hub_edges(const HubRows &h, int64_t slots, const int64_t *slot_off, int32_t K, int64_t *out,
                            hipStream_t st) {
    if (h.hi <= h.lo) return hipSuccess;
    hub_edges_kernel<<<grid_of(h.hi - h.lo, 1024), 256, 0, st>>>(h.rows + h.lo, h.hi - h.lo, h.slot_base, slot_off,
                                                                 slots, K, reinterpret_cast<unsigned long long *>(out));
    return hipGetLastError();
}

hipError_t launch_hub(bool emit, const HubRows &h, const Pruned &g, const EmitParams &ep, int64_t slots,
                      int64_t *slot_cnt, const int64_t *slot_off, hipStream_t st) {
    if (h.hi <= h.lo) return hipSuccess;
    if (!g.cid || !g.cid_row || !g.vs_cid || !g.vs_win || !h.nib || ep.row_s || ep.row_base || ep.s[0] > kHubMaxS) return hipErrorInvalidValue;
    const HubGrid grid(h.lo, h.hi, emit ? kEmitRows : kHubRows, h.kept, kDenseBits, h.first_window, kHubThreads,
                       h.launch_limit);
#define SLG_HUB(KT)                                                                                             \
    for (int64_t base = 0; base < grid.total; base += grid.cap) {                                               \
        const unsigned count = (unsigned)grid.count(base);                                                      \
        if (emit)                                                                                               \
            hub_emit_kernel<KT><<<count, kHubThreads, 0, st>>>(g, h, ep, base, grid.groups, slots, slot_off);   \
        else                                                                                                    \
            hub_count_kernel<KT><<<count, kHubThreads, 0, st>>>(g, h, ep, base, grid.groups, slots, slot_cnt);  \
    }
    if (ep.k <= 1) {
        SLG_HUB(1)
    } else if (ep.k <= 2) {
        SLG_HUB(2)
    } else {
        SLG_HUB(SLG_MAX_S)
    }
#undef SLG_HUB
    return hipGetLastError();
}

}  // namespace slg
