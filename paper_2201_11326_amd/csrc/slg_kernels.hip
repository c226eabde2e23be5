// gfx950 kernels for s-line graph construction.
//
// The path (Section III-B/C, Algorithms 2 and 3):
//   K1  prune: drop hyperedges with |e| < s_min from every vertex list
//       (degree-based pruning on both sides of a pair; a pair that meets
//       the threshold has both sizes >= s, so no edge is lost).
//   K2  plan: per kept hyperedge e_i and member v, the tail of v's list after
//       i (the partners e_j, j > i, reached through v: the upper triangle),
//       the 2-path work w_i = sum of tail lengths, and a slot table that
//       splits heavy rows by hyperedge-id range and by work.
//   K3  count overlaps |e_i n e_j| by walking every 2-path (e_i, v, e_j):
//         tiny rows (w_i <= 8): one lane sorts its partners in registers;
//         light rows (w_i <= 2048): one wavefront gathers the 2-path
//           partners into LDS, sorts them in registers (bitonic) and
//           run-length counts them;
//         heavy slots: one workgroup marks partners in an LDS bitmap over
//           the slot's id range, ranks them by prefix popcount, and counts
//           each repeated partner in an LDS counter indexed by its rank;
//           heavy vertex tails are cut into equal pieces across the
//           wavefronts.
//       The counting pass tallies every threshold's survivors (output
//       sizes) and, when memory allows, keeps each row's or slot's
//       (partner, overlap) pairs for the emit pass (the count stores).
//   K4/5 threshold-and-emit for every s_k of the ensemble from the same
//       counts (the stored overlap is the largest s for which the pair
//       survives), compacted with wavefront ballots + prefix sums. The rank
//       order is the hyperedge-id order, so rows come out sorted.
//   K6  assembly: prefix sums of per-slot counts give each slot's output
//       offset and the CSR row pointers.
// Every step is exact integer work; no floating point is involved.
#include <limits.h>

#include <type_traits>

#include "slg_device.h"
#include "slg_grid.h"
#include "slg_internal.h"

namespace slg {
namespace {

// ---------------------------------------------------------------------------
// device-wide exclusive scan (int64 output, out[n] = total)
// ---------------------------------------------------------------------------
// Several arrays per launch, since a small plan is bound by its launches (4 us
// of host time each): arrays of at most kScanSmall entries by one workgroup
// each, longer ones in three launches for all of them. With one read-back
// launch per synchronisation and one clearing of all lists, a query of 1000
// rows and six thresholds went from 66 launches to 17, 371 -> 164 us (13 and
// 141 with the light classes together). At kScanSmall entries one workgroup
// takes about as long as three launches.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kScanSmallThreads = 512, kScanSmallItems = 8;
constexpr int64_t kScanSmall = 8 * kScanSmallThreads * kScanSmallItems;

__device__ __forceinline__ int64_t scan_item(const ScanJob &j, int64_t idx) {
    if (j.bytes == 1) return as_global(static_cast<const uint8_t *>(j.in))[idx];
    if (j.bytes == 4) return as_global(static_cast<const int32_t *>(j.in))[idx];
    return as_global(static_cast<const int64_t *>(j.in))[idx];
}

// Tiles pass through LDS, so that loads and stores are whole lines and a
// thread still sums neighbours, and the next tile is loaded before this one
// is summed: 32 768 entries in 26 us without either. (Workgroups of 1024
// threads and twice the LDS waited for a free CU where several streams are
// busy: 29 us a scan beside seven other queries, now 19.)
__global__ __launch_bounds__(kScanSmallThreads) void scan_small_kernel(ScanJobs jobs) {
    constexpr int kTile = kScanSmallThreads * kScanSmallItems;
    __shared__ int64_t ws[kScanSmallThreads / 64];
    __shared__ int64_t buf[kTile + kTile / kScanSmallItems];  // an item of padding per thread
    auto at = [](int i) { return i + i / kScanSmallItems; };
    const ScanJob j = jobs.j[blockIdx.x];
    int64_t carry = 0;
    int64_t v[kScanSmallItems];
    auto load = [&](int64_t t0) {
#pragma unroll
        for (int r = 0; r < kScanSmallItems; ++r) {
            const int64_t i = t0 + r * kScanSmallThreads + threadIdx.x;
            v[r] = i < j.n ? scan_item(j, i) : 0;
        }
    };
    load(0);
    for (int64_t t0 = 0; t0 < j.n; t0 += kTile) {
#pragma unroll
        for (int r = 0; r < kScanSmallItems; ++r) buf[at(r * kScanSmallThreads + threadIdx.x)] = v[r];
        load(t0 + kTile);
        __syncthreads();
        int64_t x[kScanSmallItems], local = 0, tot;
#pragma unroll
        for (int r = 0; r < kScanSmallItems; ++r) {
            x[r] = buf[at(threadIdx.x * kScanSmallItems + r)];
            local += x[r];
        }
        int64_t run = carry + block_excl_scan<kScanSmallThreads>(local, ws, tot);
        carry += tot;
#pragma unroll
        for (int r = 0; r < kScanSmallItems; ++r) {
            buf[at(threadIdx.x * kScanSmallItems + r)] = run;
            run += x[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kScanSmallItems; ++r) {
            const int64_t i = t0 + r * kScanSmallThreads + threadIdx.x;
            if (i < j.n) as_global(j.out)[i] = buf[at(r * kScanSmallThreads + threadIdx.x)];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) as_global(j.out)[j.n] = carry;
}

// Job y's partial sums are partials[y * stride, ...).
__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(ScanJobs jobs, int64_t *__restrict__ partials,
                                                                   int64_t stride) {
    __shared__ int64_t ws[kScanThreads / 64];
    const ScanJob j = jobs.j[blockIdx.y];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    if (base >= j.n) return;
    int64_t s = 0;
    for (int t = threadIdx.x; t < kScanTile; t += kScanThreads)
        if (base + t < j.n) s += scan_item(j, base + t);
    s = wave_sum(s);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) t += ws[w];
        partials[blockIdx.y * stride + blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(1024) void scan_top_kernel(ScanJobs jobs, int64_t *__restrict__ partials,
                                                        int64_t stride) {
    __shared__ int64_t ws[16];
    int64_t *part = partials + blockIdx.x * stride;
    const int64_t nb = (jobs.j[blockIdx.x].n + kScanTile - 1) / kScanTile;
    int64_t carry = 0;
    for (int64_t base = 0; base < nb; base += 1024) {
        int64_t idx = base + threadIdx.x;
        int64_t x = idx < nb ? part[idx] : 0;
        int64_t tot;
        int64_t ex = block_excl_scan<1024>(x, ws, tot);
        if (idx < nb) part[idx] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) part[nb] = carry;
}

__global__ __launch_bounds__(kScanThreads) void scan_down_kernel(ScanJobs jobs, const int64_t *__restrict__ partials,
                                                                 int64_t stride) {
    __shared__ int64_t ws[kScanThreads / 64];
    const ScanJob j = jobs.j[blockIdx.y];
    const int64_t nb = (j.n + kScanTile - 1) / kScanTile;
    const int64_t *part = partials + blockIdx.y * stride;
    if (blockIdx.x == 0 && threadIdx.x == 0) as_global(j.out)[j.n] = nb > 0 ? part[nb] : 0;
    if ((int64_t)blockIdx.x >= nb) return;
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t local = 0;
#pragma unroll
    for (int r = 0; r < kScanItems; ++r) {
        v[r] = base + r < j.n ? scan_item(j, base + r) : 0;
        local += v[r];
    }
    int64_t tot;
    int64_t run = part[blockIdx.x] + block_excl_scan<kScanThreads>(local, ws, tot);
#pragma unroll
    for (int r = 0; r < kScanItems; ++r) {
        if (base + r < j.n) as_global(j.out)[base + r] = run;
        run += v[r];
    }
}

// Values into pinned host memory, one workgroup per entry (a launch instead
// of a copy per value).
__global__ void read_back_kernel(ReadBack rb, int64_t *host) {
    const ReadBack::Item it = rb.item[blockIdx.x];
    for (int t = threadIdx.x; t < it.n; t += blockDim.x) as_global(host)[it.at + t] = as_global(it.src)[t];
}

__global__ void fill_i64_kernel(int64_t *__restrict__ p, int64_t n, int64_t value) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n) p[idx] = value;
}

__global__ void fill_i32_kernel(int32_t *__restrict__ p, int64_t n, int32_t value) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n) p[idx] = value;
}

// ---------------------------------------------------------------------------
// K1: prune hyperedges smaller than s_min out of the vertex lists
// ---------------------------------------------------------------------------
// What is kept is one bit per hyperedge and one per incidence, in words of 64
// with the number of bits in each beside them, whose prefix sums (a 64th of an
// entry per incidence) give positions and ranks. The incidences' bits come
// from the hyperedges', which stay in L2, instead of two pointers per
// incidence. (With a byte and an int64 position per incidence, 4.4e7
// incidences of 8.8e6 hyperedges took 950 us to prune, now 215.)
__global__ __launch_bounds__(256) void row_bits_kernel(int64_t m, const int64_t *__restrict__ he_ptr, int32_t s_min,
                                                       const int32_t *__restrict__ row_s, KeepBits rows) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool keep = false;
    if (i < m) {
        const int64_t size = he_ptr[i + 1] - he_ptr[i];
        keep = size > 0 && size >= (row_s ? row_s[i] : s_min);
    }
    const unsigned long long mask = __ballot(keep);
    if (lane_id() == 0 && (i >> 6) < keep_words(m)) {
        rows.bits[i >> 6] = mask;
        rows.count[i >> 6] = (uint8_t)__popcll(mask);
    }
}

__device__ __forceinline__ int64_t kept_before(const KeepBits &k, int64_t i) {
    return k.pre[i >> 6] + __popcll(k.bits[i >> 6] & ((1ull << (i & 63)) - 1));
}

constexpr int kKeepWords = 8;  // words per wavefront, their loads in flight together

__global__ __launch_bounds__(256) void keep_incidence_kernel(int64_t nnz, const int32_t *__restrict__ v_idx, int64_t m,
                                                             const unsigned long long *__restrict__ rows,
                                                             KeepBits inc) {
    const int lane = lane_id();
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64 * kKeepWords;
    int32_t e[kKeepWords];
    unsigned long long bits[kKeepWords], mine = 0;
#pragma unroll
    for (int r = 0; r < kKeepWords; ++r) {
        const int64_t p = (w0 + r) * 64 + lane;
        e[r] = p < nnz ? v_idx[p] : -1;
    }
#pragma unroll
    for (int r = 0; r < kKeepWords; ++r) bits[r] = e[r] >= 0 && e[r] < m ? rows[e[r] >> 6] : 0ull;
#pragma unroll
    for (int r = 0; r < kKeepWords; ++r) {
        const unsigned long long mask = __ballot(bits[r] >> (e[r] & 63) & 1);
        mine = lane == r ? mask : mine;
    }
    if (lane < kKeepWords && w0 + lane < keep_words(nnz)) {
        inc.bits[w0 + lane] = mine;
        inc.count[w0 + lane] = (uint8_t)__popcll(mine);
    }
}

__global__ __launch_bounds__(256) void compact_idx_kernel(int64_t nnz, const int32_t *__restrict__ v_idx, KeepBits inc,
                                                          int32_t *__restrict__ vs_idx) {
    const int lane = lane_id();
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64 * kKeepWords;
    unsigned long long mask[kKeepWords];
    int64_t pos[kKeepWords];
    int32_t e[kKeepWords];
#pragma unroll
    for (int r = 0; r < kKeepWords; ++r) {
        const bool in = w0 + r < keep_words(nnz);
        mask[r] = in ? inc.bits[w0 + r] : 0ull;
        pos[r] = in ? inc.pre[w0 + r] : 0;
        e[r] = (w0 + r) * 64 + lane < nnz ? v_idx[(w0 + r) * 64 + lane] : 0;
    }
#pragma unroll
    for (int r = 0; r < kKeepWords; ++r)
        if (mask[r] >> lane & 1) vs_idx[pos[r] + bits_below(mask[r])] = e[r];
}

__global__ void compact_ptr_kernel(int64_t n, int64_t nnz, const int64_t *__restrict__ v_ptr, KeepBits inc,
                                   int64_t *__restrict__ vs_ptr) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v > n) return;
    int64_t q = v_ptr[v];
    q = q < 0 ? 0 : (q > nnz ? nnz : q);
    vs_ptr[v] = kept_before(inc, q);
}

// E_s positions of the kept rows (the dense tier's counter index): the rank
// of every kept row among the kept rows, its inverse, and the pruned vertex
// lists rewritten in ranks. Ranks keep the id order, so a list stays sorted
// and its tails are at the same positions.
__global__ void cid_kernel(int64_t m, KeepBits rows, int32_t *__restrict__ cid, int32_t *__restrict__ cid_row) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    const bool kept = rows.bits[i >> 6] >> (i & 63) & 1;
    const int64_t rank = kept_before(rows, i);
    cid[i] = kept ? (int32_t)rank : -1;
    if (kept) cid_row[rank] = (int32_t)i;
}

// An id outside [0, m) (a malformed vertex CSR, which the row plan flags)
// gets -1, which no window holds. vs_win keeps the low kDenseBits bits of
// each rank: windows are aligned, so that is the rank's place in its window.
__global__ void vs_cid_kernel(int64_t n, int64_t m, int64_t cap, const int64_t *__restrict__ vs_ptr,
                              const int32_t *__restrict__ vs_idx, const int32_t *__restrict__ cid,
                              int32_t *__restrict__ vs_cid, uint16_t *__restrict__ vs_win) {
    int64_t total = vs_ptr[n];
    if (total > cap) total = cap;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += stride) {
        const int32_t r = vs_idx[p];
        const int32_t c = (r >= 0 && r < m) ? cid[r] : -1;
        vs_cid[p] = c;
        vs_win[p] = (uint16_t)(c & (kDenseWindow - 1));
    }
}

// ---------------------------------------------------------------------------
// K2: per-row plan (one wavefront per hyperedge, grid-stride)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int light_class(int64_t w) {
    if (w <= kTinyMax) return 0;
    int c = 1;
    while (c < kLightClasses - 1 && w > (int64_t(64) << (c - 1))) ++c;
    return c;
}

// Per-row work estimate (Section III-E's cost: the 2-paths of row i) and
// tier. For every incidence (i, v) of a kept row: [tail_beg, tail_end) = the
// part of v's (pruned) list after i; w_i = sum of the tails; jm = largest
// partner id. Bound by the dependent loads of each incidence (the list's
// bounds, then a binary search in it), so rows of at most kSmallRow members
// are taken a group at a time by one wavefront, their members flattened: one
// incidence per lane, kPlanAhead of them searched in lockstep. (One lane per
// row walked its members one after another: 50 us on a thousand rows of 11,
// 1.02 ms on the 8.8e6 rows of a batch.) Larger rows are cut into pieces of
// kPlanPiece members, one wavefront per piece, so that a run of large rows
// (an input sorted by size) spreads over the whole grid.
constexpr int kSmallRow = 64;
constexpr int kPlanPiece = 256;
constexpr int kPlanAhead = 4;

struct RowPlanOut {
    int32_t *tail_beg, *tail_end;
    int64_t *work;
    int32_t *jmax;
    int32_t *nslots;
    uint8_t *rclass;
    int64_t *bsize;
    int32_t dense_ratio;  // the dense tier's rule (0: off)
    int32_t dense_min;
    const HubInfo *hub;  // the hub tier's choice, or null
    unsigned long long *dense_work;  // 2-paths of dense rows, then the number of hub rows and their 2-paths
};

// Members p[u] of rows i[u] (in[u]: this lane has one): their tails, the tail
// lengths w and last partners jm (-1: none); bad: the incidence is malformed.
__device__ __forceinline__ void plan_members(const Pruned &g, const int (&i)[kPlanAhead],
                                             const int (&p)[kPlanAhead], const bool (&in)[kPlanAhead],
                                             int32_t *__restrict__ tail_beg, int32_t *__restrict__ tail_end,
                                             int (&w)[kPlanAhead], int (&jm)[kPlanAhead], bool (&bad)[kPlanAhead]) {
    int v[kPlanAhead], a[kPlanAhead], e[kPlanAhead], hi[kPlanAhead];
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) v[u] = in[u] ? g.he_idx[p[u]] : -1;
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
        int64_t l = 0, h = 0;
        const bool id = v[u] >= 0 && v[u] < g.n;
        if (id) {
            l = g.vs_ptr[v[u]];
            h = g.vs_ptr[v[u] + 1];
        }
        bad[u] = in[u] && (!id || l < 0 || h < l || h > g.nnz);
        if (bad[u]) l = h = 0;
        a[u] = (int)l;
        e[u] = hi[u] = (int)h;
    }
    bool more = true;
    while (more) {
        int mid[kPlanAhead], x[kPlanAhead];
        more = false;
#pragma unroll
        for (int u = 0; u < kPlanAhead; ++u) {
            mid[u] = middle(a[u], e[u]);
            x[u] = a[u] < e[u] ? g.vs_idx[mid[u]] : 0;
        }
#pragma unroll
        for (int u = 0; u < kPlanAhead; ++u) {
            if (a[u] >= e[u]) continue;
            if (x[u] < i[u])
                a[u] = mid[u] + 1;
            else
                e[u] = mid[u];
            more |= a[u] < e[u];
        }
    }
#pragma unroll
    for (int u = 0; u < kPlanAhead; ++u) {
        // the vertex CSR must be the transpose: i is in the list
        const bool found = a[u] < hi[u] && g.vs_idx[a[u]] == i[u];
        const int beg = found ? a[u] + 1 : a[u];
        bad[u] |= in[u] && !found;
        w[u] = hi[u] - beg;
        jm[u] = beg < hi[u] ? g.vs_idx[hi[u] - 1] : -1;
        if (in[u]) {
            tail_beg[p[u]] = beg;
            tail_end[p[u]] = hi[u];
        }
    }
}

// Tier, slot count and boundary-table size of row i from its totals. hwork
// (LDS): the workgroup's 2-paths of heavy rows, then what dense_work gets. A
// heavy row goes to the dense tier when its candidate partners (the kept
// rows in (i, jm]) number at least dense_min and it has at least
// dense_ratio 2-paths per eight candidates: its slots are then the aligned
// kDenseWindow windows of E_s positions that (i, jm] touches.
__device__ __forceinline__ void plan_finish(const Pruned &g, int64_t i, int64_t p0, int64_t p1, int64_t w, int jm,
                                            bool bad, int32_t light_max, int64_t slot_work, const RowPlanOut &o,
                                            unsigned long long *ccount, unsigned long long *hwork, int *err) {
    int cls = kNone;
    int64_t ns = 0;
    if (bad) {
        atomicOr(err, 1);
    } else if (w > 0) {
        int64_t ci = -1, cj = -1;
        if (w > light_max && o.dense_ratio > 0 && g.cid && p1 - p0 < kWideMembers && jm > i && jm < g.m) {
            ci = g.cid[i];
            cj = g.cid[jm];
        }
        const int64_t crange = cj - ci;  // kept rows in (i, jm]
        if (w <= light_max) {
            cls = kLight0 + light_class(w);
            ns = 1;
        } else if (ci >= 0 && cj > ci && crange >= o.dense_min && 8 * w >= (int64_t)o.dense_ratio * crange) {
            cls = o.hub && o.hub->use && p1 - p0 <= kHubMaxMembers && w >= kHubMinRatio * crange ? kDenseHub : kDense;
            ns = (cj >> kDenseBits) - ((ci + 1) >> kDenseBits) + 1;
        } else {
            cls = (p1 - p0 >= kWideMembers) ? kHeavyWide : kHeavy;
            const int64_t range = (int64_t)jm - i;  // partners lie in [i+1, jm]
            const int64_t by_range = (range + kRangeBits - 1) / kRangeBits;
            const int64_t by_work = (w + slot_work - 1) / slot_work;
            ns = by_range > by_work ? by_range : by_work;
            if (ns > range) ns = range;
        }
    }
    o.work[i] = w;
    o.jmax[i] = jm;
    o.nslots[i] = (int32_t)ns;
    o.rclass[i] = (uint8_t)cls;
    o.bsize[i] = cls >= kHeavy && cls != kDenseHub ? (ns + 1) * (p1 - p0) : 0;  // hub rows keep no boundaries
    if (cls != kNone) atomicAdd(&ccount[cls - 1], (unsigned long long)ns);
    if (cls == kHeavy || cls == kHeavyWide) atomicAdd(hwork, (unsigned long long)w);
    if (cls == kDense) atomicAdd(hwork + 1, (unsigned long long)w);
    if (cls == kDenseHub) {
        atomicAdd(hwork + 2, 1ull);
        atomicAdd(hwork + 3, (unsigned long long)w);
    }
}

// Small rows, ROWS of them per wavefront, and the piece list of the large
// ones: a large row appends ceil(size / kPlanPiece) entries (row | piece <<
// 32), one row's pieces side by side. ROWS: 64, or 16 where 64 would leave
// the chip short of wavefronts.
template <int ROWS>
__global__ __launch_bounds__(256) void row_plan_kernel(Pruned g, int32_t s_min, int32_t light_max,
                                                       int64_t slot_work, int64_t row_lo, int64_t row_hi,
                                                       RowPlanOut o,
                                                       unsigned long long *__restrict__ class_count,
                                                       int *__restrict__ err,
                                                       unsigned long long *__restrict__ heavy_work,
                                                       int64_t *__restrict__ pieces, int64_t pieces_cap,
                                                       unsigned long long *__restrict__ num_pieces) {
    __shared__ unsigned long long ccount[kNumLists];
    __shared__ unsigned long long hwork[4];
    __shared__ int pre[4][64], pos[4][64], rjm[4][64], rbad[4][64];
    __shared__ unsigned long long rw[4][64];
    if (threadIdx.x < kNumLists) ccount[threadIdx.x] = 0;
    if (threadIdx.x < 4) hwork[threadIdx.x] = 0;
    __syncthreads();
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64 * ROWS; i0 < g.m; i0 += nwaves * ROWS) {
        const int64_t i = i0 + lane;
        unsigned long long np = 0;  // pieces of a large row
        int64_t p0 = 0, p1 = 0;
        int n = 0;           // members of a small kept row
        bool own = false;    // this lane finishes its row
        bool broken = false;
        if (lane < ROWS && i < g.m) {
            p0 = g.he_ptr[i];
            p1 = g.he_ptr[i + 1];
            broken = p0 < 0 || p1 > g.nnz || p1 < p0;  // malformed pointers
            const int64_t size = broken ? 0 : p1 - p0;
            // rows outside [row_lo, row_hi) are planned as pruned ones
            const bool kept = size > 0 && size >= (g.row_s ? g.row_s[i] : s_min) && i >= row_lo && i < row_hi;
            if (kept && size > kSmallRow)
                np = (unsigned long long)((size + kPlanPiece - 1) / kPlanPiece);
            else
                own = true;
            n = kept && own ? (int)size : 0;
        }
        const int incl = wave_incl_scan(n);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        pre[wv][lane] = incl - n;
        pos[wv][lane] = (int)p0;
        rw[wv][lane] = 0;
        rjm[wv][lane] = -1;
        rbad[wv][lane] = 0;
        wave_lds_sync();
        for (int f0 = 0; f0 < total; f0 += 64 * kPlanAhead) {
            int row[kPlanAhead], id[kPlanAhead], p[kPlanAhead], w[kPlanAhead], jm[kPlanAhead];
            bool in[kPlanAhead], bad[kPlanAhead];
#pragma unroll
            for (int u = 0; u < kPlanAhead; ++u) row[u] = 0;
#pragma unroll
            for (int step = ROWS / 2; step > 0; step >>= 1)  // largest row with pre <= f
#pragma unroll
                for (int u = 0; u < kPlanAhead; ++u)
                    if (pre[wv][row[u] + step] <= f0 + 64 * u + lane) row[u] += step;
#pragma unroll
            for (int u = 0; u < kPlanAhead; ++u) {
                const int f = f0 + 64 * u + lane;
                in[u] = f < total;
                id[u] = (int)i0 + row[u];
                p[u] = pos[wv][row[u]] + (f - pre[wv][row[u]]);
            }
            plan_members(g, id, p, in, o.tail_beg, o.tail_end, w, jm, bad);
#pragma unroll
            for (int u = 0; u < kPlanAhead; ++u) {
                if (!in[u]) continue;
                if (w[u] > 0) {
                    atomicAdd(&rw[wv][row[u]], (unsigned long long)w[u]);
                    atomicMax(&rjm[wv][row[u]], jm[u]);
                }
                if (bad[u]) rbad[wv][row[u]] = 1;
            }
        }
        wave_lds_sync();
        if (own)
            plan_finish(g, i, p0, p1, (int64_t)rw[wv][lane], rjm[wv][lane], broken || rbad[wv][lane] != 0, light_max,
                        slot_work, o, ccount, hwork, err);
        wave_lds_sync();
        // one reservation per wavefront for the pieces of its large rows
        const unsigned long long pincl = wave_incl_scan(np);
        const unsigned long long ptotal = __shfl(pincl, 63);
        if (ptotal) {
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(num_pieces, ptotal);
            base = __shfl(base, 0) + pincl - np;
            // within the capacity unless the row pointers overlap (malformed)
            for (unsigned long long k = 0; k < np; ++k) {
                if (base + k < (unsigned long long)pieces_cap)
                    pieces[base + k] = (int64_t)((unsigned long long)i | (k << 32));
                else
                    atomicOr(err, 1);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < kNumLists && ccount[threadIdx.x])
        atomicAdd(&class_count[threadIdx.x], ccount[threadIdx.x]);
    if (threadIdx.x == 0 && hwork[0]) atomicAdd(heavy_work, hwork[0]);
    if (threadIdx.x < 3 && hwork[1 + threadIdx.x]) atomicAdd(o.dense_work + threadIdx.x, hwork[1 + threadIdx.x]);
}

// One wavefront per piece of a large row: the piece's tails and its largest
// partner id, into the piece's own partial slots.
__global__ __launch_bounds__(256) void row_piece_kernel(Pruned g, int32_t *__restrict__ tail_beg,
                                                        int32_t *__restrict__ tail_end,
                                                        const int64_t *__restrict__ pieces, int64_t pieces_cap,
                                                        const unsigned long long *__restrict__ num_pieces,
                                                        int64_t *__restrict__ piece_w,
                                                        int32_t *__restrict__ piece_jm, int *__restrict__ err) {
    const int lane = lane_id();
    const int64_t count = min((int64_t)*num_pieces, pieces_cap);
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64; t < count; t += nwaves) {
        const unsigned long long e = (unsigned long long)pieces[t];
        const int64_t r = (int64_t)(e & 0xFFFFFFFFull), k = (int64_t)(e >> 32);
        const int64_t q0 = g.he_ptr[r], q1 = g.he_ptr[r + 1];
        const int64_t a = q0 + k * kPlanPiece, b = min(q1, a + kPlanPiece);
        int64_t w = 0;
        int jm = -1, rbad = 0;
        static_assert(kPlanPiece == 64 * kPlanAhead, "a piece in one go");
        int id[kPlanAhead], p[kPlanAhead], wu[kPlanAhead], ju[kPlanAhead];
        bool in[kPlanAhead], bu[kPlanAhead];
#pragma unroll
        for (int u = 0; u < kPlanAhead; ++u) {
            id[u] = (int)r;
            p[u] = (int)(a + 64 * u + lane);
            in[u] = a + 64 * u + lane < b;  // in 64 bits: the rest of the piece may lie past 2^31
        }
        plan_members(g, id, p, in, tail_beg, tail_end, wu, ju, bu);
#pragma unroll
        for (int u = 0; u < kPlanAhead; ++u) {
            if (!in[u]) continue;
            w += wu[u];
            jm = max(jm, ju[u]);
            rbad |= bu[u] ? 1 : 0;
        }
        w = wave_sum(w);
        jm = wave_max(jm);
        rbad = wave_max(rbad);
        if (lane == 0) {
            piece_w[t] = w;
            piece_jm[t] = jm;
            if (rbad) atomicOr(err, 1);
        }
    }
}

// One lane per row's first piece: the row's totals from its pieces, then the
// tier decision.
__global__ __launch_bounds__(256) void row_piece_finish_kernel(Pruned g, int32_t light_max, int64_t slot_work,
                                                               RowPlanOut o,
                                                               unsigned long long *__restrict__ class_count,
                                                               int *__restrict__ err,
                                                               unsigned long long *__restrict__ heavy_work,
                                                               const int64_t *__restrict__ pieces,
                                                               int64_t pieces_cap,
                                                               const unsigned long long *__restrict__ num_pieces,
                                                               const int64_t *__restrict__ piece_w,
                                                               const int32_t *__restrict__ piece_jm) {
    __shared__ unsigned long long ccount[kNumLists];
    __shared__ unsigned long long hwork[4];
    if (threadIdx.x < kNumLists) ccount[threadIdx.x] = 0;
    if (threadIdx.x < 4) hwork[threadIdx.x] = 0;
    __syncthreads();
    const int64_t count = min((int64_t)*num_pieces, pieces_cap);
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count;
         t += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long e = (unsigned long long)pieces[t];
        if (e >> 32) continue;  // not the row's first piece
        const int64_t r = (int64_t)(e & 0xFFFFFFFFull);
        const int64_t q0 = g.he_ptr[r], q1 = g.he_ptr[r + 1];
        const int64_t np = min((q1 - q0 + kPlanPiece - 1) / kPlanPiece, count - t);
        int64_t w = 0;
        int jm = -1;
        for (int64_t k = 0; k < np; ++k) {
            w += piece_w[t + k];
            jm = max(jm, piece_jm[t + k]);
        }
        // a malformed member has already set err
        plan_finish(g, r, q0, q1, w, jm, false, light_max, slot_work, o, ccount, hwork, err);
    }
    __syncthreads();
    if (threadIdx.x < kNumLists && ccount[threadIdx.x])
        atomicAdd(&class_count[threadIdx.x], ccount[threadIdx.x]);
    if (threadIdx.x == 0 && hwork[0]) atomicAdd(heavy_work, hwork[0]);
    if (threadIdx.x < 3 && hwork[1 + threadIdx.x]) atomicAdd(o.dense_work + threadIdx.x, hwork[1 + threadIdx.x]);
}

// A row block: rows outside [r0, r1) get no slots, no class and no boundary
// entries (from the rows phase's values of every row), and the block's
// list sizes and heavy / dense 2-paths are summed as the row plan sums them.
__global__ __launch_bounds__(256) void block_mask_kernel(int64_t m, int64_t r0, int64_t r1,
                                                         const int32_t *__restrict__ nslots_all,
                                                         const uint8_t *__restrict__ rclass_all,
                                                         const int64_t *__restrict__ bsize_all,
                                                         const int64_t *__restrict__ work,
                                                         int32_t *__restrict__ nslots, uint8_t *__restrict__ rclass,
                                                         int64_t *__restrict__ bsize,
                                                         unsigned long long *__restrict__ class_count,
                                                         unsigned long long *__restrict__ heavy_work,
                                                         unsigned long long *__restrict__ dense_work) {
    __shared__ unsigned long long cc[kNumLists];
    __shared__ unsigned long long hw, dw[3];
    if (threadIdx.x < kNumLists) cc[threadIdx.x] = 0;
    if (threadIdx.x == 0) hw = 0;
    if (threadIdx.x < 3) dw[threadIdx.x] = 0;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const bool in = i >= r0 && i < r1;
        const int c = in ? rclass_all[i] : kNone;
        const int ns = in ? nslots_all[i] : 0;
        nslots[i] = ns;
        rclass[i] = (uint8_t)c;
        bsize[i] = in ? bsize_all[i] : 0;
        if (c != kNone) atomicAdd(&cc[c - 1], (unsigned long long)ns);
        if (c == kHeavy || c == kHeavyWide) atomicAdd(&hw, (unsigned long long)work[i]);
        if (c == kDense) atomicAdd(&dw[0], (unsigned long long)work[i]);
        if (c == kDenseHub) {
            atomicAdd(&dw[1], 1ull);
            atomicAdd(&dw[2], (unsigned long long)work[i]);
        }
    }
    __syncthreads();
    if (threadIdx.x < kNumLists && cc[threadIdx.x]) atomicAdd(&class_count[threadIdx.x], cc[threadIdx.x]);
    if (threadIdx.x == 0 && hw) atomicAdd(heavy_work, hw);
    if (threadIdx.x < 3 && dw[threadIdx.x]) atomicAdd(dense_work + threadIdx.x, dw[threadIdx.x]);
}

// Tier lists filled by fill_slots_kernel.
struct LightLists {
    int32_t *l[kLightClasses];
    int64_t cap[kNumLists];  // capacity of every tier list (light, heavy, heavy-wide)
    int *err;                // set when an append would overflow a list
};

// Writes every light row's slot and appends it to its tier list, and
// reserves each heavy row's slot descriptors in the heavy lists. Rows are
// appended in blocks: a workgroup takes 256 * kFillRows rows, counts them per
// list with wavefront sums into LDS,
// reserves each list's share with one global atomic, then places its rows
// through LDS cursors (global atomics on the few list counters would
// serialise).
constexpr int kFillRows = 4;

__global__ __launch_bounds__(256) void fill_slots_kernel(
    int64_t m, const int64_t *__restrict__ he_ptr, const int64_t *__restrict__ slot_base,
    const int32_t *__restrict__ nslots, const int32_t *__restrict__ jmax,
    const uint8_t *__restrict__ rclass, const int64_t *__restrict__ bbase,
    int32_t *__restrict__ slot_row, LightLists ll, int64_t *__restrict__ hat,
    unsigned long long *__restrict__ list_fill) {
    __shared__ unsigned long long cursor[kNumLists];
    const int tid = threadIdx.x, lane = lane_id();
    const int64_t i0 = (int64_t)blockIdx.x * (256 * kFillRows);
    int cls[kFillRows], ns[kFillRows];
    int64_t base[kFillRows];
#pragma unroll
    for (int r = 0; r < kFillRows; ++r) {
        const int64_t i = i0 + r * 256 + tid;
        cls[r] = kNone;
        ns[r] = 0;
        base[r] = 0;
        if (i < m) {
            cls[r] = rclass[i];
            ns[r] = nslots[i];
            base[r] = slot_base[i];
        }
    }
    if (tid < kNumLists) cursor[tid] = 0;
    __syncthreads();
    // entries per light list: one per row (heavy descriptors are placed by
    // heavy_desc_kernel, in slot order), counted with ballots (with sums over
    // the wavefront the 1000 rows of a small graph took 13.5 us)
    for (int c = kLight0; c < kLight0 + kLightClasses; ++c) {
        int tot = 0;
#pragma unroll
        for (int r = 0; r < kFillRows; ++r) tot += __popcll(__ballot(cls[r] == c));
        if (lane == 0 && tot) atomicAdd(&cursor[c - 1], (unsigned long long)tot);
    }
    __syncthreads();
    if (tid < kNumLists && cursor[tid]) cursor[tid] = atomicAdd(&list_fill[tid], cursor[tid]);
    __syncthreads();
    for (int c = kLight0; c < kLight0 + kLightClasses; ++c) {
        unsigned long long mask[kFillRows], at = 0;
        int tot = 0;
#pragma unroll
        for (int r = 0; r < kFillRows; ++r) {
            mask[r] = __ballot(cls[r] == c);
            tot += __popcll(mask[r]);
        }
        if (!tot) continue;
        if (lane == 0) at = atomicAdd(&cursor[c - 1], (unsigned long long)tot);
        at = __shfl(at, 0);
#pragma unroll
        for (int r = 0; r < kFillRows; ++r) {
            const unsigned long long pos = at + bits_below(mask[r]);
            at += __popcll(mask[r]);
            if (cls[r] != c) continue;
            if (pos < (unsigned long long)ll.cap[c - 1]) {
                ll.l[c - 1][pos] = (int32_t)base[r];
                slot_row[base[r]] = (int32_t)(i0 + r * 256 + tid);
            } else {
                atomicOr(ll.err, 16);
            }
        }
    }
}

// Heavy slots per row, by class: the prefix sums place every heavy row's
// descriptors in row order, so each heavy list is in slot order.
// `lists`: one bit per heavy list that has slots.
__global__ void heavy_counts_kernel(int64_t m, const uint8_t *__restrict__ rclass, const int32_t *__restrict__ nslots,
                                    int lists, int32_t *__restrict__ cnt) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = rclass[i];
        for (int h = 0; h < kNumHeavyLists; ++h)
            if (lists >> h & 1) cnt[(int64_t)h * m + i] = c == kHeavy + h ? nslots[i] : 0;
    }
}

// For every c, the position of the first slot >= slots[c] in a heavy list
// ordered by slot (one thread per c).
__global__ void list_cuts_kernel(const HeavyDesc *__restrict__ desc, int64_t count,
                                 const int64_t *__restrict__ slots, int64_t n, int64_t *__restrict__ out) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const int64_t key = slots[c];
    int64_t lo = 0, hi = count;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)desc[mid].slot < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    out[c] = lo;
}

// First and one-past-last positions of the slots in [s0, s1) in a heavy
// list ordered by slot.
__global__ void heavy_range_kernel(const HeavyDesc *__restrict__ desc, int64_t count, int64_t s0, int64_t s1,
                                   int64_t *__restrict__ out) {
    if (threadIdx.x >= 2) return;
    const int64_t key = threadIdx.x == 0 ? s0 : s1;
    int64_t lo = 0, hi = count;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)desc[mid].slot < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    out[threadIdx.x] = lo;
}

// The slot descriptors of the heavy rows, one lane per slot.
struct HeavyLists {
    HeavyDesc *l[kNumHeavyLists];  // heavy, heavy-wide, dense
    int64_t cap[kNumHeavyLists];
};

__global__ __launch_bounds__(256) void heavy_desc_kernel(
    int64_t m, const int64_t *__restrict__ he_ptr, const int64_t *__restrict__ slot_base,
    const int32_t *__restrict__ nslots, const int32_t *__restrict__ jmax,
    const uint8_t *__restrict__ rclass, const int64_t *__restrict__ bbase,
    const int64_t *__restrict__ hat, int32_t *__restrict__ slot_row, HeavyLists hl,
    const int32_t *__restrict__ cid, int rows, int *__restrict__ err) {
    const int lane = lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    // `rows` rows per wavefront: each lane loads its own row's values, then the
    // heavy rows among them are written one after another (a wavefront per
    // row spent 0.43 ms on the classes of 8.8e6 rows)
    for (int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64 * rows; i0 < m; i0 += nwaves * rows) {
        const int64_t own = i0 + lane;
        const int own_cls = lane < rows && own < m ? rclass[own] : kNone;
        const bool heavy = own_cls >= kHeavy && own_cls != kDenseHub;
        int own_ns = 0, own_k = 0, own_range = 0, own_w0 = 0, own_base = 0;
        int64_t own_at = 0, own_bb = 0;
        if (heavy) {
            own_ns = nslots[own];
            own_at = hat[(own_cls - kHeavy) * (m + 1) + own];  // prefix of the class's slots
            own_base = (int32_t)slot_base[own];
            own_range = (int32_t)(jmax[own] - own);
            own_k = (int)(he_ptr[own + 1] - he_ptr[own]);
            own_bb = bbase[own];
            // dense slots: aligned windows of E_s positions from the window of
            // the row's first candidate (its own position + 1)
            own_w0 = own_cls == kDense ? (cid[own] + 1) >> kDenseBits : 0;
        }
        unsigned long long todo = __ballot(heavy);
        while (todo) {
            const int l = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            auto of = [&](int x) { return __builtin_amdgcn_readlane(x, l); };
            auto of64 = [&](int64_t x) {
                return (int64_t)((uint64_t)(uint32_t)of((int)(x >> 32)) << 32 | (uint32_t)of((int)x));
            };
            const int i = (int)i0 + l, cls = of(own_cls), h = cls - kHeavy;  // list: heavy, heavy-wide, dense
            const int ns = of(own_ns), k = of(own_k), w0 = of(own_w0), base = of(own_base);
            const int64_t at = of64(own_at), bb = of64(own_bb), range = of(own_range);
            if (at < 0 || at + ns > hl.cap[h]) {
                if (lane == 0) atomicOr(err, 16);
                continue;
            }
            HeavyDesc *lst = hl.l[h] + at;
            for (int t = lane; t < ns; t += 64) {
                HeavyDesc d;
                d.row = i;
                if (cls == kDense) {
                    d.ja = (w0 + t) << kDenseBits;
                    d.jb = (w0 + t + 1) << kDenseBits;
                } else {
                    d.ja = (int32_t)(i + 1 + range * t / ns);
                    d.jb = (int32_t)(i + 1 + range * (t + 1) / ns);
                }
                d.k = k;
                d.slot = base + t;
                d.last = t == ns - 1;
                d.bptr = bb + (int64_t)t * k;
                slot_row[base + t] = i;
                lst[t] = d;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// K3-K5 light tier: one wavefront per row, sort-and-count in registers
// ---------------------------------------------------------------------------
// Bitonic sort of 64*KPL keys; element e = lane*KPL + r lives in key[r].
template <int KPL>
__device__ __forceinline__ void wave_bitonic(int (&key)[KPL], int lane) {
    constexpr int P = 64 * KPL;
#pragma unroll
    for (int k = 2; k <= P; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j < KPL) {
#pragma unroll
                for (int r = 0; r < KPL; ++r) {
                    const int pr = r ^ j;
                    if (pr > r) {
                        const bool asc = ((lane * KPL + r) & k) == 0;
                        const int a = key[r], b = key[pr];
                        const bool sw = asc ? (a > b) : (a < b);
                        key[r] = sw ? b : a;
                        key[pr] = sw ? a : b;
                    }
                }
            } else {
                const int lx = j / KPL;
                const bool lower = (lane & lx) == 0;
#pragma unroll
                for (int r = 0; r < KPL; ++r) {
                    const int other = __shfl_xor(key[r], lx);
                    const bool asc = ((lane * KPL + r) & k) == 0;
                    key[r] = (lower == asc) ? min(key[r], other) : max(key[r], other);
                }
            }
        }
    }
}

// Rows with at most kTinyMax 2-paths: one lane per row. The lane collects
// its row's partners (the tails of its members' vertex lists), sorts them
// with a fixed 8-key network in registers, and writes the runs that reach
// each threshold to its own slot's place in the output.
using TinyKeys = int32_t[kTinyMax][256];  // column per thread: conflict-free

template <bool EMIT, bool STORE>
__device__ __forceinline__ void tiny_row(int slot, const Slots &sl, const Pruned &g, const EmitParams *ep,
                                         TinyKeys &keys, int64_t *__restrict__ slot_cnt,
                                         const int64_t *__restrict__ slot_off, const LightStore &ls) {
    static_assert(kTinyMax == 8, "8-key sorting network");
    const int tid = threadIdx.x;
    const int i = sl.row[slot];
    const int64_t p0 = g.he_ptr[i], p1 = g.he_ptr[i + 1];
    int n = 0;
    for (int64_t p = p0; p < p1 && n < kTinyMax; ++p) {
        const int end = g.tail_end[p];
        for (int q = g.tail_beg[p]; q < end && n < kTinyMax; ++q) keys[n++][tid] = g.vs_idx[q];
    }
    int k[kTinyMax];
#pragma unroll
    for (int r = 0; r < kTinyMax; ++r) k[r] = r < n ? keys[r][tid] : INT_MAX;
    // Batcher's odd-even merge sort network for 8 keys (19 compare-exchanges)
    auto cx = [&](int a, int b) {
        const int lo = min(k[a], k[b]), hi = max(k[a], k[b]);
        k[a] = lo;
        k[b] = hi;
    };
    cx(0, 1); cx(2, 3); cx(4, 5); cx(6, 7);
    cx(0, 2); cx(1, 3); cx(4, 6); cx(5, 7);
    cx(1, 2); cx(5, 6);
    cx(0, 4); cx(1, 5); cx(2, 6); cx(3, 7);
    cx(2, 4); cx(3, 5);
    cx(1, 2); cx(3, 4); cx(5, 6);
    // the head of each run of equal partners holds the overlap
    int c[kTinyMax];
#pragma unroll
    for (int r = 0; r < kTinyMax; ++r) {
        int run = 0;
        if (r < n && (r == 0 || k[r] != k[r - 1])) {
#pragma unroll
            for (int q = r; q < kTinyMax; ++q) run += (q < n && k[q] == k[r]) ? 1 : 0;
        }
        c[r] = run;  // 0 for non-heads
    }
    if (STORE) {
        const int64_t base = as_global(ls.off)[i];
        int at = 0;
#pragma unroll
        for (int r = 0; r < kTinyMax; ++r)
            if (c[r] > 0) {
                as_global(ls.key)[base + at] = k[r];
                as_global(ls.cnt)[base + at] = (uint16_t)c[r];
                ++at;
            }
        as_global(ls.n)[i] = at;
    }
    const int K = ep->k;
    const int64_t S = sl.count;
    const int id0 = ep->row_base ? as_global(ep->row_base)[i] : 0;  // caller's id of row i is i - id0
    const int srow = ep->row_s ? as_global(ep->row_s)[i] : 0;
    for (int kk = 0; kk < K; ++kk) {
        const int sk = ep->row_s ? srow : ep->s[kk];
        int64_t pos = EMIT ? slot_off[(int64_t)kk * (S + 1) + slot] - ep->out_base[kk] : 0;
        const int64_t start = pos;
        const auto col = as_global(EMIT ? ep->col[kk] : nullptr);
        const auto wo = as_global(EMIT ? ep->w[kk] : nullptr);
        const auto ro = as_global(EMIT ? ep->row[kk] : nullptr);
#pragma unroll
        for (int r = 0; r < kTinyMax; ++r) {
            if (c[r] >= sk) {  // sk >= 1, so only run heads
                if (EMIT) {
                    col[pos] = k[r] - id0;
                    wo[pos] = c[r];
                    if (ro) ro[pos] = i - id0;
                }
                ++pos;
            }
        }
        if (!EMIT) slot_cnt[(int64_t)kk * S + slot] = pos - start;
    }
}

template <bool EMIT, bool STORE>
__global__ __launch_bounds__(256) void tiny_kernel(const int32_t *__restrict__ list, int64_t count, Slots sl,
                                                   Pruned g, EmitParams prm, int64_t *__restrict__ slot_cnt,
                                                   const int64_t *__restrict__ slot_off, LightStore ls) {
    __shared__ TinyKeys keys;
    __shared__ EmitParams sp;
    stage_params(&sp, prm);
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= count) return;
    const int slot = list[t];
    if (EMIT && (slot < sp.slot_lo || slot >= sp.slot_hi)) return;  // outside the emitted chunk
    tiny_row<EMIT, STORE>(slot, sl, g, &sp, keys, slot_cnt, slot_off, ls);
}

// A wavefront's scratch for one row: its partners, and a batch of members'
// tails (start, flattened start).
template <int KPL>
struct LightSmem {
    int32_t buf[4][64 * KPL];
    int32_t seg_a[4][64];
    int32_t seg_p[4][65];
};

// STORE (counting pass): the row's partners and overlaps are also written
// to the light store, in partner order.
template <int KPL, bool EMIT, bool STORE>
__device__ __forceinline__ void light_row(int slot, const Slots &sl, const Pruned &g, const EmitParams *ep,
                                          int32_t *kb, int32_t *sa, int32_t *sp0, int64_t *__restrict__ slot_cnt,
                                          const int64_t *__restrict__ slot_off, const LightStore &ls) {
    static_assert(!(STORE && EMIT), "the store is written by the counting pass");
    constexpr int P = 64 * KPL;
    const int lane = lane_id();
    const int i = sl.row[slot];
    const int64_t p0 = g.he_ptr[i], p1 = g.he_ptr[i + 1];

    // gather the partners e_j of every 2-path (e_i, v, e_j), j > i: members
    // are taken 64 at a time; their tails are flattened and every lane finds
    // the tail of each of its positions by binary search, so all loads of a
    // batch are independent and coalesced within a tail
    int w = 0;
    for (int64_t q = p0; q < p1; q += 64) {
        const int64_t p = q + lane;
        int beg = 0, len = 0;
        if (p < p1) {
            beg = g.tail_beg[p];
            len = g.tail_end[p] - beg;
        }
        const int incl = wave_incl_scan(len);
        const int tot = __shfl(incl, 63);
        sa[lane] = beg;
        sp0[lane] = incl - len;
        if (lane == 0) sp0[64] = tot;
        wave_lds_sync();
        for (int fb = 0; fb < tot; fb += 256) {
            // largest u with sp0[u] <= f, the four positions in lockstep
            int jr[4], u[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) u[r] = 0;
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (sp0[u[r] + step] <= min(fb + lane + 64 * r, tot - 1)) u[r] += step;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                jr[r] = g.vs_idx[sa[u[r]] + (min(fb + lane + 64 * r, tot - 1) - sp0[u[r]])];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int f = fb + lane + 64 * r;
                const int e = w + f;
                if (f < tot && e < P) kb[e] = jr[r];
            }
        }
        w += tot;
        wave_lds_sync();
    }
    if (w > P) w = P;  // the planner's class bound makes this unreachable
    wave_lds_sync();

    int key[KPL];
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const int e = lane * KPL + r;
        key[r] = e < w ? kb[e] : INT_MAX;
    }
    wave_bitonic<KPL>(key, lane);
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < KPL; ++r) kb[lane * KPL + r] = key[r];
    wave_lds_sync();

    // run-length count: the head of each run of equal j holds the overlap,
    // its distance to the next head (from the last element down, by ballots:
    // walking each run took as long as the longest; 5000 skewed rows 94 us so
    // and with the searches above one after another, 55 now)
    int x[KPL], c[KPL];
    int next = w;  // the first head after row r
#pragma unroll
    for (int r = KPL - 1; r >= 0; --r) {
        const int e = r * 64 + lane;
        x[r] = e < w ? kb[e] : INT_MAX;
        const bool head = e < w && (e == 0 || kb[e - 1] != x[r]);
        const unsigned long long heads = __ballot(head);
        const unsigned long long after = lane < 63 ? heads >> (lane + 1) : 0ull;
        c[r] = head ? (after ? __ffsll(after) : next - e) : 0;  // 0 for non-heads
        if (heads) next = r * 64 + __ffsll(heads) - 1;
    }

    if (STORE) {  // every run head, in partner order
        const int64_t base = as_global(ls.off)[i];
        int tot = 0;
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            const bool head = c[r] > 0;
            const unsigned long long mask = __ballot(head);
            if (head) {
                const int64_t pos = base + tot + bits_below(mask);
                as_global(ls.key)[pos] = x[r];
                as_global(ls.cnt)[pos] = (uint16_t)c[r];
            }
            tot += __popcll(mask);
        }
        if (lane == 0) as_global(ls.n)[i] = tot;
    }

    const int K = ep->k;
    const int64_t S = sl.count;
    const int id0 = ep->row_base ? as_global(ep->row_base)[i] : 0;  // caller's id of row i is i - id0
    const int srow = ep->row_s ? as_global(ep->row_s)[i] : 0;
    for (int k = 0; k < K; ++k) {
        const int sk = ep->row_s ? srow : ep->s[k];
        int64_t base = EMIT ? slot_off[(int64_t)k * (S + 1) + slot] - ep->out_base[k] : 0;
        auto col = as_global(EMIT ? ep->col[k] : nullptr);
        auto wo = as_global(EMIT ? ep->w[k] : nullptr);
        auto ro = as_global(EMIT ? ep->row[k] : nullptr);
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            const bool surv = c[r] >= sk;  // sk >= 1, so only run heads
            const unsigned long long mask = __ballot(surv);
            if (EMIT && surv) {
                const int64_t pos = base + bits_below(mask);
                col[pos] = x[r] - id0;
                wo[pos] = c[r];
                if (ro) ro[pos] = i - id0;
            }
            base += __popcll(mask);
        }
        if (!EMIT && lane == 0) slot_cnt[(int64_t)k * S + slot] = base;
    }
}

template <int KPL, bool EMIT, bool STORE>
__global__ __launch_bounds__(256) void light_kernel(const int32_t *__restrict__ list, int64_t count,
                                                    Slots sl, Pruned g, EmitParams prm,
                                                    int64_t *__restrict__ slot_cnt,
                                                    const int64_t *__restrict__ slot_off, LightStore ls) {
    __shared__ LightSmem<KPL> sm;
    __shared__ EmitParams sp;  // thresholds and outputs, indexed by a uniform k
    stage_params(&sp, prm);
    __syncthreads();
    const int wv = threadIdx.x >> 6;
    const int64_t wid = (int64_t)blockIdx.x * 4 + wv;
    if (wid >= count) return;
    const int slot = list[wid];
    if (EMIT && (slot < sp.slot_lo || slot >= sp.slot_hi)) return;  // outside the emitted chunk
    light_row<KPL, EMIT, STORE>(slot, sl, g, &sp, sm.buf[wv], sm.seg_a[wv], sm.seg_p[wv], slot_cnt, slot_off, ls);
}

// The light lists of one launch, the class with the longest rows first:
// workgroup b takes rows of the last class whose first workgroup is <= b.
struct LightRuns {
    const int32_t *list[kLightClasses];
    int64_t count[kLightClasses];
    unsigned first[kLightClasses];  // of class kLightClasses - 1, ..., 0
    __device__ __forceinline__ int class_of(unsigned block, int64_t &group) const {
        int at = 0;
#pragma unroll
        for (int r = 1; r < kLightClasses; ++r) at = first[r] <= block ? r : at;
        group = block - first[at];
        return kLightClasses - 1 - at;
    }
};

// Counting pass of all light classes in one launch: in a small graph each
// class has too few rows for the chip and takes as long as its longest row,
// one class after another (5000 skewed rows: 185 us by class, 93 together).
template <bool STORE>
__global__ __launch_bounds__(256) void light_count_kernel(LightRuns runs, Slots sl, Pruned g, EmitParams prm,
                                                          int64_t *__restrict__ slot_cnt, LightStore ls) {
    static_assert(kLightClasses == 7, "one case per class");
    __shared__ union {
        LightSmem<32> rows;
        TinyKeys tiny;
    } sm;
    __shared__ EmitParams sp;
    stage_params(&sp, prm);
    __syncthreads();
    int64_t group;
    const int cls = runs.class_of(blockIdx.x, group), wv = threadIdx.x >> 6;
    const int64_t t = cls ? group * 4 + wv : group * 256 + threadIdx.x;
    if (t >= runs.count[cls]) return;
    const int slot = as_global(runs.list[cls])[t];
#define SLG_ROW(KPL)                                                                                               \
    light_row<KPL, false, STORE>(slot, sl, g, &sp, sm.rows.buf[wv], sm.rows.seg_a[wv], sm.rows.seg_p[wv], slot_cnt, \
                                 nullptr, ls)
    switch (cls) {
        case 0: tiny_row<false, STORE>(slot, sl, g, &sp, sm.tiny, slot_cnt, nullptr, ls); break;
        case 1: SLG_ROW(1); break;
        case 2: SLG_ROW(2); break;
        case 3: SLG_ROW(4); break;
        case 4: SLG_ROW(8); break;
        case 5: SLG_ROW(16); break;
        default: SLG_ROW(32); break;
    }
#undef SLG_ROW
}

// ---------------------------------------------------------------------------
// K3-K5 heavy tier: one workgroup per slot, LDS bitmap + rank counters
// ---------------------------------------------------------------------------
constexpr int kHW = kHeavyThreads / 64;              // wavefronts per heavy workgroup
constexpr int kSuperWords = 1024;                    // words per rank superblock (32768 bits)
constexpr int kSupers = kRangeWords / kSuperWords;

// Emit pass of all light classes from the light store: one wavefront per row
// (one lane per tiny row) reads its (partner, overlap) pairs in partner order
// and compacts every threshold's survivors with ballots (8.8e6 small rows:
// 232 us where gathering and sorting them again took 980).
__device__ __forceinline__ void tiny_store_row(int slot, const Slots &sl, const LightStore &ls, const EmitParams &sp,
                                               const int64_t *__restrict__ slot_off) {
    const int i = sl.row[slot];
    const int n = min(as_global(ls.n)[i], kTinyMax);
    const int64_t off = as_global(ls.off)[i];
    int key[kTinyMax], c[kTinyMax];
#pragma unroll
    for (int r = 0; r < kTinyMax; ++r) {
        key[r] = r < n ? as_global(ls.key)[off + r] : 0;
        c[r] = r < n ? (int)as_global(ls.cnt)[off + r] : 0;
    }
    const int id0 = sp.row_base ? as_global(sp.row_base)[i] : 0;
    const int srow = sp.row_s ? as_global(sp.row_s)[i] : 0;
    for (int kk = 0; kk < sp.k; ++kk) {
        const int sk = sp.row_s ? srow : sp.s[kk];
        int64_t pos = slot_off[(int64_t)kk * (sl.count + 1) + slot] - sp.out_base[kk];
#pragma unroll
        for (int r = 0; r < kTinyMax; ++r)
            if (c[r] >= sk) {
                as_global(sp.col[kk])[pos] = key[r] - id0;
                as_global(sp.w[kk])[pos] = c[r];
                if (sp.row[kk]) as_global(sp.row[kk])[pos] = i - id0;
                ++pos;
            }
    }
}

__global__ __launch_bounds__(256) void light_store_emit_kernel(LightRuns runs, Slots sl, LightStore ls, EmitParams prm,
                                                               const int64_t *__restrict__ slot_off) {
    __shared__ EmitParams sp;
    stage_params(&sp, prm);
    __syncthreads();
    const int lane = lane_id();
    int64_t group;
    const int cls = runs.class_of(blockIdx.x, group);
    const int64_t t = cls ? group * 4 + (threadIdx.x >> 6) : group * 256 + threadIdx.x;
    if (t >= runs.count[cls]) return;
    const int slot = as_global(runs.list[cls])[t];
    if (slot < prm.slot_lo || slot >= prm.slot_hi) return;  // outside the emitted chunk
    if (cls == 0) {
        tiny_store_row(slot, sl, ls, sp, slot_off);
        return;
    }
    const int i = sl.row[slot];
    const int n = as_global(ls.n)[i];
    const int64_t off = as_global(ls.off)[i];
    const int K = prm.k;
    const int64_t S = sl.count;
    const int id0 = prm.row_base ? as_global(prm.row_base)[i] : 0;
    const int srow = prm.row_s ? as_global(prm.row_s)[i] : 0;
    long long b[SLG_MAX_S];
    int sk[SLG_MAX_S];
#pragma unroll
    for (int kk = 0; kk < SLG_MAX_S; ++kk) {
        b[kk] = kk < K ? slot_off[(int64_t)kk * (S + 1) + slot] - sp.out_base[kk] : 0;
        sk[kk] = kk < K ? (prm.row_s ? srow : sp.s[kk]) : INT_MAX;
    }
    for (int r0 = 0; r0 < n; r0 += 64) {
        const int r = r0 + lane;
        const bool in = r < n;
        const int key = in ? as_global(ls.key)[off + r] - id0 : 0;
        const int c = in ? (int)as_global(ls.cnt)[off + r] : 0;
#pragma unroll
        for (int kk = 0; kk < SLG_MAX_S; ++kk) {
            if (kk >= K) break;
            const bool surv = c >= sk[kk];
            const unsigned long long mask = __ballot(surv);
            if (mask == 0ull) break;
            if (surv) {
                const int64_t pos = b[kk] + bits_below(mask);
                as_global(sp.col[kk])[pos] = key;
                as_global(sp.w[kk])[pos] = c;
                if (sp.row[kk]) as_global(sp.row[kk])[pos] = i - id0;
            }
            b[kk] += __popcll(mask);
        }
    }
}

__global__ void light_work_kernel(int64_t m, const uint8_t *__restrict__ rclass, const int64_t *__restrict__ work,
                                  int32_t *__restrict__ lw) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = rclass[i];
        lw[i] = (c >= kLight0 && c < kLight0 + kLightClasses) ? (int32_t)work[i] : 0;
    }
}

template <bool WIDE>
struct CounterCap {  // u16 counters packed in pairs, or u32 counters
    static constexpr int ranks = WIDE ? kRankCap / 2 : kRankCap;
};

constexpr int kThrTable = 128;  // overlaps below this find their threshold by table

struct HeavySmem {
    uint32_t bitmap[kRangeWords];        // partner j of the slot range present
    uint16_t wpre[kRangeWords];          // low 16 bits of the word's exclusive popcount prefix
    uint32_t sup[kSupers + 1];           // full prefix at each superblock start; sup[kSupers] = total
    uint32_t cnt[kRankCap / 2];          // overlap counters of the current rank window
    int32_t buf[kRankCap];               // pass-1 partners, then partner id per rank (emit)
    int32_t seg_a[kHeavyThreads];        // segment start per member of the batch
    int32_t seg_pre[kHeavyThreads + 1];  // flattened start per member of the batch
    int32_t wsum[kHW];
    int32_t nrep;                        // pass-1 repeats (partners already marked)
    int32_t wtot[SLG_MAX_S][kHW];
    unsigned long long acc[SLG_MAX_S];
    long long obase[SLG_MAX_S];
    long long wbase[SLG_MAX_S][kHW];     // output position of each wavefront's first survivor
    uint8_t thr_of[kThrTable];           // threshold index of an overlap value (0xFF: none)
};

// Rank of the first bit of word x (x < number of words in use).
__device__ __forceinline__ uint32_t word_rank(const HeavySmem &sm, int x) {
    const uint32_t base = sm.sup[x / kSuperWords];
    if ((x % kSuperWords) == 0) return base;
    return base + ((uint32_t)(sm.wpre[x] - (uint16_t)base) & 0xFFFFu);
}

// Lay out segments [a, a+len) of one batch of members for the balanced
// walk; returns the batch's 2-path count. Ends with a workgroup barrier.
__device__ __forceinline__ int layout_segments(int a, int len, HeavySmem &sm) {
    const int tid = threadIdx.x;
    int total;
    const int excl = block_excl_scan_open<kHeavyThreads>(len, sm.wsum, total);
    sm.seg_a[tid] = a;
    sm.seg_pre[tid] = excl;
    if (tid == 0) sm.seg_pre[kHeavyThreads] = total;
    __syncthreads();
    return total;
}

// Segment of member q = qb + tid from the boundary table, optionally clipped
// to [ka, kb) by binary search.
template <bool CLIP>
__device__ __forceinline__ void member_segment(const int32_t *__restrict__ vs_idx,
                                               const int32_t *__restrict__ bounds, int64_t bptr,
                                               int k, int qb, int ka, int kb, int &a, int &len) {
    const int q = qb + threadIdx.x;
    a = 0;
    len = 0;
    if (q < k) {
        a = bounds[bptr + q];
        int b = bounds[bptr + k + q];
        if (CLIP && a < b) {
            if (vs_idx[a] < ka) a = lower_bound_i32(vs_idx, a, b, ka);
            if (a < b && vs_idx[b - 1] >= kb) b = lower_bound_i32(vs_idx, a, b, kb);
        }
        len = b > a ? b - a : 0;
    }
}

// Largest u in [lo, hi] with seg_pre[u] <= f (seg_pre is non-decreasing).
__device__ __forceinline__ int segment_of(const int32_t *seg_pre, int lo, int hi, int f) {
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg_pre[mid] <= f)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Calls f(f_idx, j, valid) with every lane of the wavefront for every piece
// of the laid-out segments (valid marks the lanes that hold a partner j,
// f_idx being its position in the batch's flattened 2-path list). Each wavefront takes
// an equal share of the list (so a heavy vertex's tail is shared by all
// wavefronts) and walks it in pieces of 64*kWalkUnroll positions: every
// lane finds the segment of each of its positions by binary search between
// the piece's first and last segment, then issues all its loads together,
// so a piece costs one round trip however many tails it touches.
constexpr int kWalkUnroll = 8;

template <typename F>
__device__ __forceinline__ void walk_segments(const int32_t *__restrict__ vs_idx, int total, int nseg,
                                              const HeavySmem &sm, F &&f) {
    if (total <= 0) return;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int per = (total + kHW - 1) / kHW;
    const int c0 = wave * per;
    const int c1 = min(total, c0 + per);
    if (c0 >= c1) return;
    const int useg = min(nseg, kHeavyThreads) - 1;  // last segment of the batch
    int ufirst = segment_of(sm.seg_pre, 0, useg, c0);
    for (int pb = c0; pb < c1; pb += 64 * kWalkUnroll) {
        const int plast = min(c1, pb + 64 * kWalkUnroll) - 1;
        const int ulast = segment_of(sm.seg_pre, ufirst, useg, plast);
        // the lane's positions search [ufirst, ulast] in lockstep, with a
        // fixed step count, so that their LDS reads overlap
        int fq[kWalkUnroll], u[kWalkUnroll];
#pragma unroll
        for (int r = 0; r < kWalkUnroll; ++r) {
            fq[r] = min(pb + lane + 64 * r, plast);
            u[r] = ufirst;
        }
        for (int len = ulast - ufirst + 1; len > 1;) {
            const int half = len >> 1;
#pragma unroll
            for (int r = 0; r < kWalkUnroll; ++r)
                u[r] = sm.seg_pre[u[r] + half] <= fq[r] ? u[r] + half : u[r];
            len -= half;
        }
        int jr[kWalkUnroll];
#pragma unroll
        for (int r = 0; r < kWalkUnroll; ++r) jr[r] = vs_idx[sm.seg_a[u[r]] + (fq[r] - sm.seg_pre[u[r]])];
#pragma unroll
        for (int r = 0; r < kWalkUnroll; ++r) {
            const int fr = pb + lane + 64 * r;
            f(fr, jr[r], fr <= plast);
        }
        ufirst = ulast;
    }
}

// Largest u in [lo, hi] with seg_pre[u] <= f, for wave-uniform lo, hi and f
// (seg_pre[lo] <= f): every lane tests one of 64 evenly spaced candidates,
// so 512 segments take two LDS round trips.
__device__ __forceinline__ int wave_segment_of(const int32_t *seg_pre, int lo, int hi, int f) {
    const int lane = lane_id();
    while (hi > lo) {
        const int step = (hi - lo + 64) / 64;
        const int cand = lo + lane * step;
        const bool ok = cand <= hi && seg_pre[cand] <= f;
        lo += (__popcll(__ballot(ok)) - 1) * step;  // the candidates that pass form a prefix
        hi = min(hi, lo + step - 1);
    }
    return lo;
}

// Pass 1 of a heavy slot: marks partner j of every laid-out 2-path in the
// bitmap over [ja, ja + span). With RECORD, a 2-path whose partner was
// already marked (a repeat) is appended to buf (up to cap entries; nrep
// counts them all). The walk is that of walk_segments, with each piece's
// atomics issued together and one list reservation per piece.
// Pass 1 takes pieces of 4 positions per lane: a slot holds about 2,600
// 2-paths on the power-law workload, so larger pieces leave wavefronts idle
// at the slot's end (8 positions measured 4 % slower, 16 positions 18 %).
constexpr int kMarkUnroll = 4;

template <bool RECORD>
__device__ __forceinline__ void walk_mark(const int32_t *__restrict__ vs_idx, int total, int nseg, HeavySmem &sm,
                                          int ja, unsigned span, int cap) {
    if (total <= 0) return;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int per = (total + kHW - 1) / kHW;
    const int c0 = wave * per;
    const int c1 = min(total, c0 + per);
    if (c0 >= c1) return;
    const int useg = min(nseg, kHeavyThreads) - 1;
    int ufirst = wave_segment_of(sm.seg_pre, 0, useg, c0);
    for (int pb = c0; pb < c1; pb += 64 * kMarkUnroll) {
        const int plast = min(c1, pb + 64 * kMarkUnroll) - 1;
        const int ulast = wave_segment_of(sm.seg_pre, ufirst, useg, plast);
        int fq[kMarkUnroll], u[kMarkUnroll];
#pragma unroll
        for (int r = 0; r < kMarkUnroll; ++r) {
            fq[r] = min(pb + lane + 64 * r, plast);
            u[r] = ufirst;
        }
        for (int len = ulast - ufirst + 1; len > 1;) {
            const int half = len >> 1;
#pragma unroll
            for (int r = 0; r < kMarkUnroll; ++r)
                u[r] = sm.seg_pre[u[r] + half] <= fq[r] ? u[r] + half : u[r];
            len -= half;
        }
        int jr[kMarkUnroll];
#pragma unroll
        for (int r = 0; r < kMarkUnroll; ++r) jr[r] = vs_idx[sm.seg_a[u[r]] + (fq[r] - sm.seg_pre[u[r]])];
        // rows of the piece past its end are skipped; lanes past it OR
        // nothing into a word of their own bank
        unsigned bit[kMarkUnroll], old[kMarkUnroll];
#pragma unroll
        for (int r = 0; r < kMarkUnroll; ++r) {
            bit[r] = 0u;
            old[r] = 0u;
            if (pb + 64 * r <= plast) {  // wave-uniform
                const unsigned off = (unsigned)(jr[r] - ja);
                const bool ok = pb + lane + 64 * r <= plast && off < span;
                bit[r] = ok ? 1u << (off & 31) : 0u;
                const unsigned word = ok ? off >> 5 : (unsigned)(lane & 31);
                if (RECORD)
                    old[r] = atomicOr(&sm.bitmap[word], bit[r]);
                else
                    atomicOr(&sm.bitmap[word], bit[r]);
            }
        }
        if (RECORD) {
            unsigned long long m[kMarkUnroll];
            int tot = 0;
#pragma unroll
            for (int r = 0; r < kMarkUnroll; ++r) {
                m[r] = __ballot((old[r] & bit[r]) != 0u);
                tot += __popcll(m[r]);
            }
            if (tot) {  // wave-uniform
                int at = 0;
                if (lane == 0) at = atomicAdd(&sm.nrep, tot);
                at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
                for (int r = 0; r < kMarkUnroll; ++r) {
                    if ((old[r] & bit[r]) != 0u) {
                        const int pos = at + bits_below(m[r]);
                        if (pos < cap) sm.buf[pos] = jr[r];
                    }
                    at += __popcll(m[r]);
                }
            }
        }
        ufirst = ulast;
    }
}

// Adds one to rank r's counter and returns the count it held before.
template <bool WIDE>
__device__ __forceinline__ int count_add_rtn(uint32_t *cnt, uint32_t r) {
    if (WIDE) return (int)atomicAdd(&cnt[r], 1u);
    const unsigned sh = (r & 1u) << 4;
    return (int)((atomicAdd(&cnt[r >> 1], 1u << sh) >> sh) & 0xFFFFu);
}

template <bool WIDE>
__device__ __forceinline__ int count_get(const uint32_t *cnt, int r) {
    if (WIDE) return (int)cnt[r];
    return (int)((cnt[r >> 1] >> ((r & 1) << 4)) & 0xFFFFu);
}

// Four 256-thread workgroups per CU (4 waves per SIMD) is what the LDS
// footprint allows; the register budget is held to match (<= 128 VGPRs).
// Four slots in flight per CU hide the latency of each slot's phases.
// STORE (counting pass of non-wide slots): the pass also writes every
// slot's partners and overlaps in rank order, so that the emit pass reads
// them instead of walking the 2-paths again.
template <bool EMIT, bool WIDE, bool STORE>
__global__ __launch_bounds__(kHeavyThreads) __attribute__((amdgpu_waves_per_eu(4))) void heavy_kernel(const HeavyDesc *__restrict__ desc,
                                                              int64_t count, int64_t S,
                                                              const int32_t *__restrict__ bounds,
                                                              const int32_t *__restrict__ vs_idx,
                                                              EmitParams prm,
                                                              int64_t *__restrict__ slot_cnt,
                                                              const int64_t *__restrict__ slot_off,
                                                              unsigned long long *__restrict__ ticket,
                                                              CountStore cs) {
    static_assert(!STORE || (!EMIT && !WIDE), "the store is written by the non-wide counting pass");
    constexpr int kCap = CounterCap<WIDE>::ranks;
    __shared__ HeavySmem sm;
    __shared__ EmitParams sp;  // thresholds and outputs, indexed by a uniform k
    __shared__ int64_t next_pair;  // first slot of the pair claimed to follow the current one
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    stage_params(&sp, prm);
    if (tid == 0) next_pair = (int64_t)atomicAdd(ticket, 2ull);
    for (int x = tid; x < kRangeWords; x += kHeavyThreads) sm.bitmap[x] = 0u;
    for (int x = tid; x < kRankCap / 2; x += kHeavyThreads) sm.cnt[x] = 0u;
    if (tid < SLG_MAX_S * kHW) sm.wtot[tid / kHW][tid % kHW] = 0;
    if (tid < kThrTable) sm.thr_of[tid] = 0xFF;
    __syncthreads();
    if (tid < prm.k && prm.s[tid] < kThrTable) sm.thr_of[prm.s[tid]] = (uint8_t)tid;
    __syncthreads();
    const EmitParams *ep = &sp;
    const int K = prm.k;
    const bool row_thr = prm.row_s != nullptr;  // batched form: one threshold per row
    int64_t pair = next_pair;  // first slot of the current pair
    int64_t it = pair;         // the current slot
    if (it >= count) return;

    // Persistent workgroups claim slots two at a time from a ticket counter.
    // Software pipeline: the claim of the next pair is made during the
    // first slot of the current pair and read one slot later; the next
    // slot's descriptor, output bases, per-row values and this thread's
    // member segment are loaded while the current slot is processed.
    HeavyDesc nd = desc[it];
    int na = 0, nb = 0, nsrow = 0, nid0 = 0;
    int64_t nob = 0;
    auto prefetch = [&](const HeavyDesc &n) {
        if (tid < n.k) {
            na = bounds[n.bptr + tid];
            nb = bounds[n.bptr + n.k + tid];
        }
        if (EMIT && tid < K) nob = slot_off[(int64_t)tid * (S + 1) + n.slot] - ep->out_base[tid];
        if (ep->row_s) nsrow = as_global(ep->row_s)[n.row];  // per-row threshold (batched form)
        if (ep->row_base) nid0 = as_global(ep->row_base)[n.row];
    };
    prefetch(nd);
    unsigned long long claim = 0;  // tid 0's claim of the next pair
    while (true) {
        const HeavyDesc d = nd;
        const int ra = na, rb = nb, srow = nsrow, id0 = nid0;
        const bool first = it == pair;
        if (first && tid == 0) claim = atomicAdd(ticket, 2ull);  // read at the end of this slot

        const int i = d.row, ja = d.ja, jb = d.jb, k = d.k, slot = d.slot;
        const int s_bottom = row_thr ? srow : ep->s[0];   // smallest and largest threshold
        const int s_top = row_thr ? srow : ep->s[K - 1];
        const bool only_presence = !EMIT && !STORE && K == 1 && s_bottom <= 1;
        const int nw = (jb - ja + 31) >> 5;
        const unsigned span = (unsigned)(jb - ja);
        // bitmap and counters are all-zero here: cleared before the first
        // slot and at the end of every slot
        if (tid < SLG_MAX_S) {
            sm.acc[tid] = 0;
            sm.obase[tid] = (EMIT && tid < K) ? nob : 0;
        }
        if (tid == 0) sm.nrep = 0;
        __syncthreads();
        // the pair's second slot, else the first of the claimed pair (published
        // at the end of the current pair's first slot)
        const int64_t it_next = first ? (it + 1 < count ? it + 1 : count) : next_pair;
        const bool have_next = it_next < count;
        if (have_next) nd = desc[it_next];
        bool acc_out = !EMIT;  // slot_cnt takes the per-threshold tallies
        do {
        if (EMIT && (slot < ep->slot_lo || slot >= ep->slot_hi)) {  // outside the emitted chunk
            if (have_next) prefetch(nd);
            break;
        }

        // pass 1: mark every partner j of the slot's range. A 2-path whose
        // partner was already marked is a repeat; repeats are listed in LDS
        // (while they fit), so that pass 2 only has to count them: a
        // partner's overlap is 1 + its number of repeats.
        const bool one_batch = k <= kHeavyThreads;
        int total1 = 0;
        if (one_batch) {
            const int len = (tid < k && rb > ra) ? rb - ra : 0;
            total1 = layout_segments(ra, len, sm);
            walk_mark<true>(vs_idx, total1, k, sm, ja, span, kRankCap);
            __syncthreads();
        } else {
            for (int qb = 0; qb < k; qb += kHeavyThreads) {
                int a, len;
                member_segment<false>(vs_idx, bounds, d.bptr, k, qb, 0, 0, a, len);
                walk_mark<true>(vs_idx, layout_segments(a, len, sm), k - qb, sm, ja, span, kRankCap);
                __syncthreads();
            }
        }
        if (have_next) prefetch(nd);

        // rank of a partner = number of marked partners below it. Each thread
        // owns 8 consecutive bitmap words, read and written 16 bytes at a time
        // (words past the slot's range are zero).
        static_assert(kRangeWords == 8 * kHeavyThreads, "8 bitmap words per thread");
        const uint4 q0 = reinterpret_cast<const uint4 *>(sm.bitmap)[2 * tid];
        const uint4 q1 = reinterpret_cast<const uint4 *>(sm.bitmap)[2 * tid + 1];
        const int loc[8] = {(int)__popc(q0.x), (int)__popc(q0.y), (int)__popc(q0.z), (int)__popc(q0.w),
                            (int)__popc(q1.x), (int)__popc(q1.y), (int)__popc(q1.z), (int)__popc(q1.w)};
        int mine = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) mine += loc[r];
        int distinct;
        int run = block_excl_scan_open<kHeavyThreads>(mine, sm.wsum, distinct);
        if ((tid * 8) % kSuperWords == 0) sm.sup[tid * 8 / kSuperWords] = (uint32_t)run;
        uint32_t pk[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t lo = (uint32_t)run & 0xFFFFu;
            run += loc[2 * r];
            pk[r] = lo | (((uint32_t)run & 0xFFFFu) << 16);
            run += loc[2 * r + 1];
        }
        reinterpret_cast<uint4 *>(sm.wpre)[tid] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        if (tid == 0) sm.sup[kSupers] = (uint32_t)distinct;
        if (STORE && tid == 0) as_global(cs.n)[it] = distinct;
        __syncthreads();

        if (only_presence) {  // L_1 alone: every marked partner is an edge
            if (tid == 0) slot_cnt[slot] = distinct;
            acc_out = false;
            break;
        }

        // windows of at most kCap ranks, cut at word boundaries
        int w0 = 0;
        while (w0 < nw) {
            const uint32_t r0 = word_rank(sm, w0);
            int wl = w0 + 1, wh = nw;
            if ((uint32_t)distinct - r0 <= (uint32_t)kCap) wl = wh = nw;  // one window holds the rest
            while (wl < wh) {
                const int mid = (wl + wh + 1) >> 1;
                if ((mid == nw ? (uint32_t)distinct : word_rank(sm, mid)) - r0 <= (uint32_t)kCap)
                    wl = mid;
                else
                    wh = mid - 1;
            }
            const int w1 = wl;
            const int nr = (int)((w1 == nw ? (uint32_t)distinct : word_rank(sm, w1)) - r0);
            if (nr > 0) {
                const int nwords = WIDE ? nr : (nr + 1) >> 1;
                // every wavefront owns a contiguous range of ranks
                const int per = (((nr + kHW - 1) / kHW) + 63) & ~63;
                const int rlo = wave * per;
                const int rhi = min(nr, rlo + per);
                const bool whole = w0 == 0 && w1 == nw;
                // the repeat list serves every window of the counting pass, and
                // the single window of the emit pass (whose rank-to-partner map
                // reuses the list's storage afterwards)
                const int nrep = sm.nrep;
                const bool by_repeats = nrep <= kRankCap && (whole || !(EMIT || STORE));
                const int c_add = by_repeats ? 1 : 0;  // partners start at overlap 1
                // pass 2: count 2-paths into their partner's rank. The overlap of
                // a partner passes every value up to its final one exactly once,
                // so the 2-path that takes it to s_k makes it a survivor of
                // threshold k: one tally for the wavefront that owns its rank.
                auto add = [&](int, int j, bool valid) {
                    const unsigned off = (unsigned)(j - ja);
                    if (!valid || off >= span) return;
                    const int x = (int)(off >> 5);
                    const uint32_t r = word_rank(sm, x) + __popc(sm.bitmap[x] & ((1u << (off & 31)) - 1u)) - r0;
                    if (r >= (uint32_t)nr) return;
                    const int reached = count_add_rtn<WIDE>(sm.cnt, r) + 1 + c_add;
                    if (reached > s_top) return;
                    int hit = -1;
                    if (row_thr) {
                        hit = reached == srow ? 0 : -1;
                    } else if (reached < kThrTable) {
                        const int t = sm.thr_of[reached];
                        hit = t == 0xFF ? -1 : t;
                    } else {
                        for (int kk = 0; kk < K; ++kk) {
                            const int s = ep->s[kk];
                            if (s >= reached) {
                                hit = s == reached ? kk : -1;
                                break;
                            }
                        }
                    }
                    if (hit >= 0) atomicAdd(&sm.wtot[hit][r / per], 1);
                };
                if (by_repeats) {
                    int f = tid;
                    for (; f + 3 * kHeavyThreads < nrep; f += 4 * kHeavyThreads) {
                        const int j0 = sm.buf[f], j1 = sm.buf[f + kHeavyThreads];
                        const int j2 = sm.buf[f + 2 * kHeavyThreads], j3 = sm.buf[f + 3 * kHeavyThreads];
                        add(f, j0, true);
                        add(f, j1, true);
                        add(f, j2, true);
                        add(f, j3, true);
                    }
                    for (; f < nrep; f += kHeavyThreads) add(f, sm.buf[f], true);
                    __syncthreads();
                } else if (one_batch && whole) {
                    walk_segments(vs_idx, total1, k, sm, add);  // segments of pass 1 still laid out
                    __syncthreads();
                } else {
                    const int ka = ja + 32 * w0;
                    const int kb = min(jb, ja + 32 * w1);
                    for (int qb = 0; qb < k; qb += kHeavyThreads) {
                        int a, len;
                        member_segment<true>(vs_idx, bounds, d.bptr, k, qb, ka, kb, a, len);
                        walk_segments(vs_idx, layout_segments(a, len, sm), k - qb, sm, add);
                        __syncthreads();
                    }
                }
                // threshold 1 over the repeat list: every rank survives
                if (c_add && lane == 0 && s_bottom == 1) sm.wtot[0][wave] = rhi > rlo ? rhi - rlo : 0;
                if (EMIT || STORE) {
                    // partner of every rank of the window: neighbouring threads
                    // take neighbouring words, so a dense stretch of partners is
                    // shared out (4 % faster than each thread's own 8 words)
                    for (int x = w0 + tid; x < w1; x += kHeavyThreads) {
                        unsigned bits = sm.bitmap[x];
                        if (!bits) continue;
                        int rr = (int)(word_rank(sm, x) - r0);
                        const int jbase = ja + 32 * x;
                        do {
                            sm.buf[rr++] = jbase + __ffs(bits) - 1;
                            bits &= bits - 1u;
                        } while (bits);
                    }
                }
                __syncthreads();
                if (STORE) {  // the window's partners and overlaps, coalesced
                    static_assert(kRangeBits <= (1 << 16) && kWideMembers <= (1 << 16), "16-bit store fields");
                    const int64_t base = as_global(cs.off)[it] + r0;
                    for (int r = tid; r < nr; r += kHeavyThreads)  // whole lines, read much later
                        __builtin_nontemporal_store(
                            (uint32_t)(sm.buf[r] - ja) | ((uint32_t)(count_get<WIDE>(sm.cnt, r) + c_add) << 16),
                            &as_global(cs.ent)[base + r]);
                }
                if (tid < K) {  // each threshold's wavefront offsets and total, by one thread
                    long long b = EMIT ? sm.obase[tid] : 0;
#pragma unroll
                    for (int w = 0; w < kHW; ++w) {
                        if (EMIT) sm.wbase[tid][w] = b;
                        b += sm.wtot[tid][w];
                    }
                    if (EMIT)
                        sm.obase[tid] = b;
                    else
                        sm.acc[tid] += (unsigned long long)b;
                }
                if (EMIT && K <= 4) {
                    __syncthreads();
                    // up to four thresholds in one sweep over this wavefront's
                    // ranks: each count and partner is read once, thresholds
                    // and output positions stay in scalar registers
                    int sk4[4], left[4];
                    long long b4[4];
                    int32_t *col4[4], *w4[4], *row4[4];
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        sk4[kk] = uniform(kk < K ? (row_thr ? srow : ep->s[kk]) : INT_MAX);
                        left[kk] = uniform(kk < K ? sm.wtot[kk][wave] : 0);
                        b4[kk] = uniform(kk < K ? sm.wbase[kk][wave] : 0ll);
                        col4[kk] = uniform(kk < K ? ep->col[kk] : nullptr);
                        w4[kk] = uniform(kk < K ? ep->w[kk] : nullptr);
                        row4[kk] = uniform(kk < K ? ep->row[kk] : nullptr);
                    }
                    for (int rbase = rlo; rbase < rhi && left[0] + left[1] + left[2] + left[3] > 0; rbase += 64) {
                        const int r = rbase + lane;
                        const int c = r < rhi ? count_get<WIDE>(sm.cnt, r) + c_add : 0;
                        const bool any = c >= sk4[0];  // thresholds increase
                        const int key = any ? sm.buf[r] - id0 : 0;
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) {
                            if (left[kk] == 0) continue;  // wave-uniform
                            const bool surv = c >= sk4[kk];
                            const unsigned long long mask = __ballot(surv);
                            if (surv) {
                                const int64_t pos = b4[kk] + bits_below(mask);
                                as_global(col4[kk])[pos] = key;
                                as_global(w4[kk])[pos] = c;
                                if (row4[kk]) as_global(row4[kk])[pos] = i - id0;
                            }
                            b4[kk] += __popcll(mask);
                            left[kk] -= __popcll(mask);
                        }
                    }
                } else if (EMIT) {
                    __syncthreads();
                    // per threshold, this wavefront's survivors in rank order,
                    // compacted with ballots into consecutive positions
                    for (int kk = 0; kk < K; ++kk) {
                        int left = sm.wtot[kk][wave];
                        if (left == 0) continue;
                        const int sk = row_thr ? srow : ep->s[kk];
                        int64_t base = sm.wbase[kk][wave];
                        const auto colp = as_global(ep->col[kk]);
                        const auto wp = as_global(ep->w[kk]);
                        const auto rowp = as_global(ep->row[kk]);
                        // two groups of 64 ranks per step: their LDS reads overlap
                        for (int rbase = rlo; rbase < rhi && left > 0; rbase += 128) {
                            const int ra_ = rbase + lane, rb_ = rbase + 64 + lane;
                            const int ca = ra_ < rhi ? count_get<WIDE>(sm.cnt, ra_) + c_add : 0;
                            const int cb = rb_ < rhi ? count_get<WIDE>(sm.cnt, rb_) + c_add : 0;
                            const bool sa = ca >= sk, sb = cb >= sk;
                            const int ka_ = sa ? sm.buf[ra_] : 0;
                            const int kb_ = sb ? sm.buf[rb_] : 0;
                            const unsigned long long ma = __ballot(sa), mb = __ballot(sb);
                            const int na_ = __popcll(ma);
                            if (sa) {
                                const int64_t pos = base + bits_below(ma);
                                colp[pos] = ka_ - id0;
                                wp[pos] = ca;
                                if (rowp) rowp[pos] = i - id0;
                            }
                            if (sb) {
                                const int64_t pos = base + na_ + bits_below(mb);
                                colp[pos] = kb_ - id0;
                                wp[pos] = cb;
                                if (rowp) rowp[pos] = i - id0;
                            }
                            base += na_ + __popcll(mb);
                            left -= na_ + __popcll(mb);
                        }
                    }
                }
                __syncthreads();
                for (int x = tid; x < nwords; x += kHeavyThreads) sm.cnt[x] = 0u;
                if (tid < SLG_MAX_S * kHW) sm.wtot[tid / kHW][tid % kHW] = 0;
                if (w1 < nw) __syncthreads();  // the next window counts into cleared counters
            }
            w0 = w1;
        }
        } while (false);
        for (int x = tid; x < nw; x += kHeavyThreads) sm.bitmap[x] = 0u;
        if (first && tid == 0) next_pair = (int64_t)claim;
        __syncthreads();
        if (acc_out && tid < K) slot_cnt[(int64_t)tid * S + slot] = (int64_t)sm.acc[tid];
        if (!have_next) break;
        if (!first) pair = it_next;
        it = it_next;
    }
}

// 2-paths of every heavy slot: the lengths of its members' segments in the
// boundary table, one wavefront per slot.
__global__ __launch_bounds__(256) void slot_work_kernel(const HeavyDesc *__restrict__ desc, int64_t count,
                                                        const int32_t *__restrict__ bounds,
                                                        int64_t *__restrict__ work) {
    const int lane = lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64; t < count; t += nwaves) {
        const HeavyDesc d = desc[t];
        int64_t w = 0;
        for (int q = lane; q < d.k; q += 64) w += bounds[d.bptr + d.k + q] - bounds[d.bptr + q];
        w = wave_sum(w);
        if (lane == 0) work[t] = w;
    }
}

// Emit pass of the heavy slots from the counting pass's store: one
// wavefront per slot reads its entries in rank (partner id) order, eight
// groups of 64 ranks per step (all loads issued before any is used). Each
// threshold's survivors are compacted with ballots into a small LDS queue
// of the wavefront and written out 64 at a time, so that every global store
// is a full 256-byte row even for sparse thresholds, the first one cut so
// that the rest are aligned and past the caches (2.1e9 edges, 33 GB: 8.8 ms
// as they come, 8.0 aligned, 7.2 and 4.6 TB/s past the caches; kernels whose
// writes end within lines lose by that, the light rows' 0.81 -> 1.03 ms);
// what is left is written at the end of the slot. Thresholds increase, so a group
// with no survivor of s_k has none of the larger ones either. MAXK: 4 for
// ensembles of up to four thresholds, else SLG_MAX_S (no queues).
constexpr int kStoreGroups = 8;
constexpr int kQueue = 128;  // entries per threshold queue: < 64 kept + <= 64 appended

// Entries are (partner - ja) | overlap << 16. DENSE: ja is a window of E_s
// positions and the partner's id is cid_row[ja + low half], looked up for a
// whole group of entries at once (the lookups overlap) before they are
// queued as id << 16 | overlap. Slots are taken in list (row) order, so the
// outputs are written in order; taking them window by window kept cid_row
// in L2 but scattered the writes, and measured a third slower.
template <int MAXK, bool DENSE>
__global__ __launch_bounds__(256) void heavy_store_emit_kernel(const HeavyDesc *__restrict__ desc, int64_t count,
                                                               int64_t S, CountStore cs, EmitParams prm,
                                                               const int64_t *__restrict__ slot_off,
                                                               const int32_t *__restrict__ cid_row) {
    using E = uint32_t;                                        // stored entry
    using Q = typename std::conditional<DENSE, unsigned long long, uint32_t>::type;  // queued entry
    constexpr bool kQueued = MAXK <= 4;
    __shared__ EmitParams sp;
    __shared__ Q queue[kQueued ? 4 : 1][kQueued ? MAXK : 1][kQueued ? kQueue : 1];
    stage_params(&sp, prm);
    __syncthreads();
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int K = prm.k;
    const bool row_thr = prm.row_s != nullptr;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    // one slot: its stored entries to the outputs of every threshold
    auto emit_slot = [&](int64_t t) {
        const HeavyDesc d = desc[t];
        if (d.slot < prm.slot_lo || d.slot >= prm.slot_hi) return;  // outside the emitted chunk
        const int n = as_global(cs.n)[t];
        if (n < 0) return;  // the store was full: the slot's emit walks its 2-paths again
        const int64_t off = as_global(cs.off)[t];
        const int i = d.row;
        const int id0 = prm.row_base ? as_global(prm.row_base)[i] : 0;
        const int srow = row_thr ? as_global(prm.row_s)[i] : 0;
        const int jbase = d.ja - id0;
        const int32_t *crow = DENSE ? cid_row + d.ja : nullptr;
        long long b[MAXK];
        int sk[MAXK], fill[MAXK], need[MAXK];
#pragma unroll
        for (int kk = 0; kk < MAXK; ++kk) {
            b[kk] = kk < K ? slot_off[(int64_t)kk * (S + 1) + d.slot] - sp.out_base[kk] : 0;
            need[kk] = uniform(64 - (int)(b[kk] & 63));
            sk[kk] = kk < K ? (row_thr ? srow : sp.s[kk]) : INT_MAX;
            fill[kk] = 0;
        }
        // queued entry: DENSE, the partner's id << 16 | overlap; else the stored entry
        auto partner = [&](Q e) -> int {
            return DENSE ? (int)(e >> 16) - id0 : jbase + (int)(e & 0xFFFFu);
        };
        auto overlap = [&](Q e) -> int { return DENSE ? (int)(e & 0xFFFFu) : (int)(e >> 16); };
        // writes `m` queued entries of threshold kk (lanes below m) at b[kk]
        auto flush = [&](int kk, int m) {
            if (lane < m) {
                const Q e = queue[wave][kk][lane];
                const int64_t pos = b[kk] + lane;
                __builtin_nontemporal_store(partner(e), as_global(sp.col[kk]) + pos);
                __builtin_nontemporal_store(overlap(e), as_global(sp.w[kk]) + pos);
                if (sp.row[kk]) __builtin_nontemporal_store(i - id0, as_global(sp.row[kk]) + pos);
            }
            b[kk] += m;
        };
        for (int r0 = 0; r0 < n; r0 += 64 * kStoreGroups) {
            E e[kStoreGroups];
#pragma unroll
            for (int q = 0; q < kStoreGroups; ++q) {
                const int r = r0 + 64 * q + lane;
                e[q] = r < n ? as_global(cs.ent)[off + r] : E(0);
            }
            Q v[kStoreGroups];
#pragma unroll
            for (int q = 0; q < kStoreGroups; ++q) {
                if (DENSE)
                    v[q] = r0 + 64 * q + lane < n
                               ? ((Q)(uint32_t)as_global(crow)[e[q] & 0xFFFFu] << 16) | (Q)(e[q] >> 16)
                               : Q(0);
                else
                    v[q] = (Q)e[q];
            }
#pragma unroll
            for (int q = 0; q < kStoreGroups; ++q) {
                if (r0 + 64 * q >= n) break;  // wave-uniform
                const int c = overlap(v[q]);
#pragma unroll
                for (int kk = 0; kk < MAXK; ++kk) {
                    if (kk >= K) break;
                    const bool surv = c >= sk[kk];
                    const unsigned long long mask = __ballot(surv);
                    if (mask == 0ull) break;
                    if (kQueued) {
                        if (surv) queue[wave][kk][fill[kk] + bits_below(mask)] = v[q];
                        fill[kk] += __popcll(mask);
                        if (fill[kk] >= need[kk]) {  // up to the end of a row out, the rest moves down
                            wave_lds_sync();
                            flush(kk, need[kk]);
                            const int left = fill[kk] - need[kk];
                            const Q rest = lane < left ? queue[wave][kk][need[kk] + lane] : Q(0);
                            wave_lds_sync();
                            if (lane < left) queue[wave][kk][lane] = rest;
                            fill[kk] = left;
                            need[kk] = 64;
                        }
                    } else if (surv) {
                        const int64_t pos = b[kk] + bits_below(mask);
                        as_global(sp.col[kk])[pos] = partner(v[q]);
                        as_global(sp.w[kk])[pos] = c;
                        if (sp.row[kk]) as_global(sp.row[kk])[pos] = i - id0;
                    }
                    if (!kQueued) b[kk] += __popcll(mask);
                }
            }
        }
        if (kQueued) {
            wave_lds_sync();
#pragma unroll
            for (int kk = 0; kk < MAXK; ++kk)
                if (kk < K && fill[kk] > 0) flush(kk, fill[kk]);
            wave_lds_sync();  // the queues are reused by the next slot
        }
    };
    for (int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64; t < count; t += nwaves) emit_slot(t);
}

__global__ void sum_i32_kernel(const int32_t *__restrict__ n, int64_t count, unsigned long long *__restrict__ out) {
    unsigned long long acc = 0;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x)
        acc += (unsigned long long)n[t];
    acc = wave_sum(acc);
    if (lane_id() == 0 && acc) atomicAdd(out, acc);
}

// Edges of every threshold emitted by heavy slots (for measurement).
__global__ __launch_bounds__(256) void heavy_edges_kernel(const HeavyDesc *__restrict__ desc,
                                                          int64_t count, const int64_t *__restrict__ slot_cnt,
                                                          int64_t S, int32_t K,
                                                          unsigned long long *__restrict__ out) {
    __shared__ unsigned long long ws[4];
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long sum = 0;
    if (t < count) {
        const int slot = desc[t].slot;
        for (int k = 0; k < K; ++k) sum += (unsigned long long)slot_cnt[(int64_t)k * S + slot];
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long b = ws[0] + ws[1] + ws[2] + ws[3];
        if (b) atomicAdd(out, b);
    }
}

template <int AHEAD>
__device__ __forceinline__ void bound_members(const HeavyDesc &d, int64_t p0, const int32_t *__restrict__ vs_idx,
                                              const int32_t *__restrict__ tail_beg,
                                              const int32_t *__restrict__ tail_end, int32_t *__restrict__ bounds) {
    for (int q0 = lane_id(); q0 < d.k; q0 += 64 * AHEAD) {
        int lo[AHEAD], hi[AHEAD], end[AHEAD], first[AHEAD], last[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const bool in = q0 + 64 * u < d.k;
            lo[u] = in ? tail_beg[p0 + q0 + 64 * u] : 0;
            hi[u] = end[u] = in ? tail_end[p0 + q0 + 64 * u] : 0;
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const bool some = lo[u] < hi[u];
            first[u] = some ? vs_idx[lo[u]] : INT_MAX;
            last[u] = some ? vs_idx[hi[u] - 1] : INT_MAX;
        }
        bool more = false;
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (first[u] >= d.ja)
                hi[u] = lo[u];  // an empty tail too
            else if (last[u] < d.ja)
                lo[u] = hi[u];
            more |= lo[u] < hi[u];
        }
        while (more) {
            int mid[AHEAD], x[AHEAD];
            more = false;
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                mid[u] = middle(lo[u], hi[u]);
                x[u] = lo[u] < hi[u] ? vs_idx[mid[u]] : 0;
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if (lo[u] >= hi[u]) continue;
                if (x[u] < d.ja)
                    lo[u] = mid[u] + 1;
                else
                    hi[u] = mid[u];
                more |= lo[u] < hi[u];
            }
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int q = q0 + 64 * u;
            if (q >= d.k) continue;
            bounds[d.bptr + q] = lo[u];
            if (d.last) bounds[d.bptr + d.k + q] = end[u];
        }
    }
}

// One wavefront per heavy slot: the segment start of every member of the
// row at the slot's first partner id (and, on the row's last slot, the
// tail end). Partners of member q form a sorted tail, so the start is a
// lower bound; quick tests skip the search when the tail misses the slot.
__global__ __launch_bounds__(256) void bounds_kernel(
    const HeavyDesc *__restrict__ desc, int64_t count, const int64_t *__restrict__ he_ptr,
    const int32_t *__restrict__ vs_idx, const int32_t *__restrict__ tail_beg,
    const int32_t *__restrict__ tail_end, int32_t *__restrict__ bounds) {
    // workgroups are dealt to the 8 XCDs in turn; each XCD takes runs of 16
    // consecutive blocks (64 slots) instead, so that a row's slots (which
    // search the same vertex lists) mostly share one L2, while the runs
    // still rotate over the XCDs (rows of very different cost, e.g. sorted
    // by size, stay spread). The tail past whole rounds keeps its place.
    constexpr uint32_t kRun = 16;
    const uint32_t nb = gridDim.x, b = blockIdx.x, q = b / 8u;
    const uint32_t blk = b >= nb / (8u * kRun) * (8u * kRun) ? b : q / kRun * (8u * kRun) + b % 8u * kRun + q % kRun;
    const int lane = lane_id();
    const int64_t w = ((int64_t)blk * blockDim.x + threadIdx.x) / 64;
    if (w >= count) return;
    const HeavyDesc d = desc[w];
    const int64_t p0 = he_ptr[d.row];
    // bound by the dependent loads of a search: in rows that give a lane more
    // than one member, they are searched in lockstep (200 000 rows of a dual
    // hypergraph: 1.45 -> 1.19 ms; in fours for every row, shorter rows lose)
    if (d.k <= 64)
        bound_members<1>(d, p0, vs_idx, tail_beg, tail_end, bounds);
    else if (d.k <= 128)
        bound_members<2>(d, p0, vs_idx, tail_beg, tail_end, bounds);
    else
        bound_members<4>(d, p0, vs_idx, tail_beg, tail_end, bounds);
}

// ---------------------------------------------------------------------------
// K3-K5 dense tier: one workgroup per slot, direct LDS counters
// ---------------------------------------------------------------------------
// A dense slot is a row i and an aligned window [ja, ja + kDenseWindow) of
// E_s positions; its 2-paths are the parts of its members' tails that fall
// in the window (vertex lists in E_s positions, so the counter of partner c
// is c - ja with no search). One u32 counter per position. The walk reads
// the lists as 16-bit places in the window (c - ja = c mod kDenseWindow,
// since windows are aligned): 2 bytes per 2-path instead of 4 (6.5 % off
// the counting pass), and the counter's byte address is one shift, so a
// 2-path costs one load, one shift and one LDS add. A row of fewer than
// 2^16 members cannot reach 2^16 in a counter (the store keeps 16 bits).
constexpr int kDW = kDenseThreads / 64;                       // wavefronts per dense workgroup
constexpr int kDenseWordsPer = kDenseWindow / kDenseThreads;  // counters per thread (32)
constexpr int kDenseUnroll = 16;                              // loads in flight per lane
constexpr int kDensePiece = 64 * kDenseUnroll;                // 2-paths per wavefront step
// vs_win is allocated kDensePad entries longer: a step inside one tail
// loads whole rows past the tail's end (those values are not counted)
static_assert(kDensePad >= kDensePiece, "padding of the E_s-position lists");
static_assert(kDenseWordsPer % 4 == 0, "16-byte LDS accesses");
static_assert(kWideMembers < (1 << 16), "16-bit overlaps in the dense store");

struct DenseSmem {
    uint32_t cnt[kDenseWindow + 4];      // counters (and 4 spare words)
    int32_t seg_a[kDenseThreads];        // segment start per member of the batch
    int32_t seg_pre[kDenseThreads + 1];  // flattened start per member of the batch
    int32_t wsum[2][kDW];                // wavefront totals of a scan (two, used in turn)
    unsigned long long tally[SLG_MAX_S];
    long long base;                      // store room of the slot (or -1)
    long long chunk_at, chunk_end;       // the workgroup's store room not yet handed out
    int64_t next[2];                     // tickets claimed ahead, by slot parity
    int32_t tn;                          // the following slot's position in the descriptor list
};

// Exclusive scan over the dense workgroup. wsum is read after the scan's
// barrier: the next scan takes the other buffer, so that no second barrier
// is needed.
__device__ __forceinline__ int dense_scan(int x, int32_t *wsum, int &total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int incl = wave_incl_scan(x);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kDW; ++w) {
        const int t = wsum[w];
        pre += (w < wave) ? t : 0;
        tot += t;
    }
    total = tot;
    return pre + incl - x;
}

// Adds one to the counter at byte offset a of the counters.
__device__ __forceinline__ void dense_add(DenseSmem &sm, uint32_t a) {
    atomicAdd(reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(sm.cnt) + a), 1u);
}

// Walks the laid-out segments (2-path f of the batch is member u's tail
// position seg_a[u] + f - seg_pre[u], whose place in the window is
// vs_win[that position]) and adds one to the counter of each
// partner. Each wavefront takes an equal share of the flattened list, in
// steps of kDensePiece positions whose loads are all issued first. The
// wavefront keeps its current tail (start and end) in scalar registers: a
// step inside it (the common case: the 2-paths of a dense slot come mostly
// from long tails) takes one address and the loads' immediate offsets, with
// no LDS lookup; a step across tails finds each position's tail by binary
// search. (Keeping the next step's loads in flight while adding the
// current one's measured the same: the walk is not bound by load latency.)
__device__ __forceinline__ void dense_walk(const uint16_t *__restrict__ vs_win, int total, int nseg,
                                           DenseSmem &sm) {
    if (total <= 0) return;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int per = (total + kDW - 1) / kDW;
    const int c0 = wave * per;
    const int c1 = min(total, c0 + per);
    if (c0 >= c1) return;
    const int useg = min(nseg, kDenseThreads) - 1;
    // tail u covers flattened positions [seg_pre[u], uend); position f of it
    // is vs_win[ubase + f]
    int u = wave_segment_of(sm.seg_pre, 0, useg, c0);
    int uend = uniform(sm.seg_pre[u + 1]);
    int ubase = uniform(sm.seg_a[u] - sm.seg_pre[u]);
    // adds the step at b (its positions up to c1 - 1) from values c
    auto add_step = [&](const int (&c)[kDenseUnroll], int b) {
        const int last = min(c1, b + kDensePiece) - 1;
        if (last == b + kDensePiece - 1) {  // wave-uniform: every position of the step counts
#pragma unroll
            for (int r = 0; r < kDenseUnroll; ++r) dense_add(sm, (uint32_t)c[r] * 4u);
        } else {
#pragma unroll
            for (int r = 0; r < kDenseUnroll; ++r)
                if (b + lane + 64 * r <= last) dense_add(sm, (uint32_t)c[r] * 4u);
        }
    };
    int pb = c0;
    while (pb < c1) {
        if (pb >= uend) {
            u = wave_segment_of(sm.seg_pre, u, useg, pb);
            uend = uniform(sm.seg_pre[u + 1]);
            ubase = uniform(sm.seg_a[u] - sm.seg_pre[u]);
        }
        const int plast = min(c1, pb + kDensePiece) - 1;
        if (plast < uend) {
            // a step inside tail u
            const uint16_t *src = vs_win + ((int64_t)ubase + lane);
            int ca[kDenseUnroll];
#pragma unroll
            for (int r = 0; r < kDenseUnroll; ++r) ca[r] = src[pb + 64 * r];
            add_step(ca, pb);
            pb += kDensePiece;
        } else {
            const int ulast = wave_segment_of(sm.seg_pre, u, useg, plast);
            constexpr int kHalf = kDenseUnroll / 2;
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                const int hb = pb + 64 * kHalf * h;
                if (hb > plast) break;  // wave-uniform
                int fq[kHalf], uq[kHalf], c[kHalf];
#pragma unroll
                for (int r = 0; r < kHalf; ++r) {
                    fq[r] = min(hb + lane + 64 * r, plast);
                    uq[r] = u;
                }
                for (int len = ulast - u + 1; len > 1;) {
                    const int half = len >> 1;
#pragma unroll
                    for (int r = 0; r < kHalf; ++r)
                        uq[r] = sm.seg_pre[uq[r] + half] <= fq[r] ? uq[r] + half : uq[r];
                    len -= half;
                }
#pragma unroll
                for (int r = 0; r < kHalf; ++r) c[r] = vs_win[sm.seg_a[uq[r]] + (fq[r] - sm.seg_pre[uq[r]])];
#pragma unroll
                for (int r = 0; r < kHalf; ++r)
                    if (hb + lane + 64 * r <= plast) dense_add(sm, (uint32_t)c[r] * 4u);
            }
            u = ulast;
            uend = uniform(sm.seg_pre[u + 1]);
            ubase = uniform(sm.seg_a[u] - sm.seg_pre[u]);
            pb += kDensePiece;
        }
    }
}

// EMIT = false: the counting pass. Every threshold's survivors are tallied
// into slot_cnt; with a store, the survivors of the smallest threshold are
// kept, in partner order, for the emit pass. EMIT = true: the emit pass of
// the slots without stored survivors (every slot when there is no store),
// writing each threshold's edges in partner order at the slot's offsets.
// Persistent workgroups take slots from a ticket counter; two fit per CU
// (LDS), which takes at most 128 VGPRs (4 waves per SIMD). The next slot's
// ticket, position, descriptor and first member segments are loaded while
// the current slot is counted, so that a slot starts with no global round
// trip. Store room is taken kDenseChunk entries at a time per workgroup
// (one global atomic per chunk rather than per slot); cursor[0] is the room
// taken, cursor[1] and cursor[2] sum the survivors asked for and kept.
template <bool EMIT>
__global__ __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(4))) void dense_kernel(const HeavyDesc *__restrict__ desc, int64_t count,
                                                              const int32_t *__restrict__ order,
                                                              int64_t S, const int32_t *__restrict__ bounds,
                                                              const uint16_t *__restrict__ vs_win,
                                                              const int32_t *__restrict__ cid_row, EmitParams prm,
                                                              int64_t *__restrict__ slot_cnt,
                                                              const int64_t *__restrict__ slot_off,
                                                              unsigned long long *__restrict__ ticket,
                                                              CountStore cs, unsigned long long *__restrict__ cursor,
                                                              int64_t cap) {
    __shared__ DenseSmem sm;
    __shared__ EmitParams sp;
    const int tid = threadIdx.x, lane = lane_id();
    stage_params(&sp, prm);
    for (int x = tid; x < kDenseWindow + 4; x += kDenseThreads) sm.cnt[x] = 0u;
    if (tid == 0) {
        sm.next[0] = (int64_t)atomicAdd(ticket, 1ull);
        sm.chunk_at = 0;
        sm.chunk_end = 0;
    }
    __syncthreads();
    const int K = sp.k;
    const bool store = cs.ent != nullptr;
    // the slot of ticket tk: its position in desc (window-major order) and
    // descriptor; this thread's member segment of its first batch
    auto slot_of = [&](int64_t tk) -> int64_t { return order ? (int64_t)order[tk] : tk; };
    auto first_segment = [&](const HeavyDesc &d, int &a, int &len) {
        a = 0;
        len = 0;
        if (tid < d.k) {
            a = bounds[d.bptr + tid];
            const int b = bounds[d.bptr + d.k + tid];
            len = b > a ? b - a : 0;
        }
    };
    // zero, in a form the compiler treats as varying by lane: a load indexed
    // with it is a vector load (waited for with the vector loads, not with
    // every LDS access as a scalar load would be)
    const int64_t lane_zero = (int64_t)lane * (count >> 62);
    int64_t tk = uniform((long long)sm.next[0]);
    if (tid == 0) sm.next[1] = (int64_t)atomicAdd(ticket, 1ull);  // the following slot
    int par = 1;  // next[par] holds the following slot's ticket
    int64_t t = 0;
    HeavyDesc d{};
    int a0 = 0, len0 = 0;
    if (tk < count) {
        t = uniform((long long)slot_of(tk));
        d = desc[t];
        first_segment(d, a0, len0);
    }
    while (tk < count) {
        // the following slot's ticket is in next[par]; the previous slot's
        // counters are cleared and its reads of the shared arrays are done
        __syncthreads();
        const int64_t tkn = uniform((long long)sm.next[par]);
        // the following slot's position, loaded by one lane now and shared
        // through LDS after the walk (a scalar load would be waited for at
        // the walk's first LDS access)
        int tn_v = 0;
        if (tid == 0 && tkn < count) tn_v = order ? order[tkn + lane_zero] : (int)tkn;
        const int ja = uniform(d.ja), k = uniform(d.k);
        bool skip = false;
        if (EMIT) skip = d.slot < sp.slot_lo || d.slot >= sp.slot_hi || (store && as_global(cs.n)[t] >= 0);
        if (tid < SLG_MAX_S) sm.tally[tid] = 0ull;
        if (!skip && k > 0) {  // workgroup-uniform
            // count: every member's part of its tail inside the window
            for (int qb = 0; qb < k; qb += kDenseThreads) {
                int a = a0, len = len0;
                if (qb > 0) {
                    const int q = qb + tid;
                    a = 0;
                    len = 0;
                    if (q < k) {
                        a = bounds[d.bptr + q];
                        const int b = bounds[d.bptr + k + q];
                        len = b > a ? b - a : 0;
                    }
                }
                int total;
                const int excl = dense_scan(len, sm.wsum[0], total);
                sm.seg_a[tid] = a;
                sm.seg_pre[tid] = excl;
                if (tid == 0) sm.seg_pre[kDenseThreads] = total;
                __syncthreads();
                dense_walk(vs_win, total, k - qb, sm);
                if (tid == 0) sm.tn = tn_v;
                __syncthreads();
            }
        } else {
            if (tid == 0) sm.tn = tn_v;
            __syncthreads();
        }
        // the slot after the following one (next[par ^ 1] was read before this slot's first barrier)
        if (tid == 0) sm.next[par ^ 1] = (int64_t)atomicAdd(ticket, 1ull);
        par ^= 1;
        const int64_t tn = tkn < count ? (int64_t)sm.tn : 0;
        HeavyDesc dn{};
        if (tkn < count) dn = desc[tn + lane_zero];  // vector loads: waited for at the next slot's start
        int an = 0, lenn = 0;
        // this thread's counters: positions [tid * 32, tid * 32 + 32), read
        // 16 bytes at a time; `f(position, count)` sees each in order, and
        // with `clear` they are zeroed for the next slot. A compiler barrier
        // keeps every pass a fresh read.
        auto for_words = [&](bool clear, auto &&f) {
            __asm__ volatile("" ::: "memory");
            uint4 *q = reinterpret_cast<uint4 *>(sm.cnt) + tid * (kDenseWordsPer / 4);
#pragma unroll 2
            for (int r = 0; r < kDenseWordsPer / 4; ++r) {
                const uint4 v = q[r];
                const int x = tid * kDenseWordsPer + 4 * r;
                f(x, v.x);
                f(x + 1, v.y);
                f(x + 2, v.z);
                f(x + 3, v.w);
                if (clear) q[r] = make_uint4(0u, 0u, 0u, 0u);
            }
        };
        const unsigned s0 = (unsigned)sp.s[0];
        const auto crow = as_global(cid_row) + ja;
        if (skip) {
            if (tkn < count) first_segment(dn, an, lenn);
        } else if (!EMIT) {
            // every threshold's survivors (one pass for up to two
            // thresholds), then the survivors of the smallest kept in the store
            int n0 = 0;
            if (K <= 2) {
                const unsigned s1 = K > 1 ? (unsigned)sp.s[1] : ~0u;
                int n1 = 0;
                for_words(!store, [&](int, unsigned v) {
                    n0 += v >= s0;
                    n1 += v >= s1;
                });
                n1 = wave_sum(n1);
                if (K > 1 && lane == 0 && n1) atomicAdd(&sm.tally[1], (unsigned long long)n1);
            } else {
                for (int kk = 1; kk < K; ++kk) {
                    const unsigned sk = (unsigned)sp.s[kk];
                    int c = 0;
                    for_words(false, [&](int, unsigned v) { c += v >= sk; });
                    c = wave_sum(c);
                    if (lane == 0 && c) atomicAdd(&sm.tally[kk], (unsigned long long)c);
                }
                for_words(!store, [&](int, unsigned v) { n0 += v >= s0; });
            }
            int n;
            const int pos0 = dense_scan(n0, sm.wsum[1], n);
            if (tkn < count) first_segment(dn, an, lenn);  // the descriptor has arrived by now
            if (tid == 0) sm.tally[0] = (unsigned long long)n;
            if (store && tid == 0) {  // room for the slot's survivors, from the workgroup's chunk
                long long b = -1;
                if (n > 0) {
                    if ((long long)n > sm.chunk_end - sm.chunk_at) {
                        // a chunk, or less in a small store (a quarter of it over the workgroups)
                        long long want = cap / (4ll * (long long)gridDim.x);
                        want = want < kDenseChunk ? want : kDenseChunk;
                        want = (long long)n > want ? (long long)n : want;
                        const long long at = (long long)atomicAdd(cursor, (unsigned long long)want);
                        sm.chunk_at = at;
                        sm.chunk_end = at + want <= cap ? at + want : (at + n <= cap ? at + n : at);
                    }
                    if ((long long)n <= sm.chunk_end - sm.chunk_at) {
                        b = sm.chunk_at;
                        sm.chunk_at += n;
                        atomicAdd(cursor + 2, (unsigned long long)n);
                    }
                    atomicAdd(cursor + 1, (unsigned long long)n);
                }
                sm.base = b;
                as_global(cs.off)[t] = b < 0 ? 0 : b;
                as_global(cs.n)[t] = (n > 0 && b < 0) ? -1 : n;
            }
            __syncthreads();
            if (store) {  // window position | overlap << 16
                const long long base = sm.base;
                const auto ent = as_global(cs.ent);
                long long q0 = base + pos0;
                for_words(true, [&](int x, unsigned v) {
                    if (base >= 0 && v >= s0) ent[q0++] = (uint32_t)x | (v << 16);
                });
            }
            if (tid < K) slot_cnt[(int64_t)tid * S + d.slot] = (int64_t)sm.tally[tid];
        } else {
            // per threshold, this slot's survivors in partner order
            if (tkn < count) first_segment(dn, an, lenn);
            const int i = d.row;
            for (int kk = 0; kk < K; ++kk) {
                const unsigned sk = (unsigned)sp.s[kk];
                int n0 = 0;
                for_words(false, [&](int, unsigned v) { n0 += v >= sk; });
                int tot;
                const int pos0 = dense_scan(n0, sm.wsum[(kk + 1) & 1], tot);
                if (tot == 0) break;  // workgroup-uniform: larger thresholds have none either
                const int64_t b = slot_off[(int64_t)kk * (S + 1) + d.slot] - sp.out_base[kk];
                const auto colp = as_global(sp.col[kk]);
                const auto wp = as_global(sp.w[kk]);
                const auto rowp = as_global(sp.row[kk]);
                int64_t q0 = b + pos0;
                for_words(false, [&](int x, unsigned v) {
                    if (v >= sk) {
                        colp[q0] = crow[x];
                        wp[q0] = (int)v;
                        if (rowp) rowp[q0] = i;
                        ++q0;
                    }
                });
            }
            for_words(true, [](int, unsigned) {});  // cleared for the next slot
        }
        tk = tkn;
        t = tn;
        d = dn;
        a0 = an;
        len0 = lenn;
    }
}

__global__ void dense_keys_kernel(const HeavyDesc *__restrict__ desc, int64_t count, int32_t *__restrict__ key,
                                  int32_t *__restrict__ id) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    key[t] = desc[t].ja >> kDenseBits;
    id[t] = (int32_t)t;
}

// ---------------------------------------------------------------------------
// K6: CSR row pointers from slot offsets
// ---------------------------------------------------------------------------
__global__ void row_ptr_kernel(int64_t row_lo, int64_t row_hi, const int64_t *__restrict__ slot_base,
                               const int64_t *__restrict__ slot_off, int64_t S, EmitParams prm) {
    __shared__ EmitParams sp;
    stage_params(&sp, prm);
    __syncthreads();
    const int64_t i = row_lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > row_hi) return;
    const int64_t sb = slot_base[i];
    for (int k = 0; k < sp.k; ++k)
        as_global(sp.row_ptr[k])[i - row_lo] = slot_off[(int64_t)k * (S + 1) + sb] - sp.out_base[k];
}

// Output bytes of rows [0, i) over all thresholds, i in [0, m].
__global__ void row_bytes_kernel(int64_t m, const int64_t *__restrict__ slot_base,
                                 const int64_t *__restrict__ slot_off, int64_t S, int32_t K,
                                 int64_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > m) return;
    const int64_t sb = slot_base[i];
    int64_t b = 0;
    for (int k = 0; k < K; ++k) b += 12 * slot_off[(int64_t)k * (S + 1) + sb] + 8 * i;
    out[i] = b;
}

// out[c * K + k] = slot_off[k][slot_base[rows[c]]].
__global__ void gather_offsets_kernel(const int64_t *__restrict__ rows, int64_t count,
                                      const int64_t *__restrict__ slot_base,
                                      const int64_t *__restrict__ slot_off, int64_t S, int32_t K,
                                      int64_t *__restrict__ out) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= count) return;
    const int64_t sb = slot_base[rows[c]];
    for (int k = 0; k < K; ++k) out[c * K + k] = slot_off[(int64_t)k * (S + 1) + sb];
}

// ---------------------------------------------------------------------------
// validation
// ---------------------------------------------------------------------------
__global__ void validate_ptr_kernel(const int64_t *__restrict__ ptr, int64_t rows, int64_t nnz,
                                    int *__restrict__ err) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r > rows) return;
    const int64_t x = ptr[r];
    bool bad = x < 0 || x > nnz;
    if (r == 0) bad |= x != 0;
    if (r == rows) bad |= x != nnz;
    if (r < rows) bad |= ptr[r + 1] < x;
    if (bad) atomicOr(err, 2);
}

// One wavefront per row: ids in range and strictly increasing.
__global__ __launch_bounds__(256) void validate_rows_kernel(const int64_t *__restrict__ ptr,
                                                            const int32_t *__restrict__ idx,
                                                            int64_t rows, int64_t limit,
                                                            int *__restrict__ err) {
    const int lane = lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64; r < rows; r += nwaves) {
        const int64_t a = ptr[r], b = ptr[r + 1];
        int bad = 0;
        for (int64_t p = a + lane; p < b; p += 64) {
            const int32_t x = idx[p];
            bad |= (x < 0 || x >= limit);
            if (p > a) bad |= idx[p - 1] >= x;
        }
        if (wave_max(bad) && lane == 0) atomicOr(err, 4);
    }
}

// Every incidence (i, v) of the hyperedge CSR appears in v's list. With equal
// nnz and set-valued rows on both sides, this makes the lists transposes.
__global__ __launch_bounds__(256) void validate_transpose_kernel(
    const int64_t *__restrict__ he_ptr, const int32_t *__restrict__ he_idx, int64_t m,
    const int64_t *__restrict__ v_ptr, const int32_t *__restrict__ v_idx, int64_t n,
    int *__restrict__ err) {
    const int lane = lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64; i < m; i += nwaves) {
        int bad = 0;
        for (int64_t p = he_ptr[i] + lane; p < he_ptr[i + 1]; p += 64) {
            const int v = he_idx[p];
            if (v < 0 || v >= n) {
                bad = 1;
                continue;
            }
            const int lo = (int)v_ptr[v], hi = (int)v_ptr[v + 1];
            const int a = lower_bound_i32(v_idx, lo, hi, (int)i);
            bad |= !(a < hi && v_idx[a] == (int)i);
        }
        if (wave_max(bad) && lane == 0) atomicOr(err, 8);
    }
}

// Disjoint union of a batch of hypergraphs: graph g's hyperedges and
// vertices get ids offset by the sizes of the graphs before it.
__global__ __launch_bounds__(256) void union_kernel(const UnionPart *__restrict__ parts,
                                                    int64_t *__restrict__ he_ptr, int32_t *__restrict__ he_idx,
                                                    int64_t *__restrict__ v_ptr, int32_t *__restrict__ v_idx,
                                                    int32_t *__restrict__ row_s, int32_t *__restrict__ row_base) {
    const UnionPart u = parts[blockIdx.y];
    const int64_t lim = max(max(u.m + 1, u.n + 1), u.nnz);
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < lim; t += (int64_t)gridDim.x * blockDim.x) {
        if (t <= u.m) he_ptr[u.m_off + t] = as_global(u.he_ptr)[t] + u.nnz_off;  // the shared end entry agrees
        if (t < u.m) {
            row_s[u.m_off + t] = u.s;
            row_base[u.m_off + t] = (int32_t)u.m_off;
        }
        if (t <= u.n) v_ptr[u.n_off + t] = as_global(u.v_ptr)[t] + u.nnz_off;
        if (t < u.nnz) {
            he_idx[u.nnz_off + t] = as_global(u.he_idx)[t] + (int32_t)u.n_off;
            v_idx[u.nnz_off + t] = as_global(u.v_idx)[t] + (int32_t)u.m_off;
        }
    }
}

__global__ void gather_i64_kernel(const int64_t *__restrict__ src, const int64_t *__restrict__ idx,
                                  int64_t count, int64_t *__restrict__ out) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < count) out[c] = src[idx[c]];
}

// ---------------------------------------------------------------------------
// s-connected components (Section II-B: maximal sets of E_s joined by
// s-walks) and ID squeezing, on the emitted edge list
// ---------------------------------------------------------------------------
// label[] doubles as the union-find parent array: label[x] <= x for kept x,
// and a root is its own label. Loads and stores go to the device-coherent
// level so that concurrent hooks see each other; values only decrease, so a
// stale read still names an ancestor.
__device__ __forceinline__ int cc_load(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void cc_store(int32_t *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x's tree, halving the path on the way (each step strictly
// decreases, so the walk ends within x steps).
__device__ __forceinline__ int cc_root(int32_t *label, int x) {
    int cur = cc_load(&label[x]);
    if (cur == x) return x;
    int prev = x;
    while (true) {
        const int next = cc_load(&label[cur]);
        if (next >= cur) return cur;  // a root (next == cur)
        cc_store(&label[prev], next);
        prev = cur;
        cur = next;
    }
}

__global__ void cc_init_kernel(const int64_t *__restrict__ he_ptr, int64_t m, int32_t s, int32_t *__restrict__ label) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) label[i] = (he_ptr[i + 1] - he_ptr[i] >= s) ? (int32_t)i : -1;
}

constexpr int kHookTries = 1 << 20;  // far above any real retry count

// Joins the trees of u and v (both kept).
__device__ __forceinline__ void cc_join(int32_t *label, int u, int v, int *err) {
    int ru = cc_root(label, u), rv = cc_root(label, v);
    int tries = 0;
    while (ru != rv) {
        const int lo = min(ru, rv), hi = max(ru, rv);
        const int old = atomicCAS(&label[hi], hi, lo);  // hang the larger root under the smaller
        if (old == hi) break;
        // hi stopped being a root meanwhile: start again from the current roots
        ru = cc_root(label, lo);
        rv = cc_root(label, old);
        if (++tries >= kHookTries) {
            atomicOr(err, 1);
            break;
        }
    }
}

// A sample of an edge list: runs of kSampleRun consecutive edges out of every
// kSampleRun * every (whole cache lines: single edges spread over the list
// cost a line each, 0.3 ms instead of 0.05 for one edge in 64 of 4.1e8).
constexpr int kSampleRun = 32;
__device__ __forceinline__ int64_t sampled(int64_t t, int64_t every) {
    return t / kSampleRun * (kSampleRun * every) + t % kSampleRun;
}
__device__ __forceinline__ int64_t sample_count(int64_t n, int64_t every) {
    const int64_t run = kSampleRun * every, rest = n % run;
    return n / run * kSampleRun + (rest < kSampleRun ? rest : kSampleRun);
}

// Joins the ends of every edge. Labels are read with plain loads
// (L1 and L2); ends with the same label are in one tree already, whatever
// the age of the values (a stale label is an ancestor), and only the other
// edges walk to their roots at the device-coherent level, which misses the
// near caches. Ends at -1 never change.
constexpr int kEdgeUnroll = 4;  // edges in flight per lane

__global__ __launch_bounds__(256) void cc_hook_kernel(const int32_t *__restrict__ row, const int32_t *__restrict__ col,
                                                      int64_t num_edges, int64_t m, int32_t *label,
                                                      int *err) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x * kEdgeUnroll;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x * kEdgeUnroll + threadIdx.x; e0 < num_edges; e0 += step) {
        int u[kEdgeUnroll], v[kEdgeUnroll], lu[kEdgeUnroll], lv[kEdgeUnroll];
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) {
            const int64_t e = e0 + (int64_t)r * blockDim.x;
            u[r] = e < num_edges ? row[e] : -1;
            v[r] = e < num_edges ? col[e] : -1;
        }
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) {
            const bool in = u[r] >= 0 && u[r] < m && v[r] >= 0 && v[r] < m;
            if (!in && e0 + (int64_t)r * blockDim.x < num_edges) atomicOr(err, 4);  // not a hyperedge id
            if (!in) u[r] = -1;
            lu[r] = in ? label[u[r]] : 0;
            lv[r] = in ? label[v[r]] : 0;
        }
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) {
            if (u[r] < 0) continue;
            if (lu[r] < 0 || lv[r] < 0)  // an end outside E_s: not an edge of L_s
                atomicOr(err, 2);
            else if (lu[r] != lv[r])
                cc_join(label, u[r], v[r], err);
        }
    }
}

// Every label becomes its tree's root (no joins run meanwhile: roots keep
// their own label, so concurrent walks only see ancestors).
__global__ __launch_bounds__(256) void cc_flatten_kernel(int64_t m, int32_t *label) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    int cur = cc_load(&label[i]);
    if (cur < 0 || cur == (int)i) return;
    int next;
    while ((next = cc_load(&label[cur])) < cur) cur = next;
    cc_store(&label[i], cur);
}

// One round of hooking over a sample of the edges: of the two trees of an
// edge (labels are roots: own ids at first, flattened before every later
// round) the larger root hangs under the smallest root it meets. Links point
// down and join ends of an edge, so they form trees; a link that loses to a
// smaller root is found again by the pass over every edge. One
// fire-and-forget minimum per edge: with joins instead, all lanes chase and
// retry the same few roots (3.9 ms for the first round over 6.5e6 sampled
// edges, against 0.07 ms).
__global__ __launch_bounds__(256) void cc_min_kernel(const int32_t *__restrict__ row, const int32_t *__restrict__ col,
                                                     int64_t num_edges, int64_t every, int64_t m, int32_t *label) {
    const int64_t count = sample_count(num_edges, every);
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = sampled(t, every);
        const int u = row[e], v = col[e];
        if (u < 0 || u >= m || v < 0 || v >= m) continue;  // flagged by the pass over every edge
        const int a = label[u], b = label[v];
        const int lo = min(a, b), hi = max(a, b);
        if (lo >= 0 && lo < hi && label[hi] > lo) atomicMin(&label[hi], lo);
    }
}

// The label that most of kVotes sampled edges' ends hold (or -2).
constexpr int kVotes = 1024;
__global__ __launch_bounds__(kVotes) void cc_giant_kernel(const int32_t *__restrict__ row, int64_t num_edges, int64_t m,
                                                          const int32_t *__restrict__ label,
                                                          int32_t *__restrict__ giant) {
    __shared__ int vote[kVotes];
    __shared__ unsigned long long best;
    const int tid = threadIdx.x;
    const int u = row[num_edges / kVotes * tid];
    const int mine = u >= 0 && u < m ? label[u] : -2;
    vote[tid] = mine;
    if (tid == 0) best = 0;
    __syncthreads();
    int n = 0;
    for (int t = 0; t < kVotes; ++t) n += vote[t] == mine ? 1 : 0;
    if (mine >= 0) atomicMax(&best, ((unsigned long long)n << 32) | (unsigned)mine);
    __syncthreads();
    if (tid == 0) *giant = best ? (int32_t)(unsigned)best : -2;
}

// bits[i / 32] bit i % 32: label[i] is the giant component's.
__global__ __launch_bounds__(256) void cc_bits_kernel(int64_t m, const int32_t *__restrict__ label,
                                                      const int32_t *__restrict__ giant,
                                                      uint32_t *__restrict__ bits) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const unsigned long long b = __ballot(i < m && label[i] == *giant);
    if ((threadIdx.x & 31) == 0 && i < m) bits[i >> 5] = (uint32_t)(b >> (threadIdx.x & 32));
}

// Passes over every edge with one bit per hyperedge in LDS, so that an edge
// costs its own 8 bytes and two LDS reads: bound by the list's read. The
// gathers from a label (or flag) array in L2 ran at one lane per clock and
// CU (1.6 ms for 4.1e8 edges, 2.1 TB/s). Two sizes: four 512-thread
// workgroups per CU up to 327,680 hyperedges, one of 1,024 up to 1,245,184;
// larger graphs keep the gathers.
constexpr int kBitWords = 10240, kBitWordsLarge = 38912;
constexpr int kBitUnroll = 8;  // edges in flight per lane

__device__ __forceinline__ bool bit_of(const uint32_t *bits, int x) { return (bits[x >> 5] >> (x & 31)) & 1u; }

// Joins every edge but those inside the giant component.
template <int NT, int NW>
__global__ __launch_bounds__(NT) void cc_hook_bits_kernel(const int32_t *__restrict__ row,
                                                          const int32_t *__restrict__ col, int64_t num_edges,
                                                          int64_t m, const uint32_t *__restrict__ giant_bits,
                                                          int32_t *label, int *err) {
    __shared__ uint32_t bits[NW];
    const int words = (int)((m + 31) >> 5);
    for (int x = threadIdx.x; x < words; x += NT) bits[x] = giant_bits[x];
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * NT * kBitUnroll;
    for (int64_t e0 = (int64_t)blockIdx.x * NT * kBitUnroll + threadIdx.x; e0 < num_edges; e0 += step) {
        int u[kBitUnroll], v[kBitUnroll];
#pragma unroll
        for (int r = 0; r < kBitUnroll; ++r) {
            const int64_t e = e0 + (int64_t)r * NT;
            u[r] = e < num_edges ? row[e] : 0;
            v[r] = e < num_edges ? col[e] : 0;
        }
#pragma unroll
        for (int r = 0; r < kBitUnroll; ++r) {
            if (e0 + (int64_t)r * NT >= num_edges) continue;
            if (u[r] < 0 || u[r] >= m || v[r] < 0 || v[r] >= m) {
                atomicOr(err, 4);
                continue;
            }
            if (bit_of(bits, u[r]) && bit_of(bits, v[r])) continue;
            const int lu = label[u[r]], lv = label[v[r]];
            if (lu < 0 || lv < 0)
                atomicOr(err, 2);
            else if (lu != lv)
                cc_join(label, u[r], v[r], err);
        }
    }
}

// Marks the ends of every edge in the workgroup's own bits, then merges
// them: a word is written only where it adds bits.
template <int NT, int NW>
__global__ __launch_bounds__(NT) void mark_bits_kernel(const int32_t *__restrict__ row,
                                                       const int32_t *__restrict__ col, int64_t num_edges, int64_t m,
                                                       uint32_t *all, int *err) {
    __shared__ uint32_t bits[NW];
    const int words = (int)((m + 31) >> 5);
    for (int x = threadIdx.x; x < words; x += NT) bits[x] = 0u;
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * NT * kBitUnroll;
    for (int64_t e0 = (int64_t)blockIdx.x * NT * kBitUnroll + threadIdx.x; e0 < num_edges; e0 += step) {
        int u[kBitUnroll], v[kBitUnroll];
#pragma unroll
        for (int r = 0; r < kBitUnroll; ++r) {
            const int64_t e = e0 + (int64_t)r * NT;
            u[r] = e < num_edges ? row[e] : 0;
            v[r] = e < num_edges ? col[e] : 0;
        }
#pragma unroll
        for (int r = 0; r < kBitUnroll; ++r) {
            if (e0 + (int64_t)r * NT >= num_edges) continue;
            if (u[r] < 0 || u[r] >= m || v[r] < 0 || v[r] >= m) {
                atomicOr(err, 4);
                continue;
            }
            if (!bit_of(bits, u[r])) atomicOr(&bits[u[r] >> 5], 1u << (u[r] & 31));
            if (!bit_of(bits, v[r])) atomicOr(&bits[v[r] >> 5], 1u << (v[r] & 31));
        }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < words; x += NT) {
        const uint32_t b = bits[x];
        if (b & ~all[x]) atomicOr(&all[x], b);
    }
}

__global__ void spread_bits_kernel(int64_t m, const uint32_t *__restrict__ bits, int32_t *__restrict__ flag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) flag[i] = (int32_t)bit_of(bits, (int)i);
}

// Roots into a separate array: the trees are read, never written, here (a
// path-halving walk racing with the final stores could leave a label at an
// ancestor that is not the root).
__global__ __launch_bounds__(256) void cc_finish_kernel(int64_t m, const int32_t *__restrict__ label,
                                                        int32_t *__restrict__ out, unsigned long long *count) {
    __shared__ unsigned long long blk;
    if (threadIdx.x == 0) blk = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int root = 0;
    if (i < m) {
        int cur = label[i];
        if (cur >= 0) {
            int next;
            while ((next = label[cur]) < cur) cur = next;
            root = cur == (int)i;
        }
        out[i] = cur;
    }
    const unsigned long long b = __ballot(root);
    if ((threadIdx.x & 63) == 0 && b) atomicAdd(&blk, (unsigned long long)__popcll(b));
    __syncthreads();
    if (threadIdx.x == 0 && blk) atomicAdd(count, blk);
}

// A flag already set is not written again (most edges of a dense graph name
// ends that others have flagged; the stores to one line would serialise).
__global__ __launch_bounds__(256) void mark_ends_kernel(const int32_t *__restrict__ row,
                                                        const int32_t *__restrict__ col, int64_t num_edges, int64_t m,
                                                        int32_t *flag, int *err) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x * kEdgeUnroll;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x * kEdgeUnroll + threadIdx.x; e0 < num_edges; e0 += step) {
        int u[kEdgeUnroll], v[kEdgeUnroll], fu[kEdgeUnroll], fv[kEdgeUnroll];
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) {
            const int64_t e = e0 + (int64_t)r * blockDim.x;
            u[r] = e < num_edges ? row[e] : -1;
            v[r] = e < num_edges ? col[e] : -1;
        }
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) {
            const bool in = u[r] >= 0 && u[r] < m && v[r] >= 0 && v[r] < m;
            if (!in && e0 + (int64_t)r * blockDim.x < num_edges) atomicOr(err, 4);
            fu[r] = in ? flag[u[r]] : 1;
            fv[r] = in ? flag[v[r]] : 1;
        }
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) {
            if (!fu[r]) flag[u[r]] = 1;
            if (!fv[r]) flag[v[r]] = 1;
        }
    }
}

__global__ void squeeze_ids_kernel(int64_t m, const int32_t *__restrict__ flag, const int64_t *__restrict__ pre,
                                   int32_t *__restrict__ new_id) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) new_id[i] = flag[i] ? (int32_t)pre[i] : -1;
}

__global__ void remap_edges_kernel(int32_t *__restrict__ row, int32_t *__restrict__ col, int64_t num_edges,
                                   const int32_t *__restrict__ new_id) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < num_edges; e += stride) {
        row[e] = new_id[row[e]];
        col[e] = new_id[col[e]];
    }
}

inline unsigned grid_for(int64_t n, int threads) {
    int64_t b = (n + threads - 1) / threads;
    return (unsigned)(b < 1 ? 1 : b);
}

inline unsigned stride_grid(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > 16384) b = 16384;
    return (unsigned)(b < 1 ? 1 : b);
}

inline unsigned wave_grid(int64_t rows, int waves_per_block, int64_t cap) {
    int64_t b = (rows + waves_per_block - 1) / waves_per_block;
    if (b > cap) b = cap;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int64_t scan_partials_size(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

// A large row of S > kSmallRow members has ceil(S / 256) <= (S + 255) / 256
// <= S / 16 pieces (S >= 17): at most nnz / 16 in all when
// the rows do not overlap. The piece list holds, per piece, its entry, its 2-paths (int64)
// and its largest partner (int32): 3 * cap int64 in all.
static_assert(kPlanPiece == 256 && kSmallRow >= 16 && kSmallRow <= 64, "piece bound");
int64_t plan_pieces_cap(int64_t nnz) { return nnz / 16 + 1; }

int heavy_resident(int device) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) cus = 0;
    // the grid is shared by every variant: take the least resident one
    const void *variants[5] = {reinterpret_cast<const void *>(heavy_kernel<false, false, false>),
                               reinterpret_cast<const void *>(heavy_kernel<false, true, false>),
                               reinterpret_cast<const void *>(heavy_kernel<true, false, false>),
                               reinterpret_cast<const void *>(heavy_kernel<true, true, false>),
                               reinterpret_cast<const void *>(heavy_kernel<false, false, true>)};
    for (const void *f : variants) {
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, f, kHeavyThreads, 0) != hipSuccess) v = 0;
        per = (per == 0 || (v > 0 && v < per)) ? v : per;
    }
    if (cus <= 0) cus = 256;
    if (per <= 0) per = 1;
    return cus * per;
}

hipError_t launch_fill_i64(int64_t *p, int64_t n, int64_t value, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    fill_i64_kernel<<<grid_for(n, 256), 256, 0, st>>>(p, n, value);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t value, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    fill_i32_kernel<<<grid_for(n, 256), 256, 0, st>>>(p, n, value);
    return hipGetLastError();
}

hipError_t launch_scans(const ScanJobs &jobs, int64_t *partials, hipStream_t st) {
    if (jobs.count <= 0) return hipSuccess;
    int64_t n = 0;
    for (int t = 0; t < jobs.count; ++t) n = jobs.j[t].n > n ? jobs.j[t].n : n;
    const unsigned count = (unsigned)jobs.count;
    if (n <= kScanSmall) {
        scan_small_kernel<<<count, kScanSmallThreads, 0, st>>>(jobs);
        return hipGetLastError();
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile, stride = scan_partials_size(n);
    scan_reduce_kernel<<<dim3((unsigned)nb, count), kScanThreads, 0, st>>>(jobs, partials, stride);
    scan_top_kernel<<<count, 1024, 0, st>>>(jobs, partials, stride);
    scan_down_kernel<<<dim3((unsigned)nb, count), kScanThreads, 0, st>>>(jobs, partials, stride);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan_i64(const int64_t *in, int64_t n, int64_t *out, int64_t *partials,
                                     hipStream_t st) {
    return launch_scans(ScanJobs().add(in, n, out), partials, st);
}
hipError_t launch_exclusive_scan_i32(const int32_t *in, int64_t n, int64_t *out, int64_t *partials,
                                     hipStream_t st) {
    return launch_scans(ScanJobs().add(in, n, out), partials, st);
}
hipError_t launch_exclusive_scan_u8(const uint8_t *in, int64_t n, int64_t *out, int64_t *partials,
                                    hipStream_t st) {
    return launch_scans(ScanJobs().add(in, n, out), partials, st);
}

hipError_t launch_read_back(const ReadBack &rb, int64_t *host, hipStream_t st) {
    if (rb.count <= 0) return hipSuccess;
    read_back_kernel<<<(unsigned)rb.count, 64, 0, st>>>(rb, host);
    return hipGetLastError();
}

hipError_t launch_row_bits(int64_t m, const int64_t *he_ptr, int32_t s_min, const int32_t *row_s, const KeepBits &rows,
                           hipStream_t st) {
    row_bits_kernel<<<grid_for(keep_words(m) * 64, 256), 256, 0, st>>>(m, he_ptr, s_min, row_s, rows);
    return hipGetLastError();
}

hipError_t launch_keep_incidence(int64_t nnz, const int32_t *v_idx, int64_t m, const KeepBits &rows,
                                 const KeepBits &inc, hipStream_t st) {
    keep_incidence_kernel<<<grid_for(keep_words(nnz), 4 * kKeepWords), 256, 0, st>>>(nnz, v_idx, m, rows.bits, inc);
    return hipGetLastError();
}

hipError_t launch_compact_vertex_lists(int64_t n, int64_t nnz, const int64_t *v_ptr, const int32_t *v_idx,
                                       const KeepBits &inc, int64_t *vs_ptr, int32_t *vs_idx, hipStream_t st) {
    compact_idx_kernel<<<grid_for(keep_words(nnz), 4 * kKeepWords), 256, 0, st>>>(nnz, v_idx, inc, vs_idx);
    compact_ptr_kernel<<<grid_for(n + 1, 256), 256, 0, st>>>(n, nnz, v_ptr, inc, vs_ptr);
    return hipGetLastError();
}

hipError_t launch_cid(int64_t m, const KeepBits &rows, int32_t *cid, int32_t *cid_row, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    cid_kernel<<<grid_for(m, 256), 256, 0, st>>>(m, rows, cid, cid_row);
    return hipGetLastError();
}

hipError_t launch_vs_cid(int64_t n, int64_t m, int64_t nnz, const int64_t *vs_ptr, const int32_t *vs_idx,
                         const int32_t *cid, int32_t *vs_cid, uint16_t *vs_win, hipStream_t st) {
    if (nnz <= 0) return hipSuccess;
    vs_cid_kernel<<<stride_grid(nnz), 256, 0, st>>>(n, m, nnz, vs_ptr, vs_idx, cid, vs_cid, vs_win);
    return hipGetLastError();
}

hipError_t launch_row_plan(const Pruned &g, int32_t s_min, int32_t light_max, int64_t slot_work, int64_t row_lo,
                           int64_t row_hi, int32_t dense_ratio, int32_t dense_min, const HubInfo *hub, int32_t *tail_beg,
                           int32_t *tail_end, int64_t *work, int32_t *jmax, int32_t *nslots, uint8_t *rclass, int64_t *bsize,
                           unsigned long long *class_count, int *err, unsigned long long *heavy_work,
                           unsigned long long *dense_work, int64_t *pieces, unsigned long long *num_pieces,
                           hipStream_t st) {
    if (g.m <= 0) return hipSuccess;
    if (light_max <= 0 || light_max > kLightMax) light_max = kLightMax;
    if (slot_work <= 0) slot_work = kSlotWork;
    if (!g.cid) dense_ratio = 0;
    const RowPlanOut o{tail_beg, tail_end, work, jmax, nslots, rclass, bsize, dense_ratio, dense_min, hub, dense_work};
    auto plan = [&](auto kernel, int rows) {
        kernel<<<wave_grid((g.m + rows - 1) / rows, 4, 8192), 256, 0, st>>>(
            g, s_min, light_max, slot_work, row_lo, row_hi, o, class_count, err, heavy_work, pieces,
            plan_pieces_cap(g.nnz), num_pieces);
    };
    // 64 rows per wavefront fill the chip from about 2^17 rows on
    if (g.m >= (1 << 17))
        plan(row_plan_kernel<64>, 64);
    else
        plan(row_plan_kernel<16>, 16);
    // the piece count is known on the device only: grids for the bound
    const int64_t cap = plan_pieces_cap(g.nnz);
    int64_t *piece_w = pieces + cap;
    int32_t *piece_jm = reinterpret_cast<int32_t *>(pieces + 2 * cap);
    row_piece_kernel<<<wave_grid(cap, 4, 4096), 256, 0, st>>>(g, tail_beg, tail_end, pieces, cap, num_pieces, piece_w,
                                                              piece_jm, err);
    row_piece_finish_kernel<<<grid_for(cap, 256), 256, 0, st>>>(g, light_max, slot_work, o, class_count, err,
                                                                heavy_work, pieces, cap, num_pieces, piece_w,
                                                                piece_jm);
    return hipGetLastError();
}

hipError_t launch_fill_slots(int64_t m, const int64_t *he_ptr, const int64_t *slot_base,
                             const int32_t *nslots, const int32_t *jmax, const uint8_t *rclass,
                             const int64_t *bbase, const int32_t *cid, int64_t *hat, int32_t *hcnt,
                             int64_t *partials, int32_t *slot_row, int32_t *const *lists, HeavyDesc *const *heavy,
                             const int64_t *caps, const int64_t *planned, unsigned long long *list_fill, int *err,
                             hipStream_t st) {
    if (m <= 0) return hipSuccess;
    LightLists ll;
    for (int c = 0; c < kLightClasses; ++c) ll.l[c] = lists[c];
    for (int c = 0; c < kNumLists; ++c) ll.cap[c] = caps[c];
    ll.err = err;
    fill_slots_kernel<<<grid_for(m, 256 * kFillRows), 256, 0, st>>>(m, he_ptr, slot_base, nslots, jmax, rclass,
                                                                     bbase, slot_row, ll, hat, list_fill);
    int used = 0;
    for (int h = 0; h < kNumHeavyLists; ++h) used |= planned[kLightClasses + h] > 0 ? 1 << h : 0;
    if (!used) return hipGetLastError();
    heavy_counts_kernel<<<grid_for(m, 256) < 8192 ? grid_for(m, 256) : 8192, 256, 0, st>>>(m, rclass, nslots, used,
                                                                                          hcnt);
    ScanJobs jobs;
    for (int h = 0; h < kNumHeavyLists; ++h)
        if (used >> h & 1) jobs.add(hcnt + (int64_t)h * m, m, hat + (int64_t)h * (m + 1));
    const hipError_t e = launch_scans(jobs, partials, st);
    if (e != hipSuccess) return e;
    HeavyLists hl;
    for (int h = 0; h < kNumHeavyLists; ++h) {
        hl.l[h] = heavy[h];
        hl.cap[h] = caps[kLightClasses + h];
    }
    // fewer rows per wavefront where 64 would leave most of the chip idle
    // (37 us on 5000 rows, most of them heavy; 8 us with 8)
    const int rows = m < (1 << 17) ? 8 : 64;
    heavy_desc_kernel<<<wave_grid((m + rows - 1) / rows, 4, 8192), 256, 0, st>>>(
        m, he_ptr, slot_base, nslots, jmax, rclass, bbase, hat, slot_row, hl, cid, rows, err);
    return hipGetLastError();
}

hipError_t launch_block_mask(int64_t m, int64_t r0, int64_t r1, const int32_t *nslots_all, const uint8_t *rclass_all,
                             const int64_t *bsize_all, const int64_t *work, int32_t *nslots, uint8_t *rclass,
                             int64_t *bsize, unsigned long long *class_count, unsigned long long *heavy_work,
                             unsigned long long *dense_work, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    const unsigned grid = grid_for(m, 256) < 4096 ? grid_for(m, 256) : 4096;
    block_mask_kernel<<<grid, 256, 0, st>>>(m, r0, r1, nslots_all, rclass_all, bsize_all, work, nslots, rclass, bsize,
                                            class_count, heavy_work, dense_work);
    return hipGetLastError();
}

hipError_t launch_list_cuts(const HeavyDesc *desc, int64_t count, const int64_t *slots, int64_t n, int64_t *out,
                            hipStream_t st) {
    if (n <= 0) return hipSuccess;
    list_cuts_kernel<<<grid_for(n, 256), 256, 0, st>>>(desc, count, slots, n, out);
    return hipGetLastError();
}

hipError_t launch_heavy_range(const HeavyDesc *desc, int64_t count, int64_t s0, int64_t s1, int64_t *out,
                              hipStream_t st) {
    heavy_range_kernel<<<1, 64, 0, st>>>(desc, count, s0, s1, out);
    return hipGetLastError();
}

namespace {
// launch(runs, workgroups) for all light classes together, in as many
// launches as it takes (limit > 0: of at most that many workgroups).
template <typename F>
hipError_t light_launches(const int32_t *const *lists, const int64_t *counts, int64_t limit, F launch) {
    ClassRuns<kLightClasses> part;
    while (const unsigned grid = part.next(counts, 256, 4, max_workgroups(256, limit))) {
        LightRuns runs;
        for (int c = 0; c < kLightClasses; ++c) {
            runs.list[c] = lists[c] + part.begin[c];
            runs.count[c] = part.count[c];
            runs.first[c] = part.first[c];
        }
        launch(runs, grid);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Rows of the sorting classes up to which they are counted in one launch. It
// has the registers and LDS of its largest class, four wavefronts a SIMD:
// beyond four rows for each the classes' own launches are as fast.
constexpr int64_t kLightTogether = 16384;
// Tiny rows up to which they are counted with them. The common launch's
// registers and LDS cost a tiny row 12 ps more than a launch of its own (38
// against 27), and save at most the longest sorting row (11 us with 16 of
// them, 50 with 1000): 4.0e6 tiny rows beside 16, 1000 and 16 000 took 146,
// 151 and 305 us together, now 113, 156 and 264; 2.0e6 beside 1000 take 71
// together, 107 apart.
constexpr int64_t kTinyTogether = int64_t(3) << 20;
}  // namespace

hipError_t launch_light_count(const int32_t *const *lists, const int64_t *counts, const Slots &sl, const Pruned &g,
                              const EmitParams &ep, int64_t *slot_cnt, const LightStore *store, int64_t limit,
                              hipStream_t st) {
    int64_t rows = 0;
    for (int c = 1; c < kLightClasses; ++c) rows += counts[c];
    if (rows > kLightTogether || rows == 0) {
        for (int c = 0; c < kLightClasses; ++c) {
            const hipError_t e = launch_light(c, false, lists[c], counts[c], sl, g, ep, slot_cnt, nullptr, store, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    int64_t together[kLightClasses];
    for (int c = 0; c < kLightClasses; ++c) together[c] = counts[c];
    if (counts[0] > kTinyTogether) {
        const hipError_t e = launch_light(0, false, lists[0], counts[0], sl, g, ep, slot_cnt, nullptr, store, st);
        if (e != hipSuccess) return e;
        together[0] = 0;
    }
    return light_launches(lists, together, limit, [&](const LightRuns &runs, unsigned grid) {
        if (store)
            light_count_kernel<true><<<grid, 256, 0, st>>>(runs, sl, g, ep, slot_cnt, *store);
        else
            light_count_kernel<false><<<grid, 256, 0, st>>>(runs, sl, g, ep, slot_cnt, LightStore{});
    });
}

hipError_t launch_light(int cls, bool emit, const int32_t *list, int64_t count, const Slots &sl,
                        const Pruned &g, const EmitParams &ep, int64_t *slot_cnt,
                        const int64_t *slot_off, const LightStore *store, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    if (store && emit) return hipErrorInvalidValue;
    if (cls == 0) {  // one lane per row
        if (emit)
            tiny_kernel<true, false><<<grid_for(count, 256), 256, 0, st>>>(list, count, sl, g, ep, slot_cnt, slot_off,
                                                                           LightStore{});
        else if (store)
            tiny_kernel<false, true><<<grid_for(count, 256), 256, 0, st>>>(list, count, sl, g, ep, slot_cnt, slot_off,
                                                                           *store);
        else
            tiny_kernel<false, false><<<grid_for(count, 256), 256, 0, st>>>(list, count, sl, g, ep, slot_cnt, slot_off,
                                                                            LightStore{});
        return hipGetLastError();
    }
    const unsigned grid = grid_for(count, 4);
    const LightStore ls = store ? *store : LightStore{};
#define SLG_LIGHT(KPL)                                                                              \
    do {                                                                                           \
        if (emit)                                                                                  \
            light_kernel<KPL, true, false><<<grid, 256, 0, st>>>(list, count, sl, g, ep, slot_cnt,  \
                                                                 slot_off, ls);                    \
        else if (store)                                                                            \
            light_kernel<KPL, false, true><<<grid, 256, 0, st>>>(list, count, sl, g, ep, slot_cnt,  \
                                                                 slot_off, ls);                    \
        else                                                                                       \
            light_kernel<KPL, false, false><<<grid, 256, 0, st>>>(list, count, sl, g, ep, slot_cnt, \
                                                                  slot_off, ls);                   \
    } while (0)
    switch (cls) {
        case 1: SLG_LIGHT(1); break;
        case 2: SLG_LIGHT(2); break;
        case 3: SLG_LIGHT(4); break;
        case 4: SLG_LIGHT(8); break;
        case 5: SLG_LIGHT(16); break;
        case 6: SLG_LIGHT(32); break;
        default: return hipErrorInvalidValue;
    }
#undef SLG_LIGHT
    return hipGetLastError();
}

hipError_t launch_light_store_emit(const int32_t *const *lists, const int64_t *counts, const Slots &sl,
                                   const LightStore &store, const EmitParams &ep, const int64_t *slot_off,
                                   int64_t limit, hipStream_t st) {
    return light_launches(lists, counts, limit, [&](const LightRuns &runs, unsigned grid) {
        light_store_emit_kernel<<<grid, 256, 0, st>>>(runs, sl, store, ep, slot_off);
    });
}

hipError_t launch_light_work(int64_t m, const uint8_t *rclass, const int64_t *work, int32_t *lw, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    light_work_kernel<<<grid_for(m, 256) < 8192 ? grid_for(m, 256) : 8192, 256, 0, st>>>(m, rclass, work, lw);
    return hipGetLastError();
}

hipError_t launch_heavy(bool emit, bool wide, const HeavyDesc *desc, int64_t count, int64_t slots,
                        const int32_t *bounds, const Pruned &g, const EmitParams &ep, int64_t *slot_cnt,
                        const int64_t *slot_off, int64_t *ticket, int resident, const CountStore *store,
                        hipStream_t st) {
    if (count <= 0) return hipSuccess;
    if (store && (emit || wide)) return hipErrorInvalidValue;
    const int64_t want = resident > 0 ? resident : 512;
    const unsigned grid = (unsigned)(count < want ? count : want);
    unsigned long long *tk = reinterpret_cast<unsigned long long *>(ticket);
    const CountStore cs = store ? *store : CountStore{};
#define SLG_HEAVY(E, W, ST)                                                                          \
    heavy_kernel<E, W, ST><<<grid, kHeavyThreads, 0, st>>>(desc, count, slots, bounds, g.vs_idx, ep, slot_cnt, \
                                                           slot_off, tk, cs)
    if (emit && wide) SLG_HEAVY(true, true, false);
    else if (emit) SLG_HEAVY(true, false, false);
    else if (wide) SLG_HEAVY(false, true, false);
    else if (store) SLG_HEAVY(false, false, true);
    else SLG_HEAVY(false, false, false);
#undef SLG_HEAVY
    return hipGetLastError();
}

hipError_t launch_slot_work(const HeavyDesc *desc, int64_t count, const int32_t *bounds, int64_t *work,
                            hipStream_t st) {
    if (count <= 0) return hipSuccess;
    slot_work_kernel<<<wave_grid(count, 4, 8192), 256, 0, st>>>(desc, count, bounds, work);
    return hipGetLastError();
}

hipError_t launch_heavy_store_emit(const HeavyDesc *desc, int64_t count, int64_t slots, const CountStore &store,
                                   const EmitParams &ep, const int64_t *slot_off, const int32_t *cid_row,
                                   hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const unsigned grid = wave_grid(count, 4, 16384);
    if (cid_row) {
        if (ep.k <= 4)
            heavy_store_emit_kernel<4, true><<<grid, 256, 0, st>>>(desc, count, slots, store, ep, slot_off, cid_row);
        else
            heavy_store_emit_kernel<SLG_MAX_S, true><<<grid, 256, 0, st>>>(desc, count, slots, store, ep, slot_off,
                                                                           cid_row);
    } else if (ep.k <= 4) {
        heavy_store_emit_kernel<4, false><<<grid, 256, 0, st>>>(desc, count, slots, store, ep, slot_off, nullptr);
    } else {
        heavy_store_emit_kernel<SLG_MAX_S, false><<<grid, 256, 0, st>>>(desc, count, slots, store, ep, slot_off,
                                                                        nullptr);
    }
    return hipGetLastError();
}

hipError_t launch_dense_keys(const HeavyDesc *desc, int64_t count, int32_t *key, int32_t *id, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    dense_keys_kernel<<<grid_for(count, 256), 256, 0, st>>>(desc, count, key, id);
    return hipGetLastError();
}

hipError_t launch_dense(bool emit, const HeavyDesc *desc, int64_t count, const int32_t *order, int64_t slots,
                        const int32_t *bounds, const Pruned &g, const EmitParams &ep, int64_t *slot_cnt,
                        const int64_t *slot_off, int64_t *ticket, int resident, const CountStore *store,
                        int64_t *store_cursor, int64_t store_cap, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    if (!g.vs_win || !g.cid_row || (store && !emit && !store_cursor)) return hipErrorInvalidValue;
    const int64_t want = resident > 0 ? resident : 512;
    const unsigned grid = (unsigned)(count < want ? count : want);
    unsigned long long *tk = reinterpret_cast<unsigned long long *>(ticket);
    unsigned long long *cur = reinterpret_cast<unsigned long long *>(store_cursor);
    const CountStore cs = store ? *store : CountStore{};
    if (emit)
        dense_kernel<true><<<grid, kDenseThreads, 0, st>>>(desc, count, order, slots, bounds, g.vs_win, g.cid_row, ep,
                                                            slot_cnt, slot_off, tk, cs, cur, store_cap);
    else
        dense_kernel<false><<<grid, kDenseThreads, 0, st>>>(desc, count, order, slots, bounds, g.vs_win, g.cid_row, ep,
                                                             slot_cnt, slot_off, tk, cs, cur, store_cap);
    return hipGetLastError();
}

int dense_resident(int device) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) cus = 0;
    const void *variants[2] = {reinterpret_cast<const void *>(dense_kernel<false>),
                               reinterpret_cast<const void *>(dense_kernel<true>)};
    for (const void *f : variants) {
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, f, kDenseThreads, 0) != hipSuccess) v = 0;
        per = (per == 0 || (v > 0 && v < per)) ? v : per;
    }
    if (cus <= 0) cus = 256;
    if (per <= 0) per = 1;
    return cus * per;
}

hipError_t launch_sum_i32(const int32_t *n, int64_t count, int64_t *out, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    sum_i32_kernel<<<grid_for(count, 256) < 4096 ? grid_for(count, 256) : 4096, 256, 0, st>>>(
        n, count, reinterpret_cast<unsigned long long *>(out));
    return hipGetLastError();
}

hipError_t launch_heavy_edges(const HeavyDesc *desc, int64_t count, const int64_t *slot_cnt, int64_t S,
                              int32_t K, int64_t *out, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    heavy_edges_kernel<<<grid_for(count, 256), 256, 0, st>>>(desc, count, slot_cnt, S, K,
                                                              reinterpret_cast<unsigned long long *>(out));
    return hipGetLastError();
}

hipError_t launch_bounds(const Pruned &g, const HeavyDesc *desc, int64_t count, int32_t *bounds,
                         hipStream_t st) {
    if (count <= 0) return hipSuccess;
    bounds_kernel<<<grid_for(count, 4), 256, 0, st>>>(desc, count, g.he_ptr, g.vs_idx, g.tail_beg, g.tail_end,
                                                       bounds);
    return hipGetLastError();
}

hipError_t launch_row_ptr(int64_t row_lo, int64_t row_hi, const int64_t *slot_base,
                          const int64_t *slot_off, int64_t slots, const EmitParams &ep, hipStream_t st) {
    const int64_t n = row_hi - row_lo + 1;
    if (n <= 0) return hipSuccess;
    row_ptr_kernel<<<grid_for(n, 256), 256, 0, st>>>(row_lo, row_hi, slot_base, slot_off, slots, ep);
    return hipGetLastError();
}

hipError_t launch_row_bytes(int64_t m, const int64_t *slot_base, const int64_t *slot_off, int64_t slots,
                            int32_t K, int64_t *out, hipStream_t st) {
    row_bytes_kernel<<<grid_for(m + 1, 256), 256, 0, st>>>(m, slot_base, slot_off, slots, K, out);
    return hipGetLastError();
}

hipError_t launch_gather_offsets(const int64_t *rows, int64_t count, const int64_t *slot_base,
                                 const int64_t *slot_off, int64_t slots, int32_t K, int64_t *out,
                                 hipStream_t st) {
    if (count <= 0) return hipSuccess;
    gather_offsets_kernel<<<grid_for(count, 256), 256, 0, st>>>(rows, count, slot_base, slot_off, slots, K,
                                                                 out);
    return hipGetLastError();
}

hipError_t launch_union(const UnionPart *parts, int32_t count, int64_t max_elems, int64_t *he_ptr,
                        int32_t *he_idx, int64_t *v_ptr, int32_t *v_idx, int32_t *row_s, int32_t *row_base,
                        hipStream_t st) {
    if (count <= 0) return hipSuccess;
    int64_t bx = (max_elems + 255) / 256;
    if (bx > 256) bx = 256;
    if (bx < 1) bx = 1;
    union_kernel<<<dim3((unsigned)bx, (unsigned)count), 256, 0, st>>>(parts, he_ptr, he_idx, v_ptr, v_idx, row_s,
                                                                       row_base);
    return hipGetLastError();
}


hipError_t launch_cc_init(const int64_t *he_ptr, int64_t m, int32_t s, int32_t *label, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    cc_init_kernel<<<grid_for(m, 256), 256, 0, st>>>(he_ptr, m, s, label);
    return hipGetLastError();
}

// Lists of at least kSampleEdges edges start from a sampled forest, joined
// and flattened over growing samples, so that the pass over every edge finds
// most ends in one tree already; shorter lists take less time than the extra
// launches. 4.1e8 edges of a power-law L_1 over 2e5 hyperedges: 6.4 ms with
// every edge walking to its roots; now 1.2 ms (rounds 0.37, every edge 0.80,
// of which the list's 3.3 GB alone take 0.55).
constexpr int64_t kSampleEdges = int64_t(1) << 20;
constexpr int64_t kSampleEvery[] = {64, 32, 16};  // one edge in so many, per round

int64_t edge_bits_words(int64_t m, int64_t num_edges) {
    return num_edges >= kSampleEdges && m <= 32ll * kBitWordsLarge ? (m + 31) / 32 + 1 : 0;
}

hipError_t launch_cc_hook(const int32_t *row, const int32_t *col, int64_t num_edges, int64_t m, int32_t *label,
                          uint32_t *bits, int *err, hipStream_t st) {
    if (num_edges <= 0) return hipSuccess;
    auto grid = [](int64_t n) { return stride_grid((n + kEdgeUnroll - 1) / kEdgeUnroll); };
    if (num_edges < kSampleEdges) {
        cc_hook_kernel<<<grid(num_edges), 256, 0, st>>>(row, col, num_edges, m, label, err);
        return hipGetLastError();
    }
    const unsigned rows = grid_for(m, 256);
    for (const int64_t every : kSampleEvery) {
        cc_min_kernel<<<stride_grid(num_edges / every), 256, 0, st>>>(row, col, num_edges, every, m, label);
        cc_flatten_kernel<<<rows, 256, 0, st>>>(m, label);
    }
    if (edge_bits_words(m, num_edges) == 0) {
        cc_hook_kernel<<<grid(num_edges), 256, 0, st>>>(row, col, num_edges, m, label, err);
        return hipGetLastError();
    }
    int32_t *giant = reinterpret_cast<int32_t *>(bits + (m + 31) / 32);
    cc_giant_kernel<<<1, kVotes, 0, st>>>(row, num_edges, m, label, giant);
    cc_bits_kernel<<<rows, 256, 0, st>>>(m, label, giant, bits);
    if (m <= 32ll * kBitWords)
        cc_hook_bits_kernel<512, kBitWords><<<1024, 512, 0, st>>>(row, col, num_edges, m, bits, label, err);
    else
        cc_hook_bits_kernel<1024, kBitWordsLarge><<<256, 1024, 0, st>>>(row, col, num_edges, m, bits, label, err);
    return hipGetLastError();
}

hipError_t launch_cc_finish(int64_t m, const int32_t *label, int32_t *out, unsigned long long *count,
                            hipStream_t st) {
    if (m <= 0) return hipSuccess;
    cc_finish_kernel<<<grid_for(m, 256), 256, 0, st>>>(m, label, out, count);
    return hipGetLastError();
}

hipError_t launch_mark_ends(const int32_t *row, const int32_t *col, int64_t num_edges, int64_t m, int32_t *flag,
                            uint32_t *bits, int *err, hipStream_t st) {
    const int64_t words = edge_bits_words(m, num_edges);
    if (words == 0) {
        hipError_t e = launch_fill_i32(flag, m, 0, st);
        if (e != hipSuccess || num_edges <= 0) return e;
        mark_ends_kernel<<<stride_grid((num_edges + kEdgeUnroll - 1) / kEdgeUnroll), 256, 0, st>>>(row, col, num_edges,
                                                                                                    m, flag, err);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_i32(reinterpret_cast<int32_t *>(bits), words, 0, st);
    if (e != hipSuccess) return e;
    if (m <= 32ll * kBitWords)
        mark_bits_kernel<512, kBitWords><<<1024, 512, 0, st>>>(row, col, num_edges, m, bits, err);
    else
        mark_bits_kernel<1024, kBitWordsLarge><<<256, 1024, 0, st>>>(row, col, num_edges, m, bits, err);
    spread_bits_kernel<<<grid_for(m, 256), 256, 0, st>>>(m, bits, flag);
    return hipGetLastError();
}

hipError_t launch_squeeze_ids(int64_t m, const int32_t *flag, const int64_t *pre, int32_t *new_id, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    squeeze_ids_kernel<<<grid_for(m, 256), 256, 0, st>>>(m, flag, pre, new_id);
    return hipGetLastError();
}

hipError_t launch_remap_edges(int32_t *row, int32_t *col, int64_t num_edges, const int32_t *new_id,
                              hipStream_t st) {
    if (num_edges <= 0) return hipSuccess;
    remap_edges_kernel<<<stride_grid(num_edges), 256, 0, st>>>(row, col, num_edges, new_id);
    return hipGetLastError();
}

hipError_t launch_gather_i64(const int64_t *src, const int64_t *idx, int64_t count, int64_t *out,
                             hipStream_t st) {
    if (count <= 0) return hipSuccess;
    gather_i64_kernel<<<grid_for(count, 256), 256, 0, st>>>(src, idx, count, out);
    return hipGetLastError();
}

hipError_t launch_validate_ptr(const int64_t *ptr, int64_t rows, int64_t nnz, int *err,
                               hipStream_t st) {
    validate_ptr_kernel<<<grid_for(rows + 1, 256), 256, 0, st>>>(ptr, rows, nnz, err);
    return hipGetLastError();
}

hipError_t launch_validate_rows(const int64_t *ptr, const int32_t *idx, int64_t rows,
                                int64_t limit, int *err, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    validate_rows_kernel<<<wave_grid(rows, 4, 8192), 256, 0, st>>>(ptr, idx, rows, limit, err);
    return hipGetLastError();
}

hipError_t launch_validate_transpose(const int64_t *he_ptr, const int32_t *he_idx, int64_t m,
                                     const int64_t *v_ptr, const int32_t *v_idx, int64_t n, int *err,
                                     hipStream_t st) {
    if (m <= 0) return hipSuccess;
    validate_transpose_kernel<<<wave_grid(m, 4, 8192), 256, 0, st>>>(he_ptr, he_idx, m, v_ptr, v_idx,
                                                                      n, err);
    return hipGetLastError();
}

}  // namespace slg
