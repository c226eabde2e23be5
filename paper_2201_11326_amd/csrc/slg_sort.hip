// gfx950 kernels that turn an emitted s-line graph into a consumer-ready
// graph (Stage 4 of the framework, Section IV: the edge list becomes the
// graph's adjacency):
//   - a stable least-significant-digit radix sort of int32 keys carrying up
//     to two int32 payloads (used to transpose an edge list: sorting the
//     upper triangle by column keeps rows ascending inside every column);
//   - the symmetric CSR of L_s from its upper triangle.
// Every step is integer work and deterministic: the sort is stable, so the
// output does not depend on scheduling.
#include "slg_device.h"
#include "slg_internal.h"

namespace slg {
namespace {

constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortRounds = 128;  // rounds of kSortThreads items per chunk
constexpr int64_t kSortChunk = (int64_t)kSortThreads * kSortRounds;
constexpr int kSortBins = 1 << kSortDigitBits;

__device__ __forceinline__ int lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Digit counts of every chunk: hist[d * nchunks + c] = items of chunk c whose
// digit (key >> shift) & (2^bits - 1) is d. Digit-major, so one exclusive
// scan gives every (digit, chunk) its first output position.
__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(const int32_t *__restrict__ key, int64_t n,
                                                                 int shift, int bits, int64_t nchunks,
                                                                 int32_t *__restrict__ hist) {
    __shared__ int h[kSortBins];
    const int nb = 1 << bits;
    const unsigned mask = (unsigned)nb - 1u;
    for (int d = threadIdx.x; d < nb; d += kSortThreads) h[d] = 0;
    __syncthreads();
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const int64_t base = c * kSortChunk, end = min(n, base + kSortChunk);
        for (int64_t q = base + threadIdx.x; q < end; q += kSortThreads)
            atomicAdd(&h[((unsigned)key[q] >> shift) & mask], 1);
        __syncthreads();
        for (int d = threadIdx.x; d < nb; d += kSortThreads) {
            hist[(int64_t)d * nchunks + c] = h[d];
            h[d] = 0;
        }
        __syncthreads();
    }
}

// Stable scatter of every chunk, a tile of kSortTile items at a time. An
// item's rank among the equal digits of its tile counts such items in
// earlier rounds (LDS running counts), in lower wavefronts of its round (LDS
// counts) and in lower lanes of its wavefront (ballots on the digit bits),
// so items keep their order. The tile is then reordered by digit in LDS and
// written out in runs, which keeps the HBM writes of a digit contiguous.
// `run` holds the next output position of every digit.
constexpr int kTileRounds = 16;
constexpr int kSortTile = kSortThreads * kTileRounds;
static_assert(kSortRounds % kTileRounds == 0, "a chunk is whole tiles");

template <int NP>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(
    const int32_t *__restrict__ key_in, const int32_t *__restrict__ a_in, const int32_t *__restrict__ b_in,
    int64_t n, int shift, int bits, int64_t nchunks, const int64_t *__restrict__ off,
    int32_t *__restrict__ key_out, int32_t *__restrict__ a_out, int32_t *__restrict__ b_out) {
    __shared__ int64_t run[kSortBins];
    __shared__ int cnt[kSortBins];          // tile counts so far, then the tile's digit starts
    __shared__ int wcnt[kSortWaves][kSortBins];
    __shared__ int wsum[kSortWaves];
    __shared__ int32_t tk[kSortTile];
    __shared__ int32_t ta[NP > 0 ? kSortTile : 1];
    __shared__ int32_t tb[NP > 1 ? kSortTile : 1];
    const int nb = 1 << bits;
    const unsigned mask = (unsigned)nb - 1u;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int t = threadIdx.x; t < kSortWaves * kSortBins; t += kSortThreads) (&wcnt[0][0])[t] = 0;
    for (int t = threadIdx.x; t < kSortBins; t += kSortThreads) cnt[t] = 0;
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        for (int d = threadIdx.x; d < nb; d += kSortThreads) run[d] = off[(int64_t)d * nchunks + c];
        __syncthreads();
        for (int64_t t0 = c * kSortChunk; t0 < min(n, (c + 1) * kSortChunk); t0 += kSortTile) {
            const int tn = (int)min((int64_t)kSortTile, n - t0);  // items in this tile
            unsigned key[kTileRounds];
            int32_t pa[kTileRounds], pb[kTileRounds];
            int rk[kTileRounds];
#pragma unroll
            for (int r = 0; r < kTileRounds; ++r) {
                const int i = r * kSortThreads + threadIdx.x;
                key[r] = i < tn ? (unsigned)key_in[t0 + i] : 0u;
                if (NP > 0) pa[r] = i < tn ? a_in[t0 + i] : 0;
                if (NP > 1) pb[r] = i < tn ? b_in[t0 + i] : 0;
            }
#pragma unroll
            for (int r = 0; r < kTileRounds; ++r) {
                const bool valid = r * kSortThreads + (int)threadIdx.x < tn;
                const unsigned d = (key[r] >> shift) & mask;
                unsigned long long peers = __ballot(valid);
                for (int i = 0; i < bits; ++i) {
                    const bool bit = (d >> i) & 1u;
                    const unsigned long long bb = __ballot(bit);
                    peers &= bit ? bb : ~bb;
                }
                const int rank = lanes_below(peers);
                if (valid && rank == 0) wcnt[wave][d] = __popcll(peers);
                __syncthreads();
                int pre = 0;
                for (int w = 0; w < wave; ++w) pre += wcnt[w][d];
                rk[r] = cnt[d] + pre + rank;  // rank within the tile's digit d
                __syncthreads();
                for (int dd = threadIdx.x; dd < nb; dd += kSortThreads) {
                    int tot = 0;
#pragma unroll
                    for (int w = 0; w < kSortWaves; ++w) {
                        tot += wcnt[w][dd];
                        wcnt[w][dd] = 0;
                    }
                    cnt[dd] += tot;
                }
                __syncthreads();
            }
            // digit starts within the tile (exclusive scan of cnt)
            {
                int v[kSortBins / kSortThreads > 0 ? kSortBins / kSortThreads : 1];
                int mine = 0;
                constexpr int per = kSortBins / kSortThreads > 0 ? kSortBins / kSortThreads : 1;
#pragma unroll
                for (int j = 0; j < per; ++j) {
                    const int d = threadIdx.x * per + j;
                    v[j] = d < nb ? cnt[d] : 0;
                    mine += v[j];
                }
                int incl = mine;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int y = __shfl_up(incl, o);
                    if (lane >= o) incl += y;
                }
                if (lane == 63) wsum[wave] = incl;
                __syncthreads();
                int base = incl - mine;
                for (int w = 0; w < wave; ++w) base += wsum[w];
#pragma unroll
                for (int j = 0; j < per; ++j) {
                    const int d = threadIdx.x * per + j;
                    if (d < nb) cnt[d] = base;  // start of digit d in the tile
                    base += v[j];
                }
                __syncthreads();
            }
            // reorder by digit in LDS
#pragma unroll
            for (int r = 0; r < kTileRounds; ++r) {
                if (r * kSortThreads + (int)threadIdx.x < tn) {
                    const unsigned d = (key[r] >> shift) & mask;
                    const int q = cnt[d] + rk[r];
                    tk[q] = (int32_t)key[r];
                    if (NP > 0) ta[q] = pa[r];
                    if (NP > 1) tb[q] = pb[r];
                }
            }
            __syncthreads();
            // runs of equal digits to their places
            for (int q = threadIdx.x; q < tn; q += kSortThreads) {
                const int32_t k = tk[q];
                const unsigned d = ((unsigned)k >> shift) & mask;
                const int64_t pos = run[d] + (q - cnt[d]);
                key_out[pos] = k;
                if (NP > 0) a_out[pos] = ta[q];
                if (NP > 1) b_out[pos] = tb[q];
            }
            __syncthreads();
            // next tile: advance the digit positions, clear the counts
            for (int d = threadIdx.x; d < nb; d += kSortThreads) {
                const int end = d + 1 < nb ? cnt[d + 1] : tn;
                run[d] += end - cnt[d];
            }
            __syncthreads();
            for (int d = threadIdx.x; d < kSortBins; d += kSortThreads) cnt[d] = 0;
            __syncthreads();
        }
    }
}

// The flat kernels below give every thread kFlat items per grid step, loaded
// before any is used, so that enough loads are in flight to cover HBM
// latency.
constexpr int kFlat = 4;

// Checks that (row_ptr, row, col) is the upper triangle of a graph on m
// vertices in CSR order: row[e] = r for e in [row_ptr[r], row_ptr[r+1]),
// r < col[e] < m, columns strictly increasing along a row. err |= 1 if not.
__global__ void check_upper_kernel(const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ row,
                                   const int32_t *__restrict__ col, int64_t n, int64_t m, int *__restrict__ err) {
    bool bad = false;
    const int64_t step = (int64_t)gridDim.x * blockDim.x * kFlat;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x * kFlat + threadIdx.x; e0 < n; e0 += step) {
        int32_t r[kFlat], c[kFlat], rp[kFlat], cp[kFlat];
#pragma unroll
        for (int j = 0; j < kFlat; ++j) {
            const int64_t e = e0 + (int64_t)j * blockDim.x;
            const bool in = e < n;
            r[j] = in ? row[e] : 0;
            c[j] = in ? col[e] : 1;
            rp[j] = (in && e > 0) ? row[e - 1] : -1;
            cp[j] = (in && e > 0) ? col[e - 1] : -1;
        }
#pragma unroll
        for (int j = 0; j < kFlat; ++j) {
            const int64_t e = e0 + (int64_t)j * blockDim.x;
            if (e >= n) continue;
            if (r[j] < 0 || r[j] >= m || c[j] <= r[j] || c[j] >= m) {
                bad = true;
                continue;
            }
            if (e < row_ptr[r[j]] || e >= row_ptr[r[j] + 1]) bad = true;
            if (rp[j] == r[j] && cp[j] >= c[j]) bad = true;
        }
    }
    if (bad) atomicOr(err, 1);
}

// row_ptr must start at 0, end at n and never decrease.
__global__ void check_ptr_kernel(const int64_t *__restrict__ row_ptr, int64_t m, int64_t n, int *__restrict__ err) {
    bool bad = false;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x)
        if (row_ptr[r] > row_ptr[r + 1]) bad = true;
    if (blockIdx.x == 0 && threadIdx.x == 0 && (row_ptr[0] != 0 || row_ptr[m] != n)) bad = true;
    if (bad) atomicOr(err, 1);
}

// lower_ptr[c] = number of sorted keys below c, for c in [0, m].
__global__ void key_bounds_kernel(const int32_t *__restrict__ skey, int64_t n, int64_t m,
                                  int64_t *__restrict__ lower_ptr) {
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c <= m; c += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)skey[mid] < c)
                lo = mid + 1;
            else
                hi = mid;
        }
        lower_ptr[c] = lo;
    }
}

// Row r of the symmetric CSR is its partners below r (the transpose, rows
// ascending) followed by those above r (its own row): it starts at
// lower_ptr[r] + row_ptr[r].
__global__ void sym_ptr_kernel(const int64_t *__restrict__ lower_ptr, const int64_t *__restrict__ row_ptr,
                               int64_t m, int64_t *__restrict__ sym_ptr) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= m; r += (int64_t)gridDim.x * blockDim.x)
        sym_ptr[r] = lower_ptr[r] + row_ptr[r];
}

// Sorted entry p (column c, row i) lands at p + row_ptr[c]: the entries of
// columns below c, plus the upper entries of rows below c.
__global__ void sym_lower_kernel(const int32_t *__restrict__ skey, const int32_t *__restrict__ srow,
                                 const int32_t *__restrict__ sw, int64_t n, int64_t m,
                                 const int64_t *__restrict__ row_ptr, int32_t *__restrict__ sym_col,
                                 int32_t *__restrict__ sym_w) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x * kFlat;
    for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x * kFlat + threadIdx.x; p0 < n; p0 += step) {
        int32_t c[kFlat], r[kFlat], w[kFlat];
#pragma unroll
        for (int j = 0; j < kFlat; ++j) {
            const int64_t p = p0 + (int64_t)j * blockDim.x;
            const bool in = p < n;
            c[j] = in ? skey[p] : -1;
            r[j] = in ? srow[p] : 0;
            w[j] = (in && sw) ? sw[p] : 0;
        }
#pragma unroll
        for (int j = 0; j < kFlat; ++j) {
            const int64_t p = p0 + (int64_t)j * blockDim.x;
            if (c[j] < 0 || c[j] >= m) continue;  // past the end, or the input check has failed
            const int64_t q = p + row_ptr[c[j]];
            if (q < 0 || q >= 2 * n) continue;
            sym_col[q] = r[j];
            if (sw) sym_w[q] = w[j];
        }
    }
}

// Upper entry e of row r lands at e + lower_ptr[r + 1].
__global__ void sym_upper_kernel(const int32_t *__restrict__ row, const int32_t *__restrict__ col,
                                 const int32_t *__restrict__ w, int64_t n, int64_t m,
                                 const int64_t *__restrict__ lower_ptr, int32_t *__restrict__ sym_col,
                                 int32_t *__restrict__ sym_w) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x * kFlat;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x * kFlat + threadIdx.x; e0 < n; e0 += step) {
        int32_t r[kFlat], c[kFlat], ww[kFlat];
#pragma unroll
        for (int j = 0; j < kFlat; ++j) {
            const int64_t e = e0 + (int64_t)j * blockDim.x;
            const bool in = e < n;
            r[j] = in ? row[e] : -1;
            c[j] = in ? col[e] : 0;
            ww[j] = (in && w) ? w[e] : 0;
        }
#pragma unroll
        for (int j = 0; j < kFlat; ++j) {
            const int64_t e = e0 + (int64_t)j * blockDim.x;
            if (r[j] < 0 || r[j] >= m) continue;
            const int64_t q = e + lower_ptr[r[j] + 1];
            if (q < 0 || q >= 2 * n) continue;
            sym_col[q] = c[j];
            if (w) sym_w[q] = ww[j];
        }
    }
}

// The same by rows, one workgroup per row, where rows are long: the row's id
// is not read, and every wavefront's writes but a row's first and last are
// whole lines, past the caches. Only for pointers that passed the check (err):
// rows of others may overlap, up to n entries in each.
__global__ __launch_bounds__(256) void sym_upper_rows_kernel(const int64_t *__restrict__ row_ptr,
                                                             const int32_t *__restrict__ col,
                                                             const int32_t *__restrict__ w, int64_t n,
                                                             const int64_t *__restrict__ lower_ptr,
                                                             int32_t *__restrict__ sym_col,
                                                             int32_t *__restrict__ sym_w,
                                                             const int *__restrict__ err) {
    if (*err) return;
    const int64_t r = blockIdx.x, shift = lower_ptr[r + 1];
    const int64_t beg = max<int64_t>(row_ptr[r], 0), end = min(row_ptr[r + 1], n);
    constexpr int kAhead = 8;
    // positions in the output, from a multiple of 64 on
    for (int64_t q0 = (beg + shift) / 64 * 64 + threadIdx.x; q0 < end + shift; q0 += 256 * kAhead) {
        int32_t c[kAhead], x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t e = q0 + 256 * u - shift;
            c[u] = e >= beg && e < end ? col[e] : 0;
            x[u] = e >= beg && e < end && w ? w[e] : 0;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t q = q0 + 256 * u, e = q - shift;
            if (e < beg || e >= end || q >= 2 * n) continue;
            __builtin_nontemporal_store(c[u], sym_col + q);
            if (w) __builtin_nontemporal_store(x[u], sym_w + q);
        }
    }
}

// Edges per row from which that is faster than one thread per edge (2200 a
// row: 1.99 -> 1.43 ms for 4.4e8).
constexpr int64_t kLongRows = 256;

// ---------------------------------------------------------------------------
// Transpose of an upper triangle into the lower parts of its symmetric CSR
// ---------------------------------------------------------------------------
// A stable sort of the edges by column in two passes, high half of the
// column's bits first. Bound by HBM traffic; the general sort above took four
// passes over three arrays and a copy into place (16.6 ms for 4.4e8 edges of
// 200 000 hyperedges, 13.0 of them in its passes and their copy). Here
//   - the first pass's counts come with the check of the input;
//   - the first pass writes (row, low half) in one word beside the weight;
//   - the second pass goes bucket by bucket, so its counts are positions in
//     the whole list, give the column starts, and its items go straight to
//     their places in the output.
// A wavefront ranks kTrRounds rounds of its own contiguous items without a
// barrier (its counts in LDS, in order), so a tile has eight barriers where the
// sort above has three per round. The same edges now take 8.3 ms: 2.9 and 2.5
// in the passes (20 and 16 bytes an edge, 3.0 and 2.8 TB/s), 1.4 in the counts
// and the check, 1.4 in the upper copy. Tiles of 6144 items (three workgroups
// a CU) took 4.2 and 3.5, of 16 384 (one) 2.7 and 2.6.
constexpr int kTrThreads = 512;
constexpr int kTrWaves = kTrThreads / 64;
constexpr int kTrRounds = 16;
constexpr int kTrWaveItems = 64 * kTrRounds;
constexpr int kTrTile = kTrWaves * kTrWaveItems;

struct TransposeShape {
    int64_t n, m, chunk, chunks;  // items, vertices; items per chunk (whole tiles), first-pass chunks
    int low;                      // bits of the second digit
};

// Bucket b (columns [b << low, (b + 1) << low)): items [beg[b], beg[b + 1])
// of the first pass's output, second-pass chunks [first[b], first[b + 1]).
struct TransposeBuckets {
    int64_t *beg, *first;
};

template <int NB>
__device__ __forceinline__ void transpose_counts(const int (&h)[NB], int64_t at, int64_t step,
                                                 int32_t *__restrict__ hist) {
    for (int d = threadIdx.x; d < NB; d += kTrThreads) hist[at + d * step] = h[d];
}

// Checks that (row_ptr, row, col) is the upper triangle of a graph on m
// vertices in CSR order (row_ptr itself is check_ptr_kernel's): r < col < m,
// columns strictly increasing along a row, and each run of a row id starts
// and ends where row_ptr says, which the lanes at its ends look up. And the
// first pass's counts: hist[d * chunks + chunk] for d = col >> low.
template <int NB>
__global__ __launch_bounds__(kTrThreads) void check_count_kernel(TransposeShape s, const int64_t *__restrict__ row_ptr,
                                                                 const int32_t *__restrict__ row,
                                                                 const int32_t *__restrict__ col,
                                                                 int32_t *__restrict__ hist, int *__restrict__ err) {
    __shared__ int h[NB];
    const int lane = lane_id();
    for (int d = threadIdx.x; d < NB; d += kTrThreads) h[d] = 0;
    __syncthreads();
    bool bad = false;
    const int64_t beg = blockIdx.x * s.chunk, end = min(s.n, beg + s.chunk);
    for (int64_t e0 = beg + threadIdx.x; e0 - lane < end; e0 += kTrThreads * 8) {
        int32_t r[8], c[8], r0[8], c0[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t e = e0 + j * kTrThreads;
            r[j] = e < end ? row[e] : 0;
            c[j] = e < end ? col[e] : 1;
            r0[j] = c0[j] = -1;
            if (lane == 0 && e > 0 && e < end) {
                r0[j] = row[e - 1];
                c0[j] = col[e - 1];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t e = e0 + j * kTrThreads;
            const int ru = __shfl_up(r[j], 1), cu = __shfl_up(c[j], 1);
            const int rp = lane ? ru : r0[j], cp = lane ? cu : c0[j];
            // one count per run of equal digits
            const int d = ((unsigned)c[j] >> s.low) & (NB - 1);
            const unsigned long long heads = __ballot(lane == 0 || d != (int)(((unsigned)cu >> s.low) & (NB - 1)));
            const int live = (int)min<int64_t>(64, end - (e - lane));
            if (e >= end) continue;
            if (heads >> lane & 1) {
                const unsigned long long after = lane < 63 ? heads >> (lane + 1) : 0ull;
                atomicAdd(&h[d], min(live, after ? lane + __ffsll(after) : 64) - lane);
            }
            if (r[j] < 0 || c[j] <= r[j] || c[j] >= s.m) {
                bad = true;
                continue;
            }
            if (rp == r[j]) {
                bad |= cp >= c[j];
            } else {
                bad |= row_ptr[r[j]] != e;
                if (e > 0) bad |= rp < 0 || rp >= s.m || row_ptr[rp + 1] != e;
            }
            if (e == s.n - 1) bad |= row_ptr[r[j] + 1] != s.n;
        }
    }
    if (bad) atomicOr(err, 1);
    __syncthreads();
    transpose_counts(h, blockIdx.x, s.chunks, hist);
}

// One workgroup: the buckets from the first pass's offsets.
template <int NB>
__global__ __launch_bounds__(1024) void bucket_kernel(TransposeShape s, const int64_t *__restrict__ off,
                                                      TransposeBuckets k) {
    static_assert(NB <= 1024, "one bucket per thread");
    __shared__ int64_t ws[16];
    const int b = threadIdx.x;
    int64_t beg = s.n, q = 0, tot;
    if (b < NB) {
        beg = off[b * s.chunks];
        q = (off[(b + 1) * s.chunks] - beg + s.chunk - 1) / s.chunk;
    }
    const int64_t first = block_excl_scan<1024>(q, ws, tot);
    if (b < NB) {
        k.beg[b] = beg;
        k.first[b] = first;
    }
    if (b == 0) {
        k.beg[NB] = s.n;
        k.first[NB] = tot;
    }
}

// The bucket of second-pass chunk g, or -1 past the last; its items are
// [beg, end), its counts (off-) set at + d * step.
template <int NB>
__device__ __forceinline__ int chunk_of(const TransposeShape &s, const TransposeBuckets &k, int64_t g, int64_t &beg,
                                        int64_t &end, int64_t &at, int64_t &step) {
    if (g >= k.first[NB]) return -1;
    int b = 0;
#pragma unroll
    for (int w = NB / 2; w > 0; w >>= 1)  // the last bucket whose first chunk is <= g
        if (k.first[b + w] <= g) b += w;
    const int64_t f = k.first[b];
    step = k.first[b + 1] - f;
    beg = k.beg[b] + (g - f) * s.chunk;
    end = min(k.beg[b + 1], beg + s.chunk);
    at = f * NB + (g - f);
    return b;
}

template <int NB>
__global__ __launch_bounds__(kTrThreads) void bucket_count_kernel(TransposeShape s, TransposeBuckets k,
                                                                  const uint32_t *__restrict__ key,
                                                                  int32_t *__restrict__ hist) {
    __shared__ int h[NB];
    int64_t beg, end, at, step;
    if (chunk_of<NB>(s, k, blockIdx.x, beg, end, at, step) < 0) return;
    for (int d = threadIdx.x; d < NB; d += kTrThreads) h[d] = 0;
    __syncthreads();
    const unsigned mask = (1u << s.low) - 1u;
    for (int64_t e0 = beg + threadIdx.x; e0 < end; e0 += kTrThreads * 8) {
        uint32_t x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = e0 + j * kTrThreads < end ? key[e0 + j * kTrThreads] : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (e0 + j * kTrThreads < end) atomicAdd(&h[x[j] & mask], 1);
    }
    __syncthreads();
    transpose_counts(h, at, step, hist);
}

// lower_ptr[c]: the sorted position of column c's first item, c in [0, m];
// sym_ptr[c] beside it.
template <int NB>
__global__ void column_starts_kernel(TransposeShape s, TransposeBuckets k, const int64_t *__restrict__ off,
                                     const int64_t *__restrict__ row_ptr, int64_t *__restrict__ lower_ptr,
                                     int64_t *__restrict__ sym_ptr) {
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c <= s.m; c += (int64_t)gridDim.x * blockDim.x) {
        int64_t p = s.n;
        if (c < s.m) {
            const int64_t b = c >> s.low, d = c & ((1 << s.low) - 1), f = k.first[b], q = k.first[b + 1] - f;
            p = q > 0 ? off[f * NB + d * q] : k.beg[b];
        }
        lower_ptr[c] = p;
        sym_ptr[c] = p + row_ptr[c];
    }
}

// One chunk, a tile at a time. FIRST: (col, row, w) to (row << low | low bits
// of col, w) by the high digit; else (key, w) of one bucket to (row, w) of
// the output by the low digit.
template <int NB, bool FIRST>
__global__ __launch_bounds__(kTrThreads, 4) void transpose_kernel(
    TransposeShape s, TransposeBuckets k, const int32_t *__restrict__ key_in, const int32_t *__restrict__ row_in,
    const int32_t *__restrict__ w_in, const int64_t *__restrict__ off, const int64_t *__restrict__ row_ptr,
    int32_t *__restrict__ key_out, int32_t *__restrict__ w_out) {
    __shared__ int32_t tile[kTrTile];
    __shared__ uint16_t dig[kTrTile];
    __shared__ uint16_t cnt[kTrWaves][NB];  // counts of a wavefront, then its starts within the digit
    __shared__ int64_t run[NB];             // next output position of a digit
    __shared__ uint16_t dstart[NB];         // a digit's first place in the tile
    __shared__ int ws[kTrWaves];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int64_t beg, end, at, step;
    int64_t room = s.n;  // of the output
    if (FIRST) {
        beg = blockIdx.x * s.chunk;
        end = min(s.n, beg + s.chunk);
        at = blockIdx.x;
        step = s.chunks;
        for (int d = threadIdx.x; d < NB; d += kTrThreads) run[d] = off[at + d * step];
    } else {
        const int b = chunk_of<NB>(s, k, blockIdx.x, beg, end, at, step);
        if (b < 0) return;
        room = 2 * s.n;
        for (int d = threadIdx.x; d < NB; d += kTrThreads) {
            const int64_t c = ((int64_t)b << s.low) + d;
            // no items have these digits unless the input check has failed
            run[d] = d >> s.low || c >= s.m ? room : off[at + d * step] + row_ptr[c];
        }
    }
    const unsigned mask = (1u << s.low) - 1u;
    for (int64_t t0 = beg; t0 < end; t0 += kTrTile) {
        const int tn = (int)min((int64_t)kTrTile, end - t0);
        const int first = wave * kTrWaveItems + lane;
        uint32_t x[kTrRounds];
        int32_t y[kTrRounds], wt[kTrRounds];
        int place[kTrRounds];  // digit << 16 | rank within the wavefront's digit
#pragma unroll
        for (int r = 0; r < kTrRounds; ++r) {
            const int i = first + 64 * r;
            x[r] = i < tn ? (uint32_t)key_in[t0 + i] : 0u;
            if (FIRST) y[r] = i < tn ? row_in[t0 + i] : 0;
        }
        for (int d = lane; d < NB; d += 64) cnt[wave][d] = 0;
        volatile uint16_t *mine = cnt[wave];
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < kTrRounds; ++r) {
            const bool in = first + 64 * r < tn;  // a prefix of the lanes
            const int d = FIRST ? (int)((x[r] >> s.low) & (NB - 1)) : (int)(x[r] & mask);
            x[r] = FIRST ? (uint32_t)y[r] << s.low | (x[r] & mask) : x[r] >> s.low;  // what is written
            const unsigned long long live = __ballot(in);
            int rank, num;
            const int dp = __shfl_up(d, 1);
            if (FIRST && !__ballot(in && lane > 0 && d < dp)) {
                // one row's columns ascend: equal digits are runs of lanes
                const unsigned long long heads = __ballot(in && (lane == 0 || d != dp));
                const int head = 63 - __clzll(heads & (~0ull >> (63 - lane)) | 1ull);
                const unsigned long long after = lane < 63 ? heads & (~0ull << (lane + 1)) : 0ull;
                rank = lane - head;
                num = (after ? __ffsll(after) - 1 : __popcll(live)) - head;
            } else {
                unsigned long long peers = live;
#pragma unroll
                for (int bit = 1; bit < NB; bit <<= 1) {
                    const unsigned long long bb = __ballot(d & bit);
                    peers &= d & bit ? bb : ~bb;
                }
                rank = bits_below(peers);
                num = __popcll(peers);
            }
            const int before = mine[d];
            place[r] = d << 16 | (before + rank);
            if (in && rank == 0) mine[d] = (uint16_t)(before + num);
            wave_lds_sync();
        }
#pragma unroll
        for (int r = 0; r < kTrRounds; ++r) wt[r] = w_in && first + 64 * r < tn ? w_in[t0 + first + 64 * r] : 0;
        __syncthreads();
        // counts to starts: of each wavefront within its digit, of the digit in the tile
        {
            constexpr int per = NB / kTrThreads > 0 ? NB / kTrThreads : 1;
            int tot[per], sum = 0;
#pragma unroll
            for (int j = 0; j < per; ++j) {
                const int d = threadIdx.x * per + j;
                tot[j] = 0;
                if (d >= NB) break;
                int run_w = 0;
#pragma unroll
                for (int w = 0; w < kTrWaves; ++w) {
                    const int c = cnt[w][d];
                    cnt[w][d] = (uint16_t)run_w;
                    run_w += c;
                }
                tot[j] = run_w;
                sum += run_w;
            }
            int all;
            int st = block_excl_scan<kTrThreads>(sum, ws, all);
#pragma unroll
            for (int j = 0; j < per; ++j) {
                if (threadIdx.x * per + j < NB) dstart[threadIdx.x * per + j] = (uint16_t)st;
                st += tot[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kTrRounds; ++r) {
            const int d = place[r] >> 16;
            place[r] = dstart[d] + cnt[wave][d] + (place[r] & 0xFFFF);
            if (first + 64 * r < tn) {
                dig[place[r]] = (uint16_t)d;
                tile[place[r]] = (int32_t)x[r];
            }
        }
        __syncthreads();
        auto out = [&](int32_t *__restrict__ to) {
#pragma unroll 4
            for (int q = threadIdx.x; q < tn; q += kTrThreads) {
                const int d = dig[q];
                const int64_t pos = run[d] + (q - dstart[d]);
                if (pos >= 0 && pos < room) to[pos] = tile[q];
            }
        };
        out(key_out);
        if (w_in) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kTrRounds; ++r)
                if (first + 64 * r < tn) tile[place[r]] = wt[r];
            __syncthreads();
            out(w_out);
        }
        __syncthreads();
        // next tile: the digits' positions advance
        for (int d = threadIdx.x; d < NB; d += kTrThreads) run[d] += (d + 1 < NB ? (int)dstart[d + 1] : tn) - dstart[d];
    }
}

// Order-independent digest of an edge list: the number of edges, the sum
// of the overlaps, and the sum mod 2^64 of SplitMix64's output function
// (Steele, Lea and Flood's mixer as published by Vigna) applied to
// i * 2^32 + j, xor the overlap. Equal edge sets give equal digests in any
// order, and the digests of disjoint parts add up to the digest of their
// union, so a streamed result can be checked chunk by chunk.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x) {
    unsigned long long z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void digest_kernel(const int32_t *__restrict__ row, const int32_t *__restrict__ col,
                                                     const int32_t *__restrict__ w, int64_t n,
                                                     unsigned long long *__restrict__ out) {
    unsigned long long cnt = 0, sw = 0, h = 0;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long i = (unsigned)row[e], j = (unsigned)col[e];
        const unsigned long long x = (unsigned long long)(unsigned)w[e];
        cnt += 1;
        sw += x;
        h += splitmix64((i << 32) | j) ^ x;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        cnt += __shfl_xor(cnt, o);
        sw += __shfl_xor(sw, o);
        h += __shfl_xor(h, o);
    }
    if ((threadIdx.x & 63) == 0 && cnt) {
        atomicAdd(&out[0], cnt);
        atomicAdd(&out[1], sw);
        atomicAdd(&out[2], h);
    }
}

inline unsigned sort_grid(int64_t items, int threads, int64_t cap) {
    int64_t b = (items + threads - 1) / threads;
    if (b > cap) b = cap;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

int64_t sort_chunks(int64_t n) { return (n + kSortChunk - 1) / kSortChunk; }

int sort_passes(int key_bits) { return key_bits <= 0 ? 0 : (key_bits + kSortDigitBits - 1) / kSortDigitBits; }

hipError_t launch_sort_pass(const int32_t *key_in, const int32_t *a_in, const int32_t *b_in, int64_t n, int shift,
                            int bits, int32_t *hist, int64_t *off, int64_t *partials, int32_t *key_out,
                            int32_t *a_out, int32_t *b_out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (bits < 1 || bits > kSortDigitBits || shift < 0 || shift + bits > 32) return hipErrorInvalidValue;
    const int64_t nchunks = sort_chunks(n);
    const unsigned grid = (unsigned)(nchunks < 65536 ? nchunks : 65536);
    sort_hist_kernel<<<grid, kSortThreads, 0, st>>>(key_in, n, shift, bits, nchunks, hist);
    hipError_t e = launch_exclusive_scan_i32(hist, (int64_t)(1 << bits) * nchunks, off, partials, st);
    if (e != hipSuccess) return e;
    if (b_in)
        sort_scatter_kernel<2><<<grid, kSortThreads, 0, st>>>(key_in, a_in, b_in, n, shift, bits, nchunks, off,
                                                               key_out, a_out, b_out);
    else if (a_in)
        sort_scatter_kernel<1><<<grid, kSortThreads, 0, st>>>(key_in, a_in, nullptr, n, shift, bits, nchunks, off,
                                                               key_out, a_out, nullptr);
    else
        sort_scatter_kernel<0><<<grid, kSortThreads, 0, st>>>(key_in, nullptr, nullptr, n, shift, bits, nchunks,
                                                               off, key_out, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_digest(const int32_t *row, const int32_t *col, const int32_t *w, int64_t n,
                         unsigned long long *out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    digest_kernel<<<sort_grid(n, 256, 8192), 256, 0, st>>>(row, col, w, n, out);
    return hipGetLastError();
}

hipError_t launch_key_bounds(const int32_t *skey, int64_t n, int64_t m, int64_t *lower_ptr, hipStream_t st) {
    key_bounds_kernel<<<sort_grid(m + 1, 256, 4096), 256, 0, st>>>(skey, n, m, lower_ptr);
    return hipGetLastError();
}

// The second digit has the larger half of the bits; a packed word holds the
// row and it.
bool transpose_packs(int64_t m) { return m <= (int64_t(1) << 20); }

namespace {
int transpose_low(int64_t m) {
    int bits = 1;
    while ((int64_t(1) << bits) < m) ++bits;
    return (bits + 1) / 2;
}
int transpose_bins(int64_t m) { return m <= (int64_t(1) << 18) ? 512 : 1024; }
// Whole tiles: eight where that leaves at least 1024 chunks.
int64_t transpose_chunk(int64_t n) {
    int64_t tiles = n / (int64_t(1024) * kTrTile);
    tiles = tiles < 1 ? 1 : (tiles > 8 ? 8 : tiles);
    return tiles * kTrTile;
}
}  // namespace

int64_t transpose_counts_size(int64_t n, int64_t m) {
    const int64_t chunk = transpose_chunk(n);
    return ((n + chunk - 1) / chunk + transpose_bins(m)) * transpose_bins(m);
}

hipError_t launch_transpose(const int64_t *row_ptr, const int32_t *row, const int32_t *col, const int32_t *w,
                            int64_t n, int64_t m, const TransposeScratch &t, int64_t *lower_ptr, int64_t *sym_ptr,
                            int32_t *sym_col, int32_t *sym_w, int *err, hipStream_t st) {
    if (n <= 0 || m <= 0 || !transpose_packs(m)) return hipErrorInvalidValue;
    const int64_t chunk = transpose_chunk(n), chunks = (n + chunk - 1) / chunk;
    const int nb = transpose_bins(m);
    if (chunks + nb > INT_MAX) return hipErrorInvalidValue;
    const TransposeShape s{n, m, chunk, chunks, transpose_low(m)};
    const TransposeBuckets k{t.buckets, t.buckets + 1025};
    const unsigned g1 = (unsigned)chunks, g2 = (unsigned)(chunks + nb);
    check_ptr_kernel<<<sort_grid(m, 256, 4096), 256, 0, st>>>(row_ptr, m, n, err);
    hipError_t e;
#define SLG_TRANSPOSE(NB)                                                                                            \
    do {                                                                                                             \
        check_count_kernel<NB><<<g1, kTrThreads, 0, st>>>(s, row_ptr, row, col, t.hist, err);                        \
        if ((e = launch_exclusive_scan_i32(t.hist, chunks * NB, t.off, t.partials, st)) != hipSuccess) return e;     \
        bucket_kernel<NB><<<1, 1024, 0, st>>>(s, t.off, k);                                                          \
        transpose_kernel<NB, true><<<g1, kTrThreads, 0, st>>>(s, k, col, row, w, t.off, nullptr, t.key, t.w);        \
        if ((e = launch_fill_i32(t.hist, (chunks + NB) * NB, 0, st)) != hipSuccess) return e;                        \
        bucket_count_kernel<NB><<<g2, kTrThreads, 0, st>>>(s, k, reinterpret_cast<const uint32_t *>(t.key), t.hist); \
        if ((e = launch_exclusive_scan_i32(t.hist, (chunks + NB) * NB, t.off, t.partials, st)) != hipSuccess)        \
            return e;                                                                                                \
        column_starts_kernel<NB><<<sort_grid(m + 1, 256, 4096), 256, 0, st>>>(s, k, t.off, row_ptr, lower_ptr,       \
                                                                               sym_ptr);                             \
        transpose_kernel<NB, false><<<g2, kTrThreads, 0, st>>>(s, k, t.key, nullptr, w ? t.w : nullptr, t.off,       \
                                                                row_ptr, sym_col, sym_w);                            \
    } while (0)
    if (nb == 512)
        SLG_TRANSPOSE(512);
    else
        SLG_TRANSPOSE(1024);
#undef SLG_TRANSPOSE
    if (n / m >= kLongRows)
        sym_upper_rows_kernel<<<(unsigned)m, 256, 0, st>>>(row_ptr, col, w, n, lower_ptr, sym_col, sym_w, err);
    else
        sym_upper_kernel<<<sort_grid(n, 256 * kFlat, 16384), 256, 0, st>>>(row, col, w, n, m, lower_ptr, sym_col,
                                                                           sym_w);
    return hipGetLastError();
}

hipError_t launch_check_upper(const int64_t *row_ptr, const int32_t *row, const int32_t *col, int64_t n, int64_t m,
                              int *err, hipStream_t st) {
    check_ptr_kernel<<<sort_grid(m > 0 ? m : 1, 256, 4096), 256, 0, st>>>(row_ptr, m, n, err);
    if (n > 0) check_upper_kernel<<<sort_grid(n, 256 * kFlat, 16384), 256, 0, st>>>(row_ptr, row, col, n, m, err);
    return hipGetLastError();
}

hipError_t launch_symmetric(const int32_t *skey, const int32_t *srow, const int32_t *sw, const int64_t *row_ptr,
                            const int32_t *row, const int32_t *col, const int32_t *w, int64_t n, int64_t m,
                            int64_t *lower_ptr, int64_t *sym_ptr, int32_t *sym_col, int32_t *sym_w,
                            hipStream_t st) {
    key_bounds_kernel<<<sort_grid(m + 1, 256, 4096), 256, 0, st>>>(skey, n, m, lower_ptr);
    sym_ptr_kernel<<<sort_grid(m + 1, 256, 4096), 256, 0, st>>>(lower_ptr, row_ptr, m, sym_ptr);
    if (n > 0) {
        sym_lower_kernel<<<sort_grid(n, 256 * kFlat, 16384), 256, 0, st>>>(skey, srow, sw, n, m, row_ptr, sym_col, sym_w);
        sym_upper_kernel<<<sort_grid(n, 256 * kFlat, 16384), 256, 0, st>>>(row, col, w, n, m, lower_ptr, sym_col, sym_w);
    }
    return hipGetLastError();
}

}  // namespace slg
