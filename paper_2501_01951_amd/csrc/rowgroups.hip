// fp32 neighbor aggregation over whole matrices: columns dealt to bands, rows grouped by length.
//
// Bands.  Every XCD's 4 MiB of L2 hold 32 k of the 128-byte lines that a column slice has per node, a
// gather that misses costs four times one that hits, and an LRU cache keeps far less than the most
// popular lines.  So where a graph is dense enough the columns are dealt to bands by popularity, 26 k
// columns each and the rest in the last, and the bands are aggregated one after the other; the later
// ones add to what the earlier ones left in Z.  How many bands pay is estimated from the degree histogram
// (plan_bands).  Power law, 233 k nodes, 492 entries per row, 128 columns, 9 bands: 7.19 -> 3.44 ms, 52 -> 11
// GB read, 18 -> 83 % L2 hits (the entries that stream through the same L2 push out some of a band's lines).
//
// Groups.  Within a band rows are short, and closing them one at a time (three rounds of lane
// exchanges and a store by an eighth of the lanes, as the entry-balanced kernel of spmm.hip does)
// would take most of the time.  So they are laid out such that eight of them end together:
//
//   short rows (1 to 64 entries)  are sorted by length, longest first, and taken eight at a time:
//                                 a *group*.  Batch j of a group holds entry j of each of its eight
//                                 rows, so the eight lanes of a sub-group own one row from its first
//                                 entry to its last, add in registers and write it themselves.
//   longer rows                   are a group each: batch j holds entries 8 j .. 8 j + 7 of the row,
//                                 and the eight sub-group sums are combined once at its end.
//   very long rows                are cut into pieces, a group each, whose sums go to scratch slots
//                                 that a second kernel adds in order (deterministic, no atomics).
//
// The groups are stored one after the other as one stream of batches of eight {column, value}
// entries.  A wavefront takes the groups that start in its part of the stream, for one column slice
// of 8 lanes, so nothing crosses from one wavefront to the next.  The sort works within windows of
// 4096 consecutive rows: the padding of a group is the spread of eight neighbors in sorted order,
// while the rows written at the same time stay close together (rows sorted over the whole graph: 3 %
// slower with plain stores, 12 % with an epilogue that reads).
//
// A matrix with one band has no groups: its aggregations are those of the entry-balanced kernel.
//
// Rounding.  The entry-balanced kernel adds a row of n entries in eight chains and a tree, with an error
// variance of about n^2 / 16 + 3 n (in units of that of one addition to a sum of one entry).  A short row
// has one sub-group here, whose lanes keep four chains, one per gather in flight: over k bands
// n^2 / 8 k + (k + 3) n / 2, less from n = 9 k on.  plan_bands asks for 12 k.  Measured against 64 bits,
// the rms error of 128 columns is 0.995 of the entry-balanced kernel's for 2 bands of 30 entries per row
// (one chain: 1.26), 0.92 for 4 bands of 25 (1.19), 0.90 for 5 of 18 on a power law (1.08), 0.93 for 7 of
// 14 (1.10) and 0.64 for 9 of 55 (0.82).  The chains cost nothing (100 k nodes, 100 per row, 4 bands: 399
// us with one chain and 8 wavefronts per SIMD, 385 with four and 6; 4 and 8 wavefronts spill).
#include <cmath>

#include "agg_common.h"

namespace mixgcn {
namespace {

constexpr int kGroupRows = 8;   // rows of a group, sub-groups of a wavefront
constexpr int kMostShort = 64;  // longest row that may share a group with others
constexpr int kWindowItems = 16;
constexpr int kWindow = kBlock * kWindowItems;  // rows sorted together
// Stream positions for which the first group that starts there is tabulated (batches).
constexpr int kTabBatches = 8;
constexpr int kRowPad = 2 * kGroupRows;  // groups whose rows may be read past the end
constexpr int kStreamPad = 128 * kGroupRows;  // entries that the pipeline may read past the end

// Marks in bits 30 and 31 of the column word of the first entry of a group's last batch.
constexpr uint32_t kEndGroup = 1u << 30;  // every sub-group closes its own row
constexpr uint32_t kEndRow = 2u << 30;    // the sub-groups close one row together
constexpr uint32_t kEndPiece = 3u << 30;  // they close a piece of a row
constexpr uint32_t kPadValue = 0x80000000u;  // value word (-0.0) of an entry that stands for nothing
// A row of a group: its index and what the band is to it.
constexpr uint32_t kRowMask = 0x3FFFFFFFu;
constexpr uint32_t kNoRow = kRowMask;
constexpr uint32_t kRowAdds = 1u << 31;   // an earlier band has written the row
constexpr uint32_t kRowMore = 1u << 30;   // a later band will add to it: no epilogue yet

// Classes of the row sort: pieces, single long rows, short rows by falling length, empty rows.
constexpr int kClassPieces = 0;
constexpr int kClassLong = 1;
constexpr int kClassEmpty = kMostShort + 2;

__device__ inline int row_class(int64_t len, int64_t piece, int short_row)
{
    if (len > piece) return kClassPieces;
    if (len > short_row) return kClassLong;
    return kClassEmpty - (int)len;
}

// ---- bands ----------------------------------------------------------------------------------------

constexpr int kBandColumns = 26000;  // columns of a band: 4/5 of the lines of an XCD's L2
constexpr int kBandBits = 4;
constexpr int kMostBands = 1 << kBandBits;
// Least entries of a row per band on average: with fewer the sums lose precision (see the top).
constexpr int kBandRow = 12;
// Largest matrix that may have bands.  Above it the two forms together (24 bytes per entry) would not
// leave room for the features.
constexpr int64_t kMostEntries = 1ll << 31;
// Popularity bins, most popular first: exact up to 64 entries, 16 bins per factor of two above.
constexpr int kBins = 256;

__device__ inline int popularity_bin(int64_t len)
{
    if (len < 64) return kBins - 1 - (int)len;
    const int e = 63 - __clzll((long long)len);  // 2^e <= len
    const int b = 64 + (e - 6) * 16 + (int)((len >> (e - 4)) & 15);
    return b > kBins - 1 ? 0 : kBins - 1 - b;
}

// Rows and entries per bin, and the sort keys (row << 8 | bin).
__global__ __launch_bounds__(kBlock) void popularity_kernel(const int64_t* __restrict__ rowptr,
                                                            uint32_t n, uint64_t* __restrict__ keys,
                                                            unsigned long long* __restrict__ rows,
                                                            unsigned long long* __restrict__ entries)
{
    __shared__ unsigned long long hr[kBins], he[kBins];
    hr[threadIdx.x] = 0;
    he[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < n; r += (int64_t)gridDim.x * kBlock) {
        const int64_t len = rowptr[r + 1] - rowptr[r];
        const int b = popularity_bin(len);
        keys[r] = (uint64_t)r << 8 | (uint64_t)b;
        atomicAdd(&hr[b], 1ull);
        atomicAdd(&he[b], (unsigned long long)len);
    }
    __syncthreads();
    if (hr[threadIdx.x]) {
        atomicAdd(&rows[threadIdx.x], hr[threadIdx.x]);
        atomicAdd(&entries[threadIdx.x], he[threadIdx.x]);
    }
}

__global__ __launch_bounds__(kBlock) void band_of_column_kernel(const uint64_t* __restrict__ sorted,
                                                                uint32_t n, uint32_t per_band,
                                                                int n_bands, uint8_t* __restrict__ band)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t b = i / per_band;
    band[sorted[i] >> 8] = (uint8_t)(b < (uint32_t)n_bands ? b : n_bands - 1);
}

// Entries of every row in every band, one wavefront per row.  FILL: pos[b][r] is where the row's
// entries of band b start, and the entry indices are written there in their order in the row;
// otherwise their counts go to count[b][r].  A hub's row is a chain of steps of 64 entries, so the loads of
// eight are in flight and a step has a ballot per bit of the band, not one per band (70 M entries on 233 k
// nodes, one of them tied to all others: the whole build 13.2 -> 6.5 ms, 5.7 without the hub).
template <bool FILL>
__global__ __launch_bounds__(kBlock) void deal_entries_kernel(
    const int64_t* __restrict__ rowptr, const uint32_t* __restrict__ col,
    const uint8_t* __restrict__ band, uint32_t n, int n_bands, uint32_t* __restrict__ count,
    const uint64_t* __restrict__ pos, uint32_t* __restrict__ src)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
    if (r >= n) return;
    const int64_t e0 = rowptr[r], e1 = rowptr[r + 1];
    // lane b keeps the running count (or position) of band b
    uint64_t run = FILL && lane < n_bands ? pos[(int64_t)lane * n + r] : 0;
    // One step; mine: band of the lane's entry, -1 for none.  From a ballot per bit every lane has the
    // lanes with entries of its own entry's band and, for lane b, those of band b.
    auto deal = [&](int64_t e, int mine) {
        uint64_t same = __ballot(mine >= 0), own = same;
#pragma unroll
        for (int i = 0; i < kBandBits; ++i) {
            const uint64_t m = __ballot((mine >> i) & 1);
            same &= (mine >> i) & 1 ? m : ~m;
            own &= (lane >> i) & 1 ? m : ~m;
        }
        if (FILL) {
            const uint64_t at = __shfl((unsigned long long)run, mine & (kWave - 1), kWave);
            if (mine >= 0) src[at + __popcll(same & ((1ull << lane) - 1))] = (uint32_t)(e + lane);
        }
        run += __popcll(own);  // meaningless in lanes past the bands
    };
    constexpr int kAhead = 8;
    int64_t e = e0;
    for (; e + kAhead * kWave <= e1; e += kAhead * kWave) {
        uint32_t c[kAhead];
        int mine[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) c[j] = col[e + j * kWave + lane];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) mine[j] = band[c[j]];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) deal(e + j * kWave, mine[j]);
    }
    for (; e < e1; e += kWave) deal(e, e + lane < e1 ? band[col[e + lane]] : -1);
    if (!FILL && lane < n_bands) count[(int64_t)lane * n + r] = (uint32_t)run;
}

// rowptr of a band relative to its own entries
__global__ __launch_bounds__(kBlock) void band_rowptr_kernel(const uint64_t* __restrict__ pos,
                                                             int64_t n, int b, int n_bands,
                                                             int64_t nnz, int64_t* __restrict__ rowptr)
{
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r > n) return;
    const uint64_t* p = pos + (int64_t)b * n;
    const int64_t end = b + 1 < n_bands ? (int64_t)p[n] : nnz;
    rowptr[r] = (r < n ? (int64_t)p[r] : end) - (int64_t)p[0];
}

// Share of gathers that miss an LRU cache of `lines` lines when column classes of `count` columns
// with `entries` gathers in all are hit independently (Che's approximation: a line stays for a
// fixed number of gathers T, chosen so that the cache is full).
struct Popular {
    double count, entries;
};
double lru_misses(const Popular* c, int n, double lines)
{
    double total = 0, columns = 0;
    for (int i = 0; i < n; ++i) {
        total += c[i].entries;
        columns += c[i].count;
    }
    if (columns <= lines || total <= 0) return 0;
    double lo = 0, hi = total * 1e6;
    for (int it = 0; it < 100; ++it) {
        const double T = 0.5 * (lo + hi);
        double full = 0;
        for (int i = 0; i < n; ++i)
            if (c[i].count > 0) full += c[i].count * -expm1(-c[i].entries / c[i].count / total * T);
        (full < lines ? lo : hi) = T;
    }
    double miss = 0;
    for (int i = 0; i < n; ++i)
        if (c[i].count > 0) miss += c[i].entries * exp(-c[i].entries / c[i].count / total * lo);
    return miss / total;
}

// Number of bands for a matrix with the given rows and entries per bin (most popular first).  In
// units of a gather that misses (18 ps per line over the chip), a hit measured 0.3 to 0.38 and a row
// that a later band adds to 3 to 6 lines: its old line is read with a miss that the gathers queued
// behind it wait for, and written again.
constexpr double kHit = 0.35, kLines = 29000;
int plan_bands(const unsigned long long* rows, const unsigned long long* entries, double n, double nnz,
               RowGroups* out)
{
    constexpr double kInBand = 0.03, kRow = 5;
    const int most = nnz / n / kBandRow < kMostBands ? (int)(nnz / n / kBandRow) : kMostBands;
    int best = 1;
    double best_cost = 0;
    for (int k = 1; k <= most && (k - 1) * (double)kBandColumns < n; ++k) {
        double cost = 0;
        Popular rest[kBins];
        int n_rest = 0;
        double share[kMostBands] = {};
        double rank = 0;
        for (int i = 0; i < kBins; ++i) {
            double left = (double)rows[i];
            if (left <= 0) continue;
            const double each = (double)entries[i] / left;
            while (left > 0) {
                int b = (int)(rank / kBandColumns);
                if (b > k - 1) b = k - 1;
                double take = left;
                if (b < k - 1 && rank + take > (b + 1) * (double)kBandColumns)
                    take = (b + 1) * (double)kBandColumns - rank;
                share[b] += take * each / nnz;
                if (b == k - 1) rest[n_rest++] = Popular{take, take * each};
                rank += take;
                left -= take;
            }
        }
        for (int b = 0; b < k; ++b) {
            const double miss = b < k - 1 ? kInBand : lru_misses(rest, n_rest, kLines);
            cost += share[b] * (miss + (1 - miss) * kHit);
            if (b == 0) continue;
            for (int i = 0; i < kBins; ++i)  // rows that have an entry in the band
                if (rows[i])
                    cost += kRow * (double)rows[i] / nnz *
                            -expm1(-(double)entries[i] / (double)rows[i] * share[b]);
        }
        // Bands have to promise a fifth: the estimate takes columns and rows for independent, and
        // where popular rows prefer popular columns (R-MAT) it promises up to 15 % that are not
        // there.  Uniform columns, 100 k nodes, 100 entries per row: 566 -> 373 us with 4 bands
        // (estimate 0.81 -> 0.51); power law, 233 k nodes, 492 per row: 7.2 -> 3.5 ms with 9.
        if (k == 1) {
            out->most_cost = 0.85 * cost;  // with the launches (rowgroups_take)
            best_cost = 0.8 * cost;
        } else if (cost < best_cost) {
            out->cost = best_cost = cost;
            best = k;
        }
    }
    return best;
}

// ---- layout ---------------------------------------------------------------------------------------

// What a window of rows contributes.
struct WindowPlan {
    uint32_t cut, pieces, groups, batches;
};

// Sorts the rows of a window by class (stable) and counts what they need; one block per window.
__global__ __launch_bounds__(kBlock) void window_sort_kernel(const int64_t* __restrict__ rowptr,
                                                             uint32_t n, int64_t piece, int short_row,
                                                             uint32_t* __restrict__ sorted,
                                                             uint2* __restrict__ long_short,
                                                             WindowPlan* __restrict__ plan)
{
    __shared__ uint32_t whist[kBlock / kWave][256];
    __shared__ uint32_t base[256];
    __shared__ uint64_t scan[4];
    __shared__ uint32_t pieces, batches;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) whist[i][threadIdx.x] = 0;
    if (threadIdx.x == 0) pieces = batches = 0;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
    const int64_t first = (int64_t)blockIdx.x * kWindow;
    const int64_t row0 = first + (int64_t)w * kWindowItems * kWave + lane;
    uint32_t digit[kWindowItems], rank[kWindowItems];
    bool valid[kWindowItems];
#pragma unroll
    for (int i = 0; i < kWindowItems; ++i) {
        const int64_t r = row0 + (int64_t)i * kWave;
        valid[i] = r < n;
        const int64_t len = valid[i] ? rowptr[r + 1] - rowptr[r] : 0;
        digit[i] = (uint32_t)row_class(len, piece, short_row);
        if (valid[i] && digit[i] == kClassPieces) {
            const int64_t full = len / piece, rest = len % piece;
            atomicAdd(&pieces, (uint32_t)(full + (rest ? 1 : 0)));
            atomicAdd(&batches, (uint32_t)(full * (piece / kGroupRows) + (rest + kGroupRows - 1) / kGroupRows));
        } else if (valid[i] && digit[i] == kClassLong) {
            atomicAdd(&batches, (uint32_t)((len + kGroupRows - 1) / kGroupRows));
        }
    }
    wave_digit_ranks(digit, valid, whist, rank);
    __syncthreads();
    const int d = threadIdx.x;  // thread d: class d
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) {
        const uint32_t c = whist[i][d];
        whist[i][d] = total;
        total += c;
    }
    uint64_t all;
    const uint32_t b = (uint32_t)block_exclusive_scan_u64(total, &all, scan);
    base[d] = b;
    __syncthreads();
    const uint32_t short0 = base[kClassLong + 1];
    if (d > kClassLong && d < kClassEmpty && total > 0) {
        // a group of short rows is as long as its first row
        const uint32_t g0 = (b - short0 + kGroupRows - 1) / kGroupRows;
        const uint32_t g1 = (b - short0 + total + kGroupRows - 1) / kGroupRows;
        atomicAdd(&batches, (g1 - g0) * (uint32_t)(kClassEmpty - d));
    }
#pragma unroll
    for (int i = 0; i < kWindowItems; ++i)
        if (valid[i])
            sorted[first + base[digit[i]] + whist[w][digit[i]] + rank[i]] =
                (uint32_t)(row0 + (int64_t)i * kWave);
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t n_cut = base[kClassLong], n_long = short0 - n_cut, n_short = base[kClassEmpty] - short0;
        long_short[blockIdx.x] = make_uint2(n_long, n_short);
        plan[blockIdx.x] = WindowPlan{n_cut, pieces, pieces + n_long + (n_short + kGroupRows - 1) / kGroupRows,
                                      batches};
    }
}

struct WindowStart {
    uint64_t cut, pieces, groups, batches;
};

// Exclusive prefix sums over the windows; start[n_windows] = totals.  One block.
__global__ __launch_bounds__(kBlock) void window_scan_kernel(const WindowPlan* __restrict__ plan,
                                                             int64_t n_windows,
                                                             WindowStart* __restrict__ start)
{
    __shared__ uint64_t lds[4];
    WindowStart run{0, 0, 0, 0};
    for (int64_t i0 = 0; i0 < n_windows; i0 += kBlock) {
        const int64_t i = i0 + threadIdx.x;
        const WindowPlan p = i < n_windows ? plan[i] : WindowPlan{0, 0, 0, 0};
        WindowStart o;
        uint64_t t;
        o.cut = run.cut + block_exclusive_scan_u64(p.cut, &t, lds);
        run.cut += t;
        o.pieces = run.pieces + block_exclusive_scan_u64(p.pieces, &t, lds);
        run.pieces += t;
        o.groups = run.groups + block_exclusive_scan_u64(p.groups, &t, lds);
        run.groups += t;
        o.batches = run.batches + block_exclusive_scan_u64(p.batches, &t, lds);
        run.batches += t;
        if (i < n_windows) start[i] = o;
    }
    if (threadIdx.x == 0) start[n_windows] = run;
}

// Whether a row has entries in an earlier or a later band.
__device__ inline uint32_t band_marks(const uint32_t* __restrict__ count, int64_t n, int64_t row,
                                      int band, int n_bands)
{
    uint32_t marks = 0;
    for (int b = 0; b < n_bands; ++b)
        if (b != band && count[b * n + row]) marks |= b < band ? kRowAdds : kRowMore;
    return marks;
}

// Kinds of groups.  The eight row words of a group hold its rows; those of a long row hold the row and
// seven times kNoRow, those of a piece kNoRow alone.
constexpr uint32_t kKindShort = 0;
constexpr uint32_t kKindLong = 1;
constexpr uint32_t kKindPiece = 2;  // + slot of the piece

// Lays out the groups of a window: rows, kinds and lengths in batches; one block per window.
__global__ __launch_bounds__(kBlock) void window_groups_kernel(
    const int64_t* __restrict__ rowptr, const uint32_t* __restrict__ sorted,
    const uint2* __restrict__ long_short, const WindowStart* __restrict__ start, int64_t piece,
    const uint32_t* __restrict__ band_count, int64_t n, int band, int n_bands,
    uint32_t* __restrict__ rows, uint32_t* __restrict__ kind, uint32_t* __restrict__ len,
    uint32_t* __restrict__ cut_row, uint64_t* __restrict__ piece0)
{
    const WindowStart at = start[blockIdx.x], next = start[blockIdx.x + 1];
    const int n_cut = (int)(next.cut - at.cut);
    const int n_long = (int)long_short[blockIdx.x].x, n_short = (int)long_short[blockIdx.x].y;
    const uint32_t* const mine = sorted + (int64_t)blockIdx.x * kWindow;
    int64_t k = (int64_t)at.groups;
    int64_t slot = (int64_t)at.pieces;
    for (int i = 0; i < n_cut; ++i) {
        const uint32_t r = mine[i];
        const int64_t entries = rowptr[r + 1] - rowptr[r], count = (entries + piece - 1) / piece;
        if (threadIdx.x == 0) {
            cut_row[at.cut + i] = r | band_marks(band_count, n, r, band, n_bands);
            piece0[at.cut + i] = (uint64_t)slot;
        }
        for (int64_t p = threadIdx.x; p < count; p += kBlock) {
            const int64_t left = entries - p * piece;
            for (int j = 0; j < kGroupRows; ++j) rows[(k + p) * kGroupRows + j] = kNoRow;
            kind[k + p] = kKindPiece + (uint32_t)(slot + p);
            len[k + p] = (uint32_t)(((left < piece ? left : piece) + kGroupRows - 1) / kGroupRows);
        }
        k += count;
        slot += count;
    }
    for (int i = threadIdx.x; i < n_long; i += kBlock) {
        const uint32_t r = mine[n_cut + i];
        rows[(k + i) * kGroupRows] = r | band_marks(band_count, n, r, band, n_bands);
        for (int j = 1; j < kGroupRows; ++j) rows[(k + i) * kGroupRows + j] = kNoRow;
        kind[k + i] = kKindLong;
        len[k + i] = (uint32_t)((rowptr[r + 1] - rowptr[r] + kGroupRows - 1) / kGroupRows);
    }
    k += n_long;
    const int padded = (n_short + kGroupRows - 1) / kGroupRows * kGroupRows;
    for (int i = threadIdx.x; i < padded; i += kBlock) {
        uint32_t r = kNoRow;
        if (i < n_short) {
            r = mine[n_cut + n_long + i];
            if (i % kGroupRows == 0) {  // the first row of a group is its longest
                kind[k + i / kGroupRows] = kKindShort;
                len[k + i / kGroupRows] = (uint32_t)(rowptr[r + 1] - rowptr[r]);
            }
            r |= band_marks(band_count, n, r, band, n_bands);
        }
        rows[k * kGroupRows + i] = r;
    }
}

// tab[i] = {first group that starts at batch kTabBatches * i or later, batch where it starts}
__global__ __launch_bounds__(kBlock) void group_table_kernel(const uint64_t* __restrict__ start,
                                                             int64_t n_groups, int64_t n_batches,
                                                             int64_t n_tab, uint2* __restrict__ tab,
                                                             uint32_t* __restrict__ rows)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k > n_groups) return;
    const int64_t b = k < n_groups ? (int64_t)start[k] : n_batches;
    const int64_t i0 = k == 0 ? 0 : (int64_t)start[k - 1] / kTabBatches + 1;
    const int64_t i1 = k < n_groups ? b / kTabBatches : n_tab - 1;
    for (int64_t i = i0; i <= i1; ++i) tab[i] = make_uint2((uint32_t)k, (uint32_t)b);
    if (k == n_groups)  // the padding stands for no rows
        for (int i = 0; i < kRowPad * kGroupRows; ++i) rows[k * kGroupRows + i] = kNoRow;
}

// ---- values ---------------------------------------------------------------------------------------

// One wavefront per group: computes the matrix values of its rows (rule of the normalisation mode,
// see entry_value) and writes them to the public array, to the entry-balanced form and, with the
// columns and the end marks, to the group's batches.  rowptr and src are those of the band: its entry
// `at` is entry src[at] of the matrix.  64 consecutive entries of the stream per step: the lane with
// position i of the step handles entry i / 8 of row i % 8 of a short group.
__global__ __launch_bounds__(kBlock) void fill_groups_kernel(
    const int64_t* __restrict__ rowptr, const uint32_t* __restrict__ col,
    const float* __restrict__ dinv, int mode, float eps, int swapped,
    const uint32_t* __restrict__ rows, const uint32_t* __restrict__ kind,
    const uint64_t* __restrict__ start, const uint32_t* __restrict__ cut_row,
    const uint64_t* __restrict__ piece0, int64_t n_cut, int64_t n_groups, int64_t n_batches,
    int64_t piece,
    const uint32_t* __restrict__ src,
    float* __restrict__ val, uint2* __restrict__ cv, uint2* __restrict__ ent)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t k = (int64_t)blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
    if (k >= n_groups) {
        if (k == n_groups)
            for (int i = lane; i < kStreamPad; i += kWave)
                ent[n_batches * kGroupRows + i] = make_uint2(0u, kPadValue);
        return;
    }
    const int64_t b0 = (int64_t)start[k];
    const int64_t b1 = k + 1 < n_groups ? (int64_t)start[k + 1] : n_batches;
    const uint32_t what = kind[k];
    const bool is_short = what == kKindShort, is_piece = what >= kKindPiece;
    uint32_t row = rows[k * kGroupRows + (is_short ? lane % kGroupRows : 0)] & kRowMask;
    int64_t skip = 0;
    if (is_piece) {  // of the last cut row whose pieces start at this slot or earlier
        const int64_t slot = what - kKindPiece;
        int64_t lo = 0, hi = n_cut;
        while (lo + 1 < hi) {
            const int64_t mid = (lo + hi) / 2;
            if ((int64_t)piece0[mid] <= slot) lo = mid;
            else hi = mid;
        }
        row = cut_row[lo] & kRowMask;
        skip = (slot - (int64_t)piece0[lo]) * piece;
    }
    int64_t e0 = 0, e1 = 0;
    if (row != kNoRow) {
        e0 = rowptr[row];
        e1 = rowptr[row + 1];
    }
    if (is_piece) {
        e0 += skip;
        if (e1 - e0 > piece) e1 = e0 + piece;
    }
    const float drow = (mode == MIXGCN_NORM_SUM || row == kNoRow) ? 0.f : dinv[row];
    const uint32_t end = is_piece ? kEndPiece : is_short ? kEndGroup : kEndRow;
    for (int64_t b = b0; b < b1; b += kWave / kGroupRows) {
        const int64_t bb = b + lane / kGroupRows;  // the lane's batch
        if (bb >= b1) break;
        const int64_t at = e0 + (is_short ? bb - b0 : (b - b0) * kGroupRows + lane);
        uint2 out = make_uint2(0u, kPadValue);
        if (at < e1) {
            const int64_t e = src[at];
            const uint32_t c = col[e];
            const float v = entry_value(mode, eps, swapped, row, c, drow, dinv);
            val[e] = v;
            cv[e].y = __float_as_uint(v);
            out = make_uint2(c, __float_as_uint(v));
        } else if (e1 > e0) {
            out.x = col[src[e1 - 1]];  // a line that has just been gathered
        }
        if (bb == b1 - 1 && lane % kGroupRows == 0) out.x |= end;
        ent[bb * kGroupRows + lane % kGroupRows] = out;
    }
}

// ---- aggregation ----------------------------------------------------------------------------------

constexpr int kVec = 4;         // columns per lane, 16 bytes
constexpr int kSliceLanes = 8;  // lanes of a slice
constexpr int kSliceColumns = kSliceLanes * kVec;
using F = Feat<MIXGCN_F32>;

// Closes a row, or what one band adds to it: between bands a row waits in Z.  zraw and mbits are what Z
// and the mask hold for the lane's columns, where they are wanted (kRowAdds, mask).
template <bool EPI>
__device__ inline void finish_row(float* t, void* Z, int64_t ldz, uint32_t row, int64_t c, int epi,
                                  const F::Raw& zraw, bool masked, uint32_t mbits, int c_lo, int c_hi)
{
    if (EPI) {
        if (row & kRowAdds) {
            float o[kVec];
            F::widen(zraw, o);
#pragma unroll
            for (int i = 0; i < kVec; ++i) t[i] += o[i];
        }
        if (!(row & kRowMore)) {
            if (epi & kEpiRelu) {
#pragma unroll
                for (int i = 0; i < kVec; ++i) t[i] = fmaxf(t[i], 0.f);
            }
            if (masked) {
#pragma unroll
                for (int i = 0; i < kVec; ++i) t[i] = ((mbits >> i) & 1u) ? t[i] : 0.f;
            }
        }
    }
    store_in_range<MIXGCN_F32>(Z, (int64_t)(row & kRowMask) * ldz, c, t, c_lo, c_hi);
}

// Eight lanes of 16 bytes hold a feature row's slice, one 128-byte line.
// The pipeline is that of the entry-balanced kernel: the entries of D gathers arrive with one
// coalesced load two rounds ahead and are handed out with lane shuffles, the feature rows are
// gathered one round (D loads) ahead, two rounds are written out per trip so that no register
// of a load in flight is copied, and the loop has no side exit.
// EPI: an epilogue other than a plain store is wanted.  OFF32: offsets into H fit 32 bits and
// column indices 24 bits.  D: gathers in flight per wavefront, a batch each, at 4 (D = 8) or 6 wavefronts per SIMD.
// In bands a row is read from Z before it is added to, and the gathers behind that read wait for it: eight of them
// outlast it, where there are enough wavefronts.  us, D = 4 : 8, 128 columns, entries per band: power law, 233 k nodes of
// 492, 13 M 3570 : 3440; 150 k of 200, 5 M 1022 : 994; uniform, 60 k of 300, 6 M 467 : 462; 100 k of 100, 2.5 M 351 : 360
// (at 256 columns 693 : 677), at 20 columns 111 : 126.
template <bool EPI, bool OFF32, int D>
__global__ __launch_bounds__(kBlock, D == 8 ? 4 : 6) void aggregate_groups_kernel(
    const uint2* __restrict__ ent, const uint32_t* __restrict__ rows,
    const uint32_t* __restrict__ kind, const uint2* __restrict__ tab, int64_t n_tab, int tab_per_wave, int64_t n_waves, const void* __restrict__ H, int64_t ldh,
    void* __restrict__ Z, int64_t ldz, int c0, int width, int n_slices,
    float* __restrict__ partials, int part_stride, int epi, const uint32_t* __restrict__ mask,
    int64_t ldm, int c_lo, int c_hi)
{
    constexpr int NC = 4;  // chains of a row's sum; batch b adds to chain b % 4
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane / kSliceLanes, lj = lane % kSliceLanes;
    // Workgroups are dealt round-robin to the 8 XCDs.  1, 2, 4 or 8 slices are dealt with them, so
    // that an XCD's L2 holds lines of one slice only; any other number is taken one after the other.
    const bool dealt = (n_slices & (n_slices - 1)) == 0;
    const unsigned per_slice = gridDim.x / (unsigned)n_slices;
    const int slice = (int)(dealt ? blockIdx.x % (unsigned)n_slices : blockIdx.x / per_slice);
    const unsigned block = dealt ? blockIdx.x / (unsigned)n_slices : blockIdx.x % per_slice;
    const int64_t w = uniform64((int64_t)block * (kBlock / kWave) + (threadIdx.x >> 6));
    if (w >= n_waves) return;
    const int64_t i0 = w * tab_per_wave;
    const int64_t i1 = i0 + tab_per_wave < n_tab ? i0 + tab_per_wave : n_tab - 1;
    const uint2 t0 = tab[i0], t1 = tab[i1];
    const int nb = uniform32((int)(t1.y - t0.y));  // batches of this wavefront
    if (nb == 0) return;
    int64_t k = (int64_t)(uint32_t)uniform32((int)t0.x);
    const int64_t b0 = (int64_t)(uint32_t)uniform32((int)t0.y);
    const int cs = slice * kSliceColumns;  // first column of the slice within the pass
    const bool active = cs + lj * kVec < width;
    const int64_t c = (int64_t)c0 + cs + lj * kVec;
    const int64_t c_load = active ? c : (int64_t)c0 + cs;  // idle lanes re-read the first column
    const uint32_t pitch = (uint32_t)(ldh * F::ES);
    const uint32_t lane_off = (uint32_t)(c_load * F::ES);
    const char* const hbase = reinterpret_cast<const char*>(H) + c_load * F::ES;

    float acc[NC][kVec];
#pragma unroll
    for (int u = 0; u < NC; ++u)
#pragma unroll
        for (int i = 0; i < kVec; ++i) acc[u][i] = 0.f;
    constexpr int RE = D * kGroupRows;  // entries per round
    static_assert(RE <= kWave, "a round's entries must fit one load per lane");
    const uint2* const rent = ent + b0 * kGroupRows + (lane & (RE - 1));
    uint32_t cw[D];
    uint32_t a[D];
    F::Raw h[D];
    auto fill = [&](int u, const uint2& en) __attribute__((always_inline)) {  // slot u <- gather u of the round `en`
        cw[u] = __shfl(en.x, u * kGroupRows + sub, kWave);
        a[u] = __shfl(en.y, u * kGroupRows + sub, kWave);
        if (OFF32)  // the 24-bit multiply ignores the marks
            h[u] = *reinterpret_cast<const F::Raw*>(
                reinterpret_cast<const char*>(H) + (__umul24(cw[u], pitch) + lane_off));
        else
            h[u] = *reinterpret_cast<const F::Raw*>(
                hbase + (uint64_t)(cw[u] & kEntryColMask) * pitch);
    };
    // The rows of eight groups at a time, a word per lane, and those of the next eight in flight;
    // `row` is the lane's row of the open group.  An epilogue that reads Z or a mask gets its words
    // when the group is opened, not when it ends.
    const uint32_t* row_words = rows + k * kGroupRows + lane;
    uint32_t rv = row_words[0], rv_next = row_words[kWave];
    int g = 0;  // group within the eight
    uint32_t row = kNoRow, mbits = 0;
    F::Raw zraw = {};
    auto open = [&]() __attribute__((always_inline)) {
        row = __shfl(rv, g * kGroupRows + sub, kWave);
        if (EPI && row != kNoRow && active) {
            const int64_t r = (int64_t)(row & kRowMask);
            if (row & kRowAdds) zraw = *F::ptr(Z, r * ldz + c);
            if (mask) mbits = mask[r * ldm + (c >> 5)] >> (c & 31);
        }
    };
    open();
    auto finish = [&](uint32_t end) __attribute__((always_inline)) {
        float t[kVec];
#pragma unroll
        for (int i = 0; i < kVec; ++i) t[i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
        if (end != kEndGroup) {
            reduce_subgroups<kSliceLanes, kVec>(t);
            if (end == kEndPiece && lane < kSliceLanes && active) {
                float* p = partials + (size_t)(kind[k] - kKindPiece) * part_stride + cs + lj * kVec;
#pragma unroll
                for (int i = 0; i < kVec; ++i) p[i] = t[i];
            }
        }
        if (row != kNoRow && active)
            finish_row<EPI>(t, Z, ldz, row, c, epi, zraw, mask != nullptr, mbits, c_lo, c_hi);
#pragma unroll
        for (int u = 0; u < NC; ++u)
#pragma unroll
            for (int i = 0; i < kVec; ++i) acc[u][i] = 0.f;
        ++k;
        if (++g == kGroupRows) {
            g = 0;
            rv = rv_next;
            row_words += kWave;
            rv_next = row_words[kWave];
        }
        open();
    };
    auto round = [&](int b, const uint2& en) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            float x[kVec];
            F::widen(h[u], x);
            const float av = __uint_as_float(a[u]);
            const bool real = a[u] != kPadValue;
            uint32_t end = (uint32_t)uniform32((int)cw[u]) & ~kEntryColMask;
            if (b + u >= nb) end = 0;  // a batch of the next wavefront
            if (real) {
#pragma unroll
                for (int i = 0; i < kVec; ++i) acc[u % NC][i] = fmaf(av, x[i], acc[u % NC][i]);
            }
            if (__builtin_expect(end != 0, 0)) finish(end);
            fill(u, en);
        }
    };
    uint2 ea = rent[0];
    uint2 eb = rent[RE];
#pragma unroll
    for (int u = 0; u < D; ++u) fill(u, ea);
    for (int b = 0; b < nb; b += 2 * D) {
        ea = rent[(int64_t)(b + 2 * D) * kGroupRows];
        round(b, eb);
        eb = rent[(int64_t)(b + 3 * D) * kGroupRows];
        round(b + D, ea);
    }
}

// Adds the pieces of the rows that were cut: one block per row, its lanes along the columns.
__global__ __launch_bounds__(kWave) void sum_pieces_kernel(
    const uint32_t* __restrict__ cut_row, const uint64_t* __restrict__ piece0, int64_t n_cut,
    int64_t n_pieces, void* __restrict__ Z, int64_t ldz, int c0, int width,
    const float* __restrict__ partials, int part_stride, int epi, const uint32_t* __restrict__ mask,
    int64_t ldm, int c_lo, int c_hi)
{
    const int64_t i = blockIdx.x;
    const int j = threadIdx.x * kVec;
    if (j >= width) return;
    const int64_t k0 = (int64_t)piece0[i], k1 = i + 1 < n_cut ? (int64_t)piece0[i + 1] : n_pieces;
    float t[kVec];
#pragma unroll
    for (int v = 0; v < kVec; ++v) t[v] = 0.f;
    const float4* p = reinterpret_cast<const float4*>(partials + (size_t)k0 * part_stride + j);
    const size_t step = (size_t)part_stride / 4;
    int64_t k = k0;
    for (; k + 8 <= k1; k += 8) {  // eight loads in flight, added in order
        float4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = p[u * step];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            t[0] += q[u].x; t[1] += q[u].y; t[2] += q[u].z; t[3] += q[u].w;
        }
        p += 8 * step;
    }
    for (; k < k1; ++k, p += step) {
        const float4 q = *p;
        t[0] += q.x; t[1] += q.y; t[2] += q.z; t[3] += q.w;
    }
    const uint32_t row = cut_row[i];
    const int64_t r = (int64_t)(row & kRowMask), c = (int64_t)c0 + j;
    F::Raw zraw = {};
    if (row & kRowAdds) zraw = *F::ptr(Z, r * ldz + c);
    const uint32_t mbits = mask ? mask[r * ldm + (c >> 5)] >> (c & 31) : 0;
    finish_row<true>(t, Z, ldz, row, c, epi, zraw, mask != nullptr, mbits, c_lo, c_hi);
}

template <typename T>
int dmalloc(T** p, size_t count, hipStream_t s)
{
    return pool_alloc((void**)p, (count ? count : 1) * sizeof(T), s);
}

// Work arrays of one call, released on its stream.
struct Tmp {
    explicit Tmp(hipStream_t stream) : s(stream) {}
    hipStream_t s;
    uint64_t* keys = nullptr;
    uint64_t* alt = nullptr;
    void* sort = nullptr;
    unsigned long long* hist = nullptr;
    uint32_t* sorted = nullptr;
    uint2* long_short = nullptr;
    WindowPlan* plan = nullptr;
    WindowStart* start = nullptr;
    uint32_t* len = nullptr;
    uint32_t* count = nullptr;
    uint64_t* pos = nullptr;
    uint8_t* band = nullptr;
    ~Tmp()
    {
        pool_free_on(keys, s);
        pool_free_on(alt, s);
        pool_free_on(sort, s);
        pool_free_on(hist, s);
        pool_free_on(sorted, s);
        pool_free_on(long_short, s);
        pool_free_on(plan, s);
        pool_free_on(start, s);
        pool_free_on(len, s);
        pool_free_on(count, s);
        pool_free_on(pos, s);
        pool_free_on(band, s);
    }
};

inline unsigned blocks(int64_t threads) { return (unsigned)ceil_div(threads, kBlock); }

}  // namespace

void rowgroups_free(RowGroups* g)
{
    for (Band& b : g->bands) {
        pool_free(b.ent);
        pool_free(b.ent_t);
        pool_free(b.rows);
        pool_free(b.kind);
        pool_free(b.start);
        pool_free(b.tab);
        pool_free(b.cut_row);
        pool_free(b.piece0);
        pool_free(b.rowptr);
    }
    pool_free(g->src);
    *g = RowGroups();
}

// Streams for the values of the transpose, all or none: without memory for them its aggregations take
// the entry-balanced kernel.
int rowgroups_alloc_transpose(RowGroups* g, hipStream_t s)
{
    if (g->bands.empty() || g->bands.back().ent_t) return MIXGCN_OK;
    int rc = MIXGCN_OK;
    for (Band& b : g->bands)
        if (rc == MIXGCN_OK)
            rc = pool_alloc_async((void**)&b.ent_t, ((size_t)b.n_batches * kGroupRows + kStreamPad) * sizeof(uint2), s);
    if (rc == MIXGCN_OK) return rc;
    for (Band& b : g->bands) {
        pool_free_on(b.ent_t, s);  // nothing has used them
        b.ent_t = nullptr;
    }
    if (rc == MIXGCN_ENOMEM) (void)hipGetLastError();
    return rc == MIXGCN_ENOMEM ? MIXGCN_OK : rc;
}

namespace {

// Groups of one band, whose rows are given by rowptr.
int build_band(const int64_t* rowptr, uint32_t n, int64_t nnz, const uint32_t* band_count, int band,
               int n_bands, Band* out, hipStream_t s)
{
    Band& g = *out;
    // Pieces of 256 entries and groups of at most 32 batches keep the longest wavefront of a small
    // graph short; on large ones 1024 keep the number of slots low, and groups of up to 64 batches
    // the padding of the rows that do not fill whole batches of their own.
    const bool small = nnz < (4ll << 20);
    g.piece = small ? 256 : 1024;
    const int short_row = small ? 32 : kMostShort;
    const int64_t n_windows = ceil_div(n, kWindow);
    Tmp t(s);
    MIXGCN_TRY(dmalloc(&t.sorted, n, s));
    MIXGCN_TRY(dmalloc(&t.long_short, (size_t)n_windows, s));
    MIXGCN_TRY(dmalloc(&t.plan, (size_t)n_windows, s));
    MIXGCN_TRY(dmalloc(&t.start, (size_t)n_windows + 1, s));
    hipLaunchKernelGGL(window_sort_kernel, dim3((unsigned)n_windows), dim3(kBlock), 0, s, rowptr, n, g.piece,
                       short_row, t.sorted, t.long_short, t.plan);
    hipLaunchKernelGGL(window_scan_kernel, dim3(1), dim3(kBlock), 0, s, t.plan, n_windows, t.start);
    WindowStart h;
    MIXGCN_HIP_TRY(hipMemcpyAsync(&h, t.start + n_windows, sizeof(h), hipMemcpyDeviceToHost, s));
    MIXGCN_HIP_TRY(hipStreamSynchronize(s));
    g.n_cut = (int64_t)h.cut;
    g.n_pieces = (int64_t)h.pieces;
    g.n_groups = (int64_t)h.groups;
    g.n_batches = (int64_t)h.batches;
    g.n_tab = g.n_batches / kTabBatches + 2;

    MIXGCN_TRY(pool_alloc(&t.sort, scan_tmp_bytes(g.n_groups), s));
    MIXGCN_TRY(dmalloc(&t.len, (size_t)g.n_groups, s));
    MIXGCN_TRY(dmalloc(&g.rows, (size_t)(g.n_groups + kRowPad) * kGroupRows, s));
    MIXGCN_TRY(dmalloc(&g.kind, (size_t)g.n_groups, s));
    MIXGCN_TRY(dmalloc(&g.start, (size_t)g.n_groups, s));
    MIXGCN_TRY(dmalloc(&g.tab, (size_t)g.n_tab, s));
    MIXGCN_TRY(dmalloc(&g.cut_row, (size_t)g.n_cut, s));
    MIXGCN_TRY(dmalloc(&g.piece0, (size_t)g.n_cut, s));
    MIXGCN_TRY(dmalloc(&g.ent, (size_t)g.n_batches * kGroupRows + kStreamPad, s));
    hipLaunchKernelGGL(window_groups_kernel, dim3((unsigned)n_windows), dim3(kBlock), 0, s, rowptr, t.sorted,
                       t.long_short, t.start, g.piece, band_count, (int64_t)n, band, n_bands, g.rows, g.kind,
                       t.len, g.cut_row, g.piece0);
    MIXGCN_TRY(exclusive_scan_u32_to_u64(t.len, g.start, g.n_groups, nullptr, t.sort, s));
    hipLaunchKernelGGL(group_table_kernel, dim3(blocks(g.n_groups + 1)), dim3(kBlock), 0, s, g.start,
                       g.n_groups, g.n_batches, g.n_tab, g.tab, g.rows);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

// Host copy of the popularity histogram, and an event behind it.
struct HostHist {
    unsigned long long* p = nullptr;
    hipEvent_t ev = nullptr;
    int copy(const unsigned long long* d, hipStream_t s)
    {
        MIXGCN_TRY(host_alloc((void**)&p, 2 * kBins * sizeof(*p)));
        MIXGCN_HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        MIXGCN_HIP_TRY(hipMemcpyAsync(p, d, 2 * kBins * sizeof(*p), hipMemcpyDeviceToHost, s));
        MIXGCN_HIP_TRY(hipEventRecord(ev, s));
        queued = true;
        return MIXGCN_OK;
    }
    int wait()
    {
        MIXGCN_HIP_TRY(hipEventSynchronize(ev));
        queued = false;
        return MIXGCN_OK;
    }
    bool queued = false;
    ~HostHist()
    {
        if (queued) (void)hipEventSynchronize(ev);
        if (ev) (void)hipEventDestroy(ev);
        host_free(p);
    }
};

int build_bands(const Csr& m, uint32_t n, RowGroups* out, hipStream_t s)
{
    Tmp t(s);
    uint64_t* sorted = nullptr;
    MIXGCN_TRY(dmalloc(&t.keys, n, s));
    MIXGCN_TRY(dmalloc(&t.hist, 2 * kBins, s));
    MIXGCN_HIP_TRY(hipMemsetAsync(t.hist, 0, 2 * kBins * sizeof(unsigned long long), s));
    hipLaunchKernelGGL(popularity_kernel, dim3(blocks(n) < 512u ? blocks(n) : 512u), dim3(kBlock), 0, s,
                       m.rowptr, n, t.keys, t.hist, t.hist + kBins);
    // the row pointers are on their way to the host while the bands are planned
    HostHist h;
    MIXGCN_TRY(h.copy(t.hist, s));
    MIXGCN_TRY(csr_copy_rowptr(m, n, s));
    MIXGCN_TRY(h.wait());
    const int n_bands = plan_bands(h.p, h.p + kBins, (double)n, (double)m.nnz, out);
    if (n_bands == 1) return MIXGCN_OK;
    out->bands.resize((size_t)n_bands);

    size_t tmp_bytes = sort_tmp_bytes(n);
    const int64_t counts = (int64_t)n_bands * n;
    if (scan_tmp_bytes(counts) > tmp_bytes) tmp_bytes = scan_tmp_bytes(counts);
    MIXGCN_TRY(dmalloc(&t.alt, n, s));
    MIXGCN_TRY(pool_alloc(&t.sort, tmp_bytes, s));
    MIXGCN_TRY(dmalloc(&t.band, n, s));
    MIXGCN_TRY(dmalloc(&t.count, (size_t)counts, s));
    MIXGCN_TRY(dmalloc(&t.pos, (size_t)counts, s));
    MIXGCN_TRY(dmalloc(&out->src, (size_t)m.nnz, s));
    MIXGCN_TRY(radix_sort_u64(t.keys, t.alt, n, 8, &sorted, t.sort, s));
    uint32_t per_band = kBandColumns;
    if ((int64_t)n_bands * kBandColumns >= n) per_band = (uint32_t)ceil_div(n, n_bands);
    hipLaunchKernelGGL(band_of_column_kernel, dim3(blocks(n)), dim3(kBlock), 0, s, sorted, n, per_band,
                       n_bands, t.band);
    const dim3 grid((unsigned)ceil_div(n, kBlock / kWave));
    hipLaunchKernelGGL(deal_entries_kernel<false>, grid, dim3(kBlock), 0, s, m.rowptr, m.col, t.band, n,
                       n_bands, t.count, (const uint64_t*)nullptr, (uint32_t*)nullptr);
    MIXGCN_TRY(exclusive_scan_u32_to_u64(t.count, t.pos, counts, nullptr, t.sort, s));
    hipLaunchKernelGGL(deal_entries_kernel<true>, grid, dim3(kBlock), 0, s, m.rowptr, m.col, t.band, n,
                       n_bands, (uint32_t*)nullptr, t.pos, out->src);
    std::vector<uint64_t> first((size_t)n_bands + 1);
    for (int b = 0; b < n_bands; ++b)
        MIXGCN_HIP_TRY(hipMemcpyAsync(&first[(size_t)b], t.pos + (int64_t)b * n, 8, hipMemcpyDeviceToHost, s));
    MIXGCN_HIP_TRY(hipStreamSynchronize(s));
    first[(size_t)n_bands] = (uint64_t)m.nnz;
    for (int b = 0; b < n_bands; ++b) {
        Band& band = out->bands[(size_t)b];
        band.src0 = (int64_t)first[(size_t)b];
        MIXGCN_TRY(dmalloc(&band.rowptr, (size_t)n + 1, s));
        hipLaunchKernelGGL(band_rowptr_kernel, dim3(blocks((int64_t)n + 1)), dim3(kBlock), 0, s, t.pos,
                           (int64_t)n, b, n_bands, m.nnz, band.rowptr);
        MIXGCN_TRY(build_band(band.rowptr, n, (int64_t)first[(size_t)b + 1] - band.src0, t.count, b, n_bands,
                              &band, s));
    }
    return MIXGCN_OK;
}

}  // namespace

bool rowgroups_planned(uint32_t n, int64_t nnz)
{
    return n > (uint32_t)kBandColumns && n < kRowMask && nnz >= 2 * kBandRow * (int64_t)n && nnz <= kMostEntries;
}

// The bands and groups of a matrix with a symmetric pattern (row lengths are then the popularities of
// the columns): everything that depends on the pattern only.  None where they cannot pay, and where
// there is no memory for them.  Where they are planned it copies the row pointers to the host meanwhile, and waits for
// the stream.
int rowgroups_build(const Csr& m, uint32_t n, RowGroups* out, hipStream_t s)
{
    if (!rowgroups_planned(n, m.nnz)) return MIXGCN_OK;
    RowGroups g;
    int rc = build_bands(m, n, &g, s);
    if (rc == MIXGCN_OK && hipStreamSynchronize(s) != hipSuccess) rc = fail(MIXGCN_EHIP, "bands of the columns");
    if (rc != MIXGCN_OK) {
        (void)hipStreamSynchronize(s);  // the arrays may have work queued on them
        rowgroups_free(&g);
        if (rc != MIXGCN_ENOMEM) return rc;
        (void)hipGetLastError();
        MIXGCN_TRY(csr_copy_rowptr(m, n, s));  // (it may have been queued or not)
        MIXGCN_HIP_TRY(hipStreamSynchronize(s));
        return MIXGCN_OK;
    }
    *out = std::move(g);
    return MIXGCN_OK;
}

// Values of the matrix (mode, eps; transposed: those of its transpose on the same pattern, into
// ent_t) into val, the value words of cv, and the streams.
int rowgroups_fill(const Csr& m, const RowGroups& g, const float* dinv, int mode, float eps,
                   int swapped, bool transposed, float* val, uint2* cv, hipStream_t s)
{
    for (const Band& b : g.bands)
        hipLaunchKernelGGL(fill_groups_kernel, dim3((unsigned)ceil_div(b.n_groups + 1, kBlock / kWave)),
                           dim3(kBlock), 0, s, b.rowptr, m.col, dinv, mode, eps,
                           swapped, b.rows, b.kind, b.start, b.cut_row, b.piece0, b.n_cut, b.n_groups,
                           b.n_batches, b.piece, g.src + b.src0, val, cv,
                           transposed ? b.ent_t : b.ent);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

namespace {

int launch_groups(const Band& g, const uint2* ent, int64_t n_nodes, const void* H, int64_t ldh,
                  void* Z, int64_t ldz, int c0, int width, float* P, int part_stride, int epi,
                  const uint32_t* mask, int64_t ldm, int c_lo, int c_hi, hipStream_t s, Timer* timer,
                  int timer_kind, bool epilogue)
{
    if (g.n_batches == 0) return MIXGCN_OK;
    const int n_slices = (int)ceil_div(width, kSliceColumns);
    // A wavefront walks up to 1024 batches: its start is four dependent loads.  Half, a quarter .. of
    // that, down to 256, until the chip's 8192 wavefronts are filled seven times over (a last partial
    // filling then costs little); on small inputs further, until they are filled once.
    int per_wave = 1024 / kTabBatches;
    while (per_wave > 1) {
        const int64_t waves = ceil_div(g.n_tab, per_wave) * n_slices;
        if (waves >= (per_wave > 256 / kTabBatches ? 7 * 8192 : 8192)) break;
        per_wave /= 2;
    }
    const int64_t n_waves = ceil_div(g.n_tab - 1, per_wave);
    const int64_t grid = ceil_div(n_waves, kBlock / kWave) * n_slices;
    if (grid > 0x7FFFFFFF) return fail(MIXGCN_EINVAL, "aggregate: grid too large");
    const bool off32 = n_nodes * ldh * F::ES + (int64_t)(c0 + width) * F::ES < (1ll << 32) &&
                       ldh * F::ES < (1ll << 24) && n_nodes <= (1ll << 24);
    if (timer) MIXGCN_TRY(timer->begin(timer_kind, s));
    // the sums do not depend on D (see there)
    const bool deep = g.n_batches * n_slices >= 2400000;
#define MIXGCN_GROUPS_D(EPI, O32, D)                                                              \
    hipLaunchKernelGGL((aggregate_groups_kernel<EPI, O32, D>), dim3((unsigned)grid), dim3(kBlock), 0, s, \
                       ent, g.rows, g.kind, g.tab, g.n_tab, per_wave, n_waves, H, ldh, Z, ldz, c0, width, \
                       n_slices, P, part_stride, epi, mask, ldm, c_lo, c_hi)
#define MIXGCN_GROUPS(EPI, O32)              \
    do {                                     \
        if (deep) MIXGCN_GROUPS_D(EPI, O32, 8); \
        else MIXGCN_GROUPS_D(EPI, O32, 4);   \
    } while (0)
    if (epilogue) {
        if (off32) MIXGCN_GROUPS(true, true);
        else MIXGCN_GROUPS(true, false);
    } else {
        if (off32) MIXGCN_GROUPS(false, true);
        else MIXGCN_GROUPS(false, false);
    }
#undef MIXGCN_GROUPS
#undef MIXGCN_GROUPS_D
    if (timer) MIXGCN_TRY(timer->end(s));
    if (g.n_cut > 0)
        hipLaunchKernelGGL(sum_pieces_kernel, dim3((unsigned)g.n_cut), dim3(kWave), 0, s, g.cut_row, g.piece0,
                           g.n_cut, g.n_pieces, Z, ldz, c0, width, P, part_stride, epi, mask, ldm, c_lo,
                           c_hi);
    return MIXGCN_OK;
}

// Columns of a slot: the pass, rounded up to whole slices.
inline int slot_columns(int width) { return (int)ceil_div(width, kSliceColumns) * kSliceColumns; }

// Bytes of scratch of a pass: the slots of the pieces.
size_t pieces_scratch(const RowGroups& g, int width)
{
    int64_t slots = 0;
    for (const Band& b : g.bands) slots = b.n_pieces > slots ? b.n_pieces : slots;
    return (size_t)slots * slot_columns(width) * sizeof(float);
}

}  // namespace

// Whether a pass over all n rows takes the bands: they are there, for the values at hand too, and
//  - the pass is fp32.  bf16 rows would have to wait in fp32 between bands, in scratch of 1 KB per row,
//    which cost 1.3 times the bands of fp32;
//  - its rows are longer than 64 bytes.  Shorter ones leave half of a band's L2 empty and miss less
//    with the columns in one band, as two share a line (uniform columns, 60 k nodes, 300 per row: 107
//    us at 8 columns, in bands 137; power law, 120 k nodes, 300 per row, 16 columns: 342 and 347);
//  - a matrix of rows of up to one line does not nearly fit an L2 (uniform columns, 300 per row, 20
//    columns: 45 k nodes 122 us, in bands 134; 60 k 178 and 183; 80 k 289 and 249);
//  - there is enough of it to pay for a launch of its own per band, 10 us or 0.55 M lines with what the
//    last wavefronts leave idle (uniform columns, 45 k nodes, 80 per row, 2 bands: 49 us at 20 columns,
//    in bands 60; 145 and 146 at 128);
//  - the pieces need no more scratch than the entry-balanced kernel would, so that every caller's scratch
//    holds them.  Nothing here depends on the caller: the same call gives the same bits whatever
//    scratch it brings.
bool rowgroups_take(const RowGroups& g, int64_t n, int64_t nnz, bool values_t, int dtype, int width,
                    size_t scratch_need)
{
    if (g.bands.empty() || dtype != MIXGCN_F32 || (values_t && !g.bands.back().ent_t)) return false;
    if (width <= 16 || (width <= kSliceColumns && n * width * F::ES < (6 << 20))) return false;
    const double lines = (double)nnz * (double)ceil_div(width, kSliceColumns);
    if (g.cost + 0.55e6 * (double)(g.bands.size() - 1) / lines >= g.most_cost) return false;
    return pieces_scratch(g, width) <= scratch_need;
}

int launch_groups_pass(const RowGroups& g, bool values_t, int64_t n_nodes, const void* H, int64_t ldh,
                       void* Z, int64_t ldz, int c0, int width, float* P, int epi, const uint32_t* mask,
                       int64_t ldm, int c_lo, int c_hi, hipStream_t s, Timer* timer, int timer_kind)
{
    for (size_t i = 0; i < g.bands.size(); ++i) {
        const Band& b = g.bands[i];
        const uint2* ent = values_t ? b.ent_t : b.ent;
        // without an epilogue of its own the rows of the first band are plain stores
        const bool epilogue = epi || mask || i > 0;
        MIXGCN_TRY(launch_groups(b, ent, n_nodes, H, ldh, Z, ldz, c0, width, P, slot_columns(width), epi,
                                 mask, ldm, c_lo, c_hi, s, timer, timer_kind, epilogue));
    }
    return MIXGCN_OK;
}

}  // namespace mixgcn
