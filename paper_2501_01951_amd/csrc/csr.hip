// CSR construction of A_tilde = A + I from an edge list (paper Sec. 2.1) and the symmetric
// normalisation A_hat = D^-1/2 A_tilde D^-1/2.  Integer work: key emission, radix sort,
// duplicate removal by a tiled compaction, row pointers, per-group start rows.
#include "device_utils.h"
#include "internal.h"

namespace mixgcn {
namespace {

constexpr int kCompactItems = 8;
constexpr int kCompactTile = kBlock * kCompactItems;

// key = row << bits | col; self edges become the diagonal key when the diagonal is added anyway
// (the duplicate is removed later), otherwise the drop marker 1 << 2*bits, which sorts last.
__global__ __launch_bounds__(kBlock) void emit_keys_kernel(
    const uint32_t* __restrict__ src, const uint32_t* __restrict__ dst, uint64_t n_edges,
    uint32_t n, int bits, int symmetrize, int self_loops, int transposed,
    uint64_t* __restrict__ keys, uint32_t* __restrict__ err)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t drop = 1ull << (2 * bits);
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_edges; i += stride) {
        uint64_t u = src[i], v = dst[i];
        uint64_t k1, k2;
        if (u >= n || v >= n) {
            atomicOr(err, 1u);
            k1 = k2 = drop;
        } else if (u == v) {
            k1 = k2 = self_loops ? ((u << bits) | u) : drop;
        } else {
            if (transposed) { uint64_t t = u; u = v; v = t; }
            k1 = (u << bits) | v;
            k2 = (v << bits) | u;
        }
        keys[i] = k1;
        if (symmetrize) keys[n_edges + i] = k2;
    }
    if (self_loops) {
        const uint64_t base = (symmetrize ? 2 : 1) * n_edges;
        for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += stride)
            keys[base + u] = (u << bits) | u;
    }
}

// Keys of a wavefront for the removal of duplicates: kCompactItems * 64 consecutive ones, 64 at a time,
// with their neighbors on both sides (kNoKey past the ends).
constexpr uint64_t kNoKey = ~0ull;
struct WaveKeys {
    uint64_t key[kCompactItems];
    uint64_t prev[kCompactItems];
    uint64_t first[kCompactItems];  // lanes that hold the first key of a run of equal ones
    uint32_t count;                 // runs that start here
};

__device__ inline void load_wave_keys(const uint64_t* __restrict__ keys, int64_t n_keys, uint64_t drop,
                                      int64_t base, int lane, WaveKeys& k)
{
#pragma unroll
    for (int j = 0; j < kCompactItems; ++j) {
        const int64_t i = base + j * kWave + lane;
        k.key[j] = i < n_keys ? keys[i] : kNoKey;
    }
    uint64_t before = base > 0 && base <= n_keys ? keys[base - 1] : kNoKey;
    k.count = 0;
#pragma unroll
    for (int j = 0; j < kCompactItems; ++j) {
        const uint64_t left = __shfl_up((unsigned long long)k.key[j], 1, kWave);
        k.prev[j] = lane == 0 ? before : left;
        before = __shfl((unsigned long long)k.key[j], kWave - 1, kWave);
        k.first[j] = __ballot(k.key[j] < drop && k.key[j] != k.prev[j]);
        k.count += (uint32_t)__popcll(k.first[j]);
    }
}

__global__ __launch_bounds__(kBlock) void unique_count_kernel(const uint64_t* __restrict__ keys,
                                                              int64_t n_keys, uint64_t drop,
                                                              uint32_t* __restrict__ tile_cnt)
{
    __shared__ uint32_t count[kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
    WaveKeys k;
    load_wave_keys(keys, n_keys, drop, (int64_t)blockIdx.x * kCompactTile + w * kCompactItems * kWave,
                   lane, k);
    if (lane == 0) count[w] = k.count;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int i = 0; i < kBlock / kWave; ++i) total += count[i];
        tile_cnt[blockIdx.x] = total;
    }
}

__global__ __launch_bounds__(kBlock) void fill_i64_kernel(int64_t* p, int64_t n, int64_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Writes col/cv for every distinct key, with the mark of the last entry of a row, and rowptr[q] =
// (index of the first entry with row >= q) for every q up to the last non-empty row; later rows
// keep the preset value nnz.  Reports empty rows.  Bound by memory.  Consecutive lanes take consecutive
// keys: 33.5 M keys 0.13 ms (with eight keys per lane and the marks in a pass of their own 0.70).
__global__ __launch_bounds__(kBlock) void unique_fill_kernel(
    const uint64_t* __restrict__ keys, int64_t n_keys, uint64_t drop, int bits, uint32_t n,
    const uint64_t* __restrict__ tile_off, uint32_t* __restrict__ col,
    uint2* __restrict__ cv, int64_t* __restrict__ rowptr, uint32_t* __restrict__ any_empty)
{
    __shared__ uint32_t count[kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * kCompactTile + w * kCompactItems * kWave;
    WaveKeys k;
    load_wave_keys(keys, n_keys, drop, base, lane, k);
    const int64_t after = base + kCompactItems * kWave;
    uint64_t next_step = after < n_keys ? keys[after] : kNoKey;  // the key behind the last step
    if (lane == 0) count[w] = k.count;
    __syncthreads();
    uint64_t pos = tile_off[blockIdx.x];  // runs that start before the wave's keys
    for (int i = 0; i < w; ++i) pos += count[i];
    const uint64_t cmask = (1ull << bits) - 1;
    const uint64_t upto = ~0ull >> (kWave - 1 - lane);  // this lane and those before it
#pragma unroll
    for (int j = 0; j < kCompactItems; ++j) {
        const uint64_t key = k.key[j];
        const uint64_t right = __shfl_down((unsigned long long)key, 1, kWave);
        const uint64_t behind =
            j + 1 < kCompactItems ? __shfl((unsigned long long)k.key[j + 1 < kCompactItems ? j + 1 : j], 0, kWave)
                                  : next_step;
        const uint64_t next = lane == kWave - 1 ? behind : right;
        if (key < drop) {
            const int64_t row = (int64_t)(key >> bits);
            const uint64_t at = pos + __popcll(k.first[j] & upto) - 1;  // index of the key's run
            if ((k.first[j] >> lane) & 1) {
                const int64_t prev = k.prev[j] == kNoKey ? -1 : (int64_t)(k.prev[j] >> bits);
                for (int64_t q = prev + 1; q <= row; ++q) rowptr[q] = (int64_t)at;
                if (row > prev + 1) *any_empty = 1u;
            }
            if (key != next) {  // the last key of the run writes the entry
                const bool last = next >= drop || (int64_t)(next >> bits) != row;
                const uint32_t c = (uint32_t)(key & cmask);
                col[at] = c;
                cv[at] = make_uint2(last ? c | kEntryEndBit : c, 0u);
                if (next >= drop && row + 1 < (int64_t)n) *any_empty = 1u;
            }
        }
        pos += __popcll(k.first[j]);
    }
}

// grp_row[g] = the row that holds stored entry g * kGroupNnz (last row with rowptr <= that).
__global__ __launch_bounds__(kBlock) void group_rows_kernel(const int64_t* __restrict__ rowptr,
                                                            uint32_t n, int64_t nnz,
                                                            int64_t n_groups,
                                                            uint32_t* __restrict__ grp_row)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g > n_groups) return;
    const int64_t e = g * kGroupNnz;
    if (e >= nnz) {
        grp_row[g] = n ? n - 1 : 0;
        return;
    }
    // upper_bound(rowptr[0..n], e) - 1
    int64_t lo = 0, hi = (int64_t)n + 1;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (rowptr[mid] <= e) lo = mid + 1;
        else hi = mid;
    }
    grp_row[g] = (uint32_t)(lo - 1);
}

// Row sums of the binary matrix and the scaling vector of the mode: D^-1/2 (symmetric), D^-1
// (mean), unused (sum).
__global__ __launch_bounds__(kBlock) void degree_kernel(const int64_t* __restrict__ rowptr,
                                                        uint32_t n, int mode,
                                                        uint32_t* __restrict__ deg,
                                                        float* __restrict__ dinv)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const uint32_t d = (uint32_t)(rowptr[r + 1] - rowptr[r]);
    deg[r] = d;
    if (mode == MIXGCN_NORM_MEAN) dinv[r] = d ? (float)(1.0 / (double)d) : 0.0f;
    else dinv[r] = d ? (float)(1.0 / sqrt((double)d)) : 0.0f;
}

// One thread per stored entry, a block per group of kGroupNnz: the row of an entry is one of those that the group
// covers, so the search starts from a handful of row pointers that the block has in its L1 (over all of them it took
// most of the time).  Four groups per block, so that the columns and scales of four entries are on their way together.
// What is left are the gathers of dinv.  33.0 M entries of 2^20 rows: 656 -> 225 us; without the hints, with which the
// streams leave the L2s to dinv, 279.
constexpr int kValueGroups = 4;
static_assert(kGroupNnz == kBlock, "a thread per entry of a group");
__global__ __launch_bounds__(kBlock) void values_kernel(const int64_t* __restrict__ rowptr,
                                                        const uint32_t* __restrict__ grp_row,
                                                        const uint32_t* __restrict__ col,
                                                        const float* __restrict__ dinv,
                                                        int64_t n_groups, int64_t nnz, int mode,
                                                        float eps, int swapped,
                                                        float* __restrict__ val,
                                                        uint2* __restrict__ cv)
{
    const int64_t g0 = (int64_t)blockIdx.x * kValueGroups;
    uint32_t c[kValueGroups], row[kValueGroups];
#pragma unroll
    for (int j = 0; j < kValueGroups; ++j) {
        const int64_t e = (g0 + j) * kGroupNnz + threadIdx.x;
        c[j] = __builtin_nontemporal_load(col + (e < nnz ? e : nnz - 1));
    }
#pragma unroll
    for (int j = 0; j < kValueGroups; ++j) {
        const int64_t g = g0 + j < n_groups ? g0 + j : n_groups - 1;
        int64_t e = g * kGroupNnz + threadIdx.x;
        if (e >= nnz) e = nnz - 1;
        // the last row in [lo, hi] with rowptr <= e (rowptr[lo] <= e: the row of the group's first entry)
        uint32_t lo = grp_row[g], hi = grp_row[g + 1];
        while (lo < hi) {
            const uint32_t mid = hi - (hi - lo) / 2;
            if (rowptr[mid] <= e) lo = mid;
            else hi = mid - 1;
        }
        row[j] = lo;
    }
#pragma unroll
    for (int j = 0; j < kValueGroups; ++j) {
        const int64_t e = (g0 + j) * kGroupNnz + threadIdx.x;
        if (e >= nnz) continue;
        const float drow = mode == MIXGCN_NORM_SUM ? 0.f : dinv[row[j]];
        const float v = entry_value(mode, eps, swapped, row[j], c[j], drow, dinv);
        __builtin_nontemporal_store(v, val + e);
        __builtin_nontemporal_store(__float_as_uint(v), &cv[e].y);
    }
}

// cv_t = cv with the value words left for values_kernel to fill (same columns and row marks)
__global__ __launch_bounds__(kBlock) void copy_entries_kernel(const uint2* __restrict__ in,
                                                              uint2* __restrict__ out, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) out[i] = in[i];
}

template <typename T>
int dmalloc(T** p, size_t count, hipStream_t s)
{
    return pool_alloc((void**)p, (count ? count : 1) * sizeof(T), s);
}

template <typename T>
int dmalloc_async(T** p, size_t count, hipStream_t s)
{
    return pool_alloc_async((void**)p, (count ? count : 1) * sizeof(T), s);
}

// Work arrays of a build, released on its stream.
struct TmpBufs {
    explicit TmpBufs(hipStream_t stream) : s(stream) {}
    hipStream_t s;
    uint64_t* keys = nullptr;
    uint64_t* alt = nullptr;
    void* tmp = nullptr;
    uint32_t* flags = nullptr;
    ~TmpBufs()
    {
        pool_free_on(keys, s);
        pool_free_on(alt, s);
        pool_free_on(tmp, s);
        pool_free_on(flags, s);
    }
};

}  // namespace

void csr_free(Csr* c)
{
    pool_free(c->rowptr);
    pool_free(c->col);
    pool_free(c->cv);
    pool_free(c->val);
    pool_free(c->cv_t);
    pool_free(c->val_t);
    pool_free(c->grp_row);
    host_free(c->h_rowptr);
    rowgroups_free(&c->groups);
    *c = Csr();
}

int csr_copy_rowptr(const Csr& c, uint32_t n, hipStream_t s)
{
    MIXGCN_HIP_TRY(hipMemcpyAsync(c.h_rowptr, c.rowptr, ((size_t)n + 1) * 8, hipMemcpyDeviceToHost, s));
    return MIXGCN_OK;
}

// The row pointers are copied to the host behind the last kernel, with the wait that is there anyway (a wait of its own
// made a build of 10 k nodes 12 to 18 us longer, of 200), unless bands are planned next: then csr_copy_rowptr is still to
// be called.
int csr_from_edges(const uint32_t* d_src, const uint32_t* d_dst, uint64_t n_edges, uint32_t n,
                   bool symmetrize, bool self_loops, bool transposed, Csr* out, hipStream_t s)
{
    int bits = 1;
    while ((1ull << bits) < (uint64_t)n) ++bits;
    const uint64_t drop = 1ull << (2 * bits);
    const int sort_bits = 2 * bits + (self_loops ? 0 : 1);  // the drop marker needs one more bit
    const int64_t n_keys = (int64_t)((symmetrize ? 2 : 1) * n_edges + (self_loops ? n : 0));

    TmpBufs t(s);
    MIXGCN_TRY(dmalloc(&t.keys, (size_t)n_keys, s));
    MIXGCN_TRY(dmalloc(&t.alt, (size_t)n_keys, s));
    const int64_t n_ctiles = ceil_div(n_keys > 0 ? n_keys : 1, kCompactTile);
    size_t tmp_bytes = sort_tmp_bytes(n_keys);
    const size_t compact_bytes =
        ((size_t)n_ctiles * 4 + 255) / 256 * 256 + ((size_t)n_ctiles * 8 + 255) / 256 * 256 +
        scan_tmp_bytes(n_ctiles) + 256;
    if (compact_bytes > tmp_bytes) tmp_bytes = compact_bytes;
    MIXGCN_TRY(pool_alloc(&t.tmp, tmp_bytes, s));
    MIXGCN_TRY(dmalloc(&t.flags, 4, s));  // [0] bad endpoint, [1] empty rows, [2..3] total (u64)
    MIXGCN_HIP_TRY(hipMemsetAsync(t.flags, 0, 16, s));

    if (n_keys > 0) {
        const uint64_t work = n_edges > n ? n_edges : n;
        unsigned grid = (unsigned)((work + kBlock - 1) / kBlock);
        if (grid > 65536u) grid = 65536u;
        if (grid == 0) grid = 1;
        hipLaunchKernelGGL(emit_keys_kernel, dim3(grid), dim3(kBlock), 0, s, d_src, d_dst, n_edges,
                           n, bits, symmetrize ? 1 : 0, self_loops ? 1 : 0, transposed ? 1 : 0,
                           t.keys, t.flags);
    }
    uint64_t* sorted = t.keys;
    MIXGCN_TRY(radix_sort_u64(t.keys, t.alt, n_keys, sort_bits, &sorted, t.tmp, s));

    // distinct keys per tile -> tile offsets and nnz
    char* p = (char*)t.tmp;
    uint32_t* tile_cnt = (uint32_t*)p;
    p += ((size_t)n_ctiles * 4 + 255) / 256 * 256;
    uint64_t* tile_off = (uint64_t*)p;
    p += ((size_t)n_ctiles * 8 + 255) / 256 * 256;
    void* scan_tmp = p;
    uint64_t* d_total = (uint64_t*)(t.flags + 2);
    if (n_keys > 0) {
        hipLaunchKernelGGL(unique_count_kernel, dim3((unsigned)n_ctiles), dim3(kBlock), 0, s,
                           sorted, n_keys, drop, tile_cnt);
        MIXGCN_TRY(exclusive_scan_u32_to_u64(tile_cnt, tile_off, n_ctiles, d_total, scan_tmp, s));
    }
    uint32_t h_flags[4];
    MIXGCN_HIP_TRY(hipMemcpyAsync(h_flags, t.flags, 16, hipMemcpyDeviceToHost, s));
    MIXGCN_HIP_TRY(hipStreamSynchronize(s));
    if (h_flags[0]) return fail(MIXGCN_EINVAL, "edge endpoint >= n_nodes");
    const uint64_t nnz64 = (uint64_t)h_flags[2] | ((uint64_t)h_flags[3] << 32);
    const int64_t nnz = (int64_t)nnz64;

    Csr c;
    c.nnz = nnz;
    c.n_groups = ceil_div(nnz, kGroupNnz);
    c.nnz_padded = (c.n_groups + 1) * kGroupNnz + kEntryPad;
    int rc = MIXGCN_OK;
    do {
        if ((rc = dmalloc(&c.rowptr, (size_t)n + 1, s)) != MIXGCN_OK) break;
        if ((rc = dmalloc(&c.col, (size_t)nnz, s)) != MIXGCN_OK) break;
        if ((rc = dmalloc(&c.cv, (size_t)c.nnz_padded, s)) != MIXGCN_OK) break;
        if ((rc = dmalloc(&c.grp_row, (size_t)c.n_groups + 1, s)) != MIXGCN_OK) break;
        if (hipMemsetAsync(c.cv + nnz, 0, (size_t)(c.nnz_padded - nnz) * 8, s) != hipSuccess) {
            rc = fail(MIXGCN_EHIP, "hipMemsetAsync(cv)");
            break;
        }
        hipLaunchKernelGGL(fill_i64_kernel, dim3((unsigned)ceil_div((int64_t)n + 1, kBlock)),
                           dim3(kBlock), 0, s, c.rowptr, (int64_t)n + 1, nnz);
        if (n_keys > 0)
            hipLaunchKernelGGL(unique_fill_kernel, dim3((unsigned)n_ctiles), dim3(kBlock), 0, s,
                               sorted, n_keys, drop, bits, n, tile_off, c.col, c.cv, c.rowptr,
                               t.flags + 1);
        hipLaunchKernelGGL(group_rows_kernel, dim3((unsigned)ceil_div(c.n_groups + 1, kBlock)),
                           dim3(kBlock), 0, s, c.rowptr, n, nnz, c.n_groups, c.grp_row);
        if ((rc = host_alloc((void**)&c.h_rowptr, ((size_t)n + 1) * 8)) != MIXGCN_OK) break;
        if (!(symmetrize && rowgroups_planned(n, nnz)) && (rc = csr_copy_rowptr(c, n, s)) != MIXGCN_OK) break;
        if (hipMemcpyAsync(h_flags, t.flags, 16, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess || hipGetLastError() != hipSuccess) {
            rc = fail(MIXGCN_EHIP, "CSR fill failed");
            break;
        }
        c.has_empty_rows = h_flags[1] != 0 || (nnz == 0 && n > 0);
    } while (0);
    if (rc != MIXGCN_OK) {
        (void)hipStreamSynchronize(s);  // the arrays may have work queued on them
        csr_free(&c);
        return rc;
    }
    *out = std::move(c);
    return MIXGCN_OK;
}

namespace {

// Values of the matrix (swapped: of its transpose on the same pattern) in all stored forms.
int fill_values(const Csr& c, const float* dinv, int mode, float eps, int swapped,
                bool transposed, float* val, uint2* cv, hipStream_t s)
{
    if (c.nnz == 0) return MIXGCN_OK;
    if (!c.groups.bands.empty() && (!transposed || c.groups.bands.back().ent_t))
        return rowgroups_fill(c, c.groups, dinv, mode, eps, swapped, transposed, val, cv, s);
    hipLaunchKernelGGL(values_kernel, dim3((unsigned)ceil_div(c.n_groups, kValueGroups)), dim3(kBlock), 0, s,
                       c.rowptr, c.grp_row, c.col, dinv, c.n_groups, c.nnz, mode, eps, swapped, val, cv);
    return MIXGCN_OK;
}

}  // namespace

int normalize_graph(mixgcn_graph* g, int mode, float eps, hipStream_t s)
{
    const uint32_t n = g->n;
    if (!g->deg) MIXGCN_TRY(dmalloc_async(&g->deg, n, s));
    if (!g->dinv) MIXGCN_TRY(dmalloc_async(&g->dinv, n, s));
    if (n > 0)
        hipLaunchKernelGGL(degree_kernel, dim3((unsigned)ceil_div(n, kBlock)), dim3(kBlock), 0, s,
                           g->fwd.rowptr, n, mode, g->deg, g->dinv);
    Csr* mats[2] = {&g->fwd, g->has_transpose ? &g->tr : nullptr};
    for (Csr* c : mats) {
        if (!c) continue;
        if (!c->val) MIXGCN_TRY(dmalloc_async(&c->val, (size_t)c->nnz, s));
        MIXGCN_TRY(fill_values(*c, g->dinv, mode, eps, c == &g->tr ? 1 : 0, false, c->val, c->cv, s));
    }
    // A symmetrised graph stores one pattern for the matrix and its transpose.  The mean
    // weights are not symmetric, so the transpose gets value arrays of its own on that pattern.
    Csr& f = g->fwd;
    if (mode == MIXGCN_NORM_MEAN && (g->flags & MIXGCN_SYMMETRIZE)) {
        if (!f.val_t) MIXGCN_TRY(dmalloc_async(&f.val_t, (size_t)f.nnz, s));
        if (!f.cv_t) MIXGCN_TRY(dmalloc_async(&f.cv_t, (size_t)f.nnz_padded, s));
        MIXGCN_TRY(rowgroups_alloc_transpose(&f.groups, s));
        hipLaunchKernelGGL(copy_entries_kernel, dim3((unsigned)ceil_div(f.nnz_padded, kBlock)),
                           dim3(kBlock), 0, s, f.cv, f.cv_t, f.nnz_padded);
        MIXGCN_TRY(fill_values(f, g->dinv, mode, eps, 1, true, f.val_t, f.cv_t, s));
    }
    MIXGCN_HIP_TRY(hipGetLastError());
    g->normalized = true;
    g->norm_mode = mode;
    return MIXGCN_OK;
}

}  // namespace mixgcn
