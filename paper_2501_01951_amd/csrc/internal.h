// Internal declarations shared by the HIP sources of libmixgcn (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <string>
#include <vector>

#include "mixgcn.h"

namespace mixgcn {

// ---- error plumbing ---------------------------------------------------------------------------
void set_error(const std::string& msg);
int fail(int code, const std::string& msg);

#define MIXGCN_HIP_TRY(expr)                                                                  \
    do {                                                                                      \
        hipError_t _e = (expr);                                                               \
        if (_e != hipSuccess)                                                                 \
            return ::mixgcn::fail(_e == hipErrorOutOfMemory ? MIXGCN_ENOMEM : MIXGCN_EHIP,    \
                                  std::string(#expr) + ": " + hipGetErrorString(_e));         \
    } while (0)

#define MIXGCN_TRY(expr)         \
    do {                         \
        int _rc = (expr);        \
        if (_rc != MIXGCN_OK) return _rc; \
    } while (0)

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- graph ------------------------------------------------------------------------------------
// Granularity (in stored entries) of the table that maps an entry index to its row.
constexpr int kGroupNnz = 256;
// Padding of the kernel's entry array beyond nnz: the widest span one wavefront walks plus the
// prefetch distance of its software pipeline.
constexpr int kEntryPad = 8192;
// Bits of an entry's column word that are not part of the column index.
constexpr uint32_t kEntryEndBit = 0x80000000u;  // last stored entry of its row
constexpr uint32_t kEntryColMask = 0x3FFFFFFFu;

// Widest pass of the aggregation kernel in columns (fp32 and bf16 alike), and the bytes of row
// pieces one call can need on a graph with `nnz` stored entries, whatever its ranges.
constexpr int kAggMaxPassCols = 256;
extern int g_aggregate_whole_rows;  // measurement aid, see mixgcn_set_aggregate_whole_rows
size_t agg_scratch_bound(int64_t nnz);
size_t agg_scratch_need(int dtype, int32_t n_cols, int64_t e0, int64_t e1);

constexpr int kAggSlots = 16;
struct AggSlot {
    float* p = nullptr;
    hipStream_t stream = nullptr;
    bool bound = false;      // `stream` is meaningful (the null stream is a valid owner)
    uint64_t last_use = 0;
};

// The entries of a matrix whose columns are dealt to bands (rowgroups.hip), for aggregations over all
// rows: per band a stream of batches of eight {column, value} entries, its rows grouped by length.
struct Band {
    int64_t piece = 0;      // entries of a piece of a very long row
    int64_t n_batches = 0, n_groups = 0, n_tab = 0;
    int64_t n_cut = 0, n_pieces = 0;
    uint2* ent = nullptr;         // [8 n_batches + pad]
    uint2* ent_t = nullptr;       // the same pattern with the values of the transpose (see cv_t)
    uint32_t* rows = nullptr;     // [8 (n_groups + 16)] rows of each group
    uint32_t* kind = nullptr;     // [n_groups]
    uint64_t* start = nullptr;    // [n_groups] first batch of each group
    uint2* tab = nullptr;         // [n_tab] {group, batch} at every 8th batch
    uint32_t* cut_row = nullptr;  // [n_cut] rows that were cut into pieces
    uint64_t* piece0 = nullptr;   // [n_cut] first piece of each
    int64_t* rowptr = nullptr;    // [n + 1] of the band
    int64_t src0 = 0;             // its first entry in RowGroups::src
};
struct RowGroups {
    std::vector<Band> bands;  // empty: the columns stay in one band
    uint32_t* src = nullptr;  // [nnz] entry indices band by band
    // estimated cost of a gathered line, in units of one that misses the L2, and the most it may be for
    // the bands to pay
    double cost = 0, most_cost = 0;
};

struct Csr {
    int64_t nnz = 0;
    int64_t nnz_padded = 0;          // allocation length of cv
    int64_t n_groups = 0;            // ceil(nnz / kGroupNnz)
    int64_t* rowptr = nullptr;       // [n + 1]
    uint32_t* col = nullptr;         // [nnz]  (public form: plain ascending columns)
    float* val = nullptr;            // [nnz]  (public form)
    // The aggregation kernel's form: entry e = { col | end-of-row mark, val bits }, zero padded.
    uint2* cv = nullptr;             // [nnz_padded]
    // Values of the TRANSPOSED matrix on this same pattern (symmetrised graph whose weights are
    // not symmetric, i.e. the mean mode); null otherwise.
    uint2* cv_t = nullptr;           // [nnz_padded]
    float* val_t = nullptr;          // [nnz]
    uint32_t* grp_row = nullptr;     // [n_groups + 1] row that holds entry g * kGroupNnz
    RowGroups groups;
    int64_t* h_rowptr = nullptr;     // host copy of rowptr (host_alloc)
    bool has_empty_rows = false;
};

}  // namespace mixgcn

struct mixgcn_graph {
    uint32_t n = 0;
    uint32_t flags = 0;
    int device = 0;
    bool normalized = false;
    int norm_mode = 0;           // MIXGCN_NORM_* of the last normalisation
    bool has_transpose = false;  // a separate transpose CSR is stored in `tr`
    mixgcn::Csr fwd;
    mixgcn::Csr tr;
    uint32_t* deg = nullptr;
    float* dinv = nullptr;
    // Scratch of the aggregation kernels (pieces of the rows that cross span boundaries).  A
    // slot is bound to the stream that first asks for one and stays with it, so calls on one
    // stream share a slot (stream order keeps them apart) and calls on different streams never
    // do.  Every slot has the same size, fixed by mixgcn_normalize from the entry count (enough
    // for any row and column range); slot 0 is allocated there, further slots when a further
    // stream first aggregates this graph or ahead of time by mixgcn_graph_reserve_streams.
    mutable mixgcn::AggSlot agg_slots[mixgcn::kAggSlots];
    mutable std::mutex agg_mu;
    mutable uint64_t agg_tick = 0;
    size_t agg_slot_bytes = 0;
    // max |u - v| over the stored entries, computed on first use by the cross-layer pipeline
    mutable int64_t bandwidth = -1;
};

namespace mixgcn {

// Optional per-launch timing with HIP events recorded on the stream of the launch.
enum TimerKind {
    kTimeAggG4 = 0,  // aggregation main kernel by lane-group size: 4, 8, 16, 32, 64
    kTimeAggG8,
    kTimeAggG16,
    kTimeAggG32,
    kTimeAggG64,
    kTimeUpdateFwd,
    kTimeUpdateDgrad,
    kTimeUpdateWgrad,
    kTimeKinds
};

struct Timer {
    struct Rec {
        hipEvent_t a = nullptr, b = nullptr;
        int kind = 0;
    };
    bool enabled = false;
    std::vector<Rec> recs;
    size_t used = 0;
    int begin(int kind, hipStream_t s);
    int end(hipStream_t s);
    void reset() { used = 0; }
    void destroy();
};

}  // namespace mixgcn

struct mixgcn_pipeline {
    mixgcn::Timer timer;
    hipStream_t primary = nullptr;
    hipStream_t secondary = nullptr;
    std::vector<hipEvent_t> events;
    hipEvent_t ev_start = nullptr;
    hipEvent_t ev_done = nullptr;
};

namespace mixgcn {

// ---- device primitives (scan.hip, sort.hip) ---------------------------------------------------
// Exclusive prefix sum of n uint32 counts into uint64 offsets; total (optional, device) gets
// the sum.  tmp must hold scan_tmp_bytes(n).
size_t scan_tmp_bytes(int64_t n);
int exclusive_scan_u32_to_u64(const uint32_t* in, uint64_t* out, int64_t n, uint64_t* total,
                              void* tmp, hipStream_t s);

// Stable LSD radix sort of 64-bit keys on bits [0, n_bits).  Result ends in *sorted (either
// keys or alt).  tmp must hold sort_tmp_bytes(n).
size_t sort_tmp_bytes(int64_t n);
int radix_sort_u64(uint64_t* keys, uint64_t* alt, int64_t n, int n_bits, uint64_t** sorted,
                   void* tmp, hipStream_t s);

// ---- memory for the library's own arrays (pool.hip) ------------------------------------------
// pool_alloc: work that the caller queues on `s` may use the block at once; may wait for the device.
// pool_alloc_async: the same without that wait.  pool_alloc_unordered: any stream may use the block (no
// stream is made to wait, so it can be called while one is being recorded).
// pool_free: work on the block may be queued on any stream; pool_free_on: only work on `s` may be.
// pool_malloc: memory from the driver, not the cache, and back to it with hipFree; the cache makes room.
int pool_alloc(void** p, size_t bytes, hipStream_t s);
int pool_alloc_async(void** p, size_t bytes, hipStream_t s);
int pool_alloc_unordered(void** p, size_t bytes);
int pool_malloc(void** p, size_t bytes);
void pool_free(void* p);
void pool_free_on(void* p, hipStream_t s);
void pool_release();
// Host memory, pinned where the runtime grants it; nothing on the device may still use a block that is freed.
int host_alloc(void** p, size_t bytes);
void host_free(void* p);

// ---- scratch shared by entry points without a handle --------------------------------------------
int get_scratch(int which, size_t bytes, void** out);

// ---- kernels behind the entry points ----------------------------------------------------------
int csr_from_edges(const uint32_t* d_src, const uint32_t* d_dst, uint64_t n_edges, uint32_t n,
                   bool symmetrize, bool self_loops, bool transposed, Csr* out, hipStream_t s);
void csr_free(Csr* c);
// Queues the host copy of the row pointers; it is there once the stream has been waited for.
int csr_copy_rowptr(const Csr& c, uint32_t n, hipStream_t s);
int normalize_graph(mixgcn_graph* g, int mode, float eps, hipStream_t s);

// Whether the bands of a matrix with a symmetric pattern are planned: it is large and dense enough for them to pay.
bool rowgroups_planned(uint32_t n, int64_t nnz);
int rowgroups_build(const Csr& m, uint32_t n, RowGroups* out, hipStream_t s);
int rowgroups_alloc_transpose(RowGroups* g, hipStream_t s);
int rowgroups_fill(const Csr& m, const RowGroups& g, const float* dinv, int mode, float eps,
                   int swapped, bool transposed, float* val, uint2* cv, hipStream_t s);
void rowgroups_free(RowGroups* g);
bool rowgroups_take(const RowGroups& g, int64_t n, int64_t nnz, bool values_t, int dtype, int width,
                    size_t scratch_need);
// One fp32 pass over all rows: columns [c0, c0 + width), of which [c_lo, c_hi) are written.
int launch_groups_pass(const RowGroups& g, bool values_t, int64_t n_nodes, const void* H, int64_t ldh,
                       void* Z, int64_t ldz, int c0, int width, float* P, int epi, const uint32_t* mask,
                       int64_t ldm, int c_lo, int c_hi, hipStream_t s, Timer* timer, int timer_kind);

// Bands of the pass of `width` columns in a call whose row pieces need scratch_need bytes; 0: the
// entry-balanced kernel takes it.
int aggregate_bands(const mixgcn_graph* g, const Csr& m, bool values_t, int dtype, int width, int64_t r0,
                    int64_t r1, int epilogue, size_t scratch_need);

// mask: optional bitmap applied to the written outputs (bit c % 32 of mask[r * ldm + c / 32])
// values_t: walk the values of the transpose on the same pattern (m.cv_t: the transpose of a
// symmetrised graph with unsymmetric weights); epilogue: MIXGCN_EPI_* flags
// partials / partials_bytes: scratch for the row pieces (device); a call that would need more is
// refused with MIXGCN_EINVAL before anything is launched
int launch_aggregate(const mixgcn_graph* g, const Csr& m, bool values_t, int dtype, const void* H,
                     int64_t ldh, void* Z, int64_t ldz, int32_t c0, int32_t c1, int64_t r0,
                     int64_t r1, int epilogue, const uint32_t* mask, int64_t ldm, float* partials,
                     size_t partials_bytes, hipStream_t s, Timer* timer);
// The aggregation scratch that lives in a fixed device array of the library (one copy per
// device), for the entry point that may not allocate.
int static_agg_scratch(float** p, size_t* bytes);

// bits[r * ldb + c / 32] bit c % 32 = X[r, c] > 0; every word of a row up to ldb is written
int launch_relu_bitmap(int dtype, const void* X, int64_t ldx, int64_t n, int32_t cols,
                       uint32_t* bits, int64_t ldb, hipStream_t s);
// X <- X (.) M (bitmap M); rows are padded to 16 bytes, so the last vector is in bounds
int launch_apply_bitmap(int dtype, void* X, int64_t ldx, int64_t n, int32_t cols,
                        const uint32_t* bits, int64_t ldb, hipStream_t s);
// bit of (r, c) = upper half of SplitMix64 output r * cols + c (seed) < threshold
int launch_dropout_bitmap(uint64_t seed, int64_t n, int32_t cols, uint64_t threshold,
                          uint32_t* bits, int64_t ldb, hipStream_t s);

// G <- G (.) 1[R > 0] in place (ReLU derivative taken from the stored activation R).
int launch_relu_mask(int dtype, void* G, int64_t ldg, const void* R, int64_t ldr, int64_t n,
                     int32_t m, hipStream_t s);

// The ReLU derivative 1[R > 0] of an n x m fp32 matrix as bits: column c of row r is bit c % 4 of byte r * pitch + c / 4.
// The weight gradient writes it, the data gradient of the same layer reads it instead of R (each where p is set).
struct ReluBits {
    uint8_t* p = nullptr;
    int64_t pitch = 0;  // bytes; rows hold whole groups of 8 bytes
};
inline int64_t relu_bits_row(int32_t m) { return ceil_div(m, 32) * 8; }
// whether both products can take them
inline bool relu_bits_apply(int64_t lda, int64_t ldb, int64_t ldr, int64_t pitch)
{
    return lda < (1 << 22) && ldb < (1 << 22) && ldr < (1 << 22) && pitch < (1 << 26);
}
// whether a layer's backward pass of fp32 features is faster with them (k -> m columns)
bool relu_bits_pay(int64_t n, int32_t k, int32_t m);
int launch_update(int op, int dtype, const void* A, int64_t lda, const void* B, int64_t ldb,
                  void* C, int64_t ldc, int64_t n, int32_t k, int32_t m, const void* R,
                  int64_t ldr, float beta, hipStream_t s, Timer* timer, ReluBits bits);

// dW[k x m] = beta dW + A[n x k]^T (B (.) 1[R > 0])[n x m] of bf16 features
int launch_wgrad_bf16(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, float* C, int64_t ldc,
                      int64_t n, int32_t k, int32_t m, const uint16_t* R, int64_t ldr, float beta,
                      hipStream_t s, Timer* timer);

// the same of fp32 features, every operand as three bf16 terms
int launch_wgrad_split(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc,
                       int64_t n, int32_t k, int32_t m, const float* R, int64_t ldr, float beta,
                       hipStream_t s, Timer* timer, ReluBits bits);

// bf16 features and weights that do not fit LDS; launch_update_rows chooses it
int launch_update_bf16_deep(bool w_is_kd_major, bool relu, const uint16_t* A, int64_t lda, const float* W,
                            int64_t ldw, uint16_t* C, int64_t ldc, int64_t n, int KD, int MD,
                            const uint16_t* R, int64_t ldr, hipStream_t s);

// forward product of fp32 features on the fp32 matrix cores, weights that fit LDS
bool forward_rows_applies(int64_t n, int KD, int MD);
int launch_forward_rows(bool relu, const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc,
                        int64_t n, int KD, int MD, hipStream_t s);

// forward product of fp32 features, every operand as three bf16 terms; chosen by mixgcn_set_update_arith, and
// only where forward_split_applies says so
extern int g_update_arith;
bool forward_split_applies(int64_t lda, int64_t n, int32_t k, int32_t m);
int launch_forward_split(bool relu, const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc,
                         int64_t n, int32_t k, int32_t m, hipStream_t s);

// C[n x MD] = act((A (.) 1[R > 0])[n x KD] Wop), Wop[kk][j] = w_is_kd_major ? W[kk][j] : W[j][kk]; of fp32
// features the data gradient alone
int launch_update_rows(int dtype, bool w_is_kd_major, bool relu, const void* A, int64_t lda, const float* W,
                       int64_t ldw, void* C, int64_t ldc, int64_t n, int KD, int MD, const void* R,
                       int64_t ldr, hipStream_t s, ReluBits bits = {});

// Row slabs of a weight gradient of `tiles` output tiles over n rows: slabs of at most `most_rows`
// rows (1024 workgroups at most), and on small inputs shorter ones until every compute unit has a
// workgroup, but never below 128 rows: a slab costs its partial tile once more in the reduction, and
// a workgroup its start.  (64 x 32 over 4096 rows: 4 slabs of 1024 rows took 49 us, 32 of 128 take 9.8.)
// Shorter slabs are also more exact, the reduction adds them in fp64: 0.37 of the error there.
inline int64_t wgrad_slabs(int64_t n, int64_t tiles, int64_t most_rows)
{
    int64_t slabs = ceil_div(n, most_rows);
    const int64_t fill = ceil_div(256, tiles), finest = ceil_div(n, 128);
    if (slabs < fill) slabs = fill < finest ? fill : finest;
    const int64_t cap = tiles >= 1024 ? 1 : 1024 / tiles;
    if (slabs > cap) slabs = cap;
    return slabs < 1 ? 1 : slabs;
}

// dW = beta dW + sum of the slab partials P[slab][cells], in slab order in fp64
int launch_wgrad_reduce(const float* P, int64_t n_slabs, int64_t cells, int32_t m, float* dW,
                        int64_t ldw, float beta, hipStream_t s);

int launch_softmax_xent(int dtype, const void* logits, int64_t ldl, const int32_t* labels,
                        int64_t n, int32_t c, void* dlogits, int64_t ldd, double* loss,
                        hipStream_t s);

}  // namespace mixgcn
