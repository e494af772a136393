// Dispatch of the update products (paper Algorithm 2, update phase), the forward product H' = sigma(Z W) of
// fp32 features on the fp32 matrix cores (v_mfma_f32_32x32x2_f32) where gemm_rows_f32.hip does not take it, and the
// reduction of the slabs of a weight gradient.  A row-block kernel's workgroup owns 128 node rows: the node dimension
// is the long one, the feature dimensions are at most a few hundred.
//
// The sums of the forward product are chains of fp32 multiply-adds over the reduction index, bit for bit.
// They decide which side of zero an activation falls on, so they keep this rounding: with another one
// (three bf16 terms per operand, closer to 64 bits and up to 1.5 times as fast) a few decisions per layer
// change, and one on a hub moves a column of a weight gradient by 1e-3.
#include <type_traits>

#include "gemm_common.h"
#include "internal.h"

namespace mixgcn {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BK = 16;          // reduction depth staged per step
// Workgroups per CU that the register allocation of each kernel is held to (measured best of
// 2, 3, 4 on the 128 x 128 shapes).
constexpr int kRowblockMinBlocks = 3;
constexpr int kLdsPad = 4;      // row stride of the staged tiles = tile width + 4 floats

// acc += As[kk][a-rows] (x) Bs[kk][b-cols] over the BK staged reduction steps.  The operand
// registers of step k2 + 2 are read from LDS before the MFMAs of step k2 are issued.
// MFMA 32x32x2 operand layout: lane l supplies A[i = l % 32][k = l / 32] and B[k = l / 32][j = l % 32].
template <class S>
__device__ inline void mma_step(const float* As, const float* Bs, int wm, int wn, int lane,
                                floatx16 (&acc)[S::TM][S::TN])
{
    constexpr int LDA = S::BM + kLdsPad, LDB = S::BN + kLdsPad;
    const int li = lane & 31, lk = lane >> 5;
    const float* ap = As + lk * LDA + wm * S::TM * 32 + li;
    const float* bp = Bs + lk * LDB + wn * S::TN * 32 + li;
    float a[2][S::TM], b[2][S::TN];
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm) a[0][tm] = ap[tm * 32];
#pragma unroll
    for (int tn = 0; tn < S::TN; ++tn) b[0][tn] = bp[tn * 32];
#pragma unroll
    for (int k2 = 0; k2 < BK; k2 += 2) {
        const int cur = (k2 >> 1) & 1, nxt = cur ^ 1;
        if (k2 + 2 < BK) {
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm) a[nxt][tm] = ap[(k2 + 2) * LDA + tm * 32];
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn) b[nxt][tn] = bp[(k2 + 2) * LDB + tn * 32];
        }
#pragma unroll
        for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn)
                acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][tm], b[cur][tn],
                                                                   acc[tm][tn], 0, 0, 0);
        // keep the order written here: the LDS reads of step k2 + 2 go out before the MFMAs of
        // step k2, so their latency hides behind the matrix pipe instead of in front of it
        __builtin_amdgcn_sched_group_barrier(0x100, S::TM + S::TN, 0);  // DS reads
        __builtin_amdgcn_sched_group_barrier(0x008, S::TM * S::TN, 0);  // MFMAs
    }
}

// One 16-byte piece of an operand tile on its way from global memory to LDS.  issue() only
// starts the load (the address is clamped into the matrix, so it is unconditional and nothing
// waits on it); value() applies the zero fill outside [0, rows) x [0, cols) when the piece is
// written to LDS one step later.
struct Piece {
    float4 v;
    int nvalid;  // leading components inside the matrix (0..4)

    __device__ inline void issue(const float* __restrict__ M, int64_t ld, int64_t r, int c, int64_t rows, int cols)
    {
        const bool ok = r < rows && c < cols;
        nvalid = ok ? (cols - c < 4 ? cols - c : 4) : 0;
        const int64_t rr = r < rows ? r : rows - 1;
        const int cc = c < cols ? c : 0;
        v = *reinterpret_cast<const float4*>(M + rr * ld + cc);
    }
    // CHECKED = false: the caller knows the piece lies wholly inside the matrix
    template <bool CHECKED>
    __device__ inline float4 value() const
    {
        float4 o = v;
        if (CHECKED && nvalid < 4) {
            if (nvalid < 1) o.x = 0.f;
            if (nvalid < 2) o.y = 0.f;
            if (nvalid < 3) o.z = 0.f;
            o.w = 0.f;
        }
        return o;
    }
};

// ---- fast path: tiles that lie wholly inside their matrices, fp32 -------------------------------
// A vector instruction costs the SIMD four cycles during which its matrix core idles (measured:
// MFMA and vector work of a SIMD do not overlap on this part), so the inner loop of a tile with
// nothing to clip is written to need almost none: every global address is a scalar base (stepped
// with scalar arithmetic) plus a per-thread 32-bit offset that never changes, and every LDS
// address is a per-thread base plus an immediate.  LDS accesses go through volatile pointers so
// that the compiler keeps them as single instructions with 16-bit immediates: fused into
// two-address forms (8-bit offsets) they would need a vector add per pair to rebase.
typedef __attribute__((address_space(3))) float lds_float;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) floatx4 lds_floatx4;

// One operand tile of a step: E free indices x BK reduction indices, staged to LDS as [k][e].
//   TRANSPOSED: memory is [e][k]; an item is 4 consecutive k of one e (4 single-word writes)
//   DIRECT:     memory is [k][e]; an item is 4 consecutive e of one k (one 16-byte write)
// Item `tid` of pass p lies a whole number of rows (of memory) after item `tid` of pass 0, so one
// 32-bit offset per thread serves every pass: the pass only moves the uniform base.
template <int E, bool TRANSPOSED>
struct FastTile {
    static constexpr int LD = E + kLdsPad;
    static constexpr int ITEMS = TRANSPOSED ? E * (BK / 4) : BK * (E / 4);
    static constexpr int PASSES = (ITEMS + kBlock - 1) / kBlock;
    // rows of memory between passes, and floats of LDS between passes
    static constexpr int PASS_ROWS = TRANSPOSED ? kBlock / (BK / 4) : kBlock / (E / 4);
    static constexpr int PASS_LDS = TRANSPOSED ? PASS_ROWS : PASS_ROWS * LD;
    static_assert(PASSES == 1 || ITEMS % kBlock == 0, "whole passes");
    uint32_t goff;  // byte offset of the thread's item in the operand
    int lpos;       // float index of the item in the LDS tile
    bool on;        // the thread has an item (tiles smaller than one pass)
    float4 v[PASSES];

    __device__ inline void init(int tid, uint32_t pitch)
    {
        on = (ITEMS % kBlock == 0) || tid < ITEMS;
        const int it = on ? tid : 0;
        if (TRANSPOSED) {
            const int e = it / (BK / 4), kq = 4 * (it % (BK / 4));
            goff = (uint32_t)e * pitch + 4u * kq;
            lpos = kq * LD + e;
        } else {
            const int kk = it / (E / 4), e = 4 * (it % (E / 4));
            goff = (uint32_t)kk * pitch + 4u * e;
            lpos = kk * LD + e;
        }
    }
    // base: uniform address of the step's tile; pitch in bytes
    __device__ inline void load(const char* base, size_t pitch)
    {
        if (on) {
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
                v[p] = *reinterpret_cast<const float4*>(base + p * PASS_ROWS * pitch + goff);
        }
    }
    __device__ inline void store(float* tile) const
    {
        if (on) {
#pragma unroll
            for (int p = 0; p < PASSES; ++p) {
                if (TRANSPOSED) {
                    volatile lds_float* o = (volatile lds_float*)(tile + lpos + p * PASS_LDS);
                    o[0 * LD] = v[p].x;
                    o[1 * LD] = v[p].y;
                    o[2 * LD] = v[p].z;
                    o[3 * LD] = v[p].w;
                } else {
                    const floatx4 q = {v[p].x, v[p].y, v[p].z, v[p].w};
                    *(lds_floatx4*)(tile + lpos + p * PASS_LDS) = q;
                }
            }
        }
    }
};

// mma_step with single-word LDS reads at immediate offsets.
template <class S>
__device__ inline void mma_step_fast(const float* As, const float* Bs, int wm, int wn, int lane,
                                     floatx16 (&acc)[S::TM][S::TN])
{
    constexpr int LDA = S::BM + kLdsPad, LDB = S::BN + kLdsPad;
    const int li = lane & 31, lk = lane >> 5;
    const volatile lds_float* ap = (const volatile lds_float*)(As + lk * LDA + wm * S::TM * 32 + li);
    const volatile lds_float* bp = (const volatile lds_float*)(Bs + lk * LDB + wn * S::TN * 32 + li);
    float a[2][S::TM], b[2][S::TN];
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm) a[0][tm] = ap[tm * 32];
#pragma unroll
    for (int tn = 0; tn < S::TN; ++tn) b[0][tn] = bp[tn * 32];
#pragma unroll
    for (int k2 = 0; k2 < BK; k2 += 2) {
        const int cur = (k2 >> 1) & 1, nxt = cur ^ 1;
        if (k2 + 2 < BK) {
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm) a[nxt][tm] = ap[(k2 + 2) * LDA + tm * 32];
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn) b[nxt][tn] = bp[(k2 + 2) * LDB + tn * 32];
        }
#pragma unroll
        for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn)
                acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][tm], b[cur][tn],
                                                                   acc[tm][tn], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, S::TM + S::TN, 0);  // DS reads of step k2 + 2
        __builtin_amdgcn_sched_group_barrier(0x008, S::TM * S::TN, 0);  // MFMAs of step k2
    }
}

// The reduction loop of the fast path: nk full steps, LDS double buffered with compile-time
// buffer indices (two steps per trip) so that buffer offsets fold into the immediates.
template <class S, class TA, class TB, class LoadFn>
__device__ inline void fast_reduction(float (&As)[2][BK * (S::BM + kLdsPad)],
                                      float (&Bs)[2][BK * (S::BN + kLdsPad)], TA& ta, TB& tb,
                                      LoadFn load, int64_t nk, int wm, int wn, int lane,
                                      floatx16 (&acc)[S::TM][S::TN])
{
    load((int64_t)0);
    ta.store(As[0]);
    tb.store(Bs[0]);
    __syncthreads();
    int64_t s = 0;
    while (s + 2 < nk) {
        load(s + 1);
        mma_step_fast<S>(As[0], Bs[0], wm, wn, lane, acc);
        ta.store(As[1]);
        tb.store(Bs[1]);
        __syncthreads();
        load(s + 2);
        mma_step_fast<S>(As[1], Bs[1], wm, wn, lane, acc);
        ta.store(As[0]);
        tb.store(Bs[0]);
        __syncthreads();
        s += 2;
    }
    if (s + 1 < nk) {
        load(s + 1);
        mma_step_fast<S>(As[0], Bs[0], wm, wn, lane, acc);
        ta.store(As[1]);
        tb.store(Bs[1]);
        __syncthreads();
        mma_step_fast<S>(As[1], Bs[1], wm, wn, lane, acc);
    } else {
        mma_step_fast<S>(As[0], Bs[0], wm, wn, lane, acc);
    }
}

// ---- row-block kernel: C[n x MD] = act(A[n x KD] * B[KD x MD]) ----------------------------------
// A is staged transposed (reduction-major) so that the MFMA operand reads are unit-stride.
// LDS tiles are double buffered: one barrier per reduction step.
template <class S, bool RELU>
__global__ __launch_bounds__(kBlock, kRowblockMinBlocks) void rowblock_gemm_kernel(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    float* __restrict__ C, int64_t ldc, int64_t n, int KD, int MD, int n_col_tiles)
{
    constexpr int LDA = S::BM + kLdsPad, LDB = S::BN + kLdsPad;
    __shared__ float As[2][BK * LDA];
    __shared__ float Bs[2][BK * LDB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const unsigned lid = xcd_local_index(blockIdx.x, gridDim.x);
    const int64_t row0 = (int64_t)(lid / n_col_tiles) * S::BM;
    const int col0 = (int)(lid % n_col_tiles) * S::BN;

    floatx16 acc[S::TM][S::TN];
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < S::TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;

    // staging maps: "strided" = 4 consecutive reduction indices of one row/col per thread
    constexpr int A_PASSES = S::BM / 64;  // 64 rows per pass
    constexpr int BN_F4 = S::BN / 4;       // float4 per staged B row
    constexpr int B_ROWS_PER_PASS = kBlock / BN_F4;
    constexpr int B_PASSES = (BK + B_ROWS_PER_PASS - 1) / B_ROWS_PER_PASS;
    Piece ra[A_PASSES], rb[B_PASSES];

    auto issue_tiles = [&](int k0) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p)
            ra[p].issue(A, lda, row0 + p * 64 + tid / 4, k0 + 4 * (tid & 3), n, KD);
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kk = p * B_ROWS_PER_PASS + tid / BN_F4;
            rb[p].issue(B, ldb, k0 + (kk < BK ? kk : 0), col0 + 4 * (tid % BN_F4), KD, MD);
        }
    };
    // CHECKED = false when every piece of the two tiles lies inside its matrix (uniform): the
    // zero fill then costs no vector ALU work next to the MFMAs
    auto store_tiles_as = [&](float* as, float* bs, auto checked) {
        constexpr bool CHECKED = decltype(checked)::value;
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int i = p * 64 + tid / 4, kq = 4 * (tid & 3);
            const float4 v = ra[p].template value<CHECKED>();
            as[(kq + 0) * LDA + i] = v.x;
            as[(kq + 1) * LDA + i] = v.y;
            as[(kq + 2) * LDA + i] = v.z;
            as[(kq + 3) * LDA + i] = v.w;
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kk = p * B_ROWS_PER_PASS + tid / BN_F4;
            if (kk < BK)
                *reinterpret_cast<float4*>(&bs[kk * LDB + 4 * (tid % BN_F4)]) =
                    rb[p].template value<CHECKED>();
        }
    };
    const bool tile_inside = row0 + S::BM <= n && col0 + S::BN <= MD;
    auto store_tiles = [&](float* as, float* bs, int k0) {
        if (tile_inside && k0 + BK <= KD) store_tiles_as(as, bs, std::false_type{});
        else store_tiles_as(as, bs, std::true_type{});
    };

    const int nk = (KD + BK - 1) / BK;
    // every piece inside its matrix, whole reduction steps, 32-bit offsets within a tile
    const bool fast = tile_inside && KD % BK == 0 && lda < (1 << 22) && ldb < (1 << 22);
    if (fast) {
        FastTile<S::BM, true> ta;
        FastTile<S::BN, false> tb;
        ta.init(tid, (uint32_t)lda * 4u);
        tb.init(tid, (uint32_t)ldb * 4u);
        const char* a0 = reinterpret_cast<const char*>(A + row0 * lda);
        const char* b0 = reinterpret_cast<const char*>(B + col0);
        const size_t b_step = (size_t)BK * 4 * (size_t)ldb;
        auto load = [&](int64_t st) {
            ta.load(a0 + (size_t)st * (BK * 4), (size_t)lda * 4);
            tb.load(b0 + (size_t)st * b_step, (size_t)ldb * 4);
        };
        fast_reduction<S>(As, Bs, ta, tb, load, (int64_t)nk, wm, wn, lane, acc);
    } else {
        issue_tiles(0);
        store_tiles(As[0], Bs[0], 0);
        __syncthreads();
        for (int i = 0; i < nk; ++i) {
            const int cur = i & 1;
            if (i + 1 < nk) issue_tiles((i + 1) * BK);
            mma_step<S>(As[cur], Bs[cur], wm, wn, lane, acc);
            if (i + 1 < nk) store_tiles(As[cur ^ 1], Bs[cur ^ 1], (i + 1) * BK);
            __syncthreads();
        }
    }

    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4, col l%32
    const int li = lane & 31, lk = lane >> 5;
    if (tile_inside) {
        // no bounds to test: a scalar base per 32 x 32 tile and register, one 32-bit lane offset
        const int wmu = __builtin_amdgcn_readfirstlane(wm), wnu = __builtin_amdgcn_readfirstlane(wn);
        const uint32_t lane_off = (uint32_t)(4 * lk) * (uint32_t)ldc + (uint32_t)li;
#pragma unroll
        for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn) {
                float* tile = C + (row0 + (wmu * S::TM + tm) * 32) * ldc + col0 + (wnu * S::TN + tn) * 32;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = acc[tm][tn][v];
                    if (RELU) x = fmaxf(x, 0.f);
                    tile[(int64_t)(8 * (v / 4) + (v % 4)) * ldc + lane_off] = x;
                }
            }
        return;
    }
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < S::TN; ++tn) {
            const int c = col0 + (wn * S::TN + tn) * 32 + li;
            if (c >= MD) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t r = row0 + (wm * S::TM + tm) * 32 + 8 * (v / 4) + 4 * lk + (v % 4);
                if (r < n) {
                    float x = acc[tm][tn][v];
                    if (RELU) x = x > 0.f ? x : 0.f;
                    C[r * ldc + c] = x;
                }
            }
        }
}

// ---- data gradient over fewer than four indices: dZ[n x k] = (G (.) 1[R > 0])[n x m] W[k x m]^T -----
// At these depths a chain of fp32 multiply-adds is closer to 64 bits than the sums of three bf16 terms
// (relative error at depth 1 2.5e-8 against 3.4e-8, 2 3.1e-8 : 3.3e-8, 3 half of them zero 3.1e-8 : 3.3e-8;
// from 4 on it is not: 4.1e-8 : 3.2e-8, 16 7.3e-8 : 3.6e-8).  Bound by writing dZ: the masked rows of G of a
// workgroup wait in LDS, a thread keeps its four columns of W^T and walks the rows.  us at 2^20 rows 2 -> 256,
// plain and masked, 207 and 214 (three terms 206, 208), 3 -> 100 89 and 90 (282, 278).
constexpr int kShallowRows = 1024;  // most rows of a workgroup
template <bool MASK>
__global__ __launch_bounds__(kBlock) void shallow_dgrad_kernel(const float* __restrict__ G, int64_t ldg,
                                                               const float* __restrict__ W, int64_t ldw,
                                                               float* __restrict__ Z, int64_t ldz, int64_t n, int k,
                                                               int m, const float* __restrict__ R, int64_t ldr,
                                                               int quads, int block_rows)
{
    __shared__ float4 g[kShallowRows];
    const int64_t row0 = (int64_t)blockIdx.x * block_rows;
    const int here = n - row0 < block_rows ? (int)(n - row0) : block_rows;
    for (int i = threadIdx.x; i < here; i += kBlock) {  // (rows are padded to 16 bytes)
        float4 x = *reinterpret_cast<const float4*>(G + (row0 + i) * ldg);
        if (MASK) {
            const float4 r = *reinterpret_cast<const float4*>(R + (row0 + i) * ldr);
            x = make_float4(r.x > 0.f ? x.x : 0.f, r.y > 0.f ? x.y : 0.f, r.z > 0.f ? x.z : 0.f, 0.f);
        }
        g[i] = x;
    }
    __syncthreads();
    const int rows = kBlock / quads;  // rows per pass; the threads past them have no work
    const int sub = threadIdx.x / quads;
    const int c = 4 * ((int)blockIdx.y * quads + (int)(threadIdx.x % quads));
    if (sub >= rows || c >= k) return;
    float4 w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = *reinterpret_cast<const float4*>(W + (int64_t)(c + e < k ? c + e : c) * ldw);
    float* z = Z + (row0 + sub) * ldz + c;
    for (int i = sub; i < here; i += rows, z += rows * ldz) {
        const float4 x = g[i];
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = fmaf(x.x, w[e].x, 0.f);
            if (m > 1) o[e] = fmaf(x.y, w[e].y, o[e]);
            if (m > 2) o[e] = fmaf(x.z, w[e].z, o[e]);
        }
        if (c + 4 <= k) {
            *reinterpret_cast<float4*>(z) = make_float4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (c + e < k) z[e] = o[e];
        }
    }
}

// dW = beta * dW + sum over slabs.  A block owns 64 consecutive cells; its four waves each add
// every fourth slab (in slab order, fp64) and the four sums are combined in a fixed order, so
// the result is deterministic.
__global__ __launch_bounds__(kBlock) void wgrad_reduce_kernel(const float* __restrict__ P,
                                                              int64_t n_slabs, int64_t cells,
                                                              int MD, float* __restrict__ dW,
                                                              int64_t ldw, float beta)
{
    __shared__ double part[kBlock / kWave][kWave];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * kWave + lane;
    double s = 0.0;
    if (i < cells) {
        // eight loads in flight, added in the order of the plain loop
        constexpr int kStep = kBlock / kWave;
        int64_t b = w;
        for (; b + 7 * kStep < n_slabs; b += 8 * kStep) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = P[(size_t)(b + u * kStep) * cells + i];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)v[u];
        }
        for (; b < n_slabs; b += kStep) s += (double)P[(size_t)b * cells + i];
    }
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < cells) {
        const double t = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
        float* o = dW + (i / MD) * ldw + (i % MD);
        *o = (float)(beta != 0.f ? (double)beta * (double)*o + t : t);
    }
}

// four features as stored
template <typename T>
struct Raw4;
template <>
struct Raw4<float> {
    float4 q;
    __device__ inline float4 widen() const { return q; }
};
template <>
struct Raw4<uint16_t> {
    uint2 q;
    __device__ inline float4 widen() const
    {
        return make_float4(low_half(q.x), high_half(q.x), low_half(q.y), high_half(q.y));
    }
};

// G <- G (.) 1[R > 0], four elements per thread (bf16: zeroing keeps the bits exact).
template <typename T>
__global__ __launch_bounds__(kBlock) void relu_mask_kernel(T* __restrict__ G, int64_t ldg,
                                                           const T* __restrict__ R, int64_t ldr,
                                                           int64_t n, int m4)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * m4) return;
    const int64_t r = i / m4;
    const int c = (int)(i % m4) * 4;
    T* gp = G + r * ldg + c;
    const float4 h = reinterpret_cast<const Raw4<T>*>(R + r * ldr + c)->widen();
    if (!(h.x > 0.f)) gp[0] = (T)0;
    if (!(h.y > 0.f)) gp[1] = (T)0;
    if (!(h.z > 0.f)) gp[2] = (T)0;
    if (!(h.w > 0.f)) gp[3] = (T)0;
}

template <class S>
int launch_rowblock(bool relu, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc,
                    int64_t n, int KD, int MD, hipStream_t s)
{
    const int nct = (int)ceil_div(MD, S::BN);
    const int64_t grid = ceil_div(n, S::BM) * nct;
    if (grid <= 0) return MIXGCN_OK;
    if (grid > 0x7FFFFFFF) return fail(MIXGCN_EINVAL, "update: too many row tiles");
    if (relu)
        hipLaunchKernelGGL((rowblock_gemm_kernel<S, true>), dim3((unsigned)grid), dim3(kBlock), 0, s, A, lda, B,
                           ldb, C, ldc, n, KD, MD, nct);
    else
        hipLaunchKernelGGL((rowblock_gemm_kernel<S, false>), dim3((unsigned)grid), dim3(kBlock), 0, s, A, lda, B,
                           ldb, C, ldc, n, KD, MD, nct);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

// Whether C holds other columns than A of the rows of one buffer.
bool column_blocks(const float* A, int64_t lda, int32_t k, const float* C, int64_t ldc, int32_t m)
{
    const int64_t off = ((intptr_t)C - (intptr_t)A) / (int64_t)sizeof(float) % lda, col = off < 0 ? off + lda : off;
    return lda == ldc && col >= k && col + m <= lda;
}

// C[n x m] = act(A[n x k] W[k x m])
int forward_f32(bool relu, const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc,
                int64_t n, int32_t k, int32_t m, hipStream_t s)
{
    // A product written over its features has to read all of a row's before any of its sums are written: one column
    // tile, of up to 128 columns, by a workgroup that reads its own rows alone.
    const bool apart = C + n * ldc <= A || A + n * lda <= C || column_blocks(A, lda, k, C, ldc, m);
    if (apart && forward_rows_applies(n, k, m))
        return launch_forward_rows(relu, A, lda, W, ldw, C, ldc, n, k, m, s);
    return m > (apart ? 64 : 32) ? launch_rowblock<Shape128x128>(relu, A, lda, W, ldw, C, ldc, n, k, m, s)
                                 : launch_rowblock<Shape128x32>(relu, A, lda, W, ldw, C, ldc, n, k, m, s);
}

int shallow_dgrad(const float* G, int64_t ldg, const float* W, int64_t ldw, float* Z, int64_t ldz, int64_t n, int32_t k,
                  int32_t m, const float* R, int64_t ldr, hipStream_t s)
{
    if (n <= 0) return MIXGCN_OK;
    const int all = (int)ceil_div(k, 4), quads = all < kBlock ? all : kBlock, rows = kBlock / quads;
    // at most 16 passes of rows, as long as eight workgroups per compute unit are left
    int64_t block_rows = n / 2048 / rows * rows;
    const int64_t most = 16 * rows < kShallowRows ? 16 * rows : kShallowRows / rows * rows;
    block_rows = block_rows < rows ? rows : block_rows > most ? most : block_rows;
    const int64_t grid = ceil_div(n, block_rows);
    if (grid > 0x7FFFFFFF || ceil_div(all, quads) > 65535) return fail(MIXGCN_EINVAL, "update: too many row tiles");
    const dim3 blocks((unsigned)grid, (unsigned)ceil_div(all, quads));
    if (R)
        hipLaunchKernelGGL(shallow_dgrad_kernel<true>, blocks, dim3(kBlock), 0, s, G, ldg, W, ldw, Z, ldz, n, k, m, R,
                           ldr, quads, (int)block_rows);
    else
        hipLaunchKernelGGL(shallow_dgrad_kernel<false>, blocks, dim3(kBlock), 0, s, G, ldg, W, ldw, Z, ldz, n, k, m, R,
                           ldr, quads, (int)block_rows);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

}  // namespace

int launch_relu_mask(int dtype, void* G, int64_t ldg, const void* R, int64_t ldr, int64_t n,
                     int32_t m, hipStream_t s)
{
    const int m4 = (m + 3) / 4;  // rows are padded to 16 bytes, so the last vector is in bounds
    const int64_t total = n * m4;
    if (total == 0) return MIXGCN_OK;
    const dim3 grid((unsigned)ceil_div(total, kBlock));
    if (dtype == MIXGCN_F32)
        hipLaunchKernelGGL(relu_mask_kernel<float>, grid, dim3(kBlock), 0, s, (float*)G, ldg,
                           (const float*)R, ldr, n, m4);
    else
        hipLaunchKernelGGL(relu_mask_kernel<uint16_t>, grid, dim3(kBlock), 0, s, (uint16_t*)G, ldg,
                           (const uint16_t*)R, ldr, n, m4);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

int launch_wgrad_reduce(const float* P, int64_t n_slabs, int64_t cells, int32_t m, float* dW,
                        int64_t ldw, float beta, hipStream_t s)
{
    if (cells <= 0) return MIXGCN_OK;
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)ceil_div(cells, kWave)), dim3(kBlock),
                       0, s, P, n_slabs, cells, m, dW, ldw, beta);
    return MIXGCN_OK;
}

// Making the bits costs the weight gradient a twentieth; the data gradient gains where its column tiles are full and it
// waits for memory.  Times as fast with bits as with Hout read twice, both gradients and an aggregation of three entries
// per row: 128 -> 1024 1.06 of 2500 rows, 1.05 of 100 k, 1.00 of 10^6 (2^21 rows 8800 -> 8310 us); 64 -> 768 1.09, 1.06,
// 1.05; 256 -> 512 1.03, 1.04, 1.03; 32 -> 512 1.01, 1.10, 1.11.  96 -> 640 1.03, 1.03, 0.97.  Fewer or uneven columns,
// 256 -> 256 0.99, 1.03, 1.01, 384 -> 600 1.01, 1.04, 1.02 (0.98 of 20 k); column tiles that are not full, 320 -> 600
// 0.98, 1.00, 0.99, 192 -> 768 1.00, 1.01, 1.00 (0.98 of 20 k), 48 -> 600 1.02, 0.98, 0.94.
bool relu_bits_pay(int64_t n, int32_t k, int32_t m)
{
    const bool full = k == 32 || k == 64 || k % 128 == 0;
    if (m >= 512 && m % 128 == 0) return full || (k > 64 && k < 128 && n < (1 << 19));
    return m >= 256 && k >= 256 && full && n >= (1 << 16);
}

int launch_update(int op, int dtype, const void* A, int64_t lda, const void* B, int64_t ldb,
                  void* C, int64_t ldc, int64_t n, int32_t k, int32_t m, const void* R,
                  int64_t ldr, float beta, hipStream_t s, Timer* timer, ReluBits bits)
{
    if (op != MIXGCN_OP_WGRAD) {
        const bool fwd = op != MIXGCN_OP_DGRAD, relu = op == MIXGCN_OP_FWD_RELU;
        if (timer) MIXGCN_TRY(timer->begin(fwd ? kTimeUpdateFwd : kTimeUpdateDgrad, s));
        if (!fwd && dtype == MIXGCN_F32 && m < 4)
            MIXGCN_TRY(shallow_dgrad((const float*)A, lda, (const float*)B, ldb, (float*)C, ldc, n, k, m,
                                     (const float*)R, ldr, s));
        else if (!fwd || dtype != MIXGCN_F32)
            MIXGCN_TRY(launch_update_rows(dtype, fwd, relu, A, lda, (const float*)B, ldb, C, ldc, n, fwd ? k : m,
                                          fwd ? m : k, fwd ? nullptr : R, ldr, s, bits));
        else if (g_update_arith == MIXGCN_ARITH_BF16X3 && forward_split_applies(lda, n, k, m))
            MIXGCN_TRY(launch_forward_split(relu, (const float*)A, lda, (const float*)B, ldb, (float*)C, ldc, n, k,
                                            m, s));
        else
            MIXGCN_TRY(forward_f32(relu, (const float*)A, lda, (const float*)B, ldb, (float*)C, ldc, n, k, m, s));
        if (timer) MIXGCN_TRY(timer->end(s));
        return MIXGCN_OK;
    }
    if (dtype != MIXGCN_F32)
        return launch_wgrad_bf16((const uint16_t*)A, lda, (const uint16_t*)B, ldb, (float*)C, ldc, n, k, m,
                                 (const uint16_t*)R, ldr, beta, s, timer);
    return launch_wgrad_split((const float*)A, lda, (const float*)B, ldb, (float*)C, ldc, n, k, m, (const float*)R, ldr,
                              beta, s, timer, bits);
}

}  // namespace mixgcn
