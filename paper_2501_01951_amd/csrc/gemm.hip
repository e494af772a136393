// Dispatch of the update products (paper Algorithm 2, update phase), the reduction of the slabs of a weight
// gradient, and the weight gradient dW = Z^T dP of fp32 matrices with pitches of 2^22 elements and more on the
// fp32 matrix cores (v_mfma_f32_32x32x2_f32), with 64-bit offsets throughout; every other one runs on the bf16
// matrix cores (1.15 to 1.6 times as fast, and closer to 64 bits).
#include <type_traits>

#include "device_utils.h"
#include "internal.h"

namespace mixgcn {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BK = 16;          // reduction depth staged per step
constexpr int kWgradMinBlocks = 4;  // workgroups per CU that the register allocation is held to
constexpr int kLdsPad = 4;      // row stride of the staged tiles = tile width + 4 floats

// Tile shape: WM x WN waves (4 in total), each owning TM x TN accumulator tiles of 32 x 32.
template <int WM_, int WN_, int TM_, int TN_>
struct Shape {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_;
    static constexpr int BM = WM * TM * 32;  // extent along the A-operand free dimension
    static constexpr int BN = WN * TN * 32;  // extent along the B-operand free dimension
    static_assert(WM * WN == 4, "four waves per block");
};
using Shape128x32 = Shape<4, 1, 1, 1>;

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
// starts the loads (addresses are clamped into the matrix, so they are unconditional and
// nothing waits on them); value() applies the zero fill outside [0, rows) x [0, cols) and the
// optional ReLU-derivative mask x * 1[R > 0] when the piece is written to LDS one step later.
// Feature tensors are fp32 (float) or bf16 (uint16_t, widened to fp32 on the way to LDS and
// rounded to nearest even on the way out); weights are always fp32.
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
        return make_float4(__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xFFFF0000u),
                           __uint_as_float(q.y << 16), __uint_as_float(q.y & 0xFFFF0000u));
    }
};

__device__ inline uint16_t bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) != 0x7F800000u) u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline void store_elem(float* p, float x) { *p = x; }
__device__ inline void store_elem(uint16_t* p, float x) { *p = bf16_rne(x); }

template <bool MASK, typename T>
struct Piece {
    Raw4<T> v;
    Raw4<T> m;
    int nvalid;  // leading components inside the matrix (0..4)

    __device__ inline void issue(const T* __restrict__ M, int64_t ld, int64_t r, int c,
                                 int64_t rows, int cols, const T* __restrict__ R, int64_t ldr)
    {
        const bool ok = r < rows && c < cols;
        nvalid = ok ? (cols - c < 4 ? cols - c : 4) : 0;
        const int64_t rr = r < rows ? r : rows - 1;
        const int cc = c < cols ? c : 0;
        v = *reinterpret_cast<const Raw4<T>*>(M + rr * ld + cc);
        if (MASK) m = *reinterpret_cast<const Raw4<T>*>(R + rr * ldr + cc);
    }
    // CHECKED = false: the caller knows the piece lies wholly inside the matrix
    template <bool CHECKED = true>
    __device__ inline float4 value() const
    {
        float4 o = v.widen();
        if (MASK) {
            const float4 mm = m.widen();
            o.x = mm.x > 0.f ? o.x : 0.f;
            o.y = mm.y > 0.f ? o.y : 0.f;
            o.z = mm.z > 0.f ? o.z : 0.f;
            o.w = mm.w > 0.f ? o.w : 0.f;
        }
        if (CHECKED && nvalid < 4) {
            if (nvalid < 1) o.x = 0.f;
            if (nvalid < 2) o.y = 0.f;
            if (nvalid < 3) o.z = 0.f;
            o.w = 0.f;
        }
        return o;
    }
};

// Workgroups are dealt round-robin to the 8 XCDs.  This maps the hardware block index to a
// logical one such that consecutive logical indices run on the same XCD, so tiles that share
// an operand (the column tiles of one row block) find it in that XCD's L2.
__device__ inline unsigned xcd_local_index(unsigned bid, unsigned grid)
{
    const unsigned q = grid / 8, rem = grid % 8, x = bid % 8;
    return x * q + (x < rem ? x : rem) + bid / 8;
}

// ---- slab kernel: P[slab][KD x MD] = A[rows of slab][KD]^T * (B (.) 1[R > 0])[rows][MD] --------
// Both operands are staged exactly as they lie in memory (node-major), which already is the
// reduction-major layout the MFMA operand reads want.
template <class S, bool MASK, typename T>
__global__ __launch_bounds__(kBlock, kWgradMinBlocks) void wgrad_slab_kernel(
    const T* __restrict__ A, int64_t lda, const T* __restrict__ B, int64_t ldb,
    const T* __restrict__ R, int64_t ldr, float* __restrict__ P, int64_t n, int KD, int MD,
    int64_t rows_per_slab, int n_i_tiles, int n_j_tiles)
{
    constexpr int LDA = S::BM + kLdsPad, LDB = S::BN + kLdsPad;
    __shared__ float As[2][BK * LDA];
    __shared__ float Bs[2][BK * LDB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const int tiles = n_i_tiles * n_j_tiles;
    const unsigned lid = xcd_local_index(blockIdx.x, gridDim.x);
    const int64_t slab = lid / tiles;
    const int t = (int)(lid % tiles);
    const int i0 = (t / n_j_tiles) * S::BM, j0 = (t % n_j_tiles) * S::BN;
    const int64_t r_begin = slab * rows_per_slab;
    const int64_t r_end = (r_begin + rows_per_slab) < n ? (r_begin + rows_per_slab) : n;

    floatx16 acc[S::TM][S::TN];
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < S::TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;

    constexpr int AM_F4 = S::BM / 4, BN_F4 = S::BN / 4;
    constexpr int A_RPP = kBlock / AM_F4, B_RPP = kBlock / BN_F4;
    constexpr int A_PASSES = (BK + A_RPP - 1) / A_RPP, B_PASSES = (BK + B_RPP - 1) / B_RPP;
    Piece<false, T> ra[A_PASSES];
    Piece<MASK, T> rb[B_PASSES];

    auto issue_tiles = [&](int64_t r0) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int kk = p * A_RPP + tid / AM_F4;
            ra[p].issue(A, lda, r0 + (kk < BK ? kk : 0), i0 + 4 * (tid % AM_F4), r_end, KD, nullptr, 0);
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kk = p * B_RPP + tid / BN_F4;
            rb[p].issue(B, ldb, r0 + (kk < BK ? kk : 0), j0 + 4 * (tid % BN_F4), r_end, MD, R, ldr);
        }
    };
    auto store_tiles_as = [&](float* as, float* bs, auto checked) {
        constexpr bool CHECKED = decltype(checked)::value;
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int kk = p * A_RPP + tid / AM_F4;
            if (kk < BK)
                *reinterpret_cast<float4*>(&as[kk * LDA + 4 * (tid % AM_F4)]) =
                    ra[p].template value<CHECKED>();
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kk = p * B_RPP + tid / BN_F4;
            if (kk < BK)
                *reinterpret_cast<float4*>(&bs[kk * LDB + 4 * (tid % BN_F4)]) =
                    rb[p].template value<CHECKED>();
        }
    };
    const bool tile_inside = i0 + S::BM <= KD && j0 + S::BN <= MD;
    auto store_tiles = [&](float* as, float* bs, int64_t r0) {
        if (tile_inside && r0 + BK <= r_end) store_tiles_as(as, bs, std::false_type{});
        else store_tiles_as(as, bs, std::true_type{});
    };

    if (r_begin < r_end) {
        const int64_t nk = (r_end - r_begin + BK - 1) / BK;
        issue_tiles(r_begin);
        store_tiles(As[0], Bs[0], r_begin);
        __syncthreads();
        for (int64_t i = 0; i < nk; ++i) {
            const int cur = (int)(i & 1);
            if (i + 1 < nk) issue_tiles(r_begin + (i + 1) * BK);
            mma_step<S>(As[cur], Bs[cur], wm, wn, lane, acc);
            if (i + 1 < nk) store_tiles(As[cur ^ 1], Bs[cur ^ 1], r_begin + (i + 1) * BK);
            __syncthreads();
        }
    }
    float* out = P + (size_t)slab * KD * MD;
    const int li = lane & 31, lk = lane >> 5;
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < S::TN; ++tn) {
            const int j = j0 + (wn * S::TN + tn) * 32 + li;
            if (j >= MD) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = i0 + (wm * S::TM + tm) * 32 + 8 * (v / 4) + 4 * lk + (v % 4);
                if (i < KD) out[(size_t)i * MD + j] = acc[tm][tn][v];
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

namespace {

// C[k x m] = beta C + A[n x k]^T (B (.) mask)[n x m]
int wgrad_f32(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc, int64_t n,
              int32_t k, int32_t m, const float* R, int64_t ldr, float beta, hipStream_t s, Timer* timer)
{
    const int nit = (int)ceil_div(k, Shape128x32::BM), njt = (int)ceil_div(m, Shape128x32::BN);
    const int tiles = nit * njt;
    int64_t n_slabs = wgrad_slabs(n, tiles, 1024);
    int64_t rows_per_slab = ceil_div(ceil_div(n, n_slabs), BK) * BK;
    if (rows_per_slab < BK) rows_per_slab = BK;
    n_slabs = n > 0 ? ceil_div(n, rows_per_slab) : 1;
    const int64_t cells = (int64_t)k * m;
    void* scratch = nullptr;
    MIXGCN_TRY(get_scratch(0, (size_t)n_slabs * cells * sizeof(float), &scratch));
    float* P = (float*)scratch;
    const unsigned grid = (unsigned)(n_slabs * tiles);
    if (timer) MIXGCN_TRY(timer->begin(kTimeUpdateWgrad, s));
#define MIXGCN_WGRAD(MASK)                                                                                  \
    hipLaunchKernelGGL((wgrad_slab_kernel<Shape128x32, MASK, float>), dim3(grid), dim3(kBlock), 0, s, A, lda, \
                       B, ldb, R, ldr, P, n, k, m, rows_per_slab, nit, njt)
    if (R) MIXGCN_WGRAD(true);
    else MIXGCN_WGRAD(false);
#undef MIXGCN_WGRAD
    if (timer) MIXGCN_TRY(timer->end(s));
    MIXGCN_TRY(launch_wgrad_reduce(P, n_slabs, cells, m, C, ldc, beta, s));
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

}  // namespace

int launch_update(int op, int dtype, const void* A, int64_t lda, const void* B, int64_t ldb,
                  void* C, int64_t ldc, int64_t n, int32_t k, int32_t m, const void* R,
                  int64_t ldr, float beta, hipStream_t s, Timer* timer)
{
    if (op != MIXGCN_OP_WGRAD) {
        const bool fwd = op != MIXGCN_OP_DGRAD;
        const int kind = fwd ? kTimeUpdateFwd : kTimeUpdateDgrad;
        if (timer) MIXGCN_TRY(timer->begin(kind, s));
        MIXGCN_TRY(launch_update_rows(dtype, fwd, op == MIXGCN_OP_FWD_RELU, A, lda, (const float*)B, ldb, C, ldc,
                                      n, fwd ? k : m, fwd ? m : k, fwd ? nullptr : R, ldr, s));
        if (timer) MIXGCN_TRY(timer->end(s));
        return MIXGCN_OK;
    }
    if (dtype != MIXGCN_F32)
        return launch_wgrad_bf16((const uint16_t*)A, lda, (const uint16_t*)B, ldb, (float*)C, ldc, n, k, m,
                                 (const uint16_t*)R, ldr, beta, s, timer);
    const float *a = (const float*)A, *b = (const float*)B, *r = (const float*)R;
    float* c = (float*)C;
    if (wgrad_split_applies(lda, ldb, ldr, n))
        return launch_wgrad_split(a, lda, b, ldb, c, ldc, n, k, m, r, ldr, beta, s, timer);
    return wgrad_f32(a, lda, b, ldb, c, ldc, n, k, m, r, ldr, beta, s, timer);
}

}  // namespace mixgcn
