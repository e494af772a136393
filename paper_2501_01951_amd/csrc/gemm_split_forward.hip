// Forward product of fp32 features on the bf16 matrix cores; opt-in (mixgcn_set_update_arith), wide layers
// only.  Every fp32 operand is written as the exact sum of three bf16 terms (round to nearest at each stage),
//     x = x0 + x1 + x2,   |x1| <= 2^-8 |x|,   |x2| <= 2^-16 |x|,
// and a product a b is accumulated in fp32 from the six partial products of order 2^-16 and
// above: a2 b0, a0 b2, a1 b1, a1 b0, a0 b1, a0 b0, smallest first.  The three dropped ones are
// together below 2^-23 |a| |b|, the size of one fp32 rounding.  On this part a 32x32x16 bf16 MFMA does
// eight times the work of the 32x32x2 fp32 MFMA in half its time, so the six of them cost 3/8 of
// the fp32 path's matrix-core time.
//
// Why not the kernel of the data gradient (gemm_rows.hip), which is faster: a forward product decides
// which side of zero an activation falls on, and sums rounded otherwise exchange ReLU decisions of
// pre-activations within rounding of zero.  On a hub, one such decision moves a column of a weight gradient
// by 1e-3.  The products whose sums decide nothing are free to change their rounding, this one is not.
//
// Weights are split once per call, into the order the kernel walks them: the three terms of one
// step (16 reduction indices) of one column tile are contiguous, so a step's weights are three
// coalesced 16-byte loads per thread.  Features are split on their way from global memory to
// LDS: two conversions, four unpacks and four subtractions per term and four elements.  Vector
// instructions do not overlap with MFMAs on a SIMD, so the staging path carries nothing else:
// scalar bases plus fixed per-thread offsets, rows beyond the matrix are read from its last row
// (their results are never stored), and the reduction depth must be whole steps (the caller
// keeps the fp32 MFMA kernels otherwise).  Sums that are not finite are computed again in fp32.
//
// Pipeline of a tile: global loads run two steps ahead in two register sets; LDS is double
// buffered; the MFMA operands are themselves double buffered in registers, read from LDS one
// step before their MFMAs, so the only thing between a barrier and the next MFMA is the issue of
// those reads.  The main loop has no conditional load or store, which lets every wait on a load
// leave the other register set's loads in flight.
#include "gemm_common.h"
#include "internal.h"

namespace mixgcn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uintx4 lds_uintx4;

constexpr int BKS = 16;       // reduction depth per step = one MFMA
constexpr int LDR = BKS + 8;  // LDS row stride in bf16: 48 bytes, 16 consecutive rows hit all banks
constexpr int kPlanes = 3;

// tile of 128 x 128: 2 x 2 wavefronts of 2 x 2 accumulator tiles of 32 x 32
constexpr int WN = 2, TM = 2, TN = 2, BM = 128, BN = 128;

// The three terms of W[kk][j], zero outside W, in the order the row-block kernel walks them:
// out[column tile][step][term][j % BN][kk % 16], so that the weights of one step of one tile are
// 3 * BN * 32 contiguous bytes.
__global__ __launch_bounds__(kBlock) void split3_weights_kernel(
    const float* __restrict__ W, int64_t ldw, int rows_w, int cols_w, uint16_t* __restrict__ out, int out_rows,
    int out_cols)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= out_rows * out_cols) return;
    const int j = idx / out_cols, kk = idx % out_cols;
    float x = (kk < rows_w && j < cols_w) ? W[(int64_t)kk * ldw + j] : 0.f;
    const int nk = out_cols / BKS;
    const size_t tile = ((size_t)(j / BN) * nk + kk / BKS) * kPlanes;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
        const uint32_t h = pack_bf16(x, 0.f);
        out[((tile + p) * BN + j % BN) * BKS + kk % BKS] = (uint16_t)h;
        x -= low_half(h);
        if (!(fabsf(x) <= 3.0e38f)) x = 0.f;  // infinities and NaNs stay in the first term only
    }
}

// What one thread moves per step: two 16-byte pieces of the A tile (rows prow and prow + 64,
// four columns) and one 16-byte piece of each weight plane.
struct Stage {
    float4 a[2];
    uint4 b[kPlanes];

    __device__ inline void load(const char* a0, const char* b0, const uint32_t* aoff, uint32_t boff)
    {
        // every thread issues the same number of loads on every step, so that the wait for a
        // register set can leave the loads of the other set in flight
#pragma unroll
        for (int p = 0; p < 2; ++p) a[p] = *reinterpret_cast<const float4*>(a0 + aoff[p]);
#pragma unroll
        for (int p = 0; p < kPlanes; ++p)
            b[p] = *reinterpret_cast<const uint4*>(b0 + p * (BN * BKS * 2) + boff);
    }
    __device__ inline void store(uint16_t* as, uint16_t* bs, int apos, int bpos) const
    {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint16_t* q = as + apos + p * 64 * LDR;
            split_store<false>(a[p], a[p], 1.f, q, q + BM * LDR, q + 2 * BM * LDR);
        }
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) {
            const uintx4 v = {b[p].x, b[p].y, b[p].z, b[p].w};
            *(lds_uintx4*)(bs + p * BN * LDR + bpos) = v;
        }
    }
};

// C[n x MD] = act(A[n x KD] * W[KD x MD]); W is given as three bf16 terms in the layout of
// split3_weights_kernel, KD a multiple of BKS.
template <bool RELU>
__global__ __launch_bounds__(kBlock, 2) void forward_split_kernel(
    const float* __restrict__ A, int64_t lda, const uint16_t* __restrict__ Bp, const float* __restrict__ W,
    int64_t ldw, float* __restrict__ C, int64_t ldc, int64_t n, int KD, int MD, int n_col_tiles)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[2][kPlanes * BM * LDR];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kPlanes * BN * LDR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const unsigned lid = xcd_local_index(blockIdx.x, gridDim.x);
    const int64_t row0 = (int64_t)(lid / n_col_tiles) * BM;
    const int col0 = (int)(lid % n_col_tiles) * BN;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;

    // staging: thread -> (row tid / 4 [+ 64], columns 4 (tid % 4) ..) of A, (row tid / 2, half
    // tid % 2) of the weight planes
    // Rows are dealt to the lanes so that one LDS write cycle (16 lanes of 8 bytes, 8 lanes of 16)
    // covers rows 0, 2, 4, 6 or 1, 3, 5, 7 of a group of eight: at 12 banks per row these start at
    // banks 0, 24, 16, 8 (12, 4, 28, 20) and do not collide.
    auto dealt = [](int q) { return (q & ~7) | ((q & 3) << 1) | ((q >> 2) & 1); };
    const int prow = dealt(tid >> 2), pk = 4 * (tid & 3);
    uint32_t aoff[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        int64_t rr = row0 + p * 64 + prow;
        if (rr > n - 1) rr = n - 1;
        aoff[p] = (uint32_t)(rr - row0) * (uint32_t)lda * 4u + 4u * pk;
    }
    const int apos = prow * LDR + pk;
    const int brow = dealt(tid >> 1), bhalf = tid & 1;
    const uint32_t boff = ((uint32_t)brow * BKS + 8u * bhalf) * 2u;
    const int bpos = brow * LDR + 8 * bhalf;

    const char* a0 = reinterpret_cast<const char*>(A + row0 * lda);
    const int nk = KD / BKS;
    const char* b0 = reinterpret_cast<const char*>(
        Bp + (size_t)(lid % n_col_tiles) * nk * (kPlanes * BN * BKS));

    const int li = lane & 31, lk = lane >> 5;
    struct Operands {
        bf16x8 a[kPlanes][TM], b[kPlanes][TN];
    };
    auto read_operands = [&](Operands& o, const uint16_t* as, const uint16_t* bs) {
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                o.a[p][tm] = *reinterpret_cast<const bf16x8*>(
                    &as[p * BM * LDR + ((wm * TM + tm) * 32 + li) * LDR + 8 * lk]);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                o.b[p][tn] = *reinterpret_cast<const bf16x8*>(
                    &bs[p * BN * LDR + ((wn * TN + tn) * 32 + li) * LDR + 8 * lk]);
        }
    };
    auto mma = [&](const Operands& o) {
        // smallest partial products first; consecutive MFMAs go to different accumulators
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0};
        constexpr int pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        o.a[pa[q]][tm], o.b[pb[q]][tn], acc[tm][tn], 0, 0, 0);
    };

    // The MFMAs of step i run on operands that were read from LDS during step i - 1, while the
    // operands of step i + 1 are read and the tiles of step i + 2 are split and written over the
    // buffer that step i came from.  Two steps per trip keep every buffer and register set static.
    Stage s0, s1;
    Operands o0, o1;
    // a step beyond the last one loads the last one again (never stored): no branch around loads
    auto load = [&](Stage& st, int step) {
        const int sc = step < nk ? step : nk - 1;
        const size_t oa = (size_t)sc * (BKS * 4), ob = (size_t)sc * (kPlanes * BN * BKS * 2);
        st.load(a0 + oa, b0 + ob, aoff, boff);
    };
    load(s0, 0);
    load(s1, 1);
    s0.store(As[0], Bs[0], apos, bpos);
    load(s0, 2);
    if (nk > 1) s1.store(As[1], Bs[1], apos, bpos);
    load(s1, 3);
    __syncthreads();
    read_operands(o0, As[0], Bs[0]);
    __syncthreads();
    // main trips: both steps have two successors, so nothing in them is conditional and every
    // wait can be counted (a set's loads are awaited with the other set's five still in flight)
    int i = 0;
    for (; i + 3 < nk; i += 2) {
        read_operands(o1, As[1], Bs[1]);
        mma(o0);
        s0.store(As[0], Bs[0], apos, bpos);
        load(s0, i + 4);
        __syncthreads();
        read_operands(o0, As[0], Bs[0]);
        mma(o1);
        s1.store(As[1], Bs[1], apos, bpos);
        load(s1, i + 5);
        __syncthreads();
    }
    // the last one to three steps
    const int rem = nk - i;
    if (rem >= 2) read_operands(o1, As[1], Bs[1]);
    mma(o0);
    if (rem >= 3) s0.store(As[0], Bs[0], apos, bpos);
    if (rem >= 2) {
        __syncthreads();
        if (rem >= 3) read_operands(o0, As[0], Bs[0]);
        mma(o1);
        if (rem >= 3) mma(o0);
    }

    float z = 0.f;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) z = fmaf(acc[tm][tn][v], 0.f, z);
    const bool repair = __any(!(z == 0.f));

    // D layout: lane l, register v -> row 8 (v / 4) + 4 (l / 32) + v % 4, col l % 32
    const int wmu = __builtin_amdgcn_readfirstlane(wm), wnu = __builtin_amdgcn_readfirstlane(wn);
    const uint32_t lane_off = (uint32_t)(4 * lk) * (uint32_t)ldc + (uint32_t)li;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int ct = col0 + (wnu * TN + tn) * 32;
            const int64_t rt = row0 + (wmu * TM + tm) * 32;
            float* tile = C + rt * ldc + ct;
            if (!repair && rt + 32 <= n && ct + 32 <= MD && ldc < (1 << 22)) {
                // nothing to clip: a scalar base per register, one 32-bit lane offset
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    // as signed integers, max(bits, 0) clears exactly the values with the sign set
                    int x = __float_as_int(acc[tm][tn][v]);
                    if (RELU) x = x > 0 ? x : 0;
                    tile[(int64_t)(8 * (v / 4) + (v % 4)) * ldc + lane_off] = __int_as_float(x);
                }
            } else if (ct + li < MD) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int64_t r = rt + 8 * (v / 4) + 4 * lk + (v % 4);
                    if (r < n) {
                        float x = acc[tm][tn][v];
                        if (RELU && !repair) x = x > 0.f ? x : 0.f;
                        C[r * ldc + ct + li] = x;
                    }
                }
            }
        }
    if (__builtin_expect(repair, 0)) {
        const int64_t rt = row0 + wmu * TM * 32;
        const int ct = col0 + wnu * TN * 32;
        const int64_t r1 = rt + TM * 32 < n ? rt + TM * 32 : n;
        const int c1 = ct + TN * 32 < MD ? ct + TN * 32 : MD;
        if (rt < r1)
            repair_sums<RELU>(
                C, ldc, rt, r1, ct, c1, KD, [&](int64_t r, int k) { return A[r * lda + k]; },
                [&](int k, int c) { return W[(int64_t)k * ldw + c]; });
    }
}

}  // namespace

// Outputs of at most 64 columns and reductions of fewer than four steps are bound by their memory traffic in
// either arithmetic; 32-bit offsets inside a tile.
bool forward_split_applies(int64_t lda, int64_t n, int32_t k, int32_t m)
{
    return n > 0 && lda < (1 << 22) && m > 64 && k >= 64 && k % BKS == 0;
}

// C[n x m] = act(A[n x k] W[k x m])
int launch_forward_split(bool relu, const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc,
                         int64_t n, int32_t k, int32_t m, hipStream_t s)
{
    const int nct = (int)ceil_div(m, BN);
    const int64_t grid = ceil_div(n, BM) * nct;
    if (grid > 0x7FFFFFFF) return fail(MIXGCN_EINVAL, "update: too many row tiles");
    const int out_rows = nct * BN;
    const size_t plane = (size_t)out_rows * k;
    void* scratch = nullptr;
    MIXGCN_TRY(get_scratch(3, kPlanes * plane * sizeof(uint16_t), &scratch));
    uint16_t* planes = (uint16_t*)scratch;
    hipLaunchKernelGGL(split3_weights_kernel, dim3((unsigned)ceil_div((int64_t)plane, kBlock)), dim3(kBlock), 0, s,
                       W, ldw, k, m, planes, out_rows, k);
    if (relu)
        hipLaunchKernelGGL((forward_split_kernel<true>), dim3((unsigned)grid), dim3(kBlock), 0, s, A, lda, planes, W,
                           ldw, C, ldc, n, k, m, nct);
    else
        hipLaunchKernelGGL((forward_split_kernel<false>), dim3((unsigned)grid), dim3(kBlock), 0, s, A, lda, planes, W,
                           ldw, C, ldc, n, k, m, nct);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

}  // namespace mixgcn
