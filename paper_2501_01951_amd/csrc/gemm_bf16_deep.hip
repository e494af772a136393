// Forward product and data gradient of bf16 features whose weights do not fit LDS (more than 320 reduction
// indices of 128 output columns, 640 of 64, 1280 of 32, 2560 of 16): tiles of 128 x 128 or 128 x 32 on the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation), both operands staged through LDS.
//
// Every call first splits W = hi + lo into two bf16 terms (|W - hi - lo| < 2^-16 |W|) in the layout the B
// operand wants (output index major, reduction index contiguous, zero padded to whole tiles, and tile by tile
// in the order the kernel walks them), so that a step's weights are one dense block and are split once, not
// once per workgroup: a kernel whose workgroups each split the weights on the way through two LDS buffers took,
// us at 2^19 rows against this one, 602 -> 128 263 : 208, 513 -> 200 664 : 320, 1024 -> 256 728 : 606,
// 333 -> 77 250 : 137.
//
// MFMA 32x32x16 operand layout: lane l supplies A[i = l % 32][k = 8 (l / 32) + 0..7] and
// B[k = 8 (l / 32) + 0..7][j = l % 32] as eight consecutive bf16; D as for the fp32 32x32 MFMA.
#include "gemm_bf16_tiles.h"
#include "internal.h"

namespace mixgcn {
namespace {

// Operand element (j, kk) = transpose ? W[kk][j] : W[j][kk], zero outside W, as bf16 hi and lo
// parts, in the order the row-block kernel walks them: [column tile j / bn][step kk / BKB]
// [j % bn][kk % BKB], so that the weights of one step of one tile are bn * 64 contiguous bytes.
__device__ __host__ inline size_t split_weight_index(int j, int kk, int bn, int n_steps)
{
    return (((size_t)(j / bn) * n_steps + kk / BKB) * bn + j % bn) * BKB + kk % BKB;
}
__global__ __launch_bounds__(kBlock) void split_weights_kernel(
    const float* __restrict__ W, int64_t ldw, int rows_w, int cols_w, int transpose,
    uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, int out_rows, int out_cols, int bn)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= out_rows * out_cols) return;
    const int j = idx / out_cols, kk = idx % out_cols;
    const int r = transpose ? kk : j, c = transpose ? j : kk;
    const float x = (r < rows_w && c < cols_w) ? W[(int64_t)r * ldw + c] : 0.f;
    const uint16_t h = (uint16_t)pack_bf16(x, 0.f);
    const float rest = x - low_half(h);
    const size_t o = split_weight_index(j, kk, bn, out_cols / BKB);
    hi[o] = h;
    lo[o] = fabsf(rest) <= 3.0e38f ? (uint16_t)pack_bf16(rest, 0.f) : (uint16_t)0;
}

// ---- fast path of the row-block kernel ----------------------------------------------------------
// Vector instructions do not overlap with MFMAs on a SIMD of this part (each costs 4 cycles, an
// eighth of a 32x32x16 bf16 MFMA), and the generic staging path above spends more cycles on
// address arithmetic and zero-fill masks than the MFMAs take.  A tile whose rows all exist, with
// a reduction depth of whole steps, needs none of that: both operands are 16-byte copies from a
// scalar base plus a fixed per-thread offset to a fixed LDS position (the split weights are
// padded to whole tiles with zeros).  What is left per step is the ReLU mask, three packed 16-bit
// integer instructions and an AND per 32-bit word.
// Tile row of a thread's 16-byte pieces: rows are dealt so that the 16 lanes of one LDS write
// cycle (four rows of 64 bytes) take rows q, q + 4, q + 8, q + 12 of a group of 16, which at 20
// banks per row start 16 banks apart (0, 16, 32, 48 of 64) and do not collide.
__device__ inline int staged_row(int tid)
{
    const int x = tid >> 2;
    return (x & ~15) | ((x & 3) << 2) | ((x >> 2) & 3);
}

template <class S, bool MASK>
struct FastStage {
    static constexpr int A_PASSES = S::BM / 64;
    static constexpr int B_PASSES = (S::BN + 63) / 64;
    uint32_t aoff, roff, boff;  // bytes from the step's scalar bases
    int lpos;                   // halfword index in a staged tile
    bool b_on[B_PASSES];
    uint4 a[A_PASSES], r[A_PASSES], bh[B_PASSES], bl[B_PASSES];

    static constexpr uint32_t kPitchB = BKB * 2;  // a weight tile of one step is dense
    __device__ inline void init(int tid, uint32_t pitch_a, uint32_t pitch_r)
    {
        const int prow = staged_row(tid), pk = 8 * (tid & 3);
        aoff = (uint32_t)prow * pitch_a + 2u * pk;
        roff = (uint32_t)prow * pitch_r + 2u * pk;
        // threads beyond a narrow weight tile load a row of it again and store nothing
        boff = (uint32_t)(prow % S::BN) * kPitchB + 2u * pk;
        lpos = prow * LDT + pk;
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) b_on[p] = p * 64 + prow < S::BN;
    }
    __device__ inline void load(const char* a0, const char* r0, const char* bh0, const char* bl0,
                                size_t pitch_a, size_t pitch_r)
    {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            a[p] = *reinterpret_cast<const uint4*>(a0 + p * 64 * pitch_a + aoff);
            if (MASK) r[p] = *reinterpret_cast<const uint4*>(r0 + p * 64 * pitch_r + roff);
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            bh[p] = *reinterpret_cast<const uint4*>(bh0 + p * 64 * kPitchB + boff);
            bl[p] = *reinterpret_cast<const uint4*>(bl0 + p * 64 * kPitchB + boff);
        }
    }
    // TAIL: the last step of a reduction depth that is not a whole number of steps; `km` clears
    // the elements past the depth (what the row holds there is not part of the operand)
    template <bool TAIL = false>
    __device__ inline void store(uint16_t* as, uint16_t* bhs, uint16_t* bls,
                                 const uint4& km = uint4()) const
    {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            uint4 v = a[p];
            if (MASK) {
                v.x = keep_positive(v.x, r[p].x);
                v.y = keep_positive(v.y, r[p].y);
                v.z = keep_positive(v.z, r[p].z);
                v.w = keep_positive(v.w, r[p].w);
            }
            if (TAIL) {
                v.x &= km.x;
                v.y &= km.y;
                v.z &= km.z;
                v.w &= km.w;
            }
            lds_store16(as + lpos + p * 64 * LDT, v);
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p)
            if (b_on[p]) {
                lds_store16(bhs + lpos + p * 64 * LDT, bh[p]);
                lds_store16(bls + lpos + p * 64 * LDT, bl[p]);
            }
    }
};

// ---- row-block kernel: C[n x MD] = (A (.) 1[R > 0])[n x KD] * Bop[KD x MD] ---------------------
// Bop is given split, in the order of split_weights_kernel (bn = BN): j < n_col_tiles * BN,
// kk < ldb (a multiple of BKB), zero outside the weights.
// Occupancy decides these kernels: they are bound by memory traffic, and what hides a
// workgroup's barrier and load waits is another workgroup on the same compute unit.  The wide
// tile therefore keeps ONE set of operand tiles in LDS (two barriers per step) and one set of
// staging registers, which fits three workgroups per compute unit (34 KB of LDS, 160 registers);
// with double-buffered tiles and two register sets only two fit, and every shape of config 5 ran
// 5-24 % slower.  The narrow tile is small enough for four workgroups with double buffering.
template <class S, bool RELU, bool MASK>
__global__ __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(S::BN >= 128 ? 3 : 4, S::BN >= 128 ? 3 : 4))) void rowblock_bf16_kernel(
    const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ Bh,
    const uint16_t* __restrict__ Bl, int ldb, uint16_t* __restrict__ C, int64_t ldc, int64_t n,
    int KD, int MD, const uint16_t* __restrict__ R, int64_t ldr, int n_col_tiles)
{
    // one buffer: the operand tiles (one set for the wide tile, two for the narrow one), and
    // after the last step the output tile
    constexpr bool kDouble = S::BN < 128;
    constexpr int kTileA = S::BM * LDT, kTileB = S::BN * LDT;
    constexpr int LDC = S::BN + 4;  // output tile rows: 66 or 18 banks, 8-byte aligned
    constexpr int kSets = kDouble ? 2 : 1;
    constexpr int kOperands = kSets * (kTileA + 2 * kTileB);
    constexpr int kSmem = S::BM * LDC > kOperands ? S::BM * LDC : kOperands;
    __shared__ __attribute__((aligned(16))) uint16_t smem[kSmem];
    uint16_t *As[2], *Bhs[2], *Bls[2];
    As[0] = smem;
    As[1] = kDouble ? smem + kTileA : As[0];
    Bhs[0] = smem + kSets * kTileA;
    Bhs[1] = kDouble ? Bhs[0] + kTileB : Bhs[0];
    Bls[0] = smem + kSets * kTileA + kSets * kTileB;
    Bls[1] = kDouble ? Bls[0] + kTileB : Bls[0];
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

    // a tile row holds BKB bf16 = 4 pieces of 16 bytes; a pass of the block covers 64 tile rows
    constexpr int A_PASSES = S::BM / 64;
    constexpr int B_PASSES = (S::BN + 63) / 64;
    Piece8<MASK> ra[A_PASSES];
    uint4 rbh[B_PASSES], rbl[B_PASSES];
    const int prow = staged_row(tid), pk = 8 * (tid & 3);

    auto issue_tiles = [&](int k0) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p)
            ra[p].issue(A, lda, row0 + p * 64 + prow, k0 + pk, n, KD, R, ldr);
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int j = p * 64 + prow;
            const size_t off = split_weight_index(col0 + (j < S::BN ? j : 0), k0 + pk, S::BN, ldb / BKB);
            rbh[p] = *reinterpret_cast<const uint4*>(Bh + off);
            rbl[p] = *reinterpret_cast<const uint4*>(Bl + off);
        }
    };
    auto store_tiles = [&](uint16_t* as, uint16_t* bh, uint16_t* bl) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p)
            *reinterpret_cast<uint4*>(&as[(p * 64 + prow) * LDT + pk]) = ra[p].value();
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int j = p * 64 + prow;
            if (j < S::BN) {
                *reinterpret_cast<uint4*>(&bh[j * LDT + pk]) = rbh[p];
                *reinterpret_cast<uint4*>(&bl[j * LDT + pk]) = rbl[p];
            }
        }
    };
    const int li = lane & 31, lk = lane >> 5;
    auto mma_step = [&](const uint16_t* as, const uint16_t* bh, const uint16_t* bl) {
#pragma unroll
        for (int kc = 0; kc < BKB; kc += 16) {
            bf16x8 a[S::TM], h[S::TN], l[S::TN];
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm)
                a[tm] = lds_operand(&as[((wm * S::TM + tm) * 32 + li) * LDT + kc + 8 * lk]);
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn) {
                h[tn] = lds_operand(&bh[((wn * S::TN + tn) * 32 + li) * LDT + kc + 8 * lk]);
                l[tn] = lds_operand(&bl[((wn * S::TN + tn) * 32 + li) * LDT + kc + 8 * lk]);
            }
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < S::TN; ++tn) {
                    // weights as the first operand: the accumulators hold the tile transposed,
                    // a lane then owns one node row and four consecutive columns per register quad
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l[tn], a[tm],
                                                                          acc[tm][tn], 0, 0, 0);
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h[tn], a[tm],
                                                                          acc[tm][tn], 0, 0, 0);
                }
        }
    };

    const int nk = (KD + BKB - 1) / BKB;
    // every row of the tile exists, 32-bit offsets inside a tile, and the reduction depth is a
    // whole number of steps or the rows are long enough to read the last step whole (what lies
    // past the depth is cleared on the way to LDS)
    const bool ragged = KD % BKB != 0;
    const bool fast = row0 + S::BM <= n && lda < (1 << 22) && ldr < (1 << 22) &&
                      (!ragged || ((int64_t)nk * BKB <= lda && (!MASK || (int64_t)nk * BKB <= ldr)));
    if (fast) {
        uint4 km;
        {
            const int left = KD - (nk - 1) * BKB - pk;  // elements of this thread's piece inside
            const auto word = [&](int w) {
                return (left > 2 * w ? 0x0000FFFFu : 0u) | (left > 2 * w + 1 ? 0xFFFF0000u : 0u);
            };
            km = make_uint4(word(0), word(1), word(2), word(3));
        }
        // writes the staged step to LDS; the last step of a ragged depth goes through the mask
        auto put = [&](const FastStage<S, MASK>& st, int step, uint16_t* as, uint16_t* bhs,
                       uint16_t* bls) {
            if (ragged && step == nk - 1) st.template store<true>(as, bhs, bls, km);
            else st.template store<false>(as, bhs, bls);
        };
        // Loads beyond the last step repeat it (never stored), so that no load is conditional.
        FastStage<S, MASK> st0;
        st0.init(tid, (uint32_t)lda * 2u, (uint32_t)ldr * 2u);
        const char* a0 = reinterpret_cast<const char*>(A + row0 * lda);
        const char* r0 = MASK ? reinterpret_cast<const char*>(R + row0 * ldr) : nullptr;
        const size_t tile0 = split_weight_index(col0, 0, S::BN, ldb / BKB);
        const char* bh0 = reinterpret_cast<const char*>(Bh + tile0);
        const char* bl0 = reinterpret_cast<const char*>(Bl + tile0);
        auto load = [&](FastStage<S, MASK>& st, int step) {
            const size_t sc = (size_t)(step < nk ? step : nk - 1);
            const size_t o = sc * (BKB * 2), ob = sc * (S::BN * BKB * 2);
            st.load(a0 + o, r0 + o, bh0 + ob, bl0 + ob, (size_t)lda * 2, (size_t)ldr * 2);
        };
        if constexpr (!kDouble) {
            // one set of tiles: the loads of the next step are in flight during the products
            load(st0, 0);
            for (int i = 0; i < nk; ++i) {
                put(st0, i, As[0], Bhs[0], Bls[0]);
                load(st0, i + 1);
                __syncthreads();
                mma_step(As[0], Bhs[0], Bls[0]);
                __syncthreads();  // before the next step's tiles overwrite these
            }
        } else {
            // two sets of tiles, one barrier per step, loads one step ahead
            load(st0, 0);
            put(st0, 0, As[0], Bhs[0], Bls[0]);
            __syncthreads();
            int i = 0;
            for (; i + 2 < nk; i += 2) {
                load(st0, i + 1);
                mma_step(As[0], Bhs[0], Bls[0]);
                put(st0, i + 1, As[1], Bhs[1], Bls[1]);
                __syncthreads();
                load(st0, i + 2);
                mma_step(As[1], Bhs[1], Bls[1]);
                put(st0, i + 2, As[0], Bhs[0], Bls[0]);
                __syncthreads();
            }
            if (nk - i == 2) {
                load(st0, i + 1);
                mma_step(As[0], Bhs[0], Bls[0]);
                put(st0, i + 1, As[1], Bhs[1], Bls[1]);
                __syncthreads();
                mma_step(As[1], Bhs[1], Bls[1]);
            } else {
                mma_step(As[0], Bhs[0], Bls[0]);
            }
        }
    } else {
        issue_tiles(0);
        if constexpr (!kDouble) {
            for (int i = 0; i < nk; ++i) {
                store_tiles(As[0], Bhs[0], Bls[0]);
                if (i + 1 < nk) issue_tiles((i + 1) * BKB);
                __syncthreads();
                mma_step(As[0], Bhs[0], Bls[0]);
                __syncthreads();
            }
        } else {
            store_tiles(As[0], Bhs[0], Bls[0]);
            __syncthreads();
            for (int i = 0; i < nk; ++i) {
                const int cur = i & 1;
                if (i + 1 < nk) issue_tiles((i + 1) * BKB);
                mma_step(As[cur], Bhs[cur], Bls[cur]);
                if (i + 1 < nk) store_tiles(As[cur ^ 1], Bhs[cur ^ 1], Bls[cur ^ 1]);
                __syncthreads();
            }
        }
    }

    // Accumulator layout (transposed product): lane l, register v -> node row l % 32, column
    // 8 (v / 4) + 4 (l / 32) + v % 4 of the 32 x 32 tile.
    // Converted in pairs by the hardware, collected in LDS and written as 8-byte pieces of whole
    // rows (a lane's own elements lie in 32 different rows: written directly they would be
    // 2-byte stores scattered over as many lines).
    __syncthreads();  // every wave is done with the operand tiles
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < S::TN; ++tn)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // ReLU on the fp32 sums, one maximum per element (on the packed pairs it took six
                // instructions per word, a third of this kernel's vector work)
                float e0 = acc[tm][tn][4 * g], e1 = acc[tm][tn][4 * g + 1];
                float e2 = acc[tm][tn][4 * g + 2], e3 = acc[tm][tn][4 * g + 3];
                if (RELU) {
                    e0 = fmaxf(e0, 0.f);
                    e1 = fmaxf(e1, 0.f);
                    e2 = fmaxf(e2, 0.f);
                    e3 = fmaxf(e3, 0.f);
                }
                const uint32_t w0 = pack_bf16(e0, e1);
                const uint32_t w1 = pack_bf16(e2, e3);
                const uintx2 v = {w0, w1};
                *(lds_uintx2*)(smem + ((wm * S::TM + tm) * 32 + li) * LDC + (wn * S::TN + tn) * 32 +
                               8 * g + 4 * lk) = v;
            }
    __syncthreads();
    constexpr int CPR = S::BN / 4;     // 8-byte pieces per row
    constexpr int RPP = kBlock / CPR;  // rows per pass of the block
    const int crow = tid / CPR, cpiece = tid % CPR;
    const int c = col0 + 4 * cpiece;
    const int c_valid = c < MD ? (MD - c < 4 ? MD - c : 4) : 0;  // columns of the piece inside C
    if (c_valid == 0) return;
    uint16_t* cbase = C + row0 * ldc + c;
    const int64_t rows_left = n - row0;
#pragma unroll
    for (int p = 0; p < S::BM / RPP; ++p) {
        const int r = p * RPP + crow;
        if (r >= rows_left) break;
        const uintx2 v = *(const lds_uintx2*)(smem + r * LDC + 4 * cpiece);
        uint16_t* dst = cbase + (int64_t)r * ldc;
        if (c_valid == 4) {
            *reinterpret_cast<uint2*>(dst) = make_uint2(v.x, v.y);
        } else {
            dst[0] = (uint16_t)v.x;
            if (c_valid > 1) dst[1] = (uint16_t)(v.x >> 16);
            if (c_valid > 2) dst[2] = (uint16_t)v.y;
        }
    }
}

// C[n x out_dim] = (A (.) mask)[n x red_dim] * Wop, Wop[kk][j] = transpose_w ? W[kk][j] : W[j][kk]
template <class S>
int launch_rowblock_bf16(bool relu, const uint16_t* A, int64_t lda, const float* W, int64_t ldw,
                         int w_rows, int w_cols, bool transpose_w, uint16_t* C, int64_t ldc,
                         int64_t n, int red_dim, int out_dim, const uint16_t* R, int64_t ldr,
                         hipStream_t s)
{
    const int nct = (int)ceil_div(out_dim, S::BN);
    const int64_t grid = ceil_div(n, S::BM) * nct;
    if (grid <= 0) return MIXGCN_OK;
    if (grid > 0x7FFFFFFF) return fail(MIXGCN_EINVAL, "update: too many row tiles");
    const int out_rows = nct * S::BN, out_cols = (int)ceil_div(red_dim, BKB) * BKB;
    void* scratch = nullptr;
    MIXGCN_TRY(get_scratch(3, (size_t)2 * out_rows * out_cols * sizeof(uint16_t), &scratch));
    uint16_t* hi = (uint16_t*)scratch;
    uint16_t* lo = hi + (size_t)out_rows * out_cols;
    hipLaunchKernelGGL(split_weights_kernel, dim3((unsigned)ceil_div(out_rows * out_cols, kBlock)),
                       dim3(kBlock), 0, s, W, ldw, w_rows, w_cols, transpose_w ? 1 : 0, hi, lo,
                       out_rows, out_cols, S::BN);
#define MIXGCN_ROWBLOCK(RELU, MASK)                                                              \
    hipLaunchKernelGGL((rowblock_bf16_kernel<S, RELU, MASK>), dim3((unsigned)grid), dim3(kBlock), \
                       0, s, A, lda, hi, lo, out_cols, C, ldc, n, red_dim, out_dim, R, ldr, nct)
    if (R) MIXGCN_ROWBLOCK(false, true);
    else if (relu) MIXGCN_ROWBLOCK(true, false);
    else MIXGCN_ROWBLOCK(false, false);
#undef MIXGCN_ROWBLOCK
    return MIXGCN_OK;
}

}  // namespace

int launch_update_bf16_deep(bool w_is_kd_major, bool relu, const uint16_t* A, int64_t lda, const float* W,
                            int64_t ldw, uint16_t* C, int64_t ldc, int64_t n, int KD, int MD,
                            const uint16_t* R, int64_t ldr, hipStream_t s)
{
    const int w_rows = w_is_kd_major ? KD : MD, w_cols = w_is_kd_major ? MD : KD;
    if (MD > 64)
        MIXGCN_TRY((launch_rowblock_bf16<Shape128x128>(relu, A, lda, W, ldw, w_rows, w_cols, w_is_kd_major, C, ldc,
                                                      n, KD, MD, R, ldr, s)));
    else
        MIXGCN_TRY((launch_rowblock_bf16<Shape128x32>(relu, A, lda, W, ldw, w_rows, w_cols, w_is_kd_major, C, ldc,
                                                     n, KD, MD, R, ldr, s)));
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

}  // namespace mixgcn
