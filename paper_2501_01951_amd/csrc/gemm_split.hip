// Weight gradient of fp32 features (paper Algorithm 2, update phase) on the bf16 matrix cores.  Every
// fp32 operand is written as the exact sum of three bf16 terms (round to nearest at each stage),
//     x = x0 + x1 + x2,   |x1| <= 2^-8 |x|,   |x2| <= 2^-16 |x|,
// and a product a b is accumulated in fp32 from the six partial products of order 2^-16 and
// above: a2 b0, a0 b2, a1 b1, a1 b0, a0 b1, a0 b0, smallest first.  The three dropped ones are
// together below 2^-23 |a| |b|, the size of one fp32 rounding.
//
// Sums.  The matrix cores do not round to nearest: their sums are too low by 9e-9 of a step's partial sum on
// average, whatever the sign, and over 2^20 rows that adds up to three times the error of fp32 MFMAs.  So the
// partial products of a step of 16 rows are added up from zero, added to the running sum by the vector units,
// and odd steps are computed of the negated features and subtracted: what is lost cancels.  Relative error of
// dW against 64 bits, normal inputs, 2^20 rows 128 x 256: 2.1e-7 (without the negation 2.3e-6, fp32 MFMAs
// 5.8e-7); 11.1 M rows 128 x 128: 4.7e-7 (7.1e-6, 1.9e-6); 4096 rows 64 x 32: 0.7e-7 (fp32 MFMAs 2.1e-7).
//
// Pipeline of a tile: global loads run two steps ahead in two register sets, LDS is double buffered, one
// barrier per step; the split of the next step's tile and the products of this one are independent of each
// other.  Rows past a slab's end are read as zeros, so that the loop has no conditional load or store.
//
// What bounds it: memory on the wide layers (2^21 rows 128 x 1024 reads and masks 18.2 GB at 4.7 TB/s, a
// streaming read reaches 5.7), vector work of the splits and the sums (175 instructions beside 24 MFMAs) where
// a tile has both operands to itself.  us, fp32 MFMAs -> now: 2^20 rows 128 x 256 761 -> 619, 256 x 256
// 1280 -> 863, 256 x 47 574 -> 365, 256 x 16 315 -> 282; 2^21 rows 128 x 1024 5100 -> 3900; 11.1 M rows
// 128 x 128 3170 -> 2520; 232965 rows 602 x 128 458 -> 331; 4096 rows 64 x 100 19.7 -> 15.2.
#include <type_traits>

#include "gemm_common.h"
#include "internal.h"

namespace mixgcn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int BKS = 16;       // node rows per step = the reduction depth of one MFMA
constexpr int kPlanes = 3;

// ---- weight gradient: P[slab][KD x MD] = A[rows of slab][KD]^T * (B (.) 1[R > 0])[rows][MD] -----
// The reduction runs over node rows, the slow index of both operands in memory, while the bf16
// MFMA wants eight consecutive reduction indices per lane.  The tiles are therefore staged as
// they lie (row-major [node row][feature], three bf16 planes each, plain 8-byte writes) and the
// transposition is done by the LDS read: ds_read_b64_tr_b16 hands lane i of a group of 16 lanes
// element i % 4 of the 8 bytes addressed by lanes i / 4, i / 4 + 4, i / 4 + 8 and i / 4 + 12, so
// with lane s of the group pointing at row s / 4, features 4 (s % 4) .. + 3, every lane receives
// its own feature at four consecutive rows; two such reads are one MFMA operand.
// LDS rows are 320 bytes (128 features + pad): two groups of 16 lanes are served together (64
// banks), that is four rows of 64 bytes, which a pitch of 16 banks modulo 64 keeps apart (with
// 288-byte rows a third of the LDS cycles were bank conflicts).
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
constexpr int LDW = 128 + 32;            // halfwords per staged row
constexpr int kWPlane = BKS * LDW;       // halfwords per plane of a tile

__device__ inline bf16x8 read_transposed(const uint16_t* p)
{
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)p);
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + 4 * LDW));
    const shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 o;
    __builtin_memcpy(&o, &v, 16);
    return o;
}

// Sixteen bytes at a byte offset of a step's rows; zeros where the step has no such row.
__device__ inline float4 load16(__amdgpu_buffer_rsrc_t rows, uint32_t offset)
{
    const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)offset, 0, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}

// The rows of a step, `bytes` of them from `first` on, as a buffer: what lies past the slab's end is read as
// zeros, a step past the end reads nothing, and no load is conditional.
__device__ inline __amdgpu_buffer_rsrc_t rows_at(const char* first, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(first), 0, bytes, 0x00020000);
}

// FAR: a step of 16 rows does not fit a buffer with 32-bit offsets (pitches of 2^22 elements and more).  The
// same tiles, slabs and order with 64-bit addresses: the arithmetic does not depend on the pitch.
// BITS: the mask goes to `bits` too (see ReluBits), each byte once, by the tiles of the first 128 features (2^21 rows
// 128 x 1024 3900 -> 4200 us; the data gradient that reads it instead of R 4580 -> 3780).
template <int BN, bool MASK, bool FAR, bool BITS>
__global__ __launch_bounds__(kBlock, 2) void wgrad_split_kernel(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    const float* __restrict__ R, int64_t ldr, float* __restrict__ P, int KD, int MD,
    int64_t rows_per_slab, int64_t n_rows, int n_i_tiles, int n_j_tiles, ReluBits bits)
{
    // tile of 128 x BN: 2 x 2 wavefronts of 64 x BN / 2, or (32 columns) four of 32 x 32
    constexpr int WN = BN > 32 ? 2 : 1, TM = BN > 32 ? 2 : 1, TN = BN / WN / 32;
    constexpr int PB = BN == 128 ? 2 : 1;  // pieces of B per thread and step
    __shared__ __attribute__((aligned(16))) uint16_t As[2][kPlanes * kWPlane];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kPlanes * kWPlane];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int tiles = n_i_tiles * n_j_tiles;
    const unsigned lid = xcd_local_index(blockIdx.x, gridDim.x);
    // (scalar: the division is done in vector registers, and a buffer in those is loaded from in a loop)
    const int slab = __builtin_amdgcn_readfirstlane((int)(lid / (unsigned)tiles));
    const int t = __builtin_amdgcn_readfirstlane((int)(lid % (unsigned)tiles));
    const int i0 = (t / n_j_tiles) * 128, j0 = (t % n_j_tiles) * BN;
    const int64_t r_begin = slab * rows_per_slab;
    const int64_t r_end = (r_begin + rows_per_slab) < n_rows ? (r_begin + rows_per_slab) : n_rows;
    int left = __builtin_amdgcn_readfirstlane((int)(r_end - r_begin));  // rows from the load cursor on
    const int nk = (left + BKS - 1) / BKS;

    floatx16 acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;
    };
    clear();

    // staging: thread -> rows tid / 32 and tid / 32 + 8 of the step, features 4 (tid % 32) .. + 3 (fewer
    // columns of B: a row each; of 32 columns the second half of the threads repeats the first).  Features
    // past the matrix reach only cells of the product that are not stored: any column of the row will do.
    const int srow = tid >> 5, scol = 4 * (tid & 31);
    const int trow = tid / (BN / 4) % BKS, tcol = 4 * (tid % (BN / 4));
    const int acol = i0 + (i0 + scol < KD ? scol : 0), bcol = j0 + (j0 + tcol < MD ? tcol : 0);
    uint32_t aoff[2], boff[PB], roff[PB];
#pragma unroll
    for (int p = 0; p < 2; ++p) aoff[p] = (uint32_t)(srow + 8 * p) * (uint32_t)lda * 4u + 4u * acol;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        boff[p] = (uint32_t)(trow + 8 * p) * (uint32_t)ldb * 4u + 4u * bcol;
        roff[p] = MASK ? (uint32_t)(trow + 8 * p) * (uint32_t)ldr * 4u + 4u * bcol : 0u;
    }
    const int spos = srow * LDW + scol, tpos = trow * LDW + tcol;

    struct Regs {
        float4 a[2], b[PB], r[MASK ? PB : 1];
    };
    const char* ap = reinterpret_cast<const char*>(A + r_begin * lda);
    const char* bp = reinterpret_cast<const char*>(B + r_begin * ldb);
    const char* rp = MASK ? reinterpret_cast<const char*>(R + r_begin * ldr) : nullptr;
    const int pa = (int)lda * 4, pb = (int)ldb * 4, pr = (int)ldr * 4;
    // Four values of row `row` of the step at the load cursor, zeros past the slab's end (FAR; the slab's first
    // row exists)
    auto load_far = [&](const float* M, int64_t ld, int row, int col) {
        const bool in = row < left;
        const float4 v = *reinterpret_cast<const float4*>(M + (in ? r_end - left + row : r_begin) * ld + col);
        return in ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    auto load = [&](Regs& g) {
        if (FAR) {
#pragma unroll
            for (int p = 0; p < 2; ++p) g.a[p] = load_far(A, lda, srow + 8 * p, acol);
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                g.b[p] = load_far(B, ldb, trow + 8 * p, bcol);
                if (MASK) g.r[MASK ? p : 0] = load_far(R, ldr, trow + 8 * p, bcol);
            }
            left -= BKS;
            return;
        }
        const int rows = __builtin_amdgcn_readfirstlane(left >= BKS ? BKS : left > 0 ? left : 0);
        const auto ra = rows_at(ap, rows * pa), rb = rows_at(bp, rows * pb);
#pragma unroll
        for (int p = 0; p < 2; ++p) g.a[p] = load16(ra, aoff[p]);
#pragma unroll
        for (int p = 0; p < PB; ++p) g.b[p] = load16(rb, boff[p]);
        if (MASK) {
            const auto rr = rows_at(rp, rows * pr);
#pragma unroll
            for (int p = 0; p < PB; ++p) g.r[MASK ? p : 0] = load16(rr, roff[p]);
            rp += (int64_t)BKS * pr;
        }
        ap += (int64_t)BKS * pa;
        bp += (int64_t)BKS * pb;
        left -= BKS;
    };
    // The bytes of a step's mask.  What lies past the slab's end or the columns is outside the buffer: not stored.
    int bits_left = BITS && i0 == 0 ? left : 0;  // rows from the store cursor on
    char* bits_row = BITS ? reinterpret_cast<char*>(bits.p + r_begin * bits.pitch) : nullptr;
    const uint32_t bits_col = j0 + tcol < MD ? (uint32_t)(j0 + tcol) / 4 : 0x7FFF0000u;
    auto put_bits = [&](const Regs& g) {
        const int rows = __builtin_amdgcn_readfirstlane(bits_left >= BKS ? BKS : bits_left > 0 ? bits_left : 0);
        const auto out = rows_at(bits_row, rows * (int)bits.pitch);
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const float4 r = g.r[MASK ? p : 0];
            const int b = (r.x > 0.f ? 1 : 0) | (r.y > 0.f ? 2 : 0) | (r.z > 0.f ? 4 : 0) | (r.w > 0.f ? 8 : 0);
            __builtin_amdgcn_raw_buffer_store_b8(
                (uint8_t)b, out, (int)((uint32_t)(trow + 8 * p) * (uint32_t)bits.pitch + bits_col), 0, 0);
        }
        bits_row += BKS * bits.pitch;
        bits_left -= BKS;
    };
    auto store = [&](const Regs& g, uint16_t* as, uint16_t* bs, auto odd) {
        if (BITS) put_bits(g);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint16_t* qa = as + spos + p * 8 * LDW;
            split_store<false>(g.a[p], g.a[p], decltype(odd)::value ? -kTermScale : kTermScale, qa, qa + kWPlane,
                               qa + 2 * kWPlane);
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            uint16_t* qb = bs + tpos + p * 8 * LDW;
            split_store<MASK>(g.b[p], g.r[MASK ? p : 0], kTermScale, qb, qb + kWPlane, qb + 2 * kWPlane);
        }
    };
    // operand reads: lane -> 16-lane group (feature block, reduction half), place in the group
    const int grp = lane >> 4, gs = lane & 15;
    const int rpos = (8 * (grp >> 1) + (gs >> 2)) * LDW + 16 * (grp & 1) + 4 * (gs & 3);
    // The partial products of a step are added up from zero and then to the running sum, once per step.
    auto mma = [&](const uint16_t* as, const uint16_t* bs, auto odd) {
        constexpr int qa[6] = {2, 0, 1, 1, 0, 0};
        constexpr int qb[6] = {0, 2, 1, 0, 1, 0};
        bf16x8 a[TM][kPlanes], b[TN][kPlanes];
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                b[tn][p] = read_transposed(bs + p * kWPlane + rpos + (wn * TN + tn) * 32);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                a[tm][p] = read_transposed(as + p * kWPlane + rpos + (wm * TM + tm) * 32);
        }
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            floatx16 part[TN];
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    const floatx16 zero = {};
                    part[tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[tm][qa[q]], b[tn][qb[q]],
                                                                       q == 0 ? zero : part[tn], 0, 0, 0);
                }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[tm][tn][v] += decltype(odd)::value ? -part[tn][v] : part[tn][v];
        }
    };

    if (nk > 0) {
        constexpr std::false_type even{};
        constexpr std::true_type odd{};
        Regs g0, g1;
        load(g0);
        load(g1);
        store(g0, As[0], Bs[0], even);
        load(g0);
        __syncthreads();
        for (int i = 0; i + 1 < nk; i += 2) {
            store(g1, As[1], Bs[1], odd);
            load(g1);
            mma(As[0], Bs[0], even);
            __syncthreads();
            store(g0, As[0], Bs[0], even);
            load(g0);
            mma(As[1], Bs[1], odd);
            __syncthreads();
        }
        if (nk & 1) mma(As[0], Bs[0], even);
    }

    // D layout: lane l, register v -> row 8 (v / 4) + 4 (l / 32) + v % 4, col l % 32
    const int li = lane & 31, lk = lane >> 5;
    const int iw = i0 + wm * TM * 32, jw = j0 + wn * TN * 32;
    float z = 0.f;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool in = iw + tm * 32 + 8 * (v / 4) + 4 * lk + (v % 4) < KD && jw + tn * 32 + li < MD;
                z = fmaf(in ? acc[tm][tn][v] : 0.f, 0.f, z);
            }
    float unscale = 1.f / (kTermScale * kTermScale);
    if (__builtin_expect(r_end - r_begin < 4 || __any(!(z == 0.f)), 0)) {
        // A sum that is not finite (a term of an infinity is NaN, a value next to the largest float rounds
        // up to an infinity), or fewer than four rows, over which a chain of fp32 multiply-adds is closer to
        // 64 bits: the wavefront's tile again on the fp32 matrix cores, straight from memory.
        // 32x32x2: lane l supplies column l % 32 of reduction index l / 32.
        clear();
        unscale = 1.f;
        int ca[TM], cb[TN];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) ca[tm] = iw + tm * 32 + li < KD ? iw + tm * 32 + li : i0;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) cb[tn] = jw + tn * 32 + li < MD ? jw + tn * 32 + li : j0;
        for (int64_t r = r_begin; r < r_end; r += 2) {
            const bool in = r + lk < r_end;
            const int64_t row = in ? r + lk : r;
            float a[TM], b[TN];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const float x = A[row * lda + ca[tm]];
                a[tm] = in ? x : 0.f;
            }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const float x = B[row * ldb + cb[tn]];
                b[tn] = in && (!MASK || R[row * ldr + cb[tn]] > 0.f) ? x : 0.f;
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[tm], b[tn], acc[tm][tn], 0, 0, 0);
        }
    }

    float* out = P + (size_t)slab * KD * MD;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int j = jw + tn * 32 + li;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = iw + tm * 32 + 8 * (v / 4) + 4 * lk + (v % 4);
                if (i < KD && j < MD) out[(size_t)i * MD + j] = acc[tm][tn][v] * unscale;
            }
        }
}

}  // namespace

// dW[k x m] = beta dW + A[n x k]^T (B (.) mask)[n x m]
int launch_wgrad_split(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc, int64_t n,
                       int32_t k, int32_t m, const float* R, int64_t ldr, float beta, hipStream_t s, Timer* timer,
                       ReluBits bits)
{
    // The narrowest tile that holds the columns (2^20 rows 256 x 47: 508 us with 128 columns, 360 with 64;
    // 256 x 16: 333 with 64, 282 with 32).
    const int bn = m > 64 ? 128 : m > 32 ? 64 : 32;
    const int nit = (int)ceil_div(k, 128), njt = (int)ceil_div(m, bn), tiles = nit * njt;
    int64_t n_slabs = wgrad_slabs(n, tiles, 1024);
    int64_t rows_per_slab = ceil_div(ceil_div(n, n_slabs), BKS) * BKS;
    if (rows_per_slab < BKS) rows_per_slab = BKS;
    n_slabs = n > 0 ? ceil_div(n, rows_per_slab) : 1;  // without rows: one slab of zeros
    const bool far = lda >= (1 << 22) || ldb >= (1 << 22) || (R && ldr >= (1 << 22));
    if (bits.p && (!R || far || bn < 128)) return fail(MIXGCN_EINVAL, "update: mask bits");
    const int64_t cells = (int64_t)k * m;
    void* scratch = nullptr;
    MIXGCN_TRY(get_scratch(0, (size_t)n_slabs * cells * sizeof(float), &scratch));
    float* P = (float*)scratch;
    const unsigned grid = (unsigned)(n_slabs * tiles);
    if (timer) MIXGCN_TRY(timer->begin(kTimeUpdateWgrad, s));
#define MIXGCN_WGRAD(BN, MASK, FAR, BITS)                                                                        \
    hipLaunchKernelGGL((wgrad_split_kernel<BN, MASK, FAR, BITS>), dim3(grid), dim3(kBlock), 0, s, A, lda, B, ldb, R, \
                       ldr, P, k, m, rows_per_slab, n, nit, njt, bits)
#define MIXGCN_WGRAD_MASK(BN)                                            \
    do {                                                                 \
        if (R && far) MIXGCN_WGRAD(BN, true, true, false);               \
        else if (R) MIXGCN_WGRAD(BN, true, false, false);                \
        else if (far) MIXGCN_WGRAD(BN, false, true, false);              \
        else MIXGCN_WGRAD(BN, false, false, false);                      \
    } while (0)
    if (bits.p) MIXGCN_WGRAD(128, true, false, true);
    else if (bn == 128) MIXGCN_WGRAD_MASK(128);
    else if (bn == 64) MIXGCN_WGRAD_MASK(64);
    else MIXGCN_WGRAD_MASK(32);
#undef MIXGCN_WGRAD_MASK
#undef MIXGCN_WGRAD
    if (timer) MIXGCN_TRY(timer->end(s));
    MIXGCN_TRY(launch_wgrad_reduce(P, n_slabs, cells, m, C, ldc, beta, s));
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

}  // namespace mixgcn
