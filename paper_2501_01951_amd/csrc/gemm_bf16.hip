// Weight gradient of bf16-stored features (paper Algorithm 2, update phase) on the bf16 matrix cores:
// v_mfma_f32_32x32x16_bf16, fp32 accumulation.  Activations and gradients are bf16 in memory and enter
// the MFMA as they are.
//
// MFMA 32x32x16 operand layout: lane l supplies A[i = l % 32][k = 8 (l / 32) + 0..7] and
// B[k = 8 (l / 32) + 0..7][j = l % 32] as eight consecutive bf16; D as for the fp32 32x32 MFMA.
#include "gemm_bf16_tiles.h"
#include "internal.h"

namespace mixgcn {
namespace {

// ---- slab kernel: P[slab][KD x MD] = A[rows of slab][KD]^T * (B (.) 1[R > 0])[rows][MD] --------
// The reduction runs over node rows, which is the slow index of both operands in memory, so a
// tile is transposed on its way into LDS: a thread takes the same eight columns of two
// consecutive rows and writes eight 32-bit words, each holding one column's pair of rows.
template <class S, bool MASK>
__global__ __launch_bounds__(kBlock) void wgrad_bf16_kernel(
    const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B, int64_t ldb,
    const uint16_t* __restrict__ R, int64_t ldr, float* __restrict__ P, int64_t n, int KD, int MD,
    int64_t rows_per_slab, int n_i_tiles, int n_j_tiles)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[2][S::BM * LDT];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][S::BN * LDT];
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

    // 16 row pairs x (tile width / 8) column groups per step; one block pass covers 16 groups
    constexpr int A_PASSES = S::BM / 128 > 0 ? S::BM / 128 : 1;
    constexpr int B_PASSES = S::BN / 128 > 0 ? S::BN / 128 : 1;
    const int rp = tid / 16, cg = tid % 16;
    Piece8<false> a0[A_PASSES], a1[A_PASSES];
    Piece8<MASK> b0[B_PASSES], b1[B_PASSES];

    auto issue_tiles = [&](int64_t r0) {
        const int64_t ra = r0 + 2 * rp;
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int c = 8 * (p * 16 + cg);
            const int cc = c < S::BM ? c : 0;
            a0[p].issue(A, lda, ra, i0 + cc, r_end, KD, nullptr, 0);
            a1[p].issue(A, lda, ra + 1, i0 + cc, r_end, KD, nullptr, 0);
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int c = 8 * (p * 16 + cg);
            const int cc = c < S::BN ? c : 0;
            b0[p].issue(B, ldb, ra, j0 + cc, r_end, MD, R, ldr);
            b1[p].issue(B, ldb, ra + 1, j0 + cc, r_end, MD, R, ldr);
        }
    };
    // words of the two rows -> LDS[(column)][row pair]
    auto scatter = [&](uint16_t* tile, int c, const uint4& x, const uint4& y) {
        uint32_t* t32 = reinterpret_cast<uint32_t*>(tile);
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            t32[(c + 2 * w) * (LDT / 2) + rp] = (xs[w] & 0xFFFFu) | (ys[w] << 16);
            t32[(c + 2 * w + 1) * (LDT / 2) + rp] = (xs[w] >> 16) | (ys[w] & 0xFFFF0000u);
        }
    };
    auto store_tiles = [&](uint16_t* as, uint16_t* bs) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int c = 8 * (p * 16 + cg);
            if (c < S::BM) scatter(as, c, a0[p].value(), a1[p].value());
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int c = 8 * (p * 16 + cg);
            if (c < S::BN) scatter(bs, c, b0[p].value(), b1[p].value());
        }
    };
    const int li = lane & 31, lk = lane >> 5;
    auto mma_step = [&](const uint16_t* as, const uint16_t* bs) {
#pragma unroll
        for (int kc = 0; kc < BKB; kc += 16) {
            bf16x8 a[S::TM], b[S::TN];
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm)
                a[tm] = lds_operand(&as[((wm * S::TM + tm) * 32 + li) * LDT + kc + 8 * lk]);
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn)
                b[tn] = lds_operand(&bs[((wn * S::TN + tn) * 32 + li) * LDT + kc + 8 * lk]);
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < S::TN; ++tn)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[tm], b[tn],
                                                                          acc[tm][tn], 0, 0, 0);
        }
    };

    if (r_begin < r_end) {
        const int64_t nk = (r_end - r_begin + BKB - 1) / BKB;
        issue_tiles(r_begin);
        store_tiles(As[0], Bs[0]);
        __syncthreads();
        for (int64_t i = 0; i < nk; ++i) {
            const int cur = (int)(i & 1);
            if (i + 1 < nk) issue_tiles(r_begin + (i + 1) * BKB);
            mma_step(As[cur], Bs[cur]);
            if (i + 1 < nk) store_tiles(As[cur ^ 1], Bs[cur ^ 1]);
            __syncthreads();
        }
    }
    float* out = P + (size_t)slab * KD * MD;
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

// ---- the same product without the scattered LDS writes -------------------------------------------
// (In the kernel above the transposing 4-byte writes keep the LDS busy 80 % of the time, seven
// eighths of it with bank conflicts.)  Here the tiles are staged as they lie, row-major
// [node row][feature] with 16-byte copies, and the LDS read transposes: ds_read_b64_tr_b16 hands
// lane i of a group of 16 lanes element i % 4 of the 8 bytes addressed by lanes i / 4, i / 4 + 4,
// i / 4 + 8 and i / 4 + 12, so with lane s of the group pointing at row s / 4, features
// 4 (s % 4) .. + 3, every lane receives its own feature at four consecutive rows, and two such
// reads are one MFMA operand.  Two groups are served per cycle from 64 banks (four rows of 64
// bytes): a row pitch of 64 bytes modulo 256 keeps them apart.  Rows come in whole steps of 32; the last n % 32
// rows are a slab of their own with one step, whose other rows are zeros (the kernel above in a launch of its own took
// 6 us for them: a weight gradient of 100003 rows 128 x 128 25 -> 19.6 us, 128 x 16 17 -> 13).  Features beyond the
// matrices are zeroed with per-thread masks that do not change from step to step.
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;

template <int PITCH>
__device__ inline bf16x8 read_transposed(const uint16_t* p)
{
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)p);
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + 4 * PITCH));
    const shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 o;
    __builtin_memcpy(&o, &v, 16);
    return o;
}

template <class S, bool MASK>
__global__ __launch_bounds__(kBlock, S::BN == 128 ? 3 : 5) void wgrad_bf16_tr_kernel(
    const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B, int64_t ldb,
    const uint16_t* __restrict__ R, int64_t ldr, float* __restrict__ P, int64_t n_main, int64_t n, int KD, int MD,
    int64_t rows_per_slab, int n_i_tiles, int n_j_tiles)
{
    static_assert(S::BM == 128 && (S::BN == 128 || S::BN == 32), "tile shapes of the staging");
    constexpr int PA = 128 + 32;                         // halfwords per staged row of A
    constexpr int PB = S::BN == 128 ? 128 + 32 : 32;     // ... of B
    constexpr int B_PPR = S::BN / 8;                     // 16-byte pieces per row of B
    constexpr int B_RPP = kBlock / B_PPR;                // rows per pass of the block
    constexpr int B_PASSES = B_RPP >= BKB ? 1 : BKB / B_RPP;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][BKB * PA];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BKB * PB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const int tiles = n_i_tiles * n_j_tiles;
    // The workgroups of the rest come behind the others, which keep their even deal to the XCDs: one more on an XCD whose
    // compute units have as many each as fit evenly costs what one of the others takes (2450000 rows 256 x 64 masked,
    // 1024 workgroups and 4: 522 us, this way 435)
    const unsigned main_grid = gridDim.x - (n > n_main ? (unsigned)tiles : 0u);
    const unsigned lid = blockIdx.x < main_grid ? xcd_local_index(blockIdx.x, main_grid) : blockIdx.x;
    const int slab = __builtin_amdgcn_readfirstlane((int)(lid / (unsigned)tiles));
    const int t = (int)(lid % (unsigned)tiles);
    const int i0 = (t / n_j_tiles) * S::BM, j0 = (t % n_j_tiles) * S::BN;
    // n_main rows in whole steps, then the slab of the others
    const int64_t first = slab * rows_per_slab;
    const int rest = first < n_main ? 0 : (int)(n - n_main);
    const int64_t r_begin = rest ? n_main : first;
    const int64_t r_end = (r_begin + rows_per_slab) < n_main ? (r_begin + rows_per_slab) : n_main;
    const int nk = rest ? 0 : (int)((r_end - r_begin) / BKB);  // whole steps: the caller sees to it

    floatx16 acc[S::TM][S::TN];
#pragma unroll
    for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < S::TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;

    // staging: A rows tid / 16 and tid / 16 + 16, features 8 (tid % 16) .. + 7; B alike with its
    // own pieces per row.  A piece beyond the matrix is loaded from column 0 and masked to zero.
    auto keep_words = [](int nvalid, uint32_t* kw) {
#pragma unroll
        for (int w = 0; w < 4; ++w)
            kw[w] = (nvalid > 2 * w ? 0x0000FFFFu : 0u) | (nvalid > 2 * w + 1 ? 0xFFFF0000u : 0u);
    };
    const int arow = tid >> 4, acol = i0 + 8 * (tid & 15);
    const int a_valid = acol < KD ? (KD - acol < 8 ? KD - acol : 8) : 0;
    uint32_t a_keep[4];
    keep_words(a_valid, a_keep);
    const uint32_t a_off = ((uint32_t)arow * (uint32_t)lda + (uint32_t)(a_valid ? acol : 0)) * 2u;
    const int a_pos = arow * PA + 8 * (tid & 15);
    const int brow = tid / B_PPR, bcol = j0 + 8 * (tid % B_PPR);
    const bool b_on = brow < BKB;
    const int b_valid = bcol < MD ? (MD - bcol < 8 ? MD - bcol : 8) : 0;
    uint32_t b_keep[4];
    keep_words(b_valid, b_keep);
    const int brow_c = b_on ? brow : 0;  // idle threads of a narrow tile load row 0 again
    const uint32_t b_off = ((uint32_t)brow_c * (uint32_t)ldb + (uint32_t)(b_valid ? bcol : 0)) * 2u;
    const uint32_t r_off = MASK ? ((uint32_t)brow_c * (uint32_t)ldr + (uint32_t)(b_valid ? bcol : 0)) * 2u : 0u;
    const int b_pos = brow_c * PB + 8 * (tid % B_PPR);
    const bool inside = i0 + S::BM <= KD && j0 + S::BN <= MD;

    const char* a0 = reinterpret_cast<const char*>(A + r_begin * lda);
    const char* b0 = reinterpret_cast<const char*>(B + r_begin * ldb);
    const char* m0 = MASK ? reinterpret_cast<const char*>(R + r_begin * ldr) : nullptr;
    const size_t step_a = (size_t)BKB * 2 * (size_t)lda, step_b = (size_t)BKB * 2 * (size_t)ldb,
                 step_r = (size_t)BKB * 2 * (size_t)ldr;

    struct Regs {
        uint4 a[2], b[B_PASSES], r[B_PASSES];
    };
    // a step beyond the last one loads the last one again (never stored): no branch around loads
    auto load = [&](Regs& g, int step) {
        const size_t sc = (size_t)(step < nk ? step : nk - 1);
#pragma unroll
        for (int p = 0; p < 2; ++p)
            g.a[p] = *reinterpret_cast<const uint4*>(a0 + sc * step_a + (size_t)p * 16 * 2 * (size_t)lda + a_off);
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            g.b[p] = *reinterpret_cast<const uint4*>(b0 + sc * step_b + (size_t)p * B_RPP * 2 * (size_t)ldb + b_off);
            if (MASK)
                g.r[p] = *reinterpret_cast<const uint4*>(m0 + sc * step_r + (size_t)p * B_RPP * 2 * (size_t)ldr + r_off);
        }
    };
    auto store = [&](const Regs& g, uint16_t* as, uint16_t* bs) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint4 v = g.a[p];
            if (!inside) {
                v.x &= a_keep[0];
                v.y &= a_keep[1];
                v.z &= a_keep[2];
                v.w &= a_keep[3];
            }
            lds_store16(as + a_pos + p * 16 * PA, v);
        }
        if (b_on) {
#pragma unroll
            for (int p = 0; p < B_PASSES; ++p) {
                uint4 v = g.b[p];
                if (MASK) {
                    v.x = keep_positive(v.x, g.r[p].x);
                    v.y = keep_positive(v.y, g.r[p].y);
                    v.z = keep_positive(v.z, g.r[p].z);
                    v.w = keep_positive(v.w, g.r[p].w);
                }
                if (!inside) {
                    v.x &= b_keep[0];
                    v.y &= b_keep[1];
                    v.z &= b_keep[2];
                    v.w &= b_keep[3];
                }
                lds_store16(bs + b_pos + p * B_RPP * PB, v);
            }
        }
    };
    // operand reads: lane -> 16-lane group (feature block, reduction half), place in the group
    const int grp = lane >> 4, gs = lane & 15;
    const int rrow = 8 * (grp >> 1) + (gs >> 2), rcol = 16 * (grp & 1) + 4 * (gs & 3);
    auto step_mma = [&](const uint16_t* as, const uint16_t* bs) {
#pragma unroll
        for (int kc = 0; kc < BKB; kc += 16) {
            bf16x8 a[S::TM], b[S::TN];
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm)
                a[tm] = read_transposed<PA>(as + (kc + rrow) * PA + (wm * S::TM + tm) * 32 + rcol);
#pragma unroll
            for (int tn = 0; tn < S::TN; ++tn)
                b[tn] = read_transposed<PB>(bs + (kc + rrow) * PB + (wn * S::TN + tn) * 32 + rcol);
#pragma unroll
            for (int tm = 0; tm < S::TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < S::TN; ++tn)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[tm], b[tn], acc[tm][tn],
                                                                          0, 0, 0);
        }
    };

    if (nk > 0) {
        // LDS double buffered one step ahead, global loads two steps ahead in two register sets
        Regs g0, g1;
        load(g0, 0);
        load(g1, 1);
        store(g0, As[0], Bs[0]);
        load(g0, 2);
        __syncthreads();
        int i = 0;
        for (; i + 2 < nk; i += 2) {
            step_mma(As[0], Bs[0]);
            store(g1, As[1], Bs[1]);
            load(g1, i + 3);
            __syncthreads();
            step_mma(As[1], Bs[1]);
            store(g0, As[0], Bs[0]);
            load(g0, i + 4);
            __syncthreads();
        }
        step_mma(As[0], Bs[0]);
        if (nk - i == 2) {
            store(g1, As[1], Bs[1]);
            __syncthreads();
            step_mma(As[1], Bs[1]);
        }
    }

    if (rest) {
        Regs g;
        // (a row that does not exist: the first one, times zero)
        auto piece = [](const char* first, size_t at, uint32_t off, bool in) {
            const uint4 v = *reinterpret_cast<const uint4*>(first + (in ? at + off : (size_t)0));
            const uint32_t k = in ? ~0u : 0u;
            return make_uint4(v.x & k, v.y & k, v.z & k, v.w & k);
        };
#pragma unroll
        for (int p = 0; p < 2; ++p) g.a[p] = piece(a0, (size_t)p * 16 * 2 * (size_t)lda, a_off, arow + p * 16 < rest);
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const bool in = brow_c + p * B_RPP < rest;
            g.b[p] = piece(b0, (size_t)p * B_RPP * 2 * (size_t)ldb, b_off, in);
            if (MASK) g.r[p] = piece(m0, (size_t)p * B_RPP * 2 * (size_t)ldr, r_off, in);
        }
        store(g, As[0], Bs[0]);
        __syncthreads();
        step_mma(As[0], Bs[0]);
    }

    const int li = lane & 31, lk = lane >> 5;
    float* out = P + (size_t)slab * KD * MD;
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

}  // namespace

int launch_wgrad_bf16(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, float* C, int64_t ldc,
                      int64_t n, int32_t k, int32_t m, const uint16_t* R, int64_t ldr, float beta,
                      hipStream_t s, Timer* timer)
{
    // C[k x m] = beta C + A[n x k]^T (B (.) mask)[n x m]: with the transposing LDS reads, the last n % 32 rows too where
    // their slab fits the scratch; pitches that 32-bit offsets do not reach with the scattering kernel
    const bool wide = m > 64;
    const int bm = 128, bn = wide ? 128 : 32;
    const int nit = (int)ceil_div(k, bm), njt = (int)ceil_div(m, bn);
    const int tiles = nit * njt;
    const int64_t cells = (int64_t)k * m;
    const bool pitches_ok = lda < (1 << 25) && ldb < (1 << 25) && ldr < (1 << 25);
    const int64_t n_main = pitches_ok ? n - n % BKB : 0;
    struct Part {
        int64_t rows = 0, slabs = 0, rows_per_slab = BKB;
    };
    auto plan = [&](int64_t rows) {
        Part p;
        p.rows = rows;
        p.rows_per_slab = ceil_div(ceil_div(rows, wgrad_slabs(rows, tiles, 2048)), BKB) * BKB;
        if (p.rows_per_slab < BKB) p.rows_per_slab = BKB;
        p.slabs = rows > 0 ? ceil_div(rows, p.rows_per_slab) : 1;
        return p;
    };
    Part main_part, rest;
    if (n_main > 0) main_part = plan(n_main);
    if (n_main < n || n == 0) rest = plan(n - n_main);
    // One reduction adds the slabs of both where they fit the buffer's default size together (a
    // call recorded into a graph must not make it grow): six products over 100003 rows take 11 us
    // less than with a reduction of their own for the last 3 rows.
    const int64_t all = main_part.slabs + rest.slabs;
    const bool together = (size_t)all * cells * sizeof(float) <= ((size_t)64 << 20);
    const int64_t most = main_part.slabs > rest.slabs ? main_part.slabs : rest.slabs;
    void* scratch = nullptr;
    MIXGCN_TRY(get_scratch(0, (size_t)(together ? all : most) * cells * sizeof(float), &scratch));
    float* const P0 = (float*)scratch;
    if (timer) MIXGCN_TRY(timer->begin(kTimeUpdateWgrad, s));
    // the rest in the launch of the whole steps: one more slab
    const bool one_launch = pitches_ok && together && n % BKB != 0;
    auto slabs = [&](bool transposing_reads, int64_t row0, const Part& p, float* P) {
        const int64_t rows = p.rows, rows_per_slab = p.rows_per_slab;
        const int64_t n_slabs = p.slabs + (transposing_reads && one_launch ? 1 : 0);
        const unsigned grid = (unsigned)(n_slabs * tiles);
        const int64_t n_all = one_launch ? n : rows;
        const uint16_t* a = A + row0 * lda;
        const uint16_t* b = B + row0 * ldb;
        const uint16_t* r = R ? R + row0 * ldr : nullptr;
#define MIXGCN_WGRAD(SHAPE, MASK)                                                                             \
    do {                                                                                                      \
        if (transposing_reads)                                                                                \
            hipLaunchKernelGGL((wgrad_bf16_tr_kernel<SHAPE, MASK>), dim3(grid), dim3(kBlock), 0, s, a, lda, b, ldb, r, \
                               ldr, P, rows, n_all, k, m, rows_per_slab, nit, njt);                           \
        else                                                                                                  \
            hipLaunchKernelGGL((wgrad_bf16_kernel<SHAPE, MASK>), dim3(grid), dim3(kBlock), 0, s, a, lda, b, ldb, r, \
                               ldr, P, rows, k, m, rows_per_slab, nit, njt);                                  \
    } while (0)
        if (wide) {
            if (r) MIXGCN_WGRAD(Shape128x128, true);
            else MIXGCN_WGRAD(Shape128x128, false);
        } else {
            if (r) MIXGCN_WGRAD(Shape128x32, true);
            else MIXGCN_WGRAD(Shape128x32, false);
        }
#undef MIXGCN_WGRAD
    };
    if (main_part.slabs || one_launch) {
        slabs(true, 0, main_part, P0);
        if (!together) {
            MIXGCN_TRY(launch_wgrad_reduce(P0, main_part.slabs, cells, m, C, ldc, beta, s));
            beta = 1.f;
        }
    }
    if (rest.slabs && !one_launch) slabs(false, n_main, rest, together ? P0 + main_part.slabs * cells : P0);
    if (together || rest.slabs)
        MIXGCN_TRY(launch_wgrad_reduce(P0, together ? all : rest.slabs, cells, m, C, ldc, beta, s));
    if (timer) MIXGCN_TRY(timer->end(s));
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

}  // namespace mixgcn
