// Node update H' = sigma(Z W) of bf16 features and data gradient dZ = (dP (.) 1[R > 0]) W^T of bf16 and fp32
// ones (paper Algorithm 2, update phase) on the bf16 matrix cores: C[n x MD] = act(A[n x KD] Bop[KD x MD])
// with few columns and very many rows.  (The forward product of fp32 features keeps the fp32 rounding.)
//
// Arithmetic.  fp32 operands are written as exact sums of three bf16 terms (round to nearest at each
// stage, |x1| <= 2^-8 |x|, |x2| <= 2^-16 |x|) and a product is accumulated in fp32 from the six partial
// products of order 2^-16 and above, smallest first; the three dropped ones are together below
// 2^-23 |a| |b|, one fp32 rounding.  bf16 features enter as they are and the weights as two terms
// (|W - hi - lo| < 2^-16 |W|).
//
// Work split.  The weights of 128 output columns stay in LDS, in MFMA operand order, for as long as the
// workgroup lives (one per compute unit; what fits is kRowsLds: three terms of up to 192 reduction indices, 144 KB,
// or two of up to 320, 160 KB, and of fewer output columns twice as many each time); its eight wavefronts then walk 32-row tiles of their own without a barrier, each with
// the rows of the next two steps in flight from global memory straight to registers (16 rows of 64 bytes
// per load: such a read runs at the streaming rate, 6.1 TB/s).  No other wavefront needs a row, so
// nothing is gained from LDS, and a term split happens once.  Deeper fp32 products stream the weights
// through two LDS buffers, split on the way, one barrier per step; deeper bf16 ones have a kernel of their own.
//
// What bounds it: memory (a copy in the same pattern reaches 5.2 TB/s) up to 128 x 128, from there on
// about evenly the matrix cores and the vector work of the splits.  Six bf16 MFMAs take 3/8 of the time
// of the fp32 MFMAs they replace; on random data this part sustains 270 to 300 TFLOP/s of fp32 products
// that way, register operands only, and these kernels reach 135 to 175.  us before (tiles of 128 x 128 on
// the fp32 matrix cores, bf16: on the bf16 ones) -> now, forward and data gradient:
//   fp32 2^20 rows, data gradient plain and masked, 128 -> 128: 344 -> 240, 399 -> 313;  256 -> 256: 1164 -> 868,
//   1256 -> 1029;  602 -> 128: 1396 -> 1008, 1610 -> 1315;  11.1 M rows 128 -> 128: 3659 -> 2386
//   bf16 2.45 M rows 256 -> 256: 912 -> 690, 1150 -> 985;  100 -> 256: 562 -> 424;  100003 rows
//   128 -> 128: 24 -> 16 (the weights' own launch is gone too)
#include "gemm_common.h"
#include "internal.h"

namespace mixgcn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uintx4 lds_uintx4;

constexpr int kRowsWaves = 8;                      // most wavefronts per workgroup
constexpr int kRowsBlock = kRowsWaves * kWave;
constexpr int TM = 2;                              // 16-row tiles per wavefront
constexpr int kWaveRows = 16 * TM;
constexpr int kRowsLds = 160 * 1024;

template <int DT>
struct Terms {
    static constexpr int PA = DT == MIXGCN_F32 ? 3 : 1;  // terms of a feature
    static constexpr int PB = DT == MIXGCN_F32 ? 3 : 2;  // terms of a weight
    static constexpr int NQ = DT == MIXGCN_F32 ? 6 : 2;  // partial products
    static constexpr int NB = DT == MIXGCN_F32 ? 1 : 2;  // MFMAs along the reduction per step
    static constexpr int KC = 32 * NB;                   // reduction indices per step: 128 bytes of a row
    static constexpr int ES = DT == MIXGCN_F32 ? 4 : 2;
};
template <int DT>
__device__ constexpr int term_a(int q)
{
    constexpr int f[6] = {2, 0, 1, 1, 0, 0};
    return DT == MIXGCN_F32 ? f[q] : 0;
}
template <int DT>
__device__ constexpr int term_b(int q)
{
    constexpr int f[6] = {0, 2, 1, 0, 1, 0};
    return DT == MIXGCN_F32 ? f[q] : 1 - q;
}

// A lane of group g reads two 16-byte pieces of its row per step, piece h at byte 64 h + 16 g: the four
// groups together take 64 consecutive bytes.  First reduction index of piece h; fp32: both pieces feed one
// MFMA (elements 0 .. 3 and 4 .. 7 of the lane), bf16: one each.
template <int DT>
__device__ inline int piece_index(int g, int h)
{
    return DT == MIXGCN_F32 ? h * 16 + g * 4 : h * 32 + g * 8;
}
// Reduction index within a step of element e of lane group g in MFMA b.
template <int DT>
__device__ inline int step_index(int g, int b, int e)
{
    return DT == MIXGCN_F32 ? piece_index<DT>(g, e >> 2) + (e & 3) : piece_index<DT>(g, b) + e;
}
// Output column of row i of MFMA tile t.  bf16: two tiles interleave, so that a lane holds eight
// consecutive columns (16 bytes) of its node row.
template <int DT, int TN>
__device__ inline int tile_column(int t, int i)
{
    if (DT == MIXGCN_F32 || TN == 1) return t * 16 + i;
    return (t >> 1) * 32 + (i >> 2) * 8 + (t & 1) * 4 + (i & 3);
}

// P bf16 terms of eight fp32 values, term p in out[4 p ..]: words of two consecutive values.
// WEIGHTS: an infinity, or a value that rounds to one, stays in the first term alone.
template <int P, bool WEIGHTS>
__device__ inline void split8(const float* x, uint32_t* out)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t w = pack_bf16(a, b);
            out[4 * p + i] = w;
            if (p + 1 < P) {
                a -= low_half(w);
                b -= high_half(w);
                if (WEIGHTS) {
                    if (!(fabsf(a) <= 3.0e38f)) a = 0.f;
                    if (!(fabsf(b) <= 3.0e38f)) b = 0.f;
                }
            }
        }
    }
}

__device__ inline uint4 load_from(const char* p)
{
    const uintx4 v = load_piece<uintx4>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// v, recomputed where it is used: what is derived from it inside the main loop is not kept in registers
// from iteration to iteration.
__device__ inline int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// How the rows are masked: not, by 1[R > 0], or by the bits that the weight gradient has made of it (fp32).
constexpr int kNoMask = 0, kMaskRef = 1, kMaskBits = 2;

template <int DT, int MASK>
struct RawRows {
    uint4 a[TM][2];
    uint4 r[TM][MASK == kMaskRef ? 2 : 1];
    uint2 bits[TM];
};

struct RowsArgs {
    const void* A;
    int64_t lda;
    const float* W;
    int64_t ldw;
    void* C;
    int64_t ldc;
    int64_t n;
    int KD, MD;
    const void* R;
    int64_t ldr;
    int n_col_tiles, row_groups;
    int waves;  // wavefronts of a workgroup that walk rows (streamed weights: all); all load the weights
    ReluBits bits;
};

template <int DT, int TN, bool WT, bool RELU, int MASK, bool RESIDENT>
__global__ __launch_bounds__(kRowsBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void update_rows_kernel(RowsArgs p)
{
    using T = Terms<DT>;
    constexpr int PA = T::PA, PB = T::PB, NB = T::NB, KC = T::KC, ES = T::ES;
    constexpr int BN = TN * 16;
    constexpr int kChunk = TN * NB * PB * 512;  // halfwords of one step's weights
    extern __shared__ __attribute__((aligned(16))) uint16_t wlds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, g = lane >> 4;
    const int nch = (p.KD + KC - 1) / KC;

    // workgroups are dealt round-robin to the 8 XCDs: the column tiles of one group of rows run on the
    // same XCD, next to each other
    const int xcd = blockIdx.x % 8, q = blockIdx.x / 8;
    const int col0 = (q % p.n_col_tiles) * BN;
    const int group = (q / p.n_col_tiles) * 8 + xcd;

    // ---- weights: item = (tile, MFMA of the step, lane), eight elements, PB terms ----
    // a weight at the edge of W, or zero past it: always one load, from an address inside
    auto edge = [&](int k, int col) {
        const bool in = k < p.KD && col < p.MD;
        const int64_t kk = in ? k : 0, cc = in ? col : 0;
        const float v = p.W[WT ? kk * p.ldw + cc : cc * p.ldw + kk];
        return in ? v : 0.f;
    };
    auto load_w = [&](int c, int item, float* w) {
        item = fresh(item);
        const int t = item / (64 * NB), kb = item / 64 % NB, gg = (item >> 4) & 3;
        const int col = col0 + tile_column<DT, TN>(t, item & 15);
        const bool inside = (c + 1) * KC <= p.KD && col0 + BN <= p.MD;
        if (WT) {
            const float* src = p.W + (int64_t)(c * KC) * p.ldw + col;
            if (inside) {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = src[(int64_t)step_index<DT>(gg, kb, e) * p.ldw];
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = edge(c * KC + step_index<DT>(gg, kb, e), col);
            }
        } else {
            const float* src = p.W + (int64_t)col * p.ldw + c * KC;
            if (inside) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 v = *reinterpret_cast<const float4*>(src + step_index<DT>(gg, kb, 4 * h));
                    w[4 * h] = v.x;
                    w[4 * h + 1] = v.y;
                    w[4 * h + 2] = v.z;
                    w[4 * h + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = edge(c * KC + step_index<DT>(gg, kb, e), col);
            }
        }
    };
    auto store_w = [&](uint16_t* chunk, int item, const float* w) {
        uint32_t t[4 * PB];
        float x[8];
        item = fresh(item);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = DT == MIXGCN_F32 ? w[e] * kTermScale : w[e];
        split8<PB, true>(x, t);
        uint16_t* dst = chunk + (item >> 6) * (PB * 512) + (item & 63) * 8;
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            const uintx4 v = {t[4 * b], t[4 * b + 1], t[4 * b + 2], t[4 * b + 3]};
            *(lds_uintx4*)(dst + b * 512) = v;
        }
    };
    constexpr int kItems = TN * 64 * NB;
    constexpr int kPerThread = (kItems + kRowsBlock - 1) / kRowsBlock;  // weight items per thread and step
    float wreg[kPerThread][8];
    auto load_step_w = [&](int c) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            if (kItems % kRowsBlock == 0 || tid + i * kRowsBlock < kItems)
                load_w(c, tid + i * kRowsBlock, wreg[i]);
    };
    auto store_step_w = [&](uint16_t* chunk) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            if (kItems % kRowsBlock == 0 || tid + i * kRowsBlock < kItems)
                store_w(chunk, tid + i * kRowsBlock, wreg[i]);
    };

    // ---- rows: lane (li, g) holds row li of a 16-row tile ----
    // RESIDENT: every wavefront walks 32-row tiles of its own; otherwise the workgroup walks blocks of
    // kRowsWaves tiles together, one step at a time
    const int64_t tiles = (p.n + kWaveRows - 1) / kWaveRows;
    const int waves = RESIDENT ? p.waves : kRowsWaves;
    const int64_t stride = (int64_t)p.row_groups * waves;
    const int64_t first = (int64_t)group * waves + wave;
    int64_t count;  // tiles of this wavefront (streaming: of its workgroup's first wavefront)
    {
        const int64_t f = RESIDENT ? first : (int64_t)group * kRowsWaves;
        count = f < tiles && wave < waves ? (tiles - f + stride - 1) / stride : 0;
    }
    // Rows in flight: two steps, or one with a mask, which loads twice the bytes per step (and two would
    // not fit the registers).
    constexpr int kAhead = MASK == kMaskRef ? 1 : 2;
    RawRows<DT, MASK> raw[kAhead];
    const char* arow[TM];
    const char* rrow[TM];
    const char* brow[TM];
    int lc = 0;             // chunk the load cursor stands at
    int64_t lt = first;     // its tile
    auto point = [&]() {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            int64_t row = lt * kWaveRows + tm * 16 + li;
            if (row > p.n - 1) row = p.n - 1;
            arow[tm] = reinterpret_cast<const char*>(p.A) + row * p.lda * ES + g * 16;
            if (MASK == kMaskRef) rrow[tm] = reinterpret_cast<const char*>(p.R) + row * p.ldr * ES + g * 16;
            if (MASK == kMaskBits) brow[tm] = reinterpret_cast<const char*>(p.bits.p) + row * p.bits.pitch;
        }
    };
    const bool ragged = p.KD % KC != 0;
    // Loads of the cursor's step; in the last step of a ragged depth a piece past the end is read as zeros
    auto load = [&](RawRows<DT, MASK>& x) {
        const int off = lc * (KC * ES);
        const char* const zero = reinterpret_cast<const char*>(&g_zero_piece);
        const bool last = ragged && lc == nch - 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool out = last && lc * KC + piece_index<DT>(g, h) >= p.KD;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                x.a[tm][h] = load_from(out ? zero : arow[tm] + off + h * 64);
                if (MASK == kMaskRef) x.r[tm][h] = load_from(out ? zero : rrow[tm] + off + h * 64);
            }
        }
        if (MASK == kMaskBits) {  // the 32 columns of the step: a byte for each piece of 4, all lanes of a row the same
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) x.bits[tm] = *reinterpret_cast<const uint2*>(brow[tm] + lc * 8);
        }
        if (++lc == nch) {
            lc = 0;
            lt += stride;
            point();
        }
    };
    // ... and where the end lies inside a piece, what the row holds past it is cleared
    constexpr int kPiece = 16 / ES;
    const bool split_piece = p.KD % kPiece != 0;
    auto trim = [&](RawRows<DT, MASK>& x, int c) {
        if (!split_piece || c != nch - 1) return;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int left = p.KD - c * KC - piece_index<DT>(g, h);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                uint32_t* w = reinterpret_cast<uint32_t*>(&x.a[tm][h]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (DT == MIXGCN_F32) w[i] = left > i ? w[i] : 0u;
                    else w[i] &= (left > 2 * i ? 0x0000FFFFu : 0u) | (left > 2 * i + 1 ? 0xFFFF0000u : 0u);
                }
            }
        }
    };

    floatx4 acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[tm][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    constexpr int kWords = DT == MIXGCN_F32 ? PA : NB;  // 16-byte groups per 16-row tile
    struct Operand {
        uint32_t w[TM][4 * kWords];
    };
    auto split_rows = [&](const RawRows<DT, MASK>& x, Operand& o) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (DT == MIXGCN_F32) {
                float v[8];
                __builtin_memcpy(v, x.a[tm], 32);
                if (MASK == kMaskRef) {
                    float r[8];
                    __builtin_memcpy(r, x.r[tm], 32);
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = r[e] > 0.f ? v[e] : 0.f;
                }
                if (MASK == kMaskBits) {
                    const uint32_t w[2] = {x.bits[tm].x >> (8 * g), x.bits[tm].y >> (8 * g)};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint32_t keep = (uint32_t)((int)(w[e >> 2] << (31 - (e & 3))) >> 31);
                        v[e] = __uint_as_float(__float_as_uint(v[e]) & keep);
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] *= kTermScale;
                split8<PA, false>(v, o.w[tm]);
            } else {
                __builtin_memcpy(o.w[tm], x.a[tm], 32);
                if (MASK) {
                    uint32_t r[8];
                    __builtin_memcpy(r, x.r[tm], 32);
#pragma unroll
                    for (int i = 0; i < 8; ++i) o.w[tm][i] = keep_positive(o.w[tm][i], r[i]);
                }
            }
        }
    };
    // acc += o * chunk.  The partial products of a step are added up from zero and then to the running
    // sum, once per step: rounding the running sum for every partial product costs three times the error
    // (K = 128: 1.5e-7 against 5.5e-8, fp32 MFMA 2.0e-7).
    auto mma = [&](const Operand& o, const uint16_t* chunk) {
        const uint16_t* src = chunk + lane * 8;
        constexpr int NW = NB * PB;
        bf16x8 b[2][NW];
        floatx4 part[2][TM];
#pragma unroll
        for (int k = 0; k < NW; ++k) b[0][k] = *reinterpret_cast<const bf16x8*>(src + k * 512);
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            if (t + 1 < TN) {
#pragma unroll
                for (int k = 0; k < NW; ++k)
                    b[(t + 1) & 1][k] =
                        *reinterpret_cast<const bf16x8*>(src + ((t + 1) * NW + k) * 512);
            }
#pragma unroll
            for (int s = 0; s < T::NQ; ++s)
#pragma unroll
                for (int kb = 0; kb < NB; ++kb)
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) {
                        bf16x8 a;
                        __builtin_memcpy(&a, o.w[tm] + 4 * (DT == MIXGCN_F32 ? term_a<DT>(s) : kb), 16);
                        // weights first: the accumulators hold the tile transposed, a lane owns one node
                        // row and four consecutive columns
                        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                        part[t & 1][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            b[t & 1][kb * PB + term_b<DT>(s)], a, s + kb == 0 ? zero : part[t & 1][tm], 0, 0, 0);
                    }
            if (t > 0) {
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[tm][t - 1][v] += part[(t - 1) & 1][tm][v];
            }
        }
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[tm][TN - 1][v] += part[(TN - 1) & 1][tm][v];
        // issue order: the weights of the next tile, the products, the sums of the tile before
        __builtin_amdgcn_sched_group_barrier(0x100, NW, 0);
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            if (t + 1 < TN) __builtin_amdgcn_sched_group_barrier(0x100, NW, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NB * T::NQ * TM, 0);
            if (t > 0) __builtin_amdgcn_sched_group_barrier(0x002, 4 * TM, 0);
        }
    };

    // fp32: sums that are not finite, again in plain fp32
    auto repair = [&](int64_t row0) {
        if constexpr (DT == MIXGCN_F32) {
            const float* const A = reinterpret_cast<const float*>(p.A);
            const float* const R = reinterpret_cast<const float*>(p.R);
            const int64_t row1 = row0 + kWaveRows < p.n ? row0 + kWaveRows : p.n;
            const int col1 = col0 + BN < p.MD ? col0 + BN : p.MD;
            static_assert(!RELU, "of fp32 features the data gradient alone");
            repair_sums<false>(
                reinterpret_cast<float*>(p.C), p.ldc, row0, row1, col0, col1, p.KD,
                [&](int64_t r, int k) { return !MASK || R[r * p.ldr + k] > 0.f ? A[r * p.lda + k] : 0.f; },
                [&](int k, int c) { return p.W[WT ? (int64_t)k * p.ldw + c : (int64_t)c * p.ldw + k]; });
        }
    };
    auto write = [&](int64_t tile) {
        const int li = fresh(lane) & 15, g = fresh(lane) >> 4;
        const int64_t row0 = tile * kWaveRows;
        if (RELU) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[tm][t][v] = fmaxf(acc[tm][t][v], 0.f);
        }
        // 16-byte pieces of a lane's row: piece j holds byte 64 j + 16 g of the tile's row
        constexpr int kPieces = DT == MIXGCN_F32 ? TN : TN / 2;
        auto piece = [&](int tm, int j) {
            uintx4 o;
            if (DT == MIXGCN_F32) {
                __builtin_memcpy(&o, &acc[tm][j], 16);
            } else {
                const floatx4 &x = acc[tm][(2 * j) % TN], &y = acc[tm][(2 * j + 1) % TN];
                o = uintx4{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(y[0], y[1]),
                           pack_bf16(y[2], y[3])};
            }
            return o;
        };
        // 16 bytes from column c of the tile on, or what of them lies inside the matrix
        auto put = [&](char* row, int c, const uintx4& v) {
            if (col0 + c + 16 / ES <= p.MD) {
                __builtin_nontemporal_store(v, reinterpret_cast<uintx4*>(row + c * ES));
            } else {
#pragma unroll
                for (int e = 0; e < 16 / ES; ++e)
                    if (col0 + c + e < p.MD) {
                        if (DT == MIXGCN_F32) reinterpret_cast<uint32_t*>(row)[c + e] = v[e % 4];
                        else reinterpret_cast<uint16_t*>(row)[c + e] = (uint16_t)(v[e / 2 % 4] >> (16 * (e & 1)));
                    }
            }
        };
        if (kPieces > 0 && kPieces % 2 == 0 && row0 + kWaveRows <= p.n) {
            // Tiles whose rows all exist are written as whole 128-byte lines, eight rows at a time: lanes
            // eight apart exchange one of two neighboring pieces.  Against 64 bytes of 16 rows at a time
            // and with the write hint a copy in this pattern gains a seventh (231 -> 204 us for 1.07 GB).
            const bool lo = li < 8;
            const int c = ((lo ? 0 : 64) + g * 16) / ES;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                char* const out =
                    reinterpret_cast<char*>(p.C) + ((row0 + tm * 16 + (li & 7)) * p.ldc + col0) * ES;
                char* const out8 = out + 8 * p.ldc * ES;
#pragma unroll
                for (int j = 0; j < kPieces; j += 2) {
                    const uintx4 x = piece(tm, j), y = piece(tm, (j + 1) % (kPieces > 0 ? kPieces : 1));
                    uintx4 first, second;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const uint32_t give = lo ? y[v] : x[v];
                        const uint32_t take = (uint32_t)__builtin_amdgcn_update_dpp(
                            0, (int)give, 0x128 /* row_ror:8 */, 0xF, 0xF, true);
                        first[v] = lo ? x[v] : take;
                        second[v] = lo ? take : y[v];
                    }
                    put(out, c + j * 64 / ES, first);
                    put(out8, c + j * 64 / ES, second);
                    __builtin_amdgcn_sched_barrier(0);  // one pair's registers at a time
                }
            }
            return;
        }
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int64_t row = row0 + tm * 16 + li;
            if (row < p.n) {
                char* const out = reinterpret_cast<char*>(p.C) + (row * p.ldc + col0) * ES;
                if (kPieces > 0) {
#pragma unroll
                    for (int j = 0; j < kPieces; ++j) put(out, (j * 64 + g * 16) / ES, piece(tm, j));
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (col0 + 4 * g + v < p.MD)
                            reinterpret_cast<uint16_t*>(out)[4 * g + v] = (uint16_t)pack_bf16(acc[tm][0][v], 0.f);
                }
            }
        }
    };

    auto finish = [&](int64_t tile) {
        bool bad = false;
        if (DT == MIXGCN_F32) {
            float z = 0.f;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) z = fmaf(acc[tm][t][v], 0.f, z);
            bad = __any(!(z == 0.f));
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[tm][t][v] *= 1.f / (kTermScale * kTermScale);
        }
        write(tile);
        if (__builtin_expect(bad, 0)) repair(tile * kWaveRows);
    };

    auto pin = [](Operand& o) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int i = 0; i < 4 * kWords; ++i) asm volatile("" : "+v"(o.w[tm][i]));
    };

    // ---- the walk ----
    const int64_t steps = count * nch;
    if (!RESIDENT && steps == 0) return;  // uniform over the workgroup
    point();
    if (steps > 0) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) load(raw[i]);
    }
    if (RESIDENT) {
        // four items per thread in flight
        for (int i = tid; i < nch * kItems; i += 4 * kRowsBlock) {
            float w[4][8];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = i + u * kRowsBlock;
                if (j < nch * kItems) load_w(j / kItems, j % kItems, w[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = i + u * kRowsBlock;
                if (j < nch * kItems) store_w(wlds + j / kItems * kChunk, j % kItems, w[u]);
            }
        }
    } else {
        load_step_w(0);
        store_step_w(wlds);
        load_step_w(1);
    }
    __syncthreads();
    clear();
    if (steps == 0) return;
    int c = 0;
    int64_t tile = first;
    auto step = [&](RawRows<DT, MASK>& x, int64_t s) {
        Operand o;
        trim(x, c);
        split_rows(x, o);
        // the new loads go out after the old values have been used: a register set that is still in
        // flight is never copied (a copy waits for it)
        pin(o);
        __builtin_amdgcn_sched_barrier(0);
        if (!RESIDENT) {
            // The weights of the next step replace those of the step before this one.  They are loaded
            // before the rows of the same step: waiting for them then leaves the rows in flight.
            store_step_w(wlds + (int)((s + 1) & 1) * kChunk);
            load_step_w(c + 2 < nch ? c + 2 : c + 2 - nch);
            __builtin_amdgcn_sched_barrier(0);
        }
        load(x);
        __builtin_amdgcn_sched_barrier(0);
        mma(o, RESIDENT ? wlds + c * kChunk : wlds + (int)(s & 1) * kChunk);
        if (++c == nch) {
            c = 0;
            __builtin_amdgcn_sched_barrier(0);
            finish(tile);
            clear();
            __builtin_amdgcn_sched_barrier(0);
            tile += stride;
        }
        if (!RESIDENT) __syncthreads();
    };
    // (an odd last step of two is done once more on rows past the end, which are never stored)
    for (int64_t s = 0; s < steps; s += kAhead) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) step(raw[i], s + i);
    }
}

template <int DT, int TN, bool WT>
int launch_rows_tn(bool relu, const RowsArgs& args, hipStream_t s)
{
    RowsArgs a = args;
    constexpr int KC = Terms<DT>::KC;
    constexpr int kChunkBytes = TN * Terms<DT>::NB * Terms<DT>::PB * 1024;
    constexpr bool kBits = DT == MIXGCN_F32 && TN > 1;  // (rows of 16 columns hold no bits of 256)
    const int nch = (a.KD + KC - 1) / KC;
    const bool resident = nch * kChunkBytes <= kRowsLds;
    if (DT == MIXGCN_BF16 && !resident)
        return launch_update_bf16_deep(WT, relu, (const uint16_t*)a.A, a.lda, a.W, a.ldw, (uint16_t*)a.C, a.ldc,
                                       a.n, a.KD, a.MD, (const uint16_t*)a.R, a.ldr, s);
    a.n_col_tiles = (int)ceil_div(a.MD, TN * 16);
    const int64_t tiles = ceil_div(a.n, kWaveRows);
    const RowWalk w = plan_row_walk(tiles, a.n_col_tiles, kRowsWaves, !resident);
    a.row_groups = w.row_groups;
    a.waves = w.waves;
    const unsigned grid = w.grid;
    const unsigned lds = (unsigned)((resident ? nch : 2) * kChunkBytes);
#define MIXGCN_ROWS(RELU, MASK)                                                                       \
    do {                                                                                              \
        if (DT == MIXGCN_BF16 || resident)                                                            \
            hipLaunchKernelGGL((update_rows_kernel<DT, TN, WT, RELU, MASK, true>), dim3(grid),        \
                               dim3(kRowsBlock), lds, s, a);                                          \
        else                                                                                          \
            hipLaunchKernelGGL((update_rows_kernel<DT, TN, WT, RELU, MASK, DT == MIXGCN_BF16>),       \
                               dim3(grid), dim3(kRowsBlock), lds, s, a);                              \
    } while (0)
    if constexpr (WT) {
        if (relu) MIXGCN_ROWS(true, kNoMask);
        else MIXGCN_ROWS(false, kNoMask);
    } else {
        if (!a.R) MIXGCN_ROWS(false, kNoMask);
        else if (!kBits || !a.bits.p) MIXGCN_ROWS(false, kMaskRef);
        else if constexpr (kBits) MIXGCN_ROWS(false, kMaskBits);
    }
#undef MIXGCN_ROWS
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

template <int DT, bool WT>
int launch_rows_wt(bool relu, const RowsArgs& a, hipStream_t s)
{
    if (a.MD <= 16) return launch_rows_tn<DT, 1, WT>(relu, a, s);
    if (a.MD <= 32) return launch_rows_tn<DT, 2, WT>(relu, a, s);
    if (a.MD <= 64) return launch_rows_tn<DT, 4, WT>(relu, a, s);
    return launch_rows_tn<DT, 8, WT>(relu, a, s);
}

}  // namespace

// C[n x MD] = act((A (.) 1[R > 0])[n x KD] Wop), Wop[kk][j] = w_is_kd_major ? W[kk][j] : W[j][kk]; of fp32
// features the data gradient alone
int launch_update_rows(int dtype, bool w_is_kd_major, bool relu, const void* A, int64_t lda, const float* W,
                       int64_t ldw, void* C, int64_t ldc, int64_t n, int KD, int MD, const void* R,
                       int64_t ldr, hipStream_t s, ReluBits bits)
{
    if (n <= 0) return MIXGCN_OK;
    RowsArgs a{A, lda, W, ldw, C, ldc, n, KD, MD, R, ldr, 0, 0, 0, bits};
    if (dtype == MIXGCN_F32) return launch_rows_wt<MIXGCN_F32, false>(relu, a, s);
    return w_is_kd_major ? launch_rows_wt<MIXGCN_BF16, true>(relu, a, s)
                         : launch_rows_wt<MIXGCN_BF16, false>(relu, a, s);
}

}  // namespace mixgcn
