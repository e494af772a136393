// Node update H' = sigma(Z W) of fp32 features (paper Algorithm 2, update phase) on the fp32 matrix cores:
// C[n x MD] = act(A[n x KD] W[KD x MD]) with few columns and very many rows.  The sums are chains of fp32
// multiply-adds over the reduction index, bit for bit those of the tiles in gemm.hip, which remain for weights
// that do not fit LDS and where they are faster (column_tiles).
//
// Work split.  The weights of 32 TN output columns stay in LDS, in MFMA operand order, for as long as the workgroup
// lives (one per compute unit); its wavefronts then walk 32-row tiles of their own without a barrier, each with the
// rows of the next two steps of 16 indices in flight from global memory straight to registers (16 rows of 64 bytes
// per load).  v_mfma_f32_32x32x2_f32 wants index 2 j in lanes 0 to 31 and 2 j + 1 in lanes 32 to 63, of all 32 rows:
// eight register swaps per step put them there.  The weights are its first operand, so that a lane ends with
// consecutive columns of one row and writes 16 bytes at a time.
//
// What bounds it: the matrix cores at 78 % of their time (2^20 rows, 256 -> 256), which a loop of the same MFMAs, LDS
// reads and vector instructions alone could keep busy for 94 %.  What is between them: without the stores 1009 instead
// of 1109 us, without the row loads 1025; more or fewer wavefronts per SIMD (1, 2, 3) 1148, 1123, 1240; stores with the
// non-temporal hint 1136 instead of 1101 (128 -> 1024 at 2^21 rows 5005 : 4596).  us, tiles through LDS with a barrier
// per step (gemm.hip) : here: 2^20 rows 256 -> 256 1188 : 1110, 256 -> 47 412 : 327; 2^21 rows 128 -> 1024 4974 : 4660; 2^18
// rows 128 -> 256 171 : 164, 256 -> 16 61 : 51; 20 k rows 256 -> 128 27.7 : 19.6.
#include <type_traits>

#include "gemm_common.h"
#include "internal.h"

namespace mixgcn {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) floatx4 lds_floatx4;

constexpr int KC = 16;         // reduction indices per step: 64 bytes of a row
constexpr int kTileRows = 32;  // rows of a wavefront's tile
constexpr int kWeightsLds = 160 * 1024;

// Wavefronts of a workgroup.  A single column tile waits for memory and takes more of them.
template <int TN>
struct Walk {
    static constexpr int WAVES = TN == 1 ? 16 : 8;
    static constexpr int CHUNK = TN * KC * 32;  // floats of one step's weights
};

struct ForwardArgs {
    const float* A;
    int64_t lda;
    const float* W;
    int64_t ldw;
    float* C;
    int64_t ldc;
    int64_t n;
    int KD, MD;
    int n_col_tiles, row_groups;
    int waves;  // wavefronts of a workgroup that walk rows; all load the weights
};

// x: its odd groups of 16 lanes exchanged with the even ones of y
__device__ inline void swap16(float& x, float& y)
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(s[0]);
    y = __uint_as_float(s[1]);
}
// x: its upper half exchanged with the lower half of y
__device__ inline void swap32(float& x, float& y)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(s[0]);
    y = __uint_as_float(s[1]);
}

template <int TN, bool RELU>
__global__ __launch_bounds__(Walk<TN>::WAVES * kWave) __attribute__((amdgpu_waves_per_eu(Walk<TN>::WAVES / 4)))
void forward_rows_kernel(ForwardArgs p)
{
    constexpr int kThreads = Walk<TN>::WAVES * kWave, kChunk = Walk<TN>::CHUNK;
    constexpr int BN = TN * 32;
    extern __shared__ __attribute__((aligned(16))) float weights[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int pairs = (p.KD + 2 * KC - 1) / (2 * KC), nch = 2 * pairs;

    // workgroups are dealt round-robin to the 8 XCDs: the column tiles of one group of rows run on the same XCD,
    // next to each other
    const int xcd = blockIdx.x % 8, q = blockIdx.x / 8;
    const int col0 = (q % p.n_col_tiles) * BN;
    const int group = (q / p.n_col_tiles) * 8 + xcd;

    // ---- rows: lane (li, g) loads bytes 16 g .. 16 g + 15 of a step of rows li and 16 + li ----
    const int64_t tiles = (p.n + kTileRows - 1) / kTileRows;
    const int64_t stride = (int64_t)p.row_groups * p.waves;
    const int64_t first = (int64_t)group * p.waves + wave;
    const int64_t count = first < tiles && wave < p.waves ? (tiles - first + stride - 1) / stride : 0;
    struct Rows {
        floatx4 a[2];
    } raw[2];
    const char* arow[2];
    int lc = 0;          // step the load cursor stands at
    int64_t lt = first;  // its tile
    const uint64_t lane_row = (uint64_t)li * p.lda * 4 + g * 16;
    auto point = [&]() {
        if ((lt + 1) * kTileRows <= p.n) {
            const char* const base = reinterpret_cast<const char*>(p.A + lt * kTileRows * p.lda);
            arow[0] = base + lane_row;
            arow[1] = base + 16 * p.lda * 4 + lane_row;
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                int64_t row = lt * kTileRows + h * 16 + li;
                if (row > p.n - 1) row = p.n - 1;
                arow[h] = reinterpret_cast<const char*>(p.A + row * p.lda) + g * 16;
            }
        }
    };
    const int whole = p.KD / KC;  // steps wholly inside the depth
    const char* zero = reinterpret_cast<const char*>(&g_zero_piece);
    asm("" : "+s"(zero));  // (not looked up again in every step)
    auto load = [&](Rows& x) {
        const char* from[2] = {arow[0] + lc * (KC * 4), arow[1] + lc * (KC * 4)};
        if (lc >= whole && lc * KC + 4 * g >= p.KD)
            from[0] = from[1] = zero;
#pragma unroll
        for (int h = 0; h < 2; ++h) x.a[h] = load_piece<floatx4>(from[h]);
        if (++lc == nch) {
            lc = 0;
            lt += stride;
            point();
        }
    };
    // where the depth ends inside a piece, what the row holds past it is cleared
    const bool split_piece = p.KD % 4 != 0;
    auto trim = [&](Rows& x, int c) {
        if (!split_piece || c < whole) return;
        const int left = p.KD - c * KC - 4 * g;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) x.a[h][e] = left > e ? x.a[h][e] : 0.f;
    };

    point();
    if (count > 0) {
        load(raw[0]);
        load(raw[1]);
    }

    // ---- weights: [step][half of a step][column tile][lane][4]: what a lane feeds to four MFMAs in a row ----
    {
        constexpr int kItems = kChunk / 4;
        const int items = nch * kItems;
        for (int i = tid; i < items; i += 4 * kThreads) {  // four items per thread in flight
            floatx4 w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = i + u * kThreads;
                if (j >= items) continue;
                const int l = j & 63, t = j / 64 % TN, half = j / (64 * TN);  // half: over all steps
                const int k = half * 8 + (l >> 5), col = col0 + t * 32 + (l & 31);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // always one load, from an address inside
                    const bool in = k + 2 * e < p.KD && col < p.MD;
                    const float v = p.W[in ? (int64_t)(k + 2 * e) * p.ldw + col : 0];
                    w[u][e] = in ? v : 0.f;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = i + u * kThreads;
                if (j < items) *(lds_floatx4*)(weights + (size_t)j * 4) = w[u];
            }
        }
    }
    __syncthreads();
    if (count == 0) return;

    floatx16 acc[TN];
    floatx4 b[2][TN];
    const float* const mine = weights + lane * 4;
    auto fetch = [&](int half, floatx4 (&x)[TN]) {
#pragma unroll
        for (int t = 0; t < TN; ++t) x[t] = *reinterpret_cast<const floatx4*>(mine + (half * TN + t) * 256);
    };
    // acc += four pairs of indices (or, FIRST, = ); the weights of the next four are on their way meanwhile
    auto mma = [&](const float* o, const floatx4 (&x)[TN], auto first) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                floatx16 zero;
#pragma unroll
                for (int v = 0; v < 16; ++v) zero[v] = 0.f;
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[t][s], o[s], first && s == 0 ? zero : acc[t], 0, 0, 0);
            }
        __builtin_amdgcn_sched_group_barrier(0x100, TN, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * TN, 0);
    };
    // D layout of the 32x32 MFMA with the weights first: lane l, register v -> row l % 32, column 8 (v / 4) +
    // 4 (l / 32) + v % 4.  One register swap per pair of quads gives a lane 16 bytes of row li (x) and 16 + li (y),
    // four lanes 64 consecutive bytes.
    const int lane_col = (g & 1) * 8 + (g >> 1) * 4;
    const uint64_t lane_out = ((uint64_t)li * p.ldc + lane_col) * 4;
    auto write = [&](int64_t tile) {
        char* const base = reinterpret_cast<char*>(p.C + tile * kTileRows * p.ldc + col0) + lane_out;
        char* const base16 = base + 16 * p.ldc * 4;
        // 16 bytes of rows li and 16 + li from column 32 t + 16 j + lane_col of the tile on
        auto quads = [&](int t, int j, floatx4& x, floatx4& y) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float a = acc[t][8 * j + v], b = acc[t][8 * j + 4 + v];
                if (RELU) {
                    a = __builtin_amdgcn_fmed3f(a, 0.f, __builtin_inff());
                    b = __builtin_amdgcn_fmed3f(b, 0.f, __builtin_inff());
                }
                swap16(a, b);
                x[v] = a;
                y[v] = b;
            }
        };
        if ((tile + 1) * kTileRows <= p.n && col0 + BN <= p.MD) {
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    floatx4 x, y;
                    quads(t, j, x, y);
                    *reinterpret_cast<floatx4*>(base + (t * 32 + j * 16) * 4) = x;
                    *reinterpret_cast<floatx4*>(base16 + (t * 32 + j * 16) * 4) = y;
                }
            return;
        }
        const int64_t left = p.n - tile * kTileRows - li;
        const int cols = p.MD - col0 - lane_col;
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                floatx4 x, y;
                quads(t, j, x, y);
                const int c = t * 32 + j * 16;
                if (c + 4 <= cols) {
                    if (left > 0) *reinterpret_cast<floatx4*>(base + c * 4) = x;
                    if (left > 16) *reinterpret_cast<floatx4*>(base16 + c * 4) = y;
                } else {
#pragma unroll
                    for (int v = 0; v < 3; ++v) {
                        if (c + v < cols && left > 0) reinterpret_cast<float*>(base)[c + v] = x[v];
                        if (c + v < cols && left > 16) reinterpret_cast<float*>(base16)[c + v] = y[v];
                    }
                }
            }
    };

    // ---- the walk ----
    auto step = [&](Rows& x, int c, auto first) {
        trim(x, c);
        float o[8];
        {
            float u[4], w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u[e] = x.a[0][e];
                w[e] = x.a[1][e];
                swap16(u[e], w[e]);  // u: indices e and 8 + e of all rows, w: 4 + e and 12 + e
            }
            swap32(u[0], u[1]);  // (0 | 1) and (8 | 9)
            swap32(u[2], u[3]);
            swap32(w[0], w[1]);  // (4 | 5) and (12 | 13)
            swap32(w[2], w[3]);
            o[0] = u[0], o[1] = u[2], o[2] = w[0], o[3] = w[2];
            o[4] = u[1], o[5] = u[3], o[6] = w[1], o[7] = w[3];
        }
        // the new loads go out after the old values have been used: a register set that is still in flight is
        // never copied (a copy waits for it)
#pragma unroll
        for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(o[e]));
        __builtin_amdgcn_sched_barrier(0);
        load(x);
        __builtin_amdgcn_sched_barrier(0);
        fetch(2 * c + 1, b[1]);
        mma(o, b[0], first);
        fetch(c + 1 == nch ? 0 : 2 * c + 2, b[0]);
        mma(o + 4, b[1], std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, b[0]);
    int64_t tile = first;
    // (the first two steps of a tile are written out: the first sums start from an inline zero)
    for (int64_t i = 0; i < count; ++i, tile += stride) {
        step(raw[0], 0, std::true_type{});
        step(raw[1], 1, std::false_type{});
        for (int c = 2; c < nch; c += 2) {
            step(raw[0], c, std::false_type{});
            step(raw[1], c + 1, std::false_type{});
        }
        write(tile);
    }
}

template <int TN>
int launch_tn(bool relu, ForwardArgs a, hipStream_t s)
{
    a.n_col_tiles = (int)ceil_div(a.MD, TN * 32);
    const RowWalk w = plan_row_walk(ceil_div(a.n, kTileRows), a.n_col_tiles, Walk<TN>::WAVES, false);
    a.row_groups = w.row_groups;
    a.waves = w.waves;
    const unsigned lds = (unsigned)(2 * ceil_div(a.KD, 2 * KC) * Walk<TN>::CHUNK * sizeof(float));
    if (relu)
        hipLaunchKernelGGL((forward_rows_kernel<TN, true>), dim3(w.grid), dim3(Walk<TN>::WAVES * kWave), lds, s, a);
    else
        hipLaunchKernelGGL((forward_rows_kernel<TN, false>), dim3(w.grid), dim3(Walk<TN>::WAVES * kWave), lds, s, a);
    MIXGCN_HIP_TRY(hipGetLastError());
    return MIXGCN_OK;
}

template <int TN>
bool fits(int KD)
{
    return 2 * ceil_div(KD, 2 * KC) * Walk<TN>::CHUNK * (int64_t)sizeof(float) <= kWeightsLds;
}

// Tiles that a wavefront walks one after another, and whether they keep at least `percent` of the time of all the
// wavefronts that the chip holds.
struct Passes {
    int64_t n;
    bool full(int percent) const { return 100 * used >= percent * n * slots; }
    int64_t used, slots;
};
template <int TN>
Passes passes(int64_t n, int MD)
{
    const int64_t tiles = ceil_div(n, kTileRows), n_col_tiles = ceil_div(MD, TN * 32);
    const RowWalk w = plan_row_walk(tiles, (int)n_col_tiles, Walk<TN>::WAVES, false);
    return Passes{ceil_div(w.grid, 256) * ceil_div(tiles, (int64_t)w.row_groups * w.waves), tiles * n_col_tiles,
                  256 * Walk<TN>::WAVES};
}

// Column tiles of a product in units of 32 columns, 0 for the tiles of gemm.hip.  Figures: us, those tiles : here, or how
// many times as fast it is here.
int column_tiles(int64_t n, int KD, int MD)
{
    if (n <= 0) return 0;
    const int64_t tiles = ceil_div(n, kTileRows), blocks = ceil_div(n, 128);
    // gemm.hip: its workgroups, and whether none has a tile at an edge of the columns, or at any edge.  A small launch takes
    // as long as its slowest workgroup, and one with an edge takes half as long again.
    const int64_t grid = blocks * ceil_div(MD, MD > 64 ? 128 : 32);
    const bool even = MD % (MD > 64 ? 128 : 32) == 0 && KD % KC == 0, whole = even && n % 128 == 0;
    if (MD > 64) {
        // Where its tiles leave a fifth of the compute units idle, with none at an edge half of them, 32 columns each for
        // more wavefronts: 20 k rows 256 -> 128 27.7 : 19.6, 5000 602 -> 128 56.8 : 17.4; no edge, 16384 64 -> 128 1.06,
        // 5120 64 -> 512 0.93, 25600 256 -> 128 0.89.  As long as none of them walks two tiles (5000 rows 256 -> 602
        // 0.65) or the workgroups of the second round are few (1000 64 -> 1500 1.33, 2500 64 -> 2048 0.95).  Shallow
        // depths gain by it where few compute units have a tile at all (8000 48 -> 256 1.22, 12 k 0.98; 16 -> 128 of 8000
        // 1.31, 20 k 0.90; no edge, 5120 32 -> 256 1.02, 10 k 0.86), or one or two column tiles have columns left over
        // (25 k 16 -> 80 1.06, 4096 48 -> 602 0.89).
        if (grid <= 200) {
            const Passes p = passes<1>(n, MD);
            const int64_t most = whole ? (KD < 32 ? 0 : KD < 64 ? 64 : KD < 96 ? 110 : 128)
                                 : MD % 128 == 0 || MD > 256 ? (KD < 32 ? 64 : KD < 64 ? 130 : 200) : 200;
            const bool few = p.n == 1 || (p.n == 2 && p.used <= 2048 && KD >= (whole ? 128 : 32));
            return grid <= most && few && fits<1>(KD) ? 1 : 0;
        }
        // Otherwise 128 columns, where wavefronts walk eight tiles each that keep 93 % of their time (267 k rows 256 ->
        // 384, 87 %, 0.94; 100 k 160 -> 640, 85 %, 0.92; 2 M 256 -> 384, 93 %, 1.02), deep enough to pay for the weights,
        // and no odd step that is filled up with zeros: 2^20 rows 256 -> 256 1188 : 1110, 2^18 128 -> 256 171 : 164 (200 k
        // rows 128 -> 128, three tiles each, 75 : 82; 100 k 90 -> 768 154 : 165; 700 k 100 -> 90 212 : 215).
        const Passes p = passes<4>(n, MD);
        return KD >= 128 && ceil_div(KD, KC) % 2 == 0 && p.n >= 8 && p.full(93) && fits<4>(KD) ? 4 : 0;
    }
    // 64 columns in four tiles and more that keep 85 % of the time: 2^20 rows 256 -> 47 412 : 327, 300 k 1.08 (270 k 200 ->
    // 47, 82 %, 0.94; 233 k 128 -> 41 47 : 54).
    if (MD > 32 && KD >= 192 && tiles >= 8192) return passes<2>(n, MD).full(85) && fits<2>(KD) ? 2 : 0;
    // 32 columns.  A step is 32 indices deep here, 16 in gemm.hip: not where the last one is mostly zeros (100 k rows
    // 47 -> 32 0.80, 80 -> 24 0.95), nor for shallow depths (100 k 16 -> 32 0.72).
    if (KD < 64 || !fits<1>(KD) || 9 * KD < 8 * 32 * ceil_div(KD, 32)) return 0;
    const Passes p = passes<1>(n, MD);
    // Nearly all wavefronts with two to four tiles each: 2^18 rows 256 -> 16 1.26, 256 -> 32 1.04, 2^19 256 -> 16 1.04,
    // 2^20 no faster; 135 k rows, one tile and a little, 0.73, 400 k, three and a little, 0.85.
    if (p.n > 1) return MD <= 32 && p.n <= (even ? 2 : 4) && p.full(95) ? 1 : 0;
    // One tile each at most: not without an edge (4096 rows 64 -> 32 0.85, 12 k 256 -> 64 0.82).  10 k rows 256 -> 16 1.31,
    // 64 -> 32 1.0; past 200 of its workgroups with columns left over from 96 indices on (100 k 128 -> 16 1.09, 66 k 64 -> 8
    // 0.97), with rows alone where the workgroup at the edge is not among others of a second round, from 128 on (30 k
    // 128 -> 32 1.04, 33 k 0.85, 50 k 1.01, 66 k 0.93; 26 k 64 -> 32 0.93).
    if (whole || (MD > 32 && blocks > 200)) return 0;
    if (grid <= 200) return 1;
    return even ? KD >= 128 && grid <= 512 && (grid <= 256 || grid > 300) : KD >= 96;
}

}  // namespace

bool forward_rows_applies(int64_t n, int KD, int MD) { return column_tiles(n, KD, MD) > 0; }

int launch_forward_rows(bool relu, const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc,
                        int64_t n, int KD, int MD, hipStream_t s)
{
    if (n <= 0) return MIXGCN_OK;
    const ForwardArgs a{A, lda, W, ldw, C, ldc, n, KD, MD, 0, 0, 0};
    switch (column_tiles(n, KD, MD)) {
    case 4: return launch_tn<4>(relu, a, s);
    case 2: return launch_tn<2>(relu, a, s);
    default: return launch_tn<1>(relu, a, s);
    }
}

}  // namespace mixgcn
