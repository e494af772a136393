// Device helpers shared by the kernels of the update products.
#pragma once
#include "device_utils.h"
#include "internal.h"

namespace mixgcn {

// Tile shape: WM x WN waves (4 in total), each owning TM x TN accumulator tiles of 32 x 32.
template <int WM_, int WN_, int TM_, int TN_>
struct Shape {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_;
    static constexpr int BM = WM * TM * 32;  // extent along the A-operand free dimension
    static constexpr int BN = WN * TN * 32;  // extent along the B-operand free dimension
    static_assert(WM * WN == 4, "four waves per block");
};
using Shape128x128 = Shape<2, 2, 2, 2>;
using Shape128x32 = Shape<4, 1, 1, 1>;

// Workgroups are dealt round-robin to the 8 XCDs.  This maps the hardware block index to a
// logical one such that consecutive logical indices run on the same XCD, so tiles that share
// an operand (the column tiles of one row block) find it in that XCD's L2.
__device__ inline unsigned xcd_local_index(unsigned bid, unsigned grid)
{
    const unsigned q = grid / 8, rem = grid % 8, x = bid % 8;
    return x * q + (x < rem ? x : rem) + bid / 8;
}

// What a lane reads whose piece of a row lies past the reduction depth (nothing writes it; not const, so that the read
// stays an ordinary load from a selected address).
[[maybe_unused]] static __device__ uint4 g_zero_piece = {0u, 0u, 0u, 0u};

// (The address is settled before the load: left to itself the compiler turns a selected address into two loads behind
// branches, and waits for them where the branches meet.)
template <class V>
__device__ inline V load_piece(const char* p)
{
    typedef __attribute__((address_space(1))) const V global_piece;
    uint64_t a = (uint64_t)p;
    asm("" : "+v"(a));
    return *(global_piece*)a;
}

// two fp32 -> two bf16 (round to nearest even, the conversion instruction of this part), first argument
// in the low half
__device__ inline uint32_t pack_bf16(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    const floatx2 v = {a, b};
    const bf16x2 h = __builtin_convertvector(v, bf16x2);
    uint32_t u;
    __builtin_memcpy(&u, &h, 4);
    return u;
}
__device__ inline float low_half(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float high_half(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uintx2 lds_uintx2;

// Both operands of a product in three terms are taken times this: the terms of a float then end at 2^-133, the
// smallest bf16, or above, and are exact for every float, the subnormal ones too (unscaled, operands below 1e-33
// lose bits of the third term: relative error 3e-6 at 1e-35, 3e-4 at 1e-37).  A sum that overflows by it is not
// finite and is computed again in fp32.  Costs one multiply per operand and per sum: gradients of 2^20 rows
// 256 x 256 855 -> 863 us (weights) and 831 -> 845 (data), masked ones within noise.
constexpr float kTermScale = 65536.f;

// Four fp32 of a row on their way to LDS: the three bf16 planes of the (masked) values times
// `scale`.
template <bool MASK>
__device__ inline void split_store(const float4& a, const float4& r, float scale, uint16_t* p0, uint16_t* p1,
                                   uint16_t* p2)
{
    float4 x = a;
    if (MASK) {
        x.x = r.x > 0.f ? x.x : 0.f;
        x.y = r.y > 0.f ? x.y : 0.f;
        x.z = r.z > 0.f ? x.z : 0.f;
        x.w = r.w > 0.f ? x.w : 0.f;
    }
    x = make_float4(x.x * scale, x.y * scale, x.z * scale, x.w * scale);
    const uintx2 t0 = {pack_bf16(x.x, x.y), pack_bf16(x.z, x.w)};
    x.x -= low_half(t0.x);
    x.y -= high_half(t0.x);
    x.z -= low_half(t0.y);
    x.w -= high_half(t0.y);
    const uintx2 t1 = {pack_bf16(x.x, x.y), pack_bf16(x.z, x.w)};
    x.x -= low_half(t1.x);
    x.y -= high_half(t1.x);
    x.z -= low_half(t1.y);
    x.w -= high_half(t1.y);
    const uintx2 t2 = {pack_bf16(x.x, x.y), pack_bf16(x.z, x.w)};
    *(lds_uintx2*)p0 = t0;
    *(lds_uintx2*)p1 = t1;
    *(lds_uintx2*)p2 = t2;
}

// x with the halves zeroed whose reference half (bf16 bits) is not > 0: 1 .. 0x7F80 are the positive values up
// to +inf.  r - 1 is then below 0x7F80, and 0x7F80 less that, saturated, positive exactly for them; its negation
// has the sign bit set, which an arithmetic shift spreads over the half.
__device__ inline uint32_t keep_positive(uint32_t x, uint32_t r)
{
    typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
    typedef short short2v __attribute__((ext_vector_type(2)));
    ushort2v rr;
    __builtin_memcpy(&rr, &r, 4);
    const ushort2v one = {1, 1}, inf = {0x7F80, 0x7F80};
    const ushort2v above = __builtin_elementwise_sub_sat(inf, (ushort2v)(rr - one));
    short2v a;
    __builtin_memcpy(&a, &above, 4);
    const short2v keep = (-a) >> 15;
    uint32_t k;
    __builtin_memcpy(&k, &keep, 4);
    return x & k;
}

// The elements of rows [row0, row1) and columns [col0, col1) of C that are not finite, again as chains of fp32
// multiply-adds over the reduction index (a term of an infinity is NaN, a value next to the largest float
// rounds up to an infinity as bf16); then, with RELU, the activation of all of them.  C holds the sums of the
// calling wavefront, written by it and not yet activated.  a_at(row, k), w_at(k, col): the operands.
template <bool RELU, class FA, class FW>
__device__ inline void repair_sums(float* C, int64_t ldc, int64_t row0, int64_t row1, int col0, int col1, int KD,
                                   FA a_at, FW w_at)
{
    __threadfence();  // what the wavefront wrote is read by its other lanes
    const int cols = col1 - col0;
    const int64_t cells = cols > 0 ? (row1 - row0) * cols : 0;
    for (int64_t i = threadIdx.x & (kWave - 1); i < cells; i += kWave) {
        const int64_t row = row0 + i / cols;
        const int col = col0 + (int)(i % cols);
        float* const c = C + row * ldc + col;
        float x = __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!(fabsf(x) <= 3.402823466e38f)) {
            x = 0.f;
            for (int k = 0; k < KD; ++k) x = fmaf(a_at(row, k), w_at(k, col), x);
        } else if (!RELU) {
            continue;
        }
        *c = RELU ? fmaxf(x, 0.f) : x;
    }
}

// Workgroups of a product whose weights stay in LDS and whose wavefronts walk tiles of rows: row_groups groups of
// rows (a multiple of 8, one XCD each), one workgroup per group and column tile, `waves` walking wavefronts each.
struct RowWalk {
    int row_groups, waves;
    unsigned grid;
};
inline RowWalk plan_row_walk(int64_t tiles, int n_col_tiles, int most_waves, bool all_waves)
{
    // One workgroup per compute unit.  Where there are fewer tiles than wavefronts the workgroups get
    // fewer wavefronts rather than the chip fewer workgroups (4096 rows 64 -> 32: 16 workgroups of 8 took
    // 8.2 us, 128 of one take 5.0).
    int64_t per_xcd = 32 / n_col_tiles;
    if (per_xcd < 1) per_xcd = 1;
    // Where the column tiles leave compute units of an XCD idle that way (11 of them take 22 of 32), more
    // groups of rows and several rounds of workgroups, if that saves a tenth: a round costs a wavefront its
    // tiles, and the weights about another.  us at 2^17 rows 128 -> 1408, 2176, 4224, one round : several, bf16
    // 134 : 124, 252 : 190, 524 : 380, fp32 data gradient 321 : 300, 598 : 455, 1257 : 887; with 384 to 1280 columns
    // several rounds took up to a sixth longer.
    const auto cost = [&](int64_t groups) {
        return ceil_div(groups * n_col_tiles, 32) * (ceil_div(tiles, 8 * most_waves * groups) + 1);
    };
    int64_t least = cost(per_xcd) * 9 / 10;
    for (int64_t p = per_xcd + 1; p <= 32; ++p)
        if (cost(p) < least) {
            least = cost(p);
            per_xcd = p;
        }
    const int64_t per_group = ceil_div(tiles, 8 * per_xcd);
    const int waves = all_waves || per_group > most_waves ? most_waves : (int)per_group;
    const int64_t need = ceil_div(ceil_div(tiles, waves), 8);
    if (per_xcd > need) per_xcd = need;
    return RowWalk{(int)per_xcd * 8, waves, (unsigned)(8 * per_xcd * n_col_tiles)};
}

}  // namespace mixgcn
