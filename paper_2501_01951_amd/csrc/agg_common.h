// Device helpers shared by the two aggregation kernels: feature vectors, sub-group sums, epilogues.
#pragma once
#include <type_traits>

#include "device_utils.h"
#include "internal.h"

namespace mixgcn {
namespace {

// 16-byte feature vector: 4 fp32, or 8 bf16 widened to fp32.
template <int DT>
struct Feat {
    static constexpr int ES = DT == MIXGCN_F32 ? 4 : 2;  // bytes per stored element
    static constexpr int VEC = 16 / ES;
    static constexpr int WORDS = 4;
    using Raw = uint4;
    __device__ static inline void widen(const Raw& r, float* o)
    {
        uint32_t w[WORDS];
        __builtin_memcpy(w, &r, 16);
#pragma unroll
        for (int i = 0; i < WORDS; ++i) {
            if (DT == MIXGCN_F32) {
                o[i] = __uint_as_float(w[i]);
            } else {
                o[2 * i] = __uint_as_float(w[i] << 16);
                o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
            }
        }
    }
    // two fp32 -> two bf16, round to nearest even, by the conversion instruction of this part
    // (rounding in software made a row's end a third of the vector work of this kernel at bf16)
    __device__ static inline uint32_t pack2(float lo, float hi)
    {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float floatx2 __attribute__((ext_vector_type(2)));
        const floatx2 v = {lo, hi};
        const bf16x2 h = __builtin_convertvector(v, bf16x2);
        uint32_t u;
        __builtin_memcpy(&u, &h, 4);
        return u;
    }
    __device__ static inline void store(void* base, int64_t elem_off, const float* a)
    {
        uint32_t w[WORDS];
#pragma unroll
        for (int i = 0; i < WORDS; ++i)
            w[i] = DT == MIXGCN_F32 ? __float_as_uint(a[i]) : pack2(a[2 * i], a[(2 * i + 1) % VEC]);
        Raw r;
        __builtin_memcpy(&r, w, 16);
        *reinterpret_cast<Raw*>(reinterpret_cast<char*>(base) + elem_off * ES) = r;
    }
    __device__ static inline void store_one(void* base, int64_t elem_off, float a)
    {
        if (DT == MIXGCN_F32) reinterpret_cast<float*>(base)[elem_off] = a;
        else reinterpret_cast<uint16_t*>(base)[elem_off] = (uint16_t)pack2(a, 0.f);
    }
    __device__ static inline const Raw* ptr(const void* base, int64_t elem_off)
    {
        return reinterpret_cast<const Raw*>(reinterpret_cast<const char*>(base) + elem_off * ES);
    }
};

// Writes a lane's VEC columns [c, c + VEC) of one output row: the whole group when it
// lies inside the call's column range [c_lo, c_hi), else only the elements that do, one by one
// (a range need not start or end on a group; what lies outside it is never written).
template <int DT>
__device__ inline void store_in_range(void* Z, int64_t row_off, int64_t c, const float* t, int c_lo,
                                      int c_hi)
{
    using F = Feat<DT>;
    if (c >= c_lo && c + F::VEC <= c_hi) {
        F::store(Z, row_off + c, t);
    } else {
#pragma unroll
        for (int i = 0; i < F::VEC; ++i)
            if (c + i >= c_lo && c + i < c_hi) F::store_one(Z, row_off + c + i, t[i]);
    }
}

// A value that is the same in every lane, moved to scalar registers.
__device__ inline int uniform32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uniform64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Sum over the 64 / LPR sub-groups of a wavefront (lanes that hold the same columns).
template <int LPR, int VEC>
__device__ inline void reduce_subgroups(float* v)
{
#pragma unroll
    for (int d = LPR; d < kWave; d <<= 1)
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] += __shfl_xor(v[i], d, kWave);
}

// The same sums, in the same tree, written to out[0 .. VEC) of the lanes of sub-group 0 (out: where the
// lane's position in its slice puts them; null: nowhere).  Lanes never go through LDS: neighbors 4 and 8
// away are added by DPP, and the exchanges of halves and quarters of the wavefront are swaps of two
// registers, after which each half works on elements of its own: 10 instructions for four elements and 20
// for eight, instead of 24 and 48 of which half wait for LDS.
template <int LPR, int VEC>
__device__ inline void combine_subgroups(float* v, int lane, float* out)
{
    if constexpr (LPR > 8) {  // (the whole-row measurement mode)
        reduce_subgroups<LPR, VEC>(v);
        if (lane < LPR && out) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) out[i] = v[i];
        }
    } else {
        auto dpp = [](float x, auto ctrl) {
            return __uint_as_float(
                __builtin_amdgcn_update_dpp(0, __float_as_uint(x), decltype(ctrl)::value, 0xF, 0xF, false));
        };
        // lane i takes lane i + 4 (row rotation by 12; right where bit 2 of i is clear), then i ^ 8
        if constexpr (LPR == 4) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) v[i] += dpp(v[i], std::integral_constant<int, 0x12C>{});
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] += dpp(v[i], std::integral_constant<int, 0x128>{});
        // bit 4 of the lane: 0 sums the lower half of the elements, 1 the upper half; bit 5 halves again
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i) {
            const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + VEC / 2]),
                                                            false, false);
            v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
#pragma unroll
        for (int i = 0; i < VEC / 4; ++i) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + VEC / 4]),
                                                            false, false);
            v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
        if ((lane & 15) < LPR && out) {
            float* o = out + ((lane >> 4) & 1) * (VEC / 2) + (lane >> 5) * (VEC / 4);
#pragma unroll
            for (int i = 0; i < VEC / 4; ++i) o[i] = v[i];
        }
    }
}

// Output mask of the S-SpMM (paper Eq. 4), a bitmap: column c of row r is bit c % 32 of word
// mask[r * ldm + c / 32].  A lane's VEC consecutive columns start at a multiple of VEC, so
// their bits lie in one word.
template <int VEC>
__device__ inline void apply_mask(float* t, const uint32_t* __restrict__ mask, int64_t ldm,
                                  int64_t r, int64_t c)
{
    const uint32_t bits = mask[r * ldm + (c >> 5)] >> (c & 31);
#pragma unroll
    for (int i = 0; i < VEC; ++i) t[i] = ((bits >> i) & 1u) ? t[i] : 0.f;
}

// Epilogue flags carried in the kernels' `relu` argument (MIXGCN_EPI_* of the ABI).
constexpr int kEpiRelu = 1;        // Z = max(., 0)
constexpr int kEpiAccumulate = 2;  // Z = Z + (.): the finished row sum is added to what Z holds

template <int DT>
__device__ inline void add_stored(float* t, const void* Z, int64_t elem_off)
{
    using F = Feat<DT>;
    float o[F::VEC];
    F::widen(*F::ptr(Z, elem_off), o);
#pragma unroll
    for (int i = 0; i < F::VEC; ++i) t[i] += o[i];
}

}  // namespace
}  // namespace mixgcn
