// Tiles of bf16 features on their way through LDS: shared by the weight gradient and the deep row products.
#pragma once
#include "gemm_common.h"

namespace mixgcn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BKB = 32;       // reduction depth staged per step (bf16 elements)
constexpr int LDT = BKB + 8;  // LDS row stride: 80 bytes, so 16-byte reads of 16 rows hit all banks

// Eight bf16 of a feature tile on their way from global memory to LDS: issue() starts the
// loads from an address clamped into the matrix, value() zeroes what lies outside it and, with
// MASK, what the ReLU-derivative mask 1[R > 0] removes.
template <bool MASK>
struct Piece8 {
    uint4 v, m;
    int nvalid;  // leading elements inside the matrix (0..8)

    __device__ inline void issue(const uint16_t* __restrict__ M, int64_t ld, int64_t r, int c,
                                 int64_t rows, int cols, const uint16_t* __restrict__ R,
                                 int64_t ldr)
    {
        const bool ok = r < rows && c < cols;
        nvalid = ok ? (cols - c < 8 ? cols - c : 8) : 0;
        const int64_t rr = r < rows ? r : rows - 1;
        const int cc = c < cols ? c : 0;
        v = *reinterpret_cast<const uint4*>(M + rr * ld + cc);
        if (MASK) m = *reinterpret_cast<const uint4*>(R + rr * ldr + cc);
        else m = make_uint4(0u, 0u, 0u, 0u);
    }
    __device__ static inline uint32_t keep_word(uint32_t x, uint32_t r, int left)
    {
        uint32_t keep = 0;
        if (left > 0) keep |= 0x0000FFFFu;
        if (left > 1) keep |= 0xFFFF0000u;
        if (MASK) {
            if (!(__uint_as_float(r << 16) > 0.f)) keep &= 0xFFFF0000u;
            if (!(__uint_as_float(r & 0xFFFF0000u) > 0.f)) keep &= 0x0000FFFFu;
        }
        return x & keep;
    }
    __device__ inline uint4 value() const
    {
        uint4 o;
        o.x = keep_word(v.x, m.x, nvalid);
        o.y = keep_word(v.y, m.y, nvalid - 2);
        o.z = keep_word(v.z, m.z, nvalid - 4);
        o.w = keep_word(v.w, m.w, nvalid - 6);
        return o;
    }
};

__device__ inline bf16x8 lds_operand(const uint16_t* p)
{
    return *reinterpret_cast<const bf16x8*>(p);
}

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uintx4 lds_uintx4;
__device__ inline void lds_store16(uint16_t* p, const uint4& v)
{
    const uintx4 q = {v.x, v.y, v.z, v.w};
    *(lds_uintx4*)p = q;
}

}  // namespace mixgcn
