// Device helpers of the MFMA kernels (the two learned scorers, RANSAC).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS written by some lanes of the wave and read by others next: keep the
// compiler from moving memory operations across (the hardware keeps a wave's
// LDS operations in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ __bf16 to_bf16(float v) { return (__bf16)v; }
__device__ __forceinline__ float sigmoid(float z) { return 1.0f / (1.0f + __expf(-z)); }

__device__ __forceinline__ bf16x8 frag_at(const __bf16 *p)
{
    return *reinterpret_cast<const bf16x8 *>(p);
}
// One 16x16 tile of D += A (16 x 32) * B (32 x 16): lane l holds
// A[l % 16][8 (l / 16) ..], B[8 (l / 16) ..][l % 16] and D[4 (l / 16) ..][l % 16].
// The four lane groups' K blocks of 8 are added in turn (measured: splitting a
// step between blocks, or shifting the blocks, gives the same bits), so GEMMs
// that meet the same blocks in the same order round alike.
__device__ __forceinline__ f32x4 mma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Eight K values of one column of a position-major LDS buffer: the four
// channels of a row at p, and at q, transposed over the lane's group of 16
// (ds_read_b64_tr_b16: lane i of a group receives column i of the 4 rows x 16
// columns whose 8-byte pieces its lanes address, four lanes a row).
__device__ __forceinline__ bf16x8 transposed(const __bf16 *p, const __bf16 *q)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)q);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Exchanges of two registers by rows of 16 lanes: lane groups 0..3 hold
// a0 a1 a2 a3 and b0 b1 b2 b3 before, a0 b0 a2 b2 and a1 b1 a3 b3 after
// swap_rows, a0 a1 b0 b1 and a2 a3 b2 b3 after swap_halves.
__device__ __forceinline__ void swap_rows(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// The 1x1 layer in the registers of the convolution before it: b + sum_o w[o]
// h[o] over 16 MT channels in ascending order, one fused multiply-add each,
// for two tiles.  Lane group g holds channels 16 mt + 4 g .. + 3 of its
// column's position in both; the even groups receive all of tile 0's channels
// and return its sum, the odd ones tile 1's.
template <int MT>
__device__ __forceinline__ float ordered_dot(const float *w, const bf16x4 (&h)[2][MT], float b)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    float z = b;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const u32x2 h0 = __builtin_bit_cast(u32x2, h[0][mt]);
        const u32x2 h1 = __builtin_bit_cast(u32x2, h[1][mt]);
        uint32_t x[4][2];   // [source group][channel pair]
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t even = h0[i], odd = h1[i];
            swap_rows(even, odd);
            x[0][i] = x[2][i] = even;
            x[1][i] = x[3][i] = odd;
            swap_halves(x[0][i], x[2][i]);
            swap_halves(x[1][i], x[3][i]);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 wg = *reinterpret_cast<const f32x4 *>(w + 16 * mt + 4 * g);
            const u32x2 pair = {x[g][0], x[g][1]};
            const bf16x4 hg = __builtin_bit_cast(bf16x4, pair);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                z = fmaf(wg[j], (float)hg[j], z);
        }
    }
    return z;
}

// The values of the even lane groups' column for tile 0 and of the odd ones'
// for tile 1, both in every lane.
__device__ __forceinline__ void to_all_groups(float v, float (&tile)[2])
{
    uint32_t a = __builtin_bit_cast(uint32_t, v), b = a;
    swap_rows(a, b);
    tile[0] = __builtin_bit_cast(float, a);
    tile[1] = __builtin_bit_cast(float, b);
}

// The same value, which the compiler takes for a new one: offsets derived
// from it are computed where they are used instead of being kept in registers
// over a whole window loop (beside a gradient kernel's accumulators they
// spilled, and every reload was waited for).
__device__ __forceinline__ int fresh(int v)
{
    asm("" : "+v"(v));
    return v;
}

// ReLU and the frame / strip mask in one median: clamp to [0, +inf) where
// the activation exists (top = inf), to [0, 0] elsewhere; stored as bfloat16.
__device__ __forceinline__ bf16x4 relu_bf16(const f32x4 &acc, float top)
{
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        o[j] = to_bf16(__builtin_amdgcn_fmed3f(acc[j], 0.0f, top));
    return o;
}

// v where the activation h is positive, else zero, as bfloat16.  h is a
// ReLU's output, so positive means not all bits zero.
__device__ __forceinline__ bf16x4 relu_mask(const f32x4 &v, const bf16x4 &h)
{
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    const u16x4 bits = __builtin_bit_cast(u16x4, h);
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        o[j] = to_bf16(bits[j] != 0 ? v[j] : 0.0f);
    return o;
}

// A lane's place in the 16 x 32 fragments of its wave: column of a tile and
// lane group; for transposed reads its row 4 g + col / 4 (and the one 16 on:
// K index 8 g + e of a fragment is row 4 g + e for e < 4, 16 + 4 g + e - 4
// otherwise, in both operands) and its chunk q = col % 4 of four channels.
struct Place {
    int col, g, q, r;
    __device__ __forceinline__ explicit Place(int lane)
        : col(lane & 15), g(lane >> 4), q(col & 3), r(4 * g + (col >> 2))
    {
    }
};

}  // namespace ca
