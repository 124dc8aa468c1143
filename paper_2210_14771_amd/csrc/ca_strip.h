// Half strips walked by waves in steps: the geometry, the pixels and the
// candidates that both learned scorers' strip kernels share.
#pragma once

#include "ca_internal.h"
#include "ca_mfma.h"

namespace ca {

constexpr int kStep = 64;         // positions a wave advances by
constexpr int kStripWaves = 8;    // waves of a workgroup

// LDS written by some lanes of the wave and read by others next: keep the
// compiler from moving memory operations across (the hardware keeps a wave's
// LDS operations in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A half strip, or a part of one, as a wave walks along it.
struct StripWalk {
    const uint8_t *frame;
    int64_t along, across;   // bytes from position to position, from line to line
    int first;               // first line (may lie outside the frame)
    int L, lines;            // positions; lines of the frame
    bool packed;             // a position's 24 bytes adjoin and lie in the frame
    bool last_row;           // the frame's last pixel may be among the inputs
};

// A lane's inputs of a step, position x + lane: 24 bytes, or a dword of three
// bytes for each line.  A dword's fourth byte may belong to the next pixel or
// row; only the frame's last pixel has none.
template <int LINES>
__device__ __forceinline__ void strip_fetch(uint32_t (&px)[8], const StripWalk &k, int x, int lane)
{
    int p = x + lane;
    p = p < 0 ? 0 : (p > k.L - 1 ? k.L - 1 : p);
    const uint8_t *q = k.frame + p * k.along;
    if (k.packed) {
        __builtin_memcpy(px, q + k.first * k.across, 24);
        return;
    }
    const uint8_t *v[LINES];
#pragma unroll
    for (int j = 0; j < LINES; ++j) {
        int line = k.first + j;
        line = line < 0 ? 0 : (line > k.lines - 1 ? k.lines - 1 : line);
        v[j] = q + line * k.across;
    }
    if (k.last_row && x + kStep >= k.L) {
#pragma unroll
        for (int j = 0; j < LINES; ++j)
            px[j] = v[j][0] | (uint32_t)v[j][1] << 8 | (uint32_t)v[j][2] << 16;
    } else {
#pragma unroll
        for (int j = 0; j < LINES; ++j)
            __builtin_memcpy(&px[j], v[j], 4);
    }
}

template <int LINES>
__device__ __forceinline__ void strip_walk(StripWalk &k, const uint8_t *frames, const FrameDev &d,
                                           bool horizontal, int pos)
{
    k.frame = frames + d.offset;
    k.along = horizontal ? 3 : d.rs;
    k.across = horizontal ? d.rs : 3;
    k.first = pos - 3;
    k.L = uniform_int(horizontal ? d.W : d.H);
    k.lines = uniform_int(horizontal ? d.H : d.W);
    k.packed = !horizontal && pos >= 3 && pos + 4 < k.lines;
    k.last_row = k.first + LINES >= k.lines;
}

// Four tiles' values added over the lane groups as (0 + 1) + (2 + 3): lane
// group q receives tile q's sum.
__device__ __forceinline__ float tile_sums(const float (&v)[4])
{
    uint32_t z0 = __float_as_uint(v[0]), z1 = __float_as_uint(v[1]);
    uint32_t z2 = __float_as_uint(v[2]), z3 = __float_as_uint(v[3]);
    swap_rows(z0, z1);
    swap_rows(z2, z3);
    uint32_t low = __float_as_uint(__uint_as_float(z0) + __uint_as_float(z1));
    uint32_t high = __float_as_uint(__uint_as_float(z2) + __uint_as_float(z3));
    swap_halves(low, high);
    return __uint_as_float(low) + __uint_as_float(high);
}

// Keys whose maximum is the best-scoring pixel of a half strip (ties:
// outermost); key 0 is no pixel's.
__device__ __forceinline__ uint64_t strip_key(float z, int p, int half, int L)
{
    return ((uint64_t)__float_as_uint(sigmoid(z)) << 32)
           | (uint64_t)(0xFFFFFFFFu - (uint32_t)(half ? L - 1 - p : p));
}
__device__ __forceinline__ uint64_t wave_max(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint64_t t = __shfl_xor(v, d, 64);
        v = v > t ? v : t;
    }
    return v;
}
__device__ __forceinline__ ca_point strip_point(uint64_t key, bool horizontal, int pos, int half,
                                                int L)
{
    const int k = (int)(0xFFFFFFFFu - (uint32_t)key);
    const int i = half == 0 ? k : L - 1 - k;
    ca_point pt;
    pt.x = (int16_t)(horizontal ? i : pos);
    pt.y = (int16_t)(horizontal ? pos : i);
    pt.score = __uint_as_float((uint32_t)(key >> 32));
    return pt;
}

// Waves that share a half strip and workgroups per XCD, for `units` half strips
// an XCD of frames of at most `longest` pixels a side, at most `resident`
// workgroups an XCD and a halo of `halo` positions: the split with the fewest
// steps until the last wave ends.  Frames of one shape are taken by resident
// workgroups in turns; of several shapes (mixed) each workgroup takes one turn
// and the dispatch evens out their lengths, for about a step's time of loading
// weights.  A wave alone on a half strip of full HD takes 16 steps of some 3 us.
inline int strip_split(int32_t &parts, int units, int resident, int longest, bool mixed, int halo)
{
    int64_t best = 0;
    for (int32_t p = 1; p <= kStripWaves; p *= 2) {
        const int64_t slots = (int64_t)resident * kStripWaves;
        const int64_t turns = ((int64_t)units * p + slots - 1) / slots;
        const int64_t steps = (((longest + 1) / 2 + p - 1) / p + 2 * halo + kStep - 1) / kStep;
        const int64_t cost = turns * (steps + (mixed ? 1 : 0));
        if (p == 1 || cost < best) {
            best = cost;
            parts = p;
        }
    }
    const int sets = kStripWaves / parts;
    const int groups = (units + sets - 1) / sets;
    return mixed || groups < resident ? groups : resident;
}

}  // namespace ca
