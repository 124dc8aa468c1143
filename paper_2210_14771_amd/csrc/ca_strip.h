// Half strips walked by waves in steps: the geometry, the pixels and the
// candidates that both learned scorers' strip kernels share.
#pragma once

#include "ca_deal.h"
#include "ca_internal.h"
#include "ca_mfma.h"

namespace ca {

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

// A key of a piece of a half strip that several workgroups share, kept in `word`
// until the last of `parts` of them comes, whose key becomes the best of all
// (true) and which leaves the word zero, as it was.  Nobody waits: the word holds
// the best key so far (of the distance 14 bits suffice) and the number of keys.
__device__ __forceinline__ bool edge_merge(uint64_t *word, uint64_t &key, int parts)
{
    constexpr uint64_t kScore = 0xFFFFFFFF00000000ull, kCount = 0xFFFFu;
    const uint64_t mine = (key & kScore) | (key & 0xFFFFu) << 16;
    uint64_t old = 0;   // as the first one finds it
    for (;;) {
        const uint64_t best = mine > (old & ~kCount) ? mine : old & ~kCount;
        const uint64_t count = (old & kCount) + 1;
        if (count == (uint64_t)parts) {   // (never of the guess: parts > 1)
            __hip_atomic_store(word, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            key = (best & kScore) | 0xFFFF0000u | (best >> 16 & 0xFFFFu);
            return true;
        }
        if (__hip_atomic_compare_exchange_strong(word, &old, best | count, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return false;
    }
}

// Read-only data at a uniform address, through the scalar cache: a wave's vector
// loads would wait for its weights, and for the candidate that it stored last.
template <class T>
__device__ __forceinline__ T uniform_load(const T *p)
{
    static_assert(sizeof(T) % 4 == 0, "dwords");
    typedef uint32_t words __attribute__((ext_vector_type(sizeof(T) / 4)));
    typedef const words __attribute__((address_space(4))) *const_ptr;
    return __builtin_bit_cast(T, *(const_ptr)(uintptr_t)p);
}

// A half strip, its entries in the launch's list from `start` on.
struct StripHalf {
    int frame, unit, pos, L, start, entries;
};
// What the waves of a workgroup share: best keys (0: of the half strip that an
// earlier workgroup began, 1 + w: of the one that wave w begins and does not end),
// and the former half strip.
struct StripMeet {
    uint64_t best[kStripWaves + 1];
    StripHalf ended;
};

// The candidates of a launch: this wave's share of the half strips.
// piece(frame, horizontal, pos, half, p0, p1): the best key of positions [p0, p1)
// of a half strip.  The waves that share a half strip meet in `meet` (best keys
// zero on entry), and workgroups in the launch's edge words, at the first one's.
// All threads of the workgroup call this.  MIXED: the frames differ in shape.
// SCALAR: half strips are looked up through the scalar cache (1-D network, 64 x
// 1080p with fallback: 219 us a call otherwise, 216 so; of the 2-D network the two
// waves of a SIMD then run in step and meet in its layers: 218 us a launch
// otherwise, 228 so).
template <int HALO, bool MIXED, bool SCALAR, class Args, class Piece>
__device__ __forceinline__ void strip_shares(const Args &a, StripMeet &meet, int lane, int wv,
                                             Piece piece)
{
    const int S = a.n_h + a.n_v;
    const int n = a.n_items / S;
    const int group = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int w0 = group * kStripWaves, w = w0 + wv;
    StripDeal deal = a.deal;
    int &row = deal.row, &col = deal.col, &each = deal.each;
    auto entries_of = [&](int f) {
        const FrameDev &d = a.fd[a.frame0 + f];
        row = extent_entries(d.W, HALO, deal);
        col = extent_entries(d.H, HALO, deal);
        each = 2 * (a.n_h * row + a.n_v * col);
    };
    // entries of frames base .. base + 63 up to and with this lane's
    auto scan = [&](int base) {
        int v = 0;
        if (base + lane < n) {
            entries_of(base + lane);
            v = each;
        }
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const int t = __shfl_up(v, d, 64);
            v += lane >= d ? t : 0;
        }
        return v;
    };
    int f = 0, r = 0;   // frame, entry within it
    int t, end;
    if (!MIXED) {
        t = wave_start(deal, w);
        end = wave_start(deal, w + 1);
        f = t / each;
        r = t - f * each;
    } else {
        int upto = scan(0), total = __shfl(upto, 63, 64);
        for (int base = 64; base < n; base += 64)
            total += __shfl(scan(base), 63, 64);
        total = uniform_int(total);
        deal.share = total / (int)gridDim.x;
        deal.extra = total - deal.share * (int)gridDim.x;
        t = wave_start(deal, w);
        end = wave_start(deal, w + 1);
        r = t;
        for (int base = 0; t < end; base += 64) {
            if (base)
                upto = scan(base);
            const uint64_t later = __ballot(upto > r);
            if (later) {
                const int at = __builtin_ctzll(later);
                f = base + at;
                r -= at ? uniform_int(__shfl(upto, at - 1, 64)) : 0;
                break;
            }
            r -= uniform_int(__shfl(upto, 63, 64));
        }
    }

    auto write = [&](const StripHalf &h, uint64_t key) {
        if (lane == 0)
            a.cand[(int64_t)h.frame * (2 * S) + h.unit] =
                strip_point(key, h.unit < 2 * a.n_h, h.pos, h.unit & 1, h.L);
    };
    StripHalf h;
    int table = -1;
    bool begins = false, ends = false;   // whether this wave completes a shared half strip
    if (MIXED && t < end)
        entries_of(f);
    StripPlace q = {};
    if (t < end)
        q = strip_place(deal, a.n_h, a.n_v, r);
    while (t < end) {
        h.frame = uniform_int(a.frame0 + f);
        const FrameDev d = SCALAR ? uniform_load(a.fd + h.frame) : a.fd[h.frame];
        const bool horizontal = uniform_int(q.horizontal) != 0;
        const int half = uniform_int(q.half), at = uniform_int(q.at);
        h.entries = uniform_int(q.entries);
        h.unit = uniform_int(2 * (horizontal ? q.strip : a.n_h + q.strip)) + half;
        if (MIXED || table < 0)   // (frames of one shape share the table)
            table = uniform_int(d.table);
        const int32_t *pos = a.strips + table + (h.unit >> 1);
        h.pos = SCALAR ? uniform_load(pos) : uniform_int(*pos);
        h.start = t - at;
        h.L = uniform_int(horizontal ? d.W : d.H);
        const int h0 = half ? h.L >> 1 : 0, len = half ? h.L - (h.L >> 1) : h.L >> 1;
        const int to = min(h.entries, at + end - t);
        const int from = at ? uniform_int(wave_of(deal, h.start)) : w;   // its first wave
        auto start_of = [&](int entry, int waves) {
            return piece_start(len, HALO, entry, cuts_before(deal.share, entry, waves), deal.grain);
        };
        const int p0 = h0 + (at ? start_of(at, w - from) : 0);
        const int p1 = h0 + (to == h.entries ? len : start_of(to, w - from + 1));
        const uint64_t best = piece(d, horizontal, h.pos, half, p0, p1);
        if (to - at == h.entries) {
            write(h, best);
        } else {
            if (lane == 0)
                atomicMax((unsigned long long *)&meet.best[from < w0 ? 0 : 1 + from - w0],
                          (unsigned long long)best);
            begins = from == w;   // (the last piece then)
            if (from < w0 && wv == 0) {
                ends = true;
                meet.ended = h;
            }
        }
        t += to - at;
        if (!strip_next(deal, a.n_h, a.n_v, q)) {
            ++f;
            if (MIXED && t < end) {
                entries_of(f);
                q.entries = q.horizontal ? row : col;
            }
        }
    }
    __syncthreads();
    auto complete = [&](const StripHalf &h, uint64_t key) {
        const int first = group_of(deal, h.start);
        const int last = group_of(deal, h.start + h.entries - 1);
        bool all = true;
        if (last > first && lane == 0)
            all = edge_merge(a.edges + first, key, last - first + 1);
        if (all)
            write(h, key);
    };
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
        if (k == 0 ? begins : ends)
            complete(h, meet.best[k == 0 ? 1 + wv : 0]);
        h = meet.ended;
    }
}

}  // namespace ca
