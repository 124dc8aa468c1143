// gfx950 kernels of the paper's own learned edge scorer (arXiv 2210.14771,
// Section 2.2.4): three 3x3 convolutions with 8, 16 and 32 output features,
// each followed by a ReLU, a 1x1 convolution to one logit and a sigmoid, on
// RGBXY input (colours normalised by the training data's per-channel mean
// and standard deviation, pixel coordinates normalised to [-0.5, 0.5] about
// the image centre), applied to strips seven lines thick (the network's
// receptive field), so a strip's scores are the whole-image network's output
// on the strip's centre line.
//
// A strip is processed in windows of 128 positions: band lines 0..6 (the
// strip line -3 .. +3) of the input, lines 1..5 of layer 1, 2..4 of layer 2
// and line 3 of layer 3.  Each layer is one GEMM per output line on
// v_mfma_f32_16x16x32_bf16: activations are stored position-major
// ([line][position][channel], channels contiguous, one zero guard position
// at each end), so the 8 channels of one tap at one position are one
// 16-byte LDS load, and K = (3 da + dl) C_pad + c walks the 3x3 taps.  For a
// vertical strip the band's lines are frame columns: the weights' two
// spatial axes swap roles, so the model block holds both orientations.
// Every layer's input is zero outside the frame and beyond the strip ends
// ("same" zero padding of the whole-image network).  Weights and hidden
// activations are bfloat16, sums are float32 MFMA accumulators.
#include "ca_cnn.h"
#include "ca_launch.h"
#include "ca_mfma.h"
#include "ca_reduce.h"
#include "ca_strip.h"

namespace ca {
namespace {

constexpr int kPos = kC2Win + 2;   // positions of a buffer line, guards included
constexpr int kTrainHalo = 8;      // training windows carry logits 8 .. 119
constexpr int kTrainOut = kC2Win - 2 * kTrainHalo;
constexpr int kC2Floats = 96;      // floats of the model's float block
constexpr int kWaves = kBlock / 64;
constexpr int kC2WindowBlock = 128;   // window logits: two waves, a window each

// The A operand of a layer's GEMMs (weights [M][KP], M = 16 MT output
// channels) as this lane's MFMA fragments: loaded once, kept in registers
// for every tile of every window the workgroup computes.
template <int KP, int MT>
struct Frag {
    bf16x8 a[MT][KP / 32];
};

template <int KP, int MT>
__device__ __forceinline__ Frag<KP, MT> load_frag(const __bf16 *A)
{
    const int lane = threadIdx.x & 63;
    Frag<KP, MT> f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks)
            f.a[mt][ks] = *reinterpret_cast<const bf16x8 *>(A + (mt * 16 + (lane & 15)) * KP
                                                            + 32 * ks + 8 * (lane >> 4));
    return f;
}

// Coordinates are normalised to [-0.5, 0.5] as (2 x - (W - 1)) / (2 (W - 1)),
// taken as a product with this reciprocal.
__device__ __forceinline__ float coord_scale(int extent) { return 1.0f / (float)(2 * (extent - 1)); }

__device__ __forceinline__ bool line_in(uint32_t line_ok, int j) { return (line_ok >> j) & 1u; }

__device__ __forceinline__ uint32_t band_lines(int line, int extent)
{
    uint32_t ok = 0;
    for (int j = 0; j < kC2Band; ++j) {
        const int r = line - 3 + j;
        ok |= (r >= 0 && r < extent) ? (1u << j) : 0u;
    }
    return ok;
}

// ----------------------------------------------------------- inference --

// Learned candidates: the best-scoring pixel of each half strip (ties:
// outermost).  A wave walks along a half strip, or along a part of one, in
// steps of 64 positions with private LDS buffers and the layers' weights of the
// strip's orientation in its registers: layer l works one position per layer
// behind the input, so a step's outputs need only the step's positions of the
// layer before and its last two of the step before, which stay at the head of
// the layer's lines.  The next step's pixels are loaded while a step's layers
// run.
//
// Bound by issue: about 490 vector instructions of 4 cycles and 112 MFMAs of 16
// a step, which add up to four fifths of a SIMD's cycles.  Measured, 64 1080p
// frames, 32 + 32 strips (kernel trace): 313 us with windows of 64 positions of
// which 58 are used (770 vector instructions, mostly addresses, selects and
// conversions at the input), 245 us so.

constexpr int kC2Rows = kStep + 2;   // positions of a buffer line
struct alignas(16) Strip2dRows {     // one wave's inputs of the three layers
    __bf16 x0[kC2Band * kC2Rows * 8];
    __bf16 h1[5 * kC2Rows * 8];
    __bf16 h2[3 * kC2Rows * 16];
};

__device__ __forceinline__ void strip2d_clear(Strip2dRows &R, int lane)
{
    for (int i = lane; i < (int)(sizeof(Strip2dRows) / 16); i += 64)
        reinterpret_cast<uint4 *>(&R)[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Offset of channels c .. c + 3 (c a multiple of 4) of a position of a line of
// h2.  The two 16-byte halves are exchanged in every other group of eight
// positions, so a store's 16 positions meet all banks; a fragment read takes 8
// cycles either way.
__device__ __forceinline__ int strip2d_off16(int pos, int c)
{
    return pos * 16 + ((((c >> 3) ^ (pos >> 3)) & 1) << 3) + (c & 7);
}

// The last two positions of each line of a step become the first two of the
// next; lanes beyond the lines' dwords repeat the last one's.
template <int LINES, int C>
__device__ __forceinline__ int strip2d_at(int lane)
{
    constexpr int kWords = 2 * C / 2;   // dwords of two positions
    const int i = lane < LINES * kWords ? lane : LINES * kWords - 1;
    return i / kWords * (kC2Rows * C) + 2 * (i % kWords);
}
template <int C>
__device__ __forceinline__ uint32_t strip2d_keep(const __bf16 *X, int at)
{
    return *reinterpret_cast<const uint32_t *>(X + at + kStep * C);
}
__device__ __forceinline__ void strip2d_kept(__bf16 *X, uint32_t v, int at)
{
    *reinterpret_cast<uint32_t *>(X + at) = v;
}

__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = {to_bf16(a), to_bf16(b)};
    return __builtin_bit_cast(uint32_t, v);
}

// A position's input rows, seven lines' three bytes in px: colours normalised,
// the coordinates along and across the strip (x and y, or y and x), zeros.
// CLIP: lines may lie outside the frame, or the position outside the strip (in).
template <bool HZ, bool CLIP>
__device__ __forceinline__ void strip2d_encode(__bf16 *row, const uint32_t (&px)[8],
                                               const float (&norm)[6], float along,
                                               const float (&across)[kC2Band], uint32_t line_ok,
                                               uint32_t in)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int j = 0; j < kC2Band; ++j) {
        float c[3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            c[i] = ((float)((px[j] >> (8 * i)) & 0xFFu) - norm[i]) * norm[3 + i];
        u32x4 u = {bf16_pair(c[0], c[1]), bf16_pair(c[2], HZ ? along : across[j]),
                   bf16_pair(HZ ? across[j] : along, 0.0f), 0u};
        if (CLIP) {
            const uint32_t m = line_in(line_ok, j) ? in : 0u;
            u = u32x4{u[0] & m, u[1] & m, u[2] & m, 0u};
        }
        *reinterpret_cast<u32x4 *>(row + j * (kC2Rows * 8)) = u;
    }
}

// Bits of +inf where the step's outputs of a layer exist along the strip, of 0
// elsewhere, for this lane's column of each tile; n = the first output's
// position.
__device__ __forceinline__ void strip2d_tops(uint32_t (&top)[4], int n, int L, int lane)
{
    constexpr uint32_t kInf = 0x7F800000u;
    const bool inside = n >= 0 && n + kStep <= L;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        top[t] = kInf;
    if (!inside) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            top[t] = (uint32_t)(n + 16 * t + (lane & 15)) < (uint32_t)L ? kInf : 0u;
    }
}

// A band's geometry: which lines lie in the frame, and the coordinates, across
// the strip by line, along it as (2 p - last) scale.
struct Band {
    uint32_t line_ok;
    uint32_t line1[3], line2[3], line3;   // masks of the output lines (strip2d_tops)
    float across[kC2Band];
    float scale;
    int last;
    bool horizontal;

    __device__ __forceinline__ Band(bool hz, int line, int W, int H, int lane)
        : horizontal(hz)
    {
        const int lines = hz ? H : W;
        line_ok = band_lines(line, lines);
        // layer 1's by pairs (1, 2), (3, 4), (5, -)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            line1[i] = line_in(line_ok, 2 * i + (lane >> 5) + 1) ? 0x7F800000u : 0u;
            line2[i] = line_in(line_ok, i + 2) ? 0x7F800000u : 0u;
        }
        line3 = line_in(line_ok, 3) ? 0x7F800000u : 0u;
        const float scale_x = coord_scale(W), scale_y = coord_scale(H);
        scale = hz ? scale_x : scale_y;
        last = (hz ? W : H) - 1;
#pragma unroll
        for (int j = 0; j < kC2Band; ++j)
            across[j] = (float)(2 * (line - 3 + j) - (lines - 1)) * (hz ? scale_y : scale_x);
    }

    // A step's input rows from its pixels: p, this lane's position in the frame;
    // x, the step's first position of a strip of L.
    __device__ __forceinline__ void encode(__bf16 *x0, const uint32_t (&px)[8],
                                           const float (&norm)[6], int p, int x, int L,
                                           int lane) const
    {
        const float along = (float)(2 * p - last) * scale;
        const uint32_t in = (uint32_t)(x + lane) < (uint32_t)L ? ~0u : 0u;
        const bool whole = line_ok == 0x7Fu && x >= 0 && x + kStep <= L;
        __bf16 *row = x0 + (lane + 2) * 8;
        if (horizontal && whole)
            strip2d_encode<true, false>(row, px, norm, along, across, line_ok, in);
        else if (horizontal)
            strip2d_encode<true, true>(row, px, norm, along, across, line_ok, in);
        else if (whole)
            strip2d_encode<false, false>(row, px, norm, along, across, line_ok, in);
        else
            strip2d_encode<false, true>(row, px, norm, along, across, line_ok, in);
    }
};

// One output line (or pair of lines) of a 3x3 layer: four position tiles, all
// output-channel tiles.  SEED: the sums start at the bias (learned strips);
// else it is added to them (window logits).
template <bool SEED, int C, int MT, int KS>
__device__ __forceinline__ void strip2d_conv(f32x4 (&acc)[4][MT], const bf16x8 (&w)[MT][KS],
                                             const f32x4 (&bias)[MT], const __bf16 *X,
                                             const int (&xo)[KS])
{
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            acc[t][mt] = SEED ? bias[mt] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        bf16x8 b[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            b[t] = frag_at(X + 16 * t * C + xo[ks]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t][mt] = mma(w[mt][ks], b[t], acc[t][mt]);
    }
    if (!SEED)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[t][mt] += bias[mt];
}

// The network in a wave's registers, for one orientation at a time: A
// fragments, biases, and the lane's offsets in Strip2dRows.
template <bool SEED>
struct Strip2dNet {
    // layer 1's weights are those of output-line pairs: rows 8 .. 15, so lane
    // groups 2 and 3, are the second line's channels
    bf16x8 w1[1][3], w2[1][3], w3[2][5];
    f32x4 b1[1], b2[1], b3[2], w4[2];
    float b4;
    float norm[6];   // the colours' means, then their inverse deviations
    int xo1[3], xo2[3], xo3[5], at0, at1, at2;
    int loaded = -1;   // the orientation whose weights are held

    __device__ __forceinline__ Strip2dNet(const uint8_t *model, int lane)
    {
        const float *fb = reinterpret_cast<const float *>(model + kC2FloatsOff);
        const int col = lane & 15, g = lane >> 4;
        auto four = [&](int at) {
            f32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = fb[at + j];
            return v;
        };
        b1[0] = four(kC2FB[0] + 4 * (g & 1));
        b2[0] = four(kC2FB[1] + 4 * g);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            b3[mt] = four(kC2FB[2] + 16 * mt + 4 * g);
            w4[mt] = four(kC2FW4 + 16 * mt + 4 * g);
        }
        b4 = fb[kC2FB4];
#pragma unroll
        for (int i = 0; i < 6; ++i)
            norm[i] = __uint_as_float(uniform_int(__float_as_uint(fb[kC2FMean + i])));
        // B fragment offsets of the first tile's column: K group k = tap C / 8 +
        // channel half, tap = 3 (line) + position; the groups beyond the taps
        // have zero weights
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            const int k = 4 * ks + g, k2 = k < 9 ? k : 0;
            xo1[ks] = (k / 3 * kC2Rows + k % 3 + col) * 8;
            xo2[ks] = (k2 / 3 * kC2Rows + k2 % 3 + col) * 8;
        }
#pragma unroll
        for (int ks = 0; ks < 5; ++ks) {
            const int k = 4 * ks + g < 18 ? 4 * ks + g : 0;
            xo3[ks] = k / 6 * kC2Rows * 16 + strip2d_off16(k / 2 % 3 + col, 8 * (k & 1));
        }
        at0 = strip2d_at<kC2Band, 8>(lane);
        at1 = strip2d_at<5, 8>(lane);
        at2 = strip2d_at<3, 16>(lane);
    }

    __device__ __forceinline__ void turn_to(bool horizontal, const uint8_t *model, int lane)
    {
        if (loaded == (int)horizontal)
            return;
        const int col = lane & 15, g = lane >> 4;
        const __bf16 *A = reinterpret_cast<const __bf16 *>(model) + (horizontal ? 0 : kC2Orient);
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            w1[0][ks] = frag_at(A + kC2P1 + col * 96 + 32 * ks + 8 * g);
            w2[0][ks] = frag_at(A + kC2A2 + col * 96 + 32 * ks + 8 * g);
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int ks = 0; ks < 5; ++ks)
                w3[mt][ks] = frag_at(A + kC2A3 + (16 * mt + col) * 160 + 32 * ks + 8 * g);
        loaded = (int)horizontal;
    }

    // One step, its input rows in R.x0, x the first one's position of a strip of
    // L: the logit of position x - 3 + lane.
    __device__ __forceinline__ float step(Strip2dRows &R, const Band &band, int x, int L,
                                          int lane) const
    {
        const int col = lane & 15, g = lane >> 4;
        wave_sync();
        uint32_t top[4];
        uint32_t kept = strip2d_keep<8>(R.x0, at0);
        strip2d_tops(top, x - 1, L, lane);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            f32x4 acc[4][1];
            strip2d_conv<SEED, 8>(acc, w1, b1, R.x0 + 2 * i * kC2Rows * 8, xo1);
            if (i < 2 || g < 2)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    *reinterpret_cast<bf16x4 *>(
                        R.h1 + ((2 * i + (g >> 1)) * kC2Rows + 16 * t + col + 2) * 8
                        + 4 * (g & 1)) =
                        relu_bf16(acc[t][0], __uint_as_float(top[t] & band.line1[i]));
        }
        wave_sync();
        strip2d_kept(R.x0, kept, at0);
        kept = strip2d_keep<8>(R.h1, at1);
        strip2d_tops(top, x - 2, L, lane);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            f32x4 acc[4][1];
            strip2d_conv<SEED, 8>(acc, w2, b2, R.h1 + i * kC2Rows * 8, xo2);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                *reinterpret_cast<bf16x4 *>(R.h2 + (i * kC2Rows + 16 * t) * 16
                                            + strip2d_off16(col + 2, 4 * g)) =
                    relu_bf16(acc[t][0], __uint_as_float(top[t] & band.line2[i]));
        }
        wave_sync();
        strip2d_kept(R.h1, kept, at1);
        kept = strip2d_keep<16>(R.h2, at2);
        strip2d_tops(top, x - 3, L, lane);
        float part_z[4];   // lane group's share of each tile's 1x1 layer
        {
            f32x4 acc[4][2];
            strip2d_conv<SEED, 16>(acc, w3, b3, R.h2, xo3);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float z = 0.0f;
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    const u32x2 h = __builtin_bit_cast(
                        u32x2, relu_bf16(acc[t][mt], __uint_as_float(top[t] & band.line3)));
#pragma unroll
                    for (int e = 0; e < 2; ++e) {   // a bfloat16 is a float's upper half
                        z = fmaf(w4[mt][2 * e], __uint_as_float(h[e] << 16), z);
                        z = fmaf(w4[mt][2 * e + 1], __uint_as_float(h[e] & 0xFFFF0000u), z);
                    }
                }
                part_z[t] = z;
            }
        }
        wave_sync();
        strip2d_kept(R.h2, kept, at2);
        return b4 + tile_sums(part_z);
    }
};

template <bool MIXED>
__global__ __launch_bounds__(64 * kStripWaves, 2) void k_cnn2d_strips(Cnn2dStripArgs a)
{
    extern __shared__ __align__(16) uint8_t strip_smem[];
    __shared__ StripMeet meet;
    const int lane = threadIdx.x & 63;
    const int wv = uniform_int(threadIdx.x >> 6);
    if (threadIdx.x <= kStripWaves)
        meet.best[threadIdx.x] = 0;
    __syncthreads();
    Strip2dRows &R = reinterpret_cast<Strip2dRows *>(strip_smem)[wv];
    strip2d_clear(R, lane);
    Strip2dNet<true> net(a.model, lane);
    strip_shares<kC2Halo, MIXED, false>(a, meet, lane, wv, [&](const FrameDev &d, bool horizontal,
                                                        int pos, int half, int p0, int p1) {
        net.turn_to(horizontal, a.model, lane);
        StripWalk k;
        strip_walk<kC2Band>(k, a.frames, d, horizontal, pos);
        const Band band(horizontal, pos, uniform_int(d.W), uniform_int(d.H), lane);
        uint64_t best = 0;
        uint32_t px[8];
        int x = p0 - kC2Halo;   // first new input position of the step
        if (p0 < p1)
            strip_fetch<kC2Band>(px, k, x, lane);
        for (; p0 < p1 && x - kC2Halo < p1; x += kStep) {
            if (k.packed) {   // 21 bytes to a dword of three for each line
#pragma unroll
                for (int j = kC2Band - 1; j >= 0; --j)
                    px[j] = __builtin_amdgcn_alignbyte(px[(3 * j >> 2) + 1], px[3 * j >> 2],
                                                       3 * j & 3);
            }
            band.encode(R.x0, px, net.norm, x + lane, x, k.L, lane);
            if (x + kStep - kC2Halo < p1)
                strip_fetch<kC2Band>(px, k, x + kStep, lane);
            const float z = net.step(R, band, x, k.L, lane);
            const int p = x - kC2Halo + lane;   // column lane % 16 of tile lane / 16
            if (p >= p0 && p < p1) {
                const uint64_t key = strip_key(z, p, half, k.L);
                best = best > key ? best : key;
            }
        }
        return wave_max(best);
    });
}

// Logits of positions 8 .. 119 of rendered windows [n][8][128][3]: a window is a
// strip of two steps from position 5 on (the halo of 3 before the first logit);
// the rows that the first step finds in place of its predecessor's feed only
// positions before.  A wave takes a contiguous share of the windows (those of
// one strip have one orientation), two waves a workgroup; the next step's pixels
// are loaded while a step's layers run.  The sums run as the training kernel's:
// K from zero, then the bias.
//
// Bound by the chain of layers within a step: a wave has few windows.  Measured,
// 3,584 windows (a call): 57 us with the weights loaded and every byte encoded
// alone per window, 28.8 us by workgroups of 32 positions a wave, 22.5 us so.
__global__ __launch_bounds__(kC2WindowBlock, 2) void k_cnn2d_windows(const uint8_t *model,
                                                                     const uint8_t *win,
                                                                     const int32_t *geom,
                                                                     const int32_t *range,
                                                                     float *z_out, int n_windows)
{
    extern __shared__ __align__(16) uint8_t strip_smem[];
    const int lane = threadIdx.x & 63;
    const int wv = uniform_int(threadIdx.x >> 6);
    constexpr int kPerBlock = kC2WindowBlock / 64;
    constexpr int kFirst = kTrainHalo - kC2Halo;   // first input position
    const int64_t wave = (int64_t)blockIdx.x * kPerBlock + wv, waves = gridDim.x * kPerBlock;
    const int w_begin = (int)(wave * n_windows / waves);
    const int w_end = (int)((wave + 1) * n_windows / waves);
    Strip2dRows &R = reinterpret_cast<Strip2dRows *>(strip_smem)[wv];
    strip2d_clear(R, lane);
    uint32_t px[8];
    auto fetch = [&](int wi, int x) {
        StripWalk k;
        k.frame = win + (int64_t)wi * (8 * kC2Win * 3);
        k.along = 3;
        k.across = 3 * kC2Win;
        k.first = 0;
        k.L = kC2Win;
        k.lines = 8;
        k.packed = k.last_row = false;   // an eighth line follows the band's seven
        strip_fetch<kC2Band>(px, k, x, lane);
    };
    if (w_begin < w_end)
        fetch(w_begin, kFirst);
    Strip2dNet<false> net(model, lane);
    for (int wi = w_begin; wi < w_end; ++wi) {
        const int32_t *geo = geom + 8 * wi;
        const bool hz = uniform_int(geo[0]) != 0;
        const int line = uniform_int(geo[1]), start = uniform_int(geo[2]);
        const Band band(hz, line, uniform_int(geo[3]), uniform_int(geo[4]), lane);
        const int lo = uniform_int(min(max(range[2 * wi], 0), kC2Win));
        const int L = max(uniform_int(min(range[2 * wi + 1], kC2Win)) - lo, 0);
        net.turn_to(hz, model, lane);
#pragma unroll 1
        for (int x = kFirst; x < kC2Win; x += kStep) {
            wave_sync();
            band.encode(R.x0, px, net.norm, start + x + lane, x - lo, L, lane);
            if (x == kFirst)
                fetch(wi, x + kStep);
            else if (wi + 1 < w_end)
                fetch(wi + 1, kFirst);
            const float z = net.step(R, band, x - lo, L, lane);
            const int n = x - kC2Halo + lane;
            if (n >= kTrainHalo && n < kC2Win - kTrainHalo)
                z_out[(int64_t)wi * kTrainOut + n - kTrainHalo] = z;
        }
    }
}

// Element offset of channels c .. c + 3 (c a multiple of 4) of position row
// `pos` in a 16- or 32-channel buffer line.  With 32 channels the chunk pairs
// of a row are exchanged in every other group of four rows, so that the 16
// rows of each group of lanes that an LDS read serves together start in
// distinct bank groups (lanes 0-3, 12-15 and 20-27; 4-11, 16-19 and 28-31; the
// same of the upper half, measured; chunks permuted four ways met two-way
// conflicts: 273.3 us a training step of 14,336 windows, 271.2 us so); 8- and
// 16-channel rows need nothing at this line pitch (2 rows beyond a multiple of 16: the last tap of
// a line and the first of the next share their banks' order).
static_assert(kPos % 16 == 2 && (kC2Win / 2 + 2) % 16 == 2, "line pitch");
__device__ __forceinline__ int off16(int pos, int c) { return pos * 16 + c; }
__device__ __forceinline__ int off32(int pos, int c)
{
    return pos * 32 + (((c >> 3) ^ ((pos >> 1) & 2)) << 3) + (c & 7);
}

constexpr int kL8 = kPos * 8, kL16 = kPos * 16;   // elements of a buffer line

// f(k) of this lane's K group k = 4 ks + g (small numbers): a byte of a
// constant, one bit-field extract.
template <class F>
__device__ __forceinline__ int by_group(int ks, int g, F f)
{
    uint32_t packed = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        packed |= (uint32_t)f(4 * ks + i) << (8 * i);
    return (int)((packed >> (8 * g)) & 0xFFu);
}

// The input of a rendered window for a workgroup: pixels p, p + 32, p + 64, p +
// 96 (p = tid % 32) of band line tid / 32, fetched a window ahead (the fourth
// byte of a word is the next pixel's or, the window having eight lines, the
// next line's), encoded, and stored to [line][position][8 channels].
struct WindowInput {
    uint32_t raw[4];
    bf16x8 enc[4];
    int last_w = 0, last_h = 0;
    float rw = 0.0f, rh = 0.0f;

    static __device__ __forceinline__ bool loads(int tid) { return tid < kC2Band * 32; }

    __device__ __forceinline__ void fetch(const uint8_t *win, int wi, int tid)
    {
        if (!loads(tid))
            return;
        const uint8_t *src =
            win + (int64_t)wi * (8 * kC2Win * 3) + (tid >> 5) * (kC2Win * 3) + (tid & 31) * 3;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            __builtin_memcpy(&raw[k], src + 96 * k, 4);
    }

    // geo: the window's geometry, range: its strip range; fb: the model's
    // float block.  Positions outside the frame or the strip are zero.
    __device__ __forceinline__ void encode(const int32_t *geo, const int32_t *range,
                                           const float *fb, int tid)
    {
        const bool hz = uniform_int(geo[0]) != 0;
        const int line = uniform_int(geo[1]), start = uniform_int(geo[2]);
        const int W = uniform_int(geo[3]), H = uniform_int(geo[4]);
        const int lo = uniform_int(range[0]), hi = uniform_int(range[1]);
        if (W != last_w || H != last_h) {
            rw = coord_scale(W);
            rh = coord_scale(H);
            last_w = W;
            last_h = H;
        }
        const int t = fresh(tid);
        const int across = line - 3 + (t >> 5), n0 = t & 31;
        const bool in_line = across >= 0 && across < (hz ? H : W);
        const int x2 = 2 * (hz ? start + n0 : across) - (W - 1);
        const int y2 = 2 * (hz ? across : start + n0) - (H - 1);
        const int dx = hz ? 64 : 0, dy = 64 - dx;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int n = n0 + 32 * k;
            bf16x8 v;
#pragma unroll
            for (int c = 0; c < 3; ++c)
                v[c] = to_bf16(((float)((raw[k] >> (8 * c)) & 0xFFu) - fb[kC2FMean + c])
                               * fb[kC2FInv + c]);
            v[3] = to_bf16((float)(x2 + k * dx) * rw);
            v[4] = to_bf16((float)(y2 + k * dy) * rh);
            v[5] = v[6] = v[7] = to_bf16(0.0f);
            enc[k] = in_line && n >= lo && n < hi ? v : bf16x8{};
        }
    }

    __device__ __forceinline__ void store(__bf16 *x0, int tid) const
    {
        if (!loads(tid))
            return;
        const int t = fresh(tid);
        __bf16 *dst = x0 + (t >> 5) * kL8 + ((t & 31) + 1) * 8;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<bf16x8 *>(dst + 32 * 8 * k) = enc[k];
    }
};

// ------------------------------------------------------------- training --
//
// Per window: the forward pass; dz = scale w (sigmoid(z) - t) on the
// central positions inside the strip; the signals at the pre-activations
// dP3 = [h3 > 0] w4 dz, dP2 = [h2 > 0] (flipped-W3 convolution of dP3),
// dP1 = [h1 > 0] (flipped-W2 convolution of dP2), each stored in bfloat16;
// then the weight gradients as GEMMs whose K runs over the positions,
//   dW[o][tap][c] = sum_n dP[n][o] X[n + tap][c].
// All of it is MFMA work.  The four waves of a workgroup take 32 positions of
// the window each: two 16-position tiles of every forward-shaped GEMM and one
// K step of every weight-gradient tile, whose accumulators (28 tiles, 112
// registers) a wave keeps across its windows and the workgroup adds up at the
// end.  The weight gradients' operands are columns of position-major buffers:
// ds_read_b64_tr_b16 delivers them transposed, so a tap is a row offset and
// needs no second layout (4 rows x 16 channels a read; K index 8 g + e of a
// fragment is position 4 g + e for e < 4, 16 + 4 g + e - 4 otherwise, in both
// operands).  Taps are numbered as in the frame, so vertical strips swap a
// tap's two offsets and every window adds to the same accumulators.
//
// Bound by LDS bandwidth: about 131 fragment reads of 1 KB a wave and window
// (4,100 cycles a compute unit at 128 bytes a cycle) beside 2,400 cycles of
// MFMA a SIMD; 80 KB of LDS and 256 registers let two workgroups share a
// compute unit.  Measured, 14,336
// windows: 3137 us with the weight gradients as 4 x 4 outer products on the
// vector units (723 work units a workgroup), 295 us so (kernel trace); of a
// SIMD's cycles
// about half issue vector instructions and a fifth MFMAs.

constexpr int kDW3 = 0;                        // [32][9 taps x 16]
constexpr int kDW2 = kDW3 + 32 * 144;          // [16][9 x 8, bias, 7 spare]
constexpr int kDW1 = kDW2 + 16 * 80;           // [8][9 x 8, bias, 7 spare]
constexpr int kDB3 = kDW1 + 8 * 80;            // [32]
constexpr int kDW4 = kDB3 + 32;                // [32]
constexpr int kDB4 = kDW4 + 32;
constexpr int kDLoss = kDB4 + 1;
static_assert(kDLoss < kC2GradStride && kC2GradStride % kReduceCols == 0, "gradient layout");

struct alignas(16) GradLds {
    __bf16 w3[10 * 512];          // layer 3's A fragments, [mt 5 + ks][lane][8]
    __bf16 f3[9 * 512];           // the flipped layer 3's, [3 da + dl][lane][8]
    __bf16 x0[kC2Band * kPos * 8];
    __bf16 h1[5 * kPos * 8];
    __bf16 h2[3 * kPos * 16];
    __bf16 d[5 * kPos * 8];       // dP3 [kPos][32], later dP1 [5][kPos][8]
    __bf16 dp2[3 * kPos * 16];
    __bf16 ones[8];
    float fb[kC2Floats];
};
static_assert(kPos * 32 <= 5 * kPos * 8, "dP3 fits where dP1 is kept");
static_assert(sizeof(GradLds) <= 81920, "two workgroups per compute unit");
static_assert((2 * kDB3 + 4 * 66) * sizeof(float) <= sizeof(GradLds), "sums fit the LDS");

__global__ __launch_bounds__(kBlock, 2) void k_cnn2d_grad(Cnn2dTrainArgs a)
{
    extern __shared__ __align__(16) uint8_t c2_smem[];
    GradLds &G = *reinterpret_cast<GradLds *>(c2_smem);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    {
        uint4 *z = reinterpret_cast<uint4 *>(&G);
        for (int i = tid; i < (int)(sizeof(GradLds) / 16); i += kBlock)
            z[i] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        const float *src = reinterpret_cast<const float *>(a.model + kC2FloatsOff);
        for (int i = tid; i < kC2Floats; i += kBlock)
            G.fb[i] = src[i];
        if (tid < 8)
            G.ones[tid] = to_bf16(1.0f);
        __syncthreads();
    }
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 acc3[2][9], accb3[2], acc2[5], acc1[5];
    accb3[0] = accb3[1] = zero4;
#pragma unroll
    for (int t = 0; t < 9; ++t)
        acc3[0][t] = acc3[1][t] = zero4;
#pragma unroll
    for (int t = 0; t < 5; ++t)
        acc2[t] = acc1[t] = zero4;
    float pw4[2][4], pb4 = 0.0f, loss = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        pw4[0][j] = pw4[1][j] = 0.0f;

    // a contiguous share of the windows: those of one strip have one
    // orientation, so its weights are loaded about once a strip
    const int w_begin = (int)((int64_t)blockIdx.x * a.n / gridDim.x);
    const int w_end = (int)((int64_t)(blockIdx.x + 1) * a.n / gridDim.x);
    int cur = -1;
    // the next window's input, fetched a window ahead and encoded while dW1 runs
    WindowInput in;
    if (w_begin < w_end) {
        in.fetch(a.win, w_begin, tid);
        in.encode(a.geom + 8 * w_begin, a.range + 2 * w_begin, G.fb, tid);
    }
    for (int wi = w_begin; wi < w_end; ++wi) {
        const int32_t *geo = a.geom + 8 * wi;
        const bool hz = uniform_int(geo[0]) != 0;
        const int line = uniform_int(geo[1]);
        const int lo = uniform_int(a.range[2 * wi]), hi = uniform_int(a.range[2 * wi + 1]);
        const uint32_t line_ok = band_lines(line, uniform_int(hz ? geo[4] : geo[3]));
        const __bf16 *A = reinterpret_cast<const __bf16 *>(a.model) + (hz ? 0 : kC2Orient);
        if (cur != (int)hz) {
            cur = (int)hz;
            const int col = lane & 15, g = lane >> 4;
            for (int f = wv; f < 19; f += kWaves) {
                const __bf16 *src = f < 10 ? A + kC2A3 + ((f / 5) * 16 + col) * 160 + 32 * (f % 5)
                                           : A + kC2F3 + col * 288 + 32 * (f - 10);
                *reinterpret_cast<bf16x8 *>(G.w3 + f * 512 + lane * 8) = frag_at(src + 8 * g);
            }
        }
        in.store(G.x0, tid);
        __syncthreads();
        if (wi + 1 < w_end)
            in.fetch(a.win, wi + 1, tid);
        // targets and loss weights of this lane's two positions; where a position
        // carries no loss neither counts, nor does its logit (zero times a value
        // that is not finite is not zero)
        float tgt[2], lw[2], tops[2];
        bool carries[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int n = 32 * wv + (lane & 15) + 16 * t;
            const bool here = n >= lo && n < hi;
            const bool has = here && n >= kTrainHalo && n < kC2Win - kTrainHalo;
            carries[t] = has;
            tops[t] = here ? __builtin_inff() : 0.0f;
            const int64_t k = (int64_t)wi * kTrainOut + (has ? n - kTrainHalo : 0);
            const float target = a.target[k];
            tgt[t] = has ? target : 0.0f;
            lw[t] = has ? a.scale * a.weight[k] : 0.0f;
        }
        {
            // layer 1 by output-line pairs: lane groups 0-1 hold the first line
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const Frag<96, 1> w1 = load_frag<96, 1>(A + kC2P1);
            const f32x4 b1 = *reinterpret_cast<const f32x4 *>(G.fb + kC2FB[0] + 4 * (L.g & 1));
            int o[3];   // K group k: line k / 3 of four, dl = k % 3
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                o[ks] = by_group(ks, L.g, [](int k) { return k / 3; }) * kL8
                        + (p0 + by_group(ks, L.g, [](int k) { return k % 3; })) * 8;
            }
            // the last pair's fourth input line does not exist; its weights
            // are zero for the pair's first line and the second is dropped:
            // any finite line
            const int o_last = o[2] - (8 + L.g >= 9 ? kL8 : 0);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                f32x4 acc[2];
                acc[0] = acc[1] = zero4;
#pragma unroll
                for (int ks = 0; ks < 3; ++ks) {
                    const __bf16 *x = G.x0 + 2 * i * kL8 + (i == 2 && ks == 2 ? o_last : o[ks]);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t] = mma(w1.a[0][ks], frag_at(x + t * 128), acc[t]);
                }
                const int ln = 2 * i + (L.g >> 1);
                if (ln < 5)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        *reinterpret_cast<bf16x4 *>(G.h1 + ln * kL8 + (p0 + 16 * t + 1) * 8
                                                    + 4 * (L.g & 1)) =
                            relu_bf16(acc[t] + b1, line_in(line_ok, ln + 1) ? tops[t] : 0.0f);
            }
        }
        const Frag<96, 1> w2 = load_frag<96, 1>(A + kC2A2);
        __syncthreads();
        {
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const f32x4 b2 = *reinterpret_cast<const f32x4 *>(G.fb + kC2FB[1] + 4 * L.g);
            int o[3];   // K group k (of 9): da = k / 3, dl = k % 3
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                // (groups 9 .. 11 have zero weights: any finite values)
                o[ks] = by_group(ks, L.g, [](int k) { return k < 9 ? k / 3 : 0; }) * kL8
                        + (p0 + by_group(ks, L.g, [](int k) { return k % 3; })) * 8;
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                f32x4 acc[2];
                acc[0] = acc[1] = zero4;
#pragma unroll
                for (int ks = 0; ks < 3; ++ks)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t] = mma(w2.a[0][ks], frag_at(G.h1 + i * kL8 + o[ks] + t * 128),
                                     acc[t]);
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    *reinterpret_cast<bf16x4 *>(G.h2 + i * kL16
                                                + off16(p0 + 16 * t + 1, 4 * L.g)) =
                        relu_bf16(acc[t] + b2, line_in(line_ok, i + 2) ? tops[t] : 0.0f);
            }
        }
        __syncthreads();
        {
            // layer 3, the 1x1 layer, the loss and dP3: a position's 32
            // channels sit in the four lane groups of its column
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const int frag = (L.g * 16 + L.col) * 8;
            f32x4 acc[2][2];
            acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) {
                // K group k (of 18; two more have zero weights): tap k / 2,
                // half k % 2
                const __bf16 *x =
                    G.h2 + by_group(ks, L.g, [](int k) { return k < 18 ? k / 6 : 0; }) * kL16
                    + off16(p0 + by_group(ks, L.g, [](int k) { return k / 2 % 3; }),
                            8 * (L.g & 1));
                const bf16x8 x0 = frag_at(x), x1 = frag_at(x + 256);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const bf16x8 w = frag_at(G.w3 + (mt * 5 + ks) * 512 + frag);
                    acc[mt][0] = mma(w, x0, acc[mt][0]);
                    acc[mt][1] = mma(w, x1, acc[mt][1]);
                }
            }
            f32x4 w4[2];
            w4[0] = *reinterpret_cast<const f32x4 *>(G.fb + kC2FW4 + 4 * L.g);
            w4[1] = *reinterpret_cast<const f32x4 *>(G.fb + kC2FW4 + 16 + 4 * L.g);
            bf16x4 h[2][2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    h[t][mt] = relu_bf16(
                        acc[mt][t]
                            + *reinterpret_cast<const f32x4 *>(G.fb + kC2FB[2] + 16 * mt + 4 * L.g),
                        line_in(line_ok, 3) ? tops[t] : 0.0f);
            const int own = L.g & 1;   // this lane's tile from here
            const float z = ordered_dot(G.fb + kC2FW4, h, G.fb[kC2FB4]);
            const float lw_own = own ? lw[1] : lw[0], tgt_own = own ? tgt[1] : tgt[0];
            const bool carries_own = own ? carries[1] : carries[0];
            float dz[2];
            to_all_groups(carries_own ? lw_own * (sigmoid(z) - tgt_own) : 0.0f, dz);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                pb4 += dz[t];    // every lane group alike; the first one's is taken
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    f32x4 dp;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        pw4[mt][j] = fmaf((float)h[t][mt][j], dz[t], pw4[mt][j]);
                        dp[j] = w4[mt][j] * dz[t];
                    }
                    *reinterpret_cast<bf16x4 *>(G.d + off32(p0 + 16 * t + 1, 16 * mt + 4 * L.g)) =
                        relu_mask(dp, h[t][mt]);
                }
            }
            if (L.g < 2 && carries_own)   // -(t log s + (1 - t) log(1 - s)) = max(z, 0) - z t + log(1 + e^-|z|)
                loss += lw_own * (fmaxf(z, 0.0f) - z * tgt_own + log1pf(__expf(-fabsf(z))));
            if (tid < 8)   // guard positions of dP3
                *reinterpret_cast<bf16x8 *>(G.d + (tid >> 2) * (kPos - 1) * 32 + (tid & 3) * 8) =
                    bf16x8{};
        }
        __syncthreads();
        {
            // dP2: output line i takes tap line 2 - i of the one dP3 line
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const int frag = (L.g * 16 + L.col) * 8;
            bf16x8 x[2][3];
#pragma unroll
            for (int dl = 0; dl < 3; ++dl) {
                const __bf16 *d = G.d + off32(p0 + dl, 8 * L.g);
                x[0][dl] = frag_at(d);
                x[1][dl] = frag_at(d + 512);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                f32x4 acc[2];
                acc[0] = acc[1] = zero4;
#pragma unroll
                for (int dl = 0; dl < 3; ++dl) {
                    const bf16x8 w = frag_at(G.f3 + ((2 - i) * 3 + dl) * 512 + frag);
                    acc[0] = mma(w, x[0][dl], acc[0]);
                    acc[1] = mma(w, x[1][dl], acc[1]);
                }
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int o = i * kL16 + off16(p0 + 16 * t + 1, 4 * L.g);
                    *reinterpret_cast<bf16x4 *>(G.dp2 + o) =
                        relu_mask(acc[t], *reinterpret_cast<const bf16x4 *>(G.h2 + o));
                }
            }
        }
        {
            // dW3
            const Place L(fresh(lane));
            const int r0 = 32 * wv + L.r;
            bf16x8 p[2];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const __bf16 *d = G.d + off32(r0 + 1, 16 * mt + 4 * L.q);
                p[mt] = transposed(d, d + 512);
                const __bf16 one = to_bf16(1.0f);
                accb3[mt] = mma(p[mt], bf16x8{one, one, one, one, one, one, one, one}, accb3[mt]);
            }
            int o[3];
#pragma unroll
            for (int dl = 0; dl < 3; ++dl)
                o[dl] = off16(r0 + dl, 4 * L.q);
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const int dy = tap / 3, dx = tap % 3;
                const __bf16 *x = G.h2 + (hz ? dy * kL16 + o[dx] : dx * kL16 + o[dy]);
                const bf16x8 xt = transposed(x, x + 256);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    acc3[mt][tap] = mma(p[mt], xt, acc3[mt][tap]);
            }
        }
        const Frag<192, 1> f2 = load_frag<192, 1>(A + kC2F2);
        __syncthreads();
        {
            // dP1 by output-line pairs (i0, i0 + 1) from dP2 lines i0 - 2 ..
            // i0 + 1 (K steps of lines that do not exist are left out, or
            // read as zeros where half a step exists)
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            int od[6];   // K group k: input line k / 6 of four, dl, half
#pragma unroll
            for (int ks = 0; ks < 6; ++ks) {
                od[ks] = by_group(ks, L.g, [](int k) { return k / 6; }) * kL16
                         + off16(p0 + by_group(ks, L.g, [](int k) { return k % 6 / 2; }),
                                 8 * (L.g & 1));
            }
#pragma unroll
            for (int i0 = 0; i0 < 6; i0 += 2) {
                f32x4 acc[2];
                acc[0] = acc[1] = zero4;
#pragma unroll
                for (int ks = (i0 == 0 ? 3 : 0); ks < (i0 == 0 ? 6 : i0 == 2 ? 5 : 2); ++ks) {
                    const int last = (4 * ks + 3) / 6 + i0 - 2;   // the step's last input line
                    const bool off = last > 2 && L.g >= 6 * (5 - i0) - 4 * ks;   // line > 2
                    const int o = od[ks] + (i0 - 2) * kL16 - (off ? kL16 : 0);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        bf16x8 x = frag_at(G.dp2 + o + t * 256);
                        if (last > 2 && off)
                            x = bf16x8{};
                        acc[t] = mma(f2.a[0][ks], x, acc[t]);
                    }
                }
                const int ln = i0 + (L.g >> 1);
                if (ln < 5)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int o = ln * kL8 + (p0 + 16 * t + 1) * 8 + 4 * (L.g & 1);
                        *reinterpret_cast<bf16x4 *>(G.d + o) =
                            relu_mask(acc[t], *reinterpret_cast<const bf16x4 *>(G.h1 + o));
                    }
            }
        }
        // dW2 and dW1: a tile's 16 columns are two taps of 8 channels (chunks
        // q < 2 and q >= 2 of the lane's reads); the tenth tap reads ones, its
        // columns are the bias gradients
        const int sy = hz ? kL8 : 8, sx = hz ? 8 : kL8;
        auto tap_offset = [&](const Place &L, int r0, int t) {
            const int e = 2 * t, o = 2 * t + 1;
            return r0 * 8 + 4 * (L.q & 1)
                   + (L.q >= 2 ? (o / 3) * sy + (o % 3) * sx : (e / 3) * sy + (e % 3) * sx);
        };
        {
            const Place L(fresh(lane));
            const int r0 = 32 * wv + L.r;
            const int o = off16(r0 + 1, 4 * L.q);
            bf16x8 p[3];
#pragma unroll
            for (int r = 0; r < 3; ++r)
                p[r] = transposed(G.dp2 + r * kL16 + o, G.dp2 + r * kL16 + o + 256);
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                const bool ones = t == 4 && L.q >= 2;
                const __bf16 *x = ones ? G.ones : G.h1 + tap_offset(L, r0, t);
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const __bf16 *xr = ones ? x : x + r * kL8;
                    acc2[t] = mma(p[r], transposed(xr, ones ? x : xr + 128), acc2[t]);
                }
            }
        }
        __syncthreads();
        {
            // rows 8 .. 15 of dW1's tiles repeat rows 0 .. 7
            const Place L(fresh(lane));
            const int r0 = 32 * wv + L.r;
            const int o = (r0 + 1) * 8 + 4 * (L.q & 1);
            bf16x8 p[5];
#pragma unroll
            for (int r = 0; r < 5; ++r)
                p[r] = transposed(G.d + r * kL8 + o, G.d + r * kL8 + o + 128);
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                const bool ones = t == 4 && L.q >= 2;
                const __bf16 *x = ones ? G.ones : G.x0 + tap_offset(L, r0, t);
#pragma unroll
                for (int r = 0; r < 5; ++r) {
                    const __bf16 *xr = ones ? x : x + r * kL8;
                    acc1[t] = mma(p[r], transposed(xr, ones ? x : xr + 128), acc1[t]);
                }
            }
        }
        if (wi + 1 < w_end)
            in.encode(a.geom + 8 * (wi + 1), a.range + 2 * (wi + 1), G.fb, tid);
        __syncthreads();
    }

    // the workgroup's sums, in a fixed order: (wave 0 + wave 2) + (wave 1 +
    // wave 3)
    float *sum = reinterpret_cast<float *>(&G);
    float *tail = sum + 2 * kDB3;    // [4 waves][66]: b3, w4, b4, loss
    const int col = lane & 15, g = lane >> 4;
    auto each = [&](auto fn) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int o = 4 * g + j;
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    fn(kDW3 + (16 * mt + o) * 144 + tap * 16 + col, acc3[mt][tap][j]);
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                fn(kDW2 + o * 80 + t * 16 + col, acc2[t][j]);
                if (g < 2)
                    fn(kDW1 + o * 80 + t * 16 + col, acc1[t][j]);
            }
        }
    };
    auto over_columns = [](float v) {
#pragma unroll
        for (int d = 1; d < 16; d *= 2)
            v += __shfl_xor(v, d, 64);
        return v;
    };
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const float vw = over_columns(pw4[mt][j]);
            if (col == 0) {
                tail[66 * wv + 16 * mt + 4 * g + j] = accb3[mt][j];
                tail[66 * wv + 32 + 16 * mt + 4 * g + j] = vw;
            }
        }
    pb4 = over_columns(pb4);
    loss = over_columns(loss);
    loss += __shfl_xor(loss, 16, 64);   // lane groups 0 and 1
    if (lane == 0) {
        tail[66 * wv + 64] = pb4;
        tail[66 * wv + 65] = loss;
    }
    if (wv >= 2)
        each([&](int i, float v) { sum[(wv - 2) * kDB3 + i] = v; });
    __syncthreads();
    if (wv < 2)
        each([&](int i, float v) { sum[wv * kDB3 + i] += v; });
    __syncthreads();
    float *out = a.partial + (int64_t)blockIdx.x * kC2GradStride;
    for (int i = tid; i < kDB3; i += kBlock)
        out[i] = sum[i] + sum[kDB3 + i];
    if (tid < 66)
        out[kDB3 + tid] = (tail[tid] + tail[132 + tid]) + (tail[66 + tid] + tail[198 + tid]);
}

// Gradient in model-file order from the workgroups' sums; the normaliser
// gets zero.
__global__ __launch_bounds__(kReduceThreads) void k_cnn2d_reduce(const float *partial, int grid,
                                                                 float *grad, float *loss)
{
    __shared__ float s_sum[kReduceCols];
    column_sums(partial, grid, kC2GradStride, s_sum);
    if (threadIdx.x >= kReduceCols)
        return;
    const int i = blockIdx.x * kReduceCols + threadIdx.x;
    const float v = s_sum[threadIdx.x];
    if (i < kC2FileW[0])
        grad[i] = 0.0f;
    if (i < kDW2) {
        const int o = i / 144, k = i % 144;
        grad[kC2FileW[2] + (o * 16 + k % 16) * 9 + k / 16] = v;
    } else if (i < kDB3) {
        const int l = i < kDW1 ? 1 : 0;
        const int cin = l ? 8 : 5;
        const int r = i - (l ? kDW2 : kDW1);
        const int o = r / 80, k = r % 80;
        if (k < 72 && k % 8 < cin)
            grad[kC2FileW[l] + (o * cin + k % 8) * 9 + k / 8] = v;
        else if (k == 72)
            grad[kC2FileB[l] + o] = v;
    } else if (i < kDW4) {
        grad[kC2FileB[2] + i - kDB3] = v;
    } else if (i <= kDB4) {
        grad[kC2FileW4 + i - kDW4] = v;   // w4, then b4
    } else if (i == kDLoss) {
        *loss = v;
    }
}

// SGD with momentum on the master weights (file order), each weight's copies in
// the device model block with it (k_cnn2d_pack's layout; the padding stays): a
// repack of its own cost a launch, 1.6 us of a step.
__global__ __launch_bounds__(kBlock) void k_cnn2d_update(float *master, float *mom,
                                                         const float *grad, float lr, float mu,
                                                         uint8_t *model)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= kC2Params)
        return;
    const float m = mu * mom[i] + grad[i];
    mom[i] = m;
    const float v = master[i] - lr * m;
    master[i] = v;
    const __bf16 h = to_bf16(v);
    float *fb = reinterpret_cast<float *>(model + kC2FloatsOff);
    constexpr int cin[3] = {5, 8, 16}, cout[3] = {8, 16, 32};
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const int r = i - kC2FileW[l];
        if (r >= 0 && r < cout[l] * cin[l] * 9) {
            const int dx = r % 3, dy = r / 3 % 3, c = r / 9 % cin[l], o = r / 9 / cin[l];
#pragma unroll
            for (int orient = 0; orient < 2; ++orient) {
                __bf16 *w = reinterpret_cast<__bf16 *>(model) + orient * kC2Orient;
                const int da = orient == 0 ? dy : dx, dl = orient == 0 ? dx : dy;
                if (l > 0)
                    w[(l == 1 ? kC2A2 : kC2A3) + o * (l == 1 ? 96 : 160) + (3 * da + dl) * cin[l]
                      + c] = h;
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {   // the lines of a pair
                    if (l == 0)
                        w[kC2P1 + (8 * sl + o) * 96 + (3 * (da + sl) + dl) * 8 + c] = h;
                    if (l == 1)
                        w[kC2F2 + (8 * sl + c) * 192 + (3 * (2 - da + sl) + 2 - dl) * 16 + o] = h;
                }
                if (l == 2)
                    w[kC2F3 + c * 288 + (3 * (2 - da) + 2 - dl) * 32 + o] = h;
            }
        }
        if (i >= kC2FileB[l] && i < kC2FileB[l] + cout[l])
            fb[kC2FB[l] + i - kC2FileB[l]] = v;
    }
    if (i >= kC2FileW4 && i < kC2FileW4 + 32)
        fb[kC2FW4 + i - kC2FileW4] = (float)h;
    if (i == kC2FileB4)
        fb[kC2FB4] = v;
    if (i < 6)   // the colours' means and inverse deviations
        fb[kC2FMean + i] = v;
}

// Device model block from the float32 master weights (file order); every
// slot, padding included, is written.
__global__ __launch_bounds__(kBlock) void k_cnn2d_pack(const float *master, uint8_t *model)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    constexpr int cin[3] = {5, 8, 16};
    if (i < 2 * kC2Orient) {
        const int orient = i / kC2Orient, e = i - kC2Orient * (i / kC2Orient);
        float v = 0.0f;
        int l, o, c, da, dl;
        bool real = false;
        if (e >= kC2P1) {
            // layer 1 for two output lines at once: row m = 8 s + o is output
            // channel o of the pair's line s; K = (3 lo + dl) 8 + c over the
            // pair's four input lines lo = 0 .. 3 (tap da = lo - s)
            const int r = e - kC2P1;
            const int m = r / 96, k = r % 96;
            const int g = k / 8, sl = m / 8;
            l = 0;
            o = m % 8;
            c = k % 8;
            da = g / 3 - sl;
            dl = g % 3;
            real = c < cin[0] && da >= 0 && da < 3;
        } else if (e < kC2F2) {
            l = e < kC2A3 ? 1 : 2;
            const int r = e - (l == 1 ? kC2A2 : kC2A3), kp = l == 1 ? 96 : 160;
            const int k = r % kp, tap = k / cin[l];
            o = r / kp;
            c = k % cin[l];
            da = tap / 3;
            dl = tap % 3;
            real = tap < 9;
        } else if (e < kC2F3) {
            // flipped layer 2 for two output lines at once: row m = 8 s + c is
            // input channel c at the pair's line s; K = (3 lo + dl') 16 + o
            // over four dP2 lines lo (tap da' = lo - s)
            const int r = e - kC2F2;
            const int m = r / 192, k = r % 192;
            l = 1;
            c = m % 8;
            o = k % 16;
            const int tap = k / 16;
            da = 2 - (tap / 3 - m / 8);
            dl = 2 - tap % 3;
            real = da >= 0 && da < 3;
        } else {
            const int r = e - kC2F3;
            const int m = r / 288, k = r % 288;
            const int tap = k / 32;
            l = 2;
            c = m;
            o = k % 32;
            da = 2 - tap / 3;
            dl = 2 - tap % 3;
            real = true;
        }
        if (real) {
            const int dy = orient == 0 ? da : dl, dx = orient == 0 ? dl : da;
            v = master[kC2FileW[l] + ((o * cin[l] + c) * 3 + dy) * 3 + dx];
        }
        reinterpret_cast<__bf16 *>(model)[i] = to_bf16(v);
        return;
    }
    const int f = i - 2 * kC2Orient;
    if (f >= 96)
        return;
    float *fb = reinterpret_cast<float *>(model + kC2FloatsOff);
    float v = 0.0f;
    if (f < 8)
        v = master[kC2FileB[0] + f];
    else if (f < 24)
        v = master[kC2FileB[1] + f - 8];
    else if (f < 56)
        v = master[kC2FileB[2] + f - 24];
    else if (f < 88)
        v = (float)to_bf16(master[kC2FileW4 + f - 56]);
    else if (f == 88)
        v = master[kC2FileB4];
    else if (f < 95)
        v = master[f - 89];     // mean[3], inv_std[3]
    fb[f] = v;
}

}  // namespace

hipError_t launch_cnn2d_strips(const Cnn2dStripArgs &a, hipStream_t s, hipEvent_t start,
                               hipEvent_t stop)
{
    if (a.n_items <= 0)
        return hipSuccess;
    launch_maybe_timed(a.mixed ? k_cnn2d_strips<true> : k_cnn2d_strips<false>,
                       dim3(kXcds * a.deal.groups), dim3(64 * kStripWaves),
                       kStripWaves * sizeof(Strip2dRows), s, start, stop, a);
    return hipGetLastError();
}

hipError_t launch_cnn2d_windows(const uint8_t *model, const uint8_t *win, const int32_t *geom,
                                const int32_t *range, float *z, int n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    // four resident workgroups on each of 256 compute units
    constexpr int kPerBlock = kC2WindowBlock / 64;
    const int want = (n + kPerBlock - 1) / kPerBlock, grid = want < 1024 ? want : 1024;
    hipLaunchKernelGGL(k_cnn2d_windows, dim3(grid), dim3(kC2WindowBlock),
                       kPerBlock * sizeof(Strip2dRows), s, model, win, geom, range, z, n);
    return hipGetLastError();
}

int cnn2d_grad_blocks_per_cu()
{
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_cnn2d_grad, kBlock, sizeof(GradLds))
            != hipSuccess
        || b < 1) {
        (void)hipGetLastError();
        b = 1;
    }
    return b;
}

hipError_t launch_cnn2d_grad(const Cnn2dTrainArgs &a, int grid, hipStream_t s)
{
    if (grid <= 0)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_cnn2d_grad, dim3(grid), dim3(kBlock), sizeof(GradLds), s, a);
    return hipGetLastError();
}

hipError_t launch_cnn2d_reduce(const float *partial, int grid, float *grad_out, float *loss_out,
                               hipStream_t s)
{
    hipLaunchKernelGGL(k_cnn2d_reduce, dim3(kC2GradStride / kReduceCols), dim3(kReduceThreads), 0,
                       s, partial, grid, grad_out, loss_out);
    return hipGetLastError();
}

hipError_t launch_cnn2d_update(float *master, float *momentum, const float *grad, float lr,
                               float mom, uint8_t *model, hipStream_t s)
{
    hipLaunchKernelGGL(k_cnn2d_update, dim3((kC2Params + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                       master, momentum, grad, lr, mom, model);
    return hipGetLastError();
}

hipError_t launch_cnn2d_pack(const float *master, uint8_t *model, hipStream_t s)
{
    constexpr int slots = 2 * kC2Orient + 96;
    hipLaunchKernelGGL(k_cnn2d_pack, dim3((slots + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                       master, model);
    return hipGetLastError();
}

}  // namespace ca
