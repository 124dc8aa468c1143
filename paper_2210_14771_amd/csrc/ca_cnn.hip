// gfx950 kernels of the learned strip scorer: a 1-D CNN along each strip
// whose output probability replaces the handcrafted edge score (arXiv
// 2210.14771, Section 2.2.4).  Input at each strip position: the 3 colours
// of 8 lines (24 channels, (v - 128) / 64, exact in bfloat16); four width-5
// convolutions 24 -> 16 -> 32 -> 32 -> 16 with ReLU, a 1x1 convolution to a
// logit, a sigmoid.  Weights and hidden activations are bfloat16, sums are
// float32 (MFMA accumulators).
//
// A strip is walked in steps of 64 positions (inference), or taken in windows of
// 128 positions of which the 112 central ones have exact logits: the 8 at each
// end are the receptive-field halo (training, and logits of given windows).
// Positions beyond the strip ends are zero in every layer's input.
//
// Each convolution is one GEMM: K = tap * C_in + c over position-major
// activations (channels contiguous), so an output position's B fragments are
// rows of the activation buffer.  Tiles are v_mfma_f32_16x16x32_bf16: A =
// weights [C_out][5 C_in] (padded to a multiple of 32 with zeros), B =
// activations, 16 output channels x 16 positions per tile.
#include "ca_cnn.h"
#include "ca_launch.h"
#include "ca_mfma.h"
#include "ca_reduce.h"
#include "ca_strip.h"

namespace ca {
namespace {

// --------------------------------------------------------------- kernels --

__global__ __launch_bounds__(kBlock) void k_mfma_probe(float *out)
{
    // A[m][k] = (m * 7 + k * 3) % 11 - 5, B[k][n] = (k * 5 + n * 2) % 13 - 6,
    // small integers: every product and sum is exact in float32.
    const int lane = threadIdx.x;
    if (lane >= 64)
        return;
    __bf16 a[8], b[8];
    for (int i = 0; i < 8; ++i) {
        const int k = 8 * (lane >> 4) + i;
        a[i] = to_bf16((float)(((lane & 15) * 7 + k * 3) % 11 - 5));
        b[i] = to_bf16((float)((k * 5 + (lane & 15) * 2) % 13 - 6));
    }
    const bf16x8 av = {a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]};
    const bf16x8 bv = {b[0], b[1], b[2], b[3], b[4], b[5], b[6], b[7]};
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc, 0, 0, 0);
    for (int j = 0; j < 4; ++j)
        out[(4 * (lane >> 4) + j) * 16 + (lane & 15)] = acc[j];
}

// ---------------------------------------------------------------- strips --
//
// Learned candidates: the best-scoring pixel of each half strip (ties:
// outermost).  A wave walks along a half strip, or along a part of one, in
// steps of 64 positions: layer l works two positions per layer behind the
// input, so a step's outputs need only the step's rows of the layer before and
// its last four rows of the step before, which stay in the layer's buffer.
//
// Column c of tile j is position 4 c + j of the step, so the inputs of tile j
// at tap t are those of tile j + t at tap 0: the four tiles of a layer read
// eight B fragments where tiles of 16 neighbours would read twenty.  Rows are
// stored in four planes, row 4 i + j as row i of plane j.
//
// All weights stay in registers (230 with the rest), so two waves share a SIMD
// and eight a workgroup's LDS; each takes an equal share of the half strips' steps
// (ca_deal.h).
//
// Bound by the chain of layers within a step (LDS round trips that two waves
// cover in part) beside about 340 vector instructions and 104 MFMAs a step.
// Measured, 64 1080p frames, 32 + 32 strips (kernel trace): 277 us with windows
// of 128 positions of which 112 are used and 68 KB of fragment reads per 64
// positions; 244 us in steps of 32 positions with four waves a SIMD and the
// larger layers' weights in LDS (98 KB: bound by LDS); 173 us so (32 KB).

// A layer's input rows: 4 of the step before, then the step's 64, in four
// planes; C channels (24 padded with zeros to 32) at PITCH, ROWS a plane.
template <int PITCH, int ROWS>
struct alignas(16) StripPlanes {
    static constexpr int kPlane = ROWS * PITCH + 8;
    __bf16 v[4 * kPlane];
};

struct StripRows {               // one wave's inputs of the four convolutions
    StripPlanes<32, 17> x0;
    StripPlanes<16, 18> h1;      // K is padded: a row that stays zero
    StripPlanes<32, 17> h2, h3;
};

// Offset of channels c .. c + 3 (c a multiple of 4) of a plane's row.  64-byte
// rows start in the same banks every fourth row: their 16-byte chunks are
// permuted by f = 0, 2, 3, 1 over four groups of four rows.  All different, they
// spread a store's 16 rows over the banks; and a read, which is served by groups
// of lanes (0-3, 12-15 and 20-27; 4-11, 16-19 and 28-31; the same of the upper
// half, measured) that hold rows 0-3 and 12-15 at one chunk and 4-11 at its
// neighbour, needs f(0), f(3), f(1) ^ 1 and f(2) ^ 1 to differ as well.  (LDS
// active 50.2 -> 45.3 million cycles a launch against f = 0, 1, 2, 3.)
template <int PITCH>
__device__ __forceinline__ int strip_off(int row, int c)
{
    if (PITCH == 16)
        return row * 16 + c;
    const int f = (((row >> 2) ^ (row >> 3)) & 1) << 1 | (row >> 3 & 1);
    return row * 32 + (((c >> 3) ^ f) << 3) + (c & 7);
}

// The step's input rows, (v - 128) / 64, zero outside the strip.
__device__ __forceinline__ void strip_encode(__bf16 *X, uint32_t (&px)[8], bool packed, int x, int L,
                                             const int (&xi)[3], int lane)
{
    if (!packed) {
        // dwords j = 4 i .. 4 i + 3 of three bytes to three of four
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t a = px[4 * i], b = px[4 * i + 1], c = px[4 * i + 2], e = px[4 * i + 3];
            px[3 * i] = __builtin_amdgcn_perm(b, a, 0x04020100u);
            px[3 * i + 1] = __builtin_amdgcn_perm(c, b, 0x05040201u);
            px[3 * i + 2] = __builtin_amdgcn_perm(e, c, 0x06050402u);
        }
    }
    if (x < 0 || x + kStep > L) {
        const bool in = (uint32_t)(x + lane) < (uint32_t)L;
#pragma unroll
        for (int i = 0; i < 6; ++i)
            px[i] = in ? px[i] : 0x80808080u;   // (128 - 128) / 64 = 0
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = (float)((px[2 * i + (e >> 2)] >> (8 * (e & 3))) & 0xFFu);
            o[e] = to_bf16(fmaf(v, 1.0f / 64.0f, -2.0f));   // exact
        }
        *reinterpret_cast<bf16x8 *>(X + xi[i]) = o;
    }
}

// The last four rows of a step become the first four of the next: row 16 of
// each plane row 0 (of 16-channel planes the zero row too, as row 1, which the
// next step writes before it is read).
template <int PITCH, int ROWS>
__device__ __forceinline__ uint32_t strip_keep(const StripPlanes<PITCH, ROWS> &X, int lane)
{
    return *reinterpret_cast<const uint32_t *>(X.v + (lane >> 4) * X.kPlane + 16 * PITCH
                                               + 2 * (lane & 15));
}
template <int PITCH, int ROWS>
__device__ __forceinline__ void strip_kept(StripPlanes<PITCH, ROWS> &X, uint32_t v, int lane)
{
    *reinterpret_cast<uint32_t *>(X.v + (lane >> 4) * X.kPlane + 2 * (lane & 15)) = v;
}

// Whether the step's outputs of a layer exist: +inf inside the strip, 0
// outside, for this lane's column of each tile; n = position of the step's
// first output.
__device__ __forceinline__ void strip_tops(float (&top)[4], int n, int L, int lane)
{
    const bool inside = n >= 0 && n + kStep <= L;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        top[j] = __builtin_inff();
    if (!inside) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            top[j] = (uint32_t)(n + 4 * (lane & 15) + j) < (uint32_t)L ? __builtin_inff() : 0.0f;
    }
}

// Fragments s = 0 .. 7 of a 32-channel layer's input: positions 4 c + s, lane
// group g its channels 8 g ..; xo: the offsets of rows c and c + 1.
__device__ __forceinline__ void strip_frags(bf16x8 (&f)[8], const StripPlanes<32, 17> &X,
                                            const int (&xo)[2])
{
#pragma unroll
    for (int s = 0; s < 8; ++s)
        f[s] = frag_at(X.v + (s & 3) * X.kPlane + xo[s >> 2]);
}

template <int MT, typename Y>
__device__ __forceinline__ void strip_store(Y &out, const f32x4 (&acc)[4][MT], const int (&yo)[MT],
                                            int n, int L, int lane)
{
    float top[4];
    strip_tops(top, n, L, lane);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<bf16x4 *>(out.v + j * out.kPlane + yo[mt]) =
                relu_bf16(acc[j][mt], top[j]);
}


// The network in a wave's registers: A fragments, biases, and the lane's offsets
// in StripRows.
struct StripNet {
    bf16x8 w1[5], w2[2][3], w3[2][5], w4[5];
    f32x4 b1, b2[2], b3[2], b4, w5;
    float b5;
    // input rows of this lane's position; rows c and c + 1 of a 32-channel
    // plane; of 16 channels, K groups g / 2 of a fragment lie one position
    // apart, from plane 3 to plane 0 of the next row at every fourth; outputs
    int xi[3], xo[2], xo2[2], yo1[1], yo[2];

    __device__ __forceinline__ StripNet(const uint8_t *model, int lane)
    {
        const __bf16 *W = reinterpret_cast<const __bf16 *>(model);
        const float *fb = reinterpret_cast<const float *>(model + kCnnFloatsOff);
        const int col = lane & 15, g = lane >> 4;
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            // 24 channels a tap in the model's rows, 32 here
            w1[t] = bf16x8{};
            if (g < 3)
                w1[t] = frag_at(W + kCnnWOff[0] + col * 128 + 24 * t + 8 * g);
            w3[0][t] = frag_at(W + kCnnWOff[2] + col * 160 + 32 * t + 8 * g);
            w3[1][t] = frag_at(W + kCnnWOff[2] + (16 + col) * 160 + 32 * t + 8 * g);
            w4[t] = frag_at(W + kCnnWOff[3] + col * 160 + 32 * t + 8 * g);
        }
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            w2[0][ks] = frag_at(W + kCnnWOff[1] + col * 96 + 32 * ks + 8 * g);
            w2[1][ks] = frag_at(W + kCnnWOff[1] + (16 + col) * 96 + 32 * ks + 8 * g);
        }
        auto four = [&](int at) { return *reinterpret_cast<const f32x4 *>(fb + at + 4 * g); };
        b1 = four(kCnnBOff[0]);
        b2[0] = four(kCnnBOff[1]);
        b2[1] = four(kCnnBOff[1] + 16);
        b3[0] = four(kCnnBOff[2]);
        b3[1] = four(kCnnBOff[2] + 16);
        b4 = four(kCnnBOff[3]);
        w5 = four(kCnnW5Off);
        b5 = fb[kCnnW5Off + 16];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            xi[i] = (lane & 3) * StripPlanes<32, 17>::kPlane + strip_off<32>((lane >> 2) + 1, 8 * i);
        constexpr int kPlane2 = StripPlanes<16, 18>::kPlane;
        const int at2 = strip_off<16>(col, 8 * (g & 1));
        xo2[0] = at2 + (g >> 1) * kPlane2;
        xo2[1] = at2 + (g >> 1) * (16 - 3 * kPlane2);
        yo1[0] = strip_off<16>(col + 1, 4 * g);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            xo[i] = strip_off<32>(col + i, 8 * g);
            yo[i] = strip_off<32>(col + 1, 16 * i + 4 * g);
        }
    }

    // One step, its input rows in R.x0, x the first one's position of a strip of
    // L: the logit of position x - 8 + 4 (lane % 16) + lane / 16.
    __device__ __forceinline__ float step(StripRows &R, int x, int L, int lane) const
    {
        bf16x8 b[8];
        wave_sync();
        uint32_t kept = strip_keep(R.x0, lane);
        strip_frags(b, R.x0, xo);
        {
            f32x4 acc[4][1];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[j][0] = b1;
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j][0] = mma(w1[t], b[j + t], acc[j][0]);
            strip_store<1>(R.h1, acc, yo1, x - 2, L, lane);
        }
        wave_sync();
        strip_kept(R.x0, kept, lane);
        kept = strip_keep(R.h1, lane);
#pragma unroll
        for (int s = 0; s < 8; ++s)
            b[s] = frag_at(R.h1.v + (s & 3) * R.h1.kPlane + (s >> 2) * 16
                           + xo2[(s & 3) == 3]);
        {
            f32x4 acc[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[j][0] = b2[0];
                acc[j][1] = b2[1];
            }
#pragma unroll
            for (int ks = 0; ks < 3; ++ks)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[j][0] = mma(w2[0][ks], b[j + 2 * ks], acc[j][0]);
                    acc[j][1] = mma(w2[1][ks], b[j + 2 * ks], acc[j][1]);
                }
            strip_store<2>(R.h2, acc, yo, x - 4, L, lane);
        }
        wave_sync();
        strip_kept(R.h1, kept, lane);
        kept = strip_keep(R.h2, lane);
        strip_frags(b, R.h2, xo);
        {
            f32x4 acc[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[j][0] = b3[0];
                acc[j][1] = b3[1];
            }
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[j][0] = mma(w3[0][t], b[j + t], acc[j][0]);
                    acc[j][1] = mma(w3[1][t], b[j + t], acc[j][1]);
                }
            strip_store<2>(R.h3, acc, yo, x - 6, L, lane);
        }
        wave_sync();
        strip_kept(R.h2, kept, lane);
        kept = strip_keep(R.h3, lane);
        strip_frags(b, R.h3, xo);
        float part_z[4];   // lane group's share of each tile's 1x1 layer
        {
            f32x4 acc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[j] = b4;
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = mma(w4[t], b[j + t], acc[j]);
            float top[4];
            strip_tops(top, x - 8, L, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 h = __builtin_bit_cast(u32x2, relu_bf16(acc[j], top[j]));
                float z = 0.0f;   // a bfloat16 is a float's upper half
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    z = fmaf(w5[2 * e], __uint_as_float(h[e] << 16), z);
                    z = fmaf(w5[2 * e + 1], __uint_as_float(h[e] & 0xFFFF0000u), z);
                }
                part_z[j] = z;
            }
        }
        wave_sync();
        strip_kept(R.h3, kept, lane);
        return b5 + tile_sums(part_z);
    }
};

__device__ __forceinline__ void strip_clear(StripRows &R, int lane)
{
    for (int i = lane; i < (int)(sizeof(StripRows) / 16); i += 64)
        reinterpret_cast<uint4 *>(&R)[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Logits of the central positions of uint8 windows [n][8][128][3]: a window is a
// strip of two steps, and the rows that the first one finds in place of its
// predecessor's feed only the window's halo.  One wave a window, two a workgroup
// (a small batch spreads over more compute units); the next step's bytes are
// loaded while a step's layers run.  Bound by the chain of layers within a step:
// a wave has few windows.  Measured, 3,584 windows (a call): 43.6 us with a byte
// at a time loaded at each window's turn, 19.3 us with the window's words
// fetched ahead and tiles of 16 neighbours, 17.0 us so.
__global__ __launch_bounds__(kCnnWaveBlock, 2) void k_cnn_windows(const uint8_t *model,
                                                                  const uint8_t *win,
                                                                  const int32_t *range, float *z_out,
                                                                  int n_windows)
{
    extern __shared__ __align__(16) uint8_t cnn_smem[];
    const int lane = threadIdx.x & 63;
    const int wv = uniform_int(threadIdx.x >> 6);
    StripRows &R = reinterpret_cast<StripRows *>(cnn_smem)[wv];
    strip_clear(R, lane);
    const int waves = gridDim.x * (kCnnWaveBlock / 64);
    uint32_t px[8];
    auto fetch = [&](int wi, int x) {
        StripWalk k;
        k.frame = win + (int64_t)wi * (kCnnLines * kCnnWin * 3);
        k.along = 3;
        k.across = 3 * kCnnWin;
        k.first = 0;
        k.L = kCnnWin;
        k.lines = kCnnLines;
        k.packed = false;
        k.last_row = wi == n_windows - 1;
        strip_fetch<kCnnLines>(px, k, x, lane);
    };
    const int first = blockIdx.x * (kCnnWaveBlock / 64) + wv;
    if (first < n_windows)
        fetch(first, 0);
    const StripNet net(model, lane);
    for (int wi = first; wi < n_windows; wi += waves) {
        const int lo = uniform_int(min(max(range[2 * wi], 0), kCnnWin));
        const int L = max(uniform_int(min(range[2 * wi + 1], kCnnWin)) - lo, 0);
#pragma unroll 1
        for (int x = 0; x < kCnnWin; x += kStep) {
            wave_sync();
            strip_encode(R.x0.v, px, false, x - lo, L, net.xi, lane);
            if (x == 0)
                fetch(wi, kStep);
            else if (wi + waves < n_windows)
                fetch(wi + waves, 0);
            const float z = net.step(R, x - lo, L, lane);
            const int n = x - kCnnHalo + 4 * (lane & 15) + (lane >> 4);
            if (n >= kCnnHalo && n < kCnnWin - kCnnHalo)
                z_out[(int64_t)wi * kCnnOut + n - kCnnHalo] = z;
        }
    }
}

template <bool MIXED>
__global__ __launch_bounds__(64 * kStripWaves, 2) void k_cnn_strips(CnnStripArgs a)
{
    extern __shared__ __align__(16) uint8_t cnn_smem[];
    __shared__ StripMeet meet;
    const int lane = threadIdx.x & 63;
    const int wv = uniform_int(threadIdx.x >> 6);
    if (threadIdx.x <= kStripWaves)
        meet.best[threadIdx.x] = 0;
    __syncthreads();
    StripRows &R = reinterpret_cast<StripRows *>(cnn_smem)[wv];
    strip_clear(R, lane);
    const StripNet net(a.model, lane);
    strip_shares<kCnnHalo, MIXED, true>(a, meet, lane, wv, [&](const FrameDev &d, bool horizontal,
                                                         int pos, int half, int p0, int p1) {
        StripWalk k;
        strip_walk<kCnnLines>(k, a.frames, d, horizontal, pos);
        uint64_t best = 0;
        uint32_t px[8];
        int x = p0 - kCnnHalo;   // first new input position of the step
        if (p0 < p1)
            strip_fetch<kCnnLines>(px, k, x, lane);
        for (; p0 < p1 && x - kCnnHalo < p1; x += kStep) {
            strip_encode(R.x0.v, px, k.packed, x, k.L, net.xi, lane);
            if (x + kStep - kCnnHalo < p1)
                strip_fetch<kCnnLines>(px, k, x + kStep, lane);
            const float z = net.step(R, x, k.L, lane);
            const int p = x - kCnnHalo + 4 * (lane & 15) + (lane >> 4);
            if (p >= p0 && p < p1) {
                const uint64_t key = strip_key(z, p, half, k.L);
                best = best > key ? best : key;
            }
        }
        return wave_max(best);
    });
}

// ------------------------------------------------------------- training --
//
// Backward pass of one window, given the forward activations (bfloat16) of
// the same window.  Backward signals dP_l (the gradient at layer l's
// pre-activation, ReLU mask applied) are stored in bfloat16, sums are float32
// MFMA accumulators.  Only the central 112 logits carry a loss; every
// activation they depend on is exact within the window, so the window's
// gradients equal those of the whole strip restricted to those positions.
//
//   input gradients   dX_{l-1} = flipped-weight convolution of dP_l (a
//                     forward-shaped GEMM), masked by h_{l-1} > 0;
//   weight gradients  dW_l[o][t C_in + c] = sum_n dP_l[n][o] X[n + t - 2][c],
//                     an MFMA GEMM whose K runs over the 128 positions.
//                     Both operands are columns of position-major buffers,
//                     which ds_read_b64_tr_b16 delivers transposed, so a tap
//                     is a row offset;
//   bias gradients    the same GEMM against a column of ones.
//
// The four waves of a workgroup take 32 positions each (two tiles) in the
// forward-shaped GEMMs.  In the weight gradients wave (a, b) takes half a of
// the positions and half b of the tiles (output channels 16 b .. of the
// 32-channel layers, half of the columns of the others): 24 tiles and three
// bias columns, 108 registers kept across the workgroup's windows.  A split of
// the tiles alone reads each operand twice as often, one of the positions
// alone needs 200 registers.  The 1x1 layer, the loss and dP4 are formed in
// the registers of the last convolution.
//
// Bound by LDS reads (about 150 fragments of 1 KB a wave and window) and the
// vector instructions beside them; 77 KB of LDS and 256 registers let two
// workgroups share a compute unit.  Measured, 14,336 windows: 791 us with
// channel-major copies of the signals and element-wise gathered operands, 258
// us so (kernel trace).

// Element offset of channels c .. c + 7 (c a multiple of 4) of row `row` in
// a position-major buffer of C channels.  With 32 or 16 channels the
// 16-byte chunks of a row are permuted by row (XOR with bits of the row
// index) so that the 16 lanes of one LDS pass, which read or write 16
// consecutive rows at the same channel, hit 16 distinct groups of 4 banks
// instead of 4 (32 channels) or 8 (16 channels); 24-channel rows already do.
// The permutation depends only on row / 4 mod 4 (row / 8 mod 2), so shifting
// by whole 16-row tiles keeps it.
template <int C>
__device__ __forceinline__ int act_off(int row, int c)
{
    static_assert(C == 16 || C == 24 || C == 32, "buffer width");
    if (C == 32)
        return row * 32 + ((((c >> 3) ^ (row >> 2)) & 3) << 3) + (c & 7);
    if (C == 16)
        return row * 16 + ((((c >> 3) ^ (row >> 3)) & 1) << 3) + (c & 7);
    return row * 24 + c;
}

struct alignas(16) CnnGradLds {
    __bf16 w3[10 * 512];          // layer 3's A fragments, [5 mt + ks][lane][8]
    __bf16 f3[10 * 512];          // the flipped layer 3's
    __bf16 f4[6 * 512];           // the flipped layer 4's, [3 mt + ks]
    __bf16 x0[kCnnRows * 24];
    __bf16 h1[kCnnRows * 16];
    __bf16 h2[kCnnRows * 32];
    __bf16 h3[kCnnRows * 32];
    __bf16 d16[kCnnRows * 16];    // dP4, later dP1
    __bf16 d3[kCnnRows * 32];     // dP3
    __bf16 d2[kCnnRows * 32];     // dP2
    __bf16 ones[8];
    float fb[128];
};
static_assert(sizeof(CnnGradLds) <= 81920, "two workgroups per compute unit");
constexpr int kGradTail = 18;     // w5 [16], b5, loss
static_assert((kCnnWElems + 3 * 64 + 4 * kGradTail) * sizeof(float) <= sizeof(CnnGradLds),
              "sums fit the LDS");

__global__ __launch_bounds__(kBlock, 2) void k_cnn_grad(CnnTrainArgs a)
{
    extern __shared__ __align__(16) uint8_t cnn_smem[];
    CnnGradLds &G = *reinterpret_cast<CnnGradLds *>(cnn_smem);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = uniform_int(tid >> 6);
    const int half_n = wv >> 1, half_t = wv & 1;
    const __bf16 *W = reinterpret_cast<const __bf16 *>(a.model);
    const __bf16 *Wf = reinterpret_cast<const __bf16 *>(a.model + kCnnFlipOff);
    {
        uint4 *z = reinterpret_cast<uint4 *>(&G);
        for (int i = tid; i < (int)(sizeof(CnnGradLds) / 16); i += kBlock)
            z[i] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        const float *mf = reinterpret_cast<const float *>(a.model + kCnnFloatsOff);
        if (tid < kCnnFloats)
            G.fb[tid] = mf[tid];
        if (tid < 8)
            G.ones[tid] = to_bf16(1.0f);
        const Place L(lane);
        for (int f = wv; f < 26; f += 4) {
            const int k = f < 10 ? f : f < 20 ? f - 10 : f - 20;
            const int ks = f < 20 ? k % 5 : k % 3, mt = f < 20 ? k / 5 : k / 3;
            const __bf16 *src = f < 10   ? W + kCnnWOff[2] + (16 * mt + L.col) * 160
                                : f < 20 ? Wf + kCnnFOff[1] + (16 * mt + L.col) * 160
                                         : Wf + kCnnFOff[2] + (16 * mt + L.col) * 96;
            *reinterpret_cast<bf16x8 *>(G.w3 + f * 512 + lane * 8) = frag_at(src + 32 * ks + 8 * L.g);
        }
        __syncthreads();
    }

    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 g1[4], g2[5], g3[10], g4[5], gb2 = zero4, gb3 = zero4, gb4 = zero4;
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        g3[i] = zero4;
        if (i < 5)
            g2[i] = g4[i] = zero4;
        if (i < 4)
            g1[i] = zero4;
    }
    float pw5[4] = {0.0f, 0.0f, 0.0f, 0.0f}, pb5 = 0.0f, ploss = 0.0f;

    // The next window's bytes: position tid % 128, lines 4 (tid / 128) .. + 3,
    // fetched a window ahead.  A load is four bytes from the pixel on; line 7's
    // starts a byte early, so none leaves the window.
    uint32_t raw[4];
    auto fetch = [&](int wi) {
        const int n = tid & 127, j0 = 4 * (tid >> 7);
        const uint8_t *src =
            a.win + (int64_t)wi * (kCnnLines * kCnnWin * 3) + j0 * (kCnnWin * 3) + 3 * n;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int back = j == 3 && j0 ? 1 : 0;
            __builtin_memcpy(&raw[j], src + j * (kCnnWin * 3) - back, 4);
            raw[j] >>= 8 * back;
        }
    };
    const int w_begin = (int)((int64_t)blockIdx.x * a.n / gridDim.x);
    const int w_end = (int)((int64_t)(blockIdx.x + 1) * a.n / gridDim.x);
    if (w_begin < w_end)
        fetch(w_begin);
    for (int wi = w_begin; wi < w_end; ++wi) {
        const int lo = uniform_int(a.range[2 * wi]);
        const int hi = uniform_int(a.range[2 * wi + 1]);
        {
            const int t = fresh(tid);
            const int n = t & 127;
            const bool in = n >= lo && n < hi;
            bf16x4 o[3];
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                const float b = (float)((raw[k / 3] >> (8 * (k % 3))) & 0xFFu);
                o[k >> 2][k & 3] = to_bf16(in ? fmaf(b, 1.0f / 64.0f, -2.0f) : 0.0f);
            }
            bf16x4 *dst =
                reinterpret_cast<bf16x4 *>(G.x0 + (n + kCnnGuard) * 24 + 12 * (t >> 7));
#pragma unroll
            for (int k = 0; k < 3; ++k)
                dst[k] = o[k];
        }
        __syncthreads();
        if (wi + 1 < w_end)
            fetch(wi + 1);
        // targets and loss weights of this lane's two positions; where a position
        // carries no loss neither counts, nor does its logit (zero times a value
        // that is not finite is not zero)
        float tgt[2], lw[2], tops[2];
        bool carries[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int n = 32 * wv + (lane & 15) + 16 * t;
            const bool in = n >= lo && n < hi;
            const bool has = in && n >= kCnnHalo && n < kCnnWin - kCnnHalo;
            carries[t] = has;
            tops[t] = in ? __builtin_inff() : 0.0f;
            const int64_t j = (int64_t)wi * kCnnOut + (has ? n - kCnnHalo : 0);
            const float target = a.target[j];
            tgt[t] = has ? target : 0.0f;
            lw[t] = has ? a.weight[j] * a.scale : 0.0f;
        }
        // A fragment (mt, ks) of a layer's weights in global memory
        auto weights = [&](const __bf16 *w, const Place &L, int kp, int mt, int ks) {
            return frag_at(w + (16 * mt + L.col) * kp + 32 * ks + 8 * L.g);
        };
        {
            // layer 1: 24 -> 16
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(G.fb + kCnnBOff[0] + 4 * L.g);
            f32x4 acc[2];
            acc[0] = acc[1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 w = weights(W + kCnnWOff[0], L, 128, 0, ks);
                const __bf16 *x = G.x0 + (p0 + kCnnGuard - 2) * 24 + 32 * ks + 8 * L.g;
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = mma(w, frag_at(x + 384 * t), acc[t]);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
                *reinterpret_cast<bf16x4 *>(G.h1 + act_off<16>(p0 + 16 * t + kCnnGuard, 4 * L.g)) =
                    relu_bf16(acc[t] + bias, tops[t]);
        }
        __syncthreads();
        {
            // layer 2: 16 -> 32
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            f32x4 acc[2][2];
            acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                const __bf16 *x =
                    G.h1 + act_off<16>(p0 + kCnnGuard - 2 + 2 * ks + (L.g >> 1), 8 * (L.g & 1));
                const bf16x8 x0 = frag_at(x), x1 = frag_at(x + 256);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const bf16x8 w = weights(W + kCnnWOff[1], L, 96, mt, ks);
                    acc[mt][0] = mma(w, x0, acc[mt][0]);
                    acc[mt][1] = mma(w, x1, acc[mt][1]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    *reinterpret_cast<bf16x4 *>(
                        G.h2 + act_off<32>(p0 + 16 * t + kCnnGuard, 16 * mt + 4 * L.g)) =
                        relu_bf16(acc[mt][t]
                                      + *reinterpret_cast<const f32x4 *>(G.fb + kCnnBOff[1]
                                                                         + 16 * mt + 4 * L.g),
                                  tops[t]);
        }
        __syncthreads();
        {
            // layer 3: 32 -> 32
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const int frag = (16 * L.g + L.col) * 8;
            f32x4 acc[2][2];
            acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) {
                const __bf16 *x = G.h2 + act_off<32>(p0 + kCnnGuard - 2 + ks, 8 * L.g);
                const bf16x8 x0 = frag_at(x), x1 = frag_at(x + 512);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const bf16x8 w = frag_at(G.w3 + (5 * mt + ks) * 512 + frag);
                    acc[mt][0] = mma(w, x0, acc[mt][0]);
                    acc[mt][1] = mma(w, x1, acc[mt][1]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    *reinterpret_cast<bf16x4 *>(
                        G.h3 + act_off<32>(p0 + 16 * t + kCnnGuard, 16 * mt + 4 * L.g)) =
                        relu_bf16(acc[mt][t]
                                      + *reinterpret_cast<const f32x4 *>(G.fb + kCnnBOff[2]
                                                                         + 16 * mt + 4 * L.g),
                                  tops[t]);
        }
        __syncthreads();
        {
            // layer 4 (32 -> 16), the 1x1 layer, the loss and dP4: a position's
            // 16 channels sit in the four lane groups of its column
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(G.fb + kCnnBOff[3] + 4 * L.g);
            f32x4 acc[2];
            acc[0] = acc[1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) {
                const bf16x8 w = weights(W + kCnnWOff[3], L, 160, 0, ks);
                const __bf16 *x = G.h3 + act_off<32>(p0 + kCnnGuard - 2 + ks, 8 * L.g);
                acc[0] = mma(w, frag_at(x), acc[0]);
                acc[1] = mma(w, frag_at(x + 512), acc[1]);
            }
            bf16x4 h[2][1];
            h[0][0] = relu_bf16(acc[0] + bias, tops[0]);
            h[1][0] = relu_bf16(acc[1] + bias, tops[1]);
            const int own = L.g & 1;   // this lane's tile from here
            const float z = ordered_dot(G.fb + kCnnW5Off, h, G.fb[kCnnW5Off + 16]);
            const float lw_own = own ? lw[1] : lw[0], tgt_own = own ? tgt[1] : tgt[0];
            const bool carries_own = own ? carries[1] : carries[0];
            float dz[2];
            to_all_groups(carries_own ? lw_own * (sigmoid(z) - tgt_own) : 0.0f, dz);
            const f32x4 w5 = *reinterpret_cast<const f32x4 *>(G.fb + kCnnW5Off + 4 * L.g);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                pb5 += dz[t];    // every lane group alike; the first one's is taken
                f32x4 dp;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    pw5[j] = fmaf((float)h[t][0][j], dz[t], pw5[j]);
                    dp[j] = w5[j] * dz[t];
                }
                *reinterpret_cast<bf16x4 *>(G.d16 + act_off<16>(p0 + 16 * t + kCnnGuard, 4 * L.g)) =
                    relu_mask(dp, h[t][0]);
            }
            if (L.g < 2 && carries_own)   // soft binary cross entropy in its logit form
                ploss += lw_own * (fmaxf(z, 0.0f) - z * tgt_own + log1pf(expf(-fabsf(z))));
        }
        __syncthreads();
        const __bf16 one = to_bf16(1.0f);
        const bf16x8 ones8 = {one, one, one, one, one, one, one, one};
        {
            // dP3 = [h3 > 0] (flipped W4 * dP4)
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const int frag = (16 * L.g + L.col) * 8;
            f32x4 acc[2][2];
            acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                const __bf16 *x =
                    G.d16 + act_off<16>(p0 + kCnnGuard - 2 + 2 * ks + (L.g >> 1), 8 * (L.g & 1));
                const bf16x8 x0 = frag_at(x), x1 = frag_at(x + 256);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const bf16x8 w = frag_at(G.f4 + (3 * mt + ks) * 512 + frag);
                    acc[mt][0] = mma(w, x0, acc[mt][0]);
                    acc[mt][1] = mma(w, x1, acc[mt][1]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int o = act_off<32>(p0 + 16 * t + kCnnGuard, 16 * mt + 4 * L.g);
                    *reinterpret_cast<bf16x4 *>(G.d3 + o) =
                        relu_mask(acc[mt][t], *reinterpret_cast<const bf16x4 *>(G.h3 + o));
                }
        }
        {
            // dW4: columns 80 half_t .. + 79 (tap = tile / 2, channels 16 (tile % 2) ..)
            const Place L(fresh(lane));
            const int r = 64 * half_n + L.r + kCnnGuard;
            const __bf16 *d = G.d16 + act_off<16>(r, 4 * L.q);
            int o[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                const int tile = 5 * half_t + i;
                o[i] = act_off<32>(r - 2 + (tile >> 1), 16 * (tile & 1) + 4 * L.q);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 p = transposed(d + 512 * s, d + 512 * s + 256);
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    g4[i] = mma(p, transposed(G.h3 + o[i] + 1024 * s, G.h3 + o[i] + 1024 * s + 512),
                                g4[i]);
                gb4 = mma(p, ones8, gb4);
            }
        }
        __syncthreads();
        {
            // dP2 = [h2 > 0] (flipped W3 * dP3)
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            const int frag = (16 * L.g + L.col) * 8;
            f32x4 acc[2][2];
            acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) {
                const __bf16 *x = G.d3 + act_off<32>(p0 + kCnnGuard - 2 + ks, 8 * L.g);
                const bf16x8 x0 = frag_at(x), x1 = frag_at(x + 512);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const bf16x8 w = frag_at(G.f3 + (5 * mt + ks) * 512 + frag);
                    acc[mt][0] = mma(w, x0, acc[mt][0]);
                    acc[mt][1] = mma(w, x1, acc[mt][1]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int o = act_off<32>(p0 + 16 * t + kCnnGuard, 16 * mt + 4 * L.g);
                    *reinterpret_cast<bf16x4 *>(G.d2 + o) =
                        relu_mask(acc[mt][t], *reinterpret_cast<const bf16x4 *>(G.h2 + o));
                }
        }
        {
            // dW3: output channels 16 half_t ..
            const Place L(fresh(lane));
            const int r = 64 * half_n + L.r + kCnnGuard;
            const __bf16 *d = G.d3 + act_off<32>(r, 16 * half_t + 4 * L.q);
            int o[10];
#pragma unroll
            for (int i = 0; i < 10; ++i)
                o[i] = act_off<32>(r - 2 + (i >> 1), 16 * (i & 1) + 4 * L.q);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 p = transposed(d + 1024 * s, d + 1024 * s + 512);
#pragma unroll
                for (int i = 0; i < 10; ++i)
                    g3[i] = mma(p, transposed(G.h2 + o[i] + 1024 * s, G.h2 + o[i] + 1024 * s + 512),
                                g3[i]);
                gb3 = mma(p, ones8, gb3);
            }
        }
        __syncthreads();
        {
            // dP1 = [h1 > 0] (flipped W2 * dP2)
            const Place L(fresh(lane));
            const int p0 = 32 * wv + L.col;
            f32x4 acc[2];
            acc[0] = acc[1] = zero4;
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) {
                const bf16x8 w = weights(Wf + kCnnFOff[0], L, 160, 0, ks);
                const __bf16 *x = G.d2 + act_off<32>(p0 + kCnnGuard - 2 + ks, 8 * L.g);
                acc[0] = mma(w, frag_at(x), acc[0]);
                acc[1] = mma(w, frag_at(x + 512), acc[1]);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int o = act_off<16>(p0 + 16 * t + kCnnGuard, 4 * L.g);
                *reinterpret_cast<bf16x4 *>(G.d16 + o) =
                    relu_mask(acc[t], *reinterpret_cast<const bf16x4 *>(G.h1 + o));
            }
        }
        {
            // dW2: output channels 16 half_t .., a tile a tap
            const Place L(fresh(lane));
            const int r = 64 * half_n + L.r + kCnnGuard;
            const __bf16 *d = G.d2 + act_off<32>(r, 16 * half_t + 4 * L.q);
            int o[5];
#pragma unroll
            for (int i = 0; i < 5; ++i)
                o[i] = act_off<16>(r - 2 + i, 4 * L.q);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 p = transposed(d + 1024 * s, d + 1024 * s + 512);
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    g2[i] = mma(p, transposed(G.h1 + o[i] + 512 * s, G.h1 + o[i] + 512 * s + 256),
                                g2[i]);
                gb2 = mma(p, ones8, gb2);
            }
        }
        __syncthreads();
        {
            // dW1: columns 64 half_t .. + 63 of the 120 (contiguous in the
            // rows); columns 120 .. 127 read ones, the bias gradient
            const Place L(fresh(lane));
            const int r = 64 * half_n + L.r + kCnnGuard;
            const __bf16 *d = G.d16 + act_off<16>(r, 4 * L.q);
            const __bf16 *x = G.x0 + (r - 2) * 24 + 64 * half_t + 4 * L.q;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 p = transposed(d + 512 * s, d + 512 * s + 256);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool one_col = i == 3 && half_t == 1 && L.q >= 2;
                    const __bf16 *b = one_col ? G.ones : x + 16 * i + 768 * s;
                    g1[i] = mma(p, transposed(b, one_col ? b : b + 384), g1[i]);
                }
            }
        }
        __syncthreads();
    }

    // The workgroup's sums in a fixed order: half 1 of the positions through
    // the LDS, added to half 0's; the 1x1 layer's and the loss over all waves.
    float *sum = reinterpret_cast<float *>(&G);
    float *bias = sum + kCnnWElems;            // [3][2][32]: b4, b3, b2 by half_t (32 slots)
    float *tail = bias + 3 * 64;               // [4 waves][kGradTail]
    const Place L(lane);
    auto each = [&](auto fn) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int o = 4 * L.g + j;
#pragma unroll
            for (int i = 0; i < 10; ++i)
                fn(kCnnWOff[2] + (16 * half_t + o) * 160 + 16 * i + L.col, g3[i][j]);
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                fn(kCnnWOff[3] + o * 160 + 16 * (5 * half_t + i) + L.col, g4[i][j]);
                fn(kCnnWOff[1] + (16 * half_t + o) * 96 + 16 * i + L.col, g2[i][j]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                fn(kCnnWOff[0] + o * 128 + 16 * (4 * half_t + i) + L.col, g1[i][j]);
        }
    };
#pragma unroll
    for (int d = 1; d < 16; d *= 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            pw5[j] += __shfl_xor(pw5[j], d, 64);
        pb5 += __shfl_xor(pb5, d, 64);
        ploss += __shfl_xor(ploss, d, 64);
    }
    ploss += __shfl_xor(ploss, 16, 64);        // lane groups 0 and 1
    if (L.col == 0)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            tail[kGradTail * wv + 4 * L.g + j] = pw5[j];
    if (lane == 0) {
        tail[kGradTail * wv + 16] = pb5;
        tail[kGradTail * wv + 17] = ploss;
    }
    if (half_n == 1) {
        each([&](int i, float v) { sum[i] = v; });
        if (L.col == 0)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                bias[32 * half_t + 4 * L.g + j] = gb4[j];
                bias[64 + 32 * half_t + 4 * L.g + j] = gb3[j];
                bias[128 + 32 * half_t + 4 * L.g + j] = gb2[j];
            }
    }
    __syncthreads();
    float *out = a.partial + (int64_t)blockIdx.x * kCnnGradStride;
    if (half_n == 0) {
        each([&](int i, float v) { out[i] = v + sum[i]; });
        if (L.col == 0)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int o = 4 * L.g + j;
                float *b = out + kCnnWElems;
                if (half_t == 0)
                    b[kCnnBOff[3] + o] = gb4[j] + bias[o];
                b[kCnnBOff[2] + 16 * half_t + o] = gb3[j] + bias[64 + 32 * half_t + o];
                b[kCnnBOff[1] + 16 * half_t + o] = gb2[j] + bias[128 + 32 * half_t + o];
            }
        if (half_t == 1 && L.col == 8)         // column 120 of dW1
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int o = 4 * L.g + j;
                out[kCnnWElems + kCnnBOff[0] + o] = g1[3][j] + sum[kCnnWOff[0] + o * 128 + 120];
            }
    }
    if (tid < kGradTail)
        out[kCnnWElems + kCnnW5Off + tid] =
            (tail[tid] + tail[kGradTail + tid])
            + (tail[2 * kGradTail + tid] + tail[3 * kGradTail + tid]);
    else if (tid >= kCnnW5Off + kGradTail && tid < kCnnGradStride - kCnnWElems)
        out[kCnnWElems + tid] = 0.0f;
}

// Parameter layout of the model file (float32): per layer W[o][c][t], b[o].
struct FileLayer {
    int cin, cout, kp, woff, fw, fb;
};
__device__ __forceinline__ FileLayer file_layer(int l)
{
    switch (l) {
    case 0: return {24, 16, 128, kCnnWOff[0], 0, 1920};
    case 1: return {16, 32, 96, kCnnWOff[1], 1936, 4496};
    case 2: return {32, 32, 160, kCnnWOff[2], 4528, 9648};
    default: return {32, 16, 160, kCnnWOff[3], 9680, 12240};
    }
}
constexpr int kFileW5 = 12256;
constexpr int kFileB5 = 12272;

// Sum the workgroup partials; scatter to the model-file order.
static_assert(kCnnGradStride % kReduceCols == 0, "whole column groups");
__global__ __launch_bounds__(kReduceThreads) void k_cnn_reduce(const float *partial, int grid,
                                                               float *grad, float *loss)
{
    __shared__ float s_sum[kReduceCols];
    column_sums(partial, grid, kCnnGradStride, s_sum);
    if (threadIdx.x >= kReduceCols)
        return;
    const int i = blockIdx.x * kReduceCols + threadIdx.x;
    const float v = s_sum[threadIdx.x];
    if (i < kCnnWElems) {
        const int l = i < kCnnWOff[1] ? 0 : i < kCnnWOff[2] ? 1 : i < kCnnWOff[3] ? 2 : 3;
        const FileLayer L = file_layer(l);
        const int o = (i - L.woff) / L.kp;
        const int k = (i - L.woff) - o * L.kp;
        if (k >= 5 * L.cin)
            return;
        const int t = k / L.cin, c = k - t * L.cin;
        grad[L.fw + (o * L.cin + c) * 5 + t] = v;
        return;
    }
    const int r = i - kCnnWElems;
    if (r < 96) {
        const int l = r < kCnnBOff[1] ? 0 : r < kCnnBOff[2] ? 1 : r < kCnnBOff[3] ? 2 : 3;
        grad[file_layer(l).fb + r - kCnnBOff[l]] = v;
    } else if (r < 112) {
        grad[kFileW5 + r - 96] = v;
    } else if (r == 112) {
        grad[kFileB5] = v;
    } else if (r == 113) {
        loss[0] = v;
    }
}

// SGD with momentum (m = mu m + g, p -= lr m) on the master weights (file order),
// each weight's copies in the device model block with it (k_cnn_pack's layout; the padding stays): a
// repack of its own cost a launch, 1.8 us of a step.
__global__ __launch_bounds__(kBlock) void k_cnn_update(float *master, float *mom,
                                                       const float *grad, float lr, float mu,
                                                       uint8_t *model)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= kCnnParams)
        return;
    const float m = mu * mom[i] + grad[i];
    mom[i] = m;
    const float v = master[i] - lr * m;
    master[i] = v;
    __bf16 *w = reinterpret_cast<__bf16 *>(model);
    float *fb = reinterpret_cast<float *>(model + kCnnFloatsOff);
    __bf16 *wf = reinterpret_cast<__bf16 *>(model + kCnnFlipOff);
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const FileLayer L = file_layer(l);
        const int r = i - L.fw;
        if (r >= 0 && r < L.cout * L.cin * 5) {
            const int t = r % 5, c = r / 5 % L.cin, o = r / 5 / L.cin;
            w[L.woff + o * L.kp + t * L.cin + c] = to_bf16(v);
            if (l > 0)
                wf[kCnnFOff[l - 1] + c * (l == 3 ? 96 : 160) + (4 - t) * L.cout + o] = to_bf16(v);
        }
        if (i >= L.fb && i < L.fb + L.cout)
            fb[kCnnBOff[l] + i - L.fb] = v;
    }
    if (i >= kFileW5 && i < kFileW5 + 16)
        fb[kCnnW5Off + i - kFileW5] = (float)to_bf16(v);
    if (i == kFileB5)
        fb[kCnnW5Off + 16] = v;
}

// Device model block from float32 master weights: every slot (padding
// included) is written.
__global__ __launch_bounds__(kBlock) void k_cnn_pack(const float *master, uint8_t *model)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    __bf16 *w = reinterpret_cast<__bf16 *>(model);
    float *fb = reinterpret_cast<float *>(model + kCnnFloatsOff);
    __bf16 *wf = reinterpret_cast<__bf16 *>(model + kCnnFlipOff);
    if (i < kCnnWElems) {
        const int l = i < kCnnWOff[1] ? 0 : i < kCnnWOff[2] ? 1 : i < kCnnWOff[3] ? 2 : 3;
        const FileLayer L = file_layer(l);
        const int o = (i - L.woff) / L.kp;
        const int k = (i - L.woff) - o * L.kp;
        float v = 0.0f;
        if (k < 5 * L.cin) {
            const int t = k / L.cin, c = k - t * L.cin;
            v = master[L.fw + (o * L.cin + c) * 5 + t];
        }
        w[i] = to_bf16(v);
        return;
    }
    int r = i - kCnnWElems;
    if (r < 128) {
        float v = 0.0f;
        if (r < 96) {
            const int l = r < kCnnBOff[1] ? 0 : r < kCnnBOff[2] ? 1 : r < kCnnBOff[3] ? 2 : 3;
            v = master[file_layer(l).fb + r - kCnnBOff[l]];
        } else if (r < 112) {
            v = (float)to_bf16(master[kFileW5 + r - 96]);
        } else if (r == 112) {
            v = master[kFileB5];
        }
        fb[r] = v;
        return;
    }
    r -= 128;
    if (r < kCnnFElems) {
        // Wf_l[c][t' C_out + o] = W_l[o][c][4 - t'] for layers 2, 3, 4
        const int q = r < kCnnFOff[1] ? 0 : r < kCnnFOff[2] ? 1 : 2;
        const FileLayer L = file_layer(q + 1);
        const int kpf = q == 2 ? 96 : 160;
        const int c = (r - kCnnFOff[q]) / kpf;
        const int k = (r - kCnnFOff[q]) - c * kpf;
        float v = 0.0f;
        if (k < 5 * L.cout) {
            const int tp = k / L.cout, o = k - tp * L.cout;
            v = master[L.fw + (o * L.cin + c) * 5 + (4 - tp)];
        }
        wf[r] = to_bf16(v);
    }
}

}  // namespace

hipError_t launch_mfma_probe(float *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_mfma_probe, dim3(1), dim3(kBlock), 0, s, out);
    return hipGetLastError();
}

constexpr size_t kCnnWaveLds = (size_t)(kCnnWaveBlock / 64) * sizeof(StripRows);

hipError_t launch_cnn_windows(const uint8_t *model, const uint8_t *win, const int32_t *range,
                              float *z, int n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    const int waves = kCnnWaveBlock / 64;
    int grid = (n + waves - 1) / waves;
    grid = grid < 1024 ? grid : 1024;
    hipLaunchKernelGGL(k_cnn_windows, dim3(grid), dim3(kCnnWaveBlock), kCnnWaveLds, s, model, win,
                       range, z, n);
    return hipGetLastError();
}

int cnn_strips_blocks_per_cu()
{
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_cnn_strips<false>, 64 * kStripWaves,
                                                     kStripWaves * sizeof(StripRows))
            != hipSuccess
        || b < 1) {
        (void)hipGetLastError();
        b = 1;
    }
    return b;
}

hipError_t launch_cnn_strips(const CnnStripArgs &a, int groups_per_xcd, hipStream_t s,
                             hipEvent_t start, hipEvent_t stop)
{
    if (a.n_items <= 0)
        return hipSuccess;
    launch_maybe_timed(a.mixed ? k_cnn_strips<true> : k_cnn_strips<false>,
                       dim3(kXcds * groups_per_xcd), dim3(64 * kStripWaves),
                       kStripWaves * sizeof(StripRows), s, start, stop, a);
    return hipGetLastError();
}

}  // namespace ca

namespace ca {

hipError_t launch_cnn_grad(const CnnTrainArgs &a, int grid, hipStream_t s)
{
    if (grid <= 0)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_cnn_grad, dim3(grid), dim3(kBlock), sizeof(CnnGradLds), s, a);
    return hipGetLastError();
}

hipError_t launch_cnn_reduce(const float *partial, int grid, float *grad_out, float *loss_out,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_cnn_reduce, dim3(kCnnGradStride / kReduceCols), dim3(kReduceThreads), 0, s,
                       partial, grid, grad_out, loss_out);
    return hipGetLastError();
}

hipError_t launch_cnn_update(float *master, float *momentum, const float *grad, float lr,
                             float mom, uint8_t *model, hipStream_t s)
{
    hipLaunchKernelGGL(k_cnn_update, dim3((kCnnParams + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                       master, momentum, grad, lr, mom, model);
    return hipGetLastError();
}

hipError_t launch_cnn_pack(const float *master, uint8_t *model, hipStream_t s)
{
    constexpr int slots = kCnnWElems + 128 + kCnnFElems;
    hipLaunchKernelGGL(k_cnn_pack, dim3((slots + kBlock - 1) / kBlock), dim3(kBlock), 0, s, master,
                       model);
    return hipGetLastError();
}

}  // namespace ca
