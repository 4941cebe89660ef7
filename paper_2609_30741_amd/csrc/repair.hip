// Learned gap/edge repair network: inference and training kernels.
//
// 3x3 convolutions run as implicit GEMMs on the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulate).  Forward: rows of the GEMM
// are output channels (weights packed [cout padded to 16][9][cin padded to
// 16], each row padded with zeros to a multiple of 32), columns are 16
// consecutive pixels of one image row, the reduction runs over (tap, input
// channel).  The input-gradient pass is the same kernel
// with the weights transposed and flipped.  The weight gradient is a GEMM
// over pixels: each block accumulates its pixels into a partial, and a
// second kernel adds the partials in a fixed order, so results are
// deterministic.  Activations and gradients between layers are stored as
// bf16 [B][H][W][C], channels innermost; a layer may read or write a
// channel slice of a larger tensor (the pixel stride exceeds the slice); a
// decoder reads its upsampled channels from the coarser level and the others
// from the skip connection, so no concatenation is stored.  The images the network reads and writes are
// planar fp32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "bgs_repair.h"

namespace {

typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct LayerDef {
    int cin, cout, relu;
};
// e1a e1b e2a e2b e3a e3b d2 d1 out
constexpr int kLayers = 9;
constexpr LayerDef kNet[kLayers] = {{5, 16, 1},  {16, 16, 1}, {16, 32, 1}, {32, 32, 1}, {32, 64, 1},
                                    {64, 64, 1}, {96, 32, 1}, {48, 16, 1}, {16, 4, 0}};
enum { E1A, E1B, E2A, E2B, E3A, E3B, D2, D1, OUT };

constexpr int pad16(int v) { return (v + 15) & ~15; }

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
    // Round to nearest even (values are finite).
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------
// Convolution (forward, or input gradient with transposed weights).
// Activations and gradients are bf16 [B][H][W][C] with the channels of a
// pixel contiguous; a tensor's pixel stride (ps) is a multiple of 8 and may
// exceed the channels a layer reads or writes (a slice of a concatenation,
// or zero padding), and every buffer is 16-byte aligned.
// ---------------------------------------------------------------------------
struct ConvArgs {
    const uint16_t* in;  // channel 0 of the input
    int64_t in_bs;       // elements per image
    int in_ps;           // elements per pixel
    int cin;
    // Optional half-resolution source of input channels [0, up_c): read at
    // (y / 2, x / 2), the nearest 2x upsample, so a decoder's concatenated
    // input needs no upsampled copy.  Channel ci >= up_c is channel
    // ci - up_c of in.
    const uint16_t* up;
    int64_t up_bs;
    int up_ps;
    int up_c;
    const uint16_t* w;  // [pad16(cout)][kpad] bf16, k = tap * cpad + ci, zero for k >= 9 cpad
    int kpad;           // pad32(9 cpad)
    const float* bias;  // may be null
    int cout;           // a multiple of 4
    uint16_t* out;      // channel 0 of the output (bf16, out_bs, out_ps), or
    float* out_f;       // fp32 [B][cout][H][W] planes (exactly one is set)
    int64_t out_bs;
    int out_ps;
    const uint16_t* mask;  // may be null: output zero where mask <= 0 (layout of out)
    int64_t mask_bs;
    int mask_ps;
    // May be null: also store the 2x2 mean of the (bf16) output, [H/2][W/2]
    // pixels of pool_ps elements (H and W even).
    uint16_t* pool;
    int64_t pool_bs;
    int pool_ps;
    int relu;
    int H, W;
    // Inference: the first layer forms its input from the images
    // (kConvInput), the last one writes the repaired image (kConvOutput).
    const float* rgb;     // [B][3][H][W]
    const float* z;       // [B][H][W]
    const uint8_t* hole;  // [B][H][W]
    float* rgb_out;       // [B][3][H][W]
    float* err_out;       // [B][H][W], may be null
};
enum { kConvPlain, kConvInput, kConvOutput };

// Block: 4 waves over 64 pixels (x from blockIdx.x * 64) of R consecutive
// rows from R blockIdx.y; blockIdx.z = image * groups + group, a group
// being MT <= 4 16-row tiles of output channels.
// The block first stages input rows R blockIdx.y - 1 .. + R, x from
// blockIdx.x * 64 - 1 to + 64 (zero outside the image), of every input
// channel (padded to CPAD, a multiple of 16, with zeros) in LDS:
// [R + 2][66][CPAD + conv_pad(CPAD)] bf16, one 16-byte load and store per
// 8 channels of a pixel.  The reduction index is k = tap * CPAD + ci in
// 32-deep slices of v_mfma_f32_16x16x32_bf16; a lane's eight operands of a
// slice are eight consecutive channels of one tap, one 16-byte LDS read,
// and each weight operand serves all R rows and all of a wave's column
// tiles.
constexpr int kConvCols = 66;

constexpr int pad32(int v) { return (v + 31) & ~31; }
// Spare channel slots per staged pixel, by width, chosen by measurement
// over 0 to 32 spare slots (LDS bank-conflict counter and kernel time): the
// 16-byte operand reads of 48 and 96 channels are cheapest with none (and
// the smaller stage fits more blocks per CU: 96 channels at 800x600, 29 ->
// 23 us), those of 32 and 64 channels with 16, and 16 channels run
// fastest with 8.
constexpr int conv_pad(int cpad) { return cpad == 16 ? 8 : cpad == 32 || cpad == 64 ? 16 : 0; }
constexpr size_t conv_lds_bytes(int cpad, int rows) {
    return (size_t)(rows + 2) * kConvCols * (cpad + conv_pad(cpad)) * sizeof(uint16_t);
}

// Two floats to bf16, round to nearest even, the first in the low half.
__device__ __forceinline__ uint32_t pack_bf(float a, float b) {
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    const v2bf v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}

// Items of the fill that a thread has in flight: all of its share where
// that leaves registers, else half.
constexpr int conv_fill(int items) {
    const int u = (items + 255) / 256;
    return u <= 14 ? u : (u + 1) / 2;
}

// Input widths of the decoders, whose first channels come from the coarser
// level.
constexpr bool conv_has_up(int cpad) { return cpad == 48 || cpad == 96; }

// Network input of one pixel, eight channels: warped rgb (zero at holes),
// hole flag, 1/z (zero at holes and background), three zero slots.
__device__ __forceinline__ uint4 input_pixel(float r, float g, float b, float z, bool hole) {
    const float inv = (hole || !(z < INFINITY)) ? 0.f : 1.f / z;
    return uint4{pack_bf(hole ? 0.f : r, hole ? 0.f : g), pack_bf(hole ? 0.f : b, hole ? 1.f : 0.f), pack_bf(inv, 0.f), 0u};
}

// kMode: kConvInput and kConvOutput are the first and last layer of an
// inference pass, without the tensors (16 bytes a pixel written and read
// again, each) and the launches between them and the images.
template <int CPAD, int MT, int R, int kMode = kConvPlain>
__global__ __launch_bounds__(256) void k_conv3x3(ConvArgs a) {
    constexpr int PS = CPAD + conv_pad(CPAD);  // staged bf16 per pixel
    constexpr int G = CPAD / 8;               // 16-byte channel groups per pixel
    constexpr int SL = pad32(9 * CPAD) / 32;  // reduction slices
    extern __shared__ uint4 s_raw[];
    uint16_t* s_in = reinterpret_cast<uint16_t*>(s_raw);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int groups = (a.cout + 16 * MT - 1) / (16 * MT);
    const int y0 = blockIdx.y * R, b = blockIdx.z / groups, m0 = (blockIdx.z - b * groups) * MT;
    const int xb = blockIdx.x * 64;
    const int n = lane & 15, kg = lane >> 4;
    const int mt = min(MT, ((a.cout + 15) >> 4) - m0);
    // Wave w computes output tile m = w % MT (of the group) for CT = 4 / CW
    // consecutive 16-pixel column tiles from column tile CT (w / MT), so a
    // block reads each weight row 4 / MT times instead of 4 (MT = 3: waves
    // 0-2 take all four column tiles, wave 3 only helps with the fill).
    constexpr int CW = MT == 1 ? 4 : MT == 2 ? 2 : 1;  // waves per tile
    constexpr int CT = 4 / CW;
    const int wm = wave % MT, wc = (wave / MT) * CT;
    const bool busy = wave < MT * CW;
    // Weight operands run P slices ahead of their use in a register ring;
    // the first P are in flight during the fill.
    constexpr int P = SL < 8 ? SL : 8;
    const uint16_t* wl = a.w + (size_t)((m0 + min(wm, mt - 1)) * 16 + n) * a.kpad + 8 * kg;
    uint4 wq[P];
#pragma unroll
    for (int s = 0; s < P; ++s) wq[s] = *reinterpret_cast<const uint4*>(wl + 32 * s);
    // kConvOutput: the images' values, in flight during the fill.  Lane kg
    // holds output channel kg of its pixels (spread weight rows): a colour
    // plane, or the predicted error.
    float oq[kMode == kConvOutput ? R : 1];
    uint8_t oh[kMode == kConvOutput ? R : 1];
    if constexpr (kMode == kConvOutput) {
        static_assert(CT == 1, "the output layer has one column tile a wave");
        const int64_t hw = (int64_t)a.H * a.W;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int x = min(xb + 16 * wc + n, a.W - 1), y = min(y0 + r, a.H - 1);
            const int64_t p = (int64_t)y * a.W + x;
            oh[r] = a.hole[b * hw + p];
            oq[r] = a.rgb[(3 * b + min(kg, 2)) * hw + p];
        }
    }
    // Fill: item = (row, column, channel group), group fastest, so a wave's
    // loads walk consecutive 16-byte words of consecutive pixels.  A thread
    // takes every 256th item and steps its (row, column, group) along, with
    // 32-bit offsets from the block's corner; blocks inside the image skip
    // the bounds.  (These layers are as much bound by such arithmetic as by
    // their products: deriving every item from its number, the 48-channel
    // layer filled 57% of its issue slots with vector instructions.)  Up to
    // 14 items' loads per thread are in flight before their stores.
    // Channels at or past cin read as zero (a group past cin is not loaded:
    // it may lie beyond the tensor's pixel stride); only 16-channel inputs
    // have any.
    constexpr int items = (R + 2) * kConvCols * G, U = conv_fill(items);
    constexpr bool kUp = conv_has_up(CPAD), kPartial = CPAD == 16;
    const char* in0 = reinterpret_cast<const char*>(
        a.in + (int64_t)b * a.in_bs + ((int64_t)(y0 - 1) * a.W + (xb - 1)) * a.in_ps - a.up_c);
    // y0 and xb are even, so the corner lies in the odd half of its 2x2 block.
    const char* up0 = kUp ? reinterpret_cast<const char*>(a.up + (int64_t)b * a.up_bs +
                                                          ((int64_t)(y0 / 2 - 1) * (a.W >> 1) + xb / 2 - 1) * a.up_ps)
                          : nullptr;
    const uint32_t in_row = 2u * a.W * a.in_ps, in_px = 2u * a.in_ps, up_row = (uint32_t)(a.W >> 1) * 2u * a.up_ps,
                   up_px = 2u * a.up_ps;
    const auto fill = [&](auto inside) {
        int g = (int)threadIdx.x % G, rc = (int)threadIdx.x / G;
        int c = rc % kConvCols, r = rc / kConvCols;
#pragma unroll
        for (int i0 = 0; i0 < items; i0 += 256 * U) {
            uint4 v[U];
            int at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int ci = 8 * g;
                at[u] = rc * PS + ci;
                bool ok = i0 + 256 * u + 256 <= items || i0 + 256 * u + (int)threadIdx.x < items;
                if (!inside.value)
                    ok = ok && (unsigned)(y0 - 1 + r) < (unsigned)a.H && (unsigned)(xb - 1 + c) < (unsigned)a.W;
                if (kPartial) ok = ok && ci < a.cin;
                v[u] = uint4{0u, 0u, 0u, 0u};
                if (ok) {
                    const bool up = kUp && ci < a.up_c;
                    const char* src = up ? up0 : in0;
                    const uint32_t rr = up ? (uint32_t)(r + 1) >> 1 : (uint32_t)r, cc = up ? (uint32_t)(c + 1) >> 1 : (uint32_t)c;
                    v[u] = *reinterpret_cast<const uint4*>(
                        src + (uint32_t)(rr * (up ? up_row : in_row) + cc * (up ? up_px : in_px) + 2u * ci));
                }
                // The thread's next item, 256 on.
                constexpr int dg = 256 % G, dc = 256 / G;
                rc += dc;
                c += dc;
                if (dg) {
                    g += dg;
                    const bool carry = g >= G;
                    g -= carry ? G : 0;
                    rc += carry ? 1 : 0;
                    c += carry ? 1 : 0;
                }
#pragma unroll
                for (int k = 0; k < (dc + kConvCols) / kConvCols; ++k) {
                    const bool wrap = c >= kConvCols;
                    c -= wrap ? kConvCols : 0;
                    r += wrap ? 1 : 0;
                }
            }
            if (kPartial && a.cin < 16) {  // uniform: groups that straddle cin
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int left = a.cin - 8 * g;  // 256 % G is 0: one group per thread
                    uint32_t* q = reinterpret_cast<uint32_t*>(&v[u]);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        q[k] &= (2 * k + 1 < left ? 0xFFFF0000u : 0u) | (2 * k < left ? 0xFFFFu : 0u);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + 256 * u + 256 <= items || i0 + 256 * u + (int)threadIdx.x < items)
                    *reinterpret_cast<uint4*>(s_in + at[u]) = v[u];
        }
    };
    if constexpr (kMode == kConvInput) {
        static_assert(CPAD == 16 && PS == 24, "the network input has eight of 16 channels");
        constexpr int pixels = (R + 2) * kConvCols, V = (pixels + 255) / 256;
        const int64_t hw = (int64_t)a.H * a.W;
        const float *ib = a.rgb + 3 * b * hw, *zb = a.z + b * hw;
        const uint8_t* hb = a.hole + b * hw;
        float cr[V], cg[V], cb[V], cz[V];
        uint8_t ch[V];
        bool in[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {  // all loads first
            const int i = (int)threadIdx.x + 256 * u, r = i / kConvCols, c = i - r * kConvCols;
            const int y = y0 - 1 + r, x = xb - 1 + c;
            in[u] = i < pixels && y >= 0 && y < a.H && x >= 0 && x < a.W;
            const int64_t p = in[u] ? (int64_t)y * a.W + x : 0;
            cr[u] = ib[p];
            cg[u] = ib[hw + p];
            cb[u] = ib[2 * hw + p];
            cz[u] = zb[p];
            ch[u] = hb[p];
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int i = (int)threadIdx.x + 256 * u;
            if (i >= pixels) continue;
            uint4 v = input_pixel(cr[u], cg[u], cb[u], cz[u], ch[u] != 0);
            if (!in[u]) v = uint4{0u, 0u, 0u, 0u};
            *reinterpret_cast<uint4*>(s_in + i * PS) = v;
            *reinterpret_cast<uint4*>(s_in + i * PS + 8) = uint4{0u, 0u, 0u, 0u};
        }
    } else if (y0 > 0 && y0 + R < a.H && xb > 0 && xb + 64 < a.W) {
        fill(std::true_type{});
    } else {
        fill(std::false_type{});
    }
    __syncthreads();
    if (!busy || wm >= mt || xb + 16 * wc >= a.W) return;  // whole wave, after the block's only barrier
    v4f acc[CT][R];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[c][r] = v4f{0.f, 0.f, 0.f, 0.f};
    // A lane's operands of slice s: k = 32 s + 8 kg .. + 7, one tap and eight
    // channels.  A slice that crosses into the next tap does so at its middle
    // (CPAD is 16 or a multiple of 16 that 32-slices meet there), and the
    // next tap is one column on, or a row on and two columns back: three
    // lane bases serve every slice with constant offsets.
    static_assert(CPAD % 32 == 0 || CPAD % 32 == 16, "slices cross taps at their middle only");
    const int hi = kg >= 2 ? 1 : 0;
    const uint16_t* base0 = s_in + (16 * wc + n) * PS + 8 * kg;
    const uint16_t* base1 = base0 + hi * (PS - CPAD);
    const uint16_t* base2 = base0 + hi * ((kConvCols - 2) * PS - CPAD);
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int t0 = 32 * s / CPAD, t1 = (32 * s + 16) / CPAD;  // taps of the slice's halves
        const int off = ((t0 / 3) * kConvCols + t0 % 3) * PS + 32 * s - t0 * CPAD;
        const uint16_t* base = t1 == t0 || t1 >= 9 ? base0 : t1 % 3 ? base1 : base2;
        const v8bf av = __builtin_bit_cast(v8bf, wq[s % P]);
        if (s + P < SL) wq[s % P] = *reinterpret_cast<const uint4*>(wl + 32 * (s + P));
#pragma unroll
        for (int c = 0; c < CT; ++c) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // Past the last tap (the zero padding of the reduction) the
                // operands are zero.
                uint4 q = uint4{0u, 0u, 0u, 0u};
                if (t1 < 9 || !hi) q = *reinterpret_cast<const uint4*>(base + off + (r * kConvCols + 16 * c) * PS);
                acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(v8bf, q), acc[c][r], 0, 0, 0);
            }
        }
    }
    // Lane holds output channels co .. co + 3 of pixel column n of each
    // column tile: one 8-byte store per row and tile (cout is a multiple of 4).
    if constexpr (kMode == kConvOutput) {
        // Channels 0-2 the residual, 3 the predicted squared error.
        const int64_t hw = (int64_t)a.H * a.W;
        const float ob = a.bias[kg];
        float* op = kg < 3 ? a.rgb_out + (3 * b + kg) * hw : a.err_out ? a.err_out + b * hw : nullptr;
        if (!op) return;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int x = xb + 16 * wc + n, y = y0 + r;
            if (x >= a.W || y >= a.H) continue;
            const float res = acc[0][r][0] + ob;
            op[(int64_t)y * a.W + x] = kg < 3 ? (oh[r] ? oq[r] + res : oq[r]) : (oh[r] ? res : 0.f);
        }
        return;
    }
    const int co = (m0 + wm) * 16 + 4 * kg;
    if (co >= a.cout) return;
    float bias[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bias[j] = a.bias ? a.bias[co + j] : 0.f;
    const int64_t corner = (int64_t)y0 * a.W + xb;  // offsets from here fit 32 bits
    char* ob = a.out ? reinterpret_cast<char*>(a.out + (int64_t)b * a.out_bs + corner * a.out_ps) : nullptr;
    const char* mb = a.mask ? reinterpret_cast<const char*>(a.mask + (int64_t)b * a.mask_bs + corner * a.mask_ps) : nullptr;
    uint2 h[CT][R];  // the stored values
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int px = 16 * (wc + c) + n;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool in = xb + px < a.W && y0 + r < a.H;
            const uint32_t pix = (uint32_t)(r * a.W + px);
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = acc[c][r][j] + bias[j];
                if (a.relu) v[j] = fmaxf(v[j], 0.f);
            }
            if (in && mb) {
                const uint2 mk = *reinterpret_cast<const uint2*>(mb + 2u * (pix * a.mask_ps + co));
                if (!(__uint_as_float(mk.x << 16) > 0.f)) v[0] = 0.f;
                if (!(__uint_as_float(mk.x & 0xFFFF0000u) > 0.f)) v[1] = 0.f;
                if (!(__uint_as_float(mk.y << 16) > 0.f)) v[2] = 0.f;
                if (!(__uint_as_float(mk.y & 0xFFFF0000u) > 0.f)) v[3] = 0.f;
            }
            h[c][r] = uint2{pack_bf(v[0], v[1]), pack_bf(v[2], v[3])};
            if (!in) continue;
            if (a.out_f) {
                float* of = a.out_f + (int64_t)b * a.out_bs + (int64_t)co * a.H * a.W + corner;
#pragma unroll
                for (int j = 0; j < 4; ++j) (of + (int64_t)j * a.H * a.W)[pix] = v[j];
            } else {
                *reinterpret_cast<uint2*>(ob + 2u * (pix * a.out_ps + co)) = h[c][r];
            }
        }
    }
    if (!a.pool) return;
    // 2x2 mean of the stored values: rows r and r + 1 of the lane (R and the
    // block's first row are even), columns of lanes n and n ^ 1 (same kg),
    // summed in the order (x, y), (x + 1, y), (x, y + 1), (x + 1, y + 1).
    // With W and H even a pair of columns or rows is inside the image or
    // outside together.
    char* pb = reinterpret_cast<char*>(a.pool + (int64_t)b * a.pool_bs +
                                       ((int64_t)(y0 >> 1) * (a.W >> 1) + (xb >> 1)) * a.pool_ps);
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int px = 16 * (wc + c) + n;
#pragma unroll
        for (int r = 0; r < R; r += 2) {
            float q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u0 = j < 2 ? h[c][r].x : h[c][r].y, u2 = j < 2 ? h[c][r + 1].x : h[c][r + 1].y;
                const float s0 = __uint_as_float(j & 1 ? u0 & 0xFFFF0000u : u0 << 16);
                const float s2 = __uint_as_float(j & 1 ? u2 & 0xFFFF0000u : u2 << 16);
                const float s1 = __shfl_xor(s0, 1, 64), s3 = __shfl_xor(s2, 1, 64);
                q[j] = 0.25f * (((s0 + s1) + s2) + s3);
            }
            if ((n & 1) || xb + px >= a.W || y0 + r >= a.H) continue;
            const uint32_t pp = (uint32_t)((r >> 1) * (a.W >> 1) + (px >> 1));
            *reinterpret_cast<uint2*>(pb + 2u * (pp * a.pool_ps + co)) = uint2{pack_bf(q[0], q[1]), pack_bf(q[2], q[3])};
        }
    }
}

// ---------------------------------------------------------------------------
// Weight and bias gradients.  dW[co][ci][tap] = sum over pixels p of
// g[p, co] * in[p + tap offset, ci]: per tap a GEMM over pixels with both
// operands stored pixel by pixel, so both must be read transposed.  A block
// stages kWgRows x kWgCols pixels of the gradient and the same with a
// one-pixel border of 16 input channels in LDS as they lie in memory, and
// ds_read_b64_tr_b16 turns 4 pixels x 16 channels into an MFMA operand: a
// tap is another pixel address, and needs no realignment.  (Gathering the
// operands' elements one by one from memory, 42 us a layer on eight 128x128
// crops, was bound by its 2-byte loads.)  Three waves take a row of taps
// each, for all output channels (MT tiles of 16), so a wave holds 3 MT
// accumulator tiles and nothing is reduced across waves; wave 0 also takes
// the bias, a product with ones.  A block sums kWgRows x kWgCols items of
// its chunk and writes one partial; a second kernel adds the partials in a
// fixed order, so results are deterministic.  The layers' blocks go in one
// launch per MT after the whole backward pass, and all reductions in one:
// on the small crops of training a launch costs as much as its work.
// ---------------------------------------------------------------------------
constexpr int kWgRows = 4, kWgCols = 64, kWgPix = kWgRows * kWgCols;
constexpr int kWgInPix = (kWgRows + 2) * (kWgCols + 2);
constexpr int kWgThreads = 192;
constexpr int kWgChunks = 256;  // partials per layer at most

struct WgradJob {
    const uint16_t* g;  // layer output gradient, [B][H][W] pixels of g_ps elements
    int64_t g_bs;
    int g_ps, cout;
    const uint16_t* in;  // layer input from channel up_c on, in_ps elements per pixel
    int64_t in_bs;
    int in_ps, cin;
    const uint16_t* up;  // input channels [0, up_c), at half resolution (up_c a multiple of 16)
    int64_t up_bs;
    int up_ps, up_c;
    int B, H, W;
    int items_x, items_y;  // items per image row and column
    int items, per;        // over the batch; per chunk
    int chunks, nt;        // partials; 16-channel input tiles
    int first;             // first block: block first + chunk * nt + tile
    float* part;           // [chunk]: [tap][cout][16 nt], then [cout]
};
constexpr int kWgJobs = 4;
struct WgradJobs {
    WgradJob job[kWgJobs];
    int n;
};

typedef short v4s __attribute__((ext_vector_type(4)));

// Eight pixels' values of one channel for this lane (channel lane & 15,
// pixels 8 (lane >> 4) on), from LDS pixels of 16 channels starting at p:
// each group of 16 lanes reads four pixels as they lie and gets them
// transposed.
__device__ __forceinline__ v8bf tr_operand(const uint16_t* p, int lane) {
    const uint16_t* q = p + (8 * (lane >> 4) + ((lane & 15) >> 2)) * 16 + (lane & 3) * 4;
    typedef __attribute__((address_space(3))) v4s* lds_v4s;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(q));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(q + 4 * 16));
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int MT>
__global__ __launch_bounds__(kWgThreads) void k_wgrad(WgradJobs J) {
    __shared__ __attribute__((aligned(16))) uint16_t s_in[kWgInPix * 16];
    __shared__ __attribute__((aligned(16))) uint16_t s_g[MT * kWgPix * 16];
    int jb = 0;
    while (jb + 1 < J.n && (int)blockIdx.x >= J.job[jb + 1].first) ++jb;
    const WgradJob& a = J.job[jb];
    const int local = (int)blockIdx.x - a.first, chunk = local / a.nt, nt = local - chunk * a.nt;
    const int ci0 = 16 * nt;
    const int tid = threadIdx.x, lane = tid & 63, ky = tid >> 6;
    const bool from_up = ci0 < a.up_c;
    v4f acc[MT][3], accb[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        accb[m] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[m][k] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    const v8s one8 = {0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80};
    const v8bf ones = __builtin_bit_cast(v8bf, one8);
    const int i1 = min(a.items, (chunk + 1) * a.per);
    for (int item = chunk * a.per; item < i1; ++item) {
        const int ix = item % a.items_x, r = item / a.items_x, iy = r % a.items_y, b = r / a.items_y;
        const int x0 = ix * kWgCols, y0 = iy * kWgRows;
        // All of a thread's loads, then the stores (16 bytes: eight channels
        // of a pixel; zero outside the image and past the last channel).
        constexpr int kInWords = 2 * kWgInPix, kGWords = 2 * MT * kWgPix;
        constexpr int kInU = (kInWords + kWgThreads - 1) / kWgThreads, kGU = (kGWords + kWgThreads - 1) / kWgThreads;
        uint4 vi[kInU], vg[kGU];
#pragma unroll
        for (int u = 0; u < kInU; ++u) {
            const int w = tid + u * kWgThreads, c = ci0 + 8 * (w & 1), p = w >> 1;
            const int y = y0 + p / (kWgCols + 2) - 1, x = x0 + p % (kWgCols + 2) - 1;
            vi[u] = uint4{0u, 0u, 0u, 0u};
            if (w < kInWords && y >= 0 && y < a.H && x >= 0 && x < a.W && c < a.cin)
                vi[u] = *reinterpret_cast<const uint4*>(
                    from_up ? a.up + (int64_t)b * a.up_bs + ((int64_t)(y >> 1) * (a.W >> 1) + (x >> 1)) * a.up_ps + c
                            : a.in + (int64_t)b * a.in_bs + ((int64_t)y * a.W + x) * a.in_ps + (c - a.up_c));
        }
#pragma unroll
        for (int u = 0; u < kGU; ++u) {
            const int w = tid + u * kWgThreads, c = 8 * (w % (2 * MT)), p = w / (2 * MT);
            const int y = y0 + p / kWgCols, x = x0 + p % kWgCols;
            vg[u] = uint4{0u, 0u, 0u, 0u};
            if (w < kGWords && y < a.H && x < a.W && c < a.cout)
                vg[u] = *reinterpret_cast<const uint4*>(a.g + (int64_t)b * a.g_bs + ((int64_t)y * a.W + x) * a.g_ps + c);
        }
        __syncthreads();  // the previous item's operands have been read
#pragma unroll
        for (int u = 0; u < kInU; ++u) {
            const int w = tid + u * kWgThreads;
            if (w < kInWords) *reinterpret_cast<uint4*>(s_in + 8 * w) = vi[u];
        }
#pragma unroll
        for (int u = 0; u < kGU; ++u) {
            const int w = tid + u * kWgThreads, g8 = w % (2 * MT), p = w / (2 * MT);
            if (w < kGWords) *reinterpret_cast<uint4*>(s_g + ((g8 >> 1) * kWgPix + p) * 16 + 8 * (g8 & 1)) = vg[u];
        }
        __syncthreads();
        for (int row = 0; row < kWgRows; ++row) {
            if (y0 + row >= a.H) break;
#pragma unroll
            for (int sx = 0; sx < kWgCols; sx += 32) {
                if (x0 + sx >= a.W) break;
                v8bf ga[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m) ga[m] = tr_operand(s_g + (m * kWgPix + row * kWgCols + sx) * 16, lane);
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const v8bf ib = tr_operand(s_in + ((row + ky) * (kWgCols + 2) + sx + kx) * 16, lane);
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m][kx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ga[m], ib, acc[m][kx], 0, 0, 0);
                }
                if (ky == 0 && nt == 0) {
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ga[m], ones, accb[m], 0, 0, 0);
                }
            }
        }
    }
    // Lane holds channels co .. co + 3 of input channel ci.
    const int cinp = 16 * a.nt, n = lane & 15;
    float* pb = a.part + (size_t)chunk * (9 * a.cout * cinp + a.cout);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int co = 16 * m + 4 * (lane >> 4) + j;
            if (co >= a.cout) continue;
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) pb[(size_t)((3 * ky + kx) * a.cout + co) * cinp + ci0 + n] = acc[m][kx][j];
            if (ky == 0 && nt == 0 && n == 0) pb[(size_t)9 * a.cout * cinp + co] = accb[m][j];
        }
    }
}

// grad (each layer's W[cout][cin][9] then b[cout]) from the partials in a
// fixed order: block of 64 outputs; wave q adds the q-th quarter of the
// chunks in chunk order, then ((q0 + q1) + (q2 + q3)).
struct WgradSum {
    const float* part;
    float* grad;
    int chunks, cout, cin, cinp, first;  // first: the layer's first block
};
struct WgradSums {
    WgradSum job[kLayers];
    int n;
};

__global__ __launch_bounds__(256) void k_wgrad_reduce(WgradSums J) {
    __shared__ float s_q[4][64];
    int jb = 0;
    while (jb + 1 < J.n && (int)blockIdx.x >= J.job[jb + 1].first) ++jb;
    const WgradSum& a = J.job[jb];
    const int W = 9 * a.cout * a.cinp, n = W + a.cout;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = ((int)blockIdx.x - a.first) * 64 + lane;
    const int per = (a.chunks + 3) / 4, c0 = q * per, c1 = min(a.chunks, c0 + per);
    float s = 0.f;
    if (i < n) {
        const float* p = a.part + i;
        int c = c0;
        for (; c + 8 <= c1; c += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(c + u) * n];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; c < c1; ++c) s += p[(size_t)c * n];
    }
    s_q[q][lane] = s;
    __syncthreads();
    if (q != 0 || i >= n) return;
    const float v = (s_q[0][lane] + s_q[1][lane]) + (s_q[2][lane] + s_q[3][lane]);
    if (i >= W) {
        a.grad[a.cout * a.cin * 9 + (i - W)] = v;
        return;
    }
    const int t = i / (a.cout * a.cinp), rem = i - t * (a.cout * a.cinp), co = rem / a.cinp, ci = rem - co * a.cinp;
    if (ci < a.cin) a.grad[(co * a.cin + ci) * 9 + t] = v;
}

__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const float s = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return s;
}

// ---------------------------------------------------------------------------
// Weight packing (fp32 master -> bf16 GEMM operands), pooling, upsampling,
// gradient merges, input assembly, output and loss.
// ---------------------------------------------------------------------------
// Column k = tap * cpad + c of a packed row of kpad columns (zero from
// 9 cpad on).  Forward: row = output channel, c = input channel,
// W[row][c][tap].  Transposed (input gradient): row = input channel, c =
// output channel, W[c][row][8 - tap] (the kernel flipped).  One launch
// packs every job: job j covers elements [start[j], start[j + 1]) of the
// grid.
struct PackJob {
    const float* w;
    uint16_t* out;
    int cin, cout, transpose, cpad, kpad;
    int spread;  // output channel c in row 4 c (kConvOutput), the other rows zero
};
struct PackJobs {
    PackJob job[2 * kLayers];
    int start[2 * kLayers + 1];
    int n;
};

__global__ __launch_bounds__(256) void k_pack(PackJobs J) {
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= J.start[J.n]) return;
    int jb = 0;
    while (g >= J.start[jb + 1]) ++jb;
    const PackJob& P = J.job[jb];
    const float* __restrict__ w = P.w;
    const int cin = P.cin, cout = P.cout, transpose = P.transpose, cpad = P.cpad, kpad = P.kpad;
    const int i = g - J.start[jb];
    int m = i / kpad;
    const int k = i - m * kpad;
    if (P.spread) m = m % 4 ? cout : m / 4;
    const int t = k / cpad, c = k - t * cpad;
    float v = 0.f;
    if (t < 9) {
        if (!transpose) {
            if (m < cout && c < cin) v = w[(m * cin + c) * 9 + t];
        } else {
            if (m < cin && c < cout) v = w[(c * cin + m) * 9 + (8 - t)];
        }
    }
    P.out[i] = f2bf(v);
}

// The channel kernels below take one pixel's eight channels (one 16-byte
// word) per thread: grid over B * pixels * C / 8 (C a multiple of 8),
// channel group fastest.
__device__ __forceinline__ void unpack8(uint4 q, float* f) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = bf2f((uint16_t)(w[k] & 0xFFFFu));
        f[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16));
    }
}
__device__ __forceinline__ uint4 pack8(const float* f) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = (uint32_t)f2bf(f[2 * k]) | ((uint32_t)f2bf(f[2 * k + 1]) << 16);
    return uint4{w[0], w[1], w[2], w[3]};
}
__device__ __forceinline__ uint4 ld8(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void st8(uint16_t* p, uint4 v) { *reinterpret_cast<uint4*>(p) = v; }

// Index of this thread's (image, pixel, channel group) over n pixels per
// image; false past the end.
__device__ __forceinline__ bool item(int64_t B, int64_t n, int C, int64_t& b, int64_t& p, int& c) {
    const int G = C >> 3;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= B * n * G) return false;
    const int64_t bp = i / G;
    c = (int)(i - bp * G) * 8;
    b = bp / n;
    p = bp - b * n;
    return true;
}

// Gradient of the upsample: sum of each 2x2 block of the first C channels
// of g (g_bs, g_ps), masked by the activation act [B][H/2][W/2][C] (ReLU
// derivative), into out of that layout.
__global__ __launch_bounds__(256) void k_up_grad(const uint16_t* __restrict__ g, int64_t g_bs, int g_ps, int B, int C,
                                                 int H, int W, const uint16_t* __restrict__ act,
                                                 uint16_t* __restrict__ out) {
    const int h = H / 2, w = W / 2;
    int64_t b, p;
    int c;
    if (!item(B, (int64_t)h * w, C, b, p, c)) return;
    const int Y = (int)(p / w), X = (int)(p - (int64_t)Y * w);
    const uint16_t* q = g + b * g_bs + ((int64_t)(2 * Y) * W + 2 * X) * g_ps + c;
    float f0[8], f1[8], f2[8], f3[8], a[8], o[8];
    unpack8(ld8(q), f0);
    unpack8(ld8(q + g_ps), f1);
    unpack8(ld8(q + (int64_t)W * g_ps), f2);
    unpack8(ld8(q + (int64_t)(W + 1) * g_ps), f3);
    const int64_t oi = (b * h * w + p) * C + c;
    unpack8(ld8(act + oi), a);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = a[k] > 0.f ? ((f0[k] + f1[k]) + f2[k]) + f3[k] : 0.f;
    st8(out + oi, pack8(o));
}

// Gradient reaching an encoder activation from its skip connection (C
// channels of skip, at skip_bs, skip_ps) and from the pool below it (pg,
// [B][H/2][W/2][C]), masked by the activation (act_bs, act_ps), into out
// [B][H][W][C].
__global__ __launch_bounds__(256) void k_merge(const uint16_t* __restrict__ skip, int64_t skip_bs, int skip_ps,
                                               const uint16_t* __restrict__ pg, const uint16_t* __restrict__ act,
                                               int64_t act_bs, int act_ps, int B, int C, int H, int W,
                                               uint16_t* __restrict__ out) {
    int64_t b, p;
    int c;
    if (!item(B, (int64_t)H * W, C, b, p, c)) return;
    const int y = (int)(p / W), x = (int)(p - (int64_t)y * W);
    float sk[8], pl[8], a[8], o[8];
    unpack8(ld8(skip + b * skip_bs + p * skip_ps + c), sk);
    unpack8(ld8(pg + (b * (H / 2) * (W / 2) + (int64_t)(y >> 1) * (W / 2) + (x >> 1)) * C + c), pl);
    unpack8(ld8(act + b * act_bs + p * act_ps + c), a);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = a[k] > 0.f ? sk[k] + 0.25f * pl[k] : 0.f;
    st8(out + (b * H * W + p) * C + c, pack8(o));
}

// Network input x0 [B][H][W][8] (training: the weight gradient reads it).
__global__ __launch_bounds__(256) void k_input(const float* __restrict__ rgb, const float* __restrict__ z,
                                               const uint8_t* __restrict__ hole, int B, int HW,
                                               uint16_t* __restrict__ x0) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)B * HW) return;
    const int64_t b = i / HW, p = i - b * HW;
    const float* q = rgb + b * 3 * HW + p;
    st8(x0 + i * 8, input_pixel(q[0], q[HW], q[2 * (int64_t)HW], z[i], hole[i] != 0));
}

// Per-block hole counts.
__global__ __launch_bounds__(256) void k_count(const uint8_t* __restrict__ hole, int64_t n, float* __restrict__ part) {
    __shared__ float red[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float c = (i < n && hole[i]) ? 1.f : 0.f;
    const float s = block_sum(c, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Predicted error of each image over its holes, first step: block b of
// image y sums err and counts holes over its grid-stride pixels, into
// part[2 (y * kErrParts + b) + {0, 1}].
constexpr int kErrParts = 256;
__global__ __launch_bounds__(256) void k_err_part(const float* __restrict__ err, const uint8_t* __restrict__ hole,
                                                  int64_t HW, float* __restrict__ part) {
    __shared__ float red[4];
    const int64_t img = blockIdx.y;
    float e = 0.f, c = 0.f;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < HW; p += (int64_t)kErrParts * 256) {
        if (hole[img * HW + p]) {
            e += err[img * HW + p];
            c += 1.f;
        }
    }
    e = block_sum(e, red);
    __syncthreads();
    c = block_sum(c, red);
    if (threadIdx.x == 0) {
        part[2 * (img * kErrParts + blockIdx.x)] = e;
        part[2 * (img * kErrParts + blockIdx.x) + 1] = c;
    }
}

// Second step, one block per image: out[y] = sum e / max(1, holes).
__global__ __launch_bounds__(256) void k_err_mean(const float* __restrict__ part, float* __restrict__ out) {
    __shared__ float red[4];
    const int64_t img = blockIdx.x;
    const float* q = part + 2 * img * kErrParts;
    float e = block_sum(q[2 * threadIdx.x], red);
    __syncthreads();
    const float c = block_sum(q[2 * threadIdx.x + 1], red);
    if (threadIdx.x == 0) out[img] = e / fmaxf(c, 1.f);
}

// One block: out[0] = scale * sum of part[0, n) (fixed order per thread,
// then the block tree).
__global__ __launch_bounds__(256) void k_sum(const float* __restrict__ part, int n, const float* __restrict__ div,
                                             float* __restrict__ out) {
    __shared__ float red[4];
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    s = block_sum(s, red);
    if (threadIdx.x == 0) out[0] = div ? s / (3.f * fmaxf(div[0], 1.f)) : s;
}

// Loss terms per hole pixel: sum over channels of (pred - target)^2 plus
// 3 (e - s)^2, s the pixel's mean squared error (held constant); per-block
// partial sums (k_sum divides by 3 holes).  Gradient with respect to the
// output layer (bf16 [B][H][W][8], slots 4-7 zero): 2 d_c / (3 N) for the
// residual, 2 (e - s) / N for e.
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ rgb, const uint8_t* __restrict__ hole,
                                              const float* __restrict__ r, const float* __restrict__ target,
                                              const float* __restrict__ n_hole, int B, int HW,
                                              float* __restrict__ rgb_out, uint16_t* __restrict__ g_r,
                                              float* __restrict__ part) {
    __shared__ float red[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float e = 0.f;
    if (i < (int64_t)B * HW) {
        const int64_t b = i / HW, p = i - b * HW;
        const bool h = hole[i] != 0;
        const float nh = fmaxf(n_hole[0], 1.f);
        const float* rb = r + b * 4 * HW + p;
        float d[3], s2 = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int64_t q = (b * 3 + c) * HW + p;
            const float pred = h ? rgb[q] + rb[(int64_t)c * HW] : rgb[q];
            d[c] = h ? pred - target[q] : 0.f;
            s2 += d[c] * d[c];
            if (rgb_out) rgb_out[q] = pred;
        }
        const float de = h ? rb[3 * (int64_t)HW] - s2 / 3.f : 0.f;
        float gr[8];
#pragma unroll
        for (int c = 0; c < 3; ++c) gr[c] = 2.f * d[c] / (3.f * nh);
        gr[3] = 2.f * de / nh;
        gr[4] = gr[5] = gr[6] = gr[7] = 0.f;
        st8(g_r + i * 8, pack8(gr));
        e = s2 + 3.f * de * de;
    }
    const float sum = block_sum(e, red);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ w, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, int64_t n, float lr,
                                              float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---------------------------------------------------------------------------
// Host side: parameter offsets, workspace layout, launch sequences.
// ---------------------------------------------------------------------------
int64_t param_offset(int l) {
    int64_t o = 0;
    for (int i = 0; i < l; ++i) o += (int64_t)kNet[i].cout * kNet[i].cin * 9 + kNet[i].cout;
    return o;
}

struct Layout {
    size_t off = 0;
    size_t take(size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    }
};

struct Bufs {
    uint16_t *x0, *e1a, *e1b, *p1, *e2a, *e2b, *p2, *e3a, *e3b, *d2, *d1;
    float* r;
    uint16_t* wf[kLayers];
    uint16_t* wb[kLayers];
    // training
    uint16_t *g_r, *g_d1, *g_cat1, *g_d2, *g_cat2, *g_e3b, *g_e3a, *g_p2, *g_e2b, *g_e2a, *g_p1, *g_e1b, *g_e1a;
    float *cnt_part, *loss_part, *n_hole;
    float* part[kLayers];
    size_t bytes;
};

// Level (0: H x W, 1: halved, 2: quartered) of each layer's output.
constexpr int kLevel[kLayers] = {0, 0, 1, 1, 2, 2, 1, 0, 0};

// The weight gradient's items and chunks of layer l.
void wgrad_split(int l, int B, int H, int W, WgradJob& a) {
    a.B = B;
    a.H = H >> kLevel[l];
    a.W = W >> kLevel[l];
    a.cin = kNet[l].cin;
    a.cout = kNet[l].cout;
    a.nt = pad16(a.cin) / 16;
    a.items_x = (a.W + kWgCols - 1) / kWgCols;
    a.items_y = (a.H + kWgRows - 1) / kWgRows;
    a.items = B * a.items_y * a.items_x;  // at most 1000 * 2048 * 128
    a.per = (a.items + kWgChunks - 1) / kWgChunks;
    a.chunks = (a.items + a.per - 1) / a.per;
}

Bufs layout(int B, int H, int W, bool train, char* base) {
    Layout L;
    Bufs f{};
    const size_t h1 = (size_t)H * W, h2 = h1 / 4, h3 = h1 / 16;
    auto bf = [&](size_t elems) { return (uint16_t*)(base + L.take(elems * 2)); };
    auto fl = [&](size_t elems) { return (float*)(base + L.take(elems * 4)); };
    if (train) f.x0 = bf(B * 8 * h1);
    f.e1a = bf(B * 16 * h1);
    f.e1b = bf(B * 16 * h1);
    f.p1 = bf(B * 16 * h2);
    f.e2a = bf(B * 32 * h2);
    f.e2b = bf(B * 32 * h2);
    f.p2 = bf(B * 32 * h3);
    f.e3a = bf(B * 64 * h3);
    f.e3b = bf(B * 64 * h3);
    f.d2 = bf(B * 32 * h2);
    f.d1 = bf(B * 16 * h1);
    if (train) f.r = fl(B * 4 * h1);
    for (int l = 0; l < kLayers; ++l) {
        f.wf[l] = bf((size_t)pad16(kNet[l].cout) * pad32(9 * pad16(kNet[l].cin)));
        f.wb[l] = bf((size_t)pad16(kNet[l].cin) * pad32(9 * pad16(kNet[l].cout)));
    }
    f.cnt_part = fl((B * h1 + 255) / 256);
    f.loss_part = fl((B * h1 + 255) / 256);
    f.n_hole = fl(1);
    if (train) {
        f.g_r = bf(B * 8 * h1);
        f.g_d1 = bf(B * 16 * h1);
        f.g_cat1 = bf(B * 48 * h1);
        f.g_d2 = bf(B * 32 * h2);
        f.g_cat2 = bf(B * 96 * h2);
        f.g_e3b = bf(B * 64 * h3);
        f.g_e3a = bf(B * 64 * h3);
        f.g_p2 = bf(B * 32 * h3);
        f.g_e2b = bf(B * 32 * h2);
        f.g_e2a = bf(B * 32 * h2);
        f.g_p1 = bf(B * 16 * h2);
        f.g_e1b = bf(B * 16 * h1);
        f.g_e1a = bf(B * 16 * h1);
        for (int l = 0; l < kLayers; ++l) {
            WgradJob a{};
            wgrad_split(l, B, H, W, a);
            f.part[l] = fl((size_t)a.chunks * (9 * a.cout * 16 * a.nt + a.cout));
        }
    }
    f.bytes = L.off;
    return f;
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

// The staged channel counts the convolution kernel is built for.
constexpr bool conv_cpad_ok(int cpad) { return cpad == 16 || cpad == 32 || cpad == 48 || cpad == 64 || cpad == 96; }
constexpr bool net_cpads_ok() {
    for (int l = 0; l < kLayers; ++l)
        if (!conv_cpad_ok(pad16(kNet[l].cin)) || !conv_cpad_ok(pad16(kNet[l].cout)) ||
            conv_has_up(pad16(kNet[l].cin)) != (l == D2 || l == D1) || conv_has_up(pad16(kNet[l].cout)) ||
            (kNet[l].cin > 16 && kNet[l].cin % 16) || (kNet[l].cout > 16 && kNet[l].cout % 16))
            return false;
    return true;
}
static_assert(net_cpads_ok(), "every layer's input and output width needs a convolution instance");

template <int CPAD, int MT, int R>
void launch_conv(hipStream_t s, int B, const ConvArgs& a) {
    const int groups = (a.cout + 16 * MT - 1) / (16 * MT);
    const dim3 g((a.W + 63) / 64, (a.H + R - 1) / R, B * groups), wg(256);
    if constexpr (CPAD == 16 && MT == 1) {  // the network's first and last layer
        if (a.rgb_out) {
            hipLaunchKernelGGL((k_conv3x3<CPAD, MT, R, kConvOutput>), g, wg, conv_lds_bytes(CPAD, R), s, a);
            return;
        }
        if (a.rgb) {
            hipLaunchKernelGGL((k_conv3x3<CPAD, MT, R, kConvInput>), g, wg, conv_lds_bytes(CPAD, R), s, a);
            return;
        }
    }
    hipLaunchKernelGGL((k_conv3x3<CPAD, MT, R>), g, wg, conv_lds_bytes(CPAD, R), s, a);
}

// mt <= 2 for the tall shapes (more tiles would not fit in registers).
template <int CPAD>
constexpr bool tall_rows(int r) { return r == 8 || (CPAD > 64 && r == 4); }

template <int CPAD, int R>
void launch_conv(hipStream_t s, int B, int mt, const ConvArgs& a) {
    if constexpr (tall_rows<CPAD>(R)) {
        if (mt == 1)
            launch_conv<CPAD, 1, R>(s, B, a);
        else
            launch_conv<CPAD, 2, R>(s, B, a);
    } else {
        switch (mt) {
            case 1: launch_conv<CPAD, 1, R>(s, B, a); break;
            case 2: launch_conv<CPAD, 2, R>(s, B, a); break;
            case 3: launch_conv<CPAD, 3, R>(s, B, a); break;
            default: launch_conv<CPAD, 4, R>(s, B, a); break;
        }
    }
}

// Block shape: four output rows per block where that still leaves at least
// six blocks per CU (they share the two halo rows and each weight operand),
// else two; then fewer output tiles per block until there are at least two
// blocks per CU, since the coarse levels have few pixels (at 200x150, two
// tiles over 600 blocks beat one tile over 1200: 11.6 against 16.7 us for
// the 64-channel layer).  bgs_repair_set_block_shape may fix either choice
// (0: automatic), and may ask for eight rows (inputs of up to 64 channels)
// or four rows of 96 channels, which take at most two output tiles.
std::atomic<int> g_rows{0}, g_tiles{0};

template <int CPAD>
void launch_conv(hipStream_t s, int B, const ConvArgs& a) {
    const int tiles = (a.cout + 15) / 16;
    auto nblk = [&](int r, int mt) {
        return (int64_t)((a.W + 63) / 64) * ((a.H + r - 1) / r) * B * ((tiles + mt - 1) / mt);
    };
    const int fr = g_rows.load(), ft = g_tiles.load();
    int mt = std::min(4, tiles);
    // Largest row count offered for this width (a workgroup may take up to
    // 160 KB of LDS): 8 rows up to 64 staged channels (95 KB at 64), 4 rows
    // of 96 (85 KB).
    constexpr int kMaxRows = CPAD <= 64 ? 8 : 4;
    // Automatic: 96 staged channels keep two rows (four take 85 KB of LDS,
    // one block per CU, and measured slower: 211 against 194 us at
    // 1032x1104); taller blocks than four rows measured no better.
    int r = std::min(kMaxRows, fr ? fr : (CPAD <= 64 && nblk(4, mt) >= 6 * 256) ? 4 : 2);
    if (ft)
        mt = std::min(ft, tiles);
    else
        while (mt > 1 && nblk(r, mt) < 2 * 256) mt = (mt + 1) / 2;
    if (mt > 2 && tall_rows<CPAD>(r)) r = r == 8 && CPAD <= 64 ? 4 : 2;
    if (r == 8)
        launch_conv<CPAD, (kMaxRows >= 8 ? 8 : 2)>(s, B, mt, a);
    else if (r == 4)
        launch_conv<CPAD, (kMaxRows >= 4 ? 4 : 2)>(s, B, mt, a);
    else
        launch_conv<CPAD, 2>(s, B, mt, a);
}

// A bf16 activation or gradient tensor [B][H][W] of pixels holding ps
// elements (bs per image), from channel 0 of a slice.
struct View {
    uint16_t* p;
    int64_t bs;
    int ps;
    View at(int channel) const { return View{p + channel, bs, ps}; }
};
const View kNone{nullptr, 0, 0};

// up (optional, with up_c): the half-resolution source of the first up_c
// input channels, read through the nearest 2x upsample.  out_f (fp32
// planes) replaces out when set.
// images (first and last layer of an inference pass): see ConvArgs.
struct Images {
    const float *rgb, *z;
    const uint8_t* hole;
    float *rgb_out, *err_out;
};
void conv(hipStream_t s, int B, int H, int W, int l, bool transpose, const Bufs& f, View in, const float* params,
          View out, float* out_f, View mask, View up = kNone, int up_c = 0, View pool = kNone, Images im = Images{}) {
    ConvArgs a{};
    a.rgb = im.rgb;
    a.z = im.z;
    a.hole = im.hole;
    a.rgb_out = im.rgb_out;
    a.err_out = im.err_out;
    a.in = in.p;
    a.in_bs = in.bs;
    a.in_ps = in.ps;
    a.cin = transpose ? kNet[l].cout : kNet[l].cin;
    a.up = up.p;
    a.up_bs = up.bs;
    a.up_ps = up.ps;
    a.up_c = up.p ? up_c : 0;
    a.cout = transpose ? kNet[l].cin : kNet[l].cout;
    a.w = transpose ? f.wb[l] : f.wf[l];
    const int cpad = pad16(a.cin);
    a.kpad = pad32(9 * cpad);
    a.bias = transpose ? nullptr : params + param_offset(l) + (int64_t)kNet[l].cout * kNet[l].cin * 9;
    a.out = out.p;
    a.out_bs = out_f ? (int64_t)a.cout * H * W : out.bs;
    a.out_ps = out.ps;
    a.out_f = out_f;
    a.mask = mask.p;
    a.mask_bs = mask.bs;
    a.mask_ps = mask.ps;
    a.pool = pool.p;
    a.pool_bs = pool.bs;
    a.pool_ps = pool.ps;
    a.relu = transpose ? 0 : kNet[l].relu;
    a.H = H;
    a.W = W;
    switch (cpad) {
        case 16: launch_conv<16>(s, B, a); break;
        case 32: launch_conv<32>(s, B, a); break;
        case 48: launch_conv<48>(s, B, a); break;
        case 64: launch_conv<64>(s, B, a); break;
        default: launch_conv<96>(s, B, a); break;  // the only other width (static_assert above)
    }
}

// The tensors of one pass, as views.
struct Net {
    View x0, e1a, e1b, p1, e2a, e2b, p2, e3a, e3b, d2, d1;
    View g_r, g_d1, g_cat1, g_d2, g_cat2, g_e3b, g_e3a, g_p2, g_e2b, g_e2a, g_p1, g_e1b, g_e1a;
};

Net views(const Bufs& f, int H, int W) {
    const int64_t h1 = (int64_t)H * W, h2 = h1 / 4, h3 = h1 / 16;
    auto v = [](uint16_t* p, int c, int64_t hw) { return View{p, c * hw, c}; };
    Net n;
    n.x0 = v(f.x0, 8, h1);
    n.e1a = v(f.e1a, 16, h1);
    n.e1b = v(f.e1b, 16, h1);
    n.p1 = v(f.p1, 16, h2);
    n.e2a = v(f.e2a, 32, h2);
    n.e2b = v(f.e2b, 32, h2);
    n.p2 = v(f.p2, 32, h3);
    n.e3a = v(f.e3a, 64, h3);
    n.e3b = v(f.e3b, 64, h3);
    n.d2 = v(f.d2, 32, h2);
    n.d1 = v(f.d1, 16, h1);
    n.g_r = v(f.g_r, 8, h1);
    n.g_d1 = v(f.g_d1, 16, h1);
    n.g_cat1 = v(f.g_cat1, 48, h1);
    n.g_d2 = v(f.g_d2, 32, h2);
    n.g_cat2 = v(f.g_cat2, 96, h2);
    n.g_e3b = v(f.g_e3b, 64, h3);
    n.g_e3a = v(f.g_e3a, 64, h3);
    n.g_p2 = v(f.g_p2, 32, h3);
    n.g_e2b = v(f.g_e2b, 32, h2);
    n.g_e2a = v(f.g_e2a, 32, h2);
    n.g_p1 = v(f.g_p1, 16, h2);
    n.g_e1b = v(f.g_e1b, 16, h1);
    n.g_e1a = v(f.g_e1a, 16, h1);
    return n;
}

inline unsigned chan_blocks(int B, int64_t pixels, int C) { return blocks((int64_t)B * pixels * (C / 8)); }

// Training keeps the network's input and residual; inference (rgb_out set)
// takes the images straight into the first layer and out of the last.
void forward(hipStream_t s, int B, int H, int W, const float* params, const float* rgb, const float* z,
             const uint8_t* hole, const Bufs& f, bool train, float* rgb_out = nullptr, float* err_out = nullptr) {
    // Forward weights always; the transposed ones only for the input
    // gradient of training.
    PackJobs J{};
    J.start[0] = 0;
    for (int t = 0; t < (train ? 2 : 1); ++t)
        for (int l = 0; l < kLayers; ++l) {
            const int ci = kNet[l].cin, co = kNet[l].cout;
            PackJob& P = J.job[J.n];
            P.w = params + param_offset(l);
            P.out = t ? f.wb[l] : f.wf[l];
            P.cin = ci;
            P.cout = co;
            P.transpose = t;
            P.cpad = pad16(t ? co : ci);
            P.kpad = pad32(9 * P.cpad);
            P.spread = !train && l == OUT;
            J.start[J.n + 1] = J.start[J.n] + pad16(t ? ci : co) * P.kpad;
            ++J.n;
        }
    hipLaunchKernelGGL(k_pack, dim3(blocks(J.start[J.n])), dim3(256), 0, s, J);
    const Net n = views(f, H, W);
    const int64_t h1 = (int64_t)H * W;
    const int H2 = H / 2, W2 = W / 2, H3 = H / 4, W3 = W / 4;
    if (train)
        hipLaunchKernelGGL(k_input, dim3(blocks(B * h1)), dim3(256), 0, s, rgb, z, hole, B, (int)h1, f.x0);
    const Images none{}, first{rgb, z, hole, nullptr, nullptr}, last{rgb, nullptr, hole, rgb_out, err_out};
    conv(s, B, H, W, E1A, false, f, n.x0, params, n.e1a, nullptr, kNone, kNone, 0, kNone, train ? none : first);
    // The encoders' second convolutions also store the pooled output.
    conv(s, B, H, W, E1B, false, f, n.e1a, params, n.e1b, nullptr, kNone, kNone, 0, n.p1);
    conv(s, B, H2, W2, E2A, false, f, n.p1, params, n.e2a, nullptr, kNone);
    conv(s, B, H2, W2, E2B, false, f, n.e2a, params, n.e2b, nullptr, kNone, kNone, 0, n.p2);
    conv(s, B, H3, W3, E3A, false, f, n.p2, params, n.e3a, nullptr, kNone);
    conv(s, B, H3, W3, E3B, false, f, n.e3a, params, n.e3b, nullptr, kNone);
    // The decoders read their upsampled channels straight from the coarser
    // level.
    conv(s, B, H2, W2, D2, false, f, n.e2b, params, n.d2, nullptr, kNone, n.e3b, 64);
    conv(s, B, H, W, D1, false, f, n.e1b, params, n.d1, nullptr, kNone, n.d2, 32);
    conv(s, B, H, W, OUT, false, f, n.d1, params, kNone, train ? f.r : nullptr, kNone, kNone, 0, kNone, train ? none : last);
}

// Input gradients layer by layer, then all weight gradients (every layer's
// output gradient and input stay in the workspace).
void backward(hipStream_t s, int B, int H, int W, const float* params, const Bufs& f, float* grad) {
    const Net n = views(f, H, W);
    const int64_t h1 = (int64_t)H * W, h2 = h1 / 4;
    const int H2 = H / 2, W2 = W / 2, H3 = H / 4, W3 = W / 4;
    conv(s, B, H, W, OUT, true, f, n.g_r, params, n.g_d1, nullptr, n.d1);
    conv(s, B, H, W, D1, true, f, n.g_d1, params, n.g_cat1, nullptr, kNone);
    hipLaunchKernelGGL(k_up_grad, dim3(chan_blocks(B, h2, 32)), dim3(256), 0, s, n.g_cat1.p, n.g_cat1.bs, n.g_cat1.ps,
                       B, 32, H, W, f.d2, f.g_d2);
    conv(s, B, H2, W2, D2, true, f, n.g_d2, params, n.g_cat2, nullptr, kNone);
    hipLaunchKernelGGL(k_up_grad, dim3(chan_blocks(B, h2 / 4, 64)), dim3(256), 0, s, n.g_cat2.p, n.g_cat2.bs,
                       n.g_cat2.ps, B, 64, H2, W2, f.e3b, f.g_e3b);
    conv(s, B, H3, W3, E3B, true, f, n.g_e3b, params, n.g_e3a, nullptr, n.e3a);
    conv(s, B, H3, W3, E3A, true, f, n.g_e3a, params, n.g_p2, nullptr, kNone);
    const View sk2 = n.g_cat2.at(64), sk1 = n.g_cat1.at(32);
    hipLaunchKernelGGL(k_merge, dim3(chan_blocks(B, h2, 32)), dim3(256), 0, s, sk2.p, sk2.bs, sk2.ps, f.g_p2, n.e2b.p,
                       n.e2b.bs, n.e2b.ps, B, 32, H2, W2, f.g_e2b);
    conv(s, B, H2, W2, E2B, true, f, n.g_e2b, params, n.g_e2a, nullptr, n.e2a);
    conv(s, B, H2, W2, E2A, true, f, n.g_e2a, params, n.g_p1, nullptr, kNone);
    hipLaunchKernelGGL(k_merge, dim3(chan_blocks(B, h1, 16)), dim3(256), 0, s, sk1.p, sk1.bs, sk1.ps, f.g_p1, n.e1b.p,
                       n.e1b.bs, n.e1b.ps, B, 16, H, W, f.g_e1b);
    conv(s, B, H, W, E1B, true, f, n.g_e1b, params, n.g_e1a, nullptr, n.e1a);
    // Per layer: output gradient, input (its own channels), and the
    // upsampled source of the decoders' first channels.
    struct Src {
        View g, in, up;
        int up_c;
    };
    const Src src[kLayers] = {{n.g_e1a, n.x0, kNone, 0}, {n.g_e1b, n.e1a, kNone, 0}, {n.g_e2a, n.p1, kNone, 0},
                              {n.g_e2b, n.e2a, kNone, 0}, {n.g_e3a, n.p2, kNone, 0}, {n.g_e3b, n.e3a, kNone, 0},
                              {n.g_d2, n.e2b, n.e3b, 64}, {n.g_d1, n.e1b, n.d2, 32}, {n.g_r, n.d1, kNone, 0}};
    WgradSums S{};
    int sum_blocks = 0;
    for (int mt = 1; mt <= 4; mt *= 2) {
        WgradJobs J{};
        int nblk = 0;
        for (int l = 0; l < kLayers; ++l) {
            if (pad16(kNet[l].cout) != 16 * mt) continue;
            WgradJob& a = J.job[J.n++];
            wgrad_split(l, B, H, W, a);
            a.g = src[l].g.p;
            a.g_bs = src[l].g.bs;
            a.g_ps = src[l].g.ps;
            a.in = src[l].in.p;
            a.in_bs = src[l].in.bs;
            a.in_ps = src[l].in.ps;
            a.up = src[l].up.p;
            a.up_bs = src[l].up.bs;
            a.up_ps = src[l].up.ps;
            a.up_c = src[l].up_c;
            a.part = f.part[l];
            a.first = nblk;
            nblk += a.chunks * a.nt;
            WgradSum& q = S.job[S.n++];
            q.part = f.part[l];
            q.grad = grad + param_offset(l);
            q.chunks = a.chunks;
            q.cout = a.cout;
            q.cin = a.cin;
            q.cinp = 16 * a.nt;
            q.first = sum_blocks;
            sum_blocks += (9 * a.cout * q.cinp + a.cout + 63) / 64;
        }
        const dim3 g(nblk), b(kWgThreads);
        if (mt == 1)
            hipLaunchKernelGGL(k_wgrad<1>, g, b, 0, s, J);
        else if (mt == 2)
            hipLaunchKernelGGL(k_wgrad<2>, g, b, 0, s, J);
        else
            hipLaunchKernelGGL(k_wgrad<4>, g, b, 0, s, J);
    }
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(sum_blocks), dim3(256), 0, s, S);
}

constexpr bool wgrad_jobs_ok() {
    int n[5] = {};
    for (int l = 0; l < kLayers; ++l) {
        const int mt = pad16(kNet[l].cout) / 16;
        if (mt != 1 && mt != 2 && mt != 4) return false;
        if (++n[mt] > kWgJobs) return false;
    }
    return true;
}
static_assert(wgrad_jobs_ok(), "every layer has a weight gradient instance and a place in its launch");

bool sizes_ok(int B, int H, int W) { return B >= 1 && B <= 1000 && H >= 4 && W >= 4 && H % 4 == 0 && W % 4 == 0 && H <= 8192 && W <= 8192; }

int32_t launched() { return hipGetLastError() == hipSuccess ? BGS_OK : BGS_ERR_HIP; }

}  // namespace

extern "C" {

BGS_API int32_t bgs_repair_num_params(int64_t* n) {
    if (!n) return BGS_ERR_INVALID_ARG;
    *n = param_offset(kLayers);
    return BGS_OK;
}

BGS_API int32_t bgs_repair_workspace_size(int32_t batch, int32_t height, int32_t width, int32_t train, size_t* bytes) {
    if (!bytes || !sizes_ok(batch, height, width) || (train != 0 && train != 1)) return BGS_ERR_INVALID_ARG;
    *bytes = layout(batch, height, width, train != 0, nullptr).bytes;
    return BGS_OK;
}

BGS_API int32_t bgs_repair_forward(const float* params, int32_t batch, int32_t height, int32_t width,
                                   const float* rgb, const float* z, const uint8_t* hole, float* rgb_out,
                                   float* err_out, void* ws, size_t ws_bytes, void* hip_stream) {
    if (!params || !rgb || !z || !hole || !rgb_out || !ws || !sizes_ok(batch, height, width))
        return BGS_ERR_INVALID_ARG;
    const Bufs f = layout(batch, height, width, false, (char*)ws);
    if (ws_bytes < f.bytes) return BGS_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    (void)hipGetLastError();
    forward(s, batch, height, width, params, rgb, z, hole, f, false, rgb_out, err_out);
    return launched();
}

BGS_API int32_t bgs_repair_hole_error(const float* err, const uint8_t* hole, int32_t batch, int32_t height,
                                      int32_t width, float* out, float* scratch, void* hip_stream) {
    static_assert(kErrParts == 256, "one part per thread of the second step");
    if (!err || !hole || !out || !scratch || batch < 1 || batch > 1000 || height < 1 || width < 1 || height > 16384 ||
        width > 16384)
        return BGS_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_err_part, dim3(kErrParts, batch), dim3(256), 0, s, err, hole, (int64_t)height * width,
                       scratch);
    hipLaunchKernelGGL(k_err_mean, dim3(batch), dim3(256), 0, s, (const float*)scratch, out);
    return launched();
}

BGS_API int32_t bgs_repair_grad(const float* params, int32_t batch, int32_t height, int32_t width, const float* rgb,
                                const float* z, const uint8_t* hole, const float* target, float* grad, float* loss,
                                float* rgb_out, void* ws, size_t ws_bytes, void* hip_stream) {
    if (!params || !rgb || !z || !hole || !target || !grad || !loss || !ws || !sizes_ok(batch, height, width))
        return BGS_ERR_INVALID_ARG;
    const Bufs f = layout(batch, height, width, true, (char*)ws);
    if (ws_bytes < f.bytes) return BGS_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    (void)hipGetLastError();
    forward(s, batch, height, width, params, rgb, z, hole, f, true);
    const int HW = height * width;
    const int64_t np = (int64_t)batch * HW;
    hipLaunchKernelGGL(k_count, dim3(blocks(np)), dim3(256), 0, s, hole, np, f.cnt_part);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, (const float*)f.cnt_part, (int)blocks(np), (const float*)nullptr,
                       f.n_hole);
    hipLaunchKernelGGL(k_loss, dim3(blocks(np)), dim3(256), 0, s, rgb, hole, (const float*)f.r, target,
                       (const float*)f.n_hole, batch, HW, rgb_out, f.g_r, f.loss_part);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, (const float*)f.loss_part, (int)blocks(np),
                       (const float*)f.n_hole, loss);
    backward(s, batch, height, width, params, f, grad);
    return launched();
}

BGS_API int32_t bgs_repair_set_block_shape(int32_t rows, int32_t tiles) {
    if (!(rows == 0 || rows == 2 || rows == 4 || rows == 8) || tiles < 0 || tiles > 4) return BGS_ERR_INVALID_ARG;
    g_rows.store(rows);
    g_tiles.store(tiles);
    return BGS_OK;
}

BGS_API int32_t bgs_repair_adam(float* params, const float* grad, float* m, float* v, int64_t n, int32_t step,
                                float lr, float beta1, float beta2, float eps, void* hip_stream) {
    if (!params || !grad || !m || !v || n < 1 || step < 1 || !(lr >= 0.f) || !(beta1 >= 0.f && beta1 < 1.f) ||
        !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return BGS_ERR_INVALID_ARG;
    const float c1 = (float)(1.0 - std::pow((double)beta1, step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, step));
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_adam, dim3(blocks(n)), dim3(256), 0, (hipStream_t)hip_stream, params, grad, m, v, n, lr,
                       beta1, beta2, eps, c1, c2);
    return launched();
}

}  // extern "C"
