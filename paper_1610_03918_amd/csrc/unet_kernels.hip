// gfx950 kernels of the learned warm start: a 4-level U-Net (16/32/64/128
// channels, 3x3 convolutions, bfloat16 weights and activations, float32
// accumulation on the matrix cores) with its backward pass, loss, Adam step,
// and the maps between the Poisson problem and the network's tensors.
//
// Convolutions run as implicit GEMMs on v_mfma_f32_16x16x32_bf16: the
// weights are the M operand (output channels), the pixels the N operand and
// the K dimension walks (32-channel chunk, tap).  The input gradient is the
// same kernel with the taps flipped and the weights transposed; what follows
// a convolution (bias, ReLU, rounding, pooling, the head; in the backward
// pass the ReLU mask and the adjoints of upsampling and pooling) is its
// epilogue.  The weight gradient contracts over pixels in a split-K kernel
// whose partial sums are added in a fixed order (deterministic).
#include "unet_internal.h"

#include <algorithm>
#include <mutex>

namespace unet {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int KS = 40;           // LDS row length (bf16) of one pixel's 32-channel chunk, padded
constexpr int PC = 18;           // patch columns: 16 output columns + 2 halo

// float32 -> bfloat16, round to nearest even (finite inputs)
__device__ __forceinline__ uint32_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }

__device__ __forceinline__ bf16x8 ld8(const uint16_t *p) {
    return __builtin_bit_cast(bf16x8, *(const uint4 *)p);
}
// bf16(s) where the layer's output h (4 bfloat16) is positive, else 0.
__device__ __forceinline__ uint2 masked(const f4 &s, const uint2 &h)
{
    uint32_t y[4];
    const uint32_t m[4] = {h.x & 0xFFFFu, h.x >> 16, h.y & 0xFFFFu, h.y >> 16};
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = bf2f(m[i]) > 0.f ? f2bf(s[i]) : 0u;
    return make_uint2(y[0] | (y[1] << 16), y[2] | (y[3] << 16));
}

// The thread's index, computed anew: what follows from it is not carried in
// registers around a loop.
__device__ __forceinline__ int here()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// One thread's share of a staged patch: rows h0-1 .. h0+PR-2, columns w0-1 ..
// w0+16, CQ groups of 8 channels of the concatenation [upsampled(up), src],
// as [row][col][KP] in LDS (zeros outside the image and beyond the channel
// count).  pw: the image wraps along W (the patch never reaches farther than
// one column beyond it).  Loads go to registers first, so that the next
// patch's are in flight while the current one is multiplied, and without a
// branch around any of them (a branch per load made the compiler wait for
// each): outside the image a thread reads the tile's first pixel and stores
// zeros.
template <int PR, int CQ, int KP> struct Patch {
    static constexpr int N = PR * PC * CQ, R = (N + 255) / 256;
    u4 v[R];
    unsigned in;                 // bit k: element k lies in the image
    unsigned ok;                 // and in the channels loaded

    // Offsets d (in pixels of the source) of this thread's elements from the
    // tile's first pixel (h0, w0); half: of a source of half the resolution.
    __device__ __forceinline__ void at(int (&d)[R], int H, int W, int h0, int w0, int pw, bool half)
    {
        const bool inner = h0 > 0 && h0 + PR - 1 <= H && w0 > 0 && w0 + PC - 1 <= W;
        const int tid = here();
        in = 0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int e = tid + 256 * k, pix = e / CQ;
            const int r = pix / PC, s = pix - r * PC;
            int dh = r - 1, dw = s - 1;
            bool i = N % 256 == 0 || e < N;
            if (!inner) {
                const int h = h0 + dh;
                int w = w0 + dw;
                if (pw) w = w < 0 ? w + W : (w == W ? 0 : w);
                i = i && h >= 0 && h < H && w >= 0 && w < W;
                dw = w - w0;
            }
            in |= i ? 1u << k : 0u;
            const int o = half ? (dh >> 1) * (W >> 1) + (dw >> 1) : dh * W + dw;
            d[k] = i ? o : 0;
        }
    }
    // q = src: the source at the tile's first pixel, C channels a pixel, from channel c0 on
    __device__ __forceinline__ void load(const uint16_t *src, int C, int c0, const int (&d)[R])
    {
        const int c = c0 + 8 * (int)(threadIdx.x % CQ);
        ok = c < C ? in : 0u;
        src += c < C ? c : 0;
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = *(const u4 *)(src + (long long)d[k] * C);
    }
    // the network's input: three channels, 6 bytes a pixel
    __device__ __forceinline__ void load3(const uint16_t *src, const int (&d)[R])
    {
        ok = threadIdx.x % CQ == 0 ? in : 0u;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const uint16_t *x = src + (long long)d[k] * kInCh;
            v[k] = u4{x[0] | ((uint32_t)x[1] << 16), x[2], 0u, 0u};
        }
    }
    __device__ __forceinline__ void store(uint16_t *sp) const
    {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (N % 256 == 0 || e < N)
                *(u4 *)(sp + (e / CQ) * KP + 8 * (e % CQ)) = (ok >> k) & 1 ? v[k] : u4{0u, 0u, 0u, 0u};
        }
    }
};

// The value two lanes apart by one in their column (n ^ 1).
__device__ __forceinline__ float beside(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}

// Orders a wavefront's own LDS accesses (its lanes run together).
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// What follows a tile's sums (see k_conv).
template <int NCO, int NR, int EP>
__device__ __forceinline__ void conv_out(const ConvArgs &a, const f4 (&acc)[NCO][NR], int b, int h0, int w0, int ct0,
                                         uint16_t *sh)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4;
    // lane holds channels 16 (ct0 + j) + 4g + (0..3) of pixel column n
    const int w = w0 + n, hw = h0 + wave * NR;
#pragma unroll
    for (int j = 0; j < NCO; ++j) {
        const int co = 16 * (ct0 + j) + 4 * g;
        if (EP == EP_FWD) {
            float bb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) bb[i] = bf2f(f2bf(a.bias[co + i]));
            uint2 y[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                uint32_t q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = f2bf(fmaxf(acc[j][r][i] + bb[i], 0.f));
                y[r] = make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
                if (hw + r < a.H && w < a.W)
                    *(uint2 *)(a.out + (((size_t)b * a.H + hw + r) * a.W + w) * a.Cout + co) = y[r];
                if (NCO == 1) *(uint2 *)(sh + ((wave * NR + r) * 16 + n) * 16 + 4 * g) = y[r];
            }
            if (a.pool) {
#pragma unroll
                for (int r = 0; r < NR; r += 2) {
                    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const float v[4] = {bf2f(y[r + d].x & 0xFFFFu), bf2f(y[r + d].x >> 16),
                                            bf2f(y[r + d].y & 0xFFFFu), bf2f(y[r + d].y >> 16)};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            s[i] += v[i];
                            s[i] += beside(v[i]);
                        }
                    }
                    if ((n & 1) == 0 && hw + r < a.H && w < a.W) {
                        uint32_t q[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) q[i] = f2bf(0.25f * s[i]);
                        *(uint2 *)(a.pool + (((size_t)b * (a.H >> 1) + ((hw + r) >> 1)) * (a.W >> 1) + (w >> 1)) * a.Cout +
                                   co) = make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
                    }
                }
            }
        } else if (EP == EP_MASK) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                if (hw + r >= a.H || w >= a.W) continue;
                const size_t o = (((size_t)b * a.H + hw + r) * a.W + w) * a.Cout + co;
                *(uint2 *)(a.out + o) = masked(acc[j][r], *(const uint2 *)(a.mask + o));
            }
        } else if (EP == EP_UP) {
            if (16 * (ct0 + j) < a.Cup) {
#pragma unroll
                for (int r = 0; r < NR; r += 2) {
                    f4 s = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int d = 0; d < 2; ++d)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            s[i] += acc[j][r + d][i];
                            s[i] += beside(acc[j][r + d][i]);
                        }
                    if ((n & 1) == 0 && hw + r < a.H && w < a.W) {
                        const size_t o =
                            (((size_t)b * (a.H >> 1) + ((hw + r) >> 1)) * (a.W >> 1) + (w >> 1)) * a.Cup + co;
                        *(uint2 *)(a.out + o) = masked(s, *(const uint2 *)(a.mask + o));
                    }
                }
            } else {
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    if (hw + r >= a.H || w >= a.W) continue;
                    *(f4 *)(a.skip + (((size_t)b * a.H + hw + r) * a.W + w) * (a.Cout - a.Cup) + co - a.Cup) = acc[j][r];
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                if (hw + r >= a.H || w >= a.W) continue;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const size_t o = (((size_t)b * 2 * a.H + 2 * (hw + r) + (d >> 1)) * (2 * a.W) + 2 * w + (d & 1)) * a.Cout + co;
                    f4 s = *(const f4 *)(a.skip + o);
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[i] += 0.25f * acc[j][r][i];
                    *(uint2 *)(a.out + o) = masked(s, *(const uint2 *)(a.mask + o));
                }
            }
        }
    }
    if (EP == EP_FWD && NCO == 1) {
        if (!a.hout) return;
        // the head on the rounded values, channels in order: one pixel a lane
        // (each wave reads what it wrote)
        wave_fence();
        if (lane >= 16 * NR) return;
        const int r = lane >> 4, c = lane & 15;
        if (hw + r >= a.H || w0 + c >= a.W) return;
        const uint32_t *u = (const uint32_t *)(sh + ((wave * NR + r) * 16 + c) * 16);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            s += bf2f(u[k] & 0xFFFFu) * a.wh[2 * k];
            s += bf2f(u[k] >> 16) * a.wh[2 * k + 1];
        }
        a.hout[((size_t)b * a.H + hw + r) * a.W + w0 + c] = s + a.wh[16];
    }
}

// ---- convolution ------------------------------------------------------------
// Block: 4 waves; output tiles of 4*NR rows x 16 columns x 16*NCO channels;
// wave w owns rows w*NR .. w*NR+NR-1.  Per chunk of 32 input channels the
// patch and the tile's weights (stored in the order of the matrix operand's
// registers: 1 KiB per tap and 16 channels, read without bank conflicts) sit
// in LDS.  A wave reads its 3 (NR + 2) pixel operands once and uses each for
// the three taps of a column of the stencil, and each weight operand for NR
// rows, and issues the next chunk's global loads before the products of this
// one.  On an input of at most 16 channels (CQ 2: half the operand is
// padding, zeroed in LDS once; CIN3: the network's 3-channel input) a block
// instead walks several tiles, its XCD's in a row (neighbours share their rims
// in its L2), keeps the weights in LDS, and loads the next tile ahead.
// Every output adds its products in the order (chunk, tap), whatever the tile.
//
// Bound: level 0 by memory and LDS reads (16 channels in and out; 134 MB in 38
// us at 4 x 1024 x 512, 3.5 TB/s of 4.7), the deeper levels by the latency of
// a few chunks on few blocks.  Measured on that batch against a kernel that
// read a pixel operand for every tap and left pooling, head and masks to
// kernels of their own: forward 0.67 -> 0.41 ms, input gradients with their
// ReLU and joins 1.60 -> 0.55 ms.
//
// EP_FWD   bias, ReLU, bfloat16; optionally the 2 x 2 means (pool) and the
//          1 x 1 head (hout) of the rounded values
// EP_MASK  input gradient through the ReLU of a layer of the same level:
//          out = bf16(acc) where mask > 0
// EP_UP    input gradient of [upsampled, skip]: channels below Cup summed
//          over 2 x 2 pixels (the adjoint of copying) and masked at the
//          coarser level (out); the others to skip (float32)
// EP_DOWN  input gradient of a pooled input: each of the finer level's 2 x 2
//          pixels gets skip + acc / 4, masked
template <int NCO, int NR, int EP, int CQ, bool CIN3>
__global__ __launch_bounds__(256, NCO *NR <= 4 && CQ == 2 ? 3 : 2) void k_conv(ConvArgs a)
{
    constexpr int TX = 4 * NR, PR = TX + 2;
    constexpr bool WALK = CQ == 2;
    typedef Patch<PR, CQ, KS> P_t;
    constexpr int NW = NCO * 9 * 64, RW = (NW + 255) / 256;
    __shared__ __align__(16) uint16_t sp[PR * PC * KS];
    __shared__ __align__(16) uint16_t sw[NCO * 9 * 512];
    // the head's transposition (the padding of sp has to stay zero)
    __shared__ __align__(16) uint16_t sh[EP == EP_FWD && NCO == 1 ? TX * 256 : 8];
    const int tilesW = (a.W + 15) >> 4, tilesH = (a.H + TX - 1) / TX;
    const int ntiles = a.B * tilesH * tilesW, per = (ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3;
    const int last = min(ntiles - xcd * per, per);      // tiles xcd * per + 0 .. last - 1
    int tl = blockIdx.x >> 3;
    if (tl >= last) return;
    const int ct0 = blockIdx.y * NCO;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4;

    P_t patch;
    int d[P_t::R], dup[WALK ? 1 : P_t::R] = {};
    u4 wv[RW];
    auto load_w = [&](int ch) {
        const u4 *wt = (const u4 *)a.wt + ((size_t)ch * a.nct + ct0) * (9 * 64);
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            const int e = threadIdx.x + 256 * k;
            wv[k] = wt[NW % 256 == 0 || e < NW ? e : NW - 1];
        }
    };
    auto store_w = [&]() {
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (NW % 256 == 0 || e < NW) ((u4 *)sw)[e] = wv[k];
        }
    };
    int b, h0, w0;
    auto place = [&](int q) {
        const int tile = xcd * per + q, rest = tile / tilesW;
        w0 = 16 * (tile - rest * tilesW);
        b = rest / tilesH;
        h0 = TX * (rest - b * tilesH);
        patch.at(d, a.H, a.W, h0, w0, a.pw, false);
        if constexpr (!WALK) {
            if (a.Cu) patch.at(dup, a.H, a.W, h0, w0, a.pw, true);
        }
    };
    auto load = [&](int ch) {
        const size_t first = ((size_t)b * a.H + h0) * a.W + w0;
        if constexpr (CIN3) {
            patch.load3(a.src + first * kInCh, d);
        } else if constexpr (WALK) {
            patch.load(a.src + first * a.Cs, a.Cs, 0, d);
        } else {
            // the 32 channels of a chunk lie in up or in src as a whole
            const int c0 = ch * kKChunk;
            const bool half = c0 < a.Cu;
            const int C = half ? a.Cu : a.Cs;
            int o[P_t::R];
#pragma unroll
            for (int k = 0; k < P_t::R; ++k) o[k] = half ? dup[k] : d[k];
            patch.load(half ? a.up + (((size_t)b * (a.H >> 1) + (h0 >> 1)) * (a.W >> 1) + (w0 >> 1)) * C : a.src + first * C,
                       C, half ? c0 : c0 - a.Cu, o);
        }
    };
    auto products = [&](f4 (&acc)[NCO][NR]) {
        bf16x8 Bv[NR + 2][3];
#pragma unroll
        for (int r = 0; r < NR + 2; ++r)
#pragma unroll
            for (int dw = 0; dw < 3; ++dw) Bv[r][dw] = ld8(sp + ((wave * NR + r) * PC + n + dw) * KS + 8 * g);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int dh = t / 3, dw = t - 3 * (t / 3);
            bf16x8 A[NCO];
#pragma unroll
            for (int j = 0; j < NCO; ++j) A[j] = ld8(sw + (j * 9 + t) * 512 + lane * 8);
#pragma unroll
            for (int j = 0; j < NCO; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    acc[j][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[j], Bv[r + dh][dw], acc[j][r], 0, 0, 0);
        }
    };
    place(tl);
    load_w(0);
    load(0);
    f4 acc[NCO][NR];
    auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < NCO; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[j][r] = f4{0.f, 0.f, 0.f, 0.f};
    };
    if constexpr (!WALK) {
        clear();
        for (int ch = 0; ch < a.nchunk; ++ch) {
            if (ch) __syncthreads();
            patch.store(sp);
            store_w();
            __syncthreads();
            if (ch + 1 < a.nchunk) {
                load_w(ch + 1);
                load(ch + 1);
            }
            products(acc);
        }
        conv_out<NCO, NR, EP>(a, acc, b, h0, w0, ct0, sh);
    } else {
        for (int e = threadIdx.x; e < PR * PC * 2; e += 256)
            *(u4 *)(sp + (e >> 1) * KS + 16 + 8 * (e & 1)) = u4{0u, 0u, 0u, 0u};
        store_w();
        for (;;) {
            patch.store(sp);
            __syncthreads();
            const int hb = b, hh = h0, ww = w0;
            tl += stride;
            if (tl < last) {
                place(tl);
                load(0);
            }
            clear();
            products(acc);
            conv_out<NCO, NR, EP>(a, acc, hb, hh, ww, ct0, sh);
            if (tl >= last) return;
            __syncthreads();
        }
    }
}

// A tile of fewer rows or channels gives more blocks; below this many tiles
// the chip is not filled.
constexpr int kConvBlocks = 512;

template <int NR> static int conv_tiles(const ConvArgs &a)
{
    return a.B * ((a.H + 4 * NR - 1) / (4 * NR)) * ((a.W + 15) >> 4);
}

template <int NCO, int NR, int EP, int CQ, bool CIN3> static void conv_run(const ConvArgs &a, hipStream_t s)
{
    // walking tiles: as many blocks as run at once (three a CU), every one the same number of tiles
    const int per = (conv_tiles<NR>(a) + 7) / 8, ny = a.nct / NCO, slots = std::max(1, 96 / ny);
    const int rounds = CQ == 2 ? (per + slots - 1) / slots : 1;
    hipLaunchKernelGGL((k_conv<NCO, NR, EP, CQ, CIN3>), dim3(8 * ((per + rounds - 1) / rounds), ny), dim3(256), 0, s, a);
}

// Wide tiles read each weight operand for more pixels; of two equally wide in
// channels the taller one has the smaller rim.  Against that stand registers:
// 32 channels of 32 or more inputs ran faster in tiles of 8 rows than of 16
// (masked gradient at 512 x 256 pixels, batch 4: 23 against 29 us; forward 24
// against 26), 16 channels of 48 slower (77 against 72 us at 1024 x 512).
template <int EP, int CQ, bool CIN3> static void conv_launch(const ConvArgs &a, hipStream_t s)
{
    const int t4 = conv_tiles<4>(a) * a.nct, t2 = conv_tiles<2>(a) * a.nct;
    if constexpr (CQ == 4) {
        if (a.nct % 4 == 0 && t4 / 4 >= kConvBlocks) return conv_run<4, 4, EP, CQ, CIN3>(a, s);
    }
    if constexpr (!CIN3) {
        if (a.nct % 3 == 0 && t4 / 3 >= kConvBlocks) return conv_run<3, 4, EP, CQ, CIN3>(a, s);
        if constexpr (CQ == 2) {
            if (a.nct % 2 == 0 && t4 / 2 >= kConvBlocks) return conv_run<2, 4, EP, CQ, CIN3>(a, s);
        }
        if (a.nct % 2 == 0 && t2 / 2 >= kConvBlocks) return conv_run<2, 2, EP, CQ, CIN3>(a, s);
    }
    if (a.nct == 1 && t4 >= kConvBlocks) return conv_run<1, 4, EP, CQ, CIN3>(a, s);
    conv_run<1, 2, EP, CQ, CIN3>(a, s);
}

void launch_conv(const ConvArgs &a, int ep, hipStream_t s)
{
    const bool narrow = a.Cu + a.Cs <= 16;
    if (a.Cs == kInCh) conv_launch<EP_FWD, 2, true>(a, s);
    else if (ep == EP_FWD) narrow ? conv_launch<EP_FWD, 2, false>(a, s) : conv_launch<EP_FWD, 4, false>(a, s);
    else if (ep == EP_MASK) narrow ? conv_launch<EP_MASK, 2, false>(a, s) : conv_launch<EP_MASK, 4, false>(a, s);
    else if (ep == EP_UP) narrow ? conv_launch<EP_UP, 2, false>(a, s) : conv_launch<EP_UP, 4, false>(a, s);
    else conv_launch<EP_DOWN, 4, false>(a, s);
}

// ---- weight gradient ------------------------------------------------------
// gw[co][t][ci] = sum over pixels p of gy[p][co] * in(p + tap t)[ci]
// Block (split, tile of 16 NCO output channels, NCS groups of 16 input
// channels) walks pixel tiles of 16 x 16 (split, split + nsplit, ...).  Wave w
// owns tile rows 4w .. 4w+3 as two K steps of 32 pixels (2 rows x 16 columns;
// lane group g: row 2 step + g / 2, columns 8 (g % 2) .. +7).  Both operands
// have pixels along K while LDS holds them by pixel, so they are read with
// the transposing LDS load (4 pixels of 16 channels a lane group); the three
// taps of a stencil row share one run of 12 pixels, realigned in registers.
// The next tile's global loads are issued before this one's products.  The
// four waves' sums meet in LDS in a fixed order and leave in register order
// (1 KiB a fragment); k_wgrad_reduce adds the splits.
//
// Measured at 4 x 1024 x 512, all layers: 2.58 ms with operands gathered 16
// bits at a time, 0.50 so; the reduction 0.78 -> 0.06 ms (one launch, half
// the splits).  Bound by the latency of a tile's loads at two blocks a CU (the
// sums take 144 registers), the layers of 16 channels by memory.
constexpr int kWTX = 16;

typedef short s4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4 lds_s4;

__device__ __forceinline__ uint2 ld_tr(const uint16_t *p)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)p));
}

template <int NCO, int NCS, bool CIN3>
__global__ __launch_bounds__(256, 2) void k_wgrad(WgradArgs a)
{
    constexpr int PR = kWTX + 2, CT = 16 * NCO, GS = CT + 8, KP = 16 * NCS + 8;
    typedef Patch<PR, 2 * NCS, KP> P_t;
    constexpr int SP = PR * PC * KP, SG = kWTX * 16 * GS;
    constexpr int NF = NCO * NCS * 9 + NCO;              // fragments of a wave's sums (bias last)
    constexpr int STAGE_B = 2 * (SP + SG), RED_B = 2 * NF * 1024;
    __shared__ __align__(16) unsigned char smem[STAGE_B > RED_B ? STAGE_B : RED_B];
    uint16_t *sp = (uint16_t *)smem;
    uint16_t *sg = sp + SP;
    const int tilesW = (a.W + 15) >> 4, tilesH = (a.H + kWTX - 1) / kWTX;
    const int ntiles = a.B * tilesH * tilesW;
    const int split = blockIdx.x, co0 = blockIdx.y * CT, cs0 = a.cs0 + blockIdx.z * NCS;
    const bool with_bias = cs0 == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4;
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));

    f4 acc[NCO][NCS][9];
    f4 bacc[NCO];
#pragma unroll
    for (int j = 0; j < NCO; ++j) {
        bacc[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCS; ++c)
#pragma unroll
            for (int t = 0; t < 9; ++t) acc[j][c][t] = f4{0.f, 0.f, 0.f, 0.f};
    }

    // this block's input channels lie in up or in src as a whole
    const bool half = 16 * cs0 < a.Cu;
    const int C = half ? a.Cu : a.Cs, c0 = half ? 16 * cs0 : 16 * cs0 - a.Cu;
    const uint16_t *const src = half ? a.up : a.src;
    P_t patch;
    constexpr int RG = CT / 8;
    u4 gv[RG];
    unsigned gok = 0;
    auto load = [&](int tile) {
        const int rest = tile / tilesW, w0 = 16 * (tile - rest * tilesW);
        const int b = rest / tilesH, h0 = kWTX * (rest - b * tilesH);
        const uint16_t *gy = a.gy + (((size_t)b * a.H + h0) * a.W + w0) * a.Cout + co0;
        const bool inner = h0 + kWTX <= a.H && w0 + 16 <= a.W;
        const int tid = here();
        gok = 0;
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            const int e = tid + 256 * k, px = e / (CT / 8), q = e % (CT / 8);
            const int dh = px >> 4, dw = px & 15;
            const bool in = inner || (h0 + dh < a.H && w0 + dw < a.W);
            gok |= in ? 1u << k : 0u;
            gv[k] = *(const u4 *)(gy + (long long)(in ? dh * a.W + dw : 0) * a.Cout + 8 * q);
        }
        int d[P_t::R];
        patch.at(d, a.H, a.W, h0, w0, a.pw, half);
        const size_t first = half ? ((size_t)b * (a.H >> 1) + (h0 >> 1)) * (a.W >> 1) + (w0 >> 1)
                                  : ((size_t)b * a.H + h0) * a.W + w0;
        if constexpr (CIN3) patch.load3(src + first * kInCh, d);
        else patch.load(src + first * C, C, c0, d);
    };
    load(split);
    for (int tile = split; tile < ntiles; tile += a.nsplit) {
        if (tile != split) __syncthreads();
        patch.store(sp);
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            const int e = threadIdx.x + 256 * k;
            *(u4 *)(sg + (e / (CT / 8)) * GS + 8 * (e % (CT / 8))) = (gok >> k) & 1 ? gv[k] : u4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
        if (tile + a.nsplit < ntiles) load(tile + a.nsplit);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int R = 4 * wave + 2 * ks + (g >> 1);
            const int col = 8 * (g & 1) + (n >> 2), c4 = 4 * (n & 3);
            bf16x8 A[NCO];
#pragma unroll
            for (int j = 0; j < NCO; ++j) {
                const uint16_t *p = sg + (R * 16 + col) * GS + 16 * j + c4;
                const uint2 x = ld_tr(p), y = ld_tr(p + 4 * GS);
                A[j] = __builtin_bit_cast(bf16x8, make_uint4(x.x, x.y, y.x, y.y));
            }
#pragma unroll
            for (int dh = 0; dh < 3; ++dh) {
#pragma unroll
                for (int c = 0; c < NCS; ++c) {
                    // pixels 0 .. 11 of the run (10 used): two a register
                    const uint16_t *p = sp + ((R + dh) * PC + col) * KP + 16 * c + c4;
                    const uint2 x = ld_tr(p), y = ld_tr(p + 4 * KP);
                    uint2 z;
                    // the run's last pixels; the patch ends two columns after its right half
                    z = ld_tr(sp + ((R + dh) * PC + min(col + 8, PC - 1)) * KP + 16 * c + c4);
                    const bf16x8 B0 = __builtin_bit_cast(bf16x8, make_uint4(x.x, x.y, y.x, y.y));
                    const bf16x8 B1 = __builtin_bit_cast(
                        bf16x8, make_uint4(__builtin_amdgcn_alignbit(x.y, x.x, 16), __builtin_amdgcn_alignbit(y.x, x.y, 16),
                                           __builtin_amdgcn_alignbit(y.y, y.x, 16), __builtin_amdgcn_alignbit(z.x, y.y, 16)));
                    const bf16x8 B2 = __builtin_bit_cast(bf16x8, make_uint4(x.y, y.x, y.y, z.x));
#pragma unroll
                    for (int j = 0; j < NCO; ++j) {
                        acc[j][c][3 * dh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[j], B0, acc[j][c][3 * dh], 0, 0, 0);
                        acc[j][c][3 * dh + 1] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[j], B1, acc[j][c][3 * dh + 1], 0, 0, 0);
                        acc[j][c][3 * dh + 2] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[j], B2, acc[j][c][3 * dh + 2], 0, 0, 0);
                    }
                }
            }
            if (with_bias) {
#pragma unroll
                for (int j = 0; j < NCO; ++j)
                    bacc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[j], ones, bacc[j], 0, 0, 0);
            }
        }
    }
    // waves (0 + 1) + (2 + 3): 1 and 3 hand over, then 2
    f4 *red = (f4 *)smem;
    __syncthreads();
    auto put = [&](int half) {
        f4 *d = red + half * NF * 64 + lane;
#pragma unroll
        for (int j = 0; j < NCO; ++j) {
#pragma unroll
            for (int c = 0; c < NCS; ++c)
#pragma unroll
                for (int t = 0; t < 9; ++t) d[((j * NCS + c) * 9 + t) * 64] = acc[j][c][t];
            d[(NCO * NCS * 9 + j) * 64] = bacc[j];
        }
    };
    auto add = [&](int half) {
        const f4 *d = red + half * NF * 64 + lane;
#pragma unroll
        for (int j = 0; j < NCO; ++j) {
#pragma unroll
            for (int c = 0; c < NCS; ++c)
#pragma unroll
                for (int t = 0; t < 9; ++t) acc[j][c][t] += d[((j * NCS + c) * 9 + t) * 64];
            bacc[j] += d[(NCO * NCS * 9 + j) * 64];
        }
    };
    if (wave & 1) put(wave >> 1);
    __syncthreads();
    if (!(wave & 1)) add(wave >> 1);
    __syncthreads();
    if (wave == 2) put(1);
    __syncthreads();
    if (wave != 0) return;
    add(1);
    f4 *part = (f4 *)(a.part + (size_t)split * a.frags * 256) + lane;
#pragma unroll
    for (int j = 0; j < NCO; ++j) {
#pragma unroll
        for (int c = 0; c < NCS; ++c)
#pragma unroll
            for (int t = 0; t < 9; ++t)
                part[(size_t)((((co0 >> 4) + j) * a.ncs + cs0 + c) * 9 + t) * 64] = acc[j][c][t];
        // every column of the bias product holds the same sums
        if (with_bias && n == 0) *(f4 *)(a.bpart + (size_t)split * a.Cout + co0 + 16 * j + 4 * g) = bacc[j];
    }
}

int wgrad_tiles(int B, int H, int W) { return B * ((H + kWTX - 1) / kWTX) * ((W + 15) >> 4); }

int wgrad_splits(int B, int H, int W, int Cin, int Cout)
{
    // about two blocks per CU: each block's sums are written and read once,
    // so more splits are more traffic and fewer leave CUs idle
    // (16 output channels: half the sums a block, and twice the blocks)
    const bool wide = Cout % 32 == 0;
    const int ncs = (Cin + 15) >> 4, per = (wide ? Cout / 32 : Cout / 16) * ((ncs + 1) / 2);
    const int ns = ((wide ? kWgradBlocks : 2 * kWgradBlocks) + per - 1) / per;
    return std::max(1, std::min(ns, wgrad_tiles(B, H, W)));
}

template <int NCO> static void wgrad_run(WgradArgs a, hipStream_t s)
{
    const int ny = a.Cout / (16 * NCO), pairs = a.ncs / 2;
    a.cs0 = 0;
    if (pairs) hipLaunchKernelGGL((k_wgrad<NCO, 2, false>), dim3(a.nsplit, ny, pairs), dim3(256), 0, s, a);
    if (a.ncs & 1) {
        a.cs0 = 2 * pairs;
        hipLaunchKernelGGL((k_wgrad<NCO, 1, false>), dim3(a.nsplit, ny, 1), dim3(256), 0, s, a);
    }
}

void launch_wgrad(const WgradArgs &a, hipStream_t s)
{
    if (a.Cs == kInCh) hipLaunchKernelGGL((k_wgrad<1, 1, true>), dim3(a.nsplit, a.Cout / 16, 1), dim3(256), 0, s, a);
    else if (a.Cout % 32 == 0) wgrad_run<2>(a, s);
    else wgrad_run<1>(a, s);
}

// Sums of the split partials of every layer in one launch: a block owns one
// fragment (16 output x 16 input channels of one tap, 4 values a lane), four
// groups of lanes take every fourth split, and the groups are added in order
// (float64, deterministic).  The last blocks sum the biases, one a layer.
__global__ __launch_bounds__(256) void k_wgrad_reduce(ReduceArgs a, float *grads)
{
    __shared__ double sh[4][256];
    int k = 0;
#pragma unroll
    for (int i = 1; i < kNConv; ++i) k += (int)blockIdx.x >= a.L[i].block0 ? 1 : 0;
    if ((int)blockIdx.x >= a.wblocks) k = (int)blockIdx.x - a.wblocks;
    const ReduceLayer &L = a.L[k];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    if ((int)blockIdx.x >= a.wblocks) {
        for (int c = lane; c < L.Cout; c += 64) {
            double s = 0.0;
#pragma unroll 8
            for (int i = q; i < L.nsplit; i += 4) s += L.bpart[(size_t)i * L.Cout + c];
            sh[q][c] = s;
        }
        __syncthreads();
        for (int c = threadIdx.x; c < L.Cout; c += 256)
            grads[L.b_off + c] = (float)(((sh[0][c] + sh[1][c]) + sh[2][c]) + sh[3][c]);
        return;
    }
    const int f = blockIdx.x - L.block0;
    const f4 *p = (const f4 *)L.part + (size_t)f * 64 + lane;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int i = q; i < L.nsplit; i += 4) {
        const f4 v = p[(size_t)i * L.frags * 64];
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] += v[c];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) sh[q][c * 64 + lane] = s[c];
    __syncthreads();
    // thread -> (co, ci) of the fragment: lane (n, g) holds co = 4g + c, ci = n
    const int c = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
    const int t = f % 9, cs = (f / 9) % L.ncs, ct = f / (9 * L.ncs);
    const int co = 16 * ct + 4 * g + c, ci = 16 * cs + n;
    if (ci >= L.Cin) return;
    const int e = threadIdx.x;
    grads[L.w_off + ((long long)co * 9 + t) * L.Cin + ci] = (float)(((sh[0][e] + sh[1][e]) + sh[2][e]) + sh[3][e]);
}

void launch_wgrad_reduce(const ReduceArgs &a, float *grads, hipStream_t s)
{
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(a.wblocks + kNConv), dim3(256), 0, s, a, grads);
}

// ---- reductions over pixels: the head's gradient and the loss ----------------
// pixels per block of the reducing kernels: enough blocks to fill the chip, few enough partial sums
static int red_px(long long P) { return P >= (1 << 20) ? 4096 : P >= (1 << 18) ? 1024 : 256; }

template <int N>
__device__ __forceinline__ void block_sum_store(double (&v)[N], double *dst) {
    __shared__ double sh[N][256];
#pragma unroll
    for (int k = 0; k < N; ++k) sh[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
#pragma unroll
            for (int k = 0; k < N; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) dst[k] = sh[k][0];
    }
}

int head_bwd_blocks(long long P) { return (int)((P + red_px(P) - 1) / red_px(P)); }

__global__ void k_head_bwd(const uint16_t *h, const float *wh, const float *gout, uint16_t *gy,
                           double *part, long long P, int px) {
    double acc[17];
#pragma unroll
    for (int k = 0; k < 17; ++k) acc[k] = 0.0;
    const long long p0 = (long long)blockIdx.x * px;
    for (long long p = p0 + threadIdx.x; p < p0 + px && p < P; p += blockDim.x) {
        const float go = gout[p];
        const uint4 v0 = *(const uint4 *)(h + p * 16), v1 = *(const uint4 *)(h + p * 16 + 8);
        const uint32_t u[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        uint32_t y[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float a0 = bf2f(u[k] & 0xFFFFu), a1 = bf2f(u[k] >> 16);
            acc[2 * k] += (double)go * a0;
            acc[2 * k + 1] += (double)go * a1;
            const uint32_t g0 = a0 > 0.f ? f2bf(go * wh[2 * k]) : 0u;
            const uint32_t g1 = a1 > 0.f ? f2bf(go * wh[2 * k + 1]) : 0u;
            y[k] = g0 | (g1 << 16);
        }
        acc[16] += go;
        *(uint4 *)(gy + p * 16) = make_uint4(y[0], y[1], y[2], y[3]);
        *(uint4 *)(gy + p * 16 + 8) = make_uint4(y[4], y[5], y[6], y[7]);
    }
    block_sum_store<17>(acc, part + 17 * (size_t)blockIdx.x);
}

void launch_head_bwd(const uint16_t *h, const float *wh, const float *gout, uint16_t *gy,
                     double *part, long long P, hipStream_t s) {
    hipLaunchKernelGGL(k_head_bwd, dim3(head_bwd_blocks(P)), dim3(256), 0, s, h, wh, gout, gy, part, P, red_px(P));
}

// Sum of n values st apart by one wavefront, in a fixed order.
__device__ __forceinline__ double wave_total(const double *p, int n, int st)
{
    const int lane = threadIdx.x & 63;
    double s = 0.0;
#pragma unroll 8
    for (int k = lane; k < n; k += 64) s += p[(size_t)k * st];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    return s;
}

__global__ __launch_bounds__(1024) void k_head_finalize(const double *part, int nblk, float *gwh) {
    const int w = threadIdx.x >> 6;
    for (int k = w; k < 17; k += 16) {
        const double s = wave_total(part + k, nblk, 17);
        if ((threadIdx.x & 63) == 0) gwh[k] = (float)s;
    }
}

void launch_head_finalize(const double *part, int nblk, float *gwh, hipStream_t s) {
    hipLaunchKernelGGL(k_head_finalize, dim3(1), dim3(1024), 0, s, part, nblk, gwh);
}

// ---- masked mean-square loss ---------------------------------------------------
int loss_blocks(long long P) { return (int)((P + red_px(P) - 1) / red_px(P)); }

__global__ void k_mask_sum(const float *mask, double *part, long long P, int px) {
    double acc[1] = {0.0};
    const long long p0 = (long long)blockIdx.x * px;
    for (long long p = p0 + threadIdx.x; p < p0 + px && p < P; p += blockDim.x) acc[0] += mask[p];
    block_sum_store<1>(acc, part + blockIdx.x);
}

void launch_mask_sum(const float *mask, double *part, long long P, hipStream_t s) {
    hipLaunchKernelGGL(k_mask_sum, dim3(loss_blocks(P)), dim3(256), 0, s, mask, part, P, red_px(P));
}

// loss = sum m (out - t)^2 / sum m;  gout = 2 m (out - t) / sum m
__global__ void k_loss(const float *out, const float *target, const float *mask, const double *msum,
                       float *gout, double *part, long long P, int px) {
    double acc[1] = {0.0};
    const double inv = *msum > 0.0 ? 1.0 / *msum : 0.0;
    const long long p0 = (long long)blockIdx.x * px;
    for (long long p = p0 + threadIdx.x; p < p0 + px && p < P; p += blockDim.x) {
        const double d = (double)out[p] - (double)target[p];
        acc[0] += (double)mask[p] * d * d;
        gout[p] = (float)(2.0 * mask[p] * d * inv);
    }
    acc[0] *= inv;
    block_sum_store<1>(acc, part + blockIdx.x);
}

void launch_loss(const float *out, const float *target, const float *mask, const double *msum,
                 float *gout, double *part, long long P, hipStream_t s) {
    hipLaunchKernelGGL(k_loss, dim3(loss_blocks(P)), dim3(256), 0, s, out, target, mask, msum, gout, part, P, red_px(P));
}

__global__ void k_sum_parts(const double *part, int n, double *dst) {
    const double s = wave_total(part, n, 1);
    if (threadIdx.x == 0) *dst = s;
}

void launch_sum_parts(const double *part, int n, double *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(64), 0, s, part, n, dst);
}

// ---- parameters -------------------------------------------------------------------
// Weights of every layer as the matrix operand reads them: per 32-channel
// chunk, 16 output channels and tap one fragment of 64 lanes x 8 bfloat16
// (lane (n, g): output channel n, input channels 8g .. 8g+7), zero beyond the
// channel count.  Forward: wf; input gradient: wd, taps flipped and channels
// swapped.  A thread writes 8 values of a fragment.
__global__ __launch_bounds__(256) void k_wprep(const float *params, PrepArgs a)
{
    int k = 0;
    const int e = blockIdx.x * 256 + threadIdx.x;
#pragma unroll
    for (int i = 1; i < 2 * kNConv; ++i) k += e >= a.first[i] ? 1 : 0;
    if (e >= a.first[2 * kNConv]) return;
    const int y = k >> 1, back = k & 1;
    const int M = back ? a.Cin[y] : a.Cout[y], K = back ? a.Cout[y] : a.Cin[y];
    const int q = e - a.first[k], lane = q & 63, f = q >> 6;
    const int nct = (M + 15) >> 4, t = f % 9, ct = (f / 9) % nct, ch = f / (9 * nct);
    const int m = 16 * ct + (lane & 15), c0 = 32 * ch + 8 * (lane >> 4);
    const float *w = params + a.w_off[y];
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = c0 + i;
        v[i] = 0u;
        if (m < M && c < K) {
            const int co = back ? c : m, ci = back ? m : c, tap = back ? 8 - t : t;
            v[i] = f2bf(w[((long long)co * 9 + tap) * a.Cin[y] + ci]);
        }
    }
    *(uint4 *)((back ? a.wd[y] : a.wf[y]) + (size_t)q * 8) =
        make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}

void launch_wprep(const float *params, const PrepArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_wprep, dim3((a.first[2 * kNConv] + 255) / 256), dim3(256), 0, s, params, a);
}

__global__ void k_adam(float *p, const float *g, float *m, float *v, long long n, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

void launch_adam(float *p, const float *g, float *m, float *v, long long n, float lr, float b1,
                 float b2, float eps, float c1, float c2, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, g, m, v, n, lr,
                       b1, b2, eps, c1, c2);
}

// ---- Poisson problem <-> network tensors -----------------------------------------
// Pixel (h, w) is node (h, w) of the NX x NY node grid (h < H <= NX, w < W <= NY).
// Input channels: source term on free nodes * s_rho; free-node indicator;
// Dirichlet value * s_v on conductor nodes.  Target: phi / s_phi; mask: free.
__global__ void k_snapshot(const double *b, const double *phi, const uint8_t *nc, int NX, int NY,
                           int H, int W, float s_rho, float s_v, float s_phi, uint16_t *x,
                           float *target, float *mask) {
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= (long long)H * W) return;
    const int h = (int)(p / W), w = (int)(p % W);
    const long long node = (long long)h * NY + w;
    const bool freen = nc[node] == 0;
    const double bv = b[node];
    x[3 * p + 0] = (uint16_t)(freen ? f2bf((float)(bv * s_rho)) : 0u);
    x[3 * p + 1] = (uint16_t)(freen ? 0x3F80u : 0u);
    x[3 * p + 2] = (uint16_t)(freen ? 0u : f2bf((float)(bv * s_v)));
    if (phi) {
        target[p] = (float)(phi[node] / s_phi);
        mask[p] = freen ? 1.f : 0.f;
    }
}

void launch_snapshot(const double *b, const double *phi, const uint8_t *node_cond, int NX, int NY,
                     int H, int W, float s_rho, float s_v, float s_phi, uint16_t *x, float *target,
                     float *mask, hipStream_t s) {
    const long long n = (long long)H * W;
    hipLaunchKernelGGL(k_snapshot, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, b, phi, node_cond,
                       NX, NY, H, W, s_rho, s_v, s_phi, x, target, mask);
}

__global__ void k_guess(const float *out, const double *b, const uint8_t *nc, int NX, int NY, int H,
                        int W, float s_phi, double *guess) {
    const long long node = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (node >= (long long)NX * NY) return;
    const int i = (int)(node / NY), j = (int)(node % NY);
    double v = 0.0;
    if (nc[node] != 0) v = b[node];
    else if (i < H && j < W) v = (double)out[(long long)i * W + j] * (double)s_phi;
    guess[node] = v;
}

void launch_guess(const float *out, const double *b, const uint8_t *node_cond, int NX, int NY,
                  int H, int W, float s_phi, double *guess, hipStream_t s) {
    const long long n = (long long)NX * NY;
    hipLaunchKernelGGL(k_guess, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, b, node_cond, NX,
                       NY, H, W, s_phi, guess);
}

// ---- residual learning: samples, stored-sample loads and the corrected start --------
// The start is the linear extrapolation phi_s = 2 phi_1 - phi_2 (phi_1 when
// phi_2 is null); r = b - A phi_s on free nodes with A = 4 - (free
// neighbours), neighbours wrapping on periodic axes (a free node never lies
// on a bounded edge).  Input x [H][W][3] = (bf16(r s_r) on free nodes, free
// indicator, bf16(b s_v) on Dirichlet nodes); target t [H][W] =
// bf16((phi_t - phi_s) s_d) on free nodes.  part (may be null): per-block
// sums of r^2, (phi_t - phi_s)^2 and the free-node count, summed in block
// order by k_rsample_sum into stats.
__device__ __forceinline__ double start_at(const double *p1, const double *p2, long long n) {
    return p2 ? 2.0 * p1[n] - p2[n] : p1[n];
}

constexpr int kRsBlock = 256;

__global__ __launch_bounds__(kRsBlock) void k_rsample(const double *b, const double *p1, const double *p2,
                                                      const double *pt, const uint8_t *nc, int NX, int NY,
                                                      int px, int py, int H, int W, float s_r, float s_v,
                                                      float s_d, uint16_t *x, uint16_t *t, double *part) {
    const long long p = (long long)blockIdx.x * kRsBlock + threadIdx.x;
    double rr = 0.0, dd = 0.0, cnt = 0.0;
    if (p < (long long)H * W) {
        const int i = (int)(p / W), j = (int)(p % W);
        const long long n = (long long)i * NY + j;
        const bool freen = nc[n] == 0;
        uint16_t x0 = 0, x2 = 0, t0 = 0;
        if (freen) {
            double s = 4.0 * start_at(p1, p2, n);
            const int im = i - 1 < 0 ? (px ? NX - 1 : -1) : i - 1;
            const int ip = i + 1 >= NX ? (px ? 0 : -1) : i + 1;
            const int jm = j - 1 < 0 ? (py ? NY - 1 : -1) : j - 1;
            const int jp = j + 1 >= NY ? (py ? 0 : -1) : j + 1;
            long long q;
            if (im >= 0 && !nc[q = (long long)im * NY + j]) s -= start_at(p1, p2, q);
            if (ip >= 0 && !nc[q = (long long)ip * NY + j]) s -= start_at(p1, p2, q);
            if (jm >= 0 && !nc[q = (long long)i * NY + jm]) s -= start_at(p1, p2, q);
            if (jp >= 0 && !nc[q = (long long)i * NY + jp]) s -= start_at(p1, p2, q);
            const double r = b[n] - s;
            x0 = (uint16_t)f2bf((float)(r * s_r));
            rr = r * r;
            cnt = 1.0;
            if (pt) {
                const double d = pt[n] - start_at(p1, p2, n);
                t0 = (uint16_t)f2bf((float)(d * s_d));
                dd = d * d;
            }
        } else {
            x2 = (uint16_t)f2bf((float)(b[n] * s_v));
        }
        x[3 * p + 0] = x0;
        x[3 * p + 1] = (uint16_t)(freen ? 0x3F80u : 0u);
        x[3 * p + 2] = x2;
        if (t) t[p] = t0;
    }
    if (part) {
        double v[3] = {rr, dd, cnt};
        __shared__ double sh[3][kRsBlock];
#pragma unroll
        for (int k = 0; k < 3; ++k) sh[k][threadIdx.x] = v[k];
        __syncthreads();
        for (int off = kRsBlock / 2; off > 0; off >>= 1) {
            if ((int)threadIdx.x < off)
#pragma unroll
                for (int k = 0; k < 3; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + off];
            __syncthreads();
        }
        if (threadIdx.x == 0)
#pragma unroll
            for (int k = 0; k < 3; ++k) part[3 * (long long)blockIdx.x + k] = sh[k][0];
    }
}

// stats[k] += the sum of the nblk partials of quantity k, in block order
// (one wavefront: lane l sums blocks l, l + 64, ...; the 64 lane sums are
// then added in lane order by lane 0).
__global__ void k_rsample_sum(const double *part, int nblk, double *stats) {
    __shared__ double sh[3][64];
    const int l = threadIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int b = l; b < nblk; b += 64)
#pragma unroll
        for (int k = 0; k < 3; ++k) s[k] += part[3 * (long long)b + k];
#pragma unroll
    for (int k = 0; k < 3; ++k) sh[k][l] = s[k];
    __syncthreads();
    if (l == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double a = 0.0;
            for (int q = 0; q < 64; ++q) a += sh[k][q];
            stats[k] += a;
        }
    }
}

long long rsample_blocks(int H, int W) { return ((long long)H * W + kRsBlock - 1) / kRsBlock; }

void launch_rsample(const double *b, const double *p1, const double *p2, const double *pt,
                    const uint8_t *nc, int NX, int NY, int px, int py, int H, int W, float s_r, float s_v,
                    float s_d, uint16_t *x, uint16_t *t, double *stats, double *part, hipStream_t s) {
    const long long nb = rsample_blocks(H, W);
    hipLaunchKernelGGL(k_rsample, dim3((unsigned)nb), dim3(kRsBlock), 0, s, b, p1, p2, pt, nc, NX, NY, px, py,
                       H, W, s_r, s_v, s_d, x, t, stats ? part : nullptr);
    if (stats) hipLaunchKernelGGL(k_rsample_sum, dim3(1), dim3(64), 0, s, part, (int)nb, stats);
}

// ---- the residual sample without a caller work array ------------------------
// Its per-block partial sums live in `scratch`, a file-scope device array that
// every call on a device shares (each device holds its own copy until the
// process ends).  Host code never passes the array's name to a kernel: the
// device address comes from hipGetSymbolAddress, looked up once per device
// with that device current.  Every block writes its three partials before
// they are summed, so nothing needs clearing between calls; calls that
// overlap on one device race on the array.
constexpr long long kScratchBlocks = 16384;                 // 4,194,304 pixels of 256-pixel blocks
static __device__ __align__(256) double scratch[3 * kScratchBlocks];   // 384 KiB

namespace {
std::mutex g_scratch_mu;
constexpr int kMaxDevices = 64;
double *g_scratch_ptr[kMaxDevices] = {};
}

long long rsample_static_max_pixels() { return kScratchBlocks * kRsBlock; }

hipError_t launch_rsample_static(const double *b, const double *p1, const double *p2, const double *pt,
                                 const uint8_t *nc, int NX, int NY, int px, int py, int H, int W, float s_r,
                                 float s_v, float s_d, uint16_t *x, uint16_t *t, double *stats, hipStream_t s) {
    double *part = nullptr;
    if (stats) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (s) {
            hipDevice_t sd = 0;
            if ((e = hipStreamGetDevice(s, &sd)) != hipSuccess) return e;
            if (sd != dev) return hipErrorInvalidDevice;      // the lookup needs the stream's device current
        }
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            void *ptr = nullptr;
            if ((e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) != hipSuccess) return e;
            g_scratch_ptr[dev] = static_cast<double *>(ptr);
        }
        part = g_scratch_ptr[dev];
    }
    launch_rsample(b, p1, p2, pt, nc, NX, NY, px, py, H, W, s_r, s_v, s_d, x, t, stats, part, s);
    return hipGetLastError();
}

// A stored sample into a batch slot: the input as it is; with t, the target
// (bfloat16 -> float32) and the loss mask (the free-node channel).
__global__ void k_load(const uint16_t *xs, const uint16_t *ts, long long P, uint16_t *x, float *target,
                       float *mask) {
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    x[3 * p + 0] = xs[3 * p + 0];
    x[3 * p + 1] = xs[3 * p + 1];
    x[3 * p + 2] = xs[3 * p + 2];
    if (ts) {
        target[p] = bf2f(ts[p]);
        mask[p] = xs[3 * p + 1] ? 1.f : 0.f;
    }
}

void launch_load(const uint16_t *xs, const uint16_t *ts, long long P, uint16_t *x, float *target, float *mask,
                 hipStream_t s) {
    hipLaunchKernelGGL(k_load, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, xs, ts, P, x, target, mask);
}

// guess = phi_s + out / s_d on free nodes of the window (use_out), phi_s elsewhere.
__global__ void k_rguess(const float *out, const double *p1, const double *p2, const uint8_t *nc, int NX,
                         int NY, int H, int W, float s_d, int use_out, double *guess) {
    const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (long long)NX * NY) return;
    const int i = (int)(n / NY), j = (int)(n % NY);
    double v = start_at(p1, p2, n);
    if (use_out && nc[n] == 0 && i < H && j < W) v += (double)out[(long long)i * W + j] / (double)s_d;
    guess[n] = v;
}

void launch_rguess(const float *out, const double *p1, const double *p2, const uint8_t *nc, int NX, int NY,
                   int H, int W, float s_d, int use_out, double *guess, hipStream_t s) {
    const long long n = (long long)NX * NY;
    hipLaunchKernelGGL(k_rguess, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, p1, p2, nc, NX, NY,
                       H, W, s_d, use_out, guess);
}

// ---- time extrapolation of the potential ------------------------------------
// out = coef[0] phi[0] + coef[1] phi[1] + ... (added in this order).
__global__ void k_extrapolate_k(ExtrapArgs a) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    double s = a.c[0] * a.p[0][i];
    for (int k = 1; k < a.K; ++k) s = s + a.c[k] * a.p[k][i];
    a.out[i] = s;
}

void launch_extrapolate(const ExtrapArgs &a, hipStream_t s) {
    if (a.n <= 0) return;
    hipLaunchKernelGGL(k_extrapolate_k, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a);
}

// ---- coarse residual learning -----------------------------------------------
// Pixel (h, w) of the network stands for the f x f block of nodes
// (h f + p, w f + q), p, q < f (f divides 16), so the network's receptive
// field spans the whole grid.  Input x [H][W][3] = (bf16(R/f^2 s_r),
// bf16(F/f^2), bf16(V/f^2 s_v)) and target t [H][W] = bf16(D/f^2 s_d), with
// R, D, F the sums over the block's free nodes of the residual r of the
// extrapolated start, of (phi_t - phi_s) and of 1, and V the sum of the
// Dirichlet values of its conductor nodes; every sum adds the block's nodes
// in row-major order (p outer, q inner), starting from 0.  One block of 256
// threads covers a 16 x 16 tile of nodes: each thread computes one node's
// terms into LDS, then one thread per pixel of the tile adds its block.
// part (may be null): per-block sums, in pixel order, of (R/f^2)^2,
// (D/f^2)^2 and the count of pixels with a free node.
constexpr int kCsTile = 16;

__global__ __launch_bounds__(256) void k_csample(const double *b, const double *p1, const double *p2,
                                                 const double *pt, const uint8_t *nc, int NX, int NY, int px,
                                                 int py, int f, int H, int W, float s_r, float s_v, float s_d,
                                                 uint16_t *x, uint16_t *t, double *part) {
    __shared__ double sr[kCsTile * kCsTile], sv[kCsTile * kCsTile], sd[kCsTile * kCsTile];
    __shared__ unsigned char sf[kCsTile * kCsTile];
    __shared__ double st[3][kCsTile * kCsTile];
    const int tid = threadIdx.x;
    const int tiles_w = (W * f + kCsTile - 1) / kCsTile;
    const int bi = blockIdx.x / tiles_w, bj = blockIdx.x % tiles_w;
    const int i = bi * kCsTile + tid / kCsTile, j = bj * kCsTile + tid % kCsTile;
    double r = 0.0, v = 0.0, d = 0.0;
    unsigned char fr = 0;
    if (i < H * f && j < W * f) {
        const long long n = (long long)i * NY + j;
        if (nc[n] == 0) {
            double s = 4.0 * start_at(p1, p2, n);
            const int im = i - 1 < 0 ? (px ? NX - 1 : -1) : i - 1;
            const int ip = i + 1 >= NX ? (px ? 0 : -1) : i + 1;
            const int jm = j - 1 < 0 ? (py ? NY - 1 : -1) : j - 1;
            const int jp = j + 1 >= NY ? (py ? 0 : -1) : j + 1;
            long long q;
            if (im >= 0 && !nc[q = (long long)im * NY + j]) s -= start_at(p1, p2, q);
            if (ip >= 0 && !nc[q = (long long)ip * NY + j]) s -= start_at(p1, p2, q);
            if (jm >= 0 && !nc[q = (long long)i * NY + jm]) s -= start_at(p1, p2, q);
            if (jp >= 0 && !nc[q = (long long)i * NY + jp]) s -= start_at(p1, p2, q);
            r = b[n] - s;
            if (pt) d = pt[n] - start_at(p1, p2, n);
            fr = 1;
        } else {
            v = b[n];
        }
    }
    sr[tid] = r;
    sv[tid] = v;
    sd[tid] = d;
    sf[tid] = fr;
    __syncthreads();
    const int per = kCsTile / f;                 // pixels per tile edge
    double q0 = 0.0, q1 = 0.0, q2 = 0.0;
    if (tid < per * per) {
        const int a = tid / per, c = tid % per;
        const int h = bi * per + a, w = bj * per + c;
        if (h < H && w < W) {
            double R = 0.0, V = 0.0, D = 0.0, F = 0.0;
            for (int pp = 0; pp < f; ++pp)
                for (int qq = 0; qq < f; ++qq) {
                    const int l = (a * f + pp) * kCsTile + (c * f + qq);
                    if (sf[l]) {
                        R += sr[l];
                        D += sd[l];
                        F += 1.0;
                    } else {
                        V += sv[l];
                    }
                }
            const double inv = 1.0 / (double)(f * f);
            const long long p = (long long)h * W + w;
            const double rm = R * inv, dm = D * inv;
            x[3 * p + 0] = (uint16_t)f2bf((float)(rm * (double)s_r));
            x[3 * p + 1] = (uint16_t)f2bf((float)(F * inv));
            x[3 * p + 2] = (uint16_t)f2bf((float)(V * inv * (double)s_v));
            if (t) t[p] = (uint16_t)f2bf((float)(dm * (double)s_d));
            q0 = rm * rm;
            q1 = dm * dm;
            q2 = F > 0.0 ? 1.0 : 0.0;
        }
    }
    if (part) {
        st[0][tid] = q0;
        st[1][tid] = q1;
        st[2][tid] = q2;
        __syncthreads();
        if (tid == 0) {
            double a0 = 0.0, a1 = 0.0, a2 = 0.0;
            for (int k = 0; k < per * per; ++k) {
                a0 += st[0][k];
                a1 += st[1][k];
                a2 += st[2][k];
            }
            part[3 * (long long)blockIdx.x + 0] = a0;
            part[3 * (long long)blockIdx.x + 1] = a1;
            part[3 * (long long)blockIdx.x + 2] = a2;
        }
    }
}

long long csample_blocks(int f, int H, int W) {
    return (long long)((H * f + kCsTile - 1) / kCsTile) * ((W * f + kCsTile - 1) / kCsTile);
}

void launch_csample(const double *b, const double *p1, const double *p2, const double *pt, const uint8_t *nc,
                    int NX, int NY, int px, int py, int f, int H, int W, float s_r, float s_v, float s_d,
                    uint16_t *x, uint16_t *t, double *stats, double *part, hipStream_t s) {
    const long long nb = csample_blocks(f, H, W);
    hipLaunchKernelGGL(k_csample, dim3((unsigned)nb), dim3(kCsTile * kCsTile), 0, s, b, p1, p2, pt, nc, NX, NY,
                       px, py, f, H, W, s_r, s_v, s_d, x, t, stats ? part : nullptr);
    if (stats) hipLaunchKernelGGL(k_rsample_sum, dim3(1), dim3(64), 0, s, part, (int)nb, stats);
}

// Lower and upper pixel of node index i on an axis of n pixels of f nodes and
// the upper pixel's weight: the node lies at pixel coordinate (i + 1/2)/f - 1/2
// (pixel centres at integers); beyond [0, n - 1] the index wraps (wrap) or is
// clamped to the edge pixel.
__device__ __forceinline__ void axis_weights(int i, int f, int n, bool wrap, int &lo, int &hi, double &a) {
    const double u = ((double)i + 0.5) / (double)f - 0.5;
    const double fl = floor(u);
    a = u - fl;
    lo = (int)fl;
    hi = lo + 1;
    if (wrap) {
        lo = lo < 0 ? lo + n : lo;
        hi = hi >= n ? hi - n : hi;
    } else {
        lo = min(max(lo, 0), n - 1);
        hi = min(max(hi, 0), n - 1);
    }
}

// guess = phi_s + c / s_d on the free nodes of the covered H f x W f region
// (use_out), c the bilinear interpolation of the coarse output, weights
// (1-a)(1-b), a(1-b), (1-a)b, ab added in that order; phi_s elsewhere.  An
// axis wraps when it is periodic and covered exactly.
__global__ void k_cguess(const float *out, const double *p1, const double *p2, const uint8_t *nc, int NX,
                         int NY, int px, int py, int f, int H, int W, float s_d, int use_out, double *guess) {
    const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (long long)NX * NY) return;
    const int i = (int)(n / NY), j = (int)(n % NY);
    double v = start_at(p1, p2, n);
    if (use_out && nc[n] == 0 && i < H * f && j < W * f) {
        int h0, h1, w0, w1;
        double a, bq;
        axis_weights(i, f, H, px && H * f == NX, h0, h1, a);
        axis_weights(j, f, W, py && W * f == NY, w0, w1, bq);
        double c = (1.0 - a) * (1.0 - bq) * (double)out[(long long)h0 * W + w0];
        c = c + a * (1.0 - bq) * (double)out[(long long)h1 * W + w0];
        c = c + (1.0 - a) * bq * (double)out[(long long)h0 * W + w1];
        c = c + a * bq * (double)out[(long long)h1 * W + w1];
        v = v + c / (double)s_d;
    }
    guess[n] = v;
}

void launch_cguess(const float *out, const double *p1, const double *p2, const uint8_t *nc, int NX, int NY,
                   int px, int py, int f, int H, int W, float s_d, int use_out, double *guess, hipStream_t s) {
    const long long n = (long long)NX * NY;
    hipLaunchKernelGGL(k_cguess, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, p1, p2, nc, NX, NY, px,
                       py, f, H, W, s_d, use_out, guess);
}

} // namespace unet
