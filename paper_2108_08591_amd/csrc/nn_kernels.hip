// nn_kernels.hip -- gfx950 kernels of the convolutional encoder-decoder used
// to warm-start steady MDF-LBM solves (C ABI: include/mdfnn.h).
//
// 3x3 convolutions are implicit GEMMs on the matrix cores:
//   forward / data gradient:  M = pixels, N = output channels, K = 9 * cin,
//   weight gradient:          M = cout,   N = cin (per tap),   K = pixels,
// each a sum of v_mfma_f32_16x16x32_bf16 products (BF16 operands, FP32
// accumulation).  For that instruction lane l of a wave holds
//   A[l % 16][8 (l / 16) + j], B[8 (l / 16) + j][l % 16]   (j = 0..7)
//   C[4 (l / 16) + r][l % 16]                              (r = 0..3).
// Activations are NHWC, so one K step of 32 of the forward product (one
// tap, 32 consecutive channels) is one 16-byte chunk per pixel and weight
// row, staged through LDS as [row][32 channels]; the weight gradient, whose
// K steps are 32 pixels, stages its tiles as they lie in memory and transposes
// them as it reads them from LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "mdfnn.h"
#include "nn_rules.h"

namespace mdfnn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

__device__ __forceinline__ uint16_t f2bf(float v)
{
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ bf16x8 load8(const uint16_t *p)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ bf16x8 zero8()
{
    const uint4 v = {0u, 0u, 0u, 0u};
    return __builtin_bit_cast(bf16x8, v);
}

// ------------------------------------------------------------------ conv fwd

// LDS-staged implicit GEMM for the forward and data-gradient products, in
// runs of 128 pixels that ignore the image's rows: where its wide blocks pay
// (nn_rules.h), and for outputs not aligned to 8 bytes.
// Block: 4 waves, a 128-pixel x BN-channel output tile; wave (wm, wn) owns
// pixels [64 wm, +64) and channels [wn BN/2, +BN/2) as 4 x (BN/32) MFMA
// blocks of 16 x 16.  Each K step (one tap, 32 input channels) stages the
// shifted 128 x 32 input tile and the BN x 32 weight tile in LDS, every
// global value read once per block; the next step's global loads are
// issued before the current step's products (double-buffered LDS, one
// barrier per step).  Rows of the LDS tiles are 32 + 8 values long, so
// the 16 rows one MFMA operand reads start in distinct banks.
constexpr int kCvBM = 128;
constexpr int kCvLd = 40;

template <int BN>
__global__ void __launch_bounds__(256)
k_conv_fwd_lds(const uint16_t *__restrict__ x1, int c1, const uint16_t *__restrict__ x2, int c2,
               const uint16_t *__restrict__ w, const float *__restrict__ bias, int B, int H, int W, int cout,
               int relu, const uint16_t *__restrict__ mask, uint16_t *__restrict__ yb, float *__restrict__ yf)
{
    constexpr int NBW = BN / 32;                 // 16-wide channel blocks per wave
    __shared__ uint4 sA4[2][kCvBM * kCvLd / 8];
    __shared__ uint4 sB4[2][BN * kCvLd / 8];
    const int cin = c1 + c2;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int i = lane & 15, g = lane >> 4, wm = wave >> 1, wn = wave & 1;
    const long long M = (long long)B * H * W;
    const long long pbase = (long long)blockIdx.x * kCvBM;
    const int co0 = blockIdx.y * BN;
    // staging roles: input rows (2 per thread: pixel t / 4 and t / 4 + 64,
    // channel chunk t % 4), weight rows (co = idx / 4, chunk idx % 4)
    const int ach = t & 3;
    int spb[2], spy[2], spx[2];
    bool spv[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const long long p = pbase + (t >> 2) + 64 * r;
        spv[r] = p < M;
        const long long pp = spv[r] ? p : 0;
        spb[r] = (int)(pp / ((long long)H * W));
        const int rem = (int)(pp % ((long long)H * W));
        spy[r] = rem / W;
        spx[r] = rem % W;
    }
    const int nk = 9 * (cin / 32);
    uint4 ra[2], rb0 = uint4{0u, 0u, 0u, 0u}, rb1 = uint4{0u, 0u, 0u, 0u};
    auto fetch = [&](int ks) __attribute__((always_inline)) {
        const int tap = ks / (cin / 32), c0 = (ks % (cin / 32)) * 32;
        const int dy = tap / 3 - 1, dx = tap % 3 - 1;
        const uint16_t *src = (c0 < c1) ? x1 : x2;
        const int cs = (c0 < c1) ? c1 : c2;
        const int cc = (c0 < c1) ? c0 : c0 - c1;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int yy = spy[r] + dy, xx = spx[r] + dx;
            ra[r] = uint4{0u, 0u, 0u, 0u};
            if (spv[r] && yy >= 0 && yy < H && xx >= 0 && xx < W)
                ra[r] = *reinterpret_cast<const uint4 *>(src + (((long long)spb[r] * H + yy) * W + xx) * cs + cc +
                                                        8 * ach);
        }
        const uint16_t *wk = w + (long long)tap * cin + c0 + 8 * (t & 3);
        if (BN * 4 >= 256 || t < BN * 4) rb0 = *reinterpret_cast<const uint4 *>(wk + (long long)(co0 + (t >> 2)) * 9 * cin);
        if constexpr (BN * 4 > 256)
            rb1 = *reinterpret_cast<const uint4 *>(wk + (long long)(co0 + 64 + (t >> 2)) * 9 * cin);
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 2; ++r) sA4[buf][((t >> 2) + 64 * r) * (kCvLd / 8) + ach] = ra[r];
        if (BN * 4 >= 256 || t < BN * 4) sB4[buf][(t >> 2) * (kCvLd / 8) + (t & 3)] = rb0;
        if constexpr (BN * 4 > 256) sB4[buf][(64 + (t >> 2)) * (kCvLd / 8) + (t & 3)] = rb1;
    };
    f32x4 acc[4][NBW];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < NBW; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
    stash(0);
    __syncthreads();
    for (int ks = 0; ks < nk; ++ks) {
        const int buf = ks & 1;
        if (ks + 1 < nk) fetch(ks + 1);
        bf16x8 fa[4], fb[NBW];
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
            fa[mb] = __builtin_bit_cast(bf16x8, sA4[buf][(wm * 64 + 16 * mb + i) * (kCvLd / 8) + g]);
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
            fb[nb] = __builtin_bit_cast(bf16x8, sB4[buf][(wn * (BN / 2) + 16 * nb + i) * (kCvLd / 8) + g]);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb)
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[mb], fb[nb], acc[mb][nb], 0, 0, 0);
        if (ks + 1 < nk) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const long long p = pbase + wm * 64 + 16 * mb + 4 * g + r;
                const int co = co0 + wn * (BN / 2) + 16 * nb + i;
                if (p >= M) continue;
                float v = acc[mb][nb][r];
                if (bias) v += bias[co];
                if (relu) v = v > 0.f ? v : 0.f;
                const long long k = p * cout + co;
                if (mask && !(bf2f(mask[k]) > 0.f)) v = 0.f;
                if (yb) yb[k] = f2bf(v);
                if (yf) yf[k] = v;
            }
}

// Four consecutive output channels at k: bias, ReLU, mask, then BF16 (8-byte
// stores) or FP32 (16).
__device__ __forceinline__ void conv_out(const f32x4 &acc, const float *__restrict__ bias, int relu,
                                         const uint16_t *__restrict__ mask, uint16_t *__restrict__ yb,
                                         float *__restrict__ yf, long long k)
{
    uint16_t vm[4] = {0, 0, 0, 0}, vb[4];
    float v[4];
    if (mask) {
        const uint2 q = *reinterpret_cast<const uint2 *>(mask + k);
        __builtin_memcpy(vm, &q, 8);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        v[r] = acc[r];
        if (bias) v[r] += bias[r];
        if (relu && !(v[r] > 0.f)) v[r] = 0.f;
        if (mask && !(bf2f(vm[r]) > 0.f)) v[r] = 0.f;
        vb[r] = f2bf(v[r]);
    }
    if (yb) {
        uint2 q;
        __builtin_memcpy(&q, vb, 8);
        *reinterpret_cast<uint2 *>(yb + k) = q;
    }
    if (yf) *reinterpret_cast<float4 *>(yf + k) = float4{v[0], v[1], v[2], v[3]};
}

// The same products in smaller blocks, more of them per CU: 4 waves, two along
// the pixels (a run of 128) and two along BN output channels, the channels
// along M, so that a lane ends with four consecutive channels of a pixel,
// written as 8 bytes.  Rows of the LDS tiles are not padded: their 16-byte
// chunks are permuted by the row, so that eight consecutive rows' reads of one
// chunk lie in distinct banks; 24 KB and 88 registers (BN = 64) leave room for
// five blocks, whose products cover each other's barriers and loads.  Whether a tap of a staged
// pixel lies inside the image is a bit of a mask formed once.  The chunks of a
// tap follow each other and the taps as in k_conv_fwd_lds: the sums are the
// same bits.  (K steps of 64 channels, or 64 x 64 products per wave, need fewer
// barriers and LDS reads but leave two blocks per CU: 16 x 128 x 128 pixels, 192
// -> 64 channels 189 and 206 us, against 153 as it is.)
__device__ __forceinline__ int conv_chunk(int row, int c) { return row * 4 + (c ^ ((row >> 2) & 3)); }

template <int BN>
__global__ void __launch_bounds__(256)
k_conv_fwd_run(const uint16_t *__restrict__ x1, int c1, const uint16_t *__restrict__ x2, int c2,
               const uint16_t *__restrict__ w, const float *__restrict__ bias, int B, int H, int W, int cout, int relu,
               const uint16_t *__restrict__ mask, uint16_t *__restrict__ yb, float *__restrict__ yf)
{
    constexpr int PX = 128, MB = BN / 32, CH = 4;
    constexpr int KA = PX * CH / 256, KW = (BN * CH + 255) / 256, RS = 256 / CH;     // rows a pass of the block stages
    __shared__ uint4 sA4[2][PX * CH];
    __shared__ uint4 sB4[2][BN * CH];
    const int cin = c1 + c2;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int i = lane & 15, g = lane >> 4, wm = wave & 1, wn = wave >> 1;
    const long long M = (long long)B * H * W;
    const long long pbase = (long long)blockIdx.x * PX;
    const int co0 = blockIdx.y * BN;
    const int ch = t % CH, row0 = t / CH;
    long long pix[KA];              // pixel index of each staged row
    unsigned inside[KA];            // bit tap: the tap's pixel lies in the image
#pragma unroll
    for (int r = 0; r < KA; ++r) {
        const long long p = pbase + row0 + RS * r;
        const long long pp = p < M ? p : 0;
        const int rem = (int)(pp % ((long long)H * W));
        const int y = rem / W, x = rem % W;
        pix[r] = pp;
        inside[r] = 0;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
            if (p < M && yy >= 0 && yy < H && xx >= 0 && xx < W) inside[r] |= 1u << tap;
        }
    }
    const int nk = 9 * (cin / 32);
    uint4 ra[KA], rw[KW];
    int tap = 0, c0 = 0;            // of the next step to fetch
    auto fetch = [&]() __attribute__((always_inline)) {
        const bool first = c0 < c1;
        const uint16_t *src = first ? x1 : x2;
        const int cs = first ? c1 : c2, cc = first ? c0 : c0 - c1;
        const int shift = (tap / 3 - 1) * W + tap % 3 - 1;
#pragma unroll
        for (int r = 0; r < KA; ++r) {
            ra[r] = uint4{0u, 0u, 0u, 0u};
            if ((inside[r] >> tap) & 1u)
                ra[r] = *reinterpret_cast<const uint4 *>(src + (pix[r] + shift) * cs + cc + 8 * ch);
        }
        const uint16_t *wk = w + (long long)tap * cin + c0 + 8 * ch;
#pragma unroll
        for (int r = 0; r < KW; ++r)
            if (BN * CH % 256 == 0 || row0 + RS * r < BN)
                rw[r] = *reinterpret_cast<const uint4 *>(wk + (long long)(co0 + row0 + RS * r) * 9 * cin);
        c0 += 32;
        if (c0 == cin) { c0 = 0; ++tap; }
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < KA; ++r) sA4[buf][conv_chunk(row0 + RS * r, ch)] = ra[r];
#pragma unroll
        for (int r = 0; r < KW; ++r)
            if (BN * CH % 256 == 0 || row0 + RS * r < BN) sB4[buf][conv_chunk(row0 + RS * r, ch)] = rw[r];
    };
    f32x4 acc[MB][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch();
    stash(0);
    __syncthreads();
    for (int ks = 0; ks < nk; ++ks) {
        const int buf = ks & 1;
        if (ks + 1 < nk) fetch();
        bf16x8 fw[MB], fx[4];
#pragma unroll
        for (int m = 0; m < MB; ++m) fw[m] = __builtin_bit_cast(bf16x8, sB4[buf][conv_chunk((wn * MB + m) * 16 + i, g)]);
#pragma unroll
        for (int n = 0; n < 4; ++n) fx[n] = __builtin_bit_cast(bf16x8, sA4[buf][conv_chunk(wm * 64 + 16 * n + i, g)]);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n)
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[m], fx[n], acc[m][n], 0, 0, 0);
        if (ks + 1 < nk) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const long long p = pbase + wm * 64 + 16 * n + i;
        if (p >= M) continue;
        const long long base = p * cout + co0 + wn * MB * 16 + 4 * g;
#pragma unroll
        for (int m = 0; m < MB; ++m)
            conv_out(acc[m][n], bias ? bias + co0 + (wn * MB + m) * 16 + 4 * g : nullptr, relu, mask, yb, yf, base + 16 * m);
    }
}

// The same products for 32 input channels from a two-dimensional pixel tile.
// Block: 4 waves, 16 x 16 pixels of one image by 32 output channels; wave v
// owns rows [4v, +4) of the tile and all 32 channels as 2 x 4 MFMA blocks, the
// channels along M, so that a lane ends with four consecutive channels of one
// pixel.  The block stages the 18 x 18 input pixels around the tile and the
// weights of all nine taps (32 x 9 x 32) in LDS once and takes the nine taps'
// products from there: an input value is read from global memory 1.3 times
// instead of nine times, and one barrier serves 72 products per wave.  With one chunk of 32 channels the taps follow each other
// as in k_conv_fwd_lds, so the sums are the same bits; with more, taking a
// chunk's nine taps together would change their order.
// 16 x 256 x 256 pixels, 32 -> 32 channels: 66 us (130 us in runs of 128 pixels),
// bound by the latency of a block's only loads, three blocks per CU.  (64 output
// channels a block, two blocks per CU: 32 -> 64 channels, 1024 pixels 15.4 and 9.2
// us, 2^18 pixels 39.0 and 34.9, 2^20 pixels 139 and 116.)
constexpr int kTlPx = 18 * 18;

__global__ void __launch_bounds__(256, 3)
k_conv_fwd_tile(const uint16_t *__restrict__ x, const uint16_t *__restrict__ w, const float *__restrict__ bias, int H, int W,
                int gx, int gy, int cout,
                int relu, const uint16_t *__restrict__ mask, uint16_t *__restrict__ yb, float *__restrict__ yf)
{
    constexpr int BN = 32, MB = BN / 16;
    constexpr int NA = kTlPx * 4, KA = (NA + 255) / 256;      // 16-byte chunks of input, per thread
    constexpr int NW = 9 * BN * 4, KW = (NW + 255) / 256;     // of weights
    __shared__ uint4 sA4[kTlPx * kCvLd / 8];
    __shared__ uint4 sW4[9 * BN * kCvLd / 8];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int b = blockIdx.x / (gx * gy), tile = blockIdx.x % (gx * gy);
    const int tx0 = (tile % gx) * 16, ty0 = (tile / gx) * 16;
    const int co0 = blockIdx.y * BN;
    uint4 ra[KA], rw[KW];
#pragma unroll
    for (int r = 0; r < KA; ++r) {
        const int idx = t + 256 * r;
        const int px = idx >> 2, ch = idx & 3;
        const int yy = ty0 - 1 + px / 18, xx = tx0 - 1 + px % 18;
        ra[r] = uint4{0u, 0u, 0u, 0u};
        if (idx < NA && yy >= 0 && yy < H && xx >= 0 && xx < W)
            ra[r] = *reinterpret_cast<const uint4 *>(x + (((long long)b * H + yy) * W + xx) * 32 + 8 * ch);
    }
#pragma unroll
    for (int r = 0; r < KW; ++r) {
        const int idx = t + 256 * r;
        rw[r] = uint4{0u, 0u, 0u, 0u};
        if (NW % 256 == 0 || idx < NW)
            rw[r] = *reinterpret_cast<const uint4 *>(w + ((long long)(co0 + (idx >> 2) % BN) * 9 + (idx >> 2) / BN) * 32 +
                                                    8 * (idx & 3));
    }
#pragma unroll
    for (int r = 0; r < KA; ++r) {
        const int idx = t + 256 * r;
        if (idx < NA) sA4[(idx >> 2) * (kCvLd / 8) + (idx & 3)] = ra[r];
    }
#pragma unroll
    for (int r = 0; r < KW; ++r) {
        const int idx = t + 256 * r;
        if (NW % 256 == 0 || idx < NW) sW4[(idx >> 2) * (kCvLd / 8) + (idx & 3)] = rw[r];
    }
    f32x4 acc[MB][4];
    const uint16_t *sA = reinterpret_cast<const uint16_t *>(sA4), *sW = reinterpret_cast<const uint16_t *>(sW4);
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const int dy = tap / 3, dx = tap % 3;
        bf16x8 fw[MB], fx[4];
#pragma unroll
        for (int m = 0; m < MB; ++m) fw[m] = load8(sW + (tap * BN + 16 * m + i) * kCvLd + 8 * g);
#pragma unroll
        for (int n = 0; n < 4; ++n) fx[n] = load8(sA + ((4 * wave + n + dy) * 18 + i + dx) * kCvLd + 8 * g);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n)
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[m], fx[n], acc[m][n], 0, 0, 0);
    }
    const int xx = tx0 + i;
    if (xx >= W) return;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int yy = ty0 + 4 * wave + n;
        if (yy >= H) continue;
        const long long base = (((long long)b * H + yy) * W + xx) * cout + co0 + 4 * g;
#pragma unroll
        for (int m = 0; m < MB; ++m)
            conv_out(acc[m][n], bias ? bias + co0 + 16 * m + 4 * g : nullptr, relu, mask, yb, yf, base + 16 * m);
    }
}

// wt[ci][tap][co] = w[co][8 - tap][ci]
__global__ void __launch_bounds__(256) k_flip(const uint16_t *__restrict__ w, int cout, int cin, uint16_t *__restrict__ wt)
{
    const long long n = (long long)cout * 9 * cin;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const int ci = (int)(k / (9LL * cout));
        const int rem = (int)(k % (9LL * cout));
        const int tap = rem / cout, co = rem % cout;
        wt[k] = w[((long long)co * 9 + (8 - tap)) * cin + ci];
    }
}

// ------------------------------------------------------------------ weight grad

constexpr int kWgBlocks = 1024;    // target blocks of one weight-gradient launch

// LDS tiles of the weight gradient, [pixel row][C channels] without padding:
// the 32-byte groups of 16 channels of a row are permuted by the row (an
// exclusive or), so that the eight rows r, .. r + 3 and r + 8, .. r + 11 that
// half a wavefront reads at once lie in distinct banks for any r.
template <int C>
__device__ __forceinline__ int swz(int row)
{
    return C == 64 ? ((row >> 1) & 1) | ((row >> 2) & 2) : (row >> 3) & 1;
}

// 16-byte chunk c8 of a row, as an index of such chunks.
template <int C>
__device__ __forceinline__ int chunk_at(int row, int c8)
{
    return row * (C / 8) + (c8 ^ (swz<C>(row) << 1));
}

// Rows r, .. r + 3, channels 16 grp .. 16 grp + 15, transposed: the lane gets its
// channel (lane % 16) of the four rows.  Each lane of a group of 16 addresses
// 8 of the group's 128 bytes, the read hands them out by column.
template <int C>
__device__ __forceinline__ uint2 rows4(const uint16_t *p, int r, int grp, int i)
{
    typedef short s4 __attribute__((ext_vector_type(4)));
    using L4 = __attribute__((address_space(3))) s4;
    const int row = r + (i >> 2);
    const s4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L4 *)(p + row * C + 16 * (grp ^ swz<C>(row)) + 4 * (i & 3)));
    return __builtin_bit_cast(uint2, v);
}

// MFMA operand of the 32 pixels from row r on and 16 channels: K index 8 g + j
// is pixel 8 g + j.
template <int C>
__device__ __forceinline__ bf16x8 rows32(const uint16_t *p, int r, int grp, int i, int g)
{
    const uint2 a = rows4<C>(p, r + 8 * g, grp, i), b = rows4<C>(p, r + 8 * g + 4, grp, i);
    return __builtin_bit_cast(bf16x8, uint4{a.x, a.y, b.x, b.y});
}

// Weight gradient with all nine taps in one block.  The K dimension (pixels)
// is walked in segments of 32 consecutive pixels of one image row; per
// segment the block stages the output-gradient row segment (MT channels)
// and the input window of rows y-1..y+1 and 34 pixels (NT channels) in LDS as
// they lie in memory, [pixel][channel], and takes the products of all nine
// taps from there with the transposing LDS read: a tap is an offset of whole
// rows.  Two LDS buffers, one barrier per segment, the next segment's global loads in flight during the
// products.  NT = 64: wave v owns all MT output channels by input channels
// [16 v, +16); NT = 32: waves (wm, wn) own halves of MT by 16.  Pixels beyond
// the row end contribute zero (their dy is staged as zero); input pixels
// outside the image are zero.  Segments [s0, s1) of split blockIdx.z; partial
// sums per split are reduced in a fixed order by k_wgrad_reduce.
// Bound by the products and, behind them, the LDS reads (26 of 8 bytes per
// lane for 36 products).  16 x 128 x 128 pixels, 192 -> 64 channels: 332 us when
// the tiles were staged transposed, value by value, in three shifted copies,
// 135 us now (430 TFLOP/s).
template <int MT, int NT>
__global__ void __launch_bounds__(256, 2)
k_conv_wgrad9(const uint16_t *__restrict__ x1, int c1, const uint16_t *__restrict__ x2, int c2,
              const uint16_t *__restrict__ dyp, int B, int H, int W, int cout, int nsplit,
              float *__restrict__ partial, float *__restrict__ bpart)
{
    constexpr int MB = (NT == 64) ? MT / 16 : MT / 32;
    constexpr int NDY = 32 * MT / 8;                    // 16-byte dy chunks per segment
    constexpr int NX = 3 * 34 * NT / 8;                 // 16-byte input chunks per window
    constexpr int KX = (NX + 255) / 256;
    __shared__ uint4 ys4[2][32 * MT / 8];
    __shared__ uint4 xw4[2][3 * 34 * NT / 8];
    const int cin = c1 + c2;
    const int co0 = blockIdx.x * MT, ci0 = blockIdx.y * NT;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int wm = (NT == 64) ? 0 : wave >> 1, wn = (NT == 64) ? wave : wave & 1;
    const uint16_t *src = (ci0 < c1) ? x1 : x2;
    const int cs = (ci0 < c1) ? c1 : c2;
    const int cc = (ci0 < c1) ? ci0 : ci0 - c1;
    const int S = (W + 31) / 32;                        // segments per image row
    const long long nseg = (long long)B * H * S;
    const long long per = (nseg + nsplit - 1) / nsplit;
    const long long s0 = blockIdx.z * per, s1 = (s0 + per < nseg) ? s0 + per : nseg;
    f32x4 acc[9][MB];
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int a = 0; a < MB; ++a) acc[k][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 rdy, rx[KX];
    // bias gradient (blocks of the first input-channel tile): the thread that
    // stages dy chunk (pixel j, channels 8 c8 ..) sums those channels over the
    // block's segments; the 32 pixel slots are added in order at the end
    const bool bias = bpart != nullptr && blockIdx.y == 0;
    float bacc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bacc[e] = 0.f;
    auto fetch = [&](long long sg) __attribute__((always_inline)) {
        const int xs = (int)(sg % S) * 32;
        const long long row = sg / S;                   // b * H + y
        const int y = (int)(row % H);
        rdy = uint4{0u, 0u, 0u, 0u};
        if (t < NDY) {
            const int j = t / (MT / 8), c8 = t % (MT / 8);
            if (xs + j < W) rdy = *reinterpret_cast<const uint4 *>(dyp + (row * W + xs + j) * cout + co0 + 8 * c8);
        }
#pragma unroll
        for (int r = 0; r < KX; ++r) {
            const int idx = t + 256 * r;
            rx[r] = uint4{0u, 0u, 0u, 0u};
            if (idx < NX) {
                const int wr = idx / (34 * NT / 8), rem = idx % (34 * NT / 8);
                const int c = rem / (NT / 8), c8 = rem % (NT / 8);
                const int yy = y - 1 + wr, xx = xs - 1 + c;
                if (yy >= 0 && yy < H && xx >= 0 && xx < W)
                    rx[r] = *reinterpret_cast<const uint4 *>(src + ((row - y + yy) * W + xx) * cs + cc + 8 * c8);
            }
        }
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
        if (t < NDY) {
            ys4[buf][chunk_at<MT>(t / (MT / 8), t % (MT / 8))] = rdy;
            if (bias) {
                const uint16_t *u = reinterpret_cast<const uint16_t *>(&rdy);
#pragma unroll
                for (int e = 0; e < 8; ++e) bacc[e] += bf2f(u[e]);
            }
        }
#pragma unroll
        for (int r = 0; r < KX; ++r) {
            const int idx = t + 256 * r;
            if (idx < NX) xw4[buf][chunk_at<NT>(idx / (NT / 8), idx % (NT / 8))] = rx[r];
        }
    };
    if (s0 < s1) {
        fetch(s0);
        stash(0);
    }
    __syncthreads();
    for (long long sg = s0; sg < s1; ++sg) {
        const int buf = (int)(sg - s0) & 1;
        if (sg + 1 < s1) fetch(sg + 1);
        const uint16_t *ys = reinterpret_cast<const uint16_t *>(ys4[buf]);
        const uint16_t *xw = reinterpret_cast<const uint16_t *>(xw4[buf]);
        bf16x8 fa[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) fa[mb] = rows32<MT>(ys, 0, wm * (MT / 32) + mb, i, g);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const bf16x8 fb = rows32<NT>(xw, (tap / 3) * 34 + tap % 3, wn, i, g);     // dy = tap / 3 - 1, dx = tap % 3 - 1
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[tap][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[mb], fb, acc[tap][mb], 0, 0, 0);
        }
        if (sg + 1 < s1) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = co0 + wm * (MT / 2) + 16 * mb + 4 * g + r;
                const int ci = ci0 + 16 * wn + i;
                partial[(((long long)blockIdx.z * cout + co) * 9 + tap) * cin + ci] = acc[tap][mb][r];
            }
    if (bias) {
        // the window is free (a barrier ends the loop): reuse it as [pixel slot][co] floats
        float *red = reinterpret_cast<float *>(&xw4[0][0]);
        static_assert(32 * MT * sizeof(float) <= sizeof(xw4), "bias slots fit the input window");
        if (t < NDY) {
            const int j = t / (MT / 8), c8 = t % (MT / 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) red[j * MT + 8 * c8 + e] = bacc[e];
        }
        __syncthreads();
        if (t < MT) {
            float sum = 0.f;
            for (int j = 0; j < 32; ++j) sum += red[j * MT + t];
            bpart[(long long)blockIdx.z * cout + co0 + t] = sum;
        }
    }
}

// Sums of split partials: out[g][k] = sum of partial[sp][k] over the splits
// sp of group g = blockIdx.y ([g chunk, (g + 1) chunk)), added in split
// order, for the n weights and, in the same launch, the nb biases (nb = 0:
// none).  One group (chunk >= nsplit) gives the final sums; with several, a
// second pass over the group sums adds them in group order, so the result
// is the same fixed-order sum whatever the launch.
__global__ void __launch_bounds__(256)
k_wgrad_reduce(const float *__restrict__ partial, long long n, const float *__restrict__ bpart, int nb, int nsplit,
               int chunk, float *__restrict__ out, float *__restrict__ bout)
{
    const int g = blockIdx.y;
    const int sp0 = g * chunk, sp1 = (sp0 + chunk < nsplit) ? sp0 + chunk : nsplit;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n + nb; k += (long long)gridDim.x * 256) {
        const bool w = k < n;
        const float *src = w ? partial + k : bpart + (k - n);
        const long long stride = w ? n : nb;
        float s = 0.f;
#pragma unroll 8
        for (int sp = sp0; sp < sp1; ++sp) s += src[sp * stride];
        if (w) out[g * n + k] = s;
        else bout[(long long)g * nb + (k - n)] = s;
    }
}

// ------------------------------------------------------------------ elementwise

// The elementwise kernels move NC channels per thread: 8 (one 16-byte access
// per operand) where the channels and every pointer allow it, else 1.  They
// are bound by memory; one value per thread left them bound by the index
// arithmetic (upsampling 16 x 128 x 128 x 64 to 256 x 256: 113 us a value at a
// time).
template <int NC> struct Bf;
template <> struct Bf<1> {
    uint16_t v[1];
    static __device__ __forceinline__ Bf load(const uint16_t *p) { return {{*p}}; }
    __device__ __forceinline__ void store(uint16_t *p) const { *p = v[0]; }
};
template <> struct Bf<8> {
    uint16_t v[8];
    static __device__ __forceinline__ Bf load(const uint16_t *p)
    {
        return __builtin_bit_cast(Bf, *reinterpret_cast<const uint4 *>(p));
    }
    __device__ __forceinline__ void store(uint16_t *p) const
    {
        *reinterpret_cast<uint4 *>(p) = __builtin_bit_cast(uint4, *this);
    }
};

// Chunk k of [B][H][W][C]: its place and channel.
template <int NC>
struct Place {
    int b, y, x, c;
    __device__ __forceinline__ Place(long long k, int H, int W, int C)
    {
        const uint32_t cn = uint32_t(C) / NC;
        uint64_t q = uint64_t(k);
        if (q >> 32 == 0) {
            uint32_t r = uint32_t(q);
            c = int(r % cn) * NC;
            r /= cn;
            x = int(r % uint32_t(W));
            r /= uint32_t(W);
            y = int(r % uint32_t(H));
            b = int(r / uint32_t(H));
        } else {
            c = int(q % cn) * NC;
            q /= cn;
            x = int(q % uint32_t(W));
            q /= uint32_t(W);
            y = int(q % uint32_t(H));
            b = int(q / uint32_t(H));
        }
    }
    __device__ __forceinline__ long long at(int yy, int xx, int H, int W, int C) const
    {
        return (((long long)b * H + yy) * W + xx) * C + c;
    }
};

template <int NC>
__global__ void __launch_bounds__(256)
k_avgpool2_fwd(const uint16_t *__restrict__ x, int B, int H, int W, int C, uint16_t *__restrict__ y)
{
    const int Ho = H / 2, Wo = W / 2;
    const long long n = (long long)B * Ho * Wo * C / NC;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const Place<NC> q(k, Ho, Wo, C);
        const long long base = q.at(2 * q.y, 2 * q.x, H, W, C);
        const Bf<NC> a = Bf<NC>::load(x + base), b = Bf<NC>::load(x + base + C),
                     c = Bf<NC>::load(x + base + (long long)W * C), d = Bf<NC>::load(x + base + (long long)W * C + C);
        Bf<NC> o;
#pragma unroll
        for (int e = 0; e < NC; ++e)
            o.v[e] = f2bf(0.25f * (bf2f(a.v[e]) + bf2f(b.v[e]) + bf2f(c.v[e]) + bf2f(d.v[e])));
        o.store(y + k * NC);
    }
}

template <int NC>
__global__ void __launch_bounds__(256)
k_avgpool2_bwd(const uint16_t *__restrict__ dy, int B, int H, int W, int C, uint16_t *__restrict__ dx)
{
    const long long n = (long long)B * H * W * C / NC;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const Place<NC> q(k, H, W, C);
        const Bf<NC> a = Bf<NC>::load(dy + q.at(q.y / 2, q.x / 2, H / 2, W / 2, C));
        Bf<NC> o;
#pragma unroll
        for (int e = 0; e < NC; ++e) o.v[e] = f2bf(0.25f * bf2f(a.v[e]));
        o.store(dx + k * NC);
    }
}

template <int NC>
__global__ void __launch_bounds__(256)
k_upsample2_fwd(const uint16_t *__restrict__ x, int B, int H, int W, int C, uint16_t *__restrict__ y)
{
    const int H2 = 2 * H, W2 = 2 * W;
    const long long n = (long long)B * H2 * W2 * C / NC;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const Place<NC> q(k, H2, W2, C);
        Bf<NC>::load(x + q.at(q.y / 2, q.x / 2, H, W, C)).store(y + k * NC);
    }
}

template <int NC>
__global__ void __launch_bounds__(256)
k_upsample2_bwd(const uint16_t *__restrict__ dy, int B, int H, int W, int C, uint16_t *__restrict__ dx)
{
    const int W2 = 2 * W;
    const long long n = (long long)B * H * W * C / NC;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const Place<NC> q(k, H, W, C);
        const long long base = q.at(2 * q.y, 2 * q.x, 2 * H, W2, C);
        const Bf<NC> a = Bf<NC>::load(dy + base), b = Bf<NC>::load(dy + base + C),
                     c = Bf<NC>::load(dy + base + (long long)W2 * C), d = Bf<NC>::load(dy + base + (long long)W2 * C + C);
        Bf<NC> o;
#pragma unroll
        for (int e = 0; e < NC; ++e) o.v[e] = f2bf(bf2f(a.v[e]) + bf2f(b.v[e]) + bf2f(c.v[e]) + bf2f(d.v[e]));
        o.store(dx + k * NC);
    }
}

template <int NC>
__global__ void __launch_bounds__(256)
k_add(const uint16_t *a, const uint16_t *b, const uint16_t *mask, long long n, uint16_t *out)
{
    n /= NC;
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const Bf<NC> va = Bf<NC>::load(a + k * NC);
        Bf<NC> vb = va, vm = va, o;
        if (b) vb = Bf<NC>::load(b + k * NC);
        if (mask) vm = Bf<NC>::load(mask + k * NC);
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            float v = bf2f(va.v[e]);
            if (b) v += bf2f(vb.v[e]);
            if (mask && !(bf2f(vm.v[e]) > 0.f)) v = 0.f;
            o.v[e] = f2bf(v);
        }
        o.store(out + k * NC);
    }
}

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

// ------------------------------------------------------------------ 1x1 head

__global__ void __launch_bounds__(256)
k_head_fwd(const uint16_t *__restrict__ x, int P, int cin, const float *__restrict__ w,
           const float *__restrict__ bias, int cout, float *__restrict__ y)
{
    __shared__ float sw[32 * 32];
    __shared__ float sb[32];
    for (int k = threadIdx.x; k < cout * cin; k += 256) sw[k] = w[k];
    if (threadIdx.x < cout) sb[threadIdx.x] = bias ? bias[threadIdx.x] : 0.f;
    __syncthreads();
    const long long p = blockIdx.x * 256LL + threadIdx.x;
    if (p >= P) return;
    float xv[32];
    for (int c = 0; c < cin; ++c) xv[c] = bf2f(x[p * cin + c]);
    for (int o = 0; o < cout; ++o) {
        float s = sb[o];
        for (int c = 0; c < cin; ++c) s += sw[o * cin + c] * xv[c];
        y[p * cout + o] = s;
    }
}

__global__ void __launch_bounds__(256)
k_head_bwd_x(const float *__restrict__ dy, int P, int cin, const float *__restrict__ w, int cout,
             const uint16_t *__restrict__ mask, uint16_t *__restrict__ dx)
{
    __shared__ float sw[32 * 32];
    for (int k = threadIdx.x; k < cout * cin; k += 256) sw[k] = w[k];
    __syncthreads();
    const long long p = blockIdx.x * 256LL + threadIdx.x;
    if (p >= P) return;
    for (int c = 0; c < cin; ++c) {
        float s = 0.f;
        for (int o = 0; o < cout; ++o) s += dy[p * cout + o] * sw[o * cin + c];
        if (mask && !(bf2f(mask[p * cin + c]) > 0.f)) s = 0.f;
        dx[p * cin + c] = f2bf(s);
    }
}

// one thread per (o, c) pair (and per o for the bias), a pixel range per block
__global__ void __launch_bounds__(256)
k_head_bwd_w(const uint16_t *__restrict__ x, const float *__restrict__ dy, int P, int cin, int cout,
             int rows_per_block, float *__restrict__ partial)
{
    const int t = threadIdx.x;
    const int nw = cout * cin;
    const long long r0 = (long long)blockIdx.x * rows_per_block;
    const long long r1 = (r0 + rows_per_block < P) ? r0 + rows_per_block : P;
    if (t < nw) {
        const int o = t / cin, c = t % cin;
        float s = 0.f;
        for (long long p = r0; p < r1; ++p) s += dy[p * cout + o] * bf2f(x[p * cin + c]);
        partial[(long long)blockIdx.x * (nw + cout) + t] = s;
    } else if (t < nw + cout) {
        const int o = t - nw;
        float s = 0.f;
        for (long long p = r0; p < r1; ++p) s += dy[p * cout + o];
        partial[(long long)blockIdx.x * (nw + cout) + t] = s;
    }
}

// Sum of the block partials of one of the cin cout + cout values per block,
// in block order: the threads bring 1024 partials at a time to LDS, the first
// adds them up (a thread per value reading them one by one waited for memory
// at every addition: 474 us for 2048 partials).
__global__ void __launch_bounds__(256)
k_head_bwd_reduce(const float *__restrict__ partial, int nblk, int cin, int cout, float *__restrict__ dw,
                  float *__restrict__ db)
{
    __shared__ float part[1024];
    const int t = threadIdx.x, k = blockIdx.x;
    const int nw = cout * cin;
    float s = 0.f;
    for (int b0 = 0; b0 < nblk; b0 += 1024) {
        const int m = nblk - b0 < 1024 ? nblk - b0 : 1024;
        __syncthreads();
        for (int b = t; b < m; b += 256) part[b] = partial[(long long)(b0 + b) * (nw + cout) + k];
        __syncthreads();
        if (t == 0) {
#pragma unroll 16
            for (int b = 0; b < m; ++b) s += part[b];
        }
    }
    if (t == 0) {
        if (k < nw) dw[k] = s;
        else if (db) db[k - nw] = s;
    }
}

// The head for 32 input channels and at most 8 output channels (the
// network's), pixels read and written 16 bytes at a time; the FP32 rows of
// cout values pass through LDS, so that they are contiguous in memory too.
// The kernels above cover every other size.  Bound by memory: at 2^20 pixels
// and 7 outputs the backward pass takes 64 + 64 MB in and 64 MB out.
constexpr int kHeadC = 32, kHeadO = 8;

__global__ void __launch_bounds__(256)
k_head_fwd32(const uint16_t *__restrict__ x, int P, const float *__restrict__ w, const float *__restrict__ bias, int cout,
             float *__restrict__ y)
{
    __shared__ float sw[kHeadO * kHeadC];
    __shared__ float sb[kHeadO];
    __shared__ float sy[256 * kHeadO];
    const int t = threadIdx.x;
    for (int k = t; k < cout * kHeadC; k += 256) sw[k] = w[k];
    if (t < cout) sb[t] = bias ? bias[t] : 0.f;
    __syncthreads();
    const long long p0 = blockIdx.x * 256LL, p = p0 + t;
    if (p < P) {
        Bf<8> xv[kHeadC / 8];
#pragma unroll
        for (int q = 0; q < kHeadC / 8; ++q) xv[q] = Bf<8>::load(x + p * kHeadC + 8 * q);
        for (int o = 0; o < cout; ++o) {
            float s = sb[o];
#pragma unroll
            for (int c = 0; c < kHeadC; ++c) s += sw[o * kHeadC + c] * bf2f(xv[c / 8].v[c % 8]);
            sy[t * cout + o] = s;
        }
    }
    __syncthreads();
    const int m = int((P - p0 < 256 ? P - p0 : 256)) * cout;
    for (int k = t; k < m; k += 256) y[p0 * cout + k] = sy[k];
}

// dx: 64 pixels per block, a thread per pixel and 8 channels.
__global__ void __launch_bounds__(256)
k_head_bwd_x32(const float *__restrict__ dy, int P, const float *__restrict__ w, int cout,
               const uint16_t *__restrict__ mask, uint16_t *__restrict__ dx)
{
    __shared__ float sw[kHeadO * kHeadC];
    __shared__ float sd[64 * kHeadO];
    const int t = threadIdx.x;
    const long long p0 = blockIdx.x * 64LL, p = p0 + t / 4;
    for (int k = t; k < cout * kHeadC; k += 256) sw[k] = w[k];
    const int m = int((P - p0 < 64 ? P - p0 : 64)) * cout;
    for (int k = t; k < m; k += 256) sd[k] = dy[p0 * cout + k];
    __syncthreads();
    if (p >= P) return;
    const int c0 = (t % 4) * 8;
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.f;
    for (int o = 0; o < cout; ++o) {
        const float d = sd[(t / 4) * cout + o];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += d * sw[o * kHeadC + c0 + e];
    }
    Bf<8> vm, r;
    if (mask) vm = Bf<8>::load(mask + p * kHeadC + c0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if (mask && !(bf2f(vm.v[e]) > 0.f)) s[e] = 0.f;
        r.v[e] = f2bf(s[e]);
    }
    r.store(dx + p * kHeadC + c0);
}

// Partial dw and db of kHeadRows pixels per block, a thread per (o, c) pair
// and per o for the bias, as k_head_bwd_w and in its order, from LDS copies of
// the pixels that all threads bring in with 16-byte loads.
constexpr int kHeadRows = 512;

__global__ void __launch_bounds__(256)
k_head_bwd_w32(const uint16_t *__restrict__ x, const float *__restrict__ dy, int P, int cout, float *__restrict__ partial)
{
    __shared__ uint4 sx4[kHeadRows * kHeadC / 8];
    __shared__ float sd[kHeadRows * (kHeadO - 1)];
    const int t = threadIdx.x;
    const int nw = cout * kHeadC;
    const long long r0 = (long long)blockIdx.x * kHeadRows;
    const int rows = (int)(P - r0 < kHeadRows ? P - r0 : kHeadRows);
    for (int k = t; k < rows * (kHeadC / 8); k += 256)
        sx4[k] = *reinterpret_cast<const uint4 *>(x + r0 * kHeadC + 8 * k);
    for (int k = t; k < rows * cout; k += 256) sd[k] = dy[r0 * cout + k];
    __syncthreads();
    const uint16_t *sx = reinterpret_cast<const uint16_t *>(sx4);
    float s = 0.f;
    if (t < nw) {
        const int o = t / kHeadC, c = t % kHeadC;
#pragma unroll 8
        for (int p = 0; p < rows; ++p) s += sd[p * cout + o] * bf2f(sx[p * kHeadC + c]);
    } else if (t < nw + cout) {
        const int o = t - nw;
#pragma unroll 8
        for (int p = 0; p < rows; ++p) s += sd[p * cout + o];
    }
    if (t < nw + cout) partial[(long long)blockIdx.x * (nw + cout) + t] = s;
}

// ------------------------------------------------------------------ loss, optimiser

// pass 1: per-block partial sums of wt (d^2 summed over channels) and wt
__global__ void __launch_bounds__(256)
k_mse_partial(const float *__restrict__ y, const float *__restrict__ tg, const float *__restrict__ wt, int P,
              int C, float *__restrict__ partial)
{
    __shared__ float s1[256], s2[256];
    const long long p = blockIdx.x * 256LL + threadIdx.x;
    float a = 0.f, b = 0.f;
    if (p < P) {
        const float ww = wt[p];
        for (int c = 0; c < C; ++c) {
            const float d = y[p * C + c] - tg[p * C + c];
            a += ww * d * d;
        }
        b = ww;
    }
    s1[threadIdx.x] = a;
    s2[threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            s1[threadIdx.x] += s1[threadIdx.x + s];
            s2[threadIdx.x] += s2[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = s1[0];
        partial[2 * blockIdx.x + 1] = s2[0];
    }
}

// pass 2 (one block): totals; loss = S / (Wsum C); totals kept for pass 3
__global__ void __launch_bounds__(256)
k_mse_total(const float *__restrict__ partial, int nblk, int C, float *__restrict__ totals, float *__restrict__ loss)
{
    __shared__ float s1[256], s2[256];
    float a = 0.f, b = 0.f;
    for (int k = threadIdx.x; k < nblk; k += 256) {
        a += partial[2 * k];
        b += partial[2 * k + 1];
    }
    s1[threadIdx.x] = a;
    s2[threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            s1[threadIdx.x] += s1[threadIdx.x + s];
            s2[threadIdx.x] += s2[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        totals[0] = s1[0];
        totals[1] = s2[0];
        if (loss) *loss = s2[0] > 0.f ? s1[0] / (s2[0] * C) : 0.f;
    }
}

// pass 3: dy = 2 wt (y - t) / (Wsum C)
__global__ void __launch_bounds__(256)
k_mse_grad(const float *__restrict__ y, const float *__restrict__ tg, const float *__restrict__ wt, int P, int C,
           const float *__restrict__ totals, float *__restrict__ dy)
{
    const long long p = blockIdx.x * 256LL + threadIdx.x;
    if (p >= P) return;
    const float den = totals[1] * C;
    const float sc = den > 0.f ? 2.f * wt[p] / den : 0.f;
    for (int c = 0; c < C; ++c) dy[p * C + c] = sc * (y[p * C + c] - tg[p * C + c]);
}

__global__ void __launch_bounds__(256)
k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v, long long n,
       float lr, float b1, float b2, float eps, float c1, float c2, uint16_t *__restrict__ pb)
{
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const float gk = g[k];
        const float mk = b1 * m[k] + (1.f - b1) * gk;
        const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
        m[k] = mk;
        v[k] = vk;
        const float mh = mk / c1, vh = vk / c2;
        const float pk = p[k] - lr * mh / (sqrtf(vh) + eps);
        p[k] = pk;
        if (pb) pb[k] = f2bf(pk);
    }
}

__global__ void __launch_bounds__(256) k_to_bf16(const float *__restrict__ x, long long n, uint16_t *__restrict__ y)
{
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) y[k] = f2bf(x[k]);
}

__global__ void __launch_bounds__(256) k_to_f32(const uint16_t *__restrict__ x, long long n, float *__restrict__ y)
{
    for (long long k = blockIdx.x * 256LL + threadIdx.x; k < n; k += (long long)gridDim.x * 256) y[k] = bf2f(x[k]);
}

int grid1(long long n)
{
    long long g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

int status(hipError_t e) { return e == hipSuccess ? MDFNN_OK : MDFNN_EDEVICE; }

}  // namespace
}  // namespace mdfnn

using namespace mdfnn;

extern "C" {

int mdfnn_conv3x3_fwd(const uint16_t *x1, int c1, const uint16_t *x2, int c2, const uint16_t *w,
                      const float *bias, int B, int H, int W, int cout, int relu, const uint16_t *mask,
                      uint16_t *y_bf16, float *y_f32, void *stream)
{
    if (!x1 || !w || (!y_bf16 && !y_f32) || B < 1 || H < 1 || W < 1) return MDFNN_EINVAL;
    if (c1 < 32 || c1 % 32 || c2 < 0 || c2 % 32 || (c2 > 0 && !x2) || cout < 32 || cout % 32) return MDFNN_EINVAL;
    const long long M = (long long)B * H * W;
    if (M > (1LL << 31)) return MDFNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const unsigned gx = (unsigned)((M + kCvBM - 1) / kCvBM);
    // four channels at a time need aligned outputs; k_conv_fwd_lds writes one
    const bool wide = (reinterpret_cast<uintptr_t>(mask) % 8 == 0) && (reinterpret_cast<uintptr_t>(y_bf16) % 8 == 0) &&
                      (reinterpret_cast<uintptr_t>(y_f32) % 16 == 0);
    switch (wide ? conv_form(B, H, W, c1 + c2, cout, {bias != nullptr, mask != nullptr, !y_bf16}) : kConvLds) {
    case kConvTile: {
        const int tgx = (W + 15) / 16, tgy = (H + 15) / 16;
        hipLaunchKernelGGL(k_conv_fwd_tile, dim3((unsigned)tgx * tgy * B, cout / 32), dim3(256), 0, st, x1, w, bias, H, W,
                           tgx, tgy, cout, relu, mask, y_bf16, y_f32);
        return status(hipGetLastError());
    }
    case kConvRun32:
        hipLaunchKernelGGL(k_conv_fwd_run<32>, dim3(gx, cout / 32), dim3(256), 0, st, x1, c1, x2, c2, w, bias, B, H, W,
                           cout, relu, mask, y_bf16, y_f32);
        return status(hipGetLastError());
    case kConvRun64:
        hipLaunchKernelGGL(k_conv_fwd_run<64>, dim3(gx, cout / 64), dim3(256), 0, st, x1, c1, x2, c2, w, bias, B, H, W,
                           cout, relu, mask, y_bf16, y_f32);
        return status(hipGetLastError());
    default: break;
    }
    if (cout % 128 == 0)
        hipLaunchKernelGGL(k_conv_fwd_lds<128>, dim3(gx, cout / 128), dim3(256), 0, st, x1, c1, x2, c2, w, bias, B, H,
                           W, cout, relu, mask, y_bf16, y_f32);
    else if (cout % 64 == 0)
        hipLaunchKernelGGL(k_conv_fwd_lds<64>, dim3(gx, cout / 64), dim3(256), 0, st, x1, c1, x2, c2, w, bias, B, H, W,
                           cout, relu, mask, y_bf16, y_f32);
    else
        hipLaunchKernelGGL(k_conv_fwd_lds<32>, dim3(gx, cout / 32), dim3(256), 0, st, x1, c1, x2, c2, w, bias, B, H, W,
                           cout, relu, mask, y_bf16, y_f32);
    return status(hipGetLastError());
}

int mdfnn_conv3x3_flip(const uint16_t *w, int cout, int cin, uint16_t *wt, void *stream)
{
    if (!w || !wt || cout < 1 || cin < 1) return MDFNN_EINVAL;
    const long long n = (long long)cout * 9 * cin;
    hipLaunchKernelGGL(k_flip, dim3(grid1(n)), dim3(256), 0, static_cast<hipStream_t>(stream), w, cout, cin, wt);
    return status(hipGetLastError());
}

// Channel tiles of the weight gradient: MT output x NT input channels; a
// tile of input channels must not straddle x1 and x2.
static int wgrad_mt(int cout) { return (cout % 64 == 0) ? 64 : 32; }
static int wgrad_nt(int c1, int c2) { return (c1 % 64 == 0 && c2 % 64 == 0) ? 64 : 32; }

// Splits of the pixel segments (32 pixels of one image row each): about 1024
// blocks over the channel tiles, at least 8 segments per split.
static int wgrad_splits(int B, int H, int W, int ntiles)
{
    const long long nseg = (long long)B * H * ((W + 31) / 32);
    long long s = (kWgBlocks + ntiles - 1) / ntiles;
    if (s > nseg / 8) s = nseg / 8;
    if (s < 1) s = 1;
    return (int)s;
}

// Splits per group of the first reduction pass.
constexpr int kWgChunk = 32;

// Fixed-order sum over ns split partials of n weights and nb biases (two
// passes when ns > kWgChunk, through mid: ceil(ns / kWgChunk) * (n + nb) floats).
static hipError_t reduce_splits(const float *partial, long long n, const float *bpart, int nb, int ns, float *mid,
                                float *out, float *bout, hipStream_t st)
{
    if (ns <= kWgChunk) {
        hipLaunchKernelGGL(k_wgrad_reduce, dim3(grid1(n + nb), 1), dim3(256), 0, st, partial, n, bpart, nb, ns, ns, out,
                           bout);
        return hipGetLastError();
    }
    const int G = (ns + kWgChunk - 1) / kWgChunk;
    float *bmid = mid + (size_t)G * n;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(grid1(n + nb), G), dim3(256), 0, st, partial, n, bpart, nb, ns, kWgChunk, mid,
                       bmid);
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(grid1(n + nb), 1), dim3(256), 0, st, mid, n, bmid, nb, G, G, out, bout);
    return hipGetLastError();
}

size_t mdfnn_wgrad_scratch_bytes(int B, int H, int W, int cin, int cout)
{
    if (B < 1 || H < 1 || W < 1 || cin < 32 || cout < 32) return 0;
    // the smallest tiles give the most splits
    const int ns = wgrad_splits(B, H, W, (cout / 64 > 0 ? cout / 64 : 1) * (cin / 64 > 0 ? cin / 64 : 1));
    const size_t G = (size_t)(ns + kWgChunk - 1) / kWgChunk;
    const size_t n = (size_t)cout * 9 * cin;
    // weight and bias partials, then the group sums of both
    return ((size_t)ns * (n + cout) + G * (n + cout)) * sizeof(float) + 256;
}

int mdfnn_conv3x3_wgrad(const uint16_t *x1, int c1, const uint16_t *x2, int c2, const uint16_t *dy, int B, int H,
                        int W, int cout, float *dw, float *db, void *scratch, void *stream)
{
    if (!x1 || !dy || !dw || !scratch || B < 1 || H < 1 || W < 1) return MDFNN_EINVAL;
    const int cin = c1 + c2;
    if (c1 < 32 || c1 % 32 || c2 < 0 || c2 % 32 || (c2 > 0 && !x2) || cout < 32 || cout % 32) return MDFNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int mt = wgrad_mt(cout), nt = wgrad_nt(c1, c2);
    const int ns = wgrad_splits(B, H, W, (cout / mt) * (cin / nt));
    float *wpart = static_cast<float *>(scratch);
    float *bpart = db ? wpart + (size_t)ns * cout * 9 * cin : nullptr;
    const dim3 grid(cout / mt, cin / nt, ns);
    if (mt == 64 && nt == 64)
        hipLaunchKernelGGL((k_conv_wgrad9<64, 64>), grid, dim3(256), 0, st, x1, c1, x2, c2, dy, B, H, W, cout, ns, wpart,
                           bpart);
    else if (mt == 64)
        hipLaunchKernelGGL((k_conv_wgrad9<64, 32>), grid, dim3(256), 0, st, x1, c1, x2, c2, dy, B, H, W, cout, ns, wpart,
                           bpart);
    else if (nt == 64)
        hipLaunchKernelGGL((k_conv_wgrad9<32, 64>), grid, dim3(256), 0, st, x1, c1, x2, c2, dy, B, H, W, cout, ns, wpart,
                           bpart);
    else
        hipLaunchKernelGGL((k_conv_wgrad9<32, 32>), grid, dim3(256), 0, st, x1, c1, x2, c2, dy, B, H, W, cout, ns, wpart,
                           bpart);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return MDFNN_EDEVICE;
    const long long n = (long long)cout * 9 * cin;
    float *mid = wpart + (size_t)ns * (n + cout);
    return status(reduce_splits(wpart, n, bpart, db ? cout : 0, ns, mid, dw, db, st));
}

int mdfnn_avgpool2_fwd(const uint16_t *x, int B, int H, int W, int C, uint16_t *y, void *stream)
{
    if (!x || !y || B < 1 || H < 2 || W < 2 || H % 2 || W % 2 || C < 1) return MDFNN_EINVAL;
    const long long n = (long long)B * (H / 2) * (W / 2) * C;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && aligned16(x) && aligned16(y))
        hipLaunchKernelGGL(k_avgpool2_fwd<8>, dim3(grid1(n / 8)), dim3(256), 0, st, x, B, H, W, C, y);
    else
        hipLaunchKernelGGL(k_avgpool2_fwd<1>, dim3(grid1(n)), dim3(256), 0, st, x, B, H, W, C, y);
    return status(hipGetLastError());
}

int mdfnn_avgpool2_bwd(const uint16_t *dy, int B, int H, int W, int C, uint16_t *dx, void *stream)
{
    if (!dy || !dx || B < 1 || H < 2 || W < 2 || H % 2 || W % 2 || C < 1) return MDFNN_EINVAL;
    const long long n = (long long)B * H * W * C;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && aligned16(dy) && aligned16(dx))
        hipLaunchKernelGGL(k_avgpool2_bwd<8>, dim3(grid1(n / 8)), dim3(256), 0, st, dy, B, H, W, C, dx);
    else
        hipLaunchKernelGGL(k_avgpool2_bwd<1>, dim3(grid1(n)), dim3(256), 0, st, dy, B, H, W, C, dx);
    return status(hipGetLastError());
}

int mdfnn_upsample2_fwd(const uint16_t *x, int B, int H, int W, int C, uint16_t *y, void *stream)
{
    if (!x || !y || B < 1 || H < 1 || W < 1 || C < 1) return MDFNN_EINVAL;
    const long long n = (long long)B * 4 * H * W * C;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && aligned16(x) && aligned16(y))
        hipLaunchKernelGGL(k_upsample2_fwd<8>, dim3(grid1(n / 8)), dim3(256), 0, st, x, B, H, W, C, y);
    else
        hipLaunchKernelGGL(k_upsample2_fwd<1>, dim3(grid1(n)), dim3(256), 0, st, x, B, H, W, C, y);
    return status(hipGetLastError());
}

int mdfnn_upsample2_bwd(const uint16_t *dy, int B, int H, int W, int C, uint16_t *dx, void *stream)
{
    if (!dy || !dx || B < 1 || H < 1 || W < 1 || C < 1) return MDFNN_EINVAL;
    const long long n = (long long)B * H * W * C;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && aligned16(dy) && aligned16(dx))
        hipLaunchKernelGGL(k_upsample2_bwd<8>, dim3(grid1(n / 8)), dim3(256), 0, st, dy, B, H, W, C, dx);
    else
        hipLaunchKernelGGL(k_upsample2_bwd<1>, dim3(grid1(n)), dim3(256), 0, st, dy, B, H, W, C, dx);
    return status(hipGetLastError());
}

int mdfnn_add(const uint16_t *a, const uint16_t *b, const uint16_t *mask, long long n, uint16_t *out, void *stream)
{
    if (!a || !out || n < 0) return MDFNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n % 8 == 0 && aligned16(a) && aligned16(b) && aligned16(mask) && aligned16(out))
        hipLaunchKernelGGL(k_add<8>, dim3(grid1(n / 8)), dim3(256), 0, st, a, b, mask, n, out);
    else
        hipLaunchKernelGGL(k_add<1>, dim3(grid1(n)), dim3(256), 0, st, a, b, mask, n, out);
    return status(hipGetLastError());
}

int mdfnn_head_fwd(const uint16_t *x, int P, int cin, const float *w, const float *bias, int cout, float *y,
                   void *stream)
{
    if (!x || !w || !y || P < 1 || cin < 1 || cin > 32 || cout < 1 || cout > 32) return MDFNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nblk = (int)(((long long)P + 255) / 256);
    if (cin == kHeadC && cout <= kHeadO && aligned16(x))
        hipLaunchKernelGGL(k_head_fwd32, dim3(nblk), dim3(256), 0, st, x, P, w, bias, cout, y);
    else
        hipLaunchKernelGGL(k_head_fwd, dim3(nblk), dim3(256), 0, st, x, P, cin, w, bias, cout, y);
    return status(hipGetLastError());
}

size_t mdfnn_head_scratch_bytes(int P, int cin, int cout)
{
    const int rows = kHeadRows;
    const size_t nblk = (size_t)((P + rows - 1) / rows);
    return nblk * (size_t)(cin * cout + cout) * sizeof(float) + 256;
}

int mdfnn_head_bwd(const uint16_t *x, const float *dy, int P, int cin, const float *w, int cout, const uint16_t *mask,
                   uint16_t *dx, float *dw, float *db, void *scratch, void *stream)
{
    if (!x || !dy || !w || !dw || !scratch || P < 1 || cin < 1 || cin > 32 || cout < 1 || cout > 32 ||
        cin * cout + cout > 256)
        return MDFNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool fast = cin == kHeadC && cout <= kHeadO;
    if (dx && fast && aligned16(dx) && aligned16(mask))
        hipLaunchKernelGGL(k_head_bwd_x32, dim3((int)(((long long)P + 63) / 64)), dim3(256), 0, st, dy, P, w, cout, mask, dx);
    else if (dx)
        hipLaunchKernelGGL(k_head_bwd_x, dim3((P + 255) / 256), dim3(256), 0, st, dy, P, cin, w, cout, mask, dx);
    const int rows = kHeadRows;
    const int nblk = (P + rows - 1) / rows;
    float *part = static_cast<float *>(scratch);
    // (cin cout + cout <= 256: at most 7 outputs)
    if (fast && aligned16(x)) hipLaunchKernelGGL(k_head_bwd_w32, dim3(nblk), dim3(256), 0, st, x, dy, P, cout, part);
    else hipLaunchKernelGGL(k_head_bwd_w, dim3(nblk), dim3(256), 0, st, x, dy, P, cin, cout, rows, part);
    hipLaunchKernelGGL(k_head_bwd_reduce, dim3(cin * cout + cout), dim3(256), 0, st, part, nblk, cin, cout, dw, db);
    return status(hipGetLastError());
}

size_t mdfnn_loss_scratch_bytes(int P) { return (size_t)(2 * ((P + 255) / 256) + 2) * sizeof(float) + 256; }

int mdfnn_mse(const float *y, const float *t, const float *wt, int P, int C, float *dy, float *loss, void *scratch,
              void *stream)
{
    if (!y || !t || !wt || !dy || !scratch || P < 1 || C < 1) return MDFNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nblk = (P + 255) / 256;
    float *part = static_cast<float *>(scratch);
    float *totals = part + 2 * nblk;
    hipLaunchKernelGGL(k_mse_partial, dim3(nblk), dim3(256), 0, st, y, t, wt, P, C, part);
    hipLaunchKernelGGL(k_mse_total, dim3(1), dim3(256), 0, st, part, nblk, C, totals, loss);
    hipLaunchKernelGGL(k_mse_grad, dim3(nblk), dim3(256), 0, st, y, t, wt, P, C, totals, dy);
    return status(hipGetLastError());
}

}  // extern "C"

// ------------------------------------------------------------------ allocation-free loss

namespace mdfnn {
namespace {

// Device scratch of mdfnn_mse_noalloc: the per-block partial sums and the two
// totals of the loss, for at most kMseStaticMaxP pixels.  Each GPU holds its
// own copy for the life of the process.  In host code `scratch` names a
// host-side stand-in; kernels get the device address that
// hipGetSymbolAddress returns for the current device.
constexpr int kMseStaticMaxP = MDFNN_MSE_NOALLOC_MAX_P;
constexpr int kMseStaticFloats = 2 * ((kMseStaticMaxP + 255) / 256) + 2;
__device__ __align__(256) float scratch[kMseStaticFloats];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
float *g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's `scratch`, looked up once per device with
// that device current.
hipError_t mse_scratch(float **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<float *>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace
}  // namespace mdfnn

extern "C" {

int mdfnn_mse_noalloc(const float *y, const float *t, const float *wt, int P, int C, float *dy, float *loss,
                      void *stream)
{
    if (!y || !t || !wt || !dy || P < 1 || C < 1) return MDFNN_EINVAL;
    if (P > kMseStaticMaxP) return MDFNN_ETOOBIG;
    float *part = nullptr;
    hipError_t e = mse_scratch(&part);
    if (e != hipSuccess) return MDFNN_EDEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nblk = (P + 255) / 256;
    float *totals = part + 2 * nblk;
    // every partial and both totals are written before they are read: nothing
    // left by an earlier call is used
    hipLaunchKernelGGL(k_mse_partial, dim3(nblk), dim3(256), 0, st, y, t, wt, P, C, part);
    hipLaunchKernelGGL(k_mse_total, dim3(1), dim3(256), 0, st, part, nblk, C, totals, loss);
    hipLaunchKernelGGL(k_mse_grad, dim3(nblk), dim3(256), 0, st, y, t, wt, P, C, totals, dy);
    return status(hipGetLastError());
}

int mdfnn_adam(float *p, const float *g, float *m, float *v, long long n, float lr, float b1, float b2, float eps, int t,
               uint16_t *p_bf16, void *stream)
{
    if (!p || !g || !m || !v || n < 0 || t < 1) return MDFNN_EINVAL;
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(grid1(n)), dim3(256), 0, static_cast<hipStream_t>(stream), p, g, m, v, n, lr, b1, b2,
                       eps, c1, c2, p_bf16);
    return status(hipGetLastError());
}

int mdfnn_to_bf16(const float *x, long long n, uint16_t *y, void *stream)
{
    if (!x || !y || n < 0) return MDFNN_EINVAL;
    hipLaunchKernelGGL(k_to_bf16, dim3(grid1(n)), dim3(256), 0, static_cast<hipStream_t>(stream), x, n, y);
    return status(hipGetLastError());
}

int mdfnn_to_f32(const uint16_t *x, long long n, float *y, void *stream)
{
    if (!x || !y || n < 0) return MDFNN_EINVAL;
    hipLaunchKernelGGL(k_to_f32, dim3(grid1(n)), dim3(256), 0, static_cast<hipStream_t>(stream), x, n, y);
    return status(hipGetLastError());
}

}  // extern "C"
