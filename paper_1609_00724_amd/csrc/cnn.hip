// Learned refinement proposer on gfx950: a 4-layer 3x3 convolutional network
// (3 -> 32 -> 32 -> 32 -> 2 channels, ReLU after the hidden layers) that reads
// coarse tiles of the field-line length, its FLEDGE map (Sect. 3.6) and Bz,
// and outputs a refine-mask logit and a log10 Q estimate per pixel.  The
// network is an extension beyond the paper; the FLL-jump rule of Sect. 3.6
// stays the fallback and the reference its proposals are scored against.
//
// Every contraction runs on the matrix cores: v_mfma_f32_16x16x32_bf16 (BF16
// operands, FP32 accumulation), each wave accumulating one or more 16x16
// output tiles.
//   forward / input gradient: M = 16 pixels of a row, N = 16 output channels,
//     K = 32 (one tap's 32 input channels, or all 9 taps of a 2-3 channel
//     input packed into one chunk)
//   weight gradient: M = 16 input channels, N = 16 output channels, K = 32
//     pixels of a row; per-wave partial sums reduced in a fixed order
// Activations are BF16 NHWC with 32 channels; the network input is FP32 with
// 3 channels, the output FP32 with 2.
#include <math.h>

#include "qsq_cnn.h"
#include "qsq_internal.h"

namespace qsq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16 bits, round to nearest, ties to even (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ __bf16 as_bf(uint16_t b) { return __builtin_bit_cast(__bf16, b); }

__device__ __forceinline__ f32x4 mfma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 ld_bf16x8(const uint16_t *p)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    return __builtin_bit_cast(bf16x8, v);
}

// network shape
constexpr int kCi[4] = {3, 32, 32, 32};
constexpr int kCo[4] = {32, 32, 32, 2};

__host__ __device__ constexpr int ntile(int c) { return (c + 15) / 16; }
// channels per tap in the packed K layout of an input with fewer than 32
// channels (3 is padded to 4 so that a tap's channels fill whole dwords)
__host__ __device__ constexpr int cpad(int ci) { return ci == 3 ? 4 : ci; }
__host__ __device__ constexpr int nchunk(int ci) { return ci >= 32 ? 9 : (9 * cpad(ci) + 31) / 32; }

// ---------------------------------------------------------------------------
// Prepared weights (BF16 matrices in MFMA-friendly order + FP32 biases)
//   fwd[l]: [nchunk(Ci)][16 ntile(Co)][32]: element (kc, co, kk) multiplies
//           input channel/tap (tap = kc, ci = kk) for Ci = 32, or
//           (tap = k / cpad(Ci), ci = k % cpad(Ci), k = 32 kc + kk; zero
//           where ci >= Ci or tap >= 9) for Ci < 32
//   bwd[l] (l >= 1): the transposed, tap-flipped kernel of the input
//           gradient, a convolution from Co channels to Ci = 32: element
//           (kc, ci, kk) = W[flip(tap)][ci][c] with (tap, c) taken from
//           (kc, kk) as above with Co in the role of Ci
// Master parameters (FP32): per layer W (3, 3, Ci, Co) row-major, then b (Co).
// ---------------------------------------------------------------------------
struct PrepLayout {
    int64_t fwd[4], bwd[4], bias[4], total_u16;
};

__host__ __device__ inline int64_t master_w(int l)
{
    int64_t o = 0;
    for (int k = 0; k < l; ++k) o += 9 * kCi[k] * kCo[k] + kCo[k];
    return o;
}

__host__ __device__ inline PrepLayout prep_layout()
{
    PrepLayout p{};
    int64_t o = 0;
    for (int l = 0; l < 4; ++l) {
        p.fwd[l] = o;
        o += (int64_t)nchunk(kCi[l]) * 16 * ntile(kCo[l]) * 32;
    }
    for (int l = 0; l < 4; ++l) {
        p.bwd[l] = o;
        if (l >= 1) o += (int64_t)nchunk(kCo[l]) * 32 * 32;
    }
    o = (o + 127) & ~(int64_t)127;
    for (int l = 0; l < 4; ++l) {
        p.bias[l] = o;      // FP32 biases stored in u16 units (2 per float)
        o += 2 * 32;
    }
    p.total_u16 = o;
    return p;
}

__global__ void k_prepare(const float *params, uint16_t *prep)
{
    const PrepLayout P = prep_layout();
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // forward matrices
    for (int l = 0; l < 4; ++l) {
        const int Ci = kCi[l], Co = kCo[l], COP = 16 * ntile(Co), NK = nchunk(Ci);
        const int64_t N = (int64_t)NK * COP * 32;
        const float *W = params + master_w(l);
        for (int64_t e = t; e < N; e += (int64_t)gridDim.x * blockDim.x) {
            const int kk = (int)(e % 32), co = (int)((e / 32) % COP), kc = (int)(e / (32 * COP));
            int tap, ci;
            if (Ci >= 32) {
                tap = kc;
                ci = kk;
            } else {
                tap = (32 * kc + kk) / cpad(Ci);
                ci = (32 * kc + kk) % cpad(Ci);
            }
            const bool ok = co < Co && tap < 9 && ci < Ci;
            prep[P.fwd[l] + e] = ok ? f2bf(W[((int64_t)tap * Ci + ci) * Co + co]) : (uint16_t)0;
        }
    }
    // transposed, flipped matrices of the input gradients
    for (int l = 1; l < 4; ++l) {
        const int Ci = kCi[l], Co = kCo[l], NK = nchunk(Co);
        const int64_t N = (int64_t)NK * 32 * 32;
        const float *W = params + master_w(l);
        for (int64_t e = t; e < N; e += (int64_t)gridDim.x * blockDim.x) {
            const int kk = (int)(e % 32), ci = (int)((e / 32) % 32), kc = (int)(e / (32 * 32));
            int tap, c;
            if (Co >= 32) {
                tap = kc;
                c = kk;
            } else {
                tap = (32 * kc + kk) / cpad(Co);
                c = (32 * kc + kk) % cpad(Co);
            }
            const bool ok = tap < 9 && ci < Ci && c < Co;
            prep[P.bwd[l] + e] = ok ? f2bf(W[((int64_t)(8 - tap) * Ci + ci) * Co + c]) : (uint16_t)0;
        }
    }
    for (int l = 0; l < 4; ++l) {
        float *b = reinterpret_cast<float *>(prep + P.bias[l]);
        const float *src = params + master_w(l) + 9 * kCi[l] * kCo[l];
        for (int64_t e = t; e < 32; e += (int64_t)gridDim.x * blockDim.x) b[e] = e < kCo[l] ? src[e] : 0.0f;
    }
}

// ---------------------------------------------------------------------------
// 3x3 'same' convolution.  A workgroup of 4 waves takes kConvRows rows of a
// 64-pixel column chunk of one image, a wave a 16-pixel strip of it, all
// output channels; the wave keeps the weight operands in registers.
// 32-channel inputs (BF16): the workgroup first stages its input rows
// (kConvRows + 2, pixels x - 1 .. x + 64, zeros outside the image) in LDS with
// all loads in flight at once; lane (i, kg) then reads pixels x0 + i - 1,
// x0 + i, x0 + i + 1, channels 8 kg .. 8 kg + 7, of each row from there, in a
// window of three rows sliding down the strip.  The network input (3 channels,
// FP32) is staged the same way, as BF16 with cpad(3) channels per pixel, and the
// 9 taps' channels packed along K (cpad(3) per tap) are read from there.  Outputs (each nullable): BF16 activations (ReLU
// applied) and FP32 values.  A BF16 NHWC output of 32 channels goes
// through LDS so that each lane stores one pixel's 8 channels (16 bytes) and
// the wave a row's 1 KB with one store.  One tile's tensors are addressed
// with 32-bit byte offsets (h w <= 2^24).
// ---------------------------------------------------------------------------
struct ConvDims {
    int64_t n;
    int h, w;
};

constexpr int kConvRows = 8;   // divides h (a multiple of 32)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// buffer resource over `bytes` bytes at p (gfx9 descriptor word 3: 32-bit
// data format, untyped access); offsets at or past `bytes` read zeros and
// drop writes
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, bytes, 0x00020000);
}

// two FP32 values to a BF16 pair (round to nearest even), a in the low half
__device__ __forceinline__ uint32_t pack_bf2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

struct Row3 {
    bf16x8 m, z, p;   // the lane's pixel shifted by -1, 0, +1
};

template <int CI, int CO>
__global__ void __launch_bounds__(256) k_conv(const void *__restrict__ in, ConvDims d,
                                              const uint16_t *__restrict__ wm, const float *__restrict__ bias,
                                              bool relu, uint16_t *__restrict__ out_bf, float *__restrict__ out_f32)
{
    constexpr int NT = ntile(CO), COP = 16 * NT, NK = nchunk(CI), R = kConvRows;
    static_assert(CI == 32 || CI == 3, "BF16 activations of 32 channels, or the FP32 network input");
    const int lane = (int)(threadIdx.x & 63);
    // workgroup: R rows of a 64-pixel column chunk of one image; wave s (a
    // scalar, so that the buffer resources below are too) the 16-pixel strip
    // x0 = xc + 16 s
    const int cpr = (d.w + 63) / 64, rb = d.h / R;
    const int64_t blk = blockIdx.x / cpr;   // image * rb + row block
    const int xc = (int)(blockIdx.x % cpr) * 64, y0 = (int)(blk % rb) * R;
    const int64_t img = blk / rb;
    const int sw = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int x0 = xc + 16 * sw;
    const int i = lane & 15, kg = lane >> 4;
    const int64_t npix = (int64_t)d.h * d.w;   // pixels of one tile
    // 32-channel inputs: the workgroup's R + 2 input rows, pixels xc - 1 ..
    // xc + 64 (zeros outside the image), staged in LDS with all loads in
    // flight at once: [row][pixel][4 chunks of 8 channels]
    constexpr int PW = 66, NCH = (R + 2) * PW * 4, PER = (NCH + 255) / 256;
    uint4 *lrows = nullptr;
    if constexpr (CI >= 32) {
        __shared__ uint4 rows_lds[NCH];
        lrows = rows_lds;
        const __amdgpu_buffer_rsrc_t rs = buf_rsrc(static_cast<const uint16_t *>(in) + img * npix * 32, (int)(npix * 64));
        u32x4 tmp[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int c = (int)threadIdx.x + 256 * k;
            const int r = c / (PW * 4), rem = c % (PW * 4), px = xc - 1 + (rem >> 2), q = rem & 3;
            // rows above and below the tile lie outside the buffer range (zeros), and so
            // do the pixels left and right of it
            const int off = px >= 0 && px < d.w ? (((y0 - 1 + r) * d.w + px) * 32 + 8 * q) * 2 : (int)(npix * 64);
            tmp[k] = c < NCH ? __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int c = (int)threadIdx.x + 256 * k;
            if (c < NCH) rows_lds[c] = make_uint4(tmp[k].x, tmp[k].y, tmp[k].z, tmp[k].w);
        }
        __syncthreads();
    }
    // inputs with CI < 32 channels: the same rows as BF16 with cpad(CI)
    // channels per pixel (the pad channel zero), WPT dwords per pixel
    constexpr int WPT = cpad(CI) / 2, NPX = (R + 2) * PW;
    uint32_t *lsmall = nullptr;
    if constexpr (CI < 32) {
        __shared__ uint32_t small_lds[NPX * WPT];
        lsmall = small_lds;
        constexpr int PERS = (NPX + 255) / 256;
        uint32_t tmp[PERS][WPT];
#pragma unroll
        for (int k = 0; k < PERS; ++k) {
            const int q = (int)threadIdx.x + 256 * k;
            const int yy = y0 - 1 + q / PW, px = xc - 1 + q % PW;
#pragma unroll
            for (int j = 0; j < WPT; ++j) tmp[k][j] = 0u;
            if (q < NPX && yy >= 0 && yy < d.h && px >= 0 && px < d.w) {
                const int64_t pix = (img * d.h + yy) * d.w + px;
                const float *pf = static_cast<const float *>(in) + pix * 3;
                tmp[k][0] = (uint32_t)f2bf(pf[0]) | ((uint32_t)f2bf(pf[1]) << 16);
                tmp[k][1] = (uint32_t)f2bf(pf[2]);
            }
        }
#pragma unroll
        for (int k = 0; k < PERS; ++k) {
            const int q = (int)threadIdx.x + 256 * k;
            if (q < NPX) {
#pragma unroll
                for (int j = 0; j < WPT; ++j) small_lds[q * WPT + j] = tmp[k][j];
            }
        }
        __syncthreads();
    }
    if (x0 >= d.w) return;   // the whole wave leaves together (no barrier follows)
    bf16x8 bw[NK][NT];
#pragma unroll
    for (int kc = 0; kc < NK; ++kc)
#pragma unroll
        for (int t = 0; t < NT; ++t) bw[kc][t] = ld_bf16x8(wm + ((int64_t)(kc * COP + t * 16 + i) * 32 + 8 * kg));
    float bv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) bv[t] = bias && t * 16 + i < CO ? bias[t * 16 + i] : 0.0f;
    // BF16 NHWC output of 32 channels through the wave's LDS stage
    __shared__ uint16_t stage_all[4][16 * 32];
    uint16_t *stage = stage_all[threadIdx.x >> 6];
    auto store_nhwc = [&](uint16_t *dst, int y, const uint32_t (&hp)[NT][2]) {
        if constexpr (CO == 32) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    stage[(4 * kg + r) * 32 + 16 * t + i] = (uint16_t)(hp[t][r >> 1] >> (16 * (r & 1)));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const u32x4 q = reinterpret_cast<const u32x4 *>(stage)[lane];
            const __amdgpu_buffer_rsrc_t rs = buf_rsrc(dst + img * npix * 32, (int)(npix * 64));
            __builtin_amdgcn_raw_buffer_store_b128(q, rs, ((y * d.w + x0) * 32 + 8 * lane) * 2, 0, 0);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int co = t * 16 + i;
                if (co >= CO) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    dst[((img * d.h + y) * d.w + x0 + 4 * kg + r) * CO + co] = (uint16_t)(hp[t][r >> 1] >> (16 * (r & 1)));
            }
        }
    };
    // the lane's three shifted operands of staged row r (input row y0 - 1 + r)
    auto lds3 = [&](int r) {
        const int base = (r * PW + 16 * sw + i) * 4 + kg;
        Row3 o;
        o.m = __builtin_bit_cast(bf16x8, lrows[base]);
        o.z = __builtin_bit_cast(bf16x8, lrows[base + 4]);
        o.p = __builtin_bit_cast(bf16x8, lrows[base + 8]);
        return o;
    };
    Row3 win[3];   // input rows y - 1, y, y + 1
    if constexpr (CI >= 32) {
        win[0] = lds3(0);
        win[1] = lds3(1);
    }
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
        const int y = y0 + rr;
        f32x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (CI >= 32) {
            win[2] = lds3(rr + 2);
#pragma unroll
            for (int ty = 0; ty < 3; ++ty)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    acc[t] = mfma(win[ty].m, bw[3 * ty + 0][t], acc[t]);
                    acc[t] = mfma(win[ty].z, bw[3 * ty + 1][t], acc[t]);
                    acc[t] = mfma(win[ty].p, bw[3 * ty + 2][t], acc[t]);
                }
            win[0] = win[1];
            win[1] = win[2];
        } else {
            // the 9 taps' channels packed along K: lane kg takes taps
            // (32 kc + 8 kg) / cpad .. + 8 / cpad - 1 of chunk kc
            // (read from the staged rows: staged row rr + dy, pixel 16 s + i + dx)
            constexpr int CP = cpad(CI), TPL = 8 / CP;
#pragma unroll
            for (int kc = 0; kc < NK; ++kc) {
                uint32_t wd[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int tt = 0; tt < TPL; ++tt) {
                    const int tap = (32 * kc + 8 * kg) / CP + tt;
                    if (tap < 9) {
                        const int q = (rr + tap / 3) * PW + 16 * sw + i + tap % 3;
#pragma unroll
                        for (int j = 0; j < WPT; ++j) wd[WPT * tt + j] = lsmall[q * WPT + j];
                    }
                }
                const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(wd[0], wd[1], wd[2], wd[3]));
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma(a, bw[kc][t], acc[t]);
            }
        }
        // lane holds D[pixel 4 kg + r][channel t 16 + i]; BF16 pairs of
        // pixels (4 kg, 4 kg + 1) and (4 kg + 2, 4 kg + 3)
        float v[NT][4];
        uint32_t hp[NT][2];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[t][r] = acc[t][r] + bv[t];
                if (relu) v[t][r] = fmaxf(v[t][r], 0.0f);
            }
            hp[t][0] = pack_bf2(v[t][0], v[t][1]);
            hp[t][1] = pack_bf2(v[t][2], v[t][3]);
        }
        if (out_f32) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int co = t * 16 + i;
                if (co >= CO) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) out_f32[((img * d.h + y) * d.w + x0 + 4 * kg + r) * CO + co] = v[t][r];
            }
        }
        if (out_bf) store_nhwc(out_bf, y, hp);
    }
}

// ---------------------------------------------------------------------------
// Backward pass of a layer with 32 input channels, in one kernel: the input
// gradient dx = conv(dy, transposed flipped weights), masked where the layer's
// input activation is 0 (ReLU), and the weight and bias gradients
//   dW[tap][ci][co] = sum over pixels of x[p + tap - (1,1)][ci] dy[p][co],
// both from the same rows of dy and x in LDS (BF16 NHWC, as the convolutions
// write them).  A workgroup of 4 waves takes R rows of a 64-pixel column chunk
// of one image, two rows at a time through a ring of four staged rows per
// tensor (pixels xc - 1 .. xc + 64, zeros outside the image); the next two
// rows are loaded into registers while the present ones are used.  (Four at a
// time leaves more in flight but not the registers for it: 16 .. 160 bytes of
// scratch a lane, 55 / 62 / 126 us where two take 32 / 52 / 70.)
//   dx: wave s takes the 16-pixel strip xc + 16 s and all 32 channels, as k_conv.
//   dW: M = 16 input channels, N = 16 output channels, K = 32 pixels; wave
//     (a, b) takes that pair of channel tiles over the whole chunk (CO = 2: a
//     and the half of the chunk).  K runs along pixels, which NHWC rows hold 64
//     bytes apart: the operands come by transposing LDS reads (each 16-lane
//     group reads 4 pixels of 16 channels and gets 4 pixels of its lane's
//     channel); three reads give 12 pixels, and so the operands of the three
//     taps of a row.
// The mask comes from the staged activations by the same reads.  kBwdFirst
// (layer 1): dx, wanted by layer 0's weight gradient alone, stays in LDS, where
// dW0[tap][ci][co] = sum of x0[p + tap - (1,1)][ci] dx[p][co] is formed too
// (M = 27 (tap, ci) pairs in two tiles).  Sums go to the workgroup's slots.  A layer
// on its own takes the same kernel: kBwdPlain stores dx as it stands (FP32, no
// mask; not where dx32 is null), kBwdInput forms layer 0's sums from its dy.
// Bound by HBM: dy and x read once, dx written once.  256 tiles of 64 x 64, as
// an input gradient and a weight gradient apart (which also needed channel-major
// copies of x and dy from the kernels before them) and here: CO = 2 (138 MB)
// 42 + 25 and 32 us (4.3 TB/s), 32 channels (201 MB) 52 + 47 and 52 us (3.9
// TB/s), FIRST (147 MB) 52 + 47 + layer 0's 24 and 70 us (2.1 TB/s: the chain
// through LDS with two waves per SIMD, 218 registers).
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// 4 pixels of the lane's channel from LDS (see above): p points at the 8 bytes
// of pixel lane % 16 / 4, channels 4 (lane % 4) .. + 3 of the lane's group
__device__ __forceinline__ s16x4 lds_tr(const uint16_t *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
}

__device__ __forceinline__ bf16x8 join8(s16x4 a, s16x4 b)
{
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// rows a step; staged rows (the step's and one either side); staged pixels; a row's room
constexpr int kBwdStep = 2, kBwdHalo = 2, kRing = kBwdStep + kBwdHalo, kBwdPx = 66, kBwdRow = 68;
enum BwdOut { kBwdMasked, kBwdFirst, kBwdPlain, kBwdInput };

template <int CO, BwdOut OUT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_bwd(const uint16_t *__restrict__ dy, const uint16_t *__restrict__ x,
                                             const float *__restrict__ x0, ConvDims d, int R,
                                             const uint16_t *__restrict__ wm, uint16_t *__restrict__ dx,
                                             float *__restrict__ dx32, float *__restrict__ part,
                                             float *__restrict__ part0)
{
    constexpr bool FIRST = OUT == kBwdFirst || OUT == kBwdInput;   // layer 0's sums too
    constexpr bool BACK = OUT != kBwdInput;                        // dx and dW
    static_assert(CO == 32 || !FIRST, "layer 0's weight gradient goes with a 32-channel layer");
    constexpr int NK = nchunk(CO);
    constexpr int SLOT = 9 * 32 * CO + CO, SLOT0 = 9 * 3 * 32 + 32;
    constexpr int XCH = kBwdPx * 4, XRO = kBwdRow * 4;   // 16-byte chunks of a staged 32-channel row; of its room
    constexpr int SPX = 72;                         // dwords of a staged 2-channel row (pixel xc + p at p + 4)
    constexpr int YB = CO == 32 ? kRing * XRO * 16 : kRing * SPX * 4;
    constexpr int GB = FIRST ? kBwdStep * 64 * 64 : 4 * 16 * 64;   // dx rows, or the waves' store stages
    constexpr int X0W = 36;                         // dwords of a staged channel of x0 (pixel p at element p + 2)
    constexpr int X0B = FIRST ? 2 * kRing * 3 * X0W * 4 : 0;
    __shared__ __align__(16) unsigned char lds[kRing * XRO * 16 + YB + GB + X0B];
    uint4 *lx = reinterpret_cast<uint4 *>(lds);
    unsigned char *lyb = lds + kRing * XRO * 16;
    uint16_t *lg = reinterpret_cast<uint16_t *>(lds + kRing * XRO * 16 + YB);
    uint32_t *l0 = reinterpret_cast<uint32_t *>(lds + kRing * XRO * 16 + YB + GB);   // [copy][row][ci][X0W]
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, kg = lane >> 4;
    const int cpr = (d.w + 63) / 64, rb = d.h / R;
    const int64_t unit = blockIdx.x;
    const int xc = (int)(unit % cpr) * 64, y0 = (int)((unit / cpr) % rb) * R;
    const int64_t img = unit / ((int64_t)cpr * rb), npix = (int64_t)d.h * d.w;
    const __amdgpu_buffer_rsrc_t xrs = buf_rsrc(BACK ? x + img * npix * 32 : nullptr, (int)(npix * 64));
    const __amdgpu_buffer_rsrc_t yrs = buf_rsrc(dy + img * npix * CO, (int)(npix * CO * 2));
    const __amdgpu_buffer_rsrc_t grs = buf_rsrc(dx ? dx + img * npix * 32 : nullptr, (int)(npix * 64));
    const __amdgpu_buffer_rsrc_t zrs = buf_rsrc(FIRST ? x0 + img * npix * 3 : nullptr, (int)(npix * 12));

    // --- staging: rows r .. r + n - 1 (0 = image row y0 - 1) of both tensors
    // (rows above and below the image lie outside the buffers and read zeros,
    // and so do the pixels left and right of it)
    auto xoff = [&](int r, int c) {
        const int px = xc - 1 + (c >> 2), yy = y0 - 1 + r;
        return px >= 0 && px < d.w && yy >= 0 && yy < d.h ? ((yy * d.w + px) * 32 + 8 * (c & 3)) * 2 : (int)(npix * 64);
    };
    auto soff = [&](int r, int p) {
        const int px = xc - 1 + p, yy = y0 - 1 + r;
        return px >= 0 && px < d.w && yy >= 0 && yy < d.h ? (yy * d.w + px) * 4 : (int)(npix * 4);
    };
    auto slot_of = [](int r) { return r % kRing; };
    constexpr int PER = (kBwdStep * XCH + 255) / 256, PERS = (kBwdStep * kBwdPx + 255) / 256;
    u32x4 tx[PER], ty[CO == 32 ? PER : 1];
    uint32_t ts[PERS], tz[FIRST ? PERS : 1][2];
    auto fetch = [&](int r0, int rows) {
        if constexpr (BACK) {
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int e = tid + 256 * k, r = e / XCH, c = e % XCH;
                const int off = r < rows ? xoff(r0 + r, c) : (int)(npix * 64);
                tx[k] = __builtin_amdgcn_raw_buffer_load_b128(xrs, off, 0, 0);
                if constexpr (CO == 32) ty[k] = __builtin_amdgcn_raw_buffer_load_b128(yrs, off, 0, 0);
            }
        }
        if constexpr (CO == 2) {
#pragma unroll
            for (int k = 0; k < PERS; ++k) {
                const int e = tid + 256 * k, r = e / kBwdPx;
                ts[k] = __builtin_amdgcn_raw_buffer_load_b32(yrs, r < rows ? soff(r0 + r, e % kBwdPx) : (int)(npix * 4), 0, 0);
            }
        }
        if constexpr (FIRST) {
#pragma unroll
            for (int k = 0; k < PERS; ++k) {
                const int e = tid + 256 * k, r = e / kBwdPx;
                const int off = r < rows ? 3 * soff(r0 + r, e % kBwdPx) : (int)(npix * 12);
                const float a = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(zrs, off, 0, 0));
                const float b = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(zrs, off, 4, 0));
                const float c = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(zrs, off, 8, 0));
                tz[k][0] = (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
                tz[k][1] = f2bf(c);
            }
        }
    };
    auto put = [&](int r0, int rows) {
        if constexpr (BACK) {
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int e = tid + 256 * k, r = e / XCH, c = e % XCH;
                if (r < rows) {
                    const int q = slot_of(r0 + r) * XRO + c;
                    lx[q] = __builtin_bit_cast(uint4, tx[k]);
                    if constexpr (CO == 32) reinterpret_cast<uint4 *>(lyb)[q] = __builtin_bit_cast(uint4, ty[k]);
                }
            }
        }
        if constexpr (CO == 2 || FIRST) {
#pragma unroll
            for (int k = 0; k < PERS; ++k) {
                const int e = tid + 256 * k, r = e / kBwdPx, p = e % kBwdPx;   // pixel xc - 1 + p
                if (r >= rows) continue;
                if constexpr (CO == 2) reinterpret_cast<uint32_t *>(lyb)[slot_of(r0 + r) * SPX + p + 3] = ts[k];
                if constexpr (FIRST) {
                    // two copies of each channel, one element apart, so that a
                    // pair of pixels at any shift is an aligned dword
                    uint16_t *z = reinterpret_cast<uint16_t *>(l0) + slot_of(r0 + r) * 3 * 2 * X0W;
                    uint16_t *z1 = z + kRing * 3 * 2 * X0W;
                    const uint16_t v[3] = {(uint16_t)tz[k][0], (uint16_t)(tz[k][0] >> 16), (uint16_t)tz[k][1]};
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        z[c * 2 * X0W + p + 1] = v[c];    // pixel xc + p' at element p' + 2
                        z1[c * 2 * X0W + p] = v[c];       // and at p' + 1
                    }
                }
            }
        }
    };

    // the input gradient's weights (as k_conv's: N = 16 t + i, K = 32 kc + 8 kg)
    bf16x8 bw[NK][2];
#pragma unroll
    for (int kc = 0; kc < NK; ++kc)
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if constexpr (BACK) bw[kc][t] = ld_bf16x8(wm + ((int64_t)(kc * 32 + t * 16 + i) * 32 + 8 * kg));
    const int a = CO == 32 ? wv >> 1 : wv & 1, b = CO == 32 ? wv & 1 : 0;
    const int hfirst = CO == 32 ? 0 : wv >> 1, hlast = CO == 32 ? 2 : hfirst + 1;   // the wave's halves of the chunk
    f32x4 acc[9], acc0 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float dbs = 0.0f, dbs0 = 0.0f;
    const int x0s = xc + 16 * wv;   // the wave's strip
    // element offset of a transposing read: pixel 8 kg + i / 4, channel 4 (i % 4) of a row
    const int tro = (8 * kg + (i >> 2)) * 32 + 4 * (i & 3);

    fetch(0, kBwdHalo);
    put(0, kBwdHalo);
    fetch(kBwdHalo, kBwdStep);
    for (int g = 0; g < R; g += kBwdStep) {
        put(g + kBwdHalo, kBwdStep);
        __syncthreads();
        if (g + kBwdStep < R) fetch(g + kBwdHalo + kBwdStep, kBwdStep);
        int ro[kRing];   // ring slots of rows g .. g + 3
#pragma unroll
        for (int k = 0; k < kRing; ++k) ro[k] = slot_of(g + k);
        if constexpr (!BACK) {
            // layer 0's output gradient: dy rows g, g + 1 of the workgroup's, zeros past the image
#pragma unroll
            for (int k = 0; k < kBwdStep; ++k) {
                const int px = xc + (tid >> 2), off = px < d.w ? (((y0 + g + k) * d.w + px) * 32 + 8 * (tid & 3)) * 2 : (int)(npix * 64);
                reinterpret_cast<u32x4 *>(lg)[k * 256 + tid] = __builtin_amdgcn_raw_buffer_load_b128(yrs, off, 0, 0);
            }
        }
        // --- input gradient
        if (BACK && x0s < d.w) {
            Row3 win[3];
            auto lds3 = [&](int k) {
                const uint4 *p = reinterpret_cast<const uint4 *>(lyb) + (ro[k] * kBwdRow + 16 * wv + i) * 4 + kg;
                Row3 o;
                o.m = __builtin_bit_cast(bf16x8, p[0]);
                o.z = __builtin_bit_cast(bf16x8, p[4]);
                o.p = __builtin_bit_cast(bf16x8, p[8]);
                return o;
            };
            if constexpr (CO == 32) {
                win[0] = lds3(0);
                win[1] = lds3(1);
            }
#pragma unroll
            for (int rr = 0; rr < kBwdStep; ++rr) {
                f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
                if constexpr (CO == 32) {
                    win[2] = lds3(rr + 2);
#pragma unroll
                    for (int tyy = 0; tyy < 3; ++tyy)
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            o[t] = mfma(win[tyy].m, bw[3 * tyy + 0][t], o[t]);
                            o[t] = mfma(win[tyy].z, bw[3 * tyy + 1][t], o[t]);
                            o[t] = mfma(win[tyy].p, bw[3 * tyy + 2][t], o[t]);
                        }
                    win[0] = win[1];
                    win[1] = win[2];
                } else {
                    constexpr int TPL = 4;   // taps a lane group packs (2 channels each)
#pragma unroll
                    for (int kc = 0; kc < NK; ++kc) {
                        uint32_t wd[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                        for (int tt = 0; tt < TPL; ++tt) {
                            const int tap = (32 * kc + 8 * kg) / 2 + tt;
                            if (tap < 9)
                                wd[tt] = reinterpret_cast<const uint32_t *>(lyb)[slot_of(g + rr + tap / 3) * SPX + 16 * wv + i +
                                                                                 tap % 3 + 3];
                        }
                        const bf16x8 op = __builtin_bit_cast(bf16x8, make_uint4(wd[0], wd[1], wd[2], wd[3]));
#pragma unroll
                        for (int t = 0; t < 2; ++t) o[t] = mfma(op, bw[kc][t], o[t]);
                    }
                }
                // lane: pixels 4 kg + r of the strip, channel 16 t + i
                if constexpr (OUT == kBwdPlain) {
                    if (!dx32) continue;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            dx32[(img * npix + (int64_t)(y0 + g + rr) * d.w + x0s + 4 * kg + r) * 32 + 16 * t + i] = o[t][r];
                    continue;
                }
                // its mask by a transposing read of the staged activations
                const uint16_t *xm = reinterpret_cast<const uint16_t *>(lx) +
                                     (ro[rr + 1] * kBwdRow + 16 * wv + 1 + 4 * kg + (i >> 2)) * 32 + 4 * (i & 3);
                uint16_t *stage = FIRST ? lg + (rr * 64 + 16 * wv) * 32 : lg + wv * 16 * 32;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const s16x4 mk = lds_tr(xm + 16 * t);
                    const uint32_t p0 = pack_bf2(o[t][0], o[t][1]), p1 = pack_bf2(o[t][2], o[t][3]);
                    const uint32_t h[4] = {p0 & 0xffffu, p0 >> 16, p1 & 0xffffu, p1 >> 16};
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        stage[(4 * kg + r) * 32 + 16 * t + i] = bf2f((uint16_t)mk[r]) > 0.0f ? (uint16_t)h[r] : (uint16_t)0;
                }
                if constexpr (!FIRST) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    const u32x4 q = reinterpret_cast<const u32x4 *>(stage)[lane];
                    __builtin_amdgcn_raw_buffer_store_b128(q, grs, (((y0 + g + rr) * d.w + x0s) * 32 + 8 * lane) * 2, 0, 0);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            }
        } else if constexpr (BACK && FIRST) {
            // pixels past the image add nothing to layer 0's sums
#pragma unroll
            for (int rr = 0; rr < kBwdStep; ++rr)
                reinterpret_cast<uint4 *>(lg + (rr * 64 + 16 * wv) * 32)[lane] = make_uint4(0u, 0u, 0u, 0u);
        }
        if constexpr (BACK) {
            // --- weight gradient: x rows g .. g + 3 against dy rows g + 1, g + 2
            bf16x8 gb[kBwdStep][2];
#pragma unroll
            for (int k = 0; k < kBwdStep; ++k)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (h < hfirst || h >= hlast) continue;
                    if constexpr (CO == 32) {
                        const uint16_t *p = reinterpret_cast<const uint16_t *>(lyb) + (ro[k + 1] * kBwdRow + 1 + 32 * h) * 32 + 16 * b + tro;
                        gb[k][h] = join8(lds_tr(p), lds_tr(p + 4 * 32));
                    } else {
                        // 8 pixels of channel i < 2 from the dword rows
                        const uint32_t *p = reinterpret_cast<const uint32_t *>(lyb) + ro[k + 1] * SPX + 4 + 32 * h + 8 * kg;
                        const uint4 u = reinterpret_cast<const uint4 *>(p)[0], v = reinterpret_cast<const uint4 *>(p)[1];
                        const uint32_t w[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
                        uint32_t o[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            o[e] = i == 0 ? (w[2 * e] & 0xffffu) | (w[2 * e + 1] << 16)
                                          : i == 1 ? (w[2 * e] >> 16) | (w[2 * e + 1] & 0xffff0000u) : 0u;
                        gb[k][h] = __builtin_bit_cast(bf16x8, make_uint4(o[0], o[1], o[2], o[3]));
                    }
                    if (a == 0) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) dbs += (float)gb[k][h][j];
                    }
                }
#pragma unroll
            for (int k = 0; k < kRing; ++k)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (h < hfirst || h >= hlast) continue;
                    const uint16_t *p = reinterpret_cast<const uint16_t *>(lx) + (ro[k] * kBwdRow + 32 * h) * 32 + 16 * a + tro;
                    // staged pixels 0 .. 11 from the lane's first; the operands
                    // shifted by 0, 1, 2 are dwords 0 .. 3, their odd pairs, 1 .. 4
                    const u32x2 q0 = __builtin_bit_cast(u32x2, lds_tr(p)), q1 = __builtin_bit_cast(u32x2, lds_tr(p + 4 * 32)),
                                q2 = __builtin_bit_cast(u32x2, lds_tr(p + 8 * 32));
                    const uint32_t w[5] = {q0.x, q0.y, q1.x, q1.y, q2.x};
                    const bf16x8 xs[3] = {
                        __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3])),
                        __builtin_bit_cast(bf16x8, make_uint4(__builtin_amdgcn_alignbyte(w[1], w[0], 2),
                                                              __builtin_amdgcn_alignbyte(w[2], w[1], 2),
                                                              __builtin_amdgcn_alignbyte(w[3], w[2], 2),
                                                              __builtin_amdgcn_alignbyte(w[4], w[3], 2))),
                        __builtin_bit_cast(bf16x8, make_uint4(w[1], w[2], w[3], w[4]))};
#pragma unroll
                    for (int tyy = 0; tyy < 3; ++tyy) {
                        const int q = k - tyy;   // dy row g + 1 + q
                        if (q < 0 || q >= kBwdStep) continue;
#pragma unroll
                        for (int t = 0; t < 3; ++t) acc[3 * tyy + t] = mfma(xs[t], gb[q][h], acc[3 * tyy + t]);
                    }
                }
        }
        if constexpr (FIRST) {
            // --- layer 0: (tap, ci) pairs 16 a .. + 15 against dx channels 16 b .. + 15
            __syncthreads();
            const int m = 16 * a + i, tap = m / 3, ci = m % 3;
#pragma unroll
            for (int rr = 0; rr < kBwdStep; ++rr)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint16_t *p = lg + (rr * 64 + 32 * h) * 32 + 16 * b + tro;
                    const bf16x8 gd = join8(lds_tr(p), lds_tr(p + 4 * 32));
                    // pixels 32 h + 8 kg + tap % 3 - 1 .. + 7: element + 2 of the first copy, + 1 of the second
                    uint32_t w[4] = {0u, 0u, 0u, 0u};
                    if (m < 27) {
                        const int e = 32 * h + 8 * kg + tap % 3 - 1;
                        const uint32_t *z = l0 + ((tap % 3 == 1 ? 0 : kRing) + slot_of(g + rr + tap / 3)) * 3 * X0W + ci * X0W;
                        const int q = (tap % 3 == 1 ? e + 2 : e + 1) >> 1;
#pragma unroll
                        for (int j = 0; j < 4; ++j) w[j] = z[q + j];
                    }
                    acc0 = mfma(__builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3])), gd, acc0);
                    if (a == 0) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) dbs0 += (float)gd[j];
                    }
                }
        }
        __syncthreads();
    }
    // lane holds D[ci = a 16 + 4 kg + r][co = b 16 + i]; the slot keeps the
    // real channels only
    if constexpr (CO == 2) {
        // the two halves of the chunk, added in a fixed order
        float *red = reinterpret_cast<float *>(lds);
        if (wv >= 2) {
#pragma unroll
            for (int t = 0; t < 9; ++t) reinterpret_cast<f32x4 *>(red)[((wv & 1) * 9 + t) * 64 + lane] = acc[t];
            red[2 * 9 * 64 * 4 + (wv & 1) * 64 + lane] = dbs;
        }
        __syncthreads();
        if (wv >= 2) return;
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t] += reinterpret_cast<f32x4 *>(red)[(wv * 9 + t) * 64 + lane];
        dbs += red[2 * 9 * 64 * 4 + wv * 64 + lane];
    }
    const int co = b * 16 + i;
    if constexpr (BACK) {
        float *slot = part + unit * SLOT;
        if (co < CO) {
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) slot[(t * 32 + a * 16 + 4 * kg + r) * CO + co] = acc[t][r];
        }
        if (a == 0) {
            dbs += __shfl_xor(dbs, 16);
            dbs += __shfl_xor(dbs, 32);
            if (kg == 0 && co < CO) slot[9 * 32 * CO + co] = dbs;
        }
    }
    if constexpr (FIRST) {
        float *s0 = part0 + unit * SLOT0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * a + 4 * kg + r;   // (tap, ci)
            if (m < 27) s0[m * 32 + co] = acc0[r];
        }
        if (a == 0) {
            dbs0 += __shfl_xor(dbs0, 16);
            dbs0 += __shfl_xor(dbs0, 32);
            if (kg == 0) s0[27 * 32 + co] = dbs0;
        }
    }
}

// Slot sums in two fixed-order stages (deterministic for a given slot count):
// groups of kRedGroup consecutive slots, then the groups in order.  One pair
// of launches reduces the slots of up to four layers (a training step's
// backward pass) at once.
constexpr int kRedGroup = 64;

struct RedSeg {
    const float *part;   // the layer's slots (each: dW (tap, ci, co), then db)
    float *dw, *db;
    int64_t nw;                   // weights (9 ci co); the slot holds nw + co floats
    int64_t nslots, nout, e0;     // slots, outputs (= slot floats), first output in the job
};

struct RedJob {
    RedSeg s[4];
    int nseg;
    int64_t total;
};

// output e of the job: its segment and the offset of its value within a slot
__device__ __forceinline__ const RedSeg &red_seg(const RedJob &J, int64_t e)
{
    int k = 0;
    while (k + 1 < J.nseg && e >= J.s[k + 1].e0) ++k;
    return J.s[k];
}

// grid (outputs / 256, slot groups): tmp[group][e] = sum of its slots
__global__ void k_wgrad_reduce1(RedJob J, float *__restrict__ tmp)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= J.total) return;
    const RedSeg &g = red_seg(J, e);
    const int64_t src = e - g.e0;
    const int64_t w0 = (int64_t)blockIdx.y * kRedGroup;
    const int64_t w1 = w0 + kRedGroup < g.nslots ? w0 + kRedGroup : g.nslots;
    float acc = 0.0f;
#pragma unroll 8
    for (int64_t w = w0; w < w1; ++w) acc += g.part[w * g.nout + src];
    tmp[(int64_t)blockIdx.y * J.total + e] = acc;
}

__global__ void k_wgrad_reduce2(RedJob J, const float *__restrict__ tmp, int64_t ngroups)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= J.total) return;
    const RedSeg &g = red_seg(J, e);
    float acc = 0.0f;
#pragma unroll 8
    for (int64_t k = 0; k < ngroups; ++k) acc += tmp[k * J.total + e];
    const int64_t le = e - g.e0;
    if (le < g.nw)
        g.dw[le] = acc;
    else
        g.db[le - g.nw] = acc;
}

// ---------------------------------------------------------------------------
// loss: mean logistic loss of the mask logit + lam * mean squared error of
// log10 Q over pixels with a finite target; writes dL/d(out) as BF16 (the
// operand precision of the backward contractions) and per-block sums
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_loss(const float *out, const float *mask, const float *logq, int64_t P,
                                              float lam, uint16_t *g, double *part)
{
    __shared__ double red[256];
    double s = 0.0;
    const double invP = 1.0 / (double)P;
    // (pixel indices fit 32 bits: n h w < 2^31)
    for (int p = (int)(blockIdx.x * blockDim.x + threadIdx.x); p < (int)P; p += (int)(gridDim.x * blockDim.x)) {
        const float2 zo = reinterpret_cast<const float2 *>(out)[p];
        const float z = zo.x, qh = zo.y, t = mask[p], tq = logq[p];
        const bool valid = isfinite(tq);
        const float sp = fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));
        const float dq = valid ? qh - tq : 0.0f;
        s += (double)(sp - t * z) + (double)lam * (double)dq * (double)dq;
        const float sig = 1.0f / (1.0f + expf(-z));
        const uint16_t g0 = f2bf((float)((sig - t) * invP)), g1 = f2bf((float)(2.0 * lam * dq * invP));
        reinterpret_cast<uint32_t *>(g)[p] = (uint32_t)g0 | ((uint32_t)g1 << 16);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] * invP;
}

// one block of 256 threads: strided partial sums, then a fixed-order tree
__global__ void __launch_bounds__(256) k_sum_parts(const double *part, int n, double *out)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int k = (int)threadIdx.x; k < n; k += 256) acc += part[k];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// Adam (Kingma & Ba 2015) on the FP32 master parameters
// b1, b2 are the decay rates, ob1 = 1 - b1 and ob2 = 1 - b2 (formed in FP64
// on the host: 1 - b2 taken in FP32 from the rounded 0.999f is 1.3e-5 off),
// c1, c2 the bias corrections 1 - b^t.
// The updated parameter is also written where k_prepare would put it in the
// prepared weights (its forward matrix entry, its transposed and flipped
// input-gradient entry, or its bias), so no separate preparation pass runs;
// the zero padding of the prepared matrices is never touched.
__device__ __forceinline__ void prep_store(int64_t e, float val, uint16_t *prep)
{
    const PrepLayout P = prep_layout();
    int l = 0;
    while (l < 3 && e >= master_w(l + 1)) ++l;
    const int Ci = kCi[l], Co = kCo[l];
    const int64_t le = e - master_w(l);
    if (le >= 9LL * Ci * Co) {
        reinterpret_cast<float *>(prep + P.bias[l])[le - 9LL * Ci * Co] = val;
        return;
    }
    const int co = (int)(le % Co), ci = (int)((le / Co) % Ci), tap = (int)(le / ((int64_t)Co * Ci));
    const uint16_t hb = f2bf(val);
    {
        const int k = Ci >= 32 ? 32 * tap + ci : tap * cpad(Ci) + ci;   // K index (chunk kc = k / 32)
        prep[P.fwd[l] + ((int64_t)(k / 32) * 16 * ntile(Co) + co) * 32 + k % 32] = hb;
    }
    if (l >= 1) {
        const int tf = 8 - tap;
        const int k = Co >= 32 ? 32 * tf + co : tf * cpad(Co) + co;
        prep[P.bwd[l] + ((int64_t)(k / 32) * 32 + ci) * 32 + k % 32] = hb;
    }
}

__global__ void k_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2, float ob1,
                       float ob2, float eps, float c1, float c2, uint16_t *prep)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const float ge = g[e];
        const float me = b1 * m[e] + ob1 * ge;
        const float ve = b2 * v[e] + ob2 * ge * ge;
        m[e] = me;
        v[e] = ve;
        const float pe = p[e] - lr * (me / c1) / (sqrtf(ve / c2) + eps);
        p[e] = pe;
        prep_store(e, pe, prep);
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

uint64_t cnn_prep_bytes() { return (uint64_t)prep_layout().total_u16 * 2; }

static const uint16_t *fwd_mat(const void *prep, int l)
{
    return static_cast<const uint16_t *>(prep) + prep_layout().fwd[l];
}
static const uint16_t *bwd_mat(const void *prep, int l)
{
    return static_cast<const uint16_t *>(prep) + prep_layout().bwd[l];
}
static const float *bias_of(const void *prep, int l)
{
    return reinterpret_cast<const float *>(static_cast<const uint16_t *>(prep) + prep_layout().bias[l]);
}

hipError_t cnn_prepare(const float *params, void *prep, hipStream_t st)
{
    hipLaunchKernelGGL(k_prepare, dim3(64), dim3(256), 0, st, params, static_cast<uint16_t *>(prep));
    return hipGetLastError();
}

static void conv_launch(int l, const void *in, ConvDims d, const void *prep, bool relu, uint16_t *out_bf, float *out_f32,
                        hipStream_t st)
{
    const dim3 grid((unsigned)(d.n * (d.h / kConvRows) * ((d.w + 63) / 64))), block(256);
    const uint16_t *wm = fwd_mat(prep, l);
    const float *b = bias_of(prep, l);
    if (l == 0)
        hipLaunchKernelGGL((k_conv<3, 32>), grid, block, 0, st, in, d, wm, b, relu, out_bf, out_f32);
    else if (l == 3)
        hipLaunchKernelGGL((k_conv<32, 2>), grid, block, 0, st, in, d, wm, b, relu, out_bf, out_f32);
    else
        hipLaunchKernelGGL((k_conv<32, 32>), grid, block, 0, st, in, d, wm, b, relu, out_bf, out_f32);
}

// Rows per workgroup of layer l's weight-gradient pass: the smallest power
// of two >= 4 dividing h that keeps its slots (one per workgroup: R rows of a
// 64-pixel column chunk) at 2048 / (waves per workgroup) or fewer, h at most
// -- about 2048 waves for the 32 x 32 layers and the narrow ones alike.
static int wgrad_rows(ConvDims d, int l)
{
    const int64_t cap = 2048 / (ntile(kCi[l]) * ntile(kCo[l]));
    int R = 4;
    while (R < d.h && d.h % (2 * R) == 0 && d.n * (d.h / R) * ((d.w + 63) / 64) > cap) R *= 2;
    return R;
}

static int64_t wgrad_slots(ConvDims d, int l) { return d.n * (d.h / wgrad_rows(d, l)) * ((d.w + 63) / 64); }

// first-stage groups of a reduction: enough for the layer with the most slots
static int64_t wgrad_groups(ConvDims d)
{
    int64_t m = 0;
    for (int l = 0; l < 4; ++l) m = wgrad_slots(d, l) > m ? wgrad_slots(d, l) : m;
    return (m + kRedGroup - 1) / kRedGroup;
}

static int64_t slot_floats(int l) { return 9LL * kCi[l] * kCo[l] + kCo[l]; }

static uint64_t al256(uint64_t b) { return (b + 255) & ~(uint64_t)255; }

static uint64_t slot_bytes(ConvDims d, int l) { return al256((uint64_t)wgrad_slots(d, l) * slot_floats(l) * 4); }

// slots of one layer (the largest layer's) and its group sums
static uint64_t wgrad_part_bytes(ConvDims d)
{
    uint64_t m = 0;
    for (int l = 0; l < 4; ++l) m = slot_bytes(d, l) > m ? slot_bytes(d, l) : m;
    return m + (uint64_t)wgrad_groups(d) * (9 * 32 * 32 + 32) * 4;
}

// slots of all four layers and the group sums of the whole parameter vector
static uint64_t train_part_bytes(ConvDims d)
{
    uint64_t b = 0;
    for (int l = 0; l < 4; ++l) b += slot_bytes(d, l);
    return b + (uint64_t)wgrad_groups(d) * QSQ_CNN_PARAMS * 4;
}

uint64_t cnn_wgrad_scratch_bytes(int64_t n, int h, int w) { return wgrad_part_bytes(ConvDims{n, h, w}); }

// the slots of layer l at `part` as a segment of a reduction job
static void add_seg(int l, int64_t slots, float *part, float *dw, float *db, RedJob &J)
{
    RedSeg &g = J.s[J.nseg++];
    g.part = part;
    g.dw = dw;
    g.db = db;
    g.nw = 9LL * kCi[l] * kCo[l];
    g.nslots = slots;
    g.nout = slot_floats(l);
    g.e0 = J.total;
    J.total += g.nout;
}

static void wgrad_reduce(const RedJob &J, float *tmp, ConvDims d, hipStream_t st)
{
    const int64_t groups = wgrad_groups(d);
    hipLaunchKernelGGL(k_wgrad_reduce1, dim3(blocks_for(J.total, 256), groups), dim3(256), 0, st, J, tmp);
    hipLaunchKernelGGL(k_wgrad_reduce2, dim3(blocks_for(J.total, 256)), dim3(256), 0, st, J, (const float *)tmp,
                       groups);
}

hipError_t cnn_layer_forward(int l, const void *prep, const void *in, int64_t n, int h, int w, float *out_f32,
                             uint16_t *out_bf, hipStream_t st)
{
    conv_launch(l, in, ConvDims{n, h, w}, prep, l < 3, out_bf, out_f32, st);
    return hipGetLastError();
}

hipError_t cnn_layer_backward(int l, const void *prep, const void *in, const uint16_t *dy, int64_t n, int h, int w,
                              float *dw, float *db, float *dx_f32, void *scratch, hipStream_t st)
{
    const ConvDims d{n, h, w};
    const int R = wgrad_rows(d, l == 3 ? 3 : 1);
    const int64_t units = wgrad_slots(d, l == 3 ? 3 : 1);
    float *part = static_cast<float *>(scratch);
    const dim3 grid((unsigned)units), block(256);
    const uint16_t *act = static_cast<const uint16_t *>(in), *noact = nullptr;
    const float *none = nullptr;
    uint16_t *nodx = nullptr;
    float *nof = nullptr;
    if (l == 0)
        hipLaunchKernelGGL((k_bwd<32, kBwdInput>), grid, block, 0, st, dy, noact, static_cast<const float *>(in), d, R,
                           noact, nodx, nof, nof, part);
    else if (l == 3)
        hipLaunchKernelGGL((k_bwd<2, kBwdPlain>), grid, block, 0, st, dy, act, none, d, R, bwd_mat(prep, l), nodx, dx_f32,
                           part, nof);
    else
        hipLaunchKernelGGL((k_bwd<32, kBwdPlain>), grid, block, 0, st, dy, act, none, d, R, bwd_mat(prep, l), nodx,
                           dx_f32, part, nof);
    RedJob J{};
    add_seg(l, units, part, dw, db, J);
    uint64_t m = 0;
    for (int k = 0; k < 4; ++k) m = slot_bytes(d, k) > m ? slot_bytes(d, k) : m;
    wgrad_reduce(J, part + m / 4, d, st);
    return hipGetLastError();
}

// Workspace of the whole-network calls: 3 hidden activations (BF16, 32 ch),
// output (FP32, 2 ch), output gradient (BF16, 2 ch), two hidden gradients
// (BF16, 32 ch), gradient vector, loss partials, weight-gradient slots.
struct CnnWs {
    uint16_t *act[3], *gout, *gh[2];
    float *out, *grad, *part;
    double *lpart, *loss;
    uint64_t total;
};

constexpr int kLossBlocks = 2048;

static CnnWs ws_layout(void *base, int64_t n, int h, int w)
{
    const uint64_t P = (uint64_t)n * h * w;
    CnnWs s{};
    char *p = static_cast<char *>(base);
    uint64_t o = 0;
    auto take = [&](uint64_t bytes) {
        char *q = p ? p + o : nullptr;
        o += al256(bytes);
        return q;
    };
    for (int k = 0; k < 3; ++k) s.act[k] = reinterpret_cast<uint16_t *>(take(P * 32 * 2));
    s.out = reinterpret_cast<float *>(take(P * 2 * 4));
    s.gout = reinterpret_cast<uint16_t *>(take(P * 2 * 2));
    for (int k = 0; k < 2; ++k) s.gh[k] = reinterpret_cast<uint16_t *>(take(P * 32 * 2));
    s.grad = reinterpret_cast<float *>(take(QSQ_CNN_PARAMS * 4));
    s.lpart = reinterpret_cast<double *>(take(kLossBlocks * 8));
    s.loss = reinterpret_cast<double *>(take(8));
    s.part = reinterpret_cast<float *>(take(train_part_bytes(ConvDims{n, h, w})));
    s.total = o;
    return s;
}

uint64_t cnn_workspace_bytes(int64_t n, int h, int w) { return ws_layout(nullptr, n, h, w).total; }

// forward through the four layers
static void forward_layers(const void *prep, const float *x, ConvDims d, float *out, const CnnWs &s, hipStream_t st)
{
    conv_launch(0, x, d, prep, true, s.act[0], nullptr, st);
    conv_launch(1, s.act[0], d, prep, true, s.act[1], nullptr, st);
    conv_launch(2, s.act[1], d, prep, true, s.act[2], nullptr, st);
    conv_launch(3, s.act[2], d, prep, false, nullptr, out, st);
}

hipError_t cnn_forward(const void *prep, const float *x, int64_t n, int h, int w, float *out, void *ws, hipStream_t st)
{
    forward_layers(prep, x, ConvDims{n, h, w}, out, ws_layout(ws, n, h, w), st);
    return hipGetLastError();
}

hipError_t cnn_train_step(float *params, float *adam_m, float *adam_v, int64_t t, float lr, const float *x,
                          const float *mask, const float *logq, int64_t n, int h, int w, float lam, void *prep,
                          float *grad_out, double *loss_out, void *ws, hipStream_t st)
{
    const CnnWs s = ws_layout(ws, n, h, w);
    const ConvDims d{n, h, w};
    const int64_t P = n * h * w;
    forward_layers(prep, x, d, s.out, s, st);
    const int lb = (int)(blocks_for(P, 256) < kLossBlocks ? blocks_for(P, 256) : kLossBlocks);
    hipLaunchKernelGGL(k_loss, dim3(lb), dim3(256), 0, st, s.out, mask, logq, P, lam, s.gout, s.lpart);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, st, s.lpart, lb, loss_out ? loss_out : s.loss);
    float *g = grad_out ? grad_out : s.grad;
    // layers 4 .. 2: weight gradients and the input gradient masked by the
    // ReLU of the layer below (its BF16 activation > 0); layer 2's kernel takes
    // layer 1's weight gradient along.  Each layer's slots in a region of their
    // own; one reduction of all four layers after the last.
    RedJob J{};
    float *part[4], *next = s.part;
    for (int l = 3; l >= 0; --l) {
        part[l] = next;
        next += slot_bytes(d, l) / 4;
    }
    const float *none = nullptr;
    float *nof = nullptr;
    const int R3 = wgrad_rows(d, 3), R1 = wgrad_rows(d, 1);   // (layers 1 and 2 alike)
    const int64_t u3 = wgrad_slots(d, 3), u1 = wgrad_slots(d, 1);
    hipLaunchKernelGGL((k_bwd<2, kBwdMasked>), dim3((unsigned)u3), dim3(256), 0, st, s.gout, s.act[2], none, d, R3,
                       bwd_mat(prep, 3), s.gh[0], nof, part[3], nof);
    hipLaunchKernelGGL((k_bwd<32, kBwdMasked>), dim3((unsigned)u1), dim3(256), 0, st, s.gh[0], s.act[1], none, d, R1,
                       bwd_mat(prep, 2), s.gh[1], nof, part[2], nof);
    hipLaunchKernelGGL((k_bwd<32, kBwdFirst>), dim3((unsigned)u1), dim3(256), 0, st, s.gh[1], s.act[0], x, d, R1,
                       bwd_mat(prep, 1), (uint16_t *)nullptr, nof, part[1], part[0]);
    for (int l = 3; l >= 0; --l)
        add_seg(l, l == 3 ? u3 : u1, part[l], g + master_w(l), g + master_w(l) + 9 * kCi[l] * kCo[l], J);
    wgrad_reduce(J, next, d, st);
    // Kingma & Ba's defaults; every constant is formed in FP64 and rounded once
    const double b1 = 0.9, b2 = 0.999;
    const float c1 = (float)(1.0 - pow(b1, (double)t)), c2 = (float)(1.0 - pow(b2, (double)t));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(QSQ_CNN_PARAMS, 256)), dim3(256), 0, st, params, g, adam_m, adam_v,
                       (int64_t)QSQ_CNN_PARAMS, lr, (float)b1, (float)b2, (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f,
                       c1, c2, static_cast<uint16_t *>(prep));
    return hipGetLastError();
}

}  // namespace qsq
