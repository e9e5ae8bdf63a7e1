// BF16 MFMA kernels (gfx950) of the warm-start U-Net: implicit-GEMM
// convolution (3x3 / 3x3x3 / 1x1, forward and input gradient), weight
// gradient, 2x2(x2) stride-2 transposed convolution (as GEMM with a
// depth-to-space / space-to-depth operand mode), max pooling, ReLU backward,
// bias gradient, masked MSE, Adam, and the feature / normalisation maps that
// connect the network to the LBM.
//
// Activations are pixel-major ("channels last", N[D]HWC) BF16 with an
// explicit channel stride and offset so that concatenation is a layout
// choice: a producer writes straight into its slice of the concatenated
// buffer.  Products accumulate in FP32 on the matrix cores
// (v_mfma_f32_16x16x32_bf16).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "unet_kernels.hpp"

namespace nn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __host__ inline float bf2f(uint16_t v) {
    union { uint32_t u; float f; } c;
    c.u = (uint32_t)v << 16;
    return c.f;
}

// float -> bf16, round to nearest even (NaN kept quiet): v_cvt_pk_bf16_f32,
// which equals the integer form x + 0x7fff + (bit 16 of x) >> 16 for every
// float (all 2^32 compared); two values cost one instruction instead of 14.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t f2bf2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// 8 BF16 values of a 16-byte vector as floats, and back.
__device__ inline void unpack8(uint4 v, float (&f)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = bf2f((uint16_t)(w[k] & 0xffffu));
        f[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16));
    }
}
__device__ inline uint4 pack8(const float (&f)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = f2bf2(f[2 * k], f[2 * k + 1]);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

constexpr int BM = 64, BN = 64;          // weight-gradient output tile (rows x K entries)

// Pixel index -> (b, z, y, x) on a grid of d x h x w per sample (pixel
// counts stay below 2^31: checked on the host).
struct Pix { int b, z, y, x; };
__device__ inline Pix pix_of(long long m64, int d, int h, int w) {
    unsigned m = (unsigned)m64;
    Pix p;
    unsigned q = m / (unsigned)w;
    p.x = (int)(m - q * (unsigned)w);
    m = q;
    q = m / (unsigned)h;
    p.y = (int)(m - q * (unsigned)h);
    m = q;
    q = m / (unsigned)d;
    p.z = (int)(m - q * (unsigned)d);
    p.b = (int)q;
    return p;
}

// K entry k of the implicit im2col matrix: channel ci and stencil offset
// (normal mode: k = tap * cin + ci over a ks^dims stencil centred on the
// pixel) or fine-grid sub-pixel (S2D mode: k = sub * cin + ci reads pixel
// (2z+sz, 2y+sy, 2x+sx), sub = sx + 2 sy + 4 sz).
struct Tap { int ci, dx, dy, dz; };
__device__ inline Tap tap_of(const ConvArgs &a, int k) {
    Tap t;
    const int tap = (int)((unsigned)k / (unsigned)a.cin);
    t.ci = k - tap * a.cin;
    if (a.flags & FLAG_S2D) {
        t.dx = tap & 1; t.dy = (tap >> 1) & 1; t.dz = (tap >> 2) & 1;
    } else if (a.ks == 3) {
        t.dx = tap % 3 - 1; t.dy = (tap / 3) % 3 - 1; t.dz = a.dims == 3 ? tap / 9 - 1 : 0;
    } else {
        t.dx = t.dy = t.dz = 0;
    }
    return t;
}

// The pixel of an im2col row, resolved once: its coordinates and the element
// offset of its first input channel (normal mode: the pixel itself; S2D: the
// fine-grid pixel (2z, 2y, 2x)).
struct Row { long long base; int x, y, z; bool valid; };
__device__ inline Row row_of(const ConvArgs &a, long long m) {
    Row r;
    r.valid = m < a.M;
    const Pix p = pix_of(r.valid ? m : 0, a.d, a.h, a.w);
    r.x = p.x; r.y = p.y; r.z = p.z;
    long long px;
    if (a.flags & FLAG_S2D) {
        const int fd = a.dims == 3 ? 2 * a.d : 1, fh = 2 * a.h, fw = 2 * a.w;
        px = (((long long)p.b * fd + (a.dims == 3 ? 2 * p.z : 0)) * fh + 2 * p.y) * fw + 2 * p.x;
    } else {
        px = (((long long)p.b * a.d + p.z) * a.h + p.y) * a.w + p.x;
    }
    r.base = px * a.in_cs + a.in_co;
    return r;
}

// A K entry resolved once per step: its tap offset from a row's base and the
// stencil displacement (for the zero-padding test).
struct KOff { long long delta; int dx, dy, dz; bool valid; };
__device__ inline KOff koff_of(const ConvArgs &a, int k) {
    KOff o;
    o.valid = k < a.K;
    const Tap t = tap_of(a, o.valid ? k : 0);
    o.dx = t.dx; o.dy = t.dy; o.dz = t.dz;
    long long d;
    if (a.flags & FLAG_S2D) {
        const int fh = 2 * a.h, fw = 2 * a.w;
        d = ((long long)t.dz * fh + t.dy) * fw + t.dx;
    } else {
        d = ((long long)t.dz * a.h + t.dy) * a.w + t.dx;
    }
    o.delta = d * a.in_cs + t.ci;
    return o;
}

// 16 bytes of the im2col matrix at (row, K offset), zero outside the grid.
__device__ inline uint4 im2col_load(const ConvArgs &a, const Row &r, const KOff &o) {
    bool ok = r.valid && o.valid;
    if (!(a.flags & FLAG_S2D)) {
        const unsigned xs = (unsigned)(r.x + o.dx), ys = (unsigned)(r.y + o.dy), zs = (unsigned)(r.z + o.dz);
        ok = ok && xs < (unsigned)a.w && ys < (unsigned)a.h && zs < (unsigned)a.d;
    }
    return ok ? *(const uint4 *)(a.in + r.base + o.delta) : make_uint4(0, 0, 0, 0);
}

// (b, z, y, x) of a flat pixel index kept as a mixed-radix counter: adding
// a fixed step digit by digit needs one carry per digit (each digit of the
// step is below its radix) and no division.
struct Cursor { int x, y, z, b; };
__device__ inline Cursor cursor_of(unsigned m, const ConvArgs &a) {
    const Pix p = pix_of(m, a.d, a.h, a.w);
    return Cursor{p.x, p.y, p.z, p.b};
}
__device__ inline void cursor_add(Cursor &c, const Cursor &s, const ConvArgs &a) {
    c.x += s.x;
    int k = c.x >= a.w;
    c.x -= k ? a.w : 0;
    c.y += s.y + k;
    k = c.y >= a.h;
    c.y -= k ? a.h : 0;
    c.z += s.z + k;
    k = c.z >= a.d;
    c.z -= k ? a.d : 0;
    c.b += s.b + k;
}
__device__ inline void cursor_inc(Cursor &c, const ConvArgs &a) { cursor_add(c, Cursor{1, 0, 0, 0}, a); }

__device__ inline bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// 8 FP32 values to a 16-byte aligned place, or added to those there.
__device__ inline void store8(float *p, const float (&v)[8], bool add) {
    float4 *dst = (float4 *)p;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        float4 x = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
        if (add) {
            const float4 old = dst[k];
            x = make_float4(old.x + x.x, old.y + x.y, old.z + x.z, old.w + x.w);
        }
        dst[k] = x;
    }
}

// ReLU backward: v[k] = 0 where the 8 activations y (NaN included) are not > 0.
__device__ inline void relu_mask(float (&v)[8], uint4 y) {
    float f[8];
    unpack8(y, f);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = f[k] > 0.f ? v[k] : 0.f;
}

// Output element of GEMM cell (m, c): returns the flat index and the bias
// channel; D2S maps column c = sub * Cr + co to the fine pixel.
__device__ inline long long out_index(const ConvArgs &a, long long m, int c, int &bias_c) {
    if (a.flags & FLAG_D2S) {
        const int cr = a.ncols >> a.dims;
        const int sub = c / cr, co = c - sub * cr;
        bias_c = co;
        const Pix p = pix_of(m, a.d, a.h, a.w);
        const int sx = sub & 1, sy = (sub >> 1) & 1, sz = (sub >> 2) & 1;
        const int fd = a.dims == 3 ? 2 * a.d : 1, fh = 2 * a.h, fw = 2 * a.w;
        const int zf = a.dims == 3 ? 2 * p.z + sz : 0;
        const long long f = (((long long)p.b * fd + zf) * fh + 2 * p.y + sy) * fw + 2 * p.x + sx;
        return f * a.out_cs + a.out_co + co;
    }
    bias_c = c;
    return m * a.out_cs + a.out_co + c;
}

// C[M x ncols] = im2col(in)[M x K] * W^T, W stored [ncols][K].
// A block computes a TBM x TBN tile with four wavefronts (2 x 2, each
// TBM/2 x TBN/2 of 16 x 16 x 32 BF16 MFMA tiles) over K steps of 64.  The
// LDS tiles are double-buffered: the next step's global loads are issued
// before the current step's MFMAs and land in the other buffer, so a step
// needs one barrier.  64 x 32 tiles serve the 32- and 8-channel layers
// without computing zero columns (and keep 5 blocks per CU).
// SPLIT: blockIdx.z takes K steps [z sper, (z + 1) sper) and the block
// stores its raw FP32 products to part[z][m][c] (k_conv_reduce adds the
// splits and applies the epilogue).
// TAPS: cin % 128 == 0, so that two or more K steps lie in one tap (or S2D
// sub-pixel): its place is found once and pointers advance by 64 channels in
// between, instead of divisions and tests per load (16 x 32^2, 256 -> 256 43 ->
// 37 us, four images of 64^2, 256 -> 128 32 -> 27 us; at 64 channels, one step
// a tap, 13 -> 15 us at 256^2, 64 -> 32).
template <int TBM, int TBN, bool TAPS, bool SPLIT = false>
__global__ void __launch_bounds__(256) k_conv(ConvArgs a, float *__restrict__ part = nullptr, int sper = 0) {
    constexpr int KB = 64;
    constexpr int WM = TBM / 2, WN = TBN / 2;
    constexpr int TI = WM / 16, TJ = WN / 16;
    constexpr int AL = TBM * 8 / 256, BL = TBN * 8 / 256;   // 16-byte loads per thread
    __shared__ __align__(16) uint16_t S[2 * (TBM + TBN) * KB];
    auto As = reinterpret_cast<uint16_t(*)[TBM][KB]>(S);
    auto Bs = reinterpret_cast<uint16_t(*)[TBN][KB]>(S + 2 * TBM * KB);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const long long m0 = (long long)blockIdx.x * TBM;
    const int n0 = blockIdx.y * TBN;
    const int kq = (t & 7) * 8;
    // 128-byte LDS rows; granules exchanged by (row >> 1) & 7 for the same reason as in granule()
    const int kw = ((t & 7) ^ ((t >> 4) & 7)) * 8;
    // rows of the im2col tile this thread loads: t / 8 + 32 l; their pixels are fixed
    Row row[AL];
#pragma unroll
    for (int l = 0; l < AL; ++l) row[l] = row_of(a, m0 + (t >> 3) + 32 * l);
    uint4 ra[AL], rb[BL];
    const int s0 = SPLIT ? (int)blockIdx.z * sper : 0;
    const int steps = SPLIT ? min((a.K + KB - 1) / KB, s0 + sper) : (a.K + KB - 1) / KB;
    int tap = 0, ci = 0;
    const uint16_t *pa[AL], *pb[BL];
    bool oka[AL];
    auto place = [&] {
        const KOff o = koff_of(a, tap * a.cin);
#pragma unroll
        for (int l = 0; l < AL; ++l) {
            const unsigned xs = (unsigned)(row[l].x + o.dx), ys = (unsigned)(row[l].y + o.dy), zs = (unsigned)(row[l].z + o.dz);
            oka[l] = row[l].valid && o.valid &&
                     ((a.flags & FLAG_S2D) || (xs < (unsigned)a.w && ys < (unsigned)a.h && zs < (unsigned)a.d));
            pa[l] = a.in + row[l].base + o.delta + ci + kq;
        }
    };
    if (TAPS) {
        tap = s0 * KB / a.cin;
        ci = s0 * KB - tap * a.cin;
        place();
#pragma unroll
        for (int l = 0; l < BL; ++l) pb[l] = a.wt + (long long)(n0 + (t >> 3) + 32 * l) * a.K + s0 * KB + kq;
    }
    auto load = [&](int k0) {
        if (TAPS) {
#pragma unroll
            for (int l = 0; l < AL; ++l) {
                ra[l] = oka[l] ? *(const uint4 *)pa[l] : make_uint4(0, 0, 0, 0);
                pa[l] += KB;
            }
#pragma unroll
            for (int l = 0; l < BL; ++l) {
                rb[l] = n0 + (t >> 3) + 32 * l < a.ncols ? *(const uint4 *)pb[l] : make_uint4(0, 0, 0, 0);
                pb[l] += KB;
            }
            ci += KB;
            if (ci == a.cin) {
                ci = 0;
                ++tap;
                place();
            }
            return;
        }
        const int k = k0 + kq;
        const bool kval = k < a.K;
        const KOff ko = koff_of(a, k);
#pragma unroll
        for (int l = 0; l < AL; ++l) ra[l] = im2col_load(a, row[l], ko);
#pragma unroll
        for (int l = 0; l < BL; ++l) {
            const int n = n0 + (t >> 3) + 32 * l;
            rb[l] = n < a.ncols && kval ? *(const uint4 *)(a.wt + (long long)n * a.K + k) : make_uint4(0, 0, 0, 0);
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int l = 0; l < AL; ++l) *(uint4 *)&As[buf][(t >> 3) + 32 * l][kw] = ra[l];
#pragma unroll
        for (int l = 0; l < BL; ++l) *(uint4 *)&Bs[buf][(t >> 3) + 32 * l][kw] = rb[l];
    };
    f32x4 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    load(s0 * KB);
    stash(s0 & 1);
    __syncthreads();
    for (int s = s0; s < steps; ++s) {
        const int buf = s & 1;
        if (s + 1 < steps) load((s + 1) * KB);
#pragma unroll
        for (int kh = 0; kh < KB; kh += 32) {
            const int kr = (((kh >> 3) + (lane >> 4)) ^ ((lane >> 1) & 7)) * 8;
            bf16x8 fb[TJ];
#pragma unroll
            for (int j = 0; j < TJ; ++j) fb[j] = as_bf16x8(*(const uint4 *)&Bs[buf][wn * WN + j * 16 + (lane & 15)][kr]);
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const bf16x8 fa = as_bf16x8(*(const uint4 *)&As[buf][wm * WM + i * 16 + (lane & 15)][kr]);
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[i][j], 0, 0, 0);
            }
        }
        if (s + 1 < steps) stash(buf ^ 1);
        __syncthreads();
    }
    if (SPLIT) {
        float *dst = part + (long long)blockIdx.z * a.M * a.ncols;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int c = n0 + wn * WN + j * 16 + (lane & 15);
                if (c >= a.ncols) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const long long m = m0 + wm * WM + i * 16 + (lane >> 4) * 4 + q;
                    if (m < a.M) dst[m * a.ncols + c] = acc[i][j][q];
                }
            }
        return;
    }
    const bool d2s = (a.flags & FLAG_D2S) != 0;
    const int cr = d2s ? a.ncols >> a.dims : a.ncols;      // D2S: columns sub * cr + co
    const uintptr_t base = a.out32 ? (uintptr_t)a.out32 : (uintptr_t)a.out;
    if (((a.out_cs | a.out_co | a.mask_cs | a.mask_co) & 7) == 0 && (!d2s || (cr & 7) == 0) &&
        ((base | (uintptr_t)a.mask) & 15) == 0) {
        // the tile goes through LDS (the buffers are free after the last barrier) so that each
        // thread stores 8 consecutive channels of a pixel (of the fine pixel for D2S, whose
        // 8-column groups stay inside one sub-pixel) with 16-byte writes
        constexpr int TL = TBN + 4;
        static_assert(TBM * TL * 4 <= (int)sizeof(S), "epilogue tile must fit in the buffers");
        float *T = reinterpret_cast<float *>(S);
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int cl = wn * WN + j * 16 + (lane & 15), c = n0 + cl;
                const float b = a.bias && c < a.ncols ? a.bias[d2s ? c - (c / cr) * cr : c] : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v = acc[i][j][q] + b;
                    if (a.flags & FLAG_RELU) v = v > 0.f ? v : 0.f;
                    T[(wm * WM + i * 16 + (lane >> 4) * 4 + q) * TL + cl] = v;
                }
            }
        __syncthreads();
        constexpr int CG = TBN / 8;
        for (int e = t; e < TBM * CG; e += 256) {
            const int ml = e / CG, cl = (e - ml * CG) * 8;
            const long long m = m0 + ml;
            const int c = n0 + cl;
            if (m >= a.M || c >= a.ncols) continue;
            const float *src = &T[ml * TL + cl];
            int bc;
            const long long o = out_index(a, m, c, bc);
            if (a.out32) {
                float *dst = a.out32 + o;
                const int nk = a.ncols - c < 8 ? a.ncols - c : 8;
                if (nk == 8) {
                    float4 v0 = make_float4(src[0], src[1], src[2], src[3]);
                    float4 v1 = make_float4(src[4], src[5], src[6], src[7]);
                    if (a.flags & FLAG_ACC) {
                        const float4 o0 = *(const float4 *)dst, o1 = *(const float4 *)(dst + 4);
                        v0.x += o0.x; v0.y += o0.y; v0.z += o0.z; v0.w += o0.w;
                        v1.x += o1.x; v1.y += o1.y; v1.z += o1.z; v1.w += o1.w;
                    }
                    *(float4 *)dst = v0;
                    *(float4 *)(dst + 4) = v1;
                } else {
                    for (int k = 0; k < nk; ++k) dst[k] = (a.flags & FLAG_ACC) ? dst[k] + src[k] : src[k];
                }
                continue;
            }
            uint16_t *dst = a.out + o;
            if (c + 8 <= a.ncols) {
                float v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = src[k];
                if (a.flags & FLAG_ACC) {
                    const uint4 old = *(const uint4 *)dst;
                    const uint32_t ow[4] = {old.x, old.y, old.z, old.w};
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[k] += bf2f((uint16_t)(ow[k >> 1] >> (16 * (k & 1))));
                }
                if (a.mask) relu_mask(v, *(const uint4 *)(a.mask + m * a.mask_cs + a.mask_co + c));
                uint32_t pw[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) pw[k] = f2bf2(v[2 * k], v[2 * k + 1]);
                *(uint4 *)dst = make_uint4(pw[0], pw[1], pw[2], pw[3]);
            } else {
                for (int k = 0; k < a.ncols - c; ++k) {
                    float v = src[k];
                    if (a.flags & FLAG_ACC) v += bf2f(dst[k]);
                    if (a.mask && !(bf2f(a.mask[m * a.mask_cs + a.mask_co + c + k]) > 0.f)) v = 0.f;
                    dst[k] = f2bf(v);
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int c = n0 + wn * WN + j * 16 + (lane & 15);
            if (c >= a.ncols) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const long long m = m0 + wm * WM + i * 16 + (lane >> 4) * 4 + q;
                if (m >= a.M) continue;
                int bc;
                const long long o = out_index(a, m, c, bc);
                float v = acc[i][j][q] + (a.bias ? a.bias[bc] : 0.f);
                if (a.flags & FLAG_RELU) v = v > 0.f ? v : 0.f;
                if (a.out32) {
                    a.out32[o] = (a.flags & FLAG_ACC) ? a.out32[o] + v : v;
                } else {
                    if (a.flags & FLAG_ACC) v += bf2f(a.out[o]);
                    if (a.mask && !(bf2f(a.mask[m * a.mask_cs + a.mask_co + c]) > 0.f)) v = 0.f;
                    a.out[o] = f2bf(v);
                }
            }
        }
}

// Loads through a buffer resource: an offset past its range reads 0, which
// stands for the zero padding.
constexpr unsigned OOB = 0xFFFFFF00u;
__device__ inline __amdgpu_buffer_rsrc_t rsrc_of(const uint16_t *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, (int)bytes, 0x00020000);
}
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ inline uint4 bload16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// The same GEMM for small layers (one image, the deep levels), which are bound
// by latency: a wavefront takes 32 pixels x 32 output channels over the K range
// of one split and loads its MFMA operands straight from memory (lane l: pixel
// or channel l & 15, K entries 8 (l >> 4) ..; rows of weights permuted as in
// k_conv3x3_rows), DS K steps of 32 ahead; the S wavefronts of a tile add their
// sums in LDS in split order.  Products and splits are added in the order of
// k_conv<SPLIT> and k_conv_reduce, in one launch and without partials in
// memory.  S = 1: the block's four wavefronts take four tiles.
// cin % 32 == 0: a step lies in one tap, whose place is scalar arithmetic; the
// input and the weights are addressed by 31-bit offsets (host-checked).
__global__ void __launch_bounds__(1024) k_conv_direct(ConvArgs a, int S, int sper, unsigned in_bytes) {
    constexpr int DS = 4;                              // (6 spill)
    extern __shared__ float sums[];                    // [split][pixel tile][2][lane][4]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tiles_n = (a.ncols + 31) / 32;
    const int nb = (int)gridDim.x, q8 = nb >> 3, r8 = nb & 7, xcd = (int)blockIdx.x & 7;
    const int bt = xcd * q8 + (xcd < r8 ? xcd : r8) + ((int)blockIdx.x >> 3);
    const int tile = S == 1 ? bt * 4 + wave : bt, z = S == 1 ? 0 : wave;
    const int n0 = tile % tiles_n * 32, kl = 8 * (lane >> 4), pl = lane & 15;
    const long long m0 = (long long)(tile / tiles_n) * 32;
    const __amdgpu_buffer_rsrc_t ri = rsrc_of(a.in, in_bytes), rw = rsrc_of(a.wt, (unsigned)a.ncols * a.K * 2u);
    constexpr unsigned OUT = 0x80000000u;              // past both ranges, also with a channel offset added
    int k = z * sper * 64, tap = k / a.cin, ci = k - tap * a.cin;        // the step to load
    const int steps = (min(a.K, (z + 1) * sper * 64) - k) / 32;
    Row row[2];
    unsigned io[2], wo[2];                             // byte offsets: the tap's pixel or OUT; the weight row or OUT
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        row[i] = row_of(a, m0 + 16 * i + pl);
        const int n = n0 + 8 * (pl >> 2) + 4 * i + (pl & 3);
        wo[i] = n < a.ncols ? 2u * (unsigned)(n * a.K + kl) : OUT;
    }
    auto place = [&] {
        int dx = 0, dy = 0, dz = 0;
        if (a.ks == 3) {
            dz = a.dims == 3 ? tap / 9 - 1 : 0;
            const int t9 = a.dims == 3 ? tap % 9 : tap;
            dy = t9 / 3 - 1;
            dx = t9 % 3 - 1;
        }
        const int delta = ((dz * a.h + dy) * a.w + dx) * a.in_cs + kl;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bool ok = row[i].valid && (unsigned)(row[i].x + dx) < (unsigned)a.w &&
                            (unsigned)(row[i].y + dy) < (unsigned)a.h && (unsigned)(row[i].z + dz) < (unsigned)a.d;
            io[i] = ok ? 2u * (unsigned)((int)row[i].base + delta) : OUT;
        }
    };
    uint4 vi[DS][2], vw[DS][2];
    auto fetch = [&](int d) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            vi[d][i] = bload16(ri, io[i] + 2u * (unsigned)ci);
            vw[d][i] = bload16(rw, wo[i] + 2u * (unsigned)k);
        }
        k += 32;
        ci += 32;
        if (ci == a.cin) {
            ci = 0;
            ++tap;
            place();
        }
    };
    place();
#pragma unroll
    for (int d = 0; d < DS; ++d)
        if (d < steps) fetch(d);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < steps; s += DS)
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            if (s + d >= steps) break;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vw[d][j]), as_bf16x8(vi[d][i]), acc[i][j], 0, 0, 0);
            if (s + d + DS < steps) fetch(d);
        }
    int i0 = 0, i1 = 2;
    if (S > 1) {
        f32x4 *dst = (f32x4 *)sums;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) dst[((z * 2 + i) * 2 + j) * 64 + lane] = acc[i][j];
        __syncthreads();
        if (wave >= 2) return;
        f32x4 v[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        for (int p = 0; p < S; ++p)
#pragma unroll
            for (int j = 0; j < 2; ++j) v[j] += dst[((p * 2 + wave) * 2 + j) * 64 + lane];
        i0 = wave;
        i1 = wave + 1;
        acc[0][0] = acc[1][0] = v[0];
        acc[0][1] = acc[1][1] = v[1];
    }
    const int c = n0 + kl;                             // the lane's 8 output channels
    if (c >= a.ncols) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const long long m = m0 + 16 * i + pl;
        if (i < i0 || i >= i1 || m >= a.M) continue;
        int bc;
        const long long o = out_index(a, m, c, bc);
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v[q] = acc[i][q >> 2][q & 3] + (a.bias ? a.bias[bc + q] : 0.f);
            if (a.flags & FLAG_RELU) v[q] = v[q] > 0.f ? v[q] : 0.f;
        }
        if (a.out32) {
            store8(a.out32 + o, v, (a.flags & FLAG_ACC) != 0);
            continue;
        }
        uint16_t *dst = a.out + o;
        if (a.flags & FLAG_ACC) {
            float old[8];
            unpack8(*(const uint4 *)dst, old);
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] += old[q];
        }
        if (a.mask) relu_mask(v, *(const uint4 *)(a.mask + m * a.mask_cs + a.mask_co + c));
        *(uint4 *)dst = pack8(v);
    }
}

// 3 x 3 (3 x 3 x 3) convolution on image rows (the plane sizes must be
// multiples of 8 x 32 pixels; input channels in chunks of 32, a last, shorter
// chunk zero-filled).  Per chunk a block's input patch of 8 x 32 pixels with
// its one-pixel halo is staged in LDS once.
//
// A wavefront computes WY rows x 16 columns x 32 output channels.  It holds the
// 9 taps' weights of the chunk in registers and walks down the patch: the
// fragment of input row yi at column offset dx serves output rows yi, yi - 1
// and yi - 2 (taps dy = 0, 1, 2), so 3 (WY + 2) fragments feed its 18 WY MFMAs
// (9 WY fragments with one per tap and output row).  Every output still adds
// its taps in the order dy, dx, chunk by chunk.
//
// The weights are the A operand (rows = output channels) and row r of the
// 16-row tile j stands for channel 8 (r >> 2) + 4 j + (r & 3), so that a lane
// ends up with 8 consecutive channels of one pixel and stores them with one
// 16-byte write straight from its accumulators.
//
// Bound by memory at 32 channels (16 x 256^2, 32 -> 32: 32.5 us, 4.1 TB/s),
// by the two barriers of a stage above (64 -> 32: 57.7 us, 670 TFLOP/s; 64^2,
// 256 -> 128: 37.4 us, 1035 TFLOP/s).  A fragment per tap and output row with
// the output staged through LDS took 75 us (64 -> 32) and 97 us instead of 48
// us (32 -> 64).
constexpr int HY = 8, HX = 32, HPX = HX + 2;         // tile rows and columns, patch columns
constexpr int HP = (HY + 2) * HPX;                   // patch pixels
constexpr int HC = 32;                               // chunk channels
// 16-byte granule of channels 8 g .. 8 g + 7 in the 64-byte LDS row of pixel (or weight row) r.  A 16-byte operand
// read serves the lanes 0-3, 12-15, 20-23, 24-27 at a time, then 4-7, 8-11, 16-19, 28-31, and so on: with this
// exchange the 16 rows they touch, at whichever row they start, cover all 64 banks (rows padded to 80 bytes met
// every bank twice: 8.8 instead of 4.4 cycles a read).
__device__ inline int granule(int r, int g) { return g ^ ((r >> 1) & 2); }

// bload16 straight to LDS: lane l of the wavefront fills the 16 bytes at
// dst + 16 l (dst uniform).  Complete after lds_wait() and a barrier.
__device__ inline void bload16_lds(__amdgpu_buffer_rsrc_t r, uint16_t *dst, unsigned off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, off, 0, 0, 0);
}
__device__ inline void lds_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Blocks take TN output channels: 64 (two column halves x two channel halves,
// WY = 8), or 32 (two column halves x two row halves, WY = 4), and walk over
// `per` consecutive tiles: the next stage's patch, of this tile or of the next
// one, is loaded while the current stage multiplies.  A stage is a (chunk,
// input plane) pair: in 3D a tile stays on one plane z and, per chunk, takes
// the input planes z - 1, z, z + 1 in turn (taps dz * 9 + dy * 3 + dx), skipping
// planes outside the volume.  RES: a 2D layer of one chunk, whose weights stay
// in registers throughout; else every stage's weights pass through LDS, where
// the next stage's are loaded (straight from memory) as soon as all wavefronts
// have read the current ones.
// MODE: OUT_PLAIN BF16 output, overwritten; OUT_MASK the same behind a ReLU
// backward; OUT_ANY accumulated or FP32 (no mask).
enum { OUT_PLAIN, OUT_MASK, OUT_ANY };
template <int TN, int DIMS, bool RES, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_conv3x3_rows(ConvArgs a, int per) {
    constexpr int WY = TN == 32 ? 4 : 8;
    __shared__ __align__(16) uint16_t P[HP * HC];
    __shared__ __align__(16) uint16_t Wl[9 * TN * HC];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int tiles_x = a.w / HX, tiles_y = a.h / HY, tiles_n = (a.ncols + TN - 1) / TN;
    const int tiles = tiles_x * tiles_y * a.n * a.d;
    // blocks of one XCD (every eighth) take neighbouring runs of tiles; the channel tiles of a run are adjacent
    const int nb = (int)gridDim.x, q8 = nb >> 3, r8 = nb & 7, xcd = (int)blockIdx.x & 7;
    const int bt = xcd * q8 + (xcd < r8 ? xcd : r8) + ((int)blockIdx.x >> 3);
    const int n0 = (bt % tiles_n) * TN;
    const int i0 = (bt / tiles_n) * per, i1 = min(i0 + per, tiles);
    if (i0 >= i1) return;
    const int wx = (wave & 1) * 16, wy = TN == 32 ? (wave >> 1) * WY : 0, wn = TN == 32 ? 0 : (wave >> 1) * 32;
    constexpr int NDZ = DIMS == 3 ? 3 : 1;
    constexpr int NPL = (HP * 4 + 255) / 256;
    const int nst = ((a.cin + HC - 1) / HC) * NDZ;    // stages of a tile
    const int g8 = (t & 3) * 8;                       // the thread's channels of a pixel
    int tx = 0, ty = 0, z = 0, b = 0;                 // the tile being loaded
    auto place = [&](int i) {
        tx = i % tiles_x;
        i /= tiles_x;
        ty = i % tiles_y;
        i /= tiles_y;
        z = DIMS == 3 ? i % a.d : 0;
        b = DIMS == 3 ? i / a.d : i;
    };
    auto next_stage = [&](int st) {
        do ++st; while (DIMS == 3 && st < nst && (unsigned)(z + st % NDZ - 1) >= (unsigned)a.d);
        return st;
    };
    uint4 pv[NPL];
    auto load_patch = [&](int st) {
        const int c0 = (st / NDZ) * HC, zz = DIMS == 3 ? z + st % NDZ - 1 : 0;
        const int y0 = ty * HY - 1, x0 = tx * HX - 1;  // the patch's first pixel
        const uint16_t *in = a.in + ((((long long)b * a.d + zz) * a.h + y0) * a.w + x0) * a.in_cs + a.in_co + c0;
        const __amdgpu_buffer_rsrc_t r = rsrc_of(in, (unsigned)(((HY + 1) * a.w + HPX) * a.in_cs) * 2u);
        const bool con = c0 + g8 < a.cin;
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            const int pp = (t >> 2) + 64 * k;
            const int py = pp / HPX, px = pp - py * HPX;
            const bool on = con && pp < HP && (unsigned)(y0 + py) < (unsigned)a.h && (unsigned)(x0 + px) < (unsigned)a.w;
            pv[k] = bload16(r, on ? (unsigned)((py * a.w + px) * a.in_cs + g8) * 2u : OOB);
        }
    };
    // The stage's weights to LDS: rows (tap, then the rows of the 16-row tiles in operand order).
    auto load_weights = [&](int st) {
        const int c0 = (st / NDZ) * HC, off = n0 * a.K + (DIMS == 3 ? (st % NDZ) * 9 * a.cin : 0) + c0;
        // channels past ncols lie past the range
        const __amdgpu_buffer_rsrc_t r = rsrc_of(a.wt + off, (unsigned)(a.ncols * a.K - off) * 2u);
#pragma unroll
        for (int k = 0; k < (9 * TN * 4 + 255) / 256; ++k) {
            const int base = (4 * k + wave) * 64;
            if (base >= 9 * TN * 4) break;
            const int row = (base + lane) >> 2, g = granule(row, lane & 3) * 8;
            const int tap = row / TN, q = row - tap * TN;
            const int n = (q & ~31) + ((q & 15) >> 2) * 8 + ((q >> 4) & 1) * 4 + (q & 3);
            bload16_lds(r, Wl + base * 8, c0 + g < a.cin ? (unsigned)(n * a.K + tap * a.cin + g) * 2u : OOB);
        }
    };
    // the lane's granules of weight row (tap 0, tile 0) and of the patch pixels (0, dx)
    const uint16_t *wl = Wl + (wn + (lane & 15)) * HC + granule(lane & 15, lane >> 4) * 8;
    const uint16_t *pl[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int px = wx + (lane & 15) + dx;
        pl[dx] = P + (wy * HPX + px) * HC + granule(px, lane >> 4) * 8;
    }
    bf16x8 wf[9][2];
    auto read_weights = [&] {
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int j = 0; j < 2; ++j) wf[tap][j] = as_bf16x8(*(const uint4 *)(wl + (tap * TN + 16 * j) * HC));
    };
    f32x4 acc[WY][2];
#pragma unroll
    for (int i = 0; i < WY; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int c = n0 + wn + (lane >> 4) * 8;          // the lane's output channels
    const bool relu = (a.flags & FLAG_RELU) != 0;
    place(i0);
    int i = i0, st = next_stage(-1);
    load_patch(st);
    load_weights(st);
    if (RES) {
        lds_wait();
        __syncthreads();
        read_weights();
    }
    while (true) {
        if (!RES) lds_wait();                         // this stage's weights
        __syncthreads();                              // the previous stage's operand reads are done
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            const int pp = (t >> 2) + 64 * k;
            if (pp < HP) *(uint4 *)&P[pp * HC + granule(pp % HPX, t & 3) * 8] = pv[k];
        }
        if (!RES) read_weights();
        __syncthreads();
        // the next stage, of this tile or of the next one
        const int y = ty * HY + wy, x = tx * HX + wx + (lane & 15);
        const long long m0 = (((long long)b * a.d + z) * a.h + y) * a.w + x;
        st = next_stage(st);
        const bool last = st >= nst;
        if (last && ++i < i1) {
            place(i);
            st = next_stage(-1);
        }
        if (i < i1) {
            load_patch(st);
            if (!RES) load_weights(st);
        }
        // the fragments of row yi + 1 are read while row yi multiplies (left alone, the compiler reads each
        // fragment right before its use and waits for it)
        bf16x8 f[2][3];
        auto read_row = [&](int yi) {
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) f[yi & 1][dx] = as_bf16x8(*(const uint4 *)(pl[dx] + yi * HPX * HC));
        };
        read_row(0);
#pragma unroll
        for (int yi = 0; yi < WY + 2; ++yi) {
            if (yi + 1 < WY + 2) read_row(yi + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int o = yi - dy;
                    if (o < 0 || o >= WY) continue;
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[o][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[dy * 3 + dx][j], f[yi & 1][dx], acc[o][j], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!last) continue;
        // 8 channels of pixel (y + r, x) per lane
        if (c < a.ncols) {
            float bias[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (a.bias)
#pragma unroll
                for (int k = 0; k < 8; ++k) bias[k] = a.bias[c + k];
            constexpr int MB = 4;                     // mask loads in flight (registers)
            uint4 mk[MB];
#pragma unroll
            for (int r = 0; r < WY; ++r) {
                if (MODE == OUT_MASK && r % MB == 0)
#pragma unroll
                    for (int k = 0; k < MB; ++k)
                        mk[k] = *(const uint4 *)(a.mask + (m0 + (long long)(r + k) * a.w) * a.mask_cs + a.mask_co + c);
                const long long o = (m0 + (long long)r * a.w) * a.out_cs + a.out_co + c;
                float v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    v[k] = acc[r][k >> 2][k & 3] + bias[k];
                    v[k] = relu && !(v[k] > 0.f) ? 0.f : v[k];
                }
                if (MODE == OUT_ANY && a.out32) {
                    float *dst = a.out32 + o;
#pragma unroll
                    for (int k = 0; k < 8; ++k) dst[k] = (a.flags & FLAG_ACC) ? dst[k] + v[k] : v[k];
                    continue;
                }
                uint16_t *dst = a.out + o;
                if (MODE == OUT_ANY && (a.flags & FLAG_ACC)) {
                    float old[8];
                    unpack8(*(const uint4 *)dst, old);
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[k] += old[k];
                }
                if (MODE == OUT_MASK) relu_mask(v, mk[r % MB]);
                *(uint4 *)dst = pack8(v);
            }
        }
        if (i >= i1) break;
#pragma unroll
        for (int r = 0; r < WY; ++r) acc[r][0] = acc[r][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// 1 x 1 convolution (normal and D2S: the head, its input gradient and the
// transposed convolutions) of few input channels.  Bound by memory; nothing is
// shared between pixels, so nothing goes through LDS: a wavefront keeps the
// weights of 32 output channels in registers (KS K steps of 32) and walks over
// groups of PT x 16 pixels, whose rows of A are MFMA operands as they lie in
// memory (lane l: pixel l & 15, K entries 8 (l >> 4) ..); the next group's are
// loaded before this one's MFMAs.  Operands, channel order and stores as in
// k_conv3x3_rows; products are added in the order of k_conv.  The gw wavefronts
// of a block that take neighbouring channels read the same pixels.
//
// 16 x 256^2 (before, in k_conv's 64 x 32 and 64 x 64 tiles): 32 -> 8 in FP32
// 18 us, 5.6 TB/s (43 us); 8 -> 32 with its ReLU mask 24 us (47 us); 16 x 128^2
// 64 -> 4 x 32 D2S 28 us (49 us), 16 x 64^2 128 -> 4 x 64 26 us (29 us).
template <int KS, int PT>
__global__ void __launch_bounds__(256) k_conv1x1(ConvArgs a, int gw) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n0 = ((int)blockIdx.y * gw + wave % gw) * 32;
    if (n0 >= a.ncols) return;
    const int walkers = (int)gridDim.x * (4 / gw);
    const int tiles = (int)((a.M + 16 * PT - 1) / (16 * PT));
    const int kl = 8 * (lane >> 4), pl = lane & 15;
    bf16x8 wf[KS][2];
    bool kv[KS];
    int ko[KS];                                        // (entries past K: the pixel's first, replaced by zeros)
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int k = 32 * s + kl;
        kv[s] = k < a.K;
        ko[s] = kv[s] ? k : 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + 8 * (pl >> 2) + 4 * j + (pl & 3);
            wf[s][j] = as_bf16x8(kv[s] && n < a.ncols ? *(const uint4 *)(a.wt + (long long)n * a.K + k) : make_uint4(0, 0, 0, 0));
        }
    }
    const int c = n0 + kl;                             // the lane's output channels
    const bool d2s = (a.flags & FLAG_D2S) != 0, cv = c < a.ncols;
    const int cr = d2s ? a.ncols >> a.dims : a.ncols, bc = d2s ? c - c / cr * cr : c;
    float bias[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (a.bias && cv)
#pragma unroll
        for (int k = 0; k < 8; ++k) bias[k] = a.bias[bc + k];
    auto load = [&](int t, uint4 (&v)[PT][KS]) {
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const long long m = (long long)(t * PT + p) * 16 + pl;
            const uint16_t *src = a.in + (m < a.M ? m : 0) * a.in_cs + a.in_co;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const uint4 x = *(const uint4 *)(src + ko[s]);
                v[p][s] = kv[s] ? x : make_uint4(0, 0, 0, 0);
            }
        }
    };
    int t = (int)blockIdx.x * (4 / gw) + wave / gw;
    uint4 cur[PT][KS], nxt[PT][KS];
    if (t < tiles) load(t, cur);
    for (; t < tiles; t += walkers) {
        if (t + walkers < tiles) load(t + walkers, nxt);
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][j], as_bf16x8(cur[p][s]), acc[j], 0, 0, 0);
            const long long m = (long long)(t * PT + p) * 16 + pl;
            if (m < a.M && cv) {
                int b;
                const long long o = out_index(a, m, c, b);
                float v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    v[k] = acc[k >> 2][k & 3] + bias[k];
                    if (a.flags & FLAG_RELU) v[k] = v[k] > 0.f ? v[k] : 0.f;
                }
                if (a.out32) {
                    store8(a.out32 + o, v, (a.flags & FLAG_ACC) != 0);
                } else {
                    uint16_t *dst = a.out + o;
                    if (a.flags & FLAG_ACC) {
                        float old[8];
                        unpack8(*(const uint4 *)dst, old);
#pragma unroll
                        for (int k = 0; k < 8; ++k) v[k] += old[k];
                    }
                    if (a.mask) relu_mask(v, *(const uint4 *)(a.mask + m * a.mask_cs + a.mask_co + c));
                    *(uint4 *)dst = pack8(v);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PT; ++p)
#pragma unroll
            for (int s = 0; s < KS; ++s) cur[p][s] = nxt[p][s];
    }
}

// Weight gradient: dW[r][k] = sum_m G[m][r] * im2col(in)[m][k], G = dout
// (S2D: r = sub * Cr + co read at the fine pixel).  blockIdx.z splits the
// pixel range; partials are summed by k_sum_splits.  The contraction runs
// over pixels, which are the slow index of both operands in memory, so each
// stage of WPB pixels is transposed on its way into LDS: a thread loads 4
// consecutive pixels x 8 channels of G and of the im2col rows, swaps them in
// registers and writes one 8-byte run of 4 pixels per channel.  The next
// stage's global loads are issued before the current stage's MFMAs.
constexpr int WPB = 128, WLD = WPB + 8;          // pixels per stage; LDS rows padded by 16 B

// Column (in halfwords) of pixel col of LDS row `row`: the 16-byte granules
// of a row are XOR-swizzled by (row >> 3) & 7.  The staging writes put 4
// pixels of 8 rows that are 8 apart; unswizzled, those rows alias onto two
// bank groups (the 272-byte row stride times 8 is a multiple of 128 banks'
// worth of bytes), swizzled they spread over all banks; the MFMA operand
// reads (16 consecutive rows, one granule) stay conflict-free.
__device__ inline int wcol(int row, int col) { return (((col >> 3) ^ ((row >> 3) & 7)) << 3) | (col & 7); }

// v[j] = 8 channels of pixel j (j = 0..3) -> o[e] = channel e of pixels 0..3.
__device__ inline void transpose_4x8(const uint4 (&v)[4], uint2 (&o)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int d = e >> 1;
        const uint32_t a0 = (&v[0].x)[d], a1 = (&v[1].x)[d], a2 = (&v[2].x)[d], a3 = (&v[3].x)[d];
        // v_perm_b32 picks bytes of {hi, lo}: 0x05040100 = low halves (lo, hi), 0x07060302 = high halves
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        o[e] = make_uint2(__builtin_amdgcn_perm(a1, a0, sel), __builtin_amdgcn_perm(a3, a2, sel));
    }
}

// NARROW (at most 32 rows, the 32-channel layers): a block takes 32 rows x
// 128 columns and its four wavefronts sit side by side along the columns, so
// no MFMA works on the empty rows a 64-row tile would carry; each thread then
// loads two column groups of the im2col rows, and half the threads the rows
// of G.
template <bool NARROW, bool SUMS>
__global__ void __launch_bounds__(256) k_wgrad(ConvArgs a, const uint16_t *__restrict__ g, int g_cs,
                                               int g_co, int rows, float *__restrict__ part, float *__restrict__ bpart,
                                               long long chunk) {
    constexpr int RM = NARROW ? 32 : BM;            // rows per block
    constexpr int CN = NARROW ? 128 : BN;           // columns per block
    constexpr int NT = CN / 64;                     // column groups of 64 per thread
    __shared__ uint16_t Gs[RM][WLD];
    __shared__ uint16_t Ts[CN][WLD];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = NARROW ? 0 : (wave & 1), wn = NARROW ? wave : (wave >> 1);
    const int r0 = blockIdx.x * RM, c0 = blockIdx.y * CN;
    const long long mb = (long long)blockIdx.z * chunk;
    const long long me = mb + chunk < a.M ? mb + chunk : a.M;
    const int pg = t >> 3, cg = (t & 7) * 8;        // pixels 4 pg .. 4 pg + 3 of a stage, channels cg .. cg + 7
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool s2d_g = (a.flags & FLAG_S2D_G) != 0, s2d = (a.flags & FLAG_S2D) != 0;
    // the thread's im2col columns (tap, channel) and G channel are fixed over
    // the pixel loop: tap displacement, 32-bit offset from the pixel's first
    // channel, and the fine-grid sub-pixel of an S2D_G row
    int dx[NT], dy[NT], dz[NT], dl[NT];
    bool kv[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const KOff o = koff_of(a, c0 + 64 * n + cg);
        dx[n] = o.dx; dy[n] = o.dy; dz[n] = o.dz; dl[n] = (int)o.delta; kv[n] = o.valid;
    }
    const int r = r0 + cg;
    const bool g_rows = cg < RM && r < rows;        // this thread stages rows of G
    int gch = r, gsx = 0, gsy = 0, gsz = 0;
    if (s2d_g) {
        const int cr = rows >> a.dims, sub = r / cr;
        gch = r - sub * cr; gsx = sub & 1; gsy = (sub >> 1) & 1; gsz = (sub >> 2) & 1;
    }
    const int fd = a.dims == 3 ? 2 * a.d : 1, fh = 2 * a.h, fw = 2 * a.w;
    // coordinates of the thread's first pixel of the next stage; a stage
    // advances them by WPB pixels through the step's own digits
    Cursor cur = cursor_of((unsigned)(mb + 4 * pg), a);
    const Cursor step = cursor_of((unsigned)WPB, a);
    uint4 gv[4], tv[NT][4];
    auto load = [&](long long mm) {
        const long long m0 = mm + 4 * pg;
        const uint16_t *tp = a.in + a.in_co + m0 * a.in_cs;
        const uint16_t *gp = g + g_co + gch + m0 * g_cs;
        Cursor c = cur;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j) cursor_inc(c, a);
            const bool mv = m0 + j < me;
            gv[j] = make_uint4(0, 0, 0, 0);
            if (g_rows && mv) {
                const uint16_t *src = gp + j * g_cs;
                if (s2d_g) {
                    const int zf = a.dims == 3 ? 2 * c.z + gsz : 0;
                    const int f = ((c.b * fd + zf) * fh + 2 * c.y + gsy) * fw + 2 * c.x + gsx;
                    src = g + g_co + gch + (long long)f * g_cs;
                }
                gv[j] = *(const uint4 *)src;
            }
            const uint16_t *pix = tp + j * a.in_cs;
            if (s2d) {
                const int px = ((c.b * fd + (a.dims == 3 ? 2 * c.z : 0)) * fh + 2 * c.y) * fw + 2 * c.x;
                pix = a.in + a.in_co + (long long)px * a.in_cs;
            }
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                bool ok = mv && kv[n];
                if (!s2d)
                    ok = ok && (unsigned)(c.x + dx[n]) < (unsigned)a.w && (unsigned)(c.y + dy[n]) < (unsigned)a.h &&
                         (unsigned)(c.z + dz[n]) < (unsigned)a.d;
                tv[n][j] = ok ? *(const uint4 *)(pix + dl[n]) : make_uint4(0, 0, 0, 0);
            }
        }
        cursor_add(cur, step, a);
    };
    // SUMS: the row sums of G too (the bias gradient's partials), as products with ones in the first column tile
    const bool sums = SUMS && blockIdx.y == 0 && wn == 0;
    const bf16x8 ones = as_bf16x8(make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
    f32x4 accb[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    load(mb);
    for (long long mm = mb; mm < me; mm += WPB) {
        __syncthreads();                              // the previous stage's MFMA reads are done
        {
            uint2 o[8];
            if (g_rows) {
                transpose_4x8(gv, o);
#pragma unroll
                for (int e = 0; e < 8; ++e) *(uint2 *)&Gs[cg + e][wcol(cg + e, 4 * pg)] = o[e];
            }
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                transpose_4x8(tv[n], o);
#pragma unroll
                for (int e = 0; e < 8; ++e) *(uint2 *)&Ts[64 * n + cg + e][wcol(64 * n + cg + e, 4 * pg)] = o[e];
            }
        }
        __syncthreads();
        if (mm + WPB < me) load(mm + WPB);
#pragma unroll
        for (int kh = 0; kh < WPB; kh += 32) {
            const int kr = kh + (lane >> 4) * 8;
            bf16x8 fb[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int tr = wn * 32 + j * 16 + (lane & 15);
                fb[j] = as_bf16x8(*(const uint4 *)&Ts[tr][wcol(tr, kr)]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int gr = wm * 32 + i * 16 + (lane & 15);
                const bf16x8 fa = as_bf16x8(*(const uint4 *)&Gs[gr][wcol(gr, kr)]);
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[i][j], 0, 0, 0);
                if (sums) accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, ones, accb[i], 0, 0, 0);
            }
        }
    }
    if (sums && (lane & 15) == 0)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int rr = r0 + wm * 32 + i * 16 + (lane >> 4) * 4 + q;
                if (rr < rows) bpart[(long long)blockIdx.z * rows + rr] = accb[i][q];
            }
    float *dst = part + (long long)blockIdx.z * rows * a.K;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = c0 + wn * 32 + j * 16 + (lane & 15);
            if (c >= a.K) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int rr = r0 + wm * 32 + i * 16 + (lane >> 4) * 4 + q;
                if (rr < rows) dst[(long long)rr * a.K + c] = acc[i][j][q];
            }
        }
}

// Weight gradient of a 3 x 3 (x 3) convolution on image rows.  The generic
// kernel above gathers the im2col matrix, i.e. every input pixel 9 times, and
// transposes it in registers.  Here a group of wavefronts walks down a strip
// of 32 columns: the rows of the input (with one column of halo on each side)
// and of G are copied into LDS once, pixel-major as they lie in memory, and
// the MFMA operands, which run over the 32 pixels of a row (the contraction
// index), come out of LDS through the gfx950 transposing read
// ds_read_b64_tr_b16.  The three operands of G's last rows stay in registers,
// so that an input row's operand at column offset dx serves the taps dy = 0,
// 1, 2 at once: 2 + 3 operands are read for 18 MFMAs (11 with one per tap).
//
// Lane layout of that read: in each group of 16 lanes, lane 4e + c names the
// 8-byte block holding columns 4c .. 4c + 3 of row e, and lane i receives
// column i of the rows 0 .. 3.  An MFMA 16x16x32 operand (lane l: tile row
// or column l & 15, K entries 8 (l >> 4) .. + 7) is the pair of reads
// h = 0, 1 in which lane 16 G + 4 e + c names K entry 8 G + 4 h + e, column
// block c.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
__device__ inline v4s lds_tr(const uint16_t *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p);
}
__device__ inline bf16x8 tr_operand(const uint16_t *p0, const uint16_t *p1) {
    const v8s v = __builtin_shufflevector(lds_tr(p0), lds_tr(p1), 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// Block: RB = 32 WR rows x CB = 16 WC input channels x the 9 taps of one plane
// offset; a wavefront takes 32 rows (two m tiles) x 16 channels x 9 taps, and
// WK = 8 / (WR WC) groups of WR x WC wavefronts walk over different strips.  Their
// sums meet in LDS at the end: one block of 8 wavefronts per CU leaves half the
// partials of two blocks of 4.  PW = 16 (planes at most 16 columns wide): the
// 32 columns of a strip are those of two planes.  A strip is cut into segments
// of `len` rows; walker v (block part z, group k: v = z WK + k) takes the
// segments v per .. v per + per - 1.  Step k of a segment that starts at row y0
// meets input row y0 - 1 + k with rows y0 + k, y0 + k - 1 and y0 + k - 2 of G;
// the input reads 0 outside the plane.  Rows of G outside the segment are left
// out (wavefront-uniform branches: zeros in their place would turn a non-finite
// input into NaN, also in taps that it does not reach).  WG_NR steps are
// staged at a time: the next ones are loaded while the current ones multiply,
// and go to the other LDS buffer.
//
// A pixel is a 64-byte row of LDS (32 channels; wider blocks stack such slabs);
// its two 16-channel halves trade places in every second run of 8 pixels, so
// that the 32 lanes that a transposing read serves at a time (4 pixels each of
// two runs, 32 bytes a pixel) cover all 64 banks.  A layer of 8 input channels
// keeps 16-byte rows and computes its 8 channels twice.
//
// SUMS: the bias gradient's partials too (bpart), the row sums of G, as products of
// G's operands with ones in the blocks of the first channel tile.
//
// 16 x 256^2, 32 -> 32: 29 us (4.6 TB/s; sum of the partials 4 us), bound by
// memory; 16 x 64^2, 128 -> 128: 27 us, of which 12 us are the launch, the first
// loads and the partials and the rest the stages (twice their MFMA time); with
// an operand per tap and 128-pixel patches, one launch per plane offset and
// 400 - 630 blocks' partials, these layers took 47 and 40 us with their sums,
// and 2 x 64^3, 64 -> 32, 172 us instead of 71 us.  Six steps a stage: the same.
constexpr int WG_NR = 3;
struct WgradWalk { int len, pieces, per, sps, z; };   // segment rows, segments per strip, segments per walker,
                                                      // stages per segment, block parts

template <int PW, int WR, int WC, bool C8, bool SUMS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
k_wgrad_rows(ConvArgs a, const uint16_t *__restrict__ g, int g_cs, int g_co, int rows, float *__restrict__ part,
             float *__restrict__ bpart, WgradWalk wk) {
    constexpr int NR = WG_NR, SP = 32 / PW, HW = PW + 2, HT = SP * HW;   // strips side by side, LDS row of the input
    constexpr int RB = 32 * WR, CB = C8 ? 8 : 16 * WC, WK = 8 / (WR * WC), TG = 512 / WK;
    constexpr int XS = C8 ? 8 : 32, XCH = CB / 8, GCH = RB / 8;          // LDS pixel (halfwords), 16-byte chunks
    constexpr int XE = NR * HT * XCH, GE = NR * 32 * GCH;                // chunks of a stage
    constexpr int XN = (XE + TG - 1) / TG, GN = (GE + TG - 1) / TG;
    constexpr int XB = NR * HT * CB, GB = NR * 32 * RB + (WR > 1 ? 64 : 0);  // halfwords of a stage
    constexpr int NA = SUMS ? 80 : 72;                                   // a lane's sums
    constexpr int SUM = NA * 64 * 2 * (WK > 2 ? 8 : 4);                  // halfwords of the sums handed over
    constexpr int NL = 2 * WK * (XB + GB) > SUM ? 2 * WK * (XB + GB) : SUM;
    static_assert(NR == 3, "the G rows rotate through 3 operands");
    __shared__ __align__(16) uint16_t S[NL];
    // (readfirstlane: the group's pointers are uniform in a wavefront and belong in scalar registers)
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int kg = wave / (WR * WC), wr = wave % WR, wc = (wave / WR) % WC, u = t % TG;
    // blocks of one XCD take neighbouring parts; the tiles of a part are adjacent
    const int ndz = a.dims == 3 ? 3 : 1, tr = rows / RB, tc = a.cin / CB, tiles = tr * tc * ndz;
    const int nb = (int)gridDim.x, q8 = nb >> 3, r8 = nb & 7, xcd = (int)blockIdx.x & 7;
    const int bt = xcd * q8 + (xcd < r8 ? xcd : r8) + ((int)blockIdx.x >> 3);
    const int zp = bt / tiles, tile = bt - zp * tiles;
    const int r0 = tile % tr * RB, ci0 = tile / tr % tc * CB, dz = a.dims == 3 ? tile / (tr * tc) - 1 : 0;
    const int npx = (a.w + PW - 1) / PW, strips = a.n * a.d * npx;       // (PW = 16: one per plane)
    const int nseg = (strips + SP - 1) / SP * wk.pieces;
    uint16_t *X = S + kg * (XB + GB), *Gs = X + XB;                      // buffer 0; buffer 1 is 2nd half of S
    constexpr int BUF = WK * (XB + GB);
    constexpr int GSL = NR * 32 * 32 + (WR > 1 ? 32 : 0);                // a slab of G; two slabs start 16 banks apart

    // the thread's chunks of a stage: byte offsets from the stage's first input / G pixel (OOB: not in the plane)
    unsigned xo[XN], go[GN];
    const uint16_t *xb = a.in, *gb = g;
    int y = 0, yend = 0;                                                 // next stage's first G row, segment's end
    auto segment = [&](int sg) {
        const int st = sg / wk.pieces * SP, y0 = (sg - sg / wk.pieces * wk.pieces) * wk.len;
        const int img = st / npx, px0 = (st - img * npx) * PW;           // img = sample * d + plane
        y = y0;
        yend = sg < nseg ? min(y0 + wk.len, a.h) : y0;
        const long long pix = ((long long)img * a.h + y0) * a.w + px0;
        gb = g + g_co + r0 + pix * g_cs;
        xb = a.in + a.in_co + ci0 + (pix + ((long long)dz * a.h - 1) * a.w - 1) * a.in_cs;
#pragma unroll
        for (int k = 0; k < XN; ++k) {
            const int e = u + TG * k, cc = e % XCH, p = e / XCH % HT, row = e / (XCH * HT);
            const int half = p / HW, c = p - half * HW;
            const bool ok = e < XE && st + half < strips && (unsigned)((img + half) % a.d + dz) < (unsigned)a.d &&
                            (unsigned)(px0 + c - 1) < (unsigned)a.w;
            xo[k] = ok ? 2u * (unsigned)(((half * a.h + row) * a.w + c) * a.in_cs + 8 * cc) : OOB;
        }
#pragma unroll
        for (int k = 0; k < GN; ++k) {
            const int e = u + TG * k, cc = e % GCH, p = e / GCH % 32, row = e / (GCH * 32);
            const int half = p / PW, c = p - half * PW;
            const bool ok = e < GE && st + half < strips && px0 + c < a.w;
            go[k] = ok ? 2u * (unsigned)(((half * a.h + row) * a.w + c) * g_cs + 8 * cc) : OOB;
        }
    };
    uint4 xv[XN], gv[GN];
    auto load = [&] {
        const __amdgpu_buffer_rsrc_t rx = rsrc_of(xb, 0x80000000u), rg = rsrc_of(gb, 0x80000000u);
#pragma unroll
        for (int k = 0; k < XN; ++k) {
            const int row = (u + TG * k) / (XCH * HT);
            xv[k] = bload16(rx, (unsigned)(y - 1 + row) < (unsigned)a.h && y - 1 + row <= yend ? xo[k] : OOB);
        }
#pragma unroll
        for (int k = 0; k < GN; ++k) gv[k] = bload16(rg, y + (u + TG * k) / (GCH * 32) < yend ? go[k] : OOB);
        y += NR;
        xb += (long long)NR * a.w * a.in_cs;
        gb += (long long)NR * a.w * g_cs;
    };
    // LDS: slab of 32 channels, row, column, channel
    auto stash = [&](int buf) {
#pragma unroll
        for (int k = 0; k < XN; ++k) {
            const int e = u + TG * k, cc = e % XCH, p = e / XCH;
            const int sw = C8 ? 0 : (p % HT % HW >> 2) & 2;
            if (e < XE) *(uint4 *)&X[buf * BUF + ((cc >> 2) * NR * HT + p) * XS + ((cc & 3) ^ sw) * 8] = xv[k];
        }
#pragma unroll
        for (int k = 0; k < GN; ++k) {
            const int e = u + TG * k, cc = e % GCH, p = e / GCH;
            if (e < GE) *(uint4 *)&Gs[buf * BUF + (cc >> 2) * GSL + p * 32 + ((cc & 3) ^ ((p >> 2) & 2)) * 8] = gv[k];
        }
    };
    // the lane's transposing-read addresses (h = 0, 1) in row 0
    const int G = lane >> 4, e4 = (lane >> 2) & 3, c4 = lane & 3;
    const uint16_t *xr[3][2], *gr[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int q = 8 * G + 4 * h + e4;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            const int px = q % PW + dx;
            xr[dx][h] = X + ((wc >> 1) * NR * HT + q / PW * HW + px) * XS +
                        (C8 ? 4 * (c4 & 1) : 16 * ((wc ^ (px >> 3)) & 1) + 4 * c4);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) gr[i][h] = Gs + wr * GSL + q * 32 + 16 * (i ^ (G & 1)) + 4 * c4;
    }
    f32x4 acc[9][2];
#pragma unroll
    for (int j = 0; j < 9; ++j) acc[j][0] = acc[j][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (wave-uniform)
    const bool sums = SUMS && ci0 == 0 && dz == 0 && wc == 0;
    const bf16x8 ones = as_bf16x8(make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
    f32x4 accb[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    bf16x8 fg[3][2], fx[2][3];                         // operands of G's last three rows, of this and the next input row
#pragma unroll
    for (int k = 0; k < 3; ++k) fg[k][0] = fg[k][1] = as_bf16x8(make_uint4(0, 0, 0, 0));
    int sg = (zp * WK + kg) * wk.per, left = wk.sps;   // (segments past the last one hold no rows)
    const int total = wk.per * wk.sps;
    segment(sg);
    int gs = 0, gl = max(yend - y, 0);                 // the stage's first G row in its segment, the segment's rows
    load();
    stash(0);
    for (int st = 0; st < total; ++st) {
        const int o = (st & 1) * BUF, s0 = gs, sl = gl;
        __syncthreads();
        if (st + 1 < total) {
            gs += NR;
            if (--left == 0) {
                left = wk.sps;
                segment(++sg);
                gs = 0;
                gl = max(yend - y, 0);
            }
            load();
        }
        auto read_row = [&](int k) {
#pragma unroll
            for (int i = 0; i < 2; ++i) fg[k % 3][i] = tr_operand(gr[i][0] + o + k * 32 * 32, gr[i][1] + o + k * 32 * 32);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) fx[k & 1][dx] = tr_operand(xr[dx][0] + o + k * HT * XS, xr[dx][1] + o + k * HT * XS);
        };
        read_row(0);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            // dy = 2 uses the oldest G row, whose operand the next row's read replaces
#pragma unroll
            for (int dy = 2; dy >= 0; --dy) {
                if (dy == 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (k + 1 < NR) read_row(k + 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (__builtin_expect((unsigned)(s0 + k - dy) >= (unsigned)sl, 0)) continue;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[dy * 3 + dx][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            fg[(k + 3 - dy) % 3][i], fx[k & 1][dx], acc[dy * 3 + dx][i], 0, 0, 0);
            }
        }
        if (sums)                                      // fg[k]: G's row k of the stage
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i) accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fg[k][i], ones, accb[i], 0, 0, 0);
        if (st + 1 < total) stash((st + 1) & 1);
    }
    // The groups' sums, the upper half of them added to the lower half until one is left.  Two groups: the second
    // hands its sums over, the first adds and stores.  More: all hand theirs over, and group k adds and stores every
    // WK'th operand (a barrier a halving, the last group storing alone: 1 us more; for two groups 0.5 us less).
    f32x4 *sum = (f32x4 *)S + lane;                        // [wavefront][operand][lane]
    constexpr int NO = NA / 4;
    const int wp = wave % (WR * WC);
    __syncthreads();
    if (WK > 2 || kg == 1) {
        f32x4 *w = sum + (WK > 2 ? wave : wp) * NO * 64;
#pragma unroll
        for (int j = 0; j < 18; ++j) w[j * 64] = acc[j >> 1][j & 1];
        if (SUMS) {
            w[18 * 64] = accb[0];
            w[19 * 64] = accb[1];
        }
    }
    __syncthreads();
    // operand j, element q: tap j / 2, row r0 + 32 wr + 16 (j & 1) + 4 (lane >> 4) + q, channel ci0 + 16 wc + (lane & 15);
    // 18 and 19: the rows' sums
    float *dst = part + (long long)zp * rows * a.K + (a.dims == 3 ? 9 * (dz + 1) * a.cin : 0) + ci0 + 16 * wc + (lane & 15);
    auto store = [&](int j, f32x4 v) {
        const int rr = r0 + 32 * wr + 16 * (j & 1) + 4 * (lane >> 4);
        if (SUMS && j >= 18) {
            if ((lane & 15) == 0)
#pragma unroll
                for (int q = 0; q < 4; ++q) bpart[(long long)zp * rows + rr + q] = v[q];
        } else if (!C8 || (lane & 15) < 8) {
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[(long long)(rr + q) * a.K + (j >> 1) * a.cin] = v[q];
        }
    };
    if constexpr (WK == 2) {
        if (kg) return;
#pragma unroll
        for (int j = 0; j < 18; ++j) store(j, acc[j >> 1][j & 1] + sum[(wp * NO + j) * 64]);
        if (sums)
#pragma unroll
            for (int j = 0; j < 2; ++j) store(18 + j, accb[j] + sum[(wp * NO + 18 + j) * 64]);
        return;
    }
    for (int j = kg; j < (sums ? NO : 18); j += WK) {
        f32x4 v[WK];
#pragma unroll
        for (int k = 0; k < WK; ++k) v[k] = sum[((k * WR * WC + wp) * NO + j) * 64];
#pragma unroll
        for (int half = WK / 2; half > 0; half >>= 1)
#pragma unroll
            for (int k = 0; k < half; ++k) v[k] += v[k + half];
        store(j, v[0]);
    }
}

// Sum of split partials: a block takes 64 V outputs (V per lane, one load), its
// NW wavefronts the splits z = w, w + NW, ..., combined in wavefront order
// (deterministic).  Bound by memory: 16 wavefronts keep enough rows in flight
// where outputs are few and splits many.  The blocks from the nb'th on sum the
// splits2 partials of the n2 outputs of part2 (the bias gradient's).
template <int NW, int V>
__global__ void __launch_bounds__(64 * NW) k_sum_splits(const float *__restrict__ part, int splits, long long n,
                                                        float *__restrict__ out, int accumulate, unsigned nb,
                                                        const float *__restrict__ part2, int splits2,
                                                        long long n2, float *__restrict__ out2) {
    typedef float vec __attribute__((ext_vector_type(V)));
    __shared__ vec sh[NW][64];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned b = blockIdx.x;
    if (b >= nb) {
        b -= nb;
        part = part2;
        splits = splits2;
        n = n2;
        out = out2;
    }
    const long long i = ((long long)b * 64 + l) * V;
    vec s = 0.f;
    if (i < n)
#pragma unroll 8
        for (int z = w; z < splits; z += NW) s += *(const vec *)(part + (long long)z * n + i);
    sh[w][l] = s;
    __syncthreads();
    if (w == 0 && i < n) {
        vec v = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) v += sh[k][l];
#pragma unroll
        for (int k = 0; k < V; ++k) out[i + k] = accumulate ? out[i + k] + v[k] : v[k];
    }
}

// Sum of split partials when there are few outputs: one block per output,
// the threads stride over the splits, then a fixed-order tree (deterministic).
__global__ void __launch_bounds__(256) k_sum_splits_narrow(const float *__restrict__ part, int splits, long long n,
                                                           float *__restrict__ out, int accumulate) {
    __shared__ float sh[256];
    const long long i = blockIdx.x;
    float acc = 0.f;
    for (int z = threadIdx.x; z < splits; z += 256) acc += part[(long long)z * n + i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[i] = accumulate ? out[i] + sh[0] : sh[0];
}

// Bias gradient partials with 16-byte loads (channel stride, offset and
// count multiples of 8, C <= 2048): a thread sums 8 channels of every
// (256 / (C/8))-th pixel of the split; LDS combines the pixel lanes.
// Bias gradient partials, 8 channels per thread with 16-byte loads.  RELU:
// first the ReLU backward in the same pass, g = 0 where y <= 0 (written back),
// then the masked g is summed (the same sums, in the same order, as the two
// passes one after the other).
template <bool RELU>
__global__ void __launch_bounds__(256) k_bias_grad8(uint16_t *__restrict__ g, const uint16_t *__restrict__ y,
                                                    int cs, int co, long long npix, int C, long long chunk,
                                                    float *__restrict__ part) {
    __shared__ float sh[256 * 8];
    const int tpp = C >> 3;                    // threads per pixel
    const int ppi = 256 / tpp;                 // pixels per iteration
    const int gi = threadIdx.x % tpp, pi = threadIdx.x / tpp;
    const long long mb = (long long)blockIdx.x * chunk;
    const long long me = mb + chunk < npix ? mb + chunk : npix;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (pi < ppi)
#pragma unroll 4
        for (long long m = mb + pi; m < me; m += ppi) {
            uint4 v = *(const uint4 *)(g + m * cs + co + gi * 8);
            if (RELU) {
                const uint4 yv = *(const uint4 *)(y + m * cs + co + gi * 8);
                const uint32_t y4[4] = {yv.x, yv.y, yv.z, yv.w};
                uint32_t g4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (!(bf2f((uint16_t)(y4[j] & 0xffffu)) > 0.f)) g4[j] &= 0xffff0000u;
                    if (!(bf2f((uint16_t)(y4[j] >> 16)) > 0.f)) g4[j] &= 0x0000ffffu;
                }
                v = make_uint4(g4[0], g4[1], g4[2], g4[3]);
                *(uint4 *)(g + m * cs + co + gi * 8) = v;
            }
            const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[2 * j] += bf2f((uint16_t)(w4[j] & 0xffffu));
                acc[2 * j + 1] += bf2f((uint16_t)(w4[j] >> 16));
            }
        }
#pragma unroll
    for (int j = 0; j < 8; ++j) sh[threadIdx.x * 8 + j] = pi < ppi ? acc[j] : 0.f;
    __syncthreads();
    for (int c = threadIdx.x; c < C; c += 256) {
        const int gc = c >> 3, j = c & 7;
        float sum = 0.f;
        for (int p = 0; p < ppi; ++p) sum += sh[(p * tpp + gc) * 8 + j];
        part[(long long)blockIdx.x * C + c] = sum;
    }
}

// Bias gradient partials: part[split][c] = sum over the split's pixels.
__global__ void __launch_bounds__(256) k_bias_grad(const uint16_t *__restrict__ g, int cs, int co, long long npix,
                                                   int C, long long chunk, float *__restrict__ part) {
    __shared__ float s[4][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), pl = threadIdx.x >> 6;
    const long long mb = (long long)blockIdx.y * chunk;
    const long long me = mb + chunk < npix ? mb + chunk : npix;
    float acc = 0.f;
    if (c < C)
        for (long long m = mb + pl; m < me; m += 4) acc += bf2f(g[m * cs + co + c]);
    s[pl][threadIdx.x & 63] = acc;
    __syncthreads();
    if (pl == 0 && c < C) part[(long long)blockIdx.y * C + c] = s[0][threadIdx.x] + s[1][threadIdx.x] + s[2][threadIdx.x] + s[3][threadIdx.x];
}

__global__ void k_relu_bwd(uint16_t *__restrict__ g, const uint16_t *__restrict__ y, int cs, int co,
                           long long npix, int C) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npix * C) return;
    const long long m = i / C;
    const int c = (int)(i - m * C);
    const long long o = m * cs + co + c;
    if (!(bf2f(y[o]) > 0.f)) g[o] = 0;
}

// 2x2(x2) max pooling, stride 2; (d, h, w) is the coarse grid.
__global__ void k_pool_fwd(const uint16_t *__restrict__ in, int in_cs, int in_co, uint16_t *__restrict__ out,
                           int out_cs, int out_co, int n, int d, int h, int w, int C, int dims) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)n * d * h * w * C;
    if (i >= total) return;
    const long long m = i / C;
    const int c = (int)(i - m * C);
    const Pix p = pix_of(m, d, h, w);
    const int fd = dims == 3 ? 2 * d : 1;
    float best = -INFINITY;
    for (int sub = 0; sub < (1 << dims); ++sub) {
        const int sx = sub & 1, sy = (sub >> 1) & 1, sz = (sub >> 2) & 1;
        const int zf = dims == 3 ? 2 * p.z + sz : 0;
        const long long f = (((long long)p.b * fd + zf) * (2 * h) + 2 * p.y + sy) * (2 * w) + 2 * p.x + sx;
        best = fmaxf(best, bf2f(in[f * in_cs + in_co + c]));
    }
    out[m * out_cs + out_co + c] = f2bf(best);
}

// Routes dout to the first maximal element of each window (sub order).
__global__ void k_pool_bwd(const uint16_t *__restrict__ in, int in_cs, int in_co,
                           const uint16_t *__restrict__ gout, int g_cs, int g_co, uint16_t *__restrict__ gin,
                           int gi_cs, int gi_co, int n, int d, int h, int w, int C, int dims, int accumulate,
                           int relu) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)n * d * h * w * C;
    if (i >= total) return;
    const long long m = i / C;
    const int c = (int)(i - m * C);
    const Pix p = pix_of(m, d, h, w);
    const int fd = dims == 3 ? 2 * d : 1;
    float best = -INFINITY;
    int arg = 0;
    long long fidx[8];
    for (int sub = 0; sub < (1 << dims); ++sub) {
        const int sx = sub & 1, sy = (sub >> 1) & 1, sz = (sub >> 2) & 1;
        const int zf = dims == 3 ? 2 * p.z + sz : 0;
        fidx[sub] = (((long long)p.b * fd + zf) * (2 * h) + 2 * p.y + sy) * (2 * w) + 2 * p.x + sx;
        const float v = bf2f(in[fidx[sub] * in_cs + in_co + c]);
        if (v > best) { best = v; arg = sub; }
    }
    const float gv = bf2f(gout[m * g_cs + g_co + c]);
    for (int sub = 0; sub < (1 << dims); ++sub) {
        const long long o = fidx[sub] * gi_cs + gi_co + c;
        const float add = sub == arg ? gv : 0.f;
        if (relu && !(bf2f(in[fidx[sub] * in_cs + in_co + c]) > 0.f)) gin[o] = 0;
        else if (accumulate) { if (sub == arg) gin[o] = f2bf(bf2f(gin[o]) + add); }
        else gin[o] = f2bf(add);
    }
}

// The same two passes on 8 channels of a pixel per thread with 16-byte
// accesses (channel counts, strides and offsets multiples of 8, 16-byte
// aligned buffers); per channel the same operations in the same order.
__global__ void __launch_bounds__(256) k_pool_fwd8(const uint16_t *__restrict__ in, int in_cs, int in_co,
                                                   uint16_t *__restrict__ out, int out_cs, int out_co, int n, int d,
                                                   int h, int w, int C, int dims) {
    const int CG = C >> 3;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)n * d * h * w * CG) return;
    const long long m = i / CG;
    const int c = (int)(i - m * CG) * 8;
    const Pix p = pix_of(m, d, h, w);
    const int fd = dims == 3 ? 2 * d : 1;
    float best[8], v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) best[k] = -INFINITY;
    for (int sub = 0; sub < (1 << dims); ++sub) {
        const int sx = sub & 1, sy = (sub >> 1) & 1, sz = (sub >> 2) & 1;
        const int zf = dims == 3 ? 2 * p.z + sz : 0;
        const long long f = (((long long)p.b * fd + zf) * (2 * h) + 2 * p.y + sy) * (2 * w) + 2 * p.x + sx;
        unpack8(*(const uint4 *)(in + f * in_cs + in_co + c), v);
#pragma unroll
        for (int k = 0; k < 8; ++k) best[k] = fmaxf(best[k], v[k]);
    }
    *(uint4 *)(out + m * out_cs + out_co + c) = pack8(best);
}

// RELU: `in` holds ReLU outputs, and the sum is 0 where they are not > 0.
template <int DIMS, bool RELU>
__global__ void __launch_bounds__(256) k_pool_bwd8(const uint16_t *__restrict__ in, int in_cs, int in_co,
                                                   const uint16_t *__restrict__ gout, int g_cs, int g_co,
                                                   uint16_t *__restrict__ gin, int gi_cs, int gi_co, int n, int d,
                                                   int h, int w, int C, int accumulate) {
    constexpr int NS = 1 << DIMS;
    const int CG = C >> 3;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)n * d * h * w * CG) return;
    const long long m = i / CG;
    const int c = (int)(i - m * CG) * 8;
    const Pix p = pix_of(m, d, h, w);
    const int fd = DIMS == 3 ? 2 * d : 1;
    float best[8], v[8], gv[8];
    int arg[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) { best[k] = -INFINITY; arg[k] = 0; }
    long long fidx[NS];
    uint4 win[NS], old[NS];
#pragma unroll
    for (int sub = 0; sub < NS; ++sub) {
        const int sx = sub & 1, sy = (sub >> 1) & 1, sz = (sub >> 2) & 1;
        const int zf = DIMS == 3 ? 2 * p.z + sz : 0;
        fidx[sub] = (((long long)p.b * fd + zf) * (2 * h) + 2 * p.y + sy) * (2 * w) + 2 * p.x + sx;
        win[sub] = *(const uint4 *)(in + fidx[sub] * in_cs + in_co + c);
        if (accumulate) old[sub] = *(const uint4 *)(gin + fidx[sub] * gi_cs + gi_co + c);
    }
#pragma unroll
    for (int sub = 0; sub < NS; ++sub) {
        unpack8(win[sub], v);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (v[k] > best[k]) { best[k] = v[k]; arg[k] = sub; }
    }
    unpack8(*(const uint4 *)(gout + m * g_cs + g_co + c), gv);
#pragma unroll
    for (int sub = 0; sub < NS; ++sub) {
        float r[8];
        if (accumulate) {
            unpack8(old[sub], r);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (sub == arg[k]) r[k] = r[k] + gv[k];
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) r[k] = sub == arg[k] ? gv[k] : 0.f;
        }
        if (RELU) relu_mask(r, win[sub]);
        *(uint4 *)(gin + fidx[sub] * gi_cs + gi_co + c) = pack8(r);
    }
}

// Masked MSE over the first `creal` channels of an FP32 prediction with
// channel stride pcs: loss = scale * sum_m w_m sum_c (p - t)^2 and the BF16
// gradient (pad channels zero).  Per-block partial sums in FP64.
__global__ void __launch_bounds__(256) k_mse(const float *__restrict__ pred, int pcs, const float *__restrict__ tgt,
                                             const float *__restrict__ wpix, int creal, long long npix,
                                             float scale, uint16_t *__restrict__ dpred, double *__restrict__ part) {
    __shared__ double s[256];
    const long long m = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double l = 0.0;
    if (m < npix) {
        const float wm = wpix ? wpix[m] : 1.f;
        for (int c = 0; c < pcs; ++c) {
            float gval = 0.f;
            if (c < creal) {
                const float d = pred[m * pcs + c] - tgt[m * creal + c];
                l += (double)(wm * d * d);
                gval = 2.f * scale * wm * d;
            }
            dpred[m * pcs + c] = f2bf(gval);
        }
    }
    s[threadIdx.x] = l * scale;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

__global__ void k_sum_f64(const double *__restrict__ part, long long n, double *__restrict__ out) {
    __shared__ double s[256];
    double a = 0.0;
    for (long long i = threadIdx.x; i < n; i += 256) a += part[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

// Adam on FP32 master weights with an optional BF16 mirror.
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m1,
                       float *__restrict__ m2, uint16_t *__restrict__ wb, long long n, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    const float v = w[i] - lr * (a * c1) / (sqrtf(b * c2) + eps);
    w[i] = v;
    if (wb) wb[i] = f2bf(v);
}

__global__ void k_to_bf16(const float *__restrict__ x, uint16_t *__restrict__ y, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

// Network input: 8 channels per pixel: solid, x / (nx - 1), 200 drho_in,
// 200 drho_out, 2 (tau - 0.9), 0, 0, 0.  prm: [n][3] = (drho_in, drho_out, tau).
__global__ void k_features(const uint8_t *__restrict__ solid, const float *__restrict__ prm, int n, int d,
                           int h, int w, uint16_t *__restrict__ out) {
    const long long m = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= (long long)n * d * h * w) return;
    const Pix p = pix_of(m, d, h, w);
    const float *q = prm + 3 * p.b;
    float f[8] = {(float)solid[m], w > 1 ? (float)p.x / (float)(w - 1) : 0.f, 200.f * q[0], 200.f * q[1],
                  2.f * (q[2] - 0.9f), 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; ++c) out[m * 8 + c] = f2bf(f[c]);
}

// Stokes-scaled targets from LBM fields (and back):
//   t0 = (drho - drho_out) / (drho_in - drho_out),
//   t_{1+a} = u_a nu / (cs^2 (drho_in - drho_out)),  nu = (tau - 1/2) / 3.
__global__ void k_normalize(const float *__restrict__ drho, const float *__restrict__ u, const uint8_t *__restrict__ solid,
                            const float *__restrict__ prm, long long per_sample, int D, long long npix,
                            float *__restrict__ tgt, float *__restrict__ wpix) {
    const long long m = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= npix) return;
    const float *q = prm + 3 * (m / per_sample);
    const float dr = q[0] - q[1], nu = (q[2] - 0.5f) / 3.f;
    const float su = nu / (dr / 3.f);
    const bool fl = solid[m] == 0;
    tgt[m * (1 + D)] = fl ? (drho[m] - q[1]) / dr : 0.f;
    for (int a = 0; a < D; ++a) tgt[m * (1 + D) + 1 + a] = fl ? u[m * D + a] * su : 0.f;
    if (wpix) wpix[m] = fl ? 1.f : 0.f;
}

__global__ void k_denormalize(const float *__restrict__ pred, int pcs, const uint8_t *__restrict__ solid,
                              const float *__restrict__ prm, long long per_sample, int D, long long npix,
                              float *__restrict__ drho, float *__restrict__ u) {
    const long long m = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= npix) return;
    const float *q = prm + 3 * (m / per_sample);
    const float dr = q[0] - q[1], nu = (q[2] - 0.5f) / 3.f;
    const float su = (dr / 3.f) / nu;
    const bool fl = solid[m] == 0;
    drho[m] = fl ? q[1] + dr * pred[m * pcs] : 0.f;
    for (int a = 0; a < D; ++a) u[m * D + a] = fl ? pred[m * pcs + 1 + a] * su : 0.f;
}

// Cross-section flux balance in three launches, FP64 sums in a fixed order:
// block (p, b) sums u_x over the fluid nodes of each section x within row
// chunk p of sample b (thread t of a pass over `cols` sections takes the
// rows t / cols, t / cols + groups, ... of section t % cols; the groups are
// then added in order) into part[b][p][x]; one block per sample adds the
// chunks in order to Q(x), averages Q over the sections to Qbar and writes
// the scale factors S[b][x] = clamp(Qbar / max(Q(x), Qbar / 10), 1/4, 4)
// (all 1 when Qbar <= 0); the last launch scales every value.
constexpr int FB_MAX_W = 2048, FB_MAX_CHUNKS = 64, FB_MIN_ROWS = 16;

__host__ __device__ inline int fb_chunks(long long rows) {
    const long long c = (rows + FB_MIN_ROWS - 1) / FB_MIN_ROWS;
    return (int)(c < FB_MAX_CHUNKS ? c : FB_MAX_CHUNKS);
}

__global__ void __launch_bounds__(256) k_fb_partial(const uint8_t *__restrict__ solid, const float *__restrict__ u,
                                                    int rows, int w, int D, double *__restrict__ part) {
    __shared__ double red[256];
    const int t = threadIdx.x, p = blockIdx.x, b = blockIdx.y, P = gridDim.x;
    const long long per = (long long)rows * w;
    const int r0 = (int)((long long)rows * p / P), r1 = (int)((long long)rows * (p + 1) / P);
    for (int x0 = 0; x0 < w; x0 += 256) {
        const int cols = w - x0 < 256 ? w - x0 : 256, groups = 256 / cols;
        const int x = x0 + t % cols, g = t / cols;
        double acc = 0.0;
        if (g < groups)
            for (int r = r0 + g; r < r1; r += groups) {
                const long long m = b * per + (long long)r * w + x;
                const float v = u[m * D];
                acc += solid[m] ? 0.0 : (double)v;
            }
        red[t] = acc;
        __syncthreads();
        if (t < cols) {
            double q = 0.0;
            for (int k = 0; k < groups; ++k) q += red[k * cols + t];
            part[((long long)b * P + p) * w + x0 + t] = q;
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) k_fb_factors(const double *__restrict__ part, int P, int w,
                                                    float *__restrict__ S) {
    __shared__ double Q[FB_MAX_W];
    __shared__ double qbar;
    const int t = threadIdx.x, b = blockIdx.x;
    for (int x = t; x < w; x += 256) {
        double q = 0.0;
        for (int p = 0; p < P; ++p) q += part[((long long)b * P + p) * w + x];
        Q[x] = q;
    }
    __syncthreads();
    if (t == 0) {
        double q = 0.0;
        for (int x = 0; x < w; ++x) q += Q[x];
        qbar = q / w;
    }
    __syncthreads();
    const double qb = qbar;
    for (int x = t; x < w; x += 256) {
        double sc = 1.0;
        if (qb > 0.0) {
            sc = qb / (Q[x] > 0.1 * qb ? Q[x] : 0.1 * qb);
            sc = sc < 0.25 ? 0.25 : (sc > 4.0 ? 4.0 : sc);
        }
        S[(long long)b * w + x] = (float)sc;
    }
}

__global__ void __launch_bounds__(256) k_fb_apply(float *__restrict__ u, const float *__restrict__ S, long long n,
                                                  long long per, int w, int D) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const long long node = i / D;                      // node of the whole batch, per nodes per sample
    const long long b = node / per;
    const int x = (int)(node % w);
    u[i] *= S[b * w + x];
}

// ------------------------------------------------------------ launchers --
static inline unsigned blocks(long long n, int b) { return (unsigned)((n + b - 1) / b); }

static bool halo_ok(const ConvArgs &a) {
    const uintptr_t ob = a.out32 ? (uintptr_t)a.out32 : (uintptr_t)a.out;
    return (a.dims == 2 || a.dims == 3) && a.ks == 3 && !(a.flags & (FLAG_S2D | FLAG_D2S)) && a.cin % 8 == 0 &&
           a.h % HY == 0 &&
           a.w % HX == 0 && ((a.in_cs | a.in_co | a.out_cs | a.out_co) & 7) == 0 && ((uintptr_t)a.in & 15) == 0 &&
           ((ob | (uintptr_t)a.mask) & 15) == 0 && ((a.mask_cs | a.mask_co) & 7) == 0 &&
           18LL * a.w * a.in_cs < (1LL << 31) && (long long)a.ncols * a.K < (1LL << 31) && a.M < (1LL << 31);
}

// Sum of the K splits of a convolution, in split order, then the epilogue
// of k_conv (bias, ReLU, accumulate, FP32 or BF16 output, D2S scatter): one
// thread per output element.
__global__ void __launch_bounds__(256) k_conv_reduce(ConvArgs a, const float *__restrict__ part, int S) {
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= a.M * a.ncols) return;
    const long long m = e / a.ncols;
    const int c = (int)(e - m * a.ncols);
    float v = 0.f;
    for (int z = 0; z < S; ++z) v += part[(long long)z * a.M * a.ncols + e];
    int bc;
    const long long o = out_index(a, m, c, bc);
    v += a.bias ? a.bias[bc] : 0.f;
    if (a.flags & FLAG_RELU) v = v > 0.f ? v : 0.f;
    if (a.out32) {
        a.out32[o] = (a.flags & FLAG_ACC) ? a.out32[o] + v : v;
    } else {
        if (a.flags & FLAG_ACC) v += bf2f(a.out[o]);
        if (a.mask && !(bf2f(a.mask[m * a.mask_cs + a.mask_co + c]) > 0.f)) v = 0.f;
        a.out[o] = f2bf(v);
    }
}

// K splits for a convolution whose output tiles are too few to fill the
// GPU (the deep, low-resolution layers, whose long K loop would run on a
// few CUs): enough splits for about 1024 blocks, each at least 4 K steps of
// 64; 1 when the layer has 512 tiles or more, or takes the row kernel.
static long long conv_tiles(const ConvArgs &a) {
    return (long long)blocks(a.M, 64) * (a.ncols <= 32 ? 1 : (a.ncols + 63) / 64);
}
static bool conv_halo(const ConvArgs &a) {
    const long long tiles = halo_ok(a) ? (long long)a.n * a.d * (a.h / HY) * (a.w / HX) : 0;
    return tiles * (a.ncols <= 32 ? 1 : (a.ncols + 63) / 64) >= 512;
}
int conv_splits(const ConvArgs &a) {
    const long long tiles = conv_tiles(a);
    if (conv_halo(a) || tiles >= 512) return 1;
    const int steps = (a.K + 63) / 64;
    long long sp = (1024 + tiles - 1) / tiles;
    sp = sp < steps / 4 ? sp : steps / 4;
    if (sp < 2) return 1;
    const int sper = (int)((steps + sp - 1) / sp);
    return (steps + sper - 1) / sper;
}

// A 1 x 1 convolution over its own input (the output's channels among the
// input's): k_conv reads all channels of its pixels before it writes them (up
// to 64 columns, or split), the kernels whose wavefronts share pixels do not.
static bool in_place(const ConvArgs &a) {
    const long long d = ((intptr_t)a.out - (intptr_t)a.in) / 2 + a.out_co - a.in_co;
    return a.ks == 1 && !a.out32 && a.in_cs == a.out_cs && d > -(long long)a.ncols && d < a.cin;
}

// The direct kernel's conditions; its splits are the wavefronts of a block.
// It reads every operand from the caches for each 32 x 32 tile, so it pays while
// launches and latency dominate (us, direct against partials and k_conv_reduce):
// with splits up to 1.3e9 multiply-adds (128^2, 64 -> 64 and 32^2, 256 -> 256 11
// : 16, 128^2, 128 -> 64 19 : 22, 64^2, 256 -> 128 19 : 21, 16^3, 128 -> 128 26 :
// 23, four images of 32^2, 256 -> 256 35 : 24), up to 0.5e9 for 32 channels or
// fewer (6000 pixels, 256 -> 32 11 : 15, 8400 19 : 15); without splits up to
// 0.67e9 and 10 steps, which one wavefront walks alone (256^2, 32 -> 32 8.5 :
// 9.7; 36000 pixels, 64 -> 8 15 : 11; 1 x 1 32^2, 256 -> 512 7.3 : 6.9).
// From nine splits on, a CU holds one block, and pixels and weight rows that lie
// a multiple of 256 bytes apart load slowly: with those, one round of blocks,
// and not a few blocks of eleven splits or more (4 x 6 x 6 x 32, 128 -> 64, 288
// blocks 25 : 20; 5 x 14 x 37, 256 -> 128, 324 blocks 20 : 18; 8^3, 128 -> 64,
// 32 blocks 14.5 : 12.7; 12^3, 128 -> 64, 108 blocks 15 : 13.8, 128 -> 128, 216
// blocks 15.2 : 17.8; 16^2, 256 -> 32, 8 blocks of nine 11.0 : 10.3).
static bool direct_ok(const ConvArgs &a, int S, unsigned *in_bytes) {
    const long long tiles = (a.M + 31) / 32 * ((a.ncols + 31) / 32);
    if (in_place(a)) return false;
    if (S >= 9 && a.cin % 128 == 0 && (tiles > 256 || tiles < (S >= 11 ? 128 : 16))) return false;
    const uintptr_t ob = a.out32 ? (uintptr_t)a.out32 : (uintptr_t)a.out;
    const long long bytes = 2 * a.M * a.in_cs;
    *in_bytes = (unsigned)bytes;
    const long long most = S == 1 ? (a.K <= 320 ? 5LL << 27 : 0) : a.ncols <= 32 ? 1LL << 29 : 5LL << 28;
    return S <= 16 && a.M * ((a.ncols + 31) / 32 * 32) <= most / a.K && a.cin % 32 == 0 && !(a.flags & FLAG_S2D) &&
           bytes < (1LL << 31) && 2LL * a.ncols * a.K < (1LL << 31) && ((a.out_cs | a.out_co) & 7) == 0 &&
           (ob & 15) == 0;
}
static hipError_t conv_direct(const ConvArgs &a, int S, int sper, unsigned in_bytes, hipStream_t s) {
    const long long tiles = (long long)blocks(a.M, 32) * ((a.ncols + 31) / 32);
    hipLaunchKernelGGL(k_conv_direct, dim3((unsigned)(S == 1 ? (tiles + 3) / 4 : tiles)), dim3(64 * (S == 1 ? 4 : S)),
                       S == 1 ? 0 : 4096 * S, s, a, S, sper, in_bytes);
    return hipGetLastError();
}

hipError_t conv_split(const ConvArgs &a, float *part, int S, hipStream_t s) {
    const int steps = (a.K + 63) / 64, sper = (steps + S - 1) / S;
    unsigned in_bytes;
    if (direct_ok(a, S, &in_bytes)) return conv_direct(a, S, sper, in_bytes, s);
    const int tbn = a.ncols <= 32 ? 32 : 64;
    const dim3 grid(blocks(a.M, 64), (unsigned)((a.ncols + tbn - 1) / tbn), (unsigned)S);
    const bool taps = a.cin % 128 == 0;
#define CALL(TBN, TAPS) hipLaunchKernelGGL((k_conv<64, TBN, TAPS, true>), grid, dim3(256), 0, s, a, part, sper)
    if (tbn == 32 && taps) CALL(32, true);
    else if (tbn == 32) CALL(32, false);
    else if (taps) CALL(64, true);
    else CALL(64, false);
#undef CALL
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_conv_reduce, dim3(blocks(a.M * a.ncols, 256)), dim3(256), 0, s, a, part, S);
    return hipGetLastError();
}

hipError_t conv(const ConvArgs &a, hipStream_t s) {
    // the row kernel holds 2 blocks per CU: below 512 tiles of 8 x 32 pixels the im2col kernel fills the chip better
    if (conv_halo(a)) {
        const int tn = a.ncols <= 32 ? 32 : 64, tiles_n = (a.ncols + tn - 1) / tn;
        const long long tiles = (long long)a.n * a.d * (a.h / HY) * (a.w / HX);
        const bool res = a.dims == 2 && a.cin <= HC;
        const int mode = a.out32 || (a.flags & FLAG_ACC) ? OUT_ANY : a.mask ? OUT_MASK : OUT_PLAIN;
        // two blocks per CU, each walking over as many tiles as that leaves it
        const int runs = (512 + tiles_n - 1) / tiles_n, per = (int)((tiles + runs - 1) / runs);
        const dim3 grid((unsigned)((tiles + per - 1) / per * tiles_n));
#define LAUNCH(TN, DIMS, RES, MODE) \
    hipLaunchKernelGGL((k_conv3x3_rows<TN, DIMS, RES, MODE>), grid, dim3(256), 0, s, a, per)
#define CALL(TN, DIMS, RES)                                        \
    do {                                                           \
        if (mode == OUT_PLAIN) LAUNCH(TN, DIMS, RES, OUT_PLAIN);   \
        else if (mode == OUT_MASK) LAUNCH(TN, DIMS, RES, OUT_MASK); \
        else LAUNCH(TN, DIMS, RES, OUT_ANY);                       \
    } while (0)
        if (a.dims == 3) {
            if (tn == 32) CALL(32, 3, false);
            else CALL(64, 3, false);
        } else if (tn == 32) {
            if (res) CALL(32, 2, true);
            else CALL(32, 2, false);
        } else {
            if (res) CALL(64, 2, true);
            else CALL(64, 2, false);
        }
#undef CALL
#undef LAUNCH
        return hipGetLastError();
    }
    const uintptr_t ob = a.out32 ? (uintptr_t)a.out32 : (uintptr_t)a.out;
    // From 256 input channels on (K steps of a wavefront's weights: 64 registers) too few pixel groups are in
    // flight: 16 x 32^2, 256 -> 4 x 128 33 us against 20 us in k_conv; S2D at K = 128 gains nothing (33 us both).
    if (a.ks == 1 && a.K <= 128 && !(a.flags & FLAG_S2D) && !in_place(a) && ((a.out_cs | a.out_co) & 7) == 0 && (ob & 15) == 0) {
        const int steps = (a.K + 31) / 32, groups = (a.ncols + 31) / 32, gw = groups >= 3 ? 4 : groups;
        const int gy = (groups + gw - 1) / gw, pt = steps <= 1 ? 4 : 2;
        const long long want = (a.M + 16 * pt * (4 / gw) - 1) / (16 * pt * (4 / gw));
        // as many blocks as are resident together (5, 4 or 3 per CU), in multiples of 8 along x, so that the blocks
        // of a pixel group fall on one XCD (twice as many: 30 instead of 28 us at 64 -> 4 x 32)
        long long gx = (256 * (steps <= 1 ? 5 : steps <= 2 ? 4 : 3) / gy + 7) / 8 * 8;
        // four K steps in one to four rounds of pixel groups per wavefront: k_conv (four images of 64^2, 128 -> 4 x 64
        // 9.6 us, here 10.7; one image 5.8 and 4.6, sixteen 29 and 25)
        if (steps <= 2 || want <= gx || want >= 4 * gx) {
            if (gx > want) gx = want;
            const dim3 grid((unsigned)gx, (unsigned)gy);
#define CALL(KS, PT) hipLaunchKernelGGL((k_conv1x1<KS, PT>), grid, dim3(256), 0, s, a, gw)
            if (steps <= 1) CALL(1, 4);
            else if (steps <= 2) CALL(2, 2);
            else CALL(4, 2);
#undef CALL
            return hipGetLastError();
        }
    }
    unsigned in_bytes;
    if (a.ks == 3 && direct_ok(a, 1, &in_bytes))
        return conv_direct(a, 1, (a.K + 63) / 64, in_bytes, s);
    const int tbn = a.ncols <= 32 ? 32 : 64;
    const dim3 grid(blocks(a.M, 64), (unsigned)((a.ncols + tbn - 1) / tbn));
    const bool taps = a.cin % 128 == 0;
#define CALL(TBN, TAPS) hipLaunchKernelGGL((k_conv<64, TBN, TAPS>), grid, dim3(256), 0, s, a)
    if (tbn == 32 && taps) CALL(32, true);
    else if (tbn == 32) CALL(32, false);
    else if (taps) CALL(64, true);
    else CALL(64, false);
#undef CALL
    return hipGetLastError();
}

long long wgrad_chunk(long long M, int splits) {
    long long c = (M + splits - 1) / splits;
    return (c + WPB - 1) / WPB * WPB;
}

// Sum of z split partials into n outputs (and of z2 of part2 into n2): a block
// per output when there are few (a weight gradient of at most 1024 entries, a
// bias gradient of many splits, whose chain of loads would outlast the rest),
// else 64 or 256 outputs per block.
static hipError_t sum_splits(const float *part, int z, long long n, float *out, int accumulate, hipStream_t s,
                             const float *part2 = nullptr, int z2 = 0, long long n2 = 0, float *out2 = nullptr) {
    const bool narrow = n <= 1024 && z > 16, narrow2 = part2 && (narrow || z2 > 512);
    if (narrow2)
        hipLaunchKernelGGL(k_sum_splits_narrow, dim3((unsigned)n2), dim3(256), 0, s, part2, z2, n2, out2, accumulate);
    if (narrow) {
        hipLaunchKernelGGL(k_sum_splits_narrow, dim3((unsigned)n), dim3(256), 0, s, part, z, n, out, accumulate);
        return hipGetLastError();
    }
    if (narrow2) n2 = 0;
#define CALL(NW, V)                                                                                              \
    hipLaunchKernelGGL((k_sum_splits<NW, V>), dim3(blocks(n, 64 * V) + blocks(n2, 64 * V)), dim3(64 * NW), 0, s, \
                       part, z, n, out, accumulate, blocks(n, 64 * V), part2, z2, n2, out2)
    if (n >= 65536 && ((n | n2) & 3) == 0 && (((uintptr_t)part | (uintptr_t)part2) & 15) == 0) CALL(4, 4);
    else if (z > 32) CALL(16, 1);
    else CALL(4, 1);
#undef CALL
    return hipGetLastError();
}

// The row kernel's block shape (10 WR + WC) for a layer, or 0: 64 rows x 32
// channels, 32 rows x 64 or 32 channels (two groups), or 32 rows x 8 channels
// (four groups).  Its loads take 32-bit byte offsets from a stage's first pixel.
static int rows_shape(const ConvArgs &a, int rows, int g_cs) {
    if (a.ks != 3 || (a.flags & (FLAG_S2D | FLAG_D2S | FLAG_S2D_G)) || a.w < 16) return 0;
    const long long reach = ((a.w <= 16 ? a.h : 0) + WG_NR + 1LL) * a.w + 34;
    if (2 * reach * (a.in_cs > g_cs ? a.in_cs : g_cs) >= (1LL << 31)) return 0;
    // small layers are launch, first loads and sums, and the im2col kernel's four wavefronts have less of those
    // (us with the sum of the partials, im2col : here; 64 -> 64: 16^2 8.4 : 12, 64^2 11.5 : 12.5, 2 x 64 x 96 13.5 :
    // 14.2; 16 x 17 x 23, 128 -> 128 16.2 : 18.2; beyond it falls behind: 5 x 32 x 96, 128 -> 128 25.7 : 19.4)
    if (rows % 64 == 0 && a.cin % 32 == 0) return (double)a.M * rows * a.K <= 0.7e9 ? 0 : 22;
    if (rows % 32 == 0 && a.cin % 64 == 0) return 14;
    if (rows % 32 == 0 && a.cin % 32 == 0) return 12;
    if (rows % 32 == 0 && a.cin == 8) return 11;
    return 0;
}

template <int PW, bool SUMS>
static hipError_t launch_wgrad_rows(int shape, const ConvArgs &a, const uint16_t *g, int g_cs, int g_co, int rows,
                                    float *part, int &z, float *dw1, float *db1, hipStream_t s) {
    const int RB = shape == 22 ? 64 : 32, CB = shape == 11 ? 8 : shape == 14 ? 64 : 32;
    const int WK = shape == 11 ? 8 : shape == 12 ? 4 : 2;
    const long long tiles = (long long)(rows / RB) * (a.cin / CB) * (a.dims == 3 ? 3 : 1);
    const long long npx = (a.w + PW - 1) / PW, strips = ((long long)a.n * a.d * npx + 32 / PW - 1) / (32 / PW);
    // one block per CU at most, within the partials that the workspace holds; of the cuts of the strips into
    // segments (a segment costs two steps more than it has rows) and the numbers of walkers the one with the least
    // time: 1.2 us a stage of the longest walk, 1.8 us for a million floats of partials written and summed (128^2,
    // 128 -> 128 with 32 parts 21.5 us, with 16 19.7; 16 x 32 x 96, 64 -> 64 with 96 22, with 48 19)
    const long long zt = tiles >= 256 ? 1 : 256 / tiles, zmax = zt < z ? zt : z, n = (long long)rows * a.K;
    WgradWalk k{};
    double best = 0;
    for (int f = 4; f >= 1; --f) {
        const long long walkers = (zmax * f + 3) / 4 * WK;
        for (int pieces = 1; pieces <= 64 && (pieces == 1 || a.h >= 4 * pieces); ++pieces) {
            const int len = (a.h + pieces - 1) / pieces, sps = (len + 2 + WG_NR - 1) / WG_NR;
            const long long per = (strips * pieces + walkers - 1) / walkers;
            const long long parts = (strips * pieces + per * WK - 1) / (per * WK);
            const double cost = 1.2 * (double)(per * sps) + 1.8e-6 * (double)(parts * n);
            if (k.len && cost >= best) continue;
            best = cost;
            k = WgradWalk{len, pieces, (int)per, sps, (int)parts};
        }
    }
    z = k.z;
    float *bpart = part + z * n;
    if (z == 1 && dw1) {                       // a single part is the gradient itself
        part = dw1;
        bpart = db1;
    }
    const dim3 grid((unsigned)(tiles * z));
    if (shape == 22)
        hipLaunchKernelGGL((k_wgrad_rows<PW, 2, 2, false, SUMS>), grid, dim3(512), 0, s, a, g, g_cs, g_co, rows, part, bpart, k);
    else if (shape == 14)
        hipLaunchKernelGGL((k_wgrad_rows<PW, 1, 4, false, SUMS>), grid, dim3(512), 0, s, a, g, g_cs, g_co, rows, part, bpart, k);
    else if (shape == 12)
        hipLaunchKernelGGL((k_wgrad_rows<PW, 1, 2, false, SUMS>), grid, dim3(512), 0, s, a, g, g_cs, g_co, rows, part, bpart, k);
    else
        hipLaunchKernelGGL((k_wgrad_rows<PW, 1, 1, true, SUMS>), grid, dim3(512), 0, s, a, g, g_cs, g_co, rows, part, bpart, k);
    return hipGetLastError();
}

// Weight gradient and (db) the bias gradient of the same G, whose partials
// follow the weight gradient's.
hipError_t wgrad(const ConvArgs &a, const uint16_t *g, int g_cs, int g_co, int rows, float *part, int splits,
                 float *dw, float *db, int accumulate, hipStream_t s) {
    const long long chunk = wgrad_chunk(a.M, splits), n = (long long)rows * a.K;
    int z = (int)((a.M + chunk - 1) / chunk);
    if (const int shape = rows_shape(a, rows, g_cs)) {
        const auto f = db ? (a.w > 16 ? launch_wgrad_rows<32, true> : launch_wgrad_rows<16, true>)
                          : (a.w > 16 ? launch_wgrad_rows<32, false> : launch_wgrad_rows<16, false>);
        const hipError_t e = f(shape, a, g, g_cs, g_co, rows, part, z, accumulate ? nullptr : dw, db, s);
        if (e != hipSuccess || (z == 1 && !accumulate)) return e;
    } else {
        const dim3 grid(rows <= 32 ? 1u : (unsigned)((rows + BM - 1) / BM),
                        rows <= 32 ? (unsigned)((a.K + 127) / 128) : (unsigned)((a.K + BN - 1) / BN), (unsigned)z);
        // a single part is the gradient itself
        const bool one = z == 1 && !accumulate && !(db && (a.flags & FLAG_S2D_G) && rows > 32);
        float *bpart = one && db && rows > 32 ? db : part + z * n;
        if (one) part = dw;
#define CALL(NARROW, SUMS) \
    hipLaunchKernelGGL((k_wgrad<NARROW, SUMS>), grid, dim3(256), 0, s, a, g, g_cs, g_co, rows, part, bpart, chunk)
        // at most 32 rows: a pass of its own for the bias gradient (16 x 256^2, 8 rows: 54 us with it, 66 us with the
        // sums in the weight gradient); more rows: 128 x 64 entries 48 us with the sums, 70 us with a pass
        if (rows <= 32) CALL(true, false);
        else if (db) CALL(false, true);
        else CALL(false, false);
#undef CALL
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        if (one && (!db || rows > 32)) return hipSuccess;
        if (db && rows <= 32) {
            const hipError_t e = one ? hipSuccess : sum_splits(part, z, n, dw, accumulate, s);
            if (e != hipSuccess) return e;
            const int fine = (a.flags & FLAG_S2D_G) ? a.dims : 0;
            const long long pixels = a.M << fine;
            const int C = rows >> fine;
            // about 16K elements (32 KB) of G per split, within the z rows floats that the workspace holds
            long long sp = (pixels * C + 16383) / 16384;
            if (sp > ((long long)z << fine)) sp = (long long)z << fine;
            return bias_grad(g, g_cs, g_co, pixels, C, bpart, (int)(sp < 1 ? 1 : sp), db, accumulate, s);
        }
    }
    if (!db) return sum_splits(part, z, n, dw, accumulate, s);
    const int fine = (a.flags & FLAG_S2D_G) ? a.dims : 0;         // rows = sub * C + co: a sub is a split more
    return sum_splits(part, z, n, dw, accumulate, s, part + z * n, z << fine, rows >> fine, db);
}

bool bias_grad8_ok(const void *g, int cs, int co, int C) {
    return cs % 8 == 0 && co % 8 == 0 && C % 8 == 0 && C <= 2048 && ((uintptr_t)g & 15) == 0;
}

hipError_t relu_bwd_bias_grad(uint16_t *g, const uint16_t *y, int cs, int co, long long npix, int C, float *part,
                              int splits, float *db, int accumulate, hipStream_t s) {
    if (!bias_grad8_ok(g, cs, co, C) || ((uintptr_t)y & 15) != 0) {
        hipError_t e = relu_bwd(g, y, cs, co, npix, C, s);
        return e != hipSuccess ? e : bias_grad(g, cs, co, npix, C, part, splits, db, accumulate, s);
    }
    const long long chunk = (npix + splits - 1) / splits;
    const int z = (int)((npix + chunk - 1) / chunk);
    hipLaunchKernelGGL(k_bias_grad8<true>, dim3((unsigned)z), dim3(256), 0, s, g, y, cs, co, npix, C, chunk, part);
    return sum_splits(part, z, (long long)C, db, accumulate, s);
}

hipError_t bias_grad(const uint16_t *g, int cs, int co, long long npix, int C, float *part, int splits, float *db,
                     int accumulate, hipStream_t s) {
    const long long chunk = (npix + splits - 1) / splits;
    const int z = (int)((npix + chunk - 1) / chunk);
    if (bias_grad8_ok(g, cs, co, C)) {
        hipLaunchKernelGGL(k_bias_grad8<false>, dim3((unsigned)z), dim3(256), 0, s, (uint16_t *)g, nullptr, cs, co,
                           npix, C, chunk, part);
    } else {
        dim3 grid((unsigned)((C + 63) / 64), (unsigned)z);
        hipLaunchKernelGGL(k_bias_grad, grid, dim3(256), 0, s, g, cs, co, npix, C, chunk, part);
    }
    return sum_splits(part, z, (long long)C, db, accumulate, s);
}

hipError_t relu_bwd(uint16_t *g, const uint16_t *y, int cs, int co, long long npix, int C, hipStream_t s) {
    hipLaunchKernelGGL(k_relu_bwd, dim3(blocks(npix * C, 256)), dim3(256), 0, s, g, y, cs, co, npix, C);
    return hipGetLastError();
}

static bool vec8(int a, int b, int c, int e, int f, const void *p, const void *q) {
    return ((a | b | c | e | f) & 7) == 0 && (((uintptr_t)p | (uintptr_t)q) & 15) == 0;
}

hipError_t pool_fwd(const uint16_t *in, int in_cs, int in_co, uint16_t *out, int out_cs, int out_co, int n, int d,
                    int h, int w, int C, int dims, hipStream_t s) {
    const long long tot = (long long)n * d * h * w * C;
    if (vec8(C, in_cs, in_co, out_cs, out_co, in, out)) {
        hipLaunchKernelGGL(k_pool_fwd8, dim3(blocks(tot / 8, 256)), dim3(256), 0, s, in, in_cs, in_co, out, out_cs,
                           out_co, n, d, h, w, C, dims);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_pool_fwd, dim3(blocks(tot, 256)), dim3(256), 0, s, in, in_cs, in_co, out, out_cs, out_co,
                       n, d, h, w, C, dims);
    return hipGetLastError();
}

hipError_t pool_bwd(const uint16_t *in, int in_cs, int in_co, const uint16_t *gout, int g_cs, int g_co,
                    uint16_t *gin, int gi_cs, int gi_co, int n, int d, int h, int w, int C, int dims, int acc,
                    int relu, hipStream_t s) {
    const long long tot = (long long)n * d * h * w * C;
    if (vec8(C, in_cs, in_co, g_cs, g_co, in, gout) && vec8(gi_cs, gi_co, 0, 0, 0, gin, nullptr)) {
#define CALL(DIMS, RELU)                                                                                          \
    hipLaunchKernelGGL((k_pool_bwd8<DIMS, RELU>), dim3(blocks(tot / 8, 256)), dim3(256), 0, s, in, in_cs, in_co, \
                       gout, g_cs, g_co, gin, gi_cs, gi_co, n, d, h, w, C, acc)
        if (dims == 2 && relu) CALL(2, true);
        else if (dims == 2) CALL(2, false);
        else if (relu) CALL(3, true);
        else CALL(3, false);
#undef CALL
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_pool_bwd, dim3(blocks(tot, 256)), dim3(256), 0, s, in, in_cs, in_co, gout, g_cs, g_co, gin,
                       gi_cs, gi_co, n, d, h, w, C, dims, acc, relu);
    return hipGetLastError();
}

hipError_t mse(const float *pred, int pcs, const float *tgt, const float *wpix, int creal, long long npix,
               float scale, uint16_t *dpred, double *part, double *loss, hipStream_t s) {
    const unsigned nb = blocks(npix, 256);
    hipLaunchKernelGGL(k_mse, dim3(nb), dim3(256), 0, s, pred, pcs, tgt, wpix, creal, npix, scale, dpred, part);
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(256), 0, s, part, (long long)nb, loss);
    return hipGetLastError();
}

hipError_t adam(float *w, const float *g, float *m1, float *m2, uint16_t *wb, long long n, float lr, float b1,
                float b2, float eps, int t, hipStream_t s) {
    const float c1 = 1.f / (1.f - powf(b1, (float)t)), c2 = 1.f / (1.f - powf(b2, (float)t));
    hipLaunchKernelGGL(k_adam, dim3(blocks(n, 256)), dim3(256), 0, s, w, g, m1, m2, wb, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t to_bf16(const float *x, uint16_t *y, long long n, hipStream_t s) {
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks(n, 256)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

hipError_t features(const uint8_t *solid, const float *prm, int n, int d, int h, int w, uint16_t *out,
                    hipStream_t s) {
    hipLaunchKernelGGL(k_features, dim3(blocks((long long)n * d * h * w, 256)), dim3(256), 0, s, solid, prm, n, d, h,
                       w, out);
    return hipGetLastError();
}

hipError_t normalize(const float *drho, const float *u, const uint8_t *solid, const float *prm, long long per_sample,
                     int D, long long npix, float *tgt, float *wpix, hipStream_t s) {
    hipLaunchKernelGGL(k_normalize, dim3(blocks(npix, 256)), dim3(256), 0, s, drho, u, solid, prm, per_sample, D, npix,
                       tgt, wpix);
    return hipGetLastError();
}

long long flux_balance_workspace_bytes(int n, long long rows, int w) {
    return (long long)n * w * (fb_chunks(rows) * (long long)sizeof(double) + (long long)sizeof(float));
}

hipError_t flux_balance(const uint8_t *solid, int n, int rows, int w, int D, float *u, void *ws, hipStream_t s) {
    const int P = fb_chunks(rows);
    double *part = (double *)ws;
    float *S = (float *)(part + (long long)n * P * w);
    hipLaunchKernelGGL(k_fb_partial, dim3((unsigned)P, (unsigned)n), dim3(256), 0, s, solid, u, rows, w, D, part);
    hipLaunchKernelGGL(k_fb_factors, dim3((unsigned)n), dim3(256), 0, s, part, P, w, S);
    const long long per = (long long)rows * w, tot = (long long)n * per * D;
    hipLaunchKernelGGL(k_fb_apply, dim3(blocks(tot, 256)), dim3(256), 0, s, u, S, tot, per, w, D);
    return hipGetLastError();
}

hipError_t denormalize(const float *pred, int pcs, const uint8_t *solid, const float *prm, long long per_sample,
                       int D, long long npix, float *drho, float *u, hipStream_t s) {
    hipLaunchKernelGGL(k_denormalize, dim3(blocks(npix, 256)), dim3(256), 0, s, pred, pcs, solid, prm, per_sample, D,
                       npix, drho, u);
    return hipGetLastError();
}

}  // namespace nn

namespace nn {

// wt[c][tap'][r] = w[r][tap][c], tap' = taps - 1 - tap when flipping (the
// input gradient of a correlation is the correlation with the flipped,
// transposed kernel).
__global__ void k_wtrans(const uint16_t *__restrict__ w, uint16_t *__restrict__ wt, int rows, int taps, int cols,
                         int flip) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n = (long long)rows * taps * cols;
    if (i >= n) return;
    const int c = (int)(i % cols);
    const int tap = (int)((i / cols) % taps);
    const int r = (int)(i / ((long long)cols * taps));
    const int tp = flip ? taps - 1 - tap : tap;
    wt[((long long)c * taps + tp) * rows + r] = w[i];
}

// The same for all layers of a network, whose launches cost more than the
// transposes (the 2D network's 20: 4 us each, 7 us together).  A block moves
// one 32 x 32 tile of one tap through LDS: 64-byte rows on both sides (a single
// layer is bound by its launch and one pass of loads and stores, 1 us shorter
// without the LDS).
__global__ void __launch_bounds__(256) k_wtrans_layers(const uint16_t *__restrict__ w, uint16_t *__restrict__ wt,
                                                       WtransLayers L) {
    __shared__ uint16_t T[32][33];
    const int lane = threadIdx.x & 63;
    const int l = __popcll(__builtin_amdgcn_ballot_w64(lane < L.n && L.first[lane] <= (int)blockIdx.x)) - 1;
    const int b = (int)blockIdx.x - L.first[l], rows = L.rows[l], taps = L.taps[l], cols = L.cols[l];
    const int tc = (cols + 31) >> 5, tr = (rows + 31) >> 5;
    const int c0 = b % tc * 32, r0 = b / tc % tr * 32, tap = b / (tc * tr), tp = L.flip[l] ? taps - 1 - tap : tap;
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    w += L.off[l];
    wt += L.off[l];
#pragma unroll
    for (int k = y; k < 32; k += 8)
        if (r0 + k < rows && c0 + x < cols) T[k][x] = w[((long long)(r0 + k) * taps + tap) * cols + c0 + x];
    __syncthreads();
#pragma unroll
    for (int k = y; k < 32; k += 8)
        if (c0 + k < cols && r0 + x < rows) wt[((long long)(c0 + k) * taps + tp) * rows + r0 + x] = T[x][k];
}

hipError_t wtrans(const uint16_t *w, uint16_t *wt, int rows, int taps, int cols, int flip, hipStream_t s) {
    const long long n = (long long)rows * taps * cols;
    hipLaunchKernelGGL(k_wtrans, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, wt, rows, taps, cols, flip);
    return hipGetLastError();
}

hipError_t wtrans_layers(const uint16_t *w, uint16_t *wt, const WtransLayers &L, hipStream_t s) {
    if (L.blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_wtrans_layers, dim3((unsigned)L.blocks), dim3(256), 0, s, w, wt, L);
    return hipGetLastError();
}

}  // namespace nn
