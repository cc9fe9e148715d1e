// Kernels of the learned warm-start network: 3x3 convolutions with 64
// channels in and out on MFMA (bfloat16 operands, FP32 accumulation), the
// loss and Adam.  Images are NHWC with the spectral bins as channels (the
// voxel order of the reconstruction); weights are [co][ky][kx][ci].
//
// Convolution as implicit GEMM: output pixels x output channels, reduction
// over (tap, input channel), K = 9 * 64 = 576, in tiles of
// v_mfma_f32_16x16x32_bf16 (lane l holds A[l%16][8(l/16)..+8],
// B[8(l/16)..+8][l%16], D[4(l/16)..+4][l%16]).
#include "sgtv_device.h"
#include "sgtv_wsnet.h"

namespace sgtv {
namespace wsn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef short v4s16 __attribute__((ext_vector_type(4)));
typedef short v8s16 __attribute__((ext_vector_type(8)));

constexpr int kC = 64;                 // channels
constexpr int kK = 9 * kC;             // reduction length of one output

__device__ __forceinline__ float softplusf(float z) { return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z))); }
__device__ __forceinline__ float sigmoidf(float z) {
    return z >= 0.0f ? 1.0f / (1.0f + expf(-z)) : expf(z) / (1.0f + expf(z));
}

constexpr int kRowPix = kC + 2;                    // staged pixels per row (width 64 + halo)
constexpr int kChunks = kC / 8;                    // 16-byte chunks per pixel (8 channels each)
constexpr int kConvThreads = 512;

// LDS layout: the weights [co][tap][ci] (576 bf16 per output channel) and the
// step's input rows [row][pixel][ci], both without padding.  A 16-byte chunk
// is stored at its index XOR (row or pixel index mod 8) within each group of
// 8 chunks, so the 16 lanes that read one MFMA fragment (16 pixels or 16
// output channels at the same channel offset) hit 8 distinct 16-byte bank
// groups per half instead of one.
size_t conv_lds_bytes(int rows) {
    return (static_cast<size_t>(kC) * kK + static_cast<size_t>(rows + 2) * kRowPix * kC) * 2;
}

__device__ __forceinline__ int swz(int chunk, int key) { return (chunk & ~7) | ((chunk ^ key) & 7); }

// EP 0: out_bf16 = relu(z + b) (hidden layer); 1: out_z = z + b, out_sp =
// softplus(z + b), either may be null (last layer); 2: out_bf16 = z if mask > 0
// else 0 (gradient through the ReLU of the previous layer, no bias).
//
// Persistent workgroups of 8 waves (two per SIMD, so one wave's LDS reads
// overlap the other's MFMAs), one per CU, stage all weights in LDS once and
// walk over steps of RS output rows of one image.  RS = 8: wave w computes row
// w, 64 pixels x 64 output channels as 4 x 4 tiles, each k-step of 32 (one tap,
// 32 input channels) reading 4 pixel and 4 weight fragments for 16 MFMAs.
// Fewer rows per step share a row between 2, 4 or 8 waves (32, 16 and 16 x half
// the channels), so that a small batch has a step for every CU (conv_rows); the
// order of the additions of an output is the same for every RS.
template <int EP, int RS>
__global__ __launch_bounds__(kConvThreads) void k_conv3x3(const __bf16 *__restrict__ X,
                                                          const __bf16 *__restrict__ Wk,
                                                          const float *__restrict__ bias, int B, int H,
                                                          __bf16 *__restrict__ out_bf16,
                                                          float *__restrict__ out_z,
                                                          float *__restrict__ out_sp,
                                                          const __bf16 *__restrict__ mask) {
    constexpr int kShare = 8 / RS;                     // waves per row
    constexpr int kPT = RS == 8 ? 4 : (RS == 4 ? 2 : 1);   // pixel tiles per wave
    constexpr int kUT = RS == 1 ? 2 : 4;               // output-channel tiles per wave
    constexpr int kStageRows = RS + 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __bf16 *ws = reinterpret_cast<__bf16 *>(smem);                  // [co][576], swizzled chunks
    __bf16 *xs = ws + static_cast<size_t>(kC) * kK;                 // [row][pixel][64], swizzled
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps_per_img = (H + RS - 1) / RS;
    const int n_steps = B * steps_per_img;

    // the input rows of a step, loaded into registers (all loads in flight at once)
    constexpr int kRChunks = kStageRows * kRowPix * kChunks, kRPer = (kRChunks + kConvThreads - 1) / kConvThreads;
    u16x8 rv[kRPer];
    auto load_rows = [&](int step) {
        const int n = step / steps_per_img, y0 = (step % steps_per_img) * RS;
#pragma unroll
        for (int k = 0; k < kRPer; ++k) {
            const int i = tid + k * kConvThreads;
            const int c8 = i % kChunks, rest = i / kChunks;
            const int xc = rest % kRowPix, r = rest / kRowPix;
            const int sy = y0 - 1 + r, sx = xc - 1;
            u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (i < kRChunks && sy >= 0 && sy < H && sx >= 0 && sx < kC)
                v = *reinterpret_cast<const u16x8 *>(X + ((static_cast<size_t>(n) * H + sy) * kC + sx) * kC + c8 * 8);
            rv[k] = v;
        }
    };

    // the weights and the first step's rows in flight together, then the
    // weights to LDS
    constexpr int kWChunks = kC * (kK / 8), kWPer = kWChunks / kConvThreads;
    static_assert(kWChunks % kConvThreads == 0, "weight chunks per thread");
    {
        u16x8 wr[kWPer];
#pragma unroll
        for (int k = 0; k < kWPer; ++k) {
            const int i = tid + k * kConvThreads, co = i / (kK / 8), k8 = i % (kK / 8);
            wr[k] = *reinterpret_cast<const u16x8 *>(Wk + static_cast<size_t>(co) * kK + k8 * 8);
        }
        if (static_cast<int>(blockIdx.x) < n_steps) load_rows(blockIdx.x);
#pragma unroll
        for (int k = 0; k < kWPer; ++k) {
            const int i = tid + k * kConvThreads, co = i / (kK / 8), k8 = i % (kK / 8);
            *reinterpret_cast<u16x8 *>(ws + co * kK + swz(k8, co) * 8) = wr[k];
        }
    }

    const int li = lane & 15, g = lane >> 4;
    const int wrow = wv / kShare, share = wv % kShare;
    const int pt0 = RS == 1 ? share / 2 : share * kPT, ut0 = RS == 1 ? (share % 2) * kUT : 0;
    for (int step = blockIdx.x; step < n_steps; step += gridDim.x) {
        const int n = step / steps_per_img, y0 = (step % steps_per_img) * RS;
        __syncthreads();                               // every wave is done with the previous step's LDS
#pragma unroll
        for (int k = 0; k < kRPer; ++k) {
            const int i = tid + k * kConvThreads;
            const int c8 = i % kChunks, rest = i / kChunks, xc = rest % kRowPix;
            if (i < kRChunks) *reinterpret_cast<u16x8 *>(xs + rest * kC + swz(c8, xc) * 8) = rv[k];
        }
        __syncthreads();
        // the next step's rows load while this one computes
        if (step + static_cast<int>(gridDim.x) < n_steps) load_rows(step + gridDim.x);

        f32x4 acc[kPT][kUT];
#pragma unroll
        for (int t = 0; t < kPT; ++t)
#pragma unroll
            for (int u = 0; u < kUT; ++u) acc[t][u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (y0 + wrow < H) {
#pragma unroll 1
            for (int tap = 0; tap < 9; ++tap) {
                const int ky = tap / 3, kx = tap % 3;
                const __bf16 *row = xs + (wrow + ky) * kRowPix * kC;
#pragma unroll
                for (int c0 = 0; c0 < kC; c0 += 32) {
                    const int cc = c0 / 8 + g;         // chunk of this lane's 8 input channels
                    bf16x8 a[kPT], b[kUT];
#pragma unroll
                    for (int t = 0; t < kPT; ++t) {
                        const int px = 16 * (pt0 + t) + li + kx;
                        a[t] = *reinterpret_cast<const bf16x8 *>(row + px * kC + swz(cc, px) * 8);
                    }
#pragma unroll
                    for (int u = 0; u < kUT; ++u) {
                        const int co = 16 * (ut0 + u) + li;
                        b[u] = *reinterpret_cast<const bf16x8 *>(ws + co * kK + swz(tap * kChunks + cc, co) * 8);
                    }
#pragma unroll
                    for (int t = 0; t < kPT; ++t)
#pragma unroll
                        for (int u = 0; u < kUT; ++u)
                            acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b[u], acc[t][u], 0, 0, 0);
                }
            }
        }
        __syncthreads();                               // the staged rows are free: the outputs pass through them

        // Epilogue through LDS: the step's outputs are written to the row area in
        // their own layout, then stored as 16-byte chunks by all threads.
        const size_t base = (static_cast<size_t>(n) * H + y0) * kC * kC;   // first element of row y0
        const int rows = H - y0 < RS ? H - y0 : RS;
        if (EP != 1) {
            __bf16 *tile = xs + wrow * (kC * kC);
#pragma unroll
            for (int t = 0; t < kPT; ++t)
#pragma unroll
                for (int u = 0; u < kUT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int px = 16 * (pt0 + t) + g * 4 + r, co = 16 * (ut0 + u) + li;
                        float z = acc[t][u][r];
                        if (EP == 0) z = fmaxf(z + bias[co], 0.0f);
                        tile[px * kC + co] = static_cast<__bf16>(z);
                    }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RS; ++k) {             // one row of chunks per turn
                if (k >= rows) break;
                const int c = k * kConvThreads + tid;
                u16x8 v = *reinterpret_cast<const u16x8 *>(xs + c * 8);
                if (EP == 2) {
                    const u16x8 m = *reinterpret_cast<const u16x8 *>(mask + base + c * 8);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        __bf16 mb;
                        const unsigned short mu = m[e];
                        __builtin_memcpy(&mb, &mu, 2);
                        if (!(static_cast<float>(mb) > 0.0f)) v[e] = 0;
                    }
                }
                *reinterpret_cast<u16x8 *>(out_bf16 + base + c * 8) = v;
            }
        } else {
            // FP32 z and softplus(z), 32 pixels at a time
            float *tile = reinterpret_cast<float *>(xs);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
                for (int t = 0; t < kPT; ++t) {
                    if ((pt0 + t) / 2 != hh) continue;
#pragma unroll
                    for (int u = 0; u < kUT; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int px = 16 * (pt0 + t) + g * 4 + r - 32 * hh, co = 16 * (ut0 + u) + li;
                            tile[(wrow * 32 + px) * kC + co] = acc[t][u][r] + bias[co];
                        }
                }
                __syncthreads();
#pragma unroll
                for (int k = 0; k < RS; ++k) {         // half a row of float4 per turn
                    if (k >= rows) break;
                    const f32x4 z = *reinterpret_cast<const f32x4 *>(tile + (k * kConvThreads + tid) * 4);
                    const size_t at = base + (static_cast<size_t>(k) * kC + 32 * hh) * kC + tid * 4;
                    if (out_z) *reinterpret_cast<f32x4 *>(out_z + at) = z;
                    if (out_sp) {   // uniform: training leaves softplus(z) to the loss kernel
                        f32x4 sp;
                        sp[0] = softplusf(z[0]);
                        sp[1] = softplusf(z[1]);
                        sp[2] = softplusf(z[2]);
                        sp[3] = softplusf(z[3]);
                        *reinterpret_cast<f32x4 *>(out_sp + at) = sp;
                    }
                }
                __syncthreads();
            }
        }
    }
}

// Weight and bias gradient of one layer: dW[co][tap][ci] = sum over pixels of
// dZ[pixel][co] X[pixel + tap][ci], a GEMM with the pixels as reduction.  The
// matrix cores want eight consecutive pixels of one channel per lane; both
// operands are staged in LDS as they lie in memory ([pixel][channel]) and read
// transposed (ds_read_b64_tr_b16: of 16 lanes, lane s reads four channels
// 4 (s mod 4) .. + 3 of pixel s / 4, and lane i receives channel i of the four
// pixels).
//
// Block b: R image rows of dZ and the R + 2 rows of X around them (zero outside
// the image), wave t = tap (ky, kx) with all 64 x 64 (co, ci) outputs of its tap
// as 4 x 4 tiles of v_mfma_f32_16x16x32_bf16.  The wave of the centre tap (which
// reads every row) also sums its dZ fragments: the block's bias partials follow
// its weight partials.  Row stride of part: C*9*C + C.
//
// A 32-byte group of 16 channels is stored at its index XOR a key of the pixel
// (bits 1 and 3), so the 32 lanes that a transposed read serves together (4 + 4
// pixels, 8 apart, 32 bytes each) cover all 64 banks once.
//
// Batch 32 of 64 x 64: 20 us, bound by its phases, which follow one another in
// the one block of a CU: 38 MB of operands with the halo in, 16 k-steps a row
// pair on the matrix cores (9 waves on 4 SIMDs), 38 MB of partial sums out.  With
// channel-major copies in memory (X in three shifts) it took 30 us, and writing
// the copies 6 to 7 us in every convolution around it.
constexpr int kWgradThreads = 9 * 64;

__device__ __forceinline__ int tr_key(int px) { return ((px >> 1) & 1) | ((px >> 2) & 2); }

size_t wgrad_lds_bytes(int R) { return (static_cast<size_t>(R + 2) * kRowPix + static_cast<size_t>(R) * kC) * kC * 2; }

template <int R>
__global__ __launch_bounds__(kWgradThreads) void k_wgrad(const __bf16 *__restrict__ DZ, const __bf16 *__restrict__ X,
                                                         int H, float *__restrict__ part) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned short *xs = reinterpret_cast<unsigned short *>(smem);   // [R + 2][66][64]
    unsigned short *ds = xs + (R + 2) * kRowPix * kC;                // [R][64][64]
    const int tid = threadIdx.x, lane = tid & 63;
    const int t = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ky = t / 3, kx = t % 3;
    const int li = lane & 15, g = lane >> 4;
    const int steps = (H + R - 1) / R;
    const int n = blockIdx.x / steps, y0 = (blockIdx.x - n * steps) * R;
    {
        // all of both in flight, then to LDS
        constexpr int kXN = (R + 2) * kRowPix * kChunks, kXPer = (kXN + kWgradThreads - 1) / kWgradThreads;
        constexpr int kDN = R * kC * kChunks, kDPer = (kDN + kWgradThreads - 1) / kWgradThreads;
        const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        u16x8 xv[kXPer], dv[kDPer];
#pragma unroll
        for (int k = 0; k < kXPer; ++k) {
            const int i = tid + k * kWgradThreads, c8 = i % kChunks, rest = i / kChunks;
            const int sx = rest % kRowPix - 1, sy = y0 - 1 + rest / kRowPix;
            xv[k] = zero;
            if (i < kXN && sy >= 0 && sy < H && sx >= 0 && sx < kC)
                xv[k] = *reinterpret_cast<const u16x8 *>(X + ((static_cast<size_t>(n) * H + sy) * kC + sx) * kC + c8 * 8);
        }
#pragma unroll
        for (int k = 0; k < kDPer; ++k) {
            const int i = tid + k * kWgradThreads, y = y0 + i / (kC * kChunks);
            dv[k] = zero;
            if (i < kDN && y < H)
                dv[k] = *reinterpret_cast<const u16x8 *>(DZ + (static_cast<size_t>(n) * H + y0) * kC * kC + i * 8);
        }
#pragma unroll
        for (int k = 0; k < kXPer; ++k) {
            const int i = tid + k * kWgradThreads, c8 = i % kChunks, rest = i / kChunks;
            if (i < kXN)
                *reinterpret_cast<u16x8 *>(xs + rest * kC + (((c8 >> 1) ^ tr_key(rest % kRowPix)) * 16 + (c8 & 1) * 8)) = xv[k];
        }
#pragma unroll
        for (int k = 0; k < kDPer; ++k) {
            const int i = tid + k * kWgradThreads, c8 = i % kChunks, rest = i / kChunks;
            if (i < kDN)
                *reinterpret_cast<u16x8 *>(ds + rest * kC + (((c8 >> 1) ^ tr_key(rest % kC)) * 16 + (c8 & 1) * 8)) = dv[k];
        }
    }
    // offsets of this lane's reads: pixels 8 g + li / 4 (+ 4), channels 4 (li % 4)
    // of 16-channel group i; a step of 32 pixels does not change the key
    int ao[2][4], bo[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int pa = 8 * g + (li >> 2) + 4 * h, pb = pa + kx;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ao[h][i] = pa * kC + (i ^ tr_key(pa)) * 16 + (li & 3) * 4;
            bo[h][i] = pb * kC + (i ^ tr_key(pb)) * 16 + (li & 3) * 4;
        }
    }
    __syncthreads();
    auto read8 = [](const unsigned short *p, int o0, int o1) {
        typedef __attribute__((address_space(3))) v4s16 *Lds;
        const v4s16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds)(p + o0));
        const v4s16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds)(p + o1));
        const v8s16 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, v);
    };
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float bs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int yy = 0; yy < R; ++yy) {
        // rows outside the image add nothing, whatever dZ and X hold (uniform)
        const int y = y0 + yy, sy = y + ky - 1;
        if (y >= H || sy < 0 || sy >= H) continue;
        const unsigned short *drow = ds + yy * kC * kC, *xrow = xs + (yy + ky) * kRowPix * kC;
#pragma unroll
        for (int p0 = 0; p0 < kC; p0 += 32) {
            bf16x8 a[4], b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = read8(xrow + p0 * kC, bo[0][j], bo[1][j]);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = read8(drow + p0 * kC, ao[0][i], ao[1][i]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            if (t == 4) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) bs[i] += static_cast<float>(a[i][e]);
            }
        }
    }
    float *out = part + static_cast<int64_t>(blockIdx.x) * (kC * kK + kC);
    if (t == 4) {
        // lanes li, li + 16, li + 32, li + 48 hold pixel quarters of channel 16 i + li
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = bs[i];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (g == 0) out[kC * kK + 16 * i + li] = v;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                out[(16 * i + 4 * g + q) * kK + t * kC + 16 * j + li] = acc[i][j][q];
}

// grad[k] = sum over blocks b of part[b][k] in a fixed order: four contiguous
// quarters of the blocks summed in order, then ((q0 + q1) + (q2 + q3)).
__global__ __launch_bounds__(256) void k_block_sum(const float *__restrict__ part, int n_blocks,
                                                   int64_t len, float *__restrict__ grad) {
    __shared__ float s4[4][64];
    const int kl = threadIdx.x & 63, qt = threadIdx.x >> 6;
    const int64_t k = static_cast<int64_t>(blockIdx.x) * 64 + kl;
    const int per = (n_blocks + 3) / 4;
    const int b0 = qt * per, b1 = min(n_blocks, b0 + per);
    float acc = 0.0f;
    if (k < len) {
        // eight loads in flight, then their additions in block order
        int b = b0;
        for (; b + 8 <= b1; b += 8) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = part[static_cast<int64_t>(b + u) * len + k];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += t[u];
        }
        for (; b < b1; ++b) acc += part[static_cast<int64_t>(b) * len + k];
    }
    s4[qt][kl] = acc;
    __syncthreads();
    if (qt == 0 && k < len) grad[k] = (s4[0][kl] + s4[1][kl]) + (s4[2][kl] + s4[3][kl]);
}

// Eight values per thread: two 16-byte loads, one 16-byte store (batch 32 of
// 64 x 64: 9.8 us = 5.1 TB/s, against 11.4 us one value at a time).
__device__ __forceinline__ bf16x8 to_bf16x8(f32x4 a, f32x4 b) {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = static_cast<__bf16>(a[e]);
        v[e + 4] = static_cast<__bf16>(b[e]);
    }
    return v;
}

__global__ __launch_bounds__(256) void k_to_bf16(const float *__restrict__ x, __bf16 *__restrict__ y, int64_t n8) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n8;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(x) + 2 * i;
        reinterpret_cast<bf16x8 *>(y)[i] = to_bf16x8(p[0], p[1]);
    }
}

// FP64 partial sums of each image: grid (n_blocks, images)
__global__ __launch_bounds__(256) void k_image_partials(const float *__restrict__ x, int64_t img,
                                                        double *__restrict__ partials) {
    const f32x4 *xi = reinterpret_cast<const f32x4 *>(x + static_cast<int64_t>(blockIdx.y) * img);
    double acc = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < img / 4;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const f32x4 v = xi[i];
        acc += (static_cast<double>(v[0]) + v[1]) + (static_cast<double>(v[2]) + v[3]);
    }
    block_sum_store(acc, partials + static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x);
}

// mean of image b from its sum; 1 where the mean is not positive
__device__ __forceinline__ double image_mean(const double *sums, int64_t b, int64_t img) {
    const double m = sums[b] / static_cast<double>(img);
    return m > 0.0 ? m : 1.0;
}

// network input: x / mean(image), rounded to bfloat16; grid (blocks, images).
// One FP64 division per thread and a product per value: the quotient in FP32
// differs from a division's only where that lies within 2^-28 of a rounding
// boundary (a division per value took 20.2 us for batch 32, this takes 10.3 us).
__global__ __launch_bounds__(256) void k_scale_to_bf16(const float *__restrict__ x, const double *__restrict__ sums,
                                                       int64_t img, __bf16 *__restrict__ y) {
    const double inv = 1.0 / image_mean(sums, blockIdx.y, img);
    const int64_t base = static_cast<int64_t>(blockIdx.y) * img / 8;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < img / 8;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(x) + 2 * (base + i);
        f32x4 a = p[0], b = p[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = static_cast<float>(a[e] * inv);
            b[e] = static_cast<float>(b[e] * inv);
        }
        reinterpret_cast<bf16x8 *>(y)[base + i] = to_bf16x8(a, b);
    }
}

// start image from the network output s: c_out * s * f (ratio) or c_out * s * mean(f)
// (direct); grid (blocks, images)
__global__ __launch_bounds__(256) void k_start_image(const float *f, const float *__restrict__ s,
                                                     const double *__restrict__ sums, int64_t img, float c_out,
                                                     int ratio, float floor, float *x0) {
    const float m = static_cast<float>(image_mean(sums, blockIdx.y, img));
    const int64_t base = static_cast<int64_t>(blockIdx.y) * img / 4;
    for (int64_t i = base + static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < base + img / 4;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const f32x4 sv = reinterpret_cast<const f32x4 *>(s)[i];
        f32x4 v = f32x4{m, m, m, m};
        if (ratio) v = reinterpret_cast<const f32x4 *>(f)[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = c_out * sv[e] * v[e];
            if (floor > 0.0f) v[e] = fmaxf(v[e], floor * c_out * m);
        }
        reinterpret_cast<f32x4 *>(x0)[i] = v;
    }
}

// dZ of the last layer: 2 (out - target) / n * softplus'(z) with out =
// softplus(z) (the same function as the layer's epilogue); FP64 loss partials.
// Bound by its arithmetic (expf, log1pf and a division per value): batch 32 of
// 64 x 64 34 us, 2.4 TB/s.
__global__ __launch_bounds__(256) void k_mse_grad(const float *__restrict__ target,
                                                  const float *__restrict__ z, int64_t n,
                                                  __bf16 *__restrict__ dz,
                                                  double *__restrict__ partials) {
    double acc = 0.0;
    const float inv = 2.0f / static_cast<float>(n);
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n / 4;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const f32x4 zv = reinterpret_cast<const f32x4 *>(z)[i], tv = reinterpret_cast<const f32x4 *>(target)[i];
        bf16x4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // softplusf(z) and sigmoidf(z) from one exp(-|z|): exp(-z) for z >= 0
            // and exp(z) below, bit for bit the values of the two functions
            const float zi = zv[k];
            const float e = expf(-fabsf(zi));
            const float sp = fmaxf(zi, 0.0f) + log1pf(e);
            const float sg = (zi >= 0.0f ? 1.0f : e) / (1.0f + e);
            const float d = sp - tv[k];
            acc += static_cast<double>(d) * d;
            o[k] = static_cast<__bf16>(inv * d * sg);
        }
        reinterpret_cast<bf16x4 *>(dz)[i] = o;
    }
    block_sum_store(acc, partials + blockIdx.x);
}

// One training step's mean squared error (its sum l[0] over cnt values) added
// to the running sum acc[0], and the step to the count acc[1].
__global__ void k_loss_accumulate(const double *__restrict__ l, double cnt, double *__restrict__ acc) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        acc[0] += l[0] / cnt;
        acc[1] += 1.0;
    }
}

// 1 - beta1 and 1 - beta2 come from the host, formed in FP64: 1 - 0.999f in
// FP32 would be 0.000999987, a 1.3e-5 relative error in every second moment.
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float omb1,
                       float omb2, float eps, float c1, float c2) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + omb1 * gi;
        const float vi = b2 * v[i] + omb2 * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// bfloat16 copies of one layer's weights: forward [co][tap][ci], and the
// backward-data kernel [ci][8 - tap][co] (flipped taps, swapped channels)
__global__ void k_weights_bf16(const float *__restrict__ w, __bf16 *__restrict__ wf,
                               __bf16 *__restrict__ wb) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kC * kK) return;
    const int co = i / kK, tap = (i % kK) / kC, ci = i % kC;
    const __bf16 h = static_cast<__bf16>(w[i]);
    wf[i] = h;
    wb[(static_cast<size_t>(ci) * 9 + (8 - tap)) * kC + co] = h;
}

// ---------------------------------------------------------------- launchers
int conv_workgroups() {
    // computed once (thread-safe initialisation of a function-local static)
    static const int n = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
            return cus;
        return 256;
    }();
    return n;
}

template <int EP, int RS>
static hipError_t conv_rs(const __bf16 *X, const __bf16 *Wk, const float *bias, int B, int H, __bf16 *ob, float *oz,
                          float *osp, const __bf16 *mask, hipStream_t st) {
    static const hipError_t raised = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_conv3x3<EP, RS>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
    if (raised != hipSuccess) return raised;
    const int n_steps = B * ((H + RS - 1) / RS);
    if (n_steps == 0) return hipSuccess;
    // one workgroup per CU (the staged weights and rows take 97 to 155 KB of LDS)
    const int grid = std::min(n_steps, conv_workgroups());
    hipLaunchKernelGGL((k_conv3x3<EP, RS>), dim3(static_cast<unsigned>(grid)), dim3(kConvThreads), conv_lds_bytes(RS),
                       st, X, Wk, bias, B, H, ob, oz, osp, mask);
    return hipGetLastError();
}

// Rows per step: the most (up to 8) that still give three quarters of the CUs a
// step.  One image of 64 rows (hidden layer / last layer): 8 rows on 8 CUs
// 12.4 / 34.6 us, 1 row on 64 CUs 5.5 / 8.8 us; 7 images of 36 rows: 17.5 us with
// 8 rows on 35 CUs, 5.9 us with 1 row on 252.
static int conv_rows(int B, int H) {
    int rs = 8;
    while (rs > 1 && B * ((H + rs - 1) / rs) * 4 < 3 * conv_workgroups()) rs /= 2;
    return rs;
}

template <int EP>
static hipError_t conv_t(const __bf16 *X, const __bf16 *Wk, const float *bias, int B, int H, __bf16 *ob, float *oz,
                         float *osp, const __bf16 *mask, hipStream_t st) {
    switch (conv_rows(B, H)) {
    case 8: return conv_rs<EP, 8>(X, Wk, bias, B, H, ob, oz, osp, mask, st);
    case 4: return conv_rs<EP, 4>(X, Wk, bias, B, H, ob, oz, osp, mask, st);
    case 2: return conv_rs<EP, 2>(X, Wk, bias, B, H, ob, oz, osp, mask, st);
    default: return conv_rs<EP, 1>(X, Wk, bias, B, H, ob, oz, osp, mask, st);
    }
}

hipError_t conv_relu(const __bf16 *X, const __bf16 *Wk, const float *bias, int B, int H, __bf16 *out, hipStream_t st) {
    return conv_t<0>(X, Wk, bias, B, H, out, nullptr, nullptr, nullptr, st);
}
hipError_t conv_softplus(const __bf16 *X, const __bf16 *Wk, const float *bias, int B, int H, float *z, float *sp,
                         hipStream_t st) {
    return conv_t<1>(X, Wk, bias, B, H, nullptr, z, sp, nullptr, st);
}
hipError_t conv_masked(const __bf16 *X, const __bf16 *Wk, int B, int H, const __bf16 *mask, __bf16 *out,
                       hipStream_t st) {
    return conv_t<2>(X, Wk, nullptr, B, H, out, nullptr, nullptr, mask, st);
}

// Rows per block of the weight gradient: 8, fewer while half the CUs would have
// no block.
static int wgrad_rows(int B, int H) {
    int r = 8;
    while (r > 2 && B * ((H + r - 1) / r) < 128) r /= 2;
    return r;
}

int wgrad_blocks(int B, int H) {
    const int r = wgrad_rows(B, H);
    return B * ((H + r - 1) / r);
}

template <int R>
static hipError_t wgrad_r(const __bf16 *X, const __bf16 *DZ, int nb, int H, float *wpart, hipStream_t st) {
    static const hipError_t raised = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_wgrad<R>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
    if (raised != hipSuccess) return raised;
    hipLaunchKernelGGL(k_wgrad<R>, dim3(static_cast<unsigned>(nb)), dim3(kWgradThreads), wgrad_lds_bytes(R), st, DZ, X,
                       H, wpart);
    return hipGetLastError();
}

hipError_t conv_wgrad(const __bf16 *X, const __bf16 *DZ, int B, int H, float *wpart, float *grad, hipStream_t st) {
    const int nb = wgrad_blocks(B, H);
    if (nb == 0) return hipSuccess;
    const int r = wgrad_rows(B, H);
    hipError_t e = r == 8   ? wgrad_r<8>(X, DZ, nb, H, wpart, st)
                   : r == 4 ? wgrad_r<4>(X, DZ, nb, H, wpart, st)
                            : wgrad_r<2>(X, DZ, nb, H, wpart, st);
    if (e != hipSuccess) return e;
    const int64_t len = static_cast<int64_t>(kC) * kK + kC;
    hipLaunchKernelGGL(k_block_sum, dim3(static_cast<unsigned>((len + 63) / 64)), dim3(256), 0, st,
                       wpart, nb, len, grad);
    return hipGetLastError();
}

hipError_t to_bf16(const float *x, __bf16 *y, int64_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_to_bf16, dim3(static_cast<unsigned>(std::min<int64_t>(4096, (n / 8 + 255) / 256))),
                       dim3(256), 0, st, x, y, n / 8);
    return hipGetLastError();
}

hipError_t image_partials(const float *x, int64_t img, int n_images, int n_blocks, double *partials,
                          hipStream_t st) {
    if (n_images == 0) return hipSuccess;
    hipLaunchKernelGGL(k_image_partials, dim3(static_cast<unsigned>(n_blocks), static_cast<unsigned>(n_images)),
                       dim3(256), 0, st, x, img, partials);
    return hipGetLastError();
}

// blocks per image of the elementwise kernels: about 4096 in all
static dim3 image_grid(int64_t per_image, int n_images) {
    const int64_t most = std::max<int64_t>(1, 4096 / n_images);
    return dim3(static_cast<unsigned>(std::min<int64_t>(most, (per_image + 255) / 256)),
                static_cast<unsigned>(n_images));
}

hipError_t scale_to_bf16(const float *x, const double *sums, int64_t img, int n_images, __bf16 *y, hipStream_t st) {
    if (n_images == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scale_to_bf16, image_grid(img / 8, n_images), dim3(256), 0, st, x, sums, img, y);
    return hipGetLastError();
}

hipError_t start_image(const float *f, const float *s, const double *sums, int64_t img, int n_images, float c_out,
                       int ratio, float floor, float *x0, hipStream_t st) {
    if (n_images == 0) return hipSuccess;
    hipLaunchKernelGGL(k_start_image, image_grid(img / 4, n_images), dim3(256), 0, st, f, s, sums, img, c_out, ratio,
                       floor, x0);
    return hipGetLastError();
}

hipError_t mse_grad(const float *target, const float *z, int64_t n, __bf16 *dz, double *partials,
                    int n_blocks, hipStream_t st) {
    hipLaunchKernelGGL(k_mse_grad, dim3(static_cast<unsigned>(n_blocks)), dim3(256), 0, st, target, z, n, dz,
                       partials);
    return hipGetLastError();
}

hipError_t loss_accumulate(const double *l, double cnt, double *acc, hipStream_t st) {
    hipLaunchKernelGGL(k_loss_accumulate, dim3(1), dim3(64), 0, st, l, cnt, acc);
    return hipGetLastError();
}

hipError_t adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1,
                float b2, float omb1, float omb2, float eps, float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3(static_cast<unsigned>(std::min<int64_t>(4096, (n + 255) / 256))),
                       dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, omb1, omb2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t weights_bf16(const float *w, __bf16 *wf, __bf16 *wb, hipStream_t st) {
    hipLaunchKernelGGL(k_weights_bf16, dim3((kC * kK + 255) / 256), dim3(256), 0, st, w, wf, wb);
    return hipGetLastError();
}

}  // namespace wsn
}  // namespace sgtv
