// 3x3 convolutions of the reduced-precision U-Nets (16-bit, split bfloat16 and
// e4m3) as implicit GEMMs on the gfx950 matrix cores.
//
// Fig. 1 and Method, "U-Net Reconstruction".  M = output channels, N = output
// pixels, K = 9 taps x input channels, on 32x32 MFMA blocks of 16 channels.
//
// Activations lie in memory as the matrix cores want them: a tensor is a list
// of channel blocks, each block a dense H x W plane of 16-byte units, one unit
// holding a pixel's operands for the block's channels:
//   MODE 1 bf16    8 channels per block
//   MODE 3 fp16    8 channels per block
//   MODE 2 bf16x3  8 channels per block; the tensor's hi plane (all blocks),
//                  then its lo plane: a float32 value is split into bfloat16
//                  hi + lo when it is produced (the multiplications only ever
//                  use the two parts), product lo*hi + hi*lo + hi*hi
//   MODE 4 e4m3    16 channels per block (of the value rounded to float16)
//   MODE 5 e4m3x3  8 channels per block, 8 bytes hi then 8 bytes lo
// So the halo tile of a chunk of 16 channels is a few runs of consecutive
// units per image row, which go to LDS by direct loads (no registers, no
// vector instructions), and the lanes of an accumulator block, which hold 4
// consecutive channels of 32 consecutive pixels, store whole cache lines.
// Nothing is converted on the way in: the rounding of the next layer's operand
// is done once, where the value is produced.
//
// Sums are taken over 16-channel groups, then horizontal, then vertical taps,
// whatever the tile, so the tile choice does not change results.
#include <hip/hip_runtime.h>

#include <cmath>

#include "conv_stage.h"

namespace lnr {
namespace {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// per MODE: channel blocks (16-byte units per pixel) of a 16-channel chunk,
// planes read as separate fragments, and weight units per (tap, output channel)
template <int MODE>
struct Fmt;
template <>
struct Fmt<1> {
  static constexpr int kBlocks = 2, kPlanes = 1, kWUnits = 2;
};
template <>
struct Fmt<2> {
  static constexpr int kBlocks = 4, kPlanes = 2, kWUnits = 4;
};
template <>
struct Fmt<3> : Fmt<1> {};
template <>
struct Fmt<4> {
  static constexpr int kBlocks = 1, kPlanes = 1, kWUnits = 1;
};
template <>
struct Fmt<5> : Fmt<1> {};  // one unit holds both planes

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  const floatx2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));  // round to nearest even
}
__device__ inline uint32_t pack_f16x2(float lo, float hi) {
  const floatx2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));  // round to nearest even
}
template <int MODE>
__device__ inline uint32_t pack16x2(float lo, float hi) {
  if constexpr (MODE == 1 || MODE == 2) return pack_bf16x2(lo, hi);
  else return pack_f16x2(lo, hi);
}
// what bfloat16 rounding left of two values (hi = their packed rounding)
__device__ inline uint32_t rest_bf16x2(float f0, float f1, uint32_t hi) {
  return pack_bf16x2(f0 - __uint_as_float(hi << 16), f1 - __uint_as_float(hi & 0xFFFF0000u));
}
// two packed float16 values -> two OCP e4m3 bytes in the chosen half of `old`,
// rounded to nearest even, saturating at +-448; with LO, the e4m3 of what the
// first rounding left (x - e4m3(x)) instead
template <bool LO>
__device__ inline int f16x2_to_e4m3(uint32_t w, int old, bool high_word) {
  float f0 = (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xFFFFu));
  float f1 = (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
  f0 = fminf(fmaxf(f0, -448.f), 448.f);
  f1 = fminf(fmaxf(f1, -448.f), 448.f);
  if constexpr (LO) {
    const int h = __builtin_amdgcn_cvt_pk_fp8_f32(f0, f1, 0, false);
    f0 = f0 - __builtin_amdgcn_cvt_f32_fp8(h, 0);
    f1 = f1 - __builtin_amdgcn_cvt_f32_fp8(h, 1);
  }
  return high_word ? __builtin_amdgcn_cvt_pk_fp8_f32(f0, f1, old, true)
                   : __builtin_amdgcn_cvt_pk_fp8_f32(f0, f1, old, false);
}
// four values (as packed float16 pairs) -> four e4m3 bytes
template <bool LO>
__device__ inline uint32_t e4m3x4(uint32_t h01, uint32_t h23) {
  return (uint32_t)f16x2_to_e4m3<LO>(h23, f16x2_to_e4m3<LO>(h01, 0, false), true);
}

// v / 255 correctly rounded, v = 0 .. 255: one correction step of the product
// with the rounded reciprocal (checked for all 256 values)
__device__ inline float over255(uint32_t v) {
  const float f = (float)v, r = 1.0f / 255.0f, y = f * r;
  return fmaf(fmaf(-255.0f, y, f), r, y);
}
// network input x = (r/255, g/255, b/255, A ? D/16 : 0, A, 0, ...) of a pixel
// as operand units: u[0], and u[1] (the lo plane) for MODE 2
template <int MODE>
__device__ inline void input_units(uint32_t q, float d, uint4 *u) {
  const bool A = (q >> 24) != 0;
  const float x0 = over255(q & 255u), x1 = over255((q >> 8) & 255u), x2 = over255((q >> 16) & 255u);
  const float x3 = A ? d * 0.0625f : 0.f, x4 = A ? 1.f : 0.f;
  const uint32_t p01 = pack16x2<MODE>(x0, x1), p23 = pack16x2<MODE>(x2, x3), p4 = pack16x2<MODE>(x4, 0.f);
  if constexpr (MODE == 1 || MODE == 3) {
    u[0] = make_uint4(p01, p23, p4, 0u);
  } else if constexpr (MODE == 2) {
    u[0] = make_uint4(p01, p23, p4, 0u);
    u[1] = make_uint4(rest_bf16x2(x0, x1, p01), rest_bf16x2(x2, x3, p23), rest_bf16x2(x4, 0.f, p4), 0u);
  } else if constexpr (MODE == 4) {
    u[0] = make_uint4(e4m3x4<false>(p01, p23), e4m3x4<false>(p4, 0u), 0u, 0u);
  } else {
    u[0] = make_uint4(e4m3x4<false>(p01, p23), e4m3x4<false>(p4, 0u), e4m3x4<true>(p01, p23), e4m3x4<true>(p4, 0u));
  }
}

// acc += A x B over 16 channels of one tap
template <int MODE, typename F>
__device__ inline void mma(const F (&a)[Fmt<MODE>::kPlanes], const F (&b)[Fmt<MODE>::kPlanes], floatx16 &acc) {
  if constexpr (MODE == 1) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[0]), __builtin_bit_cast(bf16x8, b[0]),
                                                  acc, 0, 0, 0);
  } else if constexpr (MODE == 3) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a[0]), __builtin_bit_cast(f16x8, b[0]),
                                                 acc, 0, 0, 0);
  } else if constexpr (MODE == 2) {
    const bf16x8 ah = __builtin_bit_cast(bf16x8, a[0]), al = __builtin_bit_cast(bf16x8, a[1]);
    const bf16x8 bh = __builtin_bit_cast(bf16x8, b[0]), bl = __builtin_bit_cast(bf16x8, b[1]);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
  } else if constexpr (MODE == 4) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(__builtin_bit_cast(long, a[0]), __builtin_bit_cast(long, b[0]),
                                                     acc, 0, 0, 0);
  } else {
    const long ah = __builtin_bit_cast(long, make_uint2(a[0].x, a[0].y)), al = __builtin_bit_cast(long, make_uint2(a[0].z, a[0].w));
    const long bh = __builtin_bit_cast(long, make_uint2(b[0].x, b[0].y)), bl = __builtin_bit_cast(long, make_uint2(b[0].z, b[0].w));
    acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(al, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(ah, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(ah, bh, acc, 0, 0, 0);
  }
}
template <int MODE>
struct FragOf {
  using type = uint4;
};
template <>
struct FragOf<4> {
  using type = uint2;  // 8 e4m3 per lane
};

// One staged chunk of 16 input channels: nine taps, horizontal offset dx outer,
// vertical offset dy inner.  An input row's fragment, read once per dx, feeds
// the up to three taps that use it.  A: this lane's weights (half h, channel n
// of the chunk's first channel tile), B: this lane's pixel (its wave's first
// halo row, column n); UBP: units per staged channel block, LW: units per staged
// row.  A tap's fragments are read kAhead taps (8 matrix instructions or more)
// before it, and load(-1), which prepares the loads of later steps, and load(0
// .. LOADS - 1), which start them, stand between the matrix instructions of the
// first six taps, which hide their scalar instructions.  PIN keeps the compiler to that order; with the
// loads in front of the chunk and the reads in its own order the largest
// 512-channel layers at 240 x 135 took 319 us for 300, 13 x 13 pixels
// with split e4m3 operands 52.8 for 42.2; a kernel of one chunk is better left
// to it (37.4 for 35.3 us).  Branches around the loads past the last step cost
// more than the masked loads (208 x 208, split e4m3: 371 for 330 us), and a second
// copy of the chunk without loads spills.
template <int MODE, int MB, int R, int UBP, int LW, int LOADS, bool PIN, typename Load>
__device__ inline void chunk_mma(const char *A, const char *B, floatx16 (&acc)[MB][R], Load load) {
  using F = typename FragOf<MODE>::type;
  constexpr int P = Fmt<MODE>::kPlanes, WU = Fmt<MODE>::kWUnits;
  constexpr int AT = (WU / P) * 512, AP = 9 * AT, AM = P * AP;  // bytes per tap, plane, channel tile
  constexpr int kPerTap = MB * R * (MODE == 2 || MODE == 5 ? 3 : 1), kAhead = kPerTap >= 8 ? 1 : (8 + kPerTap - 1) / kPerTap;
  constexpr int kPerLoads = (LOADS + 4) / 5;  // loads per tap, all within the first five
  F a[3][3][MB][P], b[3][R + 2][P];
  auto read = [&](int s) {
    const int dx = s / 3, dy = s % 3;
#pragma unroll
    for (int i = dy == 0 ? 0 : R - 1 + dy; i < R + dy; ++i)
#pragma unroll
      for (int p = 0; p < P; ++p)
        b[dx][i][p] = *reinterpret_cast<const F *>(B + p * 2 * UBP * 16 + (i * LW + dx) * 16);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int p = 0; p < P; ++p)
        a[dx][dy][mb][p] = *reinterpret_cast<const F *>(A + mb * AM + p * AP + (dy * 3 + dx) * AT);
  };
#pragma unroll
  for (int s = 0; s < kAhead; ++s) read(s);
#pragma unroll
  for (int s = 0; s < 9; ++s) {
    if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
    if (s + kAhead < 9) read(s + kAhead);
    int l = (s - 1) * kPerLoads;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) mma<MODE>(a[s / 3][s % 3][mb], b[s / 3][r + s % 3], acc[mb][r]);
      if (LOADS > 0 && s == 0 && r == 0) load(-1);
      const int until = (s - 1) * kPerLoads + (r + 1) * kPerLoads / R;
#pragma unroll
      for (; l < until; ++l)
        if (l >= 0 && l < LOADS) load(l);
    }
  }
  if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
}
// this lane's offsets within a chunk's weights and a pixel's units
template <int MODE>
__device__ inline int lane_a(int n, int h) {
  if constexpr (MODE == 4) return n * 16 + 8 * h;
  else return (h * 32 + n) * 16;
}
template <int MODE, int UBP>
__device__ inline int lane_b(int pixel, int h) {
  if constexpr (MODE == 4) return pixel * 16 + 8 * h;
  else return (h * UBP + pixel) * 16;
}

// four values of channels c + 4h .. c + 4h + 3 of one pixel, as the operands of
// the next layer.  base: the tensor (this image), plane: bytes per channel
// block, C channels of the tensor, px: 16 times the pixel's index (below 2^32
// for every image the library takes).  Both halves of a wave (h = 0 and 1 of
// one pixel) call it together.
template <int MODE>
__device__ inline void put_operands(char *base, size_t plane, int C, int c, int h, uint32_t px, const float (&v)[4],
                                    bool live) {
  const uint32_t p01 = pack16x2<MODE>(v[0], v[1]), p23 = pack16x2<MODE>(v[2], v[3]);
  char *u = base + (size_t)(c >> 3) * plane;  // the 8-channel block
  if constexpr (MODE == 1 || MODE == 3) {
    if (live) *reinterpret_cast<uint2 *>(u + (px + 8 * h)) = make_uint2(p01, p23);
  } else if constexpr (MODE == 2) {
    if (live) {
      *reinterpret_cast<uint2 *>(u + (px + 8 * h)) = make_uint2(p01, p23);
      *reinterpret_cast<uint2 *>(u + (size_t)(C >> 3) * plane + (px + 8 * h)) =
          make_uint2(rest_bf16x2(v[0], v[1], p01), rest_bf16x2(v[2], v[3], p23));
    }
  } else if constexpr (MODE == 5) {
    // lane h = 0 writes the 8 hi bytes, lane h = 1 the 8 lo bytes
    const uint32_t hi = e4m3x4<false>(p01, p23), lo = e4m3x4<true>(p01, p23);
    const uint32_t got = (uint32_t)__shfl_xor((int)(h ? hi : lo), 32, 64);
    if (live) *reinterpret_cast<uint2 *>(u + (px + 8 * h)) = h ? make_uint2(got, lo) : make_uint2(hi, got);
  } else {
    if (live)
      *reinterpret_cast<uint32_t *>(base + (size_t)(c >> 4) * plane + (px + (c & 8) + 4 * h)) = e4m3x4<false>(p01, p23);
  }
}
// the same four values as head_kernel reads them: blocks of 8 16-bit or 4 float32 channels
template <int MODE>
__device__ inline void put_raw(char *base, size_t plane, int c, int h, uint32_t px, const float (&v)[4]) {
  if constexpr (MODE == 2)
    *reinterpret_cast<float4 *>(base + (size_t)(2 * (c >> 3) + h) * plane + px) = make_float4(v[0], v[1], v[2], v[3]);
  else
    *reinterpret_cast<uint2 *>(base + (size_t)(c >> 3) * plane + (px + 8 * h)) =
        make_uint2(pack16x2<MODE>(v[0], v[1]), pack16x2<MODE>(v[2], v[3]));
}

// the value of the lane next to this one (pixel n ^ 1)
__device__ inline float lane_xor1(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0xB1, 0xF, 0xF, true));
}
template <int MODE>
__device__ inline float scaled(float acc, float ws) {
  if constexpr (MODE == 4 || MODE == 5) return acc * ws;
  else return acc;
}

// Bias, ReLU and stores.  Accumulator register 4j + i of block (mb, r) holds
// output channel co0 + 32 mb + 8j + 4h + i of pixel (gy0 + r, gx).  s_bias,
// s_ws: the tile's 32 MB biases and weight scales in LDS; s_head: the head's
// weights [3][32 MB] (a global load here would wait for the loads in flight).
template <int MODE, int MB, int R, bool HEAD>
__device__ inline void epilogue(const Args &a, int img, int co0, int gy0, int gx, int h, const floatx16 (&acc)[MB][R],
                                const float *s_bias, const float *s_ws, const float *s_head) {
  const int H = a.H, W = a.W;
  const size_t HW = (size_t)H * W;
  if constexpr (HEAD) {
    // per row, the sums run over (mb, j, i) in order; the bias and head weights
    // of a group of 4 channels are read once for all rows
    float hs[R][3];
#pragma unroll
    for (int r = 0; r < R; ++r) hs[r][0] = hs[r][1] = hs[r][2] = 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = co0 + mb * 32 + 8 * j + 4 * h;
        if (c < a.cout) {
          const float4 b = *reinterpret_cast<const float4 *>(s_bias + c - co0);
          const float bb[4] = {b.x, b.y, b.z, b.w};
          float ws[4] = {1.f, 1.f, 1.f, 1.f};
          if constexpr (MODE == 4 || MODE == 5) {
            const float4 w4 = *reinterpret_cast<const float4 *>(s_ws + c - co0);
            ws[0] = w4.x; ws[1] = w4.y; ws[2] = w4.z; ws[3] = w4.w;
          }
          float hw[3][4];
#pragma unroll
          for (int o = 0; o < 3; ++o) {
            const float4 w = *reinterpret_cast<const float4 *>(s_head + o * 32 * MB + c);
            hw[o][0] = w.x; hw[o][1] = w.y; hw[o][2] = w.z; hw[o][3] = w.w;
          }
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float v = fmaxf(scaled<MODE>(acc[mb][r][4 * j + i], ws[i]) + bb[i], 0.f);
              hs[r][0] = fmaf(hw[0][i], v, hs[r][0]);
              hs[r][1] = fmaf(hw[1][i], v, hs[r][1]);
              hs[r][2] = fmaf(hw[2][i], v, hs[r][2]);
            }
        }
      }
    float *head_out = a.head_outs ? a.head_outs[img] : a.head_out + (size_t)img * 3 * HW;
    const float hb0 = s_head[96 * MB], hb1 = s_head[96 * MB + 1], hb2 = s_head[96 * MB + 2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int gy = gy0 + r;
      const float s0 = hs[r][0] + __shfl_xor(hs[r][0], 32, 64);
      const float s1 = hs[r][1] + __shfl_xor(hs[r][1], 32, 64);
      const float s2 = hs[r][2] + __shfl_xor(hs[r][2], 32, 64);
      if (h == 0 && gy < H && gx < W) {
        const size_t p = (size_t)gy * W + gx;
        head_out[p] = s0 + hb0;
        head_out[HW + p] = s1 + hb1;
        head_out[2 * HW + p] = s2 + hb2;
      }
    }
  } else {
    char *out = a.out + (size_t)img * a.out_bs;
    char *pool = a.out_pool ? a.out_pool + (size_t)img * a.pool_bs : nullptr;
    const size_t plane = HW * 16;
    uint32_t px[R];
    bool live[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      px[r] = ((uint32_t)(gy0 + r) * (uint32_t)W + (uint32_t)gx) * 16u;
      live[r] = gy0 + r < H && gx < W;
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (co0 + mb * 32 + 8 * j >= a.cout) continue;  // (cout is a multiple of 16: the same for both halves)
        const int c = co0 + mb * 32 + 8 * j + 4 * h;
        const float4 b = *reinterpret_cast<const float4 *>(s_bias + c - co0);
        const float bb[4] = {b.x, b.y, b.z, b.w};
        float ws[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (MODE == 4 || MODE == 5) {
          const float4 w4 = *reinterpret_cast<const float4 *>(s_ws + c - co0);
          ws[0] = w4.x; ws[1] = w4.y; ws[2] = w4.z; ws[3] = w4.w;
        }
        float v[R][4];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) v[r][i] = fmaxf(scaled<MODE>(acc[mb][r][4 * j + i], ws[i]) + bb[i], 0.f);
        const int cb = c - 4 * h;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (a.raw) {
            if (live[r]) put_raw<MODE>(out, plane, cb, h, px[r], v[r]);
          } else {
            put_operands<MODE>(out, plane, a.cout, cb, h, px[r], v[r], live[r]);
          }
        }
        if (pool) {
          // 2x2 maximum: rows r, r + 1 and the neighbouring lane's column
#pragma unroll
          for (int r = 0; r < R; r += 2) {
            float m[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              m[i] = fmaxf(v[r][i], v[r + 1][i]);
              m[i] = fmaxf(m[i], lane_xor1(m[i]));
            }
            put_operands<MODE>(pool, plane >> 2, a.cout, cb, h,
                               ((uint32_t)((gy0 + r) >> 1) * (uint32_t)(W >> 1) + (uint32_t)(gx >> 1)) * 16u, m,
                               (gx & 1) == 0 && live[r]);
          }
        }
      }
  }
}

// The convolution.  A workgroup of NW waves (NW / CW rows of waves, CW columns
// of waves over the channels) takes tiles of NW / CW * R rows x 32 columns of
// output pixels x 32 MB CW output channels; a wave owns R rows x 32 columns x
// 32 MB channels.  The 16-channel chunks of all its tiles form one stream: step
// t is multiplied from LDS while the input of step t + DI and the weights of
// step t + DW are loaded straight into the slots that step t - 1 left, with one
// barrier per step, so a tile's first chunks are on their way while the
// previous tile is finished.  Past the last step the loads are masked off, so
// every step counts the same.  Pixels outside the image are written as zeros,
// the loads leave them alone.
template <int MODE, int MB, int R, int NW, int CW, int DI, int DW, bool HEAD>
struct ConvLds {
  static constexpr int TH = NW / CW * R, CT = MB * CW;          // tile: rows, 32-channel tiles
  static constexpr int LW = 34, UB = (TH + 2) * LW;             // halo tile: units of a channel block
  static constexpr int NL = (UB + 63) / 64, UBP = NL * 64;      // in wave loads; padded
  static constexpr int INB = Fmt<MODE>::kBlocks * UBP * 16;     // bytes: a step's input
  static constexpr int WCH = Fmt<MODE>::kWUnits * 288 * 16;     // its weights per 32 channels
  static constexpr int WB = CT * WCH;
  static constexpr int kWeights = (DI + 1) * INB, kBias = kWeights + (DW + 1) * WB;
  // Two tiles' biases and weight scales.  A tile's are loaded DW steps before its
  // first step and read after its last one, while faster waves are in the next
  // step already: with DW = 1, two slots hold for tiles of two steps or more, for
  // runs of two tiles, or where every tile has the same ones (launch() sees to it).
  static constexpr int kHead = kBias + 2 * 2 * CT * 32 * 4;
  static constexpr int kBytes = kHead + (HEAD ? (3 * 32 * CT + 4) * 4 : 0);
  static constexpr int kWaves = NW == 8 || 2 * kBytes <= 160 * 1024 ? 2 : 1;  // per SIMD, as LDS has room
};
template <int MODE, int MB, int R, int NW, int CW, int DI, int DW, bool HEAD>
__global__ __launch_bounds__(64 * NW, (ConvLds<MODE, MB, R, NW, CW, DI, DW, HEAD>::kWaves)) void conv_kernel(Args a) {
  using S = ConvLds<MODE, MB, R, NW, CW, DI, DW, HEAD>;
  static_assert(!HEAD || CW == 1, "the head sums over all channels in one wave");
  static_assert(DI == DW || (DI == 2 && DW == 1), "the loads counted by wait_for");
  constexpr int CT = S::CT, TH = S::TH, LW = S::LW, NL = S::NL, UBP = S::UBP, WU = Fmt<MODE>::kWUnits;
  constexpr int NB = Fmt<MODE>::kBlocks, NK = (NL + NW - 1) / NW;                    // a wave's loads per channel block
  constexpr int NWU = CT * WU * 288, NKW = ((NWU + 63) / 64 + NW - 1) / NW;          // weight units; a wave's loads
  __shared__ __attribute__((aligned(16))) char sm[S::kBytes];

  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int wr = wv / CW, wc0 = (wv - wr * CW) * MB;  // this wave's rows [wr R, + R) and channel tiles [wc0, + MB)
  const int H = a.H, W = a.W;
  const uint32_t sm0 = lds_address(sm);
  const int nch = (a.C0 + a.C1) >> 4, nch0 = a.C0 >> 4;
  const Walk walk = my_tiles(a);
  if (walk.first >= walk.end) return;
  const int steps = (walk.end - walk.first) * nch;
  if constexpr (HEAD) {
    float *sh = reinterpret_cast<float *>(sm + S::kHead);
    for (int i = tid; i < 3 * 32 * MB; i += 64 * NW) {
      const int o = i / (32 * MB), c = i - o * (32 * MB);
      sh[i] = c < a.cout ? a.head_w[o * a.cout + c] : 0.f;
    }
    if (tid < 3) sh[96 * MB + tid] = a.head_b[tid];
  }

  // ---- weights of a step: wave load i = wv + NW k, 64 units each
  const bool resident = DW == 1 && nch <= 2 && a.ncz == 1;  // the two slots then hold every chunk
  const int wg = a.wgroup;                                  // 32-channel tiles per packed group
  const char *wptr = nullptr;
  int wT = walk.first, wc = 0, wtile = 0, wslot = 0;
  uint64_t wlanes = ~0ull;  // 0 past the last step (and where they are resident): masked loads keep the counts
  auto begin_weights = [&]() {
    if (wc != 0) return;
    if (wT >= walk.end || (resident && wtile * nch >= 2)) {
      wlanes = 0;
      return;
    }
    const int ct = __builtin_amdgcn_readfirstlane(wT % a.ncz) * CT;
    wptr = uniform(a.w + ((size_t)(wg == 2 ? ct >> 1 : ct) * nch * wg + (wg == 2 ? ct & 1 : 0)) * S::WCH + wv * 1024);
    if (wv == 0) {  // the tile's biases and weight scales
      const uint32_t db = sm0 + S::kBias + (wtile & 1) * (2 * CT * 32 * 4);
      constexpr uint64_t lanes = CT == 2 ? ~0ull : 0xFFFFFFFFull;
      load_lds4(a.bias + ct * 32, lane * 4, db, lanes);
      if constexpr (MODE == 4 || MODE == 5) load_lds4(a.wscale + ct * 32, lane * 4, db + CT * 32 * 4, lanes);
    }
  };
  auto issue_weights = [&](int k) {
    // units past the end: the load, or half of it, is masked
    uint64_t lanes = wlanes;
    if ((k + 1) * NW * 64 > NWU) {
      const int left = NWU - (wv + NW * k) * 64;
      lanes &= left >= 64 ? ~0ull : (left > 0 ? 0xFFFFFFFFull : 0ull);
    }
    load_lds16(wptr + k * NW * 1024, lane * 16, sm0 + S::kWeights + wslot * S::WB + wv * 1024 + k * NW * 1024, lanes);
  };
  auto end_weights = [&]() {
    wptr += wg * S::WCH;
    wslot = wslot == DW ? 0 : wslot + 1;
    if (++wc == nch) {
      wc = 0;
      ++wtile;
      ++wT;
    }
  };

  // ---- input: in every channel block, wave load j = wv + NW k covers units j 64 + lane
  int urow[NK], ucol[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int pos = (wv + NW * k) * 64 + lane;
    urow[k] = pos / LW;
    ucol[k] = pos - urow[k] * LW;
  }
  int iT = walk.first, ic = 0;
  int iy0 = 0, ix0 = 0, iimg = 0;
  uint32_t voff[NK];
  uint64_t lanes[NK];
  uint32_t outside = 0;  // bit k: this lane's unit of load k lies outside the image
  bool border = false;
  const char *src = nullptr;  // the chunk's first channel block, at the tile's first halo row
  size_t blk = 0, pln = 0;    // bytes per channel block and from the hi to the lo plane of the current source
  auto set_source = [&](bool second) {
    const int sh = second ? 1 : 0, Ws = W >> sh, y0 = (iy0 - 1) >> sh;
    const char *in = second ? a.in1 + (size_t)iimg * a.in1_bs : a.in0 + (size_t)iimg * a.in0_bs;
    blk = (size_t)(H >> sh) * Ws * 16;
    pln = (size_t)((second ? a.C1 : a.C0) >> 3) * blk;
    src = uniform(in + (ptrdiff_t)y0 * Ws * 16);
#pragma unroll
    for (int k = 0; k < NK; ++k)  // (unused outside the image)
      voff[k] = (uint32_t)((((iy0 - 1 + urow[k]) >> sh) - y0) * Ws + ((ix0 - 1 + ucol[k]) >> sh)) * 16u;
  };
  int islot = 0;
  auto begin_input = [&]() {
    if (ic == 0 && iT >= walk.end) {
#pragma unroll
      for (int k = 0; k < NK; ++k) lanes[k] = 0;
      border = false;
    } else if (ic == 0) {
      const Tile t = tile_at(a, iT);
      iy0 = t.ty * TH;
      ix0 = t.tx * 32;
      iimg = t.img;
      outside = 0;
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const bool any = urow[k] < TH + 2;
        const bool in = ((unsigned)(iy0 - 1 + urow[k]) < (unsigned)H) & ((unsigned)(ix0 - 1 + ucol[k]) < (unsigned)W);
        lanes[k] = __ballot(any & in);
        outside |= (any & !in) ? 1u << k : 0u;
      }
      border = __ballot(outside != 0) != 0;
    }
    if (ic == 0 || ic == nch0) set_source(ic != 0);
  };
  auto issue_input = [&](int j) {
    const int b = j / NK, k = j % NK;
    load_lds16(src + (b & 1) * blk + (MODE == 2 && b >= 2 ? pln : 0), voff[k],
               sm0 + islot * S::INB + wv * 1024 + b * UBP * 16 + k * NW * 1024, lanes[k]);
  };
  auto end_input = [&]() {
    if (border) {
#pragma unroll
      for (int k = 0; k < NK; ++k)
        if ((outside >> k) & 1u) {
#pragma unroll
          for (int b = 0; b < NB; ++b)
            *reinterpret_cast<uint4 *>(sm + islot * S::INB + wv * 1024 + b * UBP * 16 + k * NW * 1024 + lane * 16) =
                make_uint4(0u, 0u, 0u, 0u);
        }
    }
    src += (MODE == 4 ? 1 : 2) * blk;
    islot = islot == DI ? 0 : islot + 1;
    if (++ic == nch) {
      ic = 0;
      ++iT;
    }
  };

  floatx16 acc[MB][R];
  auto zero_acc = [&]() {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[mb][r][q] = 0.f;
  };
  zero_acc();
  const char *A = sm + S::kWeights + wc0 * S::WCH + lane_a<MODE>(n, h);
  const char *B = sm + lane_b<MODE, UBP>(wr * R * LW + n, h);
  constexpr int NI = NB * NK;  // a wave's input loads per step
  auto load_weights = [&]() {
    begin_weights();
#pragma unroll
    for (int k = 0; k < NKW; ++k) issue_weights(k);
    end_weights();
  };
  auto load_input = [&]() {
    begin_input();
#pragma unroll
    for (int j = 0; j < NI; ++j) issue_input(j);
    end_input();
  };
#pragma unroll
  for (int d = 0; d < DI; ++d) {
    if (d >= steps) continue;
    if (d < DW) load_weights();
    load_input();
  }
  // Before a step: its loads are done, while newer ones may be in flight: with
  // DI = 2 and DW = 1 the input of the next step, with DI = DW = D the weights and
  // the input of D - 1 steps.  (Waiting before the epilogue keeps its stores
  // out of the count; the loads of a tile's biases only make it stricter.)
  constexpr int kNewer = DI == DW ? (DI - 1) * (NKW + NI) : NI;
  static_assert(kNewer < 64, "vmcnt has six bits");
  if (steps >= DI) wait_loads<kNewer>();
  else wait_loads<0>();
  __syncthreads();
  int T = walk.first, tile = 0, c = 0, in_slot = 0, w_slot = 0;
  for (int t = 0; t < steps; ++t) {
    const char *At = A + w_slot * S::WB, *Bt = B + in_slot * S::INB;
    chunk_mma<MODE, MB, R, UBP, LW, NKW + NI, true>(At, Bt, acc, [&](int i) {
      if (i < 0) begin_weights(), begin_input();
      else if (i < NKW) issue_weights(i);
      else issue_input(i - NKW);
    });
    end_weights();
    end_input();
    wait_loads<kNewer>();
    __syncthreads();
    in_slot = in_slot == DI ? 0 : in_slot + 1;
    w_slot = w_slot == DW ? 0 : w_slot + 1;
    if (++c == nch) {
      const Tile d = tile_at(a, T);
      const float *sb = reinterpret_cast<const float *>(sm + S::kBias) + ((resident ? 0 : tile) & 1) * (2 * CT * 32) + wc0 * 32;
      epilogue<MODE, MB, R, HEAD>(a, d.img, (d.cz * CT + wc0) * 32, d.ty * TH + wr * R, d.tx * 32 + n, h, acc, sb,
                                  sb + CT * 32, reinterpret_cast<const float *>(sm + S::kHead));
      zero_acc();
      c = 0;
      ++tile;
      ++T;
    }
  }
}

// The network's first layer by itself (first levels that enc0_kernel does not
// take): one chunk, whose operands are computed from the RGBDA image.
template <int MODE, int MB, int R, int NW>
__global__ __launch_bounds__(64 * NW, 2) void first_kernel(Args a) {
  constexpr int NT = 64 * NW, TH = NW * R, LW = 34, UB = (TH + 2) * LW, UBP = (UB + 63) / 64 * 64;
  constexpr int WU = Fmt<MODE>::kWUnits, INB = Fmt<MODE>::kBlocks * UBP * 16, NV = MB * WU * 288;
  __shared__ __attribute__((aligned(16))) char sm[INB + NV * 16];
  __shared__ __attribute__((aligned(16))) float s_bias[2 * MB * 32];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const Walk walk = my_tiles(a);
  if (walk.first >= walk.end) return;
  const Tile t = tile_at(a, walk.first);
  const int ty0 = t.ty * TH, tx0 = t.tx * 32, co0 = t.cz * 32 * MB;
  const int H = a.H, W = a.W;
  // (one chunk: the channel tiles' weights follow each other, whatever the groups)
  const uint4 *wsrc = reinterpret_cast<const uint4 *>(a.w) + (size_t)(co0 >> 5) * WU * 288;
  uint4 *sw = reinterpret_cast<uint4 *>(sm + INB);
  for (int i = tid; i < NV; i += NT) sw[i] = wsrc[i];
  if (tid < MB * 32) {
    s_bias[tid] = a.bias[co0 + tid];
    s_bias[MB * 32 + tid] = (MODE == 4 || MODE == 5) ? a.wscale[co0 + tid] : 1.f;
  }
  const float *depth = a.depth + (size_t)t.img * a.rgbda_bs;
  const uint32_t *rgba = a.rgba + (size_t)t.img * a.rgbda_bs;
  constexpr int NP = (UB + NT - 1) / NT;
  uint32_t q[NP], inside = 0;
  float d[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int pos = tid + k * NT, row = pos / LW, col = pos - row * LW;
    const int gy = ty0 - 1 + row, gx = tx0 - 1 + col;
    const bool in = pos < UB && gy >= 0 && gy < H && gx >= 0 && gx < W;
    const size_t p = in ? (size_t)gy * W + gx : 0;
    q[k] = rgba[p];
    d[k] = depth[p];
    if (in) inside |= 1u << k;
  }
  const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int pos = tid + k * NT;
    if (pos >= UB) continue;
    uint4 u[2] = {zero, zero};
    if ((inside >> k) & 1u) input_units<MODE>(q[k], d[k], u);
    uint4 *s = reinterpret_cast<uint4 *>(sm) + pos;
    s[0] = u[0];
    if constexpr (MODE == 2) {
      s[UBP] = zero;
      s[2 * UBP] = u[1];
      s[3 * UBP] = zero;
    } else if constexpr (MODE != 4) {
      s[UBP] = zero;  // channels 8..15
    }
  }
  floatx16 acc[MB][R];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[mb][r][k] = 0.f;
  __syncthreads();
  const char *A = sm + INB + lane_a<MODE>(n, h), *B = sm + lane_b<MODE, UBP>(wv * R * LW + n, h);
  chunk_mma<MODE, MB, R, UBP, LW, 0, false>(A, B, acc, [](int) {});
  epilogue<MODE, MB, R, false>(a, t.img, co0, ty0 + wv * R, tx0 + n, h, acc, s_bias, s_bias + MB * 32, nullptr);
}

// The network's first two convolutions in one kernel (first level of 16 or 32
// channels).  An output tile of NW R rows x 32 columns x 32 channels of the
// second convolution needs the first one's output on a region one pixel wider
// on every side, which needs the network input one pixel wider still.  Phase 1
// computes the first convolution on the region (linear blocks of 32 of its
// pixels, the layer's weight fragments in registers) from the input's operand
// units in LDS and leaves it in LDS as the second layer's operands, zero where
// a region pixel lies outside the image (the second layer's padding).  Phase 2
// is the generic kernel's chunk loop on it.  Workgroups are persistent: both
// layers' weights are loaded once, and the next tile's RGBDA pixels are loaded
// during phase 1 and turned into operands after phase 2.  The first layer's
// output never goes to memory; its sums are the unfused launches', so the
// outputs are bit-identical to theirs.
template <int MODE, int CK1, int R, int NW>
struct Enc0Lds {
  static constexpr int XW = 36, XPix = (NW * R + 4) * XW;       // network input region
  static constexpr int LW = 34, MPix = (NW * R + 2) * LW;       // first layer's output region
  static constexpr int UBP = (MPix + 63) / 64 * 64;
  static constexpr int NCH = CK1 / 16, WCH = Fmt<MODE>::kWUnits * 288 * 16;
  // region operands of every chunk | second-layer weights | input units (plane
  // after plane) | zeros, read by the lanes of channels 8..15 | biases, scales
  static constexpr int kW1 = NCH * Fmt<MODE>::kBlocks * UBP * 16, kX = kW1 + NCH * WCH;
  static constexpr int kZ = kX + Fmt<MODE>::kPlanes * XPix * 16, ZB = (2 * XW + 3) * 16;
  static constexpr int kBias = kZ + ZB, kBytes = kBias + 4 * 32 * 4;
};
template <int MODE, int CK1, int R, int NW>
__global__ __launch_bounds__(64 * NW, 2) void enc0_kernel(Args a0, Args a1) {
  using F = typename FragOf<MODE>::type;
  using S = Enc0Lds<MODE, CK1, R, NW>;
  constexpr int NT = 64 * NW, TH = NW * R, XW = S::XW, XPix = S::XPix, LW = S::LW, MPix = S::MPix, UBP = S::UBP;
  constexpr int P = Fmt<MODE>::kPlanes, WU = Fmt<MODE>::kWUnits, NB = Fmt<MODE>::kBlocks;
  __shared__ __attribute__((aligned(16))) char sm[S::kBytes];
  char *s_w1 = sm + S::kW1, *s_x = sm + S::kX, *s_z = sm + S::kZ;
  float *s_bias = reinterpret_cast<float *>(sm + S::kBias);  // layer 0 biases, scales, layer 1 biases, scales

  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int H = a1.H, W = a1.W;
  const Walk walk = my_tiles(a1);
  if (walk.first >= walk.end) return;

  // RGBDA pixels of a tile's input region -> registers -> operand units in LDS
  constexpr int NP = (XPix + NT - 1) / NT;
  uint32_t q[NP], inside = 0;
  float d[NP];
  auto fetch = [&](int T) {
    const Tile t = tile_at(a1, T);
    const float *depth = a0.depth + (size_t)t.img * a0.rgbda_bs;
    const uint32_t *rgba = a0.rgba + (size_t)t.img * a0.rgbda_bs;
    inside = 0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int pos = tid + k * NT, row = pos / XW, col = pos - row * XW;
      const int gy = t.ty * TH - 2 + row, gx = t.tx * 32 - 2 + col;
      const bool in = pos < XPix && gy >= 0 && gy < H && gx >= 0 && gx < W;
      const size_t p = in ? (size_t)gy * W + gx : 0;
      q[k] = rgba[p];
      d[k] = depth[p];
      if (in) inside |= 1u << k;
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int pos = tid + k * NT;
      if (pos >= XPix) continue;
      uint4 u[2] = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u)};
      if ((inside >> k) & 1u) input_units<MODE>(q[k], d[k], u);
#pragma unroll
      for (int p = 0; p < P; ++p) reinterpret_cast<uint4 *>(s_x)[p * XPix + pos] = u[p];
    }
  };
  fetch(walk.first);
  // first-layer weight fragments of this lane; everything else of the weights to LDS
  F w0[9][P];
#pragma unroll
  for (int tap = 0; tap < 9; ++tap)
#pragma unroll
    for (int p = 0; p < P; ++p)
      w0[tap][p] = *reinterpret_cast<const F *>(a0.w + (p * 9 + tap) * (WU / P) * 512 + lane_a<MODE>(n, h));
  for (int i = tid; i < S::NCH * WU * 288; i += NT)
    reinterpret_cast<uint4 *>(s_w1)[i] = reinterpret_cast<const uint4 *>(a1.w)[i];
  if (tid < 32) {
    s_bias[tid] = a0.bias[tid];
    s_bias[64 + tid] = a1.bias[tid];
    s_bias[32 + tid] = (MODE == 4 || MODE == 5) ? a0.wscale[tid] : 1.f;
    s_bias[96 + tid] = (MODE == 4 || MODE == 5) ? a1.wscale[tid] : 1.f;
  }
  for (int i = tid; i < S::ZB / 16; i += NT) reinterpret_cast<uint4 *>(s_z)[i] = make_uint4(0u, 0u, 0u, 0u);
  stage();
  __syncthreads();

  for (int T = walk.first; T < walk.end; ++T) {
    const Tile t = tile_at(a1, T);
    const int ty0 = t.ty * TH, tx0 = t.tx * 32;
    const bool more = T + 1 < walk.end;
    if (more) fetch(T + 1);

    // ---- phase 1: wave w takes pixel blocks w, w + NW, ... of the region
#pragma unroll 1
    for (int blk = wv; blk * 32 < MPix; blk += NW) {
      const int m = blk * 32 + n;
      const bool live = m < MPix;
      const int mr = live ? m / LW : 0, mc = live ? m - mr * LW : 0;
      floatx16 acc;
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[k] = 0.f;
      // channels 8..15 of the network input are zero (lanes h = 1; the e4m3 unit holds them itself)
      const char *B = s_x + (mr * XW + mc) * 16 + (MODE == 4 ? 8 * h : 0);
      if (MODE != 4 && h) B = s_z;
      const int plane = (MODE != 4 && h) ? 0 : XPix * 16;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          F b[P];
#pragma unroll
          for (int p = 0; p < P; ++p) b[p] = *reinterpret_cast<const F *>(B + p * plane + (dy * XW + dx) * 16);
          mma<MODE>(w0[dy * 3 + dx], b, acc);
        }
      const int gy = ty0 - 1 + mr, gx = tx0 - 1 + mc;
      const bool inimg = gy >= 0 && gy < H && gx >= 0 && gx < W;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (8 * j >= CK1) continue;
        const int c = 8 * j + 4 * h;
        const float4 b = *reinterpret_cast<const float4 *>(s_bias + c);
        float4 ws = make_float4(1.f, 1.f, 1.f, 1.f);
        if constexpr (MODE == 4 || MODE == 5) ws = *reinterpret_cast<const float4 *>(s_bias + 32 + c);
        const float v0 = fmaxf(scaled<MODE>(acc[4 * j + 0], ws.x) + b.x, 0.f);
        const float v1 = fmaxf(scaled<MODE>(acc[4 * j + 1], ws.y) + b.y, 0.f);
        const float v2 = fmaxf(scaled<MODE>(acc[4 * j + 2], ws.z) + b.z, 0.f);
        const float v3 = fmaxf(scaled<MODE>(acc[4 * j + 3], ws.w) + b.w, 0.f);
        // as put_operands, into the chunk's blocks in LDS; zero outside the image
        const uint32_t keep = inimg ? ~0u : 0u;
        const uint32_t p01 = pack16x2<MODE>(v0, v1), p23 = pack16x2<MODE>(v2, v3);
        char *u = sm + (((j >> 1) * NB + (MODE == 4 ? 0 : (j & 1))) * UBP + m) * 16;
        if (live) {
          if constexpr (MODE == 1 || MODE == 3) {
            *reinterpret_cast<uint2 *>(u + 8 * h) = make_uint2(p01 & keep, p23 & keep);
          } else if constexpr (MODE == 2) {
            *reinterpret_cast<uint2 *>(u + 8 * h) = make_uint2(p01 & keep, p23 & keep);
            *reinterpret_cast<uint2 *>(u + 2 * UBP * 16 + 8 * h) =
                make_uint2(rest_bf16x2(v0, v1, p01) & keep, rest_bf16x2(v2, v3, p23) & keep);
          } else if constexpr (MODE == 5) {
            *reinterpret_cast<uint32_t *>(u + 4 * h) = e4m3x4<false>(p01, p23) & keep;
            *reinterpret_cast<uint32_t *>(u + 8 + 4 * h) = e4m3x4<true>(p01, p23) & keep;
          } else {
            *reinterpret_cast<uint32_t *>(u + 8 * (j & 1) + 4 * h) = e4m3x4<false>(p01, p23) & keep;
          }
        }
      }
    }
    __syncthreads();

    // ---- phase 2
    floatx16 acc[1][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[0][r][k] = 0.f;
#pragma unroll
    for (int c = 0; c < S::NCH; ++c) {
      const char *A = s_w1 + c * S::WCH + lane_a<MODE>(n, h);
      const char *B = sm + c * NB * UBP * 16 + lane_b<MODE, UBP>(wv * R * LW + n, h);
      chunk_mma<MODE, 1, R, UBP, LW, 0, true>(A, B, acc, [](int) {});
    }
    if (more) stage();
    epilogue<MODE, 1, R, false>(a1, t.img, 0, ty0 + wv * R, tx0 + n, h, acc, s_bias + 64, s_bias + 96, nullptr);
    __syncthreads();
  }
}

// 1x1 head of a layer too wide to fuse it: float32 weights [3][C], one thread
// per pixel, planar float32 output.  x: blocks of 8 16-bit channels (MODE 1, 3)
// or 4 float32 channels (MODE 2, and the float32 network).  Bound by the pixels'
// loads: U of them in flight per thread.  Four (16 channels) hide their latency
// where one leaves it open (192 channels, us with one / four: fp16 64 x 64 14.9 /
// 8.4, 1280 x 720 82.8 / 70.8; float32 64 x 64 16.9 / 8.7, 256 x 256 17.9 / 10.7);
// float32 pixels, whole cache lines each, are read at full rate by four waves per
// SIMD and more, and one then keeps the accesses in order (640 x 480 43.4 / 40.8,
// 800 x 600 66.5 / 72.5, 1920 x 1080 289 / 300).  The sums' order is the same.
template <int MODE, int U>
__global__ __launch_bounds__(256) void head_kernel(const char *__restrict__ x, int C, size_t npix,
                                                   const float *__restrict__ w, const float *__restrict__ b,
                                                   float *__restrict__ out) {
  const size_t p = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= npix) return;
  float y0 = b[0], y1 = b[1], y2 = b[2];
#pragma unroll U
  for (int c = 0; c < C; c += 4) {
    float v[4];
    if constexpr (MODE == 2) {
      const float4 q = *reinterpret_cast<const float4 *>(x + ((size_t)(c >> 2) * npix + p) * 16);
      v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
      const uint2 q = *reinterpret_cast<const uint2 *>(x + ((size_t)(c >> 3) * npix + p) * 16 + 2 * (c & 4));
      const uint32_t u[4] = {q.x & 0xFFFFu, q.x >> 16, q.y & 0xFFFFu, q.y >> 16};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[i] = MODE == 1 ? __uint_as_float(u[i] << 16) : (float)__builtin_bit_cast(_Float16, (uint16_t)u[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      y0 = fmaf(w[c + i], v[i], y0);
      y1 = fmaf(w[C + c + i], v[i], y1);
      y2 = fmaf(w[2 * C + c + i], v[i], y2);
    }
  }
  out[p] = y0;
  out[npix + p] = y1;
  out[2 * npix + p] = y2;
}

template <int MODE, int MB, int R, int NW, int CW, int DI, int DW>
hipError_t launch(const ConvCall &c, hipStream_t s) {
  using S = ConvLds<MODE, MB, R, NW, CW, DI, DW, false>;
  Args a = make_args(c);
  const int batch = c.batch < 1 ? 1 : c.batch;
  int run = 1;
  if (MB == 1 && CW == 1 && DW == 1) {
    // long runs of tiles where there are many more than the chip takes at once
    // (narrow layers, bound by memory: 430 -> 397 us for the widest at 4K)
    set_tiles(a, S::TH, 32 * S::CT, c.layer->cout_pad, batch, 1);
    run = a.ntiles / (2 * kCUs * (8 / NW));
    run = run < 1 ? 1 : (run > 8 ? 8 : run);
    // tiles of one step and different channels: runs of two (the bias slots)
    if (a.C0 + a.C1 == 16 && a.ncz > 1) run = run < 2 ? run : 2;
  }
  const int grid = set_tiles(a, S::TH, 32 * S::CT, c.layer->cout_pad, batch, run);
  if (c.head_out || c.head_outs) {
    if constexpr (CW == 1)
      conv_kernel<MODE, MB, R, NW, CW, DI, DW, true><<<grid, 64 * NW, 0, s>>>(a);
    else
      return hipErrorInvalidValue;
  } else {
    conv_kernel<MODE, MB, R, NW, CW, DI, DW, false><<<grid, 64 * NW, 0, s>>>(a);
  }
  return hipGetLastError();
}

template <int MODE>
hipError_t first_launch(const ConvCall &c, hipStream_t s) {
  Args a = make_args(c);
  const int batch = c.batch < 1 ? 1 : c.batch;
  constexpr int R = 2, NW = 4;
  if (c.layer->cout_pad % 64 == 0)
    first_kernel<MODE, 2, R, NW><<<set_tiles(a, R * NW, 64, c.layer->cout_pad, batch, 1), 64 * NW, 0, s>>>(a);
  else
    first_kernel<MODE, 1, R, NW><<<set_tiles(a, R * NW, 32, c.layer->cout_pad, batch, 1), 64 * NW, 0, s>>>(a);
  return hipGetLastError();
}

// Tiles of a layer per CU, a fraction of a round counted as a whole one while
// there are few rounds.
inline double rounds(const ConvCall &c, int rows, int channels) {
  const double t = (double)((c.W + 31) / 32) * ((c.H + rows - 1) / rows) * (c.layer->cout_pad / channels) *
                   (c.batch < 1 ? 1 : c.batch) / kCUs;
  return t > 6 ? t + 0.5 : std::ceil(t);
}
// Tile choice by the estimated time: tiles per CU times a tile's time (in units
// of 64 channels x 8 rows at full rate; a workgroup alone on its CU runs at two
// thirds of the rate of a pair).  Large layers take the tile with the most
// matrix instructions per fragment read, 64 channels x 16 rows (two rows of
// fragments more for four rows of output); halving the rows pays where that
// fills the chip (135 x 240 x 256 channels: 31.0 / 53.2 against 33.6 / 58.2
// us), and 32 channels x 8 rows, two steps in flight, where even that leaves
// CUs idle (60 x 80 x 256 channels: 12.4 / 19.8 against 15.6 / 25.1 us).  Split
// bfloat16 reads both planes: its 64 x 16 and 64 x 8 tiles take 8 waves and a CU
// each, for 2.0 and 1.1 units of time; 64 to 512 channels, us with 16 and with 8 rows:
//   0.5 rounds of 16 rows (1 of 8)  256 x 256 x 64 channels     43.0 / 31.5
//   1.0 (2)                         128 x 128 x 512             69.1 / 78.4
//   1.25 (3)                        120 x 160 x 512            111.5 / 97.2
//   2.3 (5)                         480 x 640 x 64             120.3 / 116.9
//   2.7 (6)                         360 x 480 x 128             80.1 / 87.9
//   7 (14), no longer counted whole 720 x 1280 x 64            331.9 / 363.8
// (of 168 layers, 0.02 to 16 rounds, the choice was the faster one in all but one,
// 64.0 / 63.1).  Layers of an odd number of 32-channel tiles take tiles of 32
// channels x 16 rows where those are fewer rounds by the ratio of the two tiles'
// times, which grows with the matrix work per byte; split bfloat16's are 8 waves
// and 4, a CU each.  96 output channels of 16-channel steps, us with 16 / 8 rows
// (32 -> 96 channels; rounds of 16 rows):
//            60 x 80 (0.2)   150 x 200 (0.8)  240 x 320 (1.8)  540 x 960 (12)
//   fp16       8.4 / 7.4        9.4 / 9.6       12.4 / 14.8      49.2 / 65.0
//   fp8        9.2 / 7.8        9.9 / 9.5       12.3 / 12.4      36.6 / 46.3
//   fp8x3     12.5 / 9.5       13.8 / 12.6      19.4 / 20.4      81.0 / 92.1
//   bf16x3    11.8 / 9.4       13.8 / 16.9      22.4 / 29.2     117.6 / 134.7
// (308 layers each, 64 x 64 to 2560 x 1440, against the faster of the two: always
// 16 rows 5, 6, 11 and 6% slower, always 8 rows 10, 6, 3 and 13%, the choice under
// 1%).  Any choice gives the same results.
template <int MODE>
hipError_t dispatch(const ConvCall &c, hipStream_t s) {
  const bool wide = c.layer->cout_pad % 64 == 0;
  const bool head = c.head_out || c.head_outs;
  if constexpr (MODE == 2) {
    if (!wide)
      return rounds(c, 16, 32) * 1.3 <= rounds(c, 8, 32) ? launch<MODE, 1, 2, 8, 1, 1, 1>(c, s)
                                                         : launch<MODE, 1, 2, 4, 1, 1, 1>(c, s);
    if (!head && rounds(c, 16, 64) * 2.0 > rounds(c, 8, 64) * 1.1) return launch<MODE, 1, 2, 8, 2, 1, 1>(c, s);
    return launch<MODE, 2, 2, 8, 1, 1, 1>(c, s);
  } else {
    auto cost = [&](int rows, int channels, double tile) {
      const double k = rounds(c, rows, channels);
      return (k == 1 ? 1.5 : k) * tile;
    };
    if (wide) {
      const double t64x16 = cost(16, 64, 2.0), t64x8 = cost(8, 64, 1.08), t32x8 = head ? 1e30 : cost(8, 32, 0.8);
      if (t64x16 <= t64x8 && t64x16 <= t32x8) return launch<MODE, 2, 4, 4, 1, 1, 1>(c, s);
      return t64x8 <= t32x8 ? launch<MODE, 2, 2, 4, 1, 1, 1>(c, s) : launch<MODE, 1, 2, 4, 1, 2, 2>(c, s);
    }
    constexpr double t32x16 = MODE == 5 ? 1.8 : (MODE == 4 ? 1.6 : 1.5);
    return cost(16, 32, t32x16) <= cost(8, 32, 1.0) ? launch<MODE, 1, 4, 4, 1, 2, 1>(c, s)
                                                     : launch<MODE, 1, 2, 4, 1, 2, 2>(c, s);
  }
}

template <int MODE, int CK1>
hipError_t enc0_launch_c(const ConvCall &c0, const ConvCall &c1, hipStream_t s) {
  constexpr int R = MODE == 2 ? 2 : 4, NW = MODE == 2 ? 8 : 4;
  const Args a0 = make_args(c0);
  Args a1 = make_args(c1);
  const int batch = c1.batch < 1 ? 1 : c1.batch;
  set_tiles(a1, NW * R, 32, 32, batch, 1);
  const int run = a1.ntiles / (2 * kCUs * (8 / NW));
  const int grid = set_tiles(a1, NW * R, 32, 32, batch, run < 1 ? 1 : (run > 8 ? 8 : run));
  enc0_kernel<MODE, CK1, R, NW><<<grid, 64 * NW, 0, s>>>(a0, a1);
  return hipGetLastError();
}
template <int MODE>
hipError_t enc0_launch(const ConvCall &c0, const ConvCall &c1, hipStream_t s) {
  return c1.layer->cin_pad == 32 ? enc0_launch_c<MODE, 32>(c0, c1, s) : enc0_launch_c<MODE, 16>(c0, c1, s);
}

}  // namespace

hipError_t launch_conv16(const ConvCall &c, Prec p, hipStream_t s) {
  const ConvLayer &L = *c.layer;
  const bool head = c.head_out || c.head_outs;
  if (head && (L.cout_pad > 64 || c.out_pool || c.raw_out)) return hipErrorInvalidValue;
  if (c.rgbda_depth ? (!c.rgbda_rgba || c.C1 != 0 || L.cin_pad != 16)
                    : (c.C0 % 16 || c.C1 % 16 || c.C0 + c.C1 != L.cin_pad))
    return hipErrorInvalidValue;
  if (c.C1 && (c.H % 2 || c.W % 2)) return hipErrorInvalidValue;
  if (c.out_pool && (c.H % 2 || c.W % 2)) return hipErrorInvalidValue;
  switch (p) {
    case Prec::BF16: return c.rgbda_depth ? first_launch<1>(c, s) : dispatch<1>(c, s);
    case Prec::BF16X3: return c.rgbda_depth ? first_launch<2>(c, s) : dispatch<2>(c, s);
    case Prec::FP16: return c.rgbda_depth ? first_launch<3>(c, s) : dispatch<3>(c, s);
    case Prec::FP8:
      if (!L.wscale) return hipErrorInvalidValue;
      return c.rgbda_depth ? first_launch<4>(c, s) : dispatch<4>(c, s);
    case Prec::FP8X3:
      if (!L.wscale) return hipErrorInvalidValue;
      return c.rgbda_depth ? first_launch<5>(c, s) : dispatch<5>(c, s);
    default: return hipErrorInvalidValue;
  }
}

bool enc0_fusable(const ConvLayer &l0, const ConvLayer &l1, Prec p) {
  return p != Prec::F32 && l0.cin_pad == 16 && l0.cout_pad == 32 && l1.cout_pad == 32 && l1.cin == l0.cout &&
         l1.cin_pad == l1.cin && (l1.cin_pad == 16 || l1.cin_pad == 32);
}

hipError_t launch_enc0(const ConvCall &c0, const ConvCall &c1, Prec p, hipStream_t s) {
  const ConvLayer &L0 = *c0.layer, &L1 = *c1.layer;
  if (!enc0_fusable(L0, L1, p) || !c1.out || !c1.out_pool || c1.raw_out || c1.head_out || c1.head_outs || c1.C1 ||
      c0.H != c1.H || c0.W != c1.W || c0.batch != c1.batch || !c0.rgbda_depth || !c0.rgbda_rgba ||
      c1.C0 != L1.cin_pad || c1.H % 2 || c1.W % 2)
    return hipErrorInvalidValue;
  switch (p) {
    case Prec::BF16: return enc0_launch<1>(c0, c1, s);
    case Prec::BF16X3: return enc0_launch<2>(c0, c1, s);
    case Prec::FP16: return enc0_launch<3>(c0, c1, s);
    case Prec::FP8: return enc0_launch<4>(c0, c1, s);
    case Prec::FP8X3: return enc0_launch<5>(c0, c1, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_head16(const void *x, int C, int H, int W, const ConvLayer &head, Prec p, float *out,
                         hipStream_t s) {
  const size_t npix = (size_t)H * W;
  const unsigned nb = (unsigned)((npix + 255) / 256);
  const float *w = static_cast<const float *>(head.w);
  const char *xc = static_cast<const char *>(x);
  if (p == Prec::BF16)
    head_kernel<1, 4><<<nb, 256, 0, s>>>(xc, C, npix, w, head.bias, out);
  else if ((p == Prec::BF16X3 || p == Prec::F32) && nb <= 5 * kCUs)  // float32 activations
    head_kernel<2, 4><<<nb, 256, 0, s>>>(xc, C, npix, w, head.bias, out);
  else if (p == Prec::BF16X3 || p == Prec::F32)
    head_kernel<2, 1><<<nb, 256, 0, s>>>(xc, C, npix, w, head.bias, out);
  else
    head_kernel<3, 4><<<nb, 256, 0, s>>>(xc, C, npix, w, head.bias, out);
  return hipGetLastError();
}

}  // namespace lnr
