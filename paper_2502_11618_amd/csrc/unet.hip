// Float32 U-Net convolutions on the gfx950 matrix cores.
//
// Fig. 1 and Method, "U-Net Reconstruction": a fully convolutional U-Net maps
// the depth-filtered RGBDA image to RGB.  The network's first layer is an
// implicit GEMM (M = output channels, N = output pixels, K = 9 taps x input
// channels) on v_mfma_f32_32x32x2_f32 that reads the RGBDA image itself; every
// other layer runs as Winograd F(2x2, 3x3).  The decoder's nearest-neighbour
// upsample and channel concatenation are folded into the input staging
// (channels past the skip tensor are read from the coarser tensor at
// (y/2, x/2)), the encoder's 2x2 max-pool into the epilogue of the convolution
// that feeds it, and the 1x1 head into the epilogue of the last convolution.
// (The reduced-precision networks are in conv16.hip.)
#include <hip/hip_runtime.h>

#include <atomic>

#include "lnr_internal.h"

namespace lnr {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

struct ConvArgs {
  const void *in0;
  const void *in1;
  int C0, C1, H, W;
  const void *w;
  const float *bias;
  int cout, cin_pad;
  void *out;
  void *out_pool;
  const float *head_w;
  const float *head_b;
  float *head_out;
  // batch of same-shape images: per-image strides of the tensors above in
  // elements; head_outs (device array) gives each image's planar head output
  // when set; the RGBDA images are rgbda_bs pixels apart
  int batch;
  size_t in0_bs, in1_bs, out_bs, pool_bs;
  float *const *head_outs;
  const float *rgbda_depth;
  const uint32_t *rgbda_rgba;
  size_t rgbda_bs;
  const float *wu;  // Winograd-domain weights [cout_pad][16][cin_pad], or null
};

// The network's first 3x3 convolution as implicit GEMM (M = output channels,
// N = pixels, K = 9 taps x 8 staged channels), one chunk, read from the RGBDA
// image.  Workgroup tile: 4R rows x 32 columns of output pixels x BM output
// channels; wave w owns rows [wR, wR + R).  The input tile with its halo and
// the weights ([co][tap][8]) sit in LDS.  For one horizontal tap offset dx a
// wave reads R + 2 input-row fragments and 3 MB weight fragments and feeds
// every input row to the up-to-three vertical taps that use it.  The five
// input channels are staged as (x0, x1, x2, 0 | x3, x4, 0, 0): k-step s pairs
// channel s with channel 4 + s, so the fourth step is zero and skipped.
template <int BM, int R>
__global__ __launch_bounds__(256) void first3x3_kernel(ConvArgs a) {
  constexpr int CK = 8, S = CK + 4;          // LDS floats per staged pixel / weight row
  constexpr int MB = BM / 32;
  constexpr int TH = 4 * R, TW = 32;
  constexpr int LW = TW + 2, LPix = (TH + 2) * LW;
  constexpr int NIN = (LPix + 255) / 256;
  constexpr int WROWS = 9 * BM, NWR = (WROWS * 2 + 255) / 256;
  __shared__ __attribute__((aligned(16))) float s_in[LPix * S];
  __shared__ __attribute__((aligned(16))) float s_w[WROWS * S];

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 31, h = lane >> 5;
  const int ty0 = blockIdx.y * TH, tx0 = blockIdx.x * TW;
  const int nzc = gridDim.z / a.batch;
  const int bimg = blockIdx.z / nzc;
  const int co0 = (blockIdx.z - bimg * nzc) * BM;
  const int H = a.H, W = a.W;
  const float *depth = a.rgbda_depth + (size_t)bimg * a.rgbda_bs;
  const uint32_t *rgba = a.rgbda_rgba + (size_t)bimg * a.rgbda_bs;
  float *out = static_cast<float *>(a.out) + (size_t)bimg * a.out_bs;

  uint32_t q[NIN];
  float dd[NIN];
  bool in[NIN];
#pragma unroll
  for (int k = 0; k < NIN; ++k) {
    const int pix = tid + k * 256;
    const int gy = ty0 - 1 + pix / LW, gx = tx0 - 1 + pix % LW;
    in[k] = pix < LPix && gy >= 0 && gy < H && gx >= 0 && gx < W;
    const size_t o = in[k] ? (size_t)gy * W + gx : 0;
    q[k] = rgba[o];
    dd[k] = depth[o];
  }
  const float *wsrc = static_cast<const float *>(a.w) + (size_t)co0 * 9 * CK;
  float4 pw[NWR];
#pragma unroll
  for (int k = 0; k < NWR; ++k) {
    const int i = tid + k * 256;
    pw[k] = i < WROWS * 2 ? *reinterpret_cast<const float4 *>(wsrc + (size_t)i * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int k = 0; k < NIN; ++k) {
    const int pix = tid + k * 256;
    if (pix >= LPix) continue;
    const bool A = in[k] && (q[k] >> 24) != 0;
    const float x0 = (float)(q[k] & 255u) / 255.0f, x1 = (float)((q[k] >> 8) & 255u) / 255.0f;
    const float x2 = (float)((q[k] >> 16) & 255u) / 255.0f, x3 = A ? dd[k] * 0.0625f : 0.f, x4 = A ? 1.f : 0.f;
    float *d = &s_in[pix * S];
    *reinterpret_cast<float4 *>(d) = in[k] ? make_float4(x0, x1, x2, 0.f) : make_float4(0.f, 0.f, 0.f, 0.f);
    *reinterpret_cast<float4 *>(d + 4) = make_float4(x3, x4, 0.f, 0.f);
  }
#pragma unroll
  for (int k = 0; k < NWR; ++k) {
    const int i = tid + k * 256;
    if (i < WROWS * 2) *reinterpret_cast<float4 *>(&s_w[(i >> 1) * S + (i & 1) * 4]) = pw[k];
  }
  __syncthreads();

  floatx16 acc[MB][R];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[mb][r][k] = 0.f;
  // lane (n, h) reads channels [4h, 4h + 4): pixel column n + dx of its rows, weight row (32 mb + n) * 9 + tap
  const float *bbase = s_in + (wv * R * LW + n) * S + 4 * h;
  const float *abase = s_w + n * 9 * S + 4 * h;
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) {
    float4 fa[MB][3], fb[R + 2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
        fa[mb][dy] = *reinterpret_cast<const float4 *>(abase + (mb * 32 * 9 + dy * 3 + dx) * S);
#pragma unroll
    for (int i = 0; i < R + 2; ++i) fb[i] = *reinterpret_cast<const float4 *>(bbase + (i * LW + dx) * S);
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const float4 av = fa[mb][dy], bv = fb[r + dy];
          acc[mb][r] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv.x, acc[mb][r], 0, 0, 0);
          acc[mb][r] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv.y, acc[mb][r], 0, 0, 0);
          acc[mb][r] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv.z, acc[mb][r], 0, 0, 0);
        }
  }

  // accumulator register 4j + i of block (mb, r) holds output channel
  // co0 + 32 mb + 8j + 4h + i of pixel (ty0 + wR + r, tx0 + n)
  const int gx = tx0 + n;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = co0 + mb * 32 + 8 * j + 4 * h;
      if (c >= a.cout) continue;
      const float4 b = *reinterpret_cast<const float4 *>(a.bias + c);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int gy = ty0 + wv * R + r;
        if (gy < H && gx < W)
          *reinterpret_cast<float4 *>(out + ((size_t)gy * W + gx) * a.cout + c) =
              make_float4(fmaxf(acc[mb][r][4 * j + 0] + b.x, 0.f), fmaxf(acc[mb][r][4 * j + 1] + b.y, 0.f),
                          fmaxf(acc[mb][r][4 * j + 2] + b.z, 0.f), fmaxf(acc[mb][r][4 * j + 3] + b.w, 0.f));
      }
    }
}

// 3x3 convolution in float32 by Winograd's minimal filtering F(2x2, 3x3): each
// 2x2 block of output pixels is Y = A^T [sum_c U_c (.) V_c] A with
// V_c = B^T d_c B the transform of the block's 4x4 input patch d_c of channel
// c and U_c = G g_c G^T the transform of the 3x3 filter (computed on the host);
//   B^T = [1 0 -1 0; 0 1 1 0; 0 -1 1 0; 0 1 0 -1],
//   G   = [1 0 0; 1/2 1/2 1/2; 1/2 -1/2 1/2; 0 0 1],
//   A^T = [1 1 1 0; 0 1 -1 -1].
// The channel sum is, for each of the 16 transform positions (xi, nu), a GEMM
// (output channels x blocks, K = input channels) on v_mfma_f32_32x32x2_f32:
// 16 multiplies per block and channel pair instead of 36 for the direct form.
// A tile is 8 rows x 32 columns of output pixels (4 x 16 blocks) x 32 MB output
// channels.  A workgroup has 8 waves; wave w owns transform row xi = w & 3 of
// block rows 2 (w >> 2) and 2 (w >> 2) + 1 (32 blocks, one per lane column)
// and holds the accumulators (xi, nu = 0..3) of MB blocks of 32 channels, so
// with MB = 2 its input fragments feed two MFMA blocks.  Row xi of B^T d
// combines two patch rows, so a wave reads 8 of the 16 patch pixels and
// transforms in registers.  Workgroups are persistent (one per CU) and stream
// the CK-channel chunks of their tiles through two LDS buffers, one barrier
// per chunk.  Epilogue: each wave reduces its row by A (2 values per block and
// channel) into LDS, and every thread then finishes 4 channels of one block:
// the A^T row reduction, bias, ReLU, the 2x2 output block (which is also the
// max-pool window) and the fused 1x1 head.
template <bool HEAD, int MB, int CK>
__global__ __launch_bounds__(512) void wino3x3_kernel(ConvArgs a, int ntx, int nty, int nzc, int ntiles) {
  constexpr int NT = 512, TB = 2;                    // threads; tile blocks of 2 tile rows
  constexpr int NCO = 32 * MB;                       // output channels per workgroup tile
  constexpr int NV = CK / 4;                         // staged channels CK: 16-byte vectors per pixel
  constexpr int TH = 4 * TB, TW = 32, LW = TW + 2, LPix = (TH + 2) * LW;
  // input tile in LDS, in 16-byte units (4 channels): unit of (row, col, vector v)
  // = v PX + (col & 1) PY + row HZ + (col >> 1).  Lanes read the pixels of 16
  // consecutive blocks, 2 columns apart: with even and odd columns in separate
  // planes those are 16 consecutive units, one per bank group.
  constexpr int HZ = LW / 2, PY = (TH + 2) * HZ, PX = 2 * PY;
  constexpr int CS = 16 * CK + 4;                    // LDS floats per output channel of U (+4: bank spread)
  constexpr int INP = NV * PX * 4, BUF = INP + NCO * CS;
  constexpr int PP = NT / NV;                        // pixels / U rows per staging pass
  constexpr int NIN = (LPix + PP - 1) / PP, NWR = NCO * 16 / PP;
  constexpr int ES = 2 * 32 + 4;                     // epilogue floats per tile: 2 columns x 32 channels (+4)
  constexpr int EPL = TB * 4 * 32 * ES;
  // LDS: [buffer 0][GAP][buffer 1]; the epilogue's EPL floats start at the
  // buffer just finished (0 or BUF) and may run into the gap
  constexpr int GAP = EPL > BUF ? EPL - BUF : 0, B1 = BUF + GAP;
  static_assert(NCO * 16 % PP == 0, "U rows must fill whole staging passes");
  __shared__ __attribute__((aligned(16))) float smem[2 * BUF + GAP];

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 31, h = lane >> 5;
  const int xi = wv & 3, tb = wv >> 2;
  const int H = a.H, W = a.W;
  const int Cin = a.C0 + a.C1;

  // Persistent workgroups walk a list of tiles (an 8 x 32 pixel block of one
  // image and one block of NCO output channels).  Tile order: output-channel
  // blocks of one pixel block are consecutive, then pixel blocks, then images;
  // with a grid of 8k workgroups, workgroup w (on XCD w mod 8) walks every
  // k-th tile of the w mod 8 -th eighth of the list, so tiles that share input
  // pixels run on the same XCD at about the same time.
  const int G = gridDim.x;
  int t_first, t_end, t_step;
  if (G % 8 == 0 && G < ntiles) {
    const int x = blockIdx.x & 7, per = G >> 3;
    t_first = (int)((long)x * ntiles / 8) + (blockIdx.x >> 3);
    t_end = (int)((long)(x + 1) * ntiles / 8);
    t_step = per;
  } else {
    t_first = blockIdx.x;
    t_end = ntiles;
    t_step = G;
  }
  struct TileId { int ty0, tx0, co0, bimg; };
  auto decode = [&](int T) {
    TileId d;
    const int cz = T % nzc, sp = T / nzc;
    const int nsp = ntx * nty;
    d.bimg = sp / nsp;
    const int r = sp - d.bimg * nsp;
    d.ty0 = (r / ntx) * TH;
    d.tx0 = (r % ntx) * TW;
    d.co0 = cz * NCO;
    return d;
  };

  // staging plan: this thread moves float4 qv of pixels p0, p0 + PP, ... and of
  // U rows p0, p0 + PP, ... (row r = 16 co + position)
  const int qv = (tid % NV) * 4, p0 = tid / NV;
  int lofs[NIN];
#pragma unroll
  for (int k = 0; k < NIN; ++k) {
    const int pix = p0 + k * PP, row = pix / LW, col = pix % LW;
    lofs[k] = 4 * ((qv / 4) * PX + (col & 1) * PY + row * HZ + (col >> 1));
  }
  // fetch state: the tile whose chunks are being fetched
  int off0[NIN], off1[NIN];
  const float *fin0 = nullptr, *fin1 = nullptr, *wsrc = nullptr;
  auto set_fetch_tile = [&](const TileId &d) {
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      const int pix = p0 + k * PP, row = pix / LW, col = pix % LW;
      const int gy = d.ty0 - 1 + row, gx = d.tx0 - 1 + col;
      const bool inside = pix < LPix && gy >= 0 && gy < H && gx >= 0 && gx < W;
      off0[k] = inside ? gy * W + gx : -1;
      off1[k] = inside ? (gy >> 1) * (W >> 1) + (gx >> 1) : -1;
    }
    fin0 = static_cast<const float *>(a.in0) + (size_t)d.bimg * a.in0_bs;
    fin1 = a.in1 ? static_cast<const float *>(a.in1) + (size_t)d.bimg * a.in1_bs : nullptr;
    wsrc = a.wu + ((size_t)d.co0 * 16 + p0) * a.cin_pad + qv;
  };
  const size_t wstep = (size_t)PP * a.cin_pad;
  auto fetch_in = [&](int ci, uint4 (&v)[NIN]) {
    const bool from0 = ci < a.C0;
    const size_t csrc = from0 ? a.C0 : a.C1;
    const float *src = (from0 ? fin0 + ci : fin1 + (ci - a.C0)) + qv;
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      const int o = from0 ? off0[k] : off1[k];
      const uint4 x = *reinterpret_cast<const uint4 *>(src + (size_t)(o < 0 ? 0 : o) * csrc);
      v[k] = o < 0 ? make_uint4(0u, 0u, 0u, 0u) : x;
    }
  };
  auto fetch_w = [&](int ci, uint4 (&v)[NWR]) {
#pragma unroll
    for (int k = 0; k < NWR; ++k) v[k] = *reinterpret_cast<const uint4 *>(wsrc + k * wstep + ci);
  };
  auto store_in = [&](int buf, const uint4 (&v)[NIN]) {
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      if (!((k + 1) * PP <= LPix || p0 + k * PP < LPix)) continue;
      *reinterpret_cast<uint4 *>(&smem[buf + lofs[k]]) = v[k];
    }
  };
  auto store_w = [&](int buf, const uint4 (&v)[NWR]) {
#pragma unroll
    for (int k = 0; k < NWR; ++k) {
      const int r = p0 + k * PP;
      *reinterpret_cast<uint4 *>(&smem[buf + INP + (r >> 4) * CS + (r & 15) * CK + qv]) = v[k];
    }
  };

  // lane (n, h): block (tr, tc) of the tile, channels 8g + 4h + s of
  // chunk group g at k-step s.  Row xi of B^T d is patch row ra + sg * patch row rb.
  const int tr = 2 * tb + (n >> 4), tc = n & 15;
  const int ra = xi == 0 ? 0 : (xi == 2 ? 2 : 1);
  const int rb = xi == 0 ? 2 : (xi == 1 ? 2 : (xi == 2 ? 1 : 3));
  const float sg = xi == 1 ? 1.f : -1.f;
  const int ioa = 4 * (h * PX + (2 * tr + ra) * HZ + tc);
  const int iob = 4 * (h * PX + (2 * tr + rb) * HZ + tc);
  const int iow = INP + n * CS + 4 * xi * CK + 4 * h;
  // acc[mb][nu]: positions (xi, nu) of output channels co0 + 32 mb + ... of 32 blocks
  floatx16 acc[MB][4];
  auto zero_acc = [&]() {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[mb][v][q] = 0.f;
  };
  auto compute = [&](int buf) {
    const float *pa = smem + buf + ioa, *pb = smem + buf + iob, *pu = smem + buf + iow;
#pragma unroll 1
    for (int g = 0; g < CK / 8; ++g) {
      float4 da[4], db[4], u[MB][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // column 2 tc + j of vector 2 g + h
        const int o = 4 * (2 * g * PX + (j & 1) * PY + (j >> 1));
        da[j] = *reinterpret_cast<const float4 *>(pa + o);
        db[j] = *reinterpret_cast<const float4 *>(pb + o);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 4; ++v) u[mb][v] = *reinterpret_cast<const float4 *>(pu + mb * 32 * CS + v * CK + 8 * g);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        auto comp = [s](const float4 &f) { return s == 0 ? f.x : (s == 1 ? f.y : (s == 2 ? f.z : f.w)); };
        float r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = fmaf(sg, comp(db[j]), comp(da[j]));
        const float t[4] = {r[0] - r[2], r[1] + r[2], r[2] - r[1], r[1] - r[3]};
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            acc[mb][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(u[mb][v]), t[v], acc[mb][v], 0, 0, 0);
      }
    }
  };

  // ---- epilogue of one tile into E (EPL floats of LDS nobody reads any
  // more), one block of 32 output channels at a time.  Accumulator register
  // 4j + i of acc[mb][nu] holds position (xi, nu) of channel co0 + 32 mb +
  // 8j + 4h + i for block n; each wave reduces nu by A into E, then thread
  // (block et, quad q) reduces xi by A^T for channels c .. c + 3.
  const int q = tid & 7, et = tid >> 3, etb = et >> 5, en = et & 31;
  auto epilogue = [&](float *E, const TileId &d) {
    const int gy0 = d.ty0 + 2 * (2 * etb + (en >> 4)), gx0 = d.tx0 + 2 * (en & 15);
    float *out = a.out ? static_cast<float *>(a.out) + (size_t)d.bimg * a.out_bs : nullptr;
    float *out_pool = a.out_pool ? static_cast<float *>(a.out_pool) + (size_t)d.bimg * a.pool_bs : nullptr;
    float hs[2][2][3];  // head partial sums of this thread's channels
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int col = 0; col < 2; ++col) hs[r][col][0] = hs[r][col][1] = hs[r][col][2] = 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if (mb > 0) __syncthreads();  // the previous block's readers are done with E
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float4 p0v, p1v;
        p0v.x = acc[mb][0][4 * j + 0] + acc[mb][1][4 * j + 0] + acc[mb][2][4 * j + 0];
        p0v.y = acc[mb][0][4 * j + 1] + acc[mb][1][4 * j + 1] + acc[mb][2][4 * j + 1];
        p0v.z = acc[mb][0][4 * j + 2] + acc[mb][1][4 * j + 2] + acc[mb][2][4 * j + 2];
        p0v.w = acc[mb][0][4 * j + 3] + acc[mb][1][4 * j + 3] + acc[mb][2][4 * j + 3];
        p1v.x = acc[mb][1][4 * j + 0] - acc[mb][2][4 * j + 0] - acc[mb][3][4 * j + 0];
        p1v.y = acc[mb][1][4 * j + 1] - acc[mb][2][4 * j + 1] - acc[mb][3][4 * j + 1];
        p1v.z = acc[mb][1][4 * j + 2] - acc[mb][2][4 * j + 2] - acc[mb][3][4 * j + 2];
        p1v.w = acc[mb][1][4 * j + 3] - acc[mb][2][4 * j + 3] - acc[mb][3][4 * j + 3];
        float *e = E + ((tb * 4 + xi) * 32 + n) * ES + 8 * j + 4 * h;
        *reinterpret_cast<float4 *>(e) = p0v;
        *reinterpret_cast<float4 *>(e + 32) = p1v;
      }
      __syncthreads();
      const int c = d.co0 + 32 * mb + 4 * q;
      float y[2][2][4];  // [row][column][channel]
#pragma unroll
      for (int col = 0; col < 2; ++col) {
        float4 P[4];
#pragma unroll
        for (int x = 0; x < 4; ++x)
          P[x] = *reinterpret_cast<const float4 *>(E + ((etb * 4 + x) * 32 + en) * ES + col * 32 + 4 * q);
        y[0][col][0] = P[0].x + P[1].x + P[2].x;
        y[0][col][1] = P[0].y + P[1].y + P[2].y;
        y[0][col][2] = P[0].z + P[1].z + P[2].z;
        y[0][col][3] = P[0].w + P[1].w + P[2].w;
        y[1][col][0] = P[1].x - P[2].x - P[3].x;
        y[1][col][1] = P[1].y - P[2].y - P[3].y;
        y[1][col][2] = P[1].z - P[2].z - P[3].z;
        y[1][col][3] = P[1].w - P[2].w - P[3].w;
      }
      const bool live = c < a.cout;
      float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
      if (live) b = *reinterpret_cast<const float4 *>(a.bias + c);
      const float bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
          for (int i = 0; i < 4; ++i) y[r][col][i] = fmaxf(y[r][col][i] + bb[i], 0.f);
      if constexpr (HEAD) {
        if (live) {
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                hs[r][col][0] = fmaf(a.head_w[c + i], y[r][col][i], hs[r][col][0]);
                hs[r][col][1] = fmaf(a.head_w[a.cout + c + i], y[r][col][i], hs[r][col][1]);
                hs[r][col][2] = fmaf(a.head_w[2 * a.cout + c + i], y[r][col][i], hs[r][col][2]);
              }
        }
      } else if (live) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int col = 0; col < 2; ++col) {
            const int gy = gy0 + r, gx = gx0 + col;
            if (gy < H && gx < W)
              *reinterpret_cast<float4 *>(out + ((size_t)gy * W + gx) * a.cout + c) =
                  make_float4(y[r][col][0], y[r][col][1], y[r][col][2], y[r][col][3]);
          }
        if (out_pool && gy0 < H && gx0 < W) {
          float m[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) m[i] = fmaxf(fmaxf(y[0][0][i], y[0][1][i]), fmaxf(y[1][0][i], y[1][1][i]));
          *reinterpret_cast<float4 *>(out_pool + ((size_t)(gy0 >> 1) * (W >> 1) + (gx0 >> 1)) * a.cout + c) =
              make_float4(m[0], m[1], m[2], m[3]);
        }
      }
    }
    if constexpr (HEAD) {
      // the tile holds every output channel (cout <= NCO): sum the head over
      // the block's 8 threads; thread q < 4 writes pixel (q >> 1, q & 1)
      float *head_out =
          a.head_outs ? a.head_outs[d.bimg] : (a.head_out ? a.head_out + (size_t)d.bimg * 3 * H * W : nullptr);
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int m = 1; m < 8; m <<= 1) hs[r][col][k] += __shfl_xor(hs[r][col][k], m, 64);
      if (q < 4) {
        const int r = q >> 1, col = q & 1, gy = gy0 + r, gx = gx0 + col;
        float o0 = hs[0][0][0], o1 = hs[0][0][1], o2 = hs[0][0][2];
#pragma unroll
        for (int rr = 0; rr < 2; ++rr)
#pragma unroll
          for (int cc = 0; cc < 2; ++cc)
            if (rr == r && cc == col) {
              o0 = hs[rr][cc][0];
              o1 = hs[rr][cc][1];
              o2 = hs[rr][cc][2];
            }
        if (gy < H && gx < W) {
          const size_t HW = (size_t)H * W, p = (size_t)gy * W + gx;
          head_out[p] = o0 + a.head_b[0];
          head_out[HW + p] = o1 + a.head_b[1];
          head_out[2 * HW + p] = o2 + a.head_b[2];
        }
      }
    }
  };

  // The chunks of this workgroup's tiles form one stream: chunk step t is
  // multiplied from LDS buffer t & 1 while step t + 1 (the next chunk of the
  // tile, or the first chunk of the next tile) is fetched into registers; it
  // is then written to the other buffer, which every wave finished reading
  // before the previous barrier.  After a tile's last chunk the epilogue runs
  // on the buffer just finished, so the next tile's first chunk is already
  // staged when its multiplications start.
  if (t_first >= t_end) return;
  const int nch = Cin / CK;
  TileId cur = decode(t_first);
  set_fetch_tile(cur);
  {
    uint4 v[NIN], w[NWR];
    fetch_in(0, v);
    fetch_w(0, w);
    store_in(0, v);
    store_w(0, w);
  }
  __syncthreads();
  zero_acc();
  uint4 v[NIN], w[NWR];
  int T = t_first, c = 0, buf = 0;
  for (;;) {
    const bool last = c + 1 == nch;
    const int Tn = last ? T + t_step : T;
    const bool more = Tn < t_end;
    TileId nxt = cur;
    if (more) {
      if (last) {
        nxt = decode(Tn);
        set_fetch_tile(nxt);
      }
      const int cn = last ? 0 : (c + 1) * CK;
      fetch_w(cn, w);
      fetch_in(cn, v);
    } else {
      // (defined values on every path keep the arrays in registers)
#pragma unroll
      for (int k = 0; k < NWR; ++k) w[k] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int k = 0; k < NIN; ++k) v[k] = make_uint4(0u, 0u, 0u, 0u);
    }
    compute(buf);  // one call site: the accumulators stay in place
    const int other = buf == 0 ? B1 : 0;
    if (more) {
      store_in(other, v);
      store_w(other, w);
    }
    __syncthreads();
    if (last) {
      epilogue(smem + (buf == 0 ? 0 : BUF), cur);
      if (!more) break;
      __syncthreads();  // E is read before the buffer is staged again
      zero_acc();
      cur = nxt;
      T = Tn;
      c = 0;
    } else {
      ++c;
    }
    buf = other;
  }
}

// 1x1 head of a layer too wide to fuse it: weights [3][C], one thread per
// pixel, planar output
__global__ __launch_bounds__(256) void head32_kernel(const float *__restrict__ x, int C, int npix,
                                                     const float *__restrict__ w, const float *__restrict__ b,
                                                     float *__restrict__ out) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= npix) return;
  float y0 = b[0], y1 = b[1], y2 = b[2];
  for (int c = 0; c < C; c += 4) {
    const float4 q = *reinterpret_cast<const float4 *>(x + (size_t)p * C + c);
    const float v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      y0 = fmaf(w[c + i], v[i], y0);
      y1 = fmaf(w[C + c + i], v[i], y1);
      y2 = fmaf(w[2 * C + c + i], v[i], y2);
    }
  }
  out[p] = y0;
  out[(size_t)npix + p] = y1;
  out[2 * (size_t)npix + p] = y2;
}

constexpr long kSmallGrid = 768;

// Float32 layers whose inputs come in chunks of 16 channels (all but the
// first) run as Winograd F(2x2, 3x3) in persistent workgroups, one resident
// per CU (LDS), each walking its share of the 8 x 32 pixel tiles.
template <int MB, int CK>
hipError_t wino_launch_mc(const ConvArgs &a, int cout_pad, bool head, hipStream_t s) {
  const int ntx = (a.W + 31) / 32, nty = (a.H + 7) / 8;
  const int nzc = cout_pad / (32 * MB), ntiles = ntx * nty * nzc * a.batch;
  static std::atomic<int> cus[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      return hipErrorInvalidDevice;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  const int grid = ntiles < n ? ntiles : n;
  if (head)
    wino3x3_kernel<true, MB, CK><<<grid, 512, 0, s>>>(a, ntx, nty, nzc, ntiles);
  else
    wino3x3_kernel<false, MB, CK><<<grid, 512, 0, s>>>(a, ntx, nty, nzc, ntiles);
  return hipGetLastError();
}
// Layers with a multiple of 64 output channels: tiles of 64 channels (each
// wave reuses its input fragments for two MFMA blocks), staged 8 input
// channels at a time (two LDS buffers of U for 64 channels must fit), unless
// one image gives fewer than kSmallGrid such tiles (the 135x240 level of a
// 1080p frame), where 32-channel tiles keep every CU busy; a layer with the
// fused head needs all its channels (at most 64) in one tile.  Others: 32
// channels, 16 input channels at a time.  Both take the same sums in the same
// order, so the choice does not change results.
hipError_t wino_launch(const ConvArgs &a, int cout_pad, bool head, hipStream_t s) {
  const long tiles64 = (long)((a.W + 31) / 32) * ((a.H + 7) / 8) * (cout_pad / 64);
  if (cout_pad % 64 == 0 && (tiles64 >= kSmallGrid || head)) return wino_launch_mc<2, 8>(a, cout_pad, head, s);
  return wino_launch_mc<1, 16>(a, cout_pad, head, s);
}

hipError_t first_launch(const ConvArgs &a, int cout_pad, hipStream_t s) {
  const int bm = cout_pad % 64 == 0 ? 64 : 32;
  const dim3 grid((a.W + 31) / 32, (a.H + 7) / 8, (cout_pad / bm) * a.batch);
  if (bm == 64)
    first3x3_kernel<64, 2><<<grid, 256, 0, s>>>(a);
  else
    first3x3_kernel<32, 2><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_conv3x3(const ConvCall &c, Prec p, hipStream_t s) {
  if (p != Prec::F32) return launch_conv16(c, p, s);
  const ConvLayer &L = *c.layer;
  const ConvArgs a{c.in0, c.in1, c.C0, c.C1, c.H, c.W, L.w, L.bias, L.cout, L.cin_pad, c.out, c.out_pool,
                   c.head_w, c.head_b, c.head_out, c.batch < 1 ? 1 : c.batch, c.in0_bs / 4, c.in1_bs / 4,
                   c.out_bs / 4, c.pool_bs / 4, c.head_outs, c.rgbda_depth, c.rgbda_rgba, c.rgbda_bs,
                   static_cast<const float *>(L.wu)};
  const bool head = c.head_out || c.head_outs;
  if (head && (L.cout_pad > 64 || c.out_pool)) return hipErrorInvalidValue;
  if (c.rgbda_depth) {
    if (!c.rgbda_rgba || c.C1 != 0 || L.cin_pad != 8 || head || c.out_pool) return hipErrorInvalidValue;
    return first_launch(a, L.cout_pad, s);
  }
  if (!L.wu || c.C0 % 16 || c.C1 % 16 || c.C0 + c.C1 != L.cin_pad) return hipErrorInvalidValue;
  return wino_launch(a, L.cout_pad, head, s);
}

hipError_t launch_head(const void *x, int C, int H, int W, const ConvLayer &head, Prec p, float *out, hipStream_t s) {
  if (p != Prec::F32) return launch_head16(x, C, H, W, head, p, out, s);
  const int npix = H * W;
  head32_kernel<<<(npix + 255) / 256, 256, 0, s>>>(static_cast<const float *>(x), C, npix,
                                                   static_cast<const float *>(head.w), head.bias, out);
  return hipGetLastError();
}

}  // namespace lnr
