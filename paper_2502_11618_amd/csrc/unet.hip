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

#include "conv_stage.h"

namespace lnr {
namespace {

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
__global__ __launch_bounds__(256) void first3x3_kernel(Args a) {
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
  const int nzc = (a.cout + BM - 1) / BM;
  const int bimg = blockIdx.z / nzc;
  const int co0 = (blockIdx.z - bimg * nzc) * BM;
  const int H = a.H, W = a.W;
  const float *depth = a.depth + (size_t)bimg * a.rgbda_bs;
  const uint32_t *rgba = a.rgba + (size_t)bimg * a.rgbda_bs;
  char *out = a.out + (size_t)bimg * a.out_bs;

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
  const float *wsrc = reinterpret_cast<const float *>(a.w) + (size_t)co0 * 9 * CK;
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
          *reinterpret_cast<float4 *>(out + ((size_t)(c >> 2) * H * W + (size_t)gy * W + gx) * 16) =
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
// (output channels x blocks, K = input channels) on v_mfma_f32_16x16x4_f32:
// 16 multiplies per block and channel pair instead of 36 for the direct form.
//
// Tensors lie in memory as channel blocks: planes of 16-byte units, a unit the
// 4 channels of a pixel.  A workgroup of 4 waves takes tiles of 8 rows x 32
// columns of output pixels x 16 M output channels; wave w owns row w of the 2x2
// blocks (16 of them) and keeps all 16 positions of its blocks and the tile's
// channels in accumulators, so the output transform, the 2x2 max-pool (the
// block is its window) and the 1x1 head run in registers and no accumulator
// goes through LDS.  Chunks of 8 input channels of all the workgroup's tiles
// form one stream.  In step t a wave multiplies chunk t from registers (its
// transform) and LDS (the filters); in the multiplications' shadow it reads and
// transforms chunk t + 1 and starts the loads, straight into LDS, of step
// t + 1's filters and step t + 3's input.  One barrier per step; two workgroups
// per CU (three with M = 1) cover each other's.  The instructions of a step are
// fixed in place (sched_barrier): left alone the compiler reads each filter
// right before its use and gathers the transform in front, 8% slower.
//
// LDS of a step: input units [channel quad][halo row][even columns, odd
// columns] (the lanes read columns two apart: 16 consecutive units), filters
// [16-channel tile][position][channel pair][16 channels][2].  Lane (n, kq) =
// (lane & 15, lane >> 4) multiplies channels 2 kq and 2 kq + 1 of a chunk:
// channel n of the filters' tile, block n of the wave's row.
//
// Bound by the matrix cores and, in part, by the transform's 64 additions for
// 32 M multiplications: the cores are busy 74% of 128 + 256 -> 128 channels at
// 480 x 270 (437 us), 63% of 32 -> 32 at 1920 x 1080 (196 us), which also reads
// and writes 600 MB.  With one transform per 512-thread workgroup, shared
// through LDS, and the accumulators added up there: 538 and 272 us.
typedef float floatx4 __attribute__((ext_vector_type(4)));
template <int M, bool HEAD>
struct WinoLds {
  static constexpr int TH = 8, LW = 34, HW = 17, UB = (TH + 2) * LW;  // halo tile: units per channel quad
  static constexpr int NL = (UB + 63) / 64;                           // in wave loads
  static constexpr int INB = 2 * UB * 16, WB = M * 8192;              // bytes of a step's input and filters
  static constexpr int kWeights = 3 * INB, kBias = kWeights + 2 * WB;
  static constexpr int kHead = kBias + 2 * M * 16 * 4;                // two tiles' biases
  static constexpr int kBytes = kHead + (HEAD ? (3 * 64 + 4) * 4 : 0);
};
template <int M, bool HEAD>
__global__ __launch_bounds__(256, 2) void wino_kernel(Args a) {
  using S = WinoLds<M, HEAD>;
  constexpr int NW = 4, LW = S::LW, UB = S::UB, NK = (S::NL + NW - 1) / NW;
  __shared__ __attribute__((aligned(16))) char sm[S::kBytes];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kq = lane >> 4;
  const int H = a.H, W = a.W;
  const uint32_t sm0 = lds_address(sm);
  const int nch = (a.C0 + a.C1) >> 3, nch0 = a.C0 >> 3;
  const Walk walk = my_tiles(a);
  if (walk.first >= walk.end) return;
  const int steps = (walk.end - walk.first) * nch;
  if constexpr (HEAD) {
    float *sh = reinterpret_cast<float *>(sm + S::kHead);
    for (int i = tid; i < 3 * 64; i += 64 * NW) {
      const int o = i >> 6, c = i & 63;
      sh[i] = c < a.cout ? a.head_w[o * a.cout + c] : 0.f;
    }
    if (tid < 3) sh[192 + tid] = a.head_b[tid];
  }

  // ---- filters: 2 M loads per wave and step
  const char *wptr = nullptr;
  int wT = walk.first, wc = 0, wslot = 0, wtile = 0;
  uint64_t wlanes = ~0ull;
  auto begin_weights = [&]() {
    if (wc != 0) return;
    if (wT < walk.end) {
      const int cz = __builtin_amdgcn_readfirstlane(wT % a.ncz);
      wptr = uniform(a.w + ((size_t)(cz * M >> 1) * nch * 2 + (cz * M & 1)) * 8192 + wv * 1024);
      if (wv == 0) load_lds4(a.bias + cz * M * 16, lane * 4, sm0 + S::kBias + (wtile & 1) * M * 64, (1ull << M * 16) - 1);
    } else {
      wlanes = 0;
    }
  };
  auto issue_weights = [&](int k) {
    load_lds16(wptr + k * NW * 1024, lane * 16, sm0 + S::kWeights + wslot * S::WB + wv * 1024 + k * NW * 1024, wlanes);
  };
  auto end_weights = [&]() {
    wptr += 2 * 8192;
    wslot ^= 1;
    if (++wc == nch) {
      wc = 0;
      ++wtile;
      ++wT;
    }
  };

  // ---- input: in every channel quad, wave load j = wv + NW k covers units j 64 + lane
  int urow[NK], ucol[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int pos = (wv + NW * k) * 64 + lane;
    urow[k] = pos / LW;
    const int q = pos - urow[k] * LW;
    ucol[k] = q < S::HW ? 2 * q : 2 * (q - S::HW) + 1;
  }
  int iT = walk.first, ic = 0, islot = 0;
  int iy0 = 0, ix0 = 0, iimg = 0;
  uint32_t voff[NK];
  uint64_t lanes[NK];
  uint32_t outside = 0;  // bit k: this lane's unit of load k lies outside the image
  bool border = false;
  const char *src = nullptr;  // the chunk's first channel quad, at the tile's first halo row
  size_t blk = 0;             // bytes per channel quad of the current source
  auto set_source = [&](bool second) {
    const int sh = second ? 1 : 0, Ws = W >> sh, y0 = (iy0 - 1) >> sh;
    const char *in = second ? a.in1 + (size_t)iimg * a.in1_bs : a.in0 + (size_t)iimg * a.in0_bs;
    blk = (size_t)(H >> sh) * Ws * 16;
    src = uniform(in + (ptrdiff_t)y0 * Ws * 16);
#pragma unroll
    for (int k = 0; k < NK; ++k)  // (unused outside the image)
      voff[k] = (uint32_t)((((iy0 - 1 + urow[k]) >> sh) - y0) * Ws + ((ix0 - 1 + ucol[k]) >> sh)) * 16u;
  };
  auto begin_input = [&]() {
    if (ic == 0 && iT >= walk.end) {
#pragma unroll
      for (int k = 0; k < NK; ++k) lanes[k] = 0;
      border = false;
    } else if (ic == 0) {
      const Tile t = tile_at(a, iT);
      iy0 = t.ty * S::TH;
      ix0 = t.tx * 32;
      iimg = t.img;
      outside = 0;
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const bool any = urow[k] < S::TH + 2;
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
    load_lds16(src + b * blk, voff[k], sm0 + islot * S::INB + wv * 1024 + b * UB * 16 + k * NW * 1024, lanes[k]);
  };
  auto end_input = [&]() {
    if (border) {
#pragma unroll
      for (int k = 0; k < NK; ++k)
        if ((outside >> k) & 1u) {
#pragma unroll
          for (int b = 0; b < 2; ++b)
            *reinterpret_cast<uint4 *>(sm + islot * S::INB + wv * 1024 + b * UB * 16 + k * NW * 1024 + lane * 16) =
                make_uint4(0u, 0u, 0u, 0u);
        }
    }
    src += 2 * blk;
    islot = islot == 2 ? 0 : islot + 1;
    if (++ic == nch) {
      ic = 0;
      ++iT;
    }
  };

  // acc[m][4 xi + nu]: channels 16 m + 4 kq + i of block n
  floatx4 acc[M][16];
  auto zero_acc = [&]() {
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int p = 0; p < 16; ++p) acc[m][p] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  zero_acc();
  const char *D = sm + ((kq >> 1) * UB + 2 * wv * LW + n) * 16 + (kq & 1) * 8;
  const char *U = sm + S::kWeights + lane * 8;
  float hs[2][2][3];  // head sums of the pixel tile's channels so far

  // B^T d B of a lane's channels 2 kq, 2 kq + 1, in three parts: the patch's
  // column j, B^T over its rows, B over the columns of row x
  float2 d[4][4], v[16];
  auto read_d = [&](int slot, int j) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      d[r][j] = *reinterpret_cast<const float2 *>(D + slot * S::INB + (r * LW + (j & 1) * S::HW + (j >> 1)) * 16);
  };
  auto rows = [&](int j) {
    const float2 d0 = d[0][j], d1 = d[1][j], d2 = d[2][j], d3 = d[3][j];
    d[0][j] = make_float2(d0.x - d2.x, d0.y - d2.y);
    d[1][j] = make_float2(d1.x + d2.x, d1.y + d2.y);
    d[2][j] = make_float2(d2.x - d1.x, d2.y - d1.y);
    d[3][j] = make_float2(d1.x - d3.x, d1.y - d3.y);
    // (keeps the compiler from moving the sums out of the multiplications' shadow)
#pragma unroll
    for (int r = 0; r < 4; ++r) asm volatile("" : "+v"(d[r][j].x), "+v"(d[r][j].y));
  };
  auto columns = [&](int x) {
    v[4 * x + 0] = make_float2(d[x][0].x - d[x][2].x, d[x][0].y - d[x][2].y);
    v[4 * x + 1] = make_float2(d[x][1].x + d[x][2].x, d[x][1].y + d[x][2].y);
    v[4 * x + 2] = make_float2(d[x][2].x - d[x][1].x, d[x][2].y - d[x][1].y);
    v[4 * x + 3] = make_float2(d[x][1].x - d[x][3].x, d[x][1].y - d[x][3].y);
#pragma unroll
    for (int nu = 0; nu < 4; ++nu) asm volatile("" : "+v"(v[4 * x + nu].x), "+v"(v[4 * x + nu].y));
  };
  begin_weights();
  for (int k = 0; k < 2 * M; ++k) issue_weights(k);
  end_weights();
  for (int t = 0; t < 3; ++t) {
    begin_input();
#pragma unroll
    for (int j = 0; j < 2 * NK; ++j) issue_input(j);
    end_input();
  }
  wait_loads<0>();
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    read_d(0, j);
    rows(j);
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) columns(x);
  __syncthreads();  // slot 0 is free
  int T = walk.first, tile = 0, c = 0, slot = 1;
  for (int t = 0; t < steps; ++t) {
    // step t's filters and step t + 1's input lie in LDS, step t's transform in v
    const char *Ut = U + (t & 1) * S::WB;
    float2 u[3][M];
    auto read_u = [&](int p) {
#pragma unroll
      for (int m = 0; m < M; ++m) u[p % 3][m] = *reinterpret_cast<const float2 *>(Ut + m * 8192 + p * 512);
    };
    read_u(0);
    read_u(1);
    begin_weights();
    begin_input();
    // In the multiplications' shadow: the loads of step t + 1's filters and step
    // t + 3's input (masked off past the last), the filters of two positions on, and step
    // t + 1's transform, into v as its values are used up.  (Past the last step
    // it reads a slot of earlier values, and nobody its results.)
#pragma unroll
    for (int p = 0; p < 16; ++p) {
      __builtin_amdgcn_sched_barrier(0);
      if (p + 2 < 16) read_u(p + 2);
      if (p < 4) read_d(slot, p);
      __builtin_amdgcn_sched_barrier(0);
      const float2(&f)[M] = u[p % 3];
#pragma unroll
      for (int m = 0; m < M; ++m) acc[m][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[m].x, v[p].x, acc[m][p], 0, 0, 0);
#pragma unroll
      for (int m = 0; m < M; ++m) acc[m][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[m].y, v[p].y, acc[m][p], 0, 0, 0);
      if (p % 2 && p / 2 < 2 * M) issue_weights(p / 2);
      if (p % 2 == 0 && p >= 8) issue_input(p / 2 - 4);
      if (p >= 2 && p < 6) rows(p - 2);
      if (p == 7) columns(0);
      if (p == 9) columns(1);
      if (p == 12) columns(2);
      if (p == 15) columns(3);
    }
    __builtin_amdgcn_sched_barrier(0);
    end_weights();
    end_input();
    // the input of step t + 3, the newest loads, may stay in flight
    wait_loads<2 * NK>();
    __syncthreads();
    slot = slot == 2 ? 0 : slot + 1;
    if (++c == nch) {
      // ---- epilogue: A^T M A, bias, ReLU; stores, pool or head
      const Tile tl = tile_at(a, T);
      const int gy0 = tl.ty * S::TH + 2 * wv, gx0 = tl.tx * 32 + 2 * n;
      const size_t HWp = (size_t)H * W;
      const float *sb = reinterpret_cast<const float *>(sm + S::kBias) + (tile & 1) * M * 16;
      if constexpr (HEAD) {
        if (tl.cz == 0) {
#pragma unroll
          for (int i = 0; i < 12; ++i) (&hs[0][0][0])[i] = 0.f;
        }
      }
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int c0 = (tl.cz * M + m) * 16;
        if (c0 >= a.cout) continue;  // (cout is a multiple of 16)
        const float4 b4 = *reinterpret_cast<const float4 *>(sb + 16 * m + 4 * kq);
        const floatx4 bias = {b4.x, b4.y, b4.z, b4.w};
        floatx4 y[2][2];
        {
          floatx4 P[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) P[x] = acc[m][4 * x] + acc[m][4 * x + 1] + acc[m][4 * x + 2];
          y[0][0] = P[0] + P[1] + P[2] + bias;
          y[1][0] = P[1] - P[2] - P[3] + bias;
#pragma unroll
          for (int x = 0; x < 4; ++x) P[x] = acc[m][4 * x + 1] - acc[m][4 * x + 2] - acc[m][4 * x + 3];
          y[0][1] = P[0] + P[1] + P[2] + bias;
          y[1][1] = P[1] - P[2] - P[3] + bias;
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int i = 0; i < 4; ++i) y[r][col][i] = fmaxf(y[r][col][i], 0.f);
        if constexpr (HEAD) {
          const float *sh = reinterpret_cast<const float *>(sm + S::kHead) + c0 + 4 * kq;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const float4 w4 = *reinterpret_cast<const float4 *>(sh + 64 * k);
            const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
              for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int i = 0; i < 4; ++i) hs[r][col][k] = fmaf(w[i], y[r][col][i], hs[r][col][k]);
          }
        } else {
          const size_t cb = (size_t)(c0 / 4 + kq);  // channel quad
          char *out = a.out + (size_t)tl.img * a.out_bs + cb * HWp * 16;
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int col = 0; col < 2; ++col)
              if (gy0 + r < H && gx0 + col < W)
                *reinterpret_cast<floatx4 *>(out + ((size_t)(gy0 + r) * W + gx0 + col) * 16) = y[r][col];
          if (a.out_pool && gy0 < H && gx0 < W) {
            floatx4 mx;
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[i] = fmaxf(fmaxf(y[0][0][i], y[0][1][i]), fmaxf(y[1][0][i], y[1][1][i]));
            *reinterpret_cast<floatx4 *>(a.out_pool + (size_t)tl.img * a.pool_bs + cb * (HWp >> 2) * 16 +
                                         ((size_t)(gy0 >> 1) * (W >> 1) + (gx0 >> 1)) * 16) = mx;
          }
        }
      }
      if constexpr (HEAD) {
        if (tl.cz == a.ncz - 1) {
          // sum over the lanes of a block; lane kq writes pixel (kq >> 1, kq & 1)
          const float *hb = reinterpret_cast<const float *>(sm + S::kHead) + 192;
          float o[3] = {0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
              for (int col = 0; col < 2; ++col) {
                float x = hs[r][col][k];
                x += __shfl_xor(x, 16, 64);
                x += __shfl_xor(x, 32, 64);
                if (kq == 2 * r + col) o[k] = x + hb[k];
              }
          float *head_out = a.head_outs ? a.head_outs[tl.img] : a.head_out + (size_t)tl.img * 3 * HWp;
          const int gy = gy0 + (kq >> 1), gx = gx0 + (kq & 1);
          if (gy < H && gx < W) {
            const size_t px = (size_t)gy * W + gx;
#pragma unroll
            for (int k = 0; k < 3; ++k) head_out[k * HWp + px] = o[k];
          }
        }
      }
      zero_acc();
      c = 0;
      ++tile;
      ++T;
    }
  }
}

// Launch of the float32 layers but the first, in two tile sizes: 32 channels
// (M = 2) and 16 (M = 1), which fills the chip earlier, wastes nothing on 16 and
// 48 channels, and repeats the input's transform for every 16.
struct WinoGrid {
  int units, group;  // workgroups at one run each, channel tiles that stay in one (with the fused head: all)
  float cost;
};
template <int M>
WinoGrid wino_grid(const ConvCall &c) {
  const int batch = c.batch < 1 ? 1 : c.batch, ncz = (c.layer->cout + M * 16 - 1) / (M * 16);
  WinoGrid g;
  g.group = c.head_out || c.head_outs ? ncz : 1;
  g.units = (c.W + 31) / 32 * ((c.H + WinoLds<M, false>::TH - 1) / WinoLds<M, false>::TH) * (ncz / g.group) * batch;
  // Microseconds per chunk of 8 input channels that 1, 2 (and 3, M = 1)
  // workgroups together on a CU took; a CU has no room for more.
  static constexpr float kStep[2][4] = {{0.f, 1.1f, 1.6f, 2.2f}, {0.f, 1.5f, 2.5f, 0.f}};
  constexpr int full = M == 1 ? 3 : 2;
  const int k = (g.units + kCUs - 1) / kCUs;
  g.cost = g.group * ((float)(k / full) * kStep[M - 1][full] + kStep[M - 1][k % full]);
  return g;
}
template <int M>
hipError_t wino_tiles(const ConvCall &c, const WinoGrid &g, hipStream_t s) {
  Args a = make_args(c);
  a.w = static_cast<const char *>(c.layer->wu);
  // Short layers (at most 96 input channels) of many tiles: runs of up to 4
  // tiles per workgroup, whose start then hides behind the tiles before (1080p,
  // 32 -> 32 channels: 222 us in runs of one, 205 of four; 64 -> 64: 181, 178;
  // 128 -> 128: 167, 168).  With few tiles, or longer ones, a run only leaves
  // CUs idle at the end (256 -> 256 at 240 x 135: 204, 332).
  const int slots = (M == 1 ? 3 : 2) * kCUs, steps = g.group * ((a.C0 + a.C1) / 8);
  int run = 1;
  if (steps <= 12 && g.units >= 4 * slots) {
    long long best = 0;
    for (int r = 1; r <= 4; ++r) {
      const long long t = (g.units + (long long)r * slots - 1) / ((long long)r * slots) * (r * (steps + 1) + 1);
      if (!best || t < best) best = t, run = r;
    }
  }
  const int batch = c.batch < 1 ? 1 : c.batch, cout = (a.cout + M * 16 - 1) / (M * 16) * (M * 16);
  const int grid = set_tiles(a, WinoLds<M, false>::TH, M * 16, cout, batch, run * g.group, g.group);
  if (c.head_out || c.head_outs)
    wino_kernel<M, true><<<grid, 256, 0, s>>>(a);
  else
    wino_kernel<M, false><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t wino_launch(const ConvCall &c, hipStream_t s) {
  const WinoGrid g1 = wino_grid<1>(c), g2 = wino_grid<2>(c);
  return g1.cost < g2.cost ? wino_tiles<1>(c, g1, s) : wino_tiles<2>(c, g2, s);
}

hipError_t first_launch(const ConvCall &c, hipStream_t s) {
  const Args a = make_args(c);
  const int cout_pad = c.layer->cout_pad, bm = cout_pad % 64 == 0 ? 64 : 32;
  const dim3 grid((a.W + 31) / 32, (a.H + 7) / 8, (cout_pad / bm) * (c.batch < 1 ? 1 : c.batch));
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
  const bool head = c.head_out || c.head_outs;
  if (head && (L.cout_pad > 64 || c.out_pool)) return hipErrorInvalidValue;
  if (c.rgbda_depth) {
    if (!c.rgbda_rgba || c.C1 != 0 || L.cin_pad != 8 || head || c.out_pool) return hipErrorInvalidValue;
    return first_launch(c, s);
  }
  if (!L.wu || c.C0 % 16 || c.C1 % 16 || c.C0 + c.C1 != L.cin_pad) return hipErrorInvalidValue;
  if ((c.C1 || c.out_pool) && (c.H % 2 || c.W % 2)) return hipErrorInvalidValue;
  return wino_launch(c, s);
}

hipError_t launch_head(const void *x, int C, int H, int W, const ConvLayer &head, Prec p, float *out, hipStream_t s) {
  return launch_head16(x, C, H, W, head, p, out, s);
}

}  // namespace lnr
