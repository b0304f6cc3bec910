// Shared by the U-Net's convolution kernels: layer arguments, the tile walk, and
// direct loads from memory into LDS.
#pragma once

#include <hip/hip_runtime.h>

#include "lnr_internal.h"

namespace lnr {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// a value that every lane holds alike, in scalar registers
__device__ inline const char *uniform(const char *p) {
  const uint64_t v = (uint64_t)p;
  return (const char *)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}

// Up to 64 lanes x 16 (or 4) bytes from base + voff (per lane) straight into
// LDS: lane i's bytes go to LDS address lds + 16 i (4 i); the lanes outside
// `lanes` write nothing.  Called with every lane of the wave active.  The
// instruction is issued whatever the mask, so a wave can count its loads in
// flight.  The compiler does not see the LDS write: wait_loads() and a barrier
// come before the data are read.
// m0 is overwritten, which a clobber list cannot say (the register is reserved):
// no kernel with these loads may have another user of m0 (tests/test_kernel_asm.py
// looks at the compiled code).  exec is all ones before and after.
__device__ inline void load_lds16(const char *base, uint32_t voff, uint32_t lds, uint64_t lanes) {
  asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1"
               :
               : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(voff), "s"(uniform(base)), "s"(lanes)
               : "memory");
}
__device__ inline void load_lds4(const float *base, uint32_t voff, uint32_t lds, uint64_t lanes) {
  asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dword %1, %2\n\ts_mov_b64 exec, -1"
               :
               : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(voff), "s"(base), "s"(lanes)
               : "memory");
}
// until at most N of the wave's loads (the newest) are in flight
template <int N>
__device__ inline void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ inline uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

struct Args {
  const char *in0, *in1;     // channel blocks of H x W 16-byte units; of (H/2) x (W/2) units, read nearest-upsampled
  size_t in0_bs, in1_bs;     // bytes per image of a batch
  int C0, C1, H, W;
  const char *w;             // [channel group][chunk][32-channel tile][plane][tap][half][32 channels] units
  const float *bias, *wscale;
  int cout;
  char *out, *out_pool;
  size_t out_bs, pool_bs;
  int raw;                   // store the layer for head_kernel: float16 / bfloat16 or float32 values, not operands
  const float *head_w, *head_b;
  float *head_out;
  float *const *head_outs;
  const float *depth;        // first layer: the RGBDA images, rgbda_bs pixels apart
  const uint32_t *rgba;
  size_t rgbda_bs;
  int ntx, nty, ncz, ntiles;  // tiles: columns, rows, channel tiles, all of the batch
  int per, run;               // tiles per XCD, per workgroup
  int wgroup;                 // 32-channel tiles per group of the packed weights
};

// Tiles are listed channel tiles of a pixel tile next to each other, then
// columns, rows, images.  Consecutive workgroups go to the 8 XCDs in turn; each
// XCD takes one contiguous eighth of the list, a workgroup `run` consecutive
// tiles of it, so tiles that read the same pixels run on the same XCD at about
// the same time and share its L2.
struct Walk {
  int first, end;
};
__device__ inline Walk my_tiles(const Args &a) {
  const int per = a.per, x = (int)(blockIdx.x & 7);
  const int first = (int)(blockIdx.x >> 3) * a.run, end = first + a.run < per ? first + a.run : per;
  return {x * per + first, x * per + end < a.ntiles ? x * per + end : a.ntiles};
}
struct Tile {
  int ty, tx, cz, img;
};
__device__ inline Tile tile_at(const Args &a, int T) {
  // (the divisions run on the vector unit: back to scalar registers)
  Tile t;
  const int r = __builtin_amdgcn_readfirstlane(T / a.ncz);
  t.cz = T - r * a.ncz;
  const int q = __builtin_amdgcn_readfirstlane(r / a.ntx);
  t.tx = r - q * a.ntx;
  t.img = __builtin_amdgcn_readfirstlane(q / a.nty);
  t.ty = q - t.img * a.nty;
  return t;
}

Args make_args(const ConvCall &c) {
  const ConvLayer &L = *c.layer;
  Args a{};
  a.in0 = static_cast<const char *>(c.in0);
  a.in1 = static_cast<const char *>(c.in1);
  a.in0_bs = c.in0_bs;
  a.in1_bs = c.in1_bs;
  a.C0 = c.C0;
  a.C1 = c.C1;
  a.H = c.H;
  a.W = c.W;
  a.w = static_cast<const char *>(L.w);
  a.bias = L.bias;
  a.wscale = L.wscale;
  a.cout = L.cout;
  a.out = static_cast<char *>(c.out);
  a.out_pool = static_cast<char *>(c.out_pool);
  a.out_bs = c.out_bs;
  a.pool_bs = c.pool_bs;
  a.raw = c.raw_out ? 1 : 0;
  a.head_w = c.head_w;
  a.head_b = c.head_b;
  a.head_out = c.head_out;
  a.head_outs = c.head_outs;
  a.depth = c.rgbda_depth;
  a.rgba = c.rgbda_rgba;
  a.rgbda_bs = c.rgbda_bs;
  a.wgroup = channel_group(L.cout_pad) / 32;
  return a;
}
constexpr int kCUs = 256;  // of an MI355X (tile choice only)

// Tiles of a launch, run tiles per workgroup, the XCDs' shares whole groups of
// `group` tiles; returns the grid.
int set_tiles(Args &a, int TH, int channels, int cout_pad, int batch, int run, int group = 1) {
  a.ntx = (a.W + 31) / 32;
  a.nty = (a.H + TH - 1) / TH;
  a.ncz = cout_pad / channels;
  a.ntiles = a.ntx * a.nty * a.ncz * batch;
  a.run = run;
  a.per = ((a.ntiles + 7) / 8 + group - 1) / group * group;
  return 8 * ((a.per + run - 1) / run);
}

}  // namespace
}  // namespace lnr
