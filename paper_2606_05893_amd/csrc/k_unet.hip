// Learned Poisson warm start: a 3-D U-Net (levels of 16/32/64/128
// channels, 3x3x3 convolutions, average pooling down, nearest upsampling
// and concatenation up, 1x1x1 head) with BF16 activations and weights and
// FP32 accumulation on the CDNA4 matrix cores, plus its backward pass and
// an Adam optimiser with FP32 master weights.
//
// Tensors are channels-last (D, H, W, C) BF16; padding is circular in x, y
// and zero in z.  The 3x3x3 convolution is an implicit GEMM: M = voxels,
// N = output channels, K = 27 * C_in flattened as (tap, channel) and walked
// in chunks of 32 by v_mfma_f32_16x16x32_bf16 (lane l holds row l % 16 and
// k = 8 (l / 16) .. +7 of A and B; D rows 4 (l / 16) .. +3, column l % 16).
// The input tile of a workgroup is staged in LDS per slice of 16 channels.
// The backward-data convolution is the same kernel with the kernel flipped
// and the channel roles swapped; the weight gradient is a second GEMM whose
// reduction runs over voxels, staged through LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "pic.h"
#include "pic_ctx.h"
#include "pic_device.h"

struct pic_unet;

namespace pic {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned short bf16;  // storage

__device__ __forceinline__ float bf2f(bf16 h) {
  return __uint_as_float((unsigned)h << 16);
}
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
// The gradient word g (two BF16 values) where the activations y are positive.
__device__ __forceinline__ unsigned relu_mask2(unsigned g, unsigned y) {
  const unsigned lo = __uint_as_float(y << 16) > 0.f ? g & 0xffffu : 0u;
  const unsigned hi = __uint_as_float(y & 0xffff0000u) > 0.f ? g & 0xffff0000u : 0u;
  return lo | hi;
}
// Round to nearest even (the CDNA4 conversion instruction, two at a time).
__device__ __forceinline__ unsigned f2bf2(float lo, float hi) {
  const bf16x2v h = __builtin_convertvector((f2v){lo, hi}, bf16x2v);
  unsigned r;
  __builtin_memcpy(&r, &h, 4);
  return r;
}
__device__ __forceinline__ bf16 f2bf(float x) {
  return (bf16)(f2bf2(x, 0.0f) & 0xffffu);
}

__device__ __forceinline__ bf16x8 load8(const bf16* p) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}
struct Dims {
  int D, H, W;
  long long V;
};

// Vectors of 8 BF16 channels (16 B) for the data-movement kernels; voxel
// indices fit 32 bits for every supported grid.
__device__ __forceinline__ uint4 ld16(const bf16* p) {
  return *reinterpret_cast<const uint4*>(p);
}
__device__ __forceinline__ void st16(bf16* p, uint4 v) {
  *reinterpret_cast<uint4*>(p) = v;
}
__device__ __forceinline__ void unpack8(uint4 v, float* f) {
  const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f[2 * q] = __uint_as_float(w[q] << 16);
    f[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
  }
}
__device__ __forceinline__ void voxel_xyz(unsigned v, const Dims& d, int& x,
                                          int& y, int& z) {
  x = (int)(v % (unsigned)d.W);
  const unsigned r = v / (unsigned)d.W;
  y = (int)(r % (unsigned)d.H);
  z = (int)(r / (unsigned)d.H);
}

// Packed 3^3 weights, in the order the matrix instructions take them: per 16
// output channels, 16 input channels (slice) and tap row (oz, oy) two
// fragments of 64 lanes x 8 values, lane 16 (half + 2 slot) + channel.  The
// first holds the taps ox = slot, the second ox = 2 in slot 0 and zeros.  A
// wave's load of a fragment is 1 KB in a row; read from [channel][tap][in]
// rows, 32 bytes a row, the weights took more than half of the requests of
// the 48 -> 16 layer (562 -> 476 us at 128x128x512).
constexpr int kFrag = 512;
__host__ __device__ constexpr long long frag_at(int tile, int slices, int sl, int row) {
  return (((long long)tile * slices + sl) * 9 + row) * 2 * kFrag;
}
__host__ __device__ constexpr long long wpack(int co, int ci) {
  return frag_at(co / 16, ci / 16, 0, 0);
}

// The halo of a tile for one slice of 16 input channels (x and y periodic, z
// zero-padded), held in registers between its loads and its LDS stores
// (halo_load / halo_store; HV voxels of 32 B as two planes of 16-byte
// halves), so that the loads of the next slice can be in flight while the
// current one is computed.  UP: read from a tensor at half the dims as its
// nearest upsampling (fine voxel (z, y, x) takes coarse (z/2, y/2, x/2)).
template <int HX, int HY, int HZ, int NTH>
struct HaloRegs {
  static constexpr int HV = HX * HY * HZ;
  static constexpr int PER = (2 * HV + NTH - 1) / NTH;
  uint4 v[PER];
};

template <int HX, int HY, int HZ, int NTH, bool UP>
__device__ __forceinline__ void halo_load_c(HaloRegs<HX, HY, HZ, NTH>& r,
                                            const bf16* __restrict__ in, int C, int c0,
                                            const Dims& d, int x0, int y0, int z0) {
  constexpr int HV = HX * HY * HZ;
  const bool one = d.H >= HY && d.W >= HX;
#pragma unroll
  for (int m = 0; m < r.PER; ++m) {
    const int q = (int)threadIdx.x + m * NTH;
    const int hv = q >> 1, hh = q & 1;
    const int hx = hv % HX, hy = (hv / HX) % HY, hz = hv / (HX * HY);
    const int gz = z0 + hz - 1;
    r.v[m] = make_uint4(0, 0, 0, 0);
    if (q < 2 * HV && gz >= 0 && gz < d.D) {
      int gy = y0 + hy - 1, gx = x0 + hx - 1;
      if (one) {
        gy = gy < 0 ? gy + d.H : (gy >= d.H ? gy - d.H : gy);
        gx = gx < 0 ? gx + d.W : (gx >= d.W ? gx - d.W : gx);
      } else {
        gy = (gy + d.H) % d.H;
        gx = (gx + d.W) % d.W;
      }
      size_t gv;
      if constexpr (UP)
        gv = ((size_t)(gz >> 1) * (d.H >> 1) + (gy >> 1)) * (d.W >> 1) + (gx >> 1);
      else
        gv = ((size_t)gz * d.H + gy) * d.W + gx;
      r.v[m] = ld16(in + gv * C + c0 + hh * 8);
    }
  }
}

template <int HX, int HY, int HZ, int NTH>
__device__ __forceinline__ void halo_load(HaloRegs<HX, HY, HZ, NTH>& r,
                                          const bf16* __restrict__ in, int C,
                                          const Dims& d, int x0, int y0, int z0,
                                          int sl) {
  halo_load_c<HX, HY, HZ, NTH, false>(r, in, C, sl * 16, d, x0, y0, z0);
}

// Slice sl of 'in' (CIN channels), or with CU > 0 of the concatenation
// [up(in) (CU channels, half dims), skip (CIN - CU)].
template <int CIN, int CU, int HX, int HY, int HZ, int NTH>
__device__ __forceinline__ void halo_load_cat(HaloRegs<HX, HY, HZ, NTH>& r,
                                              const bf16* __restrict__ in,
                                              const bf16* __restrict__ skip,
                                              const Dims& d, int x0, int y0, int z0,
                                              int sl) {
  if (CU > 0 && sl * 16 < CU)
    halo_load_c<HX, HY, HZ, NTH, true>(r, in, CU, sl * 16, d, x0, y0, z0);
  else if (CU > 0)
    halo_load_c<HX, HY, HZ, NTH, false>(r, skip, CIN - CU, sl * 16 - CU, d, x0, y0, z0);
  else
    halo_load_c<HX, HY, HZ, NTH, false>(r, in, CIN, sl * 16, d, x0, y0, z0);
}

template <int HX, int HY, int HZ, int NTH>
__device__ __forceinline__ void halo_store(uint4* lds, const HaloRegs<HX, HY, HZ, NTH>& r) {
  constexpr int HV = HX * HY * HZ;
#pragma unroll
  for (int m = 0; m < r.PER; ++m) {
    const int q = (int)threadIdx.x + m * NTH;
    if (q < 2 * HV) lds[(q & 1) * HV + (q >> 1)] = r.v[m];
  }
}

// The halo of slice sl straight into LDS (16-byte direct loads, no
// registers): voxel-major, lds[2 voxel + half], which is the lanes' order, as
// such a load writes lane after lane.  Planes outside the grid are zeroed.
// halo_wait, then a barrier, before it is read.
template <int HX, int HY, int HZ, int NTH, bool UP>
__device__ __forceinline__ void halo_to_lds_c(uint4* lds, const bf16* __restrict__ in,
                                              int C, int c0, const Dims& d, int x0,
                                              int y0, int z0) {
  constexpr int HV = HX * HY * HZ;
  constexpr int PER = (2 * HV + NTH - 1) / NTH;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool one = d.H >= HY && d.W >= HX;
  const int hh = threadIdx.x & 1;
  int hx = (int)(threadIdx.x >> 1) % HX, hy = (int)(threadIdx.x >> 1) / HX % HY,
      hz = (int)(threadIdx.x >> 1) / (HX * HY);
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int q = (int)threadIdx.x + m * NTH;
    if (m > 0) {  // NTH / 2 voxels on
      constexpr int D = NTH / 2;
      hx += D % HX;
      if (hx >= HX) { hx -= HX; ++hy; }
      hy += D / HX % HY;
      if (hy >= HY) { hy -= HY; ++hz; }
      hz += D / (HX * HY);
    }
    const int gz = z0 + hz - 1;
    if (q >= 2 * HV) continue;
    if (gz >= 0 && gz < d.D) {
      int gy = y0 + hy - 1, gx = x0 + hx - 1;
      if (one) {
        gy = gy < 0 ? gy + d.H : (gy >= d.H ? gy - d.H : gy);
        gx = gx < 0 ? gx + d.W : (gx >= d.W ? gx - d.W : gx);
      } else {
        gy = (gy + d.H) % d.H;
        gx = (gx + d.W) % d.W;
      }
      size_t gv;
      if constexpr (UP)
        gv = ((size_t)(gz >> 1) * (d.H >> 1) + (gy >> 1)) * (d.W >> 1) + (gx >> 1);
      else
        gv = ((size_t)gz * d.H + gy) * d.W + gx;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(in + gv * C + c0 + hh * 8),
          (__attribute__((address_space(3))) void*)(lds + m * NTH + wave * 64), 16, 0, 0);
    } else {
      lds[q] = make_uint4(0, 0, 0, 0);
    }
  }
}

template <int CIN, int CU, int HX, int HY, int HZ, int NTH>
__device__ __forceinline__ void halo_to_lds(uint4* lds, const bf16* __restrict__ in,
                                            const bf16* __restrict__ skip,
                                            const Dims& d, int x0, int y0, int z0,
                                            int sl) {
  if (CU > 0 && sl * 16 < CU)
    halo_to_lds_c<HX, HY, HZ, NTH, true>(lds, in, CU, sl * 16, d, x0, y0, z0);
  else if (CU > 0)
    halo_to_lds_c<HX, HY, HZ, NTH, false>(lds, skip, CIN - CU, sl * 16 - CU, d, x0, y0, z0);
  else
    halo_to_lds_c<HX, HY, HZ, NTH, false>(lds, in, CIN, sl * 16, d, x0, y0, z0);
}

// This wave's direct loads have landed (vmcnt 0).
__device__ __forceinline__ void halo_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// out = conv(in) for the backward-data shapes of the decoders' concatenations
// (48, 96 and 192 output channels).  A workgroup owns 48 output channels of a
// tile of 16 (x) x 8 x 4 voxels; per slice of 16 input channels it stages the
// tile's halo (x and y periodic, z zero-padded) in LDS, the two 8-channel
// halves of a voxel in separate planes, and the slice's weights in operand
// order.  A K-chunk of 32 is two taps x 16 channels (lane group g = lane / 16:
// tap 2c + g / 2, channels 8 (g % 2) .. +7).  Each wave owns eight rows of 16
// voxels and the three column tiles (the product taken as W X, so a lane ends
// with four consecutive channels of one voxel): 8 + 3 LDS reads for 24
// products, below the LDS rate.  The coarse part (the first 2 CIN channels) and
// the skip part of the gradient go to tensors of their own.  With one slice the weights are staged once and the workgroup
// runs over many tiles.
//
// Bound: matrix products and the staging they wait for.  With the weights read
// from the cache for every four rows the kernel waited on those loads: 16 -> 48
// at 128x128x512 832 us, 32 -> 96 at half of that 651, 64 -> 192 at a quarter
// 590; 356, 207 and 106 now.
template <int CIN>
__global__ void __launch_bounds__(256, 2) k_conv3w(const bf16* __restrict__ in,
                                                   const bf16* __restrict__ Wk,
                                                   bf16* __restrict__ gup,
                                                   bf16* __restrict__ gskip, Dims d, int nsp) {
  constexpr int NT = 3, MT = 8, TY = 8, TZ = 4;
  constexpr int HX = 18, HY = TY + 2, HZ = TZ + 2;
  constexpr int HV = HX * HY * HZ;
  constexpr int NS = CIN / 16;
  __shared__ uint4 lds[HV * 2];
  __shared__ uint4 lw[14 * NT * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntx = (d.W + 15) / 16, nty = (d.H + TY - 1) / TY, ntz = (d.D + TZ - 1) / TZ;
  const int ntiles = ntx * nty * ntz;
  // 2 CIN channels of the coarse part, CIN of the skip part.
  constexpr int groups = CIN / 16, CU = 2 * CIN;
  // The channel groups of one run of tiles are neighbours on one XCD.
  const int bi = (int)xcd_block(blockIdx.x, gridDim.x);
  const int cg = bi % groups, wg = bi / groups;
  const int t0 = (int)((long long)ntiles * wg / nsp);
  const int t1 = (int)((long long)ntiles * (wg + 1) / nsp);
  const int kg = lane >> 4, rl = lane & 15;
  auto stage_w = [&](int sl) {
    for (int e = threadIdx.x; e < 14 * NT * 64; e += 256) {
      const int l = e & 63, cn = e >> 6, nt = cn % NT, ch = cn / NT;
      const int tap = 2 * ch + (l >> 5);
      uint4 v = make_uint4(0, 0, 0, 0);
      if (tap < 27)
        v = ld16(Wk + frag_at(cg * NT + nt, NS, sl, tap / 3) + (tap % 3 == 2 ? kFrag : 0) +
                 (((tap % 3 & 1) * 2 + ((l >> 4) & 1)) * 16 + (l & 15)) * 8);
      lw[e] = v;
    }
  };
  if (NS == 1) stage_w(0);
  const uint4* la = lds + (kg & 1) * HV + rl;
  HaloRegs<HX, HY, HZ, 256> hr;
  auto load = [&](int t, int sl) {
    const int tx = t % ntx, r = t / ntx;
    halo_load(hr, in, CIN, d, tx * 16, (r % nty) * TY, (r / nty) * TZ, sl);
  };
  // The next tile's halo is in flight during the products where the weights
  // stay; restaging them beside it would spill.
  if (NS == 1 && t0 < t1) load(t0, 0);
  for (int t = t0; t < t1; ++t) {
    f4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[m][n] = f4{0.f, 0.f, 0.f, 0.f};
    for (int sl = 0; sl < NS; ++sl) {
      if (NS > 1) load(t, sl);
      halo_store(lds, hr);
      if (NS > 1) stage_w(sl);
      __syncthreads();
      if (NS == 1 && t + 1 < t1) load(t + 1, 0);
#pragma unroll 2
      for (int ch = 0; ch < 14; ++ch) {
        // Chunk 13 holds tap 26 and a slot of zero weights.
        const int tap = min(2 * ch + (kg >> 1), 26);
        const int oz = tap / 9, oy = (tap / 3) % 3, ox = tap % 3;
        bf16x8 b[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const uint4 w = lw[(ch * NT + n) * 64 + lane];
          __builtin_memcpy(&b[n], &w, 16);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          // Rows wave * 8 + m: y = m, z = wave.
          const uint4 w = la[((wave + oz) * HY + m + oy) * HX + ox];
          bf16x8 a;
          __builtin_memcpy(&a, &w, 16);
#pragma unroll
          for (int n = 0; n < NT; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[n], a, acc[m][n], 0, 0, 0);
        }
      }
      __syncthreads();
    }
    const int tx = t % ntx, r = t / ntx;
    const int gx = tx * 16 + rl, y0 = (r % nty) * TY, gz = (r / nty) * TZ + wave;
    if (gz < d.D && gx < d.W)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (y0 + m >= d.H) continue;
        const size_t v = ((size_t)gz * d.H + y0 + m) * d.W + gx;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          // Four consecutive channels of one voxel, of one part.
          const int c = cg * 48 + n * 16, c4 = c + 4 * kg;
          uint2 w;
          w.x = f2bf2(acc[m][n][0], acc[m][n][1]);
          w.y = f2bf2(acc[m][n][2], acc[m][n][3]);
          *reinterpret_cast<uint2*>(c < CU ? gup + v * CU + c4 : gskip + v * CIN + (c4 - CU)) = w;
        }
      }
  }
}

// out = act(conv(in) + bias), register-blocked over output rows; with a mask
// (backward data: the activations the gradient goes to) the stored values are
// zeroed where it is not positive.  A
// workgroup owns an output tile of 16 (x) x 4WY x 4WZ voxels and stages its
// halo per slice of 16 input channels in LDS (32 bytes a voxel).  Each wave
// owns one 16-channel tile of C_out and a block of 4 x 4 output rows (y, z)
// of 16 voxels.  An input row of the halo is one MFMA operand whose K of 32
// is two x-offsets of the row (x offsets 0 and 1, or 2 and a slot whose
// weights are zero), so one LDS read of an input row serves every output
// row it reaches, up to nine (three z by three y offsets), and the wave's
// 18 weight fragments of the slice (3 z x 3 y offsets x 2 x-pairs) stay in
// registers: per slice a wave reads 6 x 6 x 2 input fragments for 288
// MFMAs (a quarter of the second pair's products are with zero weights),
// against one read per MFMA when the operand is formed per tap.  The
// product is taken as W X (rows: output channels, columns: voxels), so a
// lane ends with four consecutive channels of one voxel, stored as one
// 8-byte word.
//
// With CU > 0 the input is the decoder's concatenation [up(in), skip]
// formed in the staging (in: CU channels at half the dims; skip: CIN - CU
// channels), so the concatenated tensor is never written.
template <int CIN, int COUT, int WY, int WZ, int CU = 0, bool MASK = false>
__global__ void __launch_bounds__(64 * (COUT / 16) * WY * WZ) k_conv3r(
    const bf16* __restrict__ in, const bf16* __restrict__ skip,
    const bf16* __restrict__ Wk, const float* __restrict__ bias,
    bf16* __restrict__ out, Dims d, int relu, const bf16* __restrict__ mask) {
  static_assert(CU % 16 == 0 && CU < CIN, "concatenation split on slices");
  constexpr int NTC = COUT / 16, RY = 4, RZ = 4;
  constexpr int TX = 16, TY = WY * RY, TZ = WZ * RZ;
  constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;
  constexpr int HV = HX * HY * HZ;
  constexpr int NTH = 64 * NTC * WY * WZ;
  constexpr int NS = CIN / 16;
  static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channel multiples of 16");
  constexpr int NB = NS > 1 ? 2 : 1;
  __shared__ uint4 lds[NB][HV * 2];
  // The wave index is uniform: scalar, so the per-row tests are scalar.
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nt = wave % NTC, sp = wave / NTC;
  const int wy = sp % WY, wz = sp / WY;
  const int ntx = (d.W + TX - 1) / TX, nty = (d.H + TY - 1) / TY;
  int bi = (int)xcd_block(blockIdx.x, gridDim.x);
  const int tx = bi % ntx;
  bi /= ntx;
  const int ty = bi % nty, tz = bi / nty;
  const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
  const int kg = lane >> 4, rl = lane & 15;
  const int half = kg & 1, slot = kg >> 1;
  const bf16* wlane = Wk + lane * 8;
  f4 acc[RZ][RY];
#pragma unroll
  for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
    for (int yo = 0; yo < RY; ++yo) acc[zo][yo] = f4{0.f, 0.f, 0.f, 0.f};
  // The next slice's halo goes to the other buffer while this one is
  // computed.
  halo_to_lds<CIN, CU, HX, HY, HZ, NTH>(lds[0], in, skip, d, x0, y0, z0, 0);
  for (int sl = 0; sl < NS; ++sl) {
    // Weight fragments of the slice: taps ox = slot, and ox = 2 in slot 0
    // (zero in slot 1).
    bf16x8 wa[3][3], wb[3][3];
#pragma unroll
    for (int oz = 0; oz < 3; ++oz)
#pragma unroll
      for (int oy = 0; oy < 3; ++oy) {
        const bf16* w = wlane + frag_at(nt, NS, sl, oz * 3 + oy);
        wa[oz][oy] = load8(w);
        wb[oz][oy] = load8(w + kFrag);
      }
    halo_wait();
    __syncthreads();
    if (sl + 1 < NS)
      halo_to_lds<CIN, CU, HX, HY, HZ, NTH>(lds[(sl + 1) % NB], in, skip, d, x0, y0, z0, sl + 1);
    const uint4* lh = lds[sl % NB] + half + 2 * rl;
#pragma unroll
    for (int iz = 0; iz < RZ + 2; ++iz)
#pragma unroll
      for (int iy = 0; iy < RY + 2; ++iy) {
        const int hv = ((wz * RZ + iz) * HY + (wy * RY + iy)) * HX;
        // Slot 1 of the second fragment reads the x + 2 voxel too (its
        // weights are zero): no divergent load.
        bf16x8 fa, fb;
        {
          const uint4 w0 = lh[2 * (hv + slot)], w1 = lh[2 * (hv + 2)];
          __builtin_memcpy(&fa, &w0, 16);
          __builtin_memcpy(&fb, &w1, 16);
        }
        // The products of one fragment go to distinct accumulators, so the
        // MFMAs of a pass are independent.
#pragma unroll
        for (int oz = 0; oz < 3; ++oz)
#pragma unroll
          for (int oy = 0; oy < 3; ++oy) {
            const int zo = iz - oz, yo = iy - oy;
            if (zo >= 0 && zo < RZ && yo >= 0 && yo < RY)
              acc[zo][yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[oz][oy], fa, acc[zo][yo], 0, 0, 0);
          }
#pragma unroll
        for (int oz = 0; oz < 3; ++oz)
#pragma unroll
          for (int oy = 0; oy < 3; ++oy) {
            const int zo = iz - oz, yo = iy - oy;
            if (zo >= 0 && zo < RZ && yo >= 0 && yo < RY)
              acc[zo][yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[oz][oy], fb, acc[zo][yo], 0, 0, 0);
          }
      }
  }
  // Lane: voxel x0 + rl, channels nt * 16 + 4 kg .. +3.
  const int x = x0 + rl;
  const int c0 = nt * 16 + 4 * kg;
  float bv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) bv[j] = bias ? bias[c0 + j] : 0.0f;
  if (x < d.W) {
    // The mask words of all rows in flight before the first is needed.
    uint2 mw[RZ][RY];
    if constexpr (MASK)
#pragma unroll
      for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
        for (int yo = 0; yo < RY; ++yo) {
          const int gy = min(y0 + wy * RY + yo, d.H - 1), gz = min(z0 + wz * RZ + zo, d.D - 1);
          mw[zo][yo] = *reinterpret_cast<const uint2*>(
              mask + (((size_t)gz * d.H + gy) * d.W + x) * COUT + c0);
        }
#pragma unroll
    for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
      for (int yo = 0; yo < RY; ++yo) {
        const int gy = y0 + wy * RY + yo, gz = z0 + wz * RZ + zo;
        if (gy >= d.H || gz >= d.D) continue;
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = acc[zo][yo][j] + bv[j];
          if (relu) v[j] = fmaxf(v[j], 0.0f);
        }
        uint2 w;
        w.x = f2bf2(v[0], v[1]);
        w.y = f2bf2(v[2], v[3]);
        const size_t o = (((size_t)gz * d.H + gy) * d.W + x) * COUT + c0;
        if constexpr (MASK) {
          w.x = relu_mask2(w.x, mw[zo][yo].x);
          w.y = relu_mask2(w.y, mw[zo][yo].y);
        }
        *reinterpret_cast<uint2*>(out + o) = w;
      }
  }
}

// k_conv3r for 16 output channels as a persistent kernel: as many
// workgroups as the GPU holds at once, each taking a contiguous run of
// tiles (of one XCD's range, so that neighbouring tiles share its L2), its
// (tile, slice) items in turn; with one slice the weight fragments are
// loaded once per workgroup.
//
// Bound: the matrix products (a quarter with zero weights) take 216 of the
// 476 us of 48 -> 16 at 128x128x512 at the clock they run at; the rest is the
// loads a workgroup waits for that its neighbour does not cover.  The halo
// goes straight to LDS, so the registers (242 a lane) let two workgroups
// share a compute unit; held in registers beside the products (351 a lane,
// one workgroup) it took 840 us, of which the loads and LDS stores were 430
// (16 -> 16: 231 -> 166).  The mask of the backward form costs 55 us in its
// epilogue, as a pass of its own 126.
template <int CIN, int CU = 0, bool MASK = false>
__global__ void __launch_bounds__(256, 2) k_conv3p(
    const bf16* __restrict__ in, const bf16* __restrict__ skip,
    const bf16* __restrict__ Wk, const float* __restrict__ bias,
    bf16* __restrict__ out, Dims d, int relu, const bf16* __restrict__ mask) {
  static_assert(CU % 16 == 0 && CU < CIN && CIN % 16 == 0, "channel slices");
  constexpr int RY = 4, RZ = 4, WY = 2;
  constexpr int TX = 16, TY = 8, TZ = 8;
  constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;
  constexpr int HV = HX * HY * HZ;
  constexpr int NTH = 256;
  constexpr int NS = CIN / 16;
  __shared__ uint4 lds[HV * 2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wy = wave % WY, wz = wave / WY;
  const int ntx = (d.W + TX - 1) / TX, nty = (d.H + TY - 1) / TY;
  const int ntiles = ntx * nty * ((d.D + TZ - 1) / TZ);
  const int per = (ntiles + (int)gridDim.x - 1) / (int)gridDim.x;
  const int lo = (int)xcd_block(blockIdx.x, gridDim.x) * per;
  const int hi = lo + per < ntiles ? lo + per : ntiles;
  if (lo >= hi) return;
  const int nitems = (hi - lo) * NS;
  const int kg = lane >> 4, rl = lane & 15;
  const int half = kg & 1, slot = kg >> 1;
  const bf16* wlane = Wk + lane * 8;
  const int c0 = 4 * kg;
  float bv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) bv[j] = bias ? bias[c0 + j] : 0.0f;
  auto origin = [&](int t, int& x0, int& y0, int& z0) {
    x0 = (t % ntx) * TX;
    y0 = ((t / ntx) % nty) * TY;
    z0 = (t / (ntx * nty)) * TZ;
  };
  f4 acc[RZ][RY];
#pragma unroll
  for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
    for (int yo = 0; yo < RY; ++yo) acc[zo][yo] = f4{0.f, 0.f, 0.f, 0.f};
  bf16x8 wa[3][3], wb[3][3];
  auto load_w = [&](int sl) {
#pragma unroll
    for (int oz = 0; oz < 3; ++oz)
#pragma unroll
      for (int oy = 0; oy < 3; ++oy) {
        const bf16* w = wlane + frag_at(0, NS, sl, oz * 3 + oy);
        wa[oz][oy] = load8(w);
        wb[oz][oy] = load8(w + kFrag);
      }
  };
  if (NS == 1) load_w(0);
  for (int j = 0; j < nitems; ++j) {
    const int t = lo + j / NS, sl = j % NS;
    {
      int x0, y0, z0;
      origin(t, x0, y0, z0);
      halo_to_lds<CIN, CU, HX, HY, HZ, NTH>(lds, in, skip, d, x0, y0, z0, sl);
    }
    if (NS > 1) load_w(sl);
    halo_wait();
    __syncthreads();
    const uint4* lh = lds + half + 2 * (rl + (wz * RZ * HY + wy * RY) * HX);
    // The input rows in a ring of three, each read two rows ahead of its
    // MFMAs so that the LDS latency is covered.
    constexpr int NP = (RZ + 2) * (RY + 2);
    uint4 ring[3][2];
    auto fetch = [&](int p, uint4 (&r)[2]) {
      const int hv = ((p / (RY + 2)) * HY + p % (RY + 2)) * HX;
      r[0] = lh[2 * (hv + slot)];
      r[1] = lh[2 * (hv + 2)];
    };
    fetch(0, ring[0]);
    fetch(1, ring[1]);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int iz = p / (RY + 2), iy = p % (RY + 2);
      if (p + 2 < NP) fetch(p + 2, ring[(p + 2) % 3]);
      {
        bf16x8 fa, fb;
        __builtin_memcpy(&fa, &ring[p % 3][0], 16);
        __builtin_memcpy(&fb, &ring[p % 3][1], 16);
#pragma unroll
        for (int oz = 0; oz < 3; ++oz)
#pragma unroll
          for (int oy = 0; oy < 3; ++oy) {
            const int zo = iz - oz, yo = iy - oy;
            if (zo >= 0 && zo < RZ && yo >= 0 && yo < RY)
              acc[zo][yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[oz][oy], fa, acc[zo][yo], 0, 0, 0);
          }
#pragma unroll
        for (int oz = 0; oz < 3; ++oz)
#pragma unroll
          for (int oy = 0; oy < 3; ++oy) {
            const int zo = iz - oz, yo = iy - oy;
            if (zo >= 0 && zo < RZ && yo >= 0 && yo < RY)
              acc[zo][yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[oz][oy], fb, acc[zo][yo], 0, 0, 0);
          }
      }
    }
    if (sl == NS - 1) {
      int x0, y0, z0;
      origin(t, x0, y0, z0);
      const int x = x0 + rl;
      // The mask words of all rows in flight before the first is needed.
      uint2 mw[RZ][RY];
      if constexpr (MASK)
#pragma unroll
        for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
          for (int yo = 0; yo < RY; ++yo) {
            const int gx = min(x, d.W - 1), gy = min(y0 + wy * RY + yo, d.H - 1),
                      gz = min(z0 + wz * RZ + zo, d.D - 1);
            mw[zo][yo] = *reinterpret_cast<const uint2*>(
                mask + (((size_t)gz * d.H + gy) * d.W + gx) * 16 + c0);
          }
#pragma unroll
      for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
        for (int yo = 0; yo < RY; ++yo) {
          const int gy = y0 + wy * RY + yo, gz = z0 + wz * RZ + zo;
          if (x < d.W && gy < d.H && gz < d.D) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              v[q] = acc[zo][yo][q] + bv[q];
              if (relu) v[q] = fmaxf(v[q], 0.0f);
            }
            uint2 w;
            w.x = f2bf2(v[0], v[1]);
            w.y = f2bf2(v[2], v[3]);
            if constexpr (MASK) {
              w.x = relu_mask2(w.x, mw[zo][yo].x);
              w.y = relu_mask2(w.y, mw[zo][yo].y);
            }
            *reinterpret_cast<uint2*>(out + (((size_t)gz * d.H + gy) * d.W + x) * 16 + c0) = w;
          }
          acc[zo][yo] = f4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __syncthreads();
  }
}

// Four rows of 16 bf16 read from LDS transposed (ds_read_b64_tr_b16): within
// 16 lanes, lane 4r + c supplies the address of row r's elements 4c .. 4c + 3
// and lane i receives element i of the four rows.
typedef short s4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4v* lds_s4;
__device__ __forceinline__ bf16x8 lds_tr8(const char* r0, const char* r4) {
  s4v v[2];
  v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)r0);
  v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)r4);
  bf16x8 r;
  __builtin_memcpy(&r, v, 16);
  return r;
}

// Weight gradient dW[co][tap][ci] += sum_v g[v][co] x[v + tap][ci] as a GEMM
// whose K runs over voxels: an MFMA takes 32 voxels (two rows of 16, P planes
// apart) of 16 output channels of g against the same rows of x shifted by the
// tap (with CU > 0 x is the decoder's concatenation formed in the staging, as in
// the forward pass), and a wave keeps the 27 taps' 16 x 16 sums of one (co tile, ci slice)
// pair in registers over every tile its workgroup visits.  The voxel-major
// operands come straight from the channels-last halo by transposing LDS reads,
// so a tap's shift is an address offset.  A wave holds the g rows of a YB x P
// block of row pairs and reads each x row pair of the surrounding halo once
// per x shift for every (dy, dz) that reaches it: 3 (YB + 2)(P + 2) + YB P
// fragment reads for 27 YB P products.  A workgroup's waves take WM tiles of
// output channels and split the tile's y rows WK ways; their sums meet in LDS
// and go to dW as one atomic add per element and workgroup.
//
// Bound: the latency between two barriers (staging stores, fragment reads,
// products) at two wavefronts a SIMD, which the 27 accumulators cost; the LDS
// reads alone take 0.95 of the matrix time with YB = 2 and 0.7 with YB = 4.
// YB = 4 for 32 output channels spilled beside the prefetched tile (96 -> 32
// at 64x64x256: 358 us against 203), three wavefronts a SIMD spilled
// everywhere (16 -> 16: 414 against 158), and without the prefetch 48 -> 16
// took 806 us against 491.  At 128x128x512, against one 32-voxel chunk at a
// time gathered through LDS by 2-byte reads: 16 -> 16 1944 -> 158 us, 48 -> 16
// 4979 -> 491, 96 -> 32 1298 -> 203, 64 -> 64 194 -> 79.
template <int COUT>
struct WgTile {
  static constexpr int M = COUT / 16;
  static constexpr int WM = M < 4 ? M : 4, WK = 4 / WM;
  static constexpr int YB = M <= 2 ? 2 : 4, P = 2;
  static constexpr int TY = YB * WK, TZ = 2 * P;
  static constexpr int HY = TY + 2, HZ = TZ + 2, HV = 18 * HY * HZ;
  static constexpr int GV = 16 * TY * TZ;
};

// The bias sums of the workgroup's four waves (wave w: output channel tile
// w % wm) joined in LDS and added by one request: the 16 floats of a tile are
// one line, and an add per wave and row from every workgroup queued on it for
// 100 us.
__device__ __forceinline__ void bias_out(float* lds, f4 accb, float* db, int wm, bool on) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((lane & 15) == 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) lds[wave * 16 + 4 * (lane >> 4) + j] = accb[j];
  __syncthreads();
  if (on && (int)threadIdx.x < 16 * wm) {
    float v = 0.f;
    for (int w = threadIdx.x >> 4; w < 4; w += wm) v += lds[w * 16 + (threadIdx.x & 15)];
    atomicAdd(&db[threadIdx.x], v);
  }
  __syncthreads();
}

template <int CIN, int COUT, int CU>
__global__ void __launch_bounds__(256, 2) k_wgrad3(const bf16* __restrict__ x,
                                                   const bf16* __restrict__ skip,
                                                   const bf16* __restrict__ g,
                                                   float* __restrict__ dW,
                                                   float* __restrict__ db, Dims d, int nsp) {
  using T = WgTile<COUT>;
  constexpr int WM = T::WM, WK = T::WK, YB = T::YB, P = T::P;
  constexpr int TY = T::TY, TZ = T::TZ, HY = T::HY, HZ = T::HZ, HV = T::HV, GV = T::GV;
  constexpr int kRed = WK > 1 ? WM * 27 * 256 * 4 / 16 : 0;  // sums' exchange, uint4
  constexpr int kStage = 2 * HV + 2 * GV * WM;
  // Halo of x (two planes of 16-byte halves), then g per co tile alike.
  __shared__ uint4 lds[kStage > kRed ? kStage : kRed];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % WM, wk = wave / WM;
  // The pairs of one run of tiles are neighbours, so they share its lines in
  // one XCD's L2.
  constexpr int kPairs = (CIN / 16) * (COUT / 16 / WM);
  const int bi = (int)xcd_block(blockIdx.x, gridDim.x);
  const int pair = bi % kPairs, wg = bi / kPairs;
  const int sl = pair % (CIN / 16), mg = pair / (CIN / 16) * WM;
  const int ntx = (d.W + 15) / 16, nty = (d.H + TY - 1) / TY, ntz = (d.D + TZ - 1) / TZ;
  const int ntiles = ntx * nty * ntz;
  const char* lx = reinterpret_cast<const char*>(lds);
  const char* lg = lx + (size_t)(2 * HV + 2 * GV * wm) * 16;
  // This lane's part of a transposed read: row (q >> 2) of four voxels, 8-byte
  // part q & 3; lane group kg takes voxels 8 (kg & 1) of the pair's row kg >> 1.
  const int q = lane & 15, kg = lane >> 4;
  const int vx = 8 * (kg & 1) + (q >> 2);
  const int offx = ((q >> 1) & 1) * HV * 16 + (q & 1) * 8 +
                   (((kg >> 1) * P * HY + wk * YB) * 18 + vx) * 16;
  const int offg = ((q >> 1) & 1) * GV * 16 + (q & 1) * 8 +
                   (((kg >> 1) * P * TY + wk * YB) * 16 + vx) * 16;
  f4 acc[27];
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  f4 accb = f4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  // Neighbouring tiles share halo voxels: a contiguous run per workgroup.
  const int t0 = (int)((long long)ntiles * wg / nsp);
  const int t1 = (int)((long long)ntiles * (wg + 1) / nsp);
  // The next tile's loads are in flight while the current one is multiplied.
  constexpr int PER = 2 * GV * WM / 256;
  HaloRegs<18, HY, HZ, 256> hr;
  uint4 gr[PER];
  auto load = [&](int t) {
    const int tx = t % ntx, r = t / ntx;
    const int x0 = tx * 16, y0 = (r % nty) * TY, z0 = (r / nty) * TZ;
    halo_load_cat<CIN, CU>(hr, x, skip, d, x0, y0, z0, sl);
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int e = (int)threadIdx.x + m * 256;
      const int c8 = e % (2 * WM), v = e / (2 * WM);
      const int gx = x0 + (v & 15), gy = y0 + (v >> 4) % TY, gz = z0 + (v >> 4) / TY;
      gr[m] = make_uint4(0, 0, 0, 0);
      if (gx < d.W && gy < d.H && gz < d.D)
        gr[m] = ld16(g + (((size_t)gz * d.H + gy) * d.W + gx) * COUT + mg * 16 + c8 * 8);
    }
  };
  if (t0 < t1) load(t0);
  for (int t = t0; t < t1; ++t) {
    halo_store(lds, hr);
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int e = (int)threadIdx.x + m * 256;
      lds[2 * HV + (e % (2 * WM)) * GV + e / (2 * WM)] = gr[m];
    }
    __syncthreads();
    if (t + 1 < t1) load(t + 1);
    bf16x8 a[YB][P];
#pragma unroll
    for (int y = 0; y < YB; ++y)
#pragma unroll
      for (int z = 0; z < P; ++z) {
        const char* p = lg + offg + (z * TY + y) * 16 * 16;
        a[y][z] = lds_tr8(p, p + 64);
      }
#pragma unroll
    for (int hz = 0; hz < P + 2; ++hz)
#pragma unroll
      for (int hy = 0; hy < YB + 2; ++hy)
#pragma unroll
        for (int ox = 0; ox < 3; ++ox) {
          const char* p = lx + offx + ((hz * HY + hy) * 18 + ox) * 16;
          const bf16x8 b = lds_tr8(p, p + 64);
#pragma unroll
          for (int oz = 0; oz < 3; ++oz)
#pragma unroll
            for (int oy = 0; oy < 3; ++oy) {
              const int y = hy - oy, z = hz - oz;
              if (y >= 0 && y < YB && z >= 0 && z < P)
                acc[(oz * 3 + oy) * 3 + ox] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    a[y][z], b, acc[(oz * 3 + oy) * 3 + ox], 0, 0, 0);
            }
        }
    // The bias gradient: the same rows against columns of ones.
    if (CIN == 16 || sl == 0)
#pragma unroll
      for (int y = 0; y < YB; ++y)
#pragma unroll
        for (int z = 0; z < P; ++z)
          accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[y][z], ones, accb, 0, 0, 0);
    __syncthreads();
  }
  bias_out(reinterpret_cast<float*>(lds), accb, db + mg * 16, WM, sl == 0);
  if constexpr (WK > 1) {
    f4* red = reinterpret_cast<f4*>(lds) + wm * 27 * 64 + lane;
    for (int k = 1; k < WK; ++k) {
      if (wk == k)
#pragma unroll
        for (int t = 0; t < 27; ++t) red[t * 64] = acc[t];
      __syncthreads();
      if (wk == 0)
#pragma unroll
        for (int t = 0; t < 27; ++t) acc[t] = acc[t] + red[t * 64];
      __syncthreads();
    }
  }
  if (wk) return;
  const int co0 = (mg + wm) * 16 + 4 * kg, ci = sl * 16 + q;
#pragma unroll
  for (int t = 0; t < 27; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      atomicAdd(&dW[(long long)(co0 + j) * (27 * CIN) + t * CIN + ci], acc[t][j]);
}

// First layer (2 input channels): FP32 arithmetic, 16 outputs per voxel.
// The weights are indexed uniformly across the wave, so they come through
// the scalar cache as operands of the vector FMAs.
__global__ void __launch_bounds__(256) k_conv_first(
    const float* __restrict__ in, const float* __restrict__ W,  // [16][27][2]
    const float* __restrict__ b, bf16* __restrict__ out, Dims d) {
  const unsigned v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= (unsigned long long)d.V) return;
  int x, y, z;
  voxel_xyz(v, d, x, y, z);
  float acc[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) acc[c] = b[c];
#pragma unroll 3
  for (int tap = 0; tap < 27; ++tap) {
    const int zz = z + tap / 9 - 1;
    int yy = y + (tap / 3) % 3 - 1, xx = x + tap % 3 - 1;
    yy = yy < 0 ? yy + d.H : (yy >= d.H ? yy - d.H : yy);
    xx = xx < 0 ? xx + d.W : (xx >= d.W ? xx - d.W : xx);
    float2 i2 = make_float2(0.f, 0.f);
    if (zz >= 0 && zz < d.D)
      i2 = reinterpret_cast<const float2*>(in)[((unsigned)zz * d.H + yy) * d.W + xx];
#pragma unroll
    for (int c = 0; c < 16; ++c)
      acc[c] = fmaf(W[c * 54 + tap * 2 + 1], i2.y, fmaf(W[c * 54 + tap * 2], i2.x, acc[c]));
  }
  unsigned w[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float a0 = acc[2 * q] > 0.f ? acc[2 * q] : 0.f;
    const float a1 = acc[2 * q + 1] > 0.f ? acc[2 * q + 1] : 0.f;
    w[q] = (unsigned)f2bf(a0) | ((unsigned)f2bf(a1) << 16);
  }
  st16(out + (size_t)v * 16, make_uint4(w[0], w[1], w[2], w[3]));
  st16(out + (size_t)v * 16 + 8, make_uint4(w[4], w[5], w[6], w[7]));
}

// dW and db of the first layer, the same way: an FP32 input value is the exact
// sum of three BF16 ones (8 bits of its 24 each), so the products with the BF16
// gradient stay exact and are summed in FP32.  A halo voxel is 16 bytes: three
// parts of each of its two channels and two zeros, and a transposed read of 32
// bytes takes two x neighbours at once, columns 8 s + 3 c + part for shift s:
// x shifts -1 and 0 in one product, +1 in another (its second half, shift +2,
// is dropped).  18 products per row pair and (dy, dz), against 27 sums over
// all voxels in turn on the vector units, which read g 27 times: 1207 us at
// 128x128x512, 189 now.
__global__ void __launch_bounds__(256, 2) k_wgrad_first(const float* __restrict__ in,
                                                        const bf16* __restrict__ g,
                                                        float* __restrict__ dW,
                                                        float* __restrict__ db, Dims d, int nsp) {
  using T = WgTile<16>;
  constexpr int YB = T::YB, P = T::P, TY = T::TY, TZ = T::TZ, HY = T::HY;
  constexpr int HV = T::HV, GV = T::GV;
  // One voxel of slack: the last row's shift +2 (dropped) reads past it.
  constexpr int kRed = 18 * 256 * 4 / 16;
  constexpr int kStage = HV + 1 + 2 * GV;
  __shared__ uint4 lds[kStage > kRed ? kStage : kRed];
  const int lane = threadIdx.x & 63, wk = threadIdx.x >> 6;
  const int ntx = (d.W + 15) / 16, nty = (d.H + TY - 1) / TY, ntz = (d.D + TZ - 1) / TZ;
  const int ntiles = ntx * nty * ntz;
  const int wg = (int)xcd_block(blockIdx.x, gridDim.x);
  const char* lx = reinterpret_cast<const char*>(lds);
  const char* lg = lx + (size_t)(HV + 1) * 16;
  const int q = lane & 15, kg = lane >> 4;
  const int vx = 8 * (kg & 1) + (q >> 2);
  const int offx = (((kg >> 1) * P * HY + wk * YB) * 18 + vx) * 16 + (q & 3) * 8;
  const int offg = ((q >> 1) & 1) * GV * 16 + (q & 1) * 8 +
                   (((kg >> 1) * P * TY + wk * YB) * 16 + vx) * 16;
  f4 acc[18], accb = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 18; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  if (threadIdx.x == 0) lds[HV] = make_uint4(0, 0, 0, 0);
  constexpr int PX = (HV + 255) / 256, PG = 2 * GV / 256;
  float2 xr[PX];
  uint4 gr[PG];
  auto load = [&](int t) {
    const int tx = t % ntx, r = t / ntx;
    const int x0 = tx * 16, y0 = (r % nty) * TY, z0 = (r / nty) * TZ;
#pragma unroll
    for (int m = 0; m < PX; ++m) {
      const int hv = (int)threadIdx.x + m * 256;
      const int hx = hv % 18, hy = (hv / 18) % HY, gz = z0 + hv / (18 * HY) - 1;
      xr[m] = make_float2(0.f, 0.f);
      if (hv < HV && gz >= 0 && gz < d.D) {
        const int gy = (y0 + hy - 1 + d.H) % d.H, gx = (x0 + hx - 1 + d.W) % d.W;
        xr[m] = reinterpret_cast<const float2*>(in)[((size_t)gz * d.H + gy) * d.W + gx];
      }
    }
#pragma unroll
    for (int m = 0; m < PG; ++m) {
      const int e = (int)threadIdx.x + m * 256;
      const int v = e >> 1;
      const int gx = x0 + (v & 15), gy = y0 + (v >> 4) % TY, gz = z0 + (v >> 4) / TY;
      gr[m] = make_uint4(0, 0, 0, 0);
      if (gx < d.W && gy < d.H && gz < d.D)
        gr[m] = ld16(g + (((size_t)gz * d.H + gy) * d.W + gx) * 16 + (e & 1) * 8);
    }
  };
  // Three parts of a value; an infinity or NaN is its first part alone.
  auto split = [](float v, unsigned short (&p)[3]) {
    p[0] = f2bf(v);
    const float r1 = v - bf2f(p[0]);
    const bool fin = fabsf(bf2f(p[0])) < INFINITY;
    p[1] = fin ? f2bf(r1) : (bf16)0;
    p[2] = fin ? f2bf(r1 - bf2f(p[1])) : (bf16)0;
  };
  const int t0 = (int)((long long)ntiles * wg / nsp);
  const int t1 = (int)((long long)ntiles * (wg + 1) / nsp);
  if (t0 < t1) load(t0);
  for (int t = t0; t < t1; ++t) {
#pragma unroll
    for (int m = 0; m < PX; ++m) {
      const int hv = (int)threadIdx.x + m * 256;
      unsigned short a[3], b[3];
      split(xr[m].x, a);
      split(xr[m].y, b);
      if (hv < HV)
        lds[hv] = make_uint4(a[0] | (unsigned)a[1] << 16, a[2] | (unsigned)b[0] << 16,
                             b[1] | (unsigned)b[2] << 16, 0u);
    }
#pragma unroll
    for (int m = 0; m < PG; ++m) {
      const int e = (int)threadIdx.x + m * 256;
      lds[HV + 1 + (e & 1) * GV + (e >> 1)] = gr[m];
    }
    __syncthreads();
    if (t + 1 < t1) load(t + 1);
    bf16x8 a[YB][P];
#pragma unroll
    for (int y = 0; y < YB; ++y)
#pragma unroll
      for (int z = 0; z < P; ++z) {
        const char* p = lg + offg + (z * TY + y) * 16 * 16;
        a[y][z] = lds_tr8(p, p + 64);
        accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[y][z], ones, accb, 0, 0, 0);
      }
#pragma unroll
    for (int hz = 0; hz < P + 2; ++hz)
#pragma unroll
      for (int hy = 0; hy < YB + 2; ++hy)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const char* p = lx + offx + ((hz * HY + hy) * 18 + 2 * s2) * 16;
          const bf16x8 b = lds_tr8(p, p + 64);
#pragma unroll
          for (int oz = 0; oz < 3; ++oz)
#pragma unroll
            for (int oy = 0; oy < 3; ++oy) {
              const int y = hy - oy, z = hz - oz;
              if (y >= 0 && y < YB && z >= 0 && z < P)
                acc[(oz * 3 + oy) * 2 + s2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    a[y][z], b, acc[(oz * 3 + oy) * 2 + s2], 0, 0, 0);
            }
        }
    __syncthreads();
  }
  bias_out(reinterpret_cast<float*>(lds), accb, db, 1, true);
  f4* red = reinterpret_cast<f4*>(lds) + lane;
  for (int k = 1; k < 4; ++k) {
    if (wk == k)
#pragma unroll
      for (int t = 0; t < 18; ++t) red[t * 64] = acc[t];
    __syncthreads();
    if (wk == 0)
#pragma unroll
      for (int t = 0; t < 18; ++t) acc[t] = acc[t] + red[t * 64];
    __syncthreads();
  }
  if (wk) return;
  // Column 8 s + 3 c + part of product pair s2: the three parts' sums join in
  // the first part's lane.
  const int c = (q & 7) / 3, shift = q >> 3;
  const bool own = (q & 7) == 0 || (q & 7) == 3;
#pragma unroll
  for (int t = 0; t < 18; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = acc[t][j] + (__shfl_down(acc[t][j], 1) + __shfl_down(acc[t][j], 2));
      const int ox = 2 * (t & 1) + shift;
      if (own && ox < 3) atomicAdd(&dW[(4 * kg + j) * 54 + ((t >> 1) * 3 + ox) * 2 + c], v);
    }
}

// Average pooling 2^3 (out dims d = input dims / 2), 8 channels a thread.
__global__ void k_pool(const bf16* __restrict__ in, bf16* __restrict__ out,
                       Dims d, int C) {
  const unsigned G = (unsigned)C / 8;
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (unsigned long long)d.V * G) return;
  const unsigned v = t / G, g = t % G;
  int x, y, z;
  voxel_xyz(v, d, x, y, z);
  const unsigned W2 = 2 * d.W, H2 = 2 * d.H;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int e = 0; e < 2; ++e) {
        float f[8];
        unpack8(ld16(in + ((size_t)((2 * z + a) * H2 + 2 * y + b) * W2 + 2 * x + e) * C + 8 * g), f);
#pragma unroll
        for (int q = 0; q < 8; ++q) s[q] = s[q] + f[q];
      }
  unsigned w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    w[q] = (unsigned)f2bf(s[2 * q] * 0.125f) | ((unsigned)f2bf(s[2 * q + 1] * 0.125f) << 16);
  st16(out + (size_t)v * C + 8 * g, make_uint4(w[0], w[1], w[2], w[3]));
}

// Pre-activation gradient of an encoder level's output: the skip part of the
// decoder's concatenation gradient plus the gradient through pooling, gcoarse[parent] / 8, where the output y is
// positive (fine dims d), 8 channels a thread.
__global__ void k_pool_bwd_add(const bf16* __restrict__ gc, const bf16* __restrict__ gskip,
                               const bf16* __restrict__ y8, bf16* __restrict__ gpre, Dims d,
                               int C) {
  const unsigned G = (unsigned)C / 8;
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (unsigned long long)d.V * G) return;
  const unsigned v = t / G, g = t % G;
  int x, y, z;
  voxel_xyz(v, d, x, y, z);
  const unsigned p = ((unsigned)(z / 2) * (d.H / 2) + y / 2) * (d.W / 2) + x / 2;
  const uint4 m = ld16(y8 + (size_t)v * C + 8 * g);
  float a[8], b[8];
  unpack8(ld16(gskip + (size_t)v * C + 8 * g), a);
  unpack8(ld16(gc + (size_t)p * C + 8 * g), b);
  const unsigned mw[4] = {m.x, m.y, m.z, m.w};
  unsigned w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    w[q] = relu_mask2(f2bf2(a[2 * q] + b[2 * q] * 0.125f, a[2 * q + 1] + b[2 * q + 1] * 0.125f),
                      mw[q]);
  st16(gpre + (size_t)v * C + 8 * g, make_uint4(w[0], w[1], w[2], w[3]));
}

// The concatenation gradient's coarse part summed over the 8 children, where
// the coarse output yc is positive (coarse dims dc); 8 channels a thread.
__global__ void k_split_up(const bf16* __restrict__ gup, int Cu,
                           const bf16* __restrict__ yc, bf16* __restrict__ gpre, Dims dc) {
  const unsigned G = (unsigned)Cu / 8;
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (unsigned long long)dc.V * G) return;
  const unsigned p = t / G, g = t % G;
  int x, y, z;
  voxel_xyz(p, dc, x, y, z);
  const unsigned W2 = 2 * dc.W, H2 = 2 * dc.H;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int e = 0; e < 2; ++e) {
        float f[8];
        unpack8(ld16(gup + ((size_t)((2 * z + a) * H2 + 2 * y + b) * W2 + 2 * x + e) * Cu + 8 * g), f);
#pragma unroll
        for (int q = 0; q < 8; ++q) s[q] = s[q] + f[q];
      }
  const uint4 m = ld16(yc + (size_t)p * Cu + 8 * g);
  const unsigned mw[4] = {m.x, m.y, m.z, m.w};
  unsigned w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = relu_mask2(f2bf2(s[2 * q], s[2 * q + 1]), mw[q]);
  st16(gpre + (size_t)p * Cu + 8 * g, make_uint4(w[0], w[1], w[2], w[3]));
}

// Head: out[v] = sum_c w[c] y[v][c] + b, FP32 output.
__global__ void k_head(const bf16* __restrict__ y, const float* __restrict__ w,
                       float* __restrict__ out, long long V) {
  const unsigned v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= (unsigned long long)V) return;
  float f[16];
  unpack8(ld16(y + (size_t)v * 16), f);
  unpack8(ld16(y + (size_t)v * 16 + 8), f + 8);
  float s = w[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) s = s + w[c] * f[c];
  out[v] = s;
}

// Loss (mean squared error) partials and the output gradient.
__global__ void k_mse(const float* __restrict__ out, const float* __restrict__ t,
                      float* __restrict__ gout, long long V,
                      double* __restrict__ part) {
  __shared__ double s[256];
  double a = 0.0;
  for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < V;
       v += (long long)gridDim.x * blockDim.x) {
    const float df = out[v] - t[v];
    a += (double)df * df;
    gout[v] = 2.0f * df / (float)V;
  }
  s[threadIdx.x] = a;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// Residual loss: q = A e on the unknown planes (z >= k0), e = c - t there
// and zero below k0 and beyond the top plane; A is the scaled 7-point
// operator (x, y periodic; a Neumann bottom, k0 = 0, mirrors plane 1).
// Block partials of sum q^2.
__device__ __forceinline__ float res_e(const float* c, const float* t, int z,
                                       unsigned row, int k0, int D) {
  return (z >= k0 && z < D) ? c[row] - t[row] : 0.0f;
}

__global__ void k_res_q(const float* __restrict__ c, const float* __restrict__ t,
                        float* __restrict__ q, Dims d, int k0,
                        double* __restrict__ part) {
  __shared__ double s[256];
  double a = 0.0;
  const unsigned plane = (unsigned)d.H * d.W;
  for (unsigned long long vv = blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x;
       vv < (unsigned long long)d.V; vv += (unsigned long long)gridDim.x * blockDim.x) {
    const unsigned v = (unsigned)vv;
    int x, y, z;
    voxel_xyz(v, d, x, y, z);
    float r = 0.0f;
    if (z >= k0) {
      const unsigned base = (unsigned)z * plane;
      const int xm = x ? x - 1 : d.W - 1, xp = x + 1 < d.W ? x + 1 : 0;
      const int ym = y ? y - 1 : d.H - 1, yp = y + 1 < d.H ? y + 1 : 0;
      const float e0 = c[v] - t[v];
      float xy = res_e(c, t, z, base + y * d.W + xm, k0, d.D) +
                 res_e(c, t, z, base + y * d.W + xp, k0, d.D);
      xy = xy + (res_e(c, t, z, base + ym * d.W + x, k0, d.D) +
                 res_e(c, t, z, base + yp * d.W + x, k0, d.D));
      float zz;
      if (z == 0)
        zz = 2.0f * res_e(c, t, 1, v + plane, k0, d.D);
      else
        zz = res_e(c, t, z - 1, v - plane, k0, d.D) +
             res_e(c, t, z + 1, v + plane, k0, d.D);
      r = 6.0f * e0 - xy - zz;
    }
    q[v] = r;
    a += (double)r * r;
  }
  s[threadIdx.x] = a;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// gout = (2 / V) A^T q on the unknown planes (row z-1 = 0 of a Neumann
// bottom reaches plane 1 with coefficient 2).
__global__ void k_res_g(const float* __restrict__ q, float* __restrict__ gout,
                        Dims d, int k0, float scale) {
  const unsigned v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= (unsigned long long)d.V) return;
  int x, y, z;
  voxel_xyz(v, d, x, y, z);
  float g = 0.0f;
  if (z >= k0) {
    const unsigned plane = (unsigned)d.H * d.W, base = (unsigned)z * plane;
    const int xm = x ? x - 1 : d.W - 1, xp = x + 1 < d.W ? x + 1 : 0;
    const int ym = y ? y - 1 : d.H - 1, yp = y + 1 < d.H ? y + 1 : 0;
    float xy = q[base + y * d.W + xm] + q[base + y * d.W + xp];
    xy = xy + (q[base + ym * d.W + x] + q[base + yp * d.W + x]);
    float zz = 0.0f;
    if (z - 1 >= k0) zz = (z - 1 == 0 ? 2.0f : 1.0f) * q[v - plane];
    if (z + 1 < d.D) zz = zz + q[v + plane];
    g = (6.0f * q[v] - xy - zz) * scale;
  }
  gout[v] = g;
}

// Head backward: the last layer's pre-activation gradient gout[v] w[c] where
// y > 0; dw[c] += sum gout y; db += sum.
__global__ void __launch_bounds__(256) k_head_bwd(
    const float* __restrict__ gout, const bf16* __restrict__ y,
    const float* __restrict__ w, bf16* __restrict__ gy, float* __restrict__ dw,
    long long V) {
  __shared__ float s[17][256];
  float acc[17];
#pragma unroll
  for (int c = 0; c < 17; ++c) acc[c] = 0.f;
  for (unsigned long long v = blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x;
       v < (unsigned long long)V; v += (unsigned long long)gridDim.x * blockDim.x) {
    const float go = gout[v];
    float f[16];
    const uint4 ya = ld16(y + (size_t)v * 16), yb = ld16(y + (size_t)v * 16 + 8);
    unpack8(ya, f);
    unpack8(yb, f + 8);
    const unsigned m[8] = {ya.x, ya.y, ya.z, ya.w, yb.x, yb.y, yb.z, yb.w};
    unsigned o[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = relu_mask2(f2bf2(go * w[2 * q], go * w[2 * q + 1]), m[q]);
    st16(gy + (size_t)v * 16, make_uint4(o[0], o[1], o[2], o[3]));
    st16(gy + (size_t)v * 16 + 8, make_uint4(o[4], o[5], o[6], o[7]));
#pragma unroll
    for (int c = 0; c < 16; ++c) acc[c] = acc[c] + go * f[c];
    acc[16] = acc[16] + go;
  }
#pragma unroll
  for (int c = 0; c < 17; ++c) s[c][threadIdx.x] = acc[c];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o)
      for (int c = 0; c < 17; ++c) s[c][threadIdx.x] += s[c][threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x < 17) atomicAdd(&dw[threadIdx.x], s[threadIdx.x][0]);
}

__global__ void k_sum_d(const double* __restrict__ part, int n, double* out) {
  __shared__ double s[256];
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) a += part[i];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = s[0];
}

// Adam with FP32 master weights (Kingma & Ba): bias-corrected moments.
__global__ void k_adam(float* __restrict__ p, float* __restrict__ m,
                       float* __restrict__ v, const float* __restrict__ g,
                       long long n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// BF16 fragments (see kFrag) of a layer's weights W[co][tap][ci]: forward Wk
// of its co output channels, backward-data Wd, whose output channels are ci
// and whose taps are mirrored.
__global__ void k_pack_w(const float* __restrict__ W, int ci_n, int co_n,
                         bf16* __restrict__ Wk, bf16* __restrict__ Wd) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long n = wpack(co_n, ci_n);
  if (i >= 2 * n) return;
  const bool back = i >= n;
  const int in_n = back ? co_n : ci_n;
  long long q = back ? i - n : i;
  bf16* dst = (back ? Wd : Wk) + q;
  const int e = (int)(q % 8), lane = (int)(q / 8 % 64), second = (int)(q / kFrag % 2);
  q /= 2 * kFrag;
  const int row = (int)(q % 9), sl = (int)(q / 9 % (in_n / 16)), tile = (int)(q / 9 / (in_n / 16));
  const int kg = lane / 16, slot = kg / 2;
  const int o = tile * 16 + lane % 16, c = sl * 16 + (kg & 1) * 8 + e;
  const int tap = row * 3 + (second ? 2 : slot);
  if (second && slot) {
    *dst = 0;
    return;
  }
  *dst = f2bf(back ? W[((long long)c * 27 + 26 - tap) * ci_n + o]
                   : W[((long long)o * 27 + tap) * ci_n + c]);
}

}  // namespace
}  // namespace pic

// ============================================================================
// Host side.
// ============================================================================
namespace {

using pic::bf16;
using pic::Dims;

struct LayerSpec {
  int ci, co;
};
constexpr int kNL = 14;
constexpr LayerSpec kLayers[kNL] = {
    {2, 16},   {16, 16},  {16, 32}, {32, 32}, {32, 64},  {64, 64},  {64, 128},
    {128, 128}, {192, 64}, {64, 64}, {96, 32}, {32, 32},  {48, 16},  {16, 16}};
enum { E0A, E0B, E1A, E1B, E2A, E2B, BA, BB, D2A, D2B, D1A, D1B, D0A, D0B };
// Level of each layer's voxels.
constexpr int kLevel[kNL] = {0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 1, 1, 0, 0};

long long param_count() {
  long long n = 0;
  for (int l = 0; l < kNL; ++l) n += (long long)kLayers[l].co * 27 * kLayers[l].ci + kLayers[l].co;
  return n + 17;
}

// Workgroups (and partial sums) of the loss.
constexpr int kLossParts = 2048;

}  // namespace

struct pic_unet {
  hipStream_t stream;
  int D, H, W;                 // maximum grid
  char* ws;
  size_t bytes;
  long long np;                // parameters
  float *p, *m, *v, *g;        // master, moments, gradient
  long long woff[kNL], boff[kNL], hoff;
  bf16 *wk[kNL], *wd[kNL];     // BF16 forward / backward-data weights
  // Activations (BF16, channels-last).
  float* x_in;                 // (V0, 2) FP32 input
  bf16 *y[kNL];                // layer outputs
  bf16 *p0, *p1, *p2;          // pooled
  float *out, *gout, *target;
  // Gradient scratch per level: buffers of the level's widest tensor.
  bf16 *ga[4], *gb[4], *gs[4];
  double* dpart;
  int t;                       // Adam step
  int loss_mode, loss_k0;      // PIC_UNET_LOSS_*, first unknown plane
  float* q;                    // residual of the error (residual loss)
  std::string err;
};

namespace {

struct Carve {
  char* base;
  size_t off;
  template <typename T>
  T* take(long long n) {
    off = (off + 255) / 256 * 256;
    T* r = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += (size_t)(n > 0 ? n : 1) * sizeof(T);
    return r;
  }
};

size_t unet_carve(pic_unet* u, char* base) {
  Carve cv{base, 0};
  const long long V0 = (long long)u->D * u->H * u->W;
  long long Vl[4];
  for (int l = 0; l < 4; ++l) Vl[l] = V0 >> (3 * l);
  u->np = param_count();
  u->p = cv.take<float>(u->np);
  u->m = cv.take<float>(u->np);
  u->v = cv.take<float>(u->np);
  u->g = cv.take<float>(u->np);
  long long off = 0;
  for (int l = 0; l < kNL; ++l) {
    u->woff[l] = off;
    off += (long long)kLayers[l].co * 27 * kLayers[l].ci;
    u->boff[l] = off;
    off += kLayers[l].co;
    u->wk[l] = cv.take<bf16>(pic::wpack(kLayers[l].co, kLayers[l].ci));
    u->wd[l] = cv.take<bf16>(pic::wpack(kLayers[l].ci, kLayers[l].co));
  }
  u->hoff = off;
  u->x_in = cv.take<float>(2 * V0);
  for (int l = 0; l < kNL; ++l) u->y[l] = cv.take<bf16>(Vl[kLevel[l]] * kLayers[l].co);
  u->p0 = cv.take<bf16>(Vl[1] * 16);
  u->p1 = cv.take<bf16>(Vl[2] * 32);
  u->p2 = cv.take<bf16>(Vl[3] * 64);
  u->out = cv.take<float>(V0);
  u->gout = cv.take<float>(V0);
  u->target = cv.take<float>(V0);
  const int widest[4] = {48, 96, 192, 128};
  for (int l = 0; l < 4; ++l) {
    u->ga[l] = cv.take<bf16>(Vl[l] * widest[l]);
    u->gb[l] = cv.take<bf16>(Vl[l] * widest[l]);
    u->gs[l] = cv.take<bf16>(Vl[l] * widest[l]);
  }
  u->dpart = cv.take<double>(kLossParts + 1);
  u->q = cv.take<float>(V0);
  return cv.off + 256;
}

inline unsigned nb(long long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

Dims dims_at(const pic_unet* u, int D, int H, int W, int level) {
  Dims d;
  d.D = D >> level;
  d.H = H >> level;
  d.W = W >> level;
  d.V = (long long)d.D * d.H * d.W;
  return d;
}

// Workgroups of k_conv3p<CIN, CU> the current device holds at once.
template <int CIN, int CU, bool MASK>
unsigned conv3p_slots() {
  static unsigned cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!cached[dev]) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pic::k_conv3p<CIN, CU, MASK>, 256, 0) !=
            hipSuccess || per_cu < 1)
      per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
      cus = 256;
    cached[dev] = (unsigned)(per_cu * cus);
  }
  return cached[dev];
}

template <int CIN, int CU, bool MASK>
void conv3p_launch(hipStream_t st, const bf16* in, const bf16* skip, const bf16* Wk,
                   const float* b, bf16* out, Dims d, int relu, const bf16* mask) {
  const long long ntiles = (long long)((d.W + 15) / 16) * ((d.H + 7) / 8) * ((d.D + 7) / 8);
  const unsigned slots = conv3p_slots<CIN, CU, MASK>();
  const unsigned grid = ntiles < (long long)slots ? (unsigned)ntiles : slots;
  pic::k_conv3p<CIN, CU, MASK><<<grid, 256, 0, st>>>(in, skip, Wk, b, out, d, relu, mask);
}

// The register-blocked k_conv3r for 32 to 128 output channels, its persistent
// form k_conv3p for 16.
template <int CIN, int COUT, bool MASK>
void conv_launch(hipStream_t st, const bf16* in, const bf16* Wk, const float* b,
                 bf16* out, Dims d, int relu, const bf16* mask) {
  if constexpr (COUT == 16) {
    conv3p_launch<CIN, 0, MASK>(st, in, nullptr, Wk, b, out, d, relu, mask);
  } else {
    constexpr int WY = 1, WZ = COUT >= 64 ? 1 : 2;
    constexpr int TY = 4 * WY, TZ = 4 * WZ;
    const long long nbk = (long long)((d.W + 15) / 16) * ((d.H + TY - 1) / TY) *
                          ((d.D + TZ - 1) / TZ);
    pic::k_conv3r<CIN, COUT, WY, WZ, 0, MASK>
        <<<(unsigned)nbk, 64 * (COUT / 16) * WY * WZ, 0, st>>>(in, nullptr, Wk, b, out, d, relu, mask);
  }
}

// Dispatch of the (C_in, C_out) pairs the network and its backward use.
bool conv(hipStream_t st, int cin, int cout, const bf16* in, const bf16* Wk,
          const float* b, bf16* out, Dims d, int relu, const bf16* mask = nullptr) {
#define PIC_CONV(CI, CO)                                                   \
  if (cin == CI && cout == CO) {                                           \
    if (mask)                                                              \
      conv_launch<CI, CO, true>(st, in, Wk, b, out, d, relu, mask);        \
    else                                                                   \
      conv_launch<CI, CO, false>(st, in, Wk, b, out, d, relu, nullptr);    \
    return true;                                                           \
  }
  PIC_CONV(16, 16) PIC_CONV(16, 32) PIC_CONV(32, 32) PIC_CONV(32, 64)
  PIC_CONV(64, 64) PIC_CONV(64, 128) PIC_CONV(128, 128)
  // backward-data shapes (channels swapped)
  PIC_CONV(32, 16) PIC_CONV(64, 32) PIC_CONV(128, 64)
#undef PIC_CONV
  return false;
}

// Gradient of a decoder's concatenation (cin channels in, 3 cin out), its part
// of the upsampled coarse output and its skip part.  One round of resident
// workgroups (two on each of 256 CUs) over the channel groups with one slice,
// whose weights stay; else runs half as long.  A training sample's gradient on
// 128x128x512 with 256 / 512 / 768 / 1024 workgroups for 16 channels: 5922 /
// 5796 / 5830 / 5807 us; with 256 / 512 / 1024 / 2048 for 32 and 64: 5979 /
// 5808 / 5815 / 5807.
bool conv_cat_grad(hipStream_t st, int cin, const bf16* in, const bf16* Wk, bf16* gup, bf16* gskip,
                   Dims d) {
  const long long ntiles = (long long)((d.W + 15) / 16) * ((d.H + 7) / 8) * ((d.D + 3) / 4);
  const int groups = cin / 16;
  const int nsp = (int)std::min<long long>(ntiles, (cin == 16 ? 512 : 1024) / groups);
  const unsigned grid = (unsigned)(groups * nsp);
  if (cin == 16)
    pic::k_conv3w<16><<<grid, 256, 0, st>>>(in, Wk, gup, gskip, d, nsp);
  else if (cin == 32)
    pic::k_conv3w<32><<<grid, 256, 0, st>>>(in, Wk, gup, gskip, d, nsp);
  else if (cin == 64)
    pic::k_conv3w<64><<<grid, 256, 0, st>>>(in, Wk, gup, gskip, d, nsp);
  else
    return false;
  return true;
}

// Decoder convolution of [up(coarse) (CU channels), skip] without the
// concatenated tensor (inference).
template <int CIN, int COUT, int CU>
void conv_upcat_launch(hipStream_t st, const bf16* coarse, const bf16* skip,
                       const bf16* Wk, const float* b, bf16* out, Dims d) {
  if constexpr (COUT == 16) {
    conv3p_launch<CIN, CU, false>(st, coarse, skip, Wk, b, out, d, 1, nullptr);
  } else {
    constexpr int WY = 1, WZ = COUT == 64 ? 1 : 2;
    constexpr int TY = 4 * WY, TZ = 4 * WZ;
    const long long nbk = (long long)((d.W + 15) / 16) * ((d.H + TY - 1) / TY) *
                          ((d.D + TZ - 1) / TZ);
    pic::k_conv3r<CIN, COUT, WY, WZ, CU><<<(unsigned)nbk, 64 * (COUT / 16) * WY * WZ, 0, st>>>(
        coarse, skip, Wk, b, out, d, 1, nullptr);
  }
}

// One round of resident workgroups (two on each of 256 CUs, as the kernels'
// launch bounds have it) over all (co, ci) pairs, at least two tiles each: every
// workgroup ends with 27 x 256 atomic adds per pair.  A training sample's
// gradient with 256 / 512 / 768 / 1024 workgroups: 6477 / 5813 / 6135 / 6055 us
// on 128x128x512, 1616 / 1639 / 1709 / 1779 on 128x128x64; below that the same.
template <int COUT>
long long wgrad_runs(Dims d, int pairs) {
  using T = pic::WgTile<COUT>;
  const long long ntiles = (long long)((d.W + 15) / 16) * ((d.H + T::TY - 1) / T::TY) *
                           ((d.D + T::TZ - 1) / T::TZ);
  return std::max(1LL, std::min<long long>(512 / pairs, (ntiles + 1) / 2));
}

// dW and db of a layer with input x, or with CU > 0 the concatenation of up(x)
// and skip.
template <int CIN, int COUT, int CU>
void wgrad_launch(hipStream_t st, const bf16* x, const bf16* skip, const bf16* g, float* dW,
                  float* db, Dims d) {
  const int pairs = (CIN / 16) * ((COUT / 16) / pic::WgTile<COUT>::WM);
  const long long runs = wgrad_runs<COUT>(d, pairs);
  pic::k_wgrad3<CIN, COUT, CU><<<(unsigned)(pairs * runs), 256, 0, st>>>(x, skip, g, dW, db, d,
                                                                         (int)runs);
}

bool wgrad(hipStream_t st, int cin, int cout, const bf16* x, const bf16* skip, const bf16* g,
           float* dW, float* db, Dims d) {
#define PIC_WG(CI, CO, CU)                                                 \
  if (cin == CI && cout == CO) {                                           \
    wgrad_launch<CI, CO, CU>(st, x, skip, g, dW, db, d);                   \
    return true;                                                           \
  }
  PIC_WG(16, 16, 0) PIC_WG(16, 32, 0) PIC_WG(32, 32, 0) PIC_WG(32, 64, 0) PIC_WG(64, 64, 0)
  PIC_WG(64, 128, 0) PIC_WG(128, 128, 0) PIC_WG(192, 64, 128) PIC_WG(96, 32, 64)
  PIC_WG(48, 16, 32)
#undef PIC_WG
  return false;
}

void pack_weights(pic_unet* u) {
  for (int l = 0; l < kNL; ++l) {
    const LayerSpec& s = kLayers[l];
    if (l == E0A) continue;  // FP32 first layer
    pic::k_pack_w<<<nb(2 * pic::wpack(s.co, s.ci)), 256, 0, u->stream>>>(
        u->p + u->woff[l], s.ci, s.co, u->wk[l], u->wd[l]);
  }
}

// Forward pass of a D x H x W grid (input already in x_in); out -> u->out.
// The decoders form their concatenations in the staging.
bool unet_forward(pic_unet* u, int D, int H, int W) {
  hipStream_t st = u->stream;
  Dims d0 = dims_at(u, D, H, W, 0), d1 = dims_at(u, D, H, W, 1),
       d2 = dims_at(u, D, H, W, 2), d3 = dims_at(u, D, H, W, 3);
  const float* P = u->p;
  pic::k_conv_first<<<nb(d0.V), 256, 0, st>>>(u->x_in, P + u->woff[E0A],
                                             P + u->boff[E0A], u->y[E0A], d0);
  bool ok = true;
  auto L = [&](int l, const bf16* in, Dims d) {
    ok = ok && conv(st, kLayers[l].ci, kLayers[l].co, in, u->wk[l],
                    P + u->boff[l], u->y[l], d, 1);
  };
  L(E0B, u->y[E0A], d0);
  pic::k_pool<<<nb(d1.V * 2), 256, 0, st>>>(u->y[E0B], u->p0, d1, 16);
  L(E1A, u->p0, d1);
  L(E1B, u->y[E1A], d1);
  pic::k_pool<<<nb(d2.V * 4), 256, 0, st>>>(u->y[E1B], u->p1, d2, 32);
  L(E2A, u->p1, d2);
  L(E2B, u->y[E2A], d2);
  pic::k_pool<<<nb(d3.V * 8), 256, 0, st>>>(u->y[E2B], u->p2, d3, 64);
  L(BA, u->p2, d3);
  L(BB, u->y[BA], d3);
  conv_upcat_launch<192, 64, 128>(st, u->y[BB], u->y[E2B], u->wk[D2A], P + u->boff[D2A],
                                  u->y[D2A], d2);
  L(D2B, u->y[D2A], d2);
  conv_upcat_launch<96, 32, 64>(st, u->y[D2B], u->y[E1B], u->wk[D1A], P + u->boff[D1A],
                                u->y[D1A], d1);
  L(D1B, u->y[D1A], d1);
  conv_upcat_launch<48, 16, 32>(st, u->y[D1B], u->y[E0B], u->wk[D0A], P + u->boff[D0A],
                                u->y[D0A], d0);
  L(D0B, u->y[D0A], d0);
  pic::k_head<<<nb(d0.V), 256, 0, st>>>(u->y[D0B], P + u->hoff, u->out, d0.V);
  return ok;
}

// Backward pass from u->gout into u->g (zeroed here).
bool unet_backward(pic_unet* u, int D, int H, int W) {
  hipStream_t st = u->stream;
  Dims d[4];
  for (int l = 0; l < 4; ++l) d[l] = dims_at(u, D, H, W, l);
  hipMemsetAsync(u->g, 0, u->np * sizeof(float), st);
  float* G = u->g;
  bool ok = true;
  // Head; ga[0]: pre-activation gradient of the last layer.
  pic::k_head_bwd<<<512, 256, 0, st>>>(u->gout, u->y[D0B], u->p + u->hoff,
                                       u->ga[0], G + u->hoff, d[0].V);
  // Layer backward: the pre-activation gradient g -> dW, db and the input
  // gradient, with mask the pre-activation gradient of the layer whose output
  // the mask is.
  auto back = [&](int l, const bf16* g, const bf16* in, bf16* gx, const bf16* mask) {
    const LayerSpec& s = kLayers[l];
    const Dims& dd = d[kLevel[l]];
    ok = ok && wgrad(st, s.ci, s.co, in, nullptr, g, G + u->woff[l], G + u->boff[l], dd);
    ok = ok && conv(st, s.co, s.ci, g, u->wd[l], nullptr, gx, dd, 0, mask);
  };
  // Decoder of level lv (layers A, B; the coarser output up and the level's
  // encoder output skip, cs channels): the gradient of skip is left in gs[lv],
  // the pre-activation gradient of up in ga[lv + 1].
  auto decoder = [&](int lv, int A, int B, int up, int skip, int cs) {
    back(B, u->ga[lv], u->y[A], u->gb[lv], u->y[A]);
    ok = ok && wgrad(st, 3 * cs, cs, u->y[up], u->y[skip], u->gb[lv], G + u->woff[A],
                     G + u->boff[A], d[lv]);
    ok = ok && conv_cat_grad(st, cs, u->gb[lv], u->wd[A], u->ga[lv], u->gs[lv], d[lv]);
    pic::k_split_up<<<nb(d[lv + 1].V * (cs / 4)), 256, 0, st>>>(u->ga[lv], 2 * cs, u->y[up],
                                                               u->ga[lv + 1], d[lv + 1]);
  };
  decoder(0, D0A, D0B, D1B, E0B, 16);
  decoder(1, D1A, D1B, D2B, E1B, 32);
  decoder(2, D2A, D2B, BB, E2B, 64);
  // Bottom.
  back(BB, u->ga[3], u->y[BA], u->gb[3], u->y[BA]);
  back(BA, u->gb[3], u->p2, u->ga[3], nullptr);  // grad of p2 (64)
  // Encoder of level lv: skip gradient + pooled gradient of its output B.
  auto encoder = [&](int lv, int A, int B, const bf16* pooled, int cs) {
    pic::k_pool_bwd_add<<<nb(d[lv].V * (cs / 8)), 256, 0, st>>>(u->ga[lv + 1], u->gs[lv], u->y[B],
                                                              u->gb[lv], d[lv], cs);
    back(B, u->gb[lv], u->y[A], u->gs[lv], u->y[A]);
    if (pooled) back(A, u->gs[lv], pooled, u->ga[lv], nullptr);
  };
  encoder(2, E2A, E2B, u->p1, 64);
  encoder(1, E1A, E1B, u->p0, 32);
  encoder(0, E0A, E0B, nullptr, 16);
  // First layer: weights only.
  const long long runs = wgrad_runs<16>(d[0], 1);
  pic::k_wgrad_first<<<(unsigned)runs, 256, 0, st>>>(u->x_in, u->gs[0], G + u->woff[E0A],
                                                     G + u->boff[E0A], d[0], (int)runs);
  return ok;
}

pic_status unet_check(pic_unet* u, int D, int H, int W) {
  if (!u) return PIC_ERR_ARG;
  if (D < 8 || H < 8 || W < 8 || (D & 7) || (H & 7) || (W & 7) || D > u->D ||
      H > u->H || W > u->W || (long long)D * H * W > (long long)u->D * u->H * u->W)
    return PIC_ERR_ARG;
  return PIC_OK;
}

}  // namespace

bool pic_unet_fits(const pic_unet* u, int D, int H, int W) {
  return unet_check(const_cast<pic_unet*>(u), D, H, W) == PIC_OK;
}

// Inference for the solve's warm start: the network reads x in place and
// runs on the solver's stream.
bool pic_unet_infer(pic_unet* u, const float* x, int D, int H, int W,
                    hipStream_t st, const float** out) {
  if (unet_check(u, D, H, W) != PIC_OK) return false;
  float* keep_x = u->x_in;
  hipStream_t keep_st = u->stream;
  u->x_in = const_cast<float*>(x);
  u->stream = st;
  const bool ok = unet_forward(u, D, H, W);
  u->x_in = keep_x;
  u->stream = keep_st;
  *out = u->out;
  return ok;
}

extern "C" {

int64_t pic_unet_param_count(void) { return param_count(); }

pic_status pic_unet_workspace_bytes(int32_t D, int32_t H, int32_t W,
                                    size_t* bytes) {
  if (!bytes || D < 8 || H < 8 || W < 8 || (D & 7) || (H & 7) || (W & 7))
    return PIC_ERR_ARG;
  pic_unet u;
  u.D = D; u.H = H; u.W = W;
  *bytes = unet_carve(&u, nullptr);
  return PIC_OK;
}

pic_status pic_unet_init(int32_t D, int32_t H, int32_t W, void* ws,
                         size_t bytes, void* stream, pic_unet** out) {
  if (!out) return PIC_ERR_ARG;
  *out = nullptr;
  size_t need = 0;
  if (pic_unet_workspace_bytes(D, H, W, &need) != PIC_OK || !ws || bytes < need)
    return PIC_ERR_ARG;
  pic_unet* u = new (std::nothrow) pic_unet();
  if (!u) return PIC_ERR_STATE;
  u->D = D; u->H = H; u->W = W;
  u->stream = reinterpret_cast<hipStream_t>(stream);
  char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) / 256 * 256);
  u->ws = reinterpret_cast<char*>(ws);
  u->bytes = bytes;
  unet_carve(u, base);
  u->t = 0;
  u->loss_mode = PIC_UNET_LOSS_MSE;
  u->loss_k0 = 1;
  if (hipMemsetAsync(ws, 0, bytes, u->stream) != hipSuccess ||
      hipStreamSynchronize(u->stream) != hipSuccess) {
    delete u;
    return PIC_ERR_HIP;
  }
  *out = u;
  return PIC_OK;
}

void pic_unet_destroy(pic_unet* u) { delete u; }

pic_status pic_unet_set_loss(pic_unet* u, int32_t mode, int32_t k0) {
  if (!u || (mode != PIC_UNET_LOSS_MSE && mode != PIC_UNET_LOSS_RESIDUAL) ||
      (k0 != 0 && k0 != 1))
    return PIC_ERR_ARG;
  u->loss_mode = mode;
  u->loss_k0 = k0;
  return PIC_OK;
}

const char* pic_unet_last_error(const pic_unet* u) {
  return u ? u->err.c_str() : "null U-Net";
}

pic_status pic_unet_set_params(pic_unet* u, const float* params) {
  if (!u || !params) return PIC_ERR_ARG;
  if (hipMemcpyAsync(u->p, params, u->np * sizeof(float), hipMemcpyDeviceToDevice,
                     u->stream) != hipSuccess)
    return PIC_ERR_HIP;
  hipMemsetAsync(u->m, 0, u->np * sizeof(float), u->stream);
  hipMemsetAsync(u->v, 0, u->np * sizeof(float), u->stream);
  u->t = 0;
  pack_weights(u);
  return hipStreamSynchronize(u->stream) == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

pic_status pic_unet_get_params(pic_unet* u, float* params) {
  if (!u || !params) return PIC_ERR_ARG;
  if (hipMemcpyAsync(params, u->p, u->np * sizeof(float), hipMemcpyDeviceToDevice,
                     u->stream) != hipSuccess ||
      hipStreamSynchronize(u->stream) != hipSuccess)
    return PIC_ERR_HIP;
  return PIC_OK;
}

pic_status pic_unet_forward(pic_unet* u, const float* input, int32_t D,
                            int32_t H, int32_t W, float* out) {
  const pic_status c = unet_check(u, D, H, W);
  if (c != PIC_OK) return c;
  if (!input || !out) return PIC_ERR_ARG;
  const long long V = (long long)D * H * W;
  hipMemcpyAsync(u->x_in, input, 2 * V * sizeof(float), hipMemcpyDeviceToDevice,
                 u->stream);
  if (!unet_forward(u, D, H, W)) return PIC_ERR_STATE;
  hipMemcpyAsync(out, u->out, V * sizeof(float), hipMemcpyDeviceToDevice, u->stream);
  return hipStreamSynchronize(u->stream) == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

// Loss and parameter gradient of one sample (no update).
pic_status pic_unet_gradients(pic_unet* u, const float* input,
                              const float* target, int32_t D, int32_t H,
                              int32_t W, float* grad, double* loss) {
  const pic_status c = unet_check(u, D, H, W);
  if (c != PIC_OK) return c;
  if (!input || !target) return PIC_ERR_ARG;
  const long long V = (long long)D * H * W;
  hipStream_t st = u->stream;
  hipMemcpyAsync(u->x_in, input, 2 * V * sizeof(float), hipMemcpyDeviceToDevice, st);
  hipMemcpyAsync(u->target, target, V * sizeof(float), hipMemcpyDeviceToDevice, st);
  if (!unet_forward(u, D, H, W)) return PIC_ERR_STATE;
  if (u->loss_mode == PIC_UNET_LOSS_RESIDUAL) {
    const Dims d0 = dims_at(u, D, H, W, 0);
    pic::k_res_q<<<kLossParts, 256, 0, st>>>(u->out, u->target, u->q, d0, u->loss_k0, u->dpart);
    pic::k_res_g<<<nb(V), 256, 0, st>>>(u->q, u->gout, d0, u->loss_k0, 2.0f / (float)V);
  } else {
    pic::k_mse<<<kLossParts, 256, 0, st>>>(u->out, u->target, u->gout, V, u->dpart);
  }
  pic::k_sum_d<<<1, 256, 0, st>>>(u->dpart, kLossParts, u->dpart + kLossParts);
  if (!unet_backward(u, D, H, W)) return PIC_ERR_STATE;
  if (grad)
    hipMemcpyAsync(grad, u->g, u->np * sizeof(float), hipMemcpyDeviceToDevice, st);
  double l = 0.0;
  hipMemcpyAsync(&l, u->dpart + kLossParts, sizeof(double), hipMemcpyDeviceToHost, st);
  if (hipStreamSynchronize(st) != hipSuccess) return PIC_ERR_HIP;
  if (loss) *loss = l / (double)V;
  return PIC_OK;
}

// One Adam step on one sample; returns the sample's loss before the step.
pic_status pic_unet_train_step(pic_unet* u, const float* input,
                               const float* target, int32_t D, int32_t H,
                               int32_t W, float lr, float beta1, float beta2,
                               float eps, double* loss) {
  const pic_status s = pic_unet_gradients(u, input, target, D, H, W, nullptr, loss);
  if (s != PIC_OK) return s;
  u->t += 1;
  const float c1 = 1.f - powf(beta1, (float)u->t);
  const float c2 = 1.f - powf(beta2, (float)u->t);
  pic::k_adam<<<nb(u->np), 256, 0, u->stream>>>(u->p, u->m, u->v, u->g, u->np,
                                                 lr, beta1, beta2, eps, c1, c2);
  pack_weights(u);
  return hipStreamSynchronize(u->stream) == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

}  // extern "C"
