// Kernels of the warm-start network: 3x3x3 convolutions with periodic
// (circular) padding as implicit GEMMs on BF16 MFMA (v_mfma_f32_16x16x32_bf16,
// FP32 accumulation), plus the pooling, upsampling, activation, loss and
// optimiser kernels the network needs.  C ABI in include/lbm_nn.h.
//
// Tensors are channels-last: x[((n*D + z)*H + y)*W + x][c].  Convolution
// weights are w[co][tap][ci], tap = (dz+1)*9 + (dy+1)*3 + (dx+1).  BF16
// tensors are raw 16-bit patterns (uint16_t) on the device.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "lbm_nn_prepared.h"

#define NN_API extern "C" __attribute__((visibility("default")))

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) {
  return __builtin_bit_cast(float, (uint32_t)h << 16);
}
// round to nearest, ties to even (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t b = __builtin_bit_cast(uint32_t, f);
  if ((b & 0x7F800000u) == 0x7F800000u && (b & 0x007FFFFFu)) return (uint16_t)((b >> 16) | 0x40u);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}

struct Shape {
  int n, d, h, w;
  long long m;  // n*d*h*w voxels
};

// Output of a forward convolution: the FP32 pre-activation y, or (ACT) the
// BF16 activation a = bf16(relu ? max(y, 0) : y) that the next layer reads,
// without the FP32 round trip through memory.
template <bool ACT>
__device__ __forceinline__ void store_out(void* out, long long i, float v, int relu) {
  if constexpr (ACT)
    static_cast<uint16_t*>(out)[i] = f2bf(relu ? fmaxf(v, 0.f) : v);
  else
    static_cast<float*>(out)[i] = v;
}

// store_out of four consecutive values as one word (i a multiple of 4, out
// aligned to the word)
template <bool ACT>
__device__ __forceinline__ void store_out4(void* out, long long i, float v0, float v1, float v2,
                                           float v3, int relu) {
  if constexpr (ACT) {
    const uint32_t lo = (uint32_t)f2bf(relu ? fmaxf(v0, 0.f) : v0) |
                        ((uint32_t)f2bf(relu ? fmaxf(v1, 0.f) : v1) << 16);
    const uint32_t hi = (uint32_t)f2bf(relu ? fmaxf(v2, 0.f) : v2) |
                        ((uint32_t)f2bf(relu ? fmaxf(v3, 0.f) : v3) << 16);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + i) = make_uint2(lo, hi);
  } else {
    *reinterpret_cast<float4*>(static_cast<float*>(out) + i) = make_float4(v0, v1, v2, v3);
  }
}

// voxel index -> (n, z, y, x)
__device__ __forceinline__ void unflatten(long long m, const Shape& s, int& n, int& z, int& y,
                                          int& x) {
  x = (int)(m % s.w);
  long long r = m / s.w;
  y = (int)(r % s.h);
  r /= s.h;
  z = (int)(r % s.d);
  n = (int)(r / s.d);
}

// voxel shifted by tap t with periodic wrap
__device__ __forceinline__ long long neighbour(int n, int z, int y, int x, int t, const Shape& s) {
  const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
  int zz = z + dz, yy = y + dy, xx = x + dx;
  zz = zz < 0 ? zz + s.d : (zz >= s.d ? zz - s.d : zz);
  yy = yy < 0 ? yy + s.h : (yy >= s.h ? yy - s.h : yy);
  xx = xx < 0 ? xx + s.w : (xx >= s.w ? xx - s.w : xx);
  return (((long long)n * s.d + zz) * s.h + yy) * s.w + xx;
}

// Packed weights of a convolution (nn_conv3d_pack_weights): the MFMA weight
// operands in the order the forward kernels read them.  Fragment (row tile ct,
// step q) holds the 16 rows 16 ct.. of output channels and the four octets
// 4 q.. of K = 27 ci, lane l's 16 bytes (row l % 16, octet l / 16) at 16 l; zeros
// past the last row or octet.  A fragment is then one 1 KB run, where the
// rows of w[co][27][ci] give 16 segments of 64 bytes (the
// weight reads of the spatial kernel: 192 -> 64 channels at 32^3 x 4 105 -> 82 us,
// 1050 TFLOP/s; 96 -> 32 at 64^3 x 4 200 -> 187 us; of the halo kernel: 128 -> 256 at
// 8^3 x 4 30 -> 14 us, 384 -> 128 at one 16^3 box 83 -> 34 us).
__host__ __device__ __forceinline__ int k_steps(int ci) { return (27 * (ci >> 3) + 3) >> 2; }

// ---------------------------------------------------------------- forward
// y[m][co] = bias[co] + sum_{tap, ci} x[m + off(tap)][ci] * w[co][tap][ci]:
// an implicit GEMM with M = voxels, N = co and K = 27 ci (ci % 8 == 0).  MFMA
// operands (v_mfma_f32_16x16x32_bf16): lane l supplies row/column l % 16 and
// the 8 consecutive k of octet l / 16; the result holds rows 4 (l / 16) + i,
// column l % 16.
constexpr int kPad = 8;

// Tiled forward convolution for boxes of many tiles that are no multiple of
// the spatial tile, and for any input the kernels below do not take: block
// tile 128 voxels x BN output channels
// (BN = 16, 32 or 64), K = 27 ci staged 64 at a time through LDS.  Each of
// the 4 wavefronts owns 32 voxel rows (two 16-row MFMA tiles) against all
// BN/16 column tiles.  The 27 neighbour voxels of the block's 128 rows are
// tabulated in LDS once, so the gather of a K stage is a table lookup plus
// the tap/channel position of the thread's 8-element granule, advanced
// incrementally.  The next stage's global loads are issued into registers
// before the current stage's MFMAs (one stage of prefetch).
template <int BN, bool PK, bool ACT>
__global__ __launch_bounds__(256) void conv_fwd_tiled_kernel(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ w,
                                                             const float* __restrict__ bias,
                                                             void* __restrict__ y, Shape s,
                                                             int ci, int co, int relu) {
  constexpr int BM = 128, BK = 64, LD = BK + 8;
  constexpr int NBG = BN * BK / 8;          // B granules per stage
  constexpr int NB = (NBG + 255) / 256;     // B granules per thread (at most)
  constexpr int NT = BN / 16;               // column tiles
  __shared__ __attribute__((aligned(16))) uint16_t As[BM * LD];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LD];
  __shared__ int nbr[27 * BM];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long m0 = (long long)blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  const int K = 27 * ci, steps = k_steps(ci);
  for (int i = tid; i < 27 * BM; i += 256) {
    const int t = i / BM, r = i - t * BM;
    const long long m = m0 + r;
    int v = -1;
    if (m < s.m) {
      int vn, vz, vy, vx;
      unflatten(m, s, vn, vz, vy, vx);
      v = (int)neighbour(vn, vz, vy, vx, t, s);
    }
    nbr[i] = v;
  }
  // this thread's granules: rows (tid >> 3) + 32 i of A, B rows from g = tid + 256 i,
  // all at K offset koff = 8 (tid & 7) within the stage
  const int koff = 8 * (tid & 7);
  int ta = 0, ca = koff;
  while (ca >= ci) {
    ca -= ci;
    ++ta;
  }
  __syncthreads();

  // packed weights: thread tid + 256 i takes its 16 bytes of a fragment (row
  // tile ct + 2 i, first or second half of the stage) in the fragment's order,
  // so that a wavefront reads 1 KB in a row (in the order of the rows of LDS
  // its 16-byte words lay 256 bytes apart: 192 -> 64 channels at 4 x 28 x 33 x 35
  // 211 us, 180 from unpacked weights)
  const int ct = (n0 >> 4) + (tid >> 7), half = (tid >> 6) & 1;
  const uint16_t* wfrag = w + ((long long)ct * steps + half) * 512 + lane * 8;

  uint4 ra[4], rb[NB];
  auto gload = [&](int k0) {
    const bool kin = k0 + koff < K;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ra[i] = make_uint4(0, 0, 0, 0);
      if (kin) {
        const int v = nbr[ta * BM + (tid >> 3) + 32 * i];
        if (v >= 0) ra[i] = *reinterpret_cast<const uint4*>(x + (long long)v * ci + ca);
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int g = tid + 256 * i;
      rb[i] = make_uint4(0, 0, 0, 0);
      if constexpr (PK) {
        if (g < NBG && 16 * (ct + 2 * i) < co && (k0 >> 5) + half < steps)
          rb[i] = *reinterpret_cast<const uint4*>(wfrag + (2 * i * steps + (k0 >> 5)) * 512LL);
      } else {
        const int col = n0 + (g >> 3);
        if (g < NBG && kin && col < co)
          rb[i] = *reinterpret_cast<const uint4*>(w + (long long)col * K + k0 + koff);
      }
    }
  };
  f32x4 acc[2][NT];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[r][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  gload(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<uint4*>(&As[((tid >> 3) + 32 * i) * LD + koff]) = ra[i];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int g = tid + 256 * i;
      const int at = PK ? (16 * (g >> 7) + (lane & 15)) * LD + 32 * half + 8 * (lane >> 4)
                        : (g >> 3) * LD + koff;
      if (g < NBG) *reinterpret_cast<uint4*>(&Bs[at]) = rb[i];
    }
    __syncthreads();
    if (k0 + BK < K) {
      ca += BK;
      while (ca >= ci) {
        ca -= ci;
        ++ta;
      }
      gload(k0 + BK);
    }
#pragma unroll
    for (int ks = 0; ks < BK; ks += 32) {
      const int kk = ks + 8 * (lane >> 4);
      const bf16x8 a0 = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const uint4*>(&As[(wv * 32 + (lane & 15)) * LD + kk]));
      const bf16x8 a1 = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const uint4*>(&As[(wv * 32 + 16 + (lane & 15)) * LD + kk]));
#pragma unroll
      for (int b = 0; b < NT; ++b) {
        const bf16x8 bf = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const uint4*>(&Bs[(b * 16 + (lane & 15)) * LD + kk]));
        acc[0][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bf, acc[0][b], 0, 0, 0);
        acc[1][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bf, acc[1][b], 0, 0, 0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int col = n0 + b * 16 + (lane & 15);
    if (col >= co) continue;
    const float bb = bias ? bias[col] : 0.f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const long long row = m0 + wv * 32 + r * 16 + (lane >> 4) * 4 + i;
        if (row < s.m) store_out<ACT>(y, row * co + col, acc[r][b][i] + bb, relu);
      }
  }
}

// Spatially tiled forward convolution for ci % 32 == 0 and box edges that
// are multiples of 4 x 8 x 8 (z, y, x).  The four wavefronts of a block are
// WZ = 4 / WC z layers times WC groups of 16 NT output channels; a wavefront
// computes MT MFMA tiles of 16 voxels (TX = 16: one x row each, TX = 8: two x
// rows of 8), i.e. RPM MT rows of its layer.  The input is taken 32 channels
// at a time: the halo of the block's tile (periodic wrap) goes straight from
// global memory to LDS (16 bytes per lane, no registers).
//
// The kernel is bound by what feeds the matrix cores, so the work is arranged
// for operand reuse.  A voxel fragment (16 voxels x 32 channels at one x
// shift) is read from LDS once per dz and serves every row of the
// wavefront's patch that it is a dy neighbour of, up to three; the weights of
// the nine taps of a dz sit in registers and are replaced tap row by tap row
// as the sweep over the input rows passes their last use.  Per 32 channels a
// wavefront with MT = 8 then reads 90 voxel and 54 weight fragments for 432
// MFMAs, against 108 LDS reads per 216 MFMAs for one read per tap and row.
// Every output still adds its taps in the order dz, dy, dx (the sweep over
// input rows meets dy = 0, 1, 2 of an output row in that order), so the
// results do not depend on MT, WC or TX.
//
// The weights are the MFMA's row operand: a lane then holds four consecutive
// output channels of one voxel and stores them as one word.
//
// LDS: halo voxel (row R = hz HY + hy, column hx) starts at 64 (R P + hx)
// bytes, P the row pitch (20 or 12); its four 16-byte channel octets are
// permuted by (hx >> 1) ^ 2 R (mod 4), so that 8 consecutive voxels of a row
// read at one octet cover all banks.
//
// 96 -> 32 channels at 64^3 x 4 (174 GFLOP), BF16 output: 316 -> 200 us (870
// TFLOP/s) against one LDS read per tap and row, 187 us (930) from packed
// weights; 192 -> 64 at 32^3 x 4: 182 -> 105, packed 82 us (1050 TFLOP/s).
constexpr int kTZ = 4, kTY = 8, kTX = 8;
constexpr int kCC = 32;                 // channels per chunk

// 16 bytes per lane from global memory to LDS: lane l's go to lds + 16 l (lds
// the same in every lane).
__device__ __forceinline__ void load_to_lds(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// Consecutive workgroups go to the eight XCDs in turn; work item of block b of
// n so that each XCD takes a contiguous range of items (neighbouring tiles
// share halo lines in its L2; the first n % 8 XCDs take one item more).
__device__ __forceinline__ int xcd_item(int b, int n) {
  const int x = b % 8, r = n % 8;
  return x * (n / 8) + (x < r ? x : r) + b / 8;
}

template <int TX, int MT, int NT, int WC, bool PK, bool ACT>
__global__ __launch_bounds__(256, 2) void conv_fwd_spatial_kernel(const uint16_t* __restrict__ x,
                                                                  const uint16_t* __restrict__ w,
                                                                  const float* __restrict__ bias,
                                                                  void* __restrict__ y, Shape s,
                                                                  int ci, int co, int relu,
                                                                  int vec) {
  constexpr int WZ = 4 / WC, RPM = 16 / TX;
  constexpr int TY = RPM * MT;                   // rows of the tile
  constexpr int HZ = WZ + 2, HY = TY + 2, P = TX + 4;
  static_assert(HY % 2 == 0, "the octet permutation needs an even number of halo rows");
  constexpr int NQ = (HZ * HY * P * 4 + 63) / 64;  // wavefront loads of a staging pass
  constexpr int NL = (NQ + 3) / 4;                 // ... per wavefront (at most)
  __shared__ __attribute__((aligned(16))) unsigned char Hs[NQ * 1024];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wz = wv / WC, wc = wv % WC;
  // work item: tile (x, then y, then z, then n) and group of 16 NT WC channels
  const int cgs = (co + 16 * NT * WC - 1) / (16 * NT * WC);
  int t = xcd_item(blockIdx.x, gridDim.x);
  const int n0 = (t % cgs) * 16 * NT * WC + 16 * NT * wc;
  t /= cgs;
  const int tx_n = s.w / TX, ty_n = s.h / TY, tz_n = s.d / WZ;
  const int x0 = (t % tx_n) * TX;
  t /= tx_n;
  const int y0 = (t % ty_n) * TY;
  t /= ty_n;
  const int z0 = (t % tz_n) * WZ;
  const int bn_ = t / tz_n;
  const int col = lane & 15, oct = lane >> 4;
  const int lx = col & (TX - 1), ly = col / TX;

  // this lane's source granule (16 bytes of a voxel) of each staging load
  uint32_t src[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int g = (wv + 4 * i) * 64 + lane;
    const int hv = g >> 2;
    int R = hv / P, hx = hv - R * P;
    const int o = (g & 3) ^ ((hx >> 1) & 3) ^ ((R & 1) << 1);
    if (hx >= TX + 2) hx = 0;      // pitch padding: any voxel
    if (R >= HZ * HY) R = 0;       // past the halo
    const int hz = R / HY, hy = R - hz * HY;
    int zz = z0 + hz - 1, yy = y0 + hy - 1, xx = x0 + hx - 1;
    zz = zz < 0 ? zz + s.d : (zz >= s.d ? zz - s.d : zz);
    yy = yy < 0 ? yy + s.h : (yy >= s.h ? yy - s.h : yy);
    xx = xx < 0 ? xx + s.w : (xx >= s.w ? xx - s.w : xx);
    src[i] = (uint32_t)(((bn_ * s.d + zz) * s.h + yy) * s.w + xx) * (uint32_t)(ci >> 3) + (uint32_t)o;
  }
  // LDS byte of this lane's 16 bytes of a voxel fragment: x shift dx, row
  // parity, plus a constant per row
  int la[3][2];
#pragma unroll
  for (int dx = 0; dx < 3; ++dx)
#pragma unroll
    for (int par = 0; par < 2; ++par)
      la[dx][par] = ((wz * HY + ly) * P + lx + dx) * 64 +
                    16 * (oct ^ (((lx + dx) >> 1) & 3) ^ (((ly + par) & 1) << 1));

  // weight fragments: row co = n0 + 16 b + col, channels c0 + 8 oct
  // (rows past co repeat others; their results are not stored)
  const uint16_t* wrow[NT];
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int c = n0 + 16 * b + col, ct = (n0 >> 4) + b;
    wrow[b] = PK ? w + (long long)(16 * ct < co ? ct : 0) * k_steps(ci) * 512 + lane * 8
                 : w + (long long)(c < co ? c : 0) * 27 * ci + 8 * oct;
  }
  uint4 wf[9][NT];
  auto load_weights = [&](int dy, int off) {  // taps (dz, dy, 0..2) at off = 9 dz ci + c0
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int b = 0; b < NT; ++b)
        wf[3 * dy + dx][b] =
            *reinterpret_cast<const uint4*>(wrow[b] + (off + (3 * dy + dx) * ci) * (PK ? 16 : 1));
  };

  f32x4 acc[MT][NT];
#pragma unroll
  for (int r = 0; r < MT; ++r)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[r][b] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int dy = 0; dy < 3; ++dy) load_weights(dy, 0);
  for (int c0 = 0; c0 < ci; c0 += kCC) {
    if (c0) __syncthreads();  // the previous chunk's reads are done
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int q = wv + 4 * i;
      if (q < NQ)
        load_to_lds(reinterpret_cast<const uint4*>(x) + (unsigned long long)(src[i] + (uint32_t)(c0 >> 3)),
                    Hs + q * 1024);
    }
    __builtin_amdgcn_s_waitcnt(0);  // every load has written its LDS bytes
    __syncthreads();
#pragma unroll 1
    for (int dz = 0; dz < 3; ++dz) {
      const unsigned char* hz = Hs + dz * (HY * P * 64);
      // the weights that follow: next dz, or dz = 0 of the next chunk (the
      // last chunk loads its first ones again: never used)
      const int next = dz < 2 ? 9 * (dz + 1) * ci + c0 : (c0 + kCC < ci ? c0 + kCC : c0);
#pragma unroll
      for (int r = 0; r <= RPM * (MT - 1) + 2; ++r) {  // first halo row of the fragment
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
          const bf16x8 a = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const uint4*>(hz + la[dx][r & 1] + r * (P * 64)));
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
            if (r < dy || (r - dy) % RPM || (r - dy) / RPM >= MT) continue;
            const int m = (r - dy) / RPM;
#pragma unroll
            for (int b = 0; b < NT; ++b)
              acc[m][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, wf[3 * dy + dx][b]), a, acc[m][b], 0, 0, 0);
          }
        }
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
          if (r == RPM * (MT - 1) + dy) load_weights(dy, next);
      }
    }
  }
  // channels 4 oct + i of channel tile b, voxel col of voxel tile m
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int c = n0 + 16 * b + 4 * oct;
    float bb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bb[i] = bias && c + i < co ? bias[c + i] : 0.f;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const long long v =
          (((long long)bn_ * s.d + z0 + wz) * s.h + y0 + RPM * m + ly) * s.w + x0 + lx;
      if (vec && c + 4 <= co) {
        store_out4<ACT>(y, v * co + c, acc[m][b][0] + bb[0], acc[m][b][1] + bb[1],
                        acc[m][b][2] + bb[2], acc[m][b][3] + bb[3], relu);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (c + i < co) store_out<ACT>(y, v * co + c + i, acc[m][b][i] + bb[i], relu);
      }
    }
  }
}

// Forward convolution for any box with all channels of the halo in LDS: the
// small levels of the network, whose tiles are too few for the kernel above,
// channel counts that are no multiple of 32 (the network's 8-channel input
// and the head's gradient), and boxes that are no multiple of its tiles.
//
// The four wavefronts of a block are WZ = 4 / WC z layers times WC groups of
// 16 NT output channels; a wavefront computes MT tiles of 2 x 8 voxels (y, x),
// 2 MT rows of its layer.  K = 27 ci is taken in the order of the weights'
// memory, tap by tap, as octets of 8 channels, four octets per MFMA (lane
// group oct takes octet 4 q + oct of step q; with 8 channels that is one tap
// each).  A table in LDS holds each octet's halo offset, so a lane's voxel
// fragment is one table read and MT 16-byte reads.  Octets past K read the
// zeroed voxel behind the halo against zero weights.  Voxels outside the box
// are computed on wrapped inputs and not stored.
//
// These launches are bound by latency and by the weights, which every
// wavefront reads once in a row (L2 resident): they are loaded U steps ahead.
// Halo voxels are an odd number of octets apart in LDS (8 consecutive ones read
// at one octet then cover all banks) and loaded straight from global memory; the
// padding lanes of even channel counts load a neighbour's bytes that nothing
// reads.
//
// Against 128-voxel tiles gathered stage by stage (conv_fwd_tiled_kernel), BF16
// output: 8 -> 32 channels at 64^3 x 4 117 -> 40 us; 128 -> 256 at 8^3 x 4 56
// -> 30 us, 14 from packed weights; 384 -> 128 at one 16^3 box 145 -> 83, 34 us.
constexpr int kRX = 8, kRHX = kRX + 2;  // x extent of a tile, of its halo

template <int MT, int WC>
constexpr int rows_halo() {  // halo voxels of a block's tile
  return (4 / WC + 2) * (2 * MT + 2) * kRHX;
}
// LDS bytes: the halo in whole wavefront loads, a zero voxel octet, the table
template <int MT, int WC>
size_t rows_lds(int ci) {
  const size_t halo = (size_t)rows_halo<MT, WC>() * ((ci / 8) | 1) * 16;
  return (halo + 1023) / 1024 * 1024 + 16 + (size_t)((27 * (ci / 8) + 3) / 4 * 4) * 4;
}

template <int MT, int NT, int WC, bool PK, bool ACT>
__global__ __launch_bounds__(256) void conv_fwd_rows_kernel(const uint16_t* __restrict__ x,
                                                            const uint16_t* __restrict__ w,
                                                            const float* __restrict__ bias,
                                                            void* __restrict__ y, Shape s, int ci,
                                                            int co, int relu, int vec) {
  constexpr int WZ = 4 / WC, HY = 2 * MT + 2, HV = rows_halo<MT, WC>(), U = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char Rs[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wz = wv / WC, wc = wv % WC;
  const int cgs = (co + 16 * NT * WC - 1) / (16 * NT * WC);
  int t = xcd_item(blockIdx.x, gridDim.x);
  const int n0 = (t % cgs) * 16 * NT * WC + 16 * NT * wc;
  t /= cgs;
  const int tx_n = (s.w + kRX - 1) / kRX, ty_n = (s.h + 2 * MT - 1) / (2 * MT),
            tz_n = (s.d + WZ - 1) / WZ;
  const int x0 = (t % tx_n) * kRX;
  t /= tx_n;
  const int y0 = (t % ty_n) * 2 * MT;
  t /= ty_n;
  const int z0 = (t % tz_n) * WZ;
  const int bn_ = t / tz_n;
  const int g8 = ci >> 3, gs = g8 | 1;  // octets of a voxel; with its padding
  const int nq = (HV * gs + 63) >> 6;
  const int octets = 27 * g8, steps = (octets + 3) >> 2;
  unsigned char* zero = Rs + nq * 1024;
  int* tab = reinterpret_cast<int*>(zero + 16);

  for (int q = wv; q < nq; q += 4) {
    const int g = q * 64 + lane;
    int v = g / gs, o = g - v * gs;
    if (o >= g8) o = 0;
    if (v >= HV) v = 0;
    const int R = v / kRHX, hx = v - R * kRHX;
    const int hz = R / HY, hy = R - hz * HY;
    // wrapped coordinates; past the far halo of a partial tile: the first cell
    int zz = z0 + hz - 1, yy = y0 + hy - 1, xx = x0 + hx - 1;
    zz = zz < 0 ? zz + s.d : (zz >= s.d ? (zz == s.d ? 0 : z0) : zz);
    yy = yy < 0 ? yy + s.h : (yy >= s.h ? (yy == s.h ? 0 : y0) : yy);
    xx = xx < 0 ? xx + s.w : (xx >= s.w ? (xx == s.w ? 0 : x0) : xx);
    const long long m = (((long long)bn_ * s.d + zz) * s.h + yy) * s.w + xx;
    load_to_lds(reinterpret_cast<const uint4*>(x) + (m * g8 + o), Rs + q * 1024);
  }
  const int zoff = nq * 1024;
  for (int i = tid; i < 4 * steps; i += 256) {
    const int tap = i / g8, o = i - tap * g8;
    const int dz = tap / 9, dy = (tap / 3) % 3, dx = tap % 3;
    tab[i] = i < octets ? ((dz * HY + dy) * kRHX + dx) * (gs * 16) + o * 16 : -1;
  }
  if (tid < 4) reinterpret_cast<uint32_t*>(zero)[tid] = 0;

  const int col = lane & 15, oct = lane >> 4;
  const int lx = col & 7, ly = col >> 3;
  const int base = ((wz * HY + ly) * kRHX + lx) * (gs * 16);
  const int mstep = 2 * kRHX * gs * 16;  // next voxel tile: two rows on
  // weight rows co = n0 + 16 b + col (rows past co repeat row 0; their results
  // are not stored).  Every load is unconditional, so that the compiler keeps
  // all of them in flight; octets past K load the row's last one.
  const uint16_t* wrow[NT];
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int c = n0 + 16 * b + col, ct = (n0 >> 4) + b;
    wrow[b] = PK ? w + (long long)(16 * ct < co ? ct : 0) * steps * 512 + lane * 8
                 : w + (long long)(c < co ? c : 0) * 27 * ci;
  }
  uint4 wf[2][U][NT];
  auto load_weights = [&](uint4 (&f)[U][NT], int q0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = 4 * (q0 + u) + oct;
#pragma unroll
      for (int b = 0; b < NT; ++b)
        f[u][b] = *reinterpret_cast<const uint4*>(
            wrow[b] + (PK ? 512 * (q0 + u < steps ? q0 + u : 0)
                          : 8 * (i < octets ? i : octets - 1)));
    }
  };
  f32x4 acc[MT][NT];
#pragma unroll
  for (int r = 0; r < MT; ++r)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[r][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](const uint4 (&f)[NT], int off) {
    const int at = off < 0 ? zoff : base + off, am = off < 0 ? 0 : mstep;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const bf16x8 a =
          __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(Rs + at + m * am));
#pragma unroll
      for (int b = 0; b < NT; ++b)
        acc[m][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[b]), a,
                                                            acc[m][b], 0, 0, 0);
    }
  };
  // U steps whose octets all lie within K
  auto compute = [&](const uint4 (&f)[U][NT], int q0) {
    int off[U];
#pragma unroll
    for (int u = 0; u < U; ++u) off[u] = tab[4 * (q0 + u) + oct];
#pragma unroll
    for (int u = 0; u < U; ++u) step(f[u], off[u]);
  };
  // the last steps: weights of octets past K are zero
  auto compute_tail = [&](uint4 (&f)[U][NT], int q0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (q0 + u >= steps) break;
      if (4 * (q0 + u) + oct >= octets)
#pragma unroll
        for (int b = 0; b < NT; ++b) f[u][b] = make_uint4(0, 0, 0, 0);
      step(f[u], tab[4 * (q0 + u) + oct]);
    }
  };
  load_weights(wf[0], 0);
  __builtin_amdgcn_s_waitcnt(0);  // every load has written its LDS bytes
  __syncthreads();
  int q0 = 0;
  for (; 4 * (q0 + 2 * U) <= octets; q0 += 2 * U) {
    load_weights(wf[1], q0 + U);
    compute(wf[0], q0);
    load_weights(wf[0], q0 + 2 * U);
    compute(wf[1], q0 + U);
  }
  if (q0 < steps) {
    load_weights(wf[1], q0 + U);
    compute_tail(wf[0], q0);
    compute_tail(wf[1], q0 + U);
  }
  // channels 4 oct + i of channel tile b, voxel col of voxel tile m
  const int zz = z0 + wz, xx = x0 + lx;
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int c = n0 + 16 * b + 4 * oct;
    float bb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bb[i] = bias && c + i < co ? bias[c + i] : 0.f;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int yy = y0 + 2 * m + ly;
      if (zz >= s.d || yy >= s.h || xx >= s.w) continue;
      const long long v = (((long long)bn_ * s.d + zz) * s.h + yy) * s.w + xx;
      if (vec && c + 4 <= co) {
        store_out4<ACT>(y, v * co + c, acc[m][b][0] + bb[0], acc[m][b][1] + bb[1],
                        acc[m][b][2] + bb[2], acc[m][b][3] + bb[3], relu);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (c + i < co) store_out<ACT>(y, v * co + c + i, acc[m][b][i] + bb[i], relu);
      }
    }
  }
}

// Tiled weight gradient: dw[co][tap][ci] = sum over the voxels v of dy[v][co]
// x[v + off(tap)][ci], an MFMA GEMM whose K runs over the voxels of tiles of
// TZ x TY x TX (TX a multiple of 8), 32 voxels (four x octets, in z, y, x order)
// per step.  Block (g, chunk, co tile) adds up its steps in order for 16 CT
// input and 16 RT output channels (what LDS holds for channels past ci or co
// only reaches sums that are not stored) and writes its sum to part[g]; fold_splits_kernel adds the partials in order.  Two
// orders of the voxels (BwdwTiles): the tiles g, g + G, g + 2G, ... of
// 4 x 8 x 8, for boxes of many of them; or consecutive voxels of the box, in
// tiles of whole rows.
//
// Both operands need 8 consecutive voxels of one channel per lane, while
// tensors (and the LDS tiles) are channels-last: gfx950's transposing LDS read
// (ds_read_b64_tr_b16: 16 lanes read 4 voxels x 16 channels and each gets the
// 4 voxels of one channel) does that without a transposed copy.  The 10
// voxels of an octet's halo row serve the three x shifts: shift 0 and 2 are
// register pairs of the same reads, shift 1 takes four 16-bit funnel shifts, so
// a wavefront reads 1.5 instead of 3 operands per (dz, dy).
//
// The four wavefronts share the outputs, not the voxels, so that every sum
// keeps its order: CT input-channel tiles times 4 / CT equal shares of the
// units (dz, dy, co tile) of three taps each (CT = RT = 2: 9 units, 27
// accumulators; 9.5 operand reads per 27 MFMAs).  Halo and gradient go straight
// from global memory to LDS; where LDS allows, into the other of two buffers
// while the current tile is computed, else a second block on the CU computes
// meanwhile.
//
// LDS: voxel v of a tile at 32 CT (32 RT) bytes; with 64 bytes the two 32-byte
// halves are swapped where v & 2, so that the 4 voxels of a transposing read
// cover all banks.  The halo's rows hold TX + 2 voxels and two of padding, or,
// where tiles are whole rows of the box, the TX voxels alone: a read's four
// voxels are addressed lane by lane, so the periodic wrap in x is one of
// addresses (xtab), and a load fills whole kilobytes.
//
// Against transposed copies written to LDS two bytes at a time, and the general
// kernel for boxes of few tiles (bit-identical), whole calls with their fold in a
// short loop: 96 -> 32 channels at 64^3 x 4 641 -> 245 us, 192 -> 64 at 32^3 x 4 311
// -> 123 us, 384 -> 128 at 16^3 x 4 317 -> 105 us, 128 -> 256 at 8^3 x 4 49 -> 27 us.
// In a training step, where the clock is up, this kernel alone takes 195 to 207
// us (840 to 890 TFLOP/s) for the first and 109 to 113 us for the second, their
// folds 10 us each.
struct BwdwTiles {
  int tz, ty, tx;      // tile
  int ntx, nty, ntz;   // tiles per row, per plane of rows, per box
  int steps;           // steps of 32 voxels per tile
  int tiles;           // tiles in all
  int stride;          // > 0: tiles g, g + stride, ...; 0: consecutive voxels,
  int split_steps;     // ... this many steps per split
  int buffers;         // LDS buffers (1 or 2)
  uint32_t by_tx, by_hy;  // ceil(2^32 / tx), ceil(2^32 / (ty + 2)): divisions by __umulhi
};
constexpr int kBwdwMaxOctets = 32;  // octets of a tile (256 voxels)

typedef short s16x4 __attribute__((ext_vector_type(4)));

// 16 bytes per active lane from global memory to LDS byte address lds + 16
// lane, not tracked by the compiler, which would otherwise wait for it before
// any LDS read: lds_loads_done() before the barrier that publishes them.  The
// load takes its LDS address from M0, a reserved register that an asm statement
// cannot name as clobbered: it is put back, so that what the compiler keeps
// there holds.
__device__ __forceinline__ void load_to_lds_async(const void* g, uint32_t lds) {
  uint32_t m0;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
      "global_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
      : "=&s"(m0)
      : "s"(lds), "v"(g)
      : "memory");
}
__device__ __forceinline__ void lds_loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// 4 voxels of one channel per lane (see above)
__device__ __forceinline__ uint2 read_transposed(const unsigned char* p) {
  return __builtin_bit_cast(
      uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
}

// Bytes of one LDS buffer (halo, gradient), and of a block's LDS.
__host__ __device__ inline int bwdw_pitch(const BwdwTiles& g) {  // voxels
  return g.stride ? g.tx + 4 : g.tx;
}
__host__ __device__ inline int bwdw_halo_bytes(const BwdwTiles& g, int xv) {
  return ((g.tz + 2) * (g.ty + 2) * bwdw_pitch(g) * xv + 1023) / 1024 * 1024;
}
__host__ __device__ inline int bwdw_buffer_bytes(const BwdwTiles& g, int xv, int dv) {
  return bwdw_halo_bytes(g, xv) + g.tz * g.ty * g.tx * dv;
}

// One step for the units [U0, U1) of a wavefront: unit u = (pair u / RT, co
// tile u % RT).
template <int RT, int U0, int U1, int NA>
__device__ __forceinline__ void bwdw_step(const unsigned char* xs, const int (&xoff)[3],
                                          const unsigned char* dr, int dv, int half, int row,
                                          int plane, f32x4 (&acc)[NA]) {
  bf16x8 a[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const unsigned char* q = dr + (RT == 2 ? (r ^ half) * 32 : 0);
    const uint2 lo = read_transposed(q), hi = read_transposed(q + 4 * dv);
    a[r] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
  }
#pragma unroll
  for (int p = U0 / RT; p * RT < U1; ++p) {
    const unsigned char* q = xs + (p / 3) * plane + (p % 3) * row;
    const uint2 v0 = read_transposed(q + xoff[0]), v4 = read_transposed(q + xoff[1]),
                v8 = read_transposed(q + xoff[2]);
    const uint4 b[3] = {
        make_uint4(v0.x, v0.y, v4.x, v4.y),
        make_uint4(__builtin_amdgcn_alignbit(v0.y, v0.x, 16),
                   __builtin_amdgcn_alignbit(v4.x, v0.y, 16),
                   __builtin_amdgcn_alignbit(v4.y, v4.x, 16),
                   __builtin_amdgcn_alignbit(v8.x, v4.y, 16)),
        make_uint4(v0.y, v4.x, v4.y, v8.x)};
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int u = p * RT + r;
      if (u < U0 || u >= U1) continue;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
        acc[3 * (u - U0) + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            a[r], __builtin_bit_cast(bf16x8, b[dx]), acc[3 * (u - U0) + dx], 0, 0, 0);
    }
  }
}

// f(integral constant I) for the wavefront-uniform index I of N: the share's
// whole loop is compiled per share, since a branch inside the loop made the
// compiler copy every accumulator on each step.
template <int N, int I = 0, class F>
__device__ __forceinline__ void for_share(int share, F&& f) {
  if constexpr (I == N - 1) {
    f(std::integral_constant<int, I>{});
  } else {
    if (share == I)
      f(std::integral_constant<int, I>{});
    else
      for_share<N, I + 1>(share, f);
  }
}

template <int RT, int CT>
__global__ __launch_bounds__(256, 2) void conv_bwdw_tile_kernel(const uint16_t* __restrict__ x,
                                                                const uint16_t* __restrict__ dy,
                                                                float* __restrict__ part, Shape s,
                                                                int ci, int co, BwdwTiles g) {
  constexpr int XV = 32 * CT, DV = 32 * RT;              // bytes of a voxel in LDS
  constexpr int NV = 4, NW = NV / CT, U = 9 * RT;        // wavefronts, shares, units
  extern __shared__ __attribute__((aligned(16))) unsigned char Ls[];
  // LDS byte, for either channel tile, of the 12 voxels from x - 1 on of an
  // octet's row
  __shared__ int xtab[2][kBwdwMaxOctets * 12];
  const int tid = threadIdx.x, lane = tid & 63, oct = lane >> 4, i16 = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ct = wv % CT, share = wv / CT;
  const int c0 = blockIdx.y * 16 * CT, o0 = blockIdx.z * 16 * RT;
  const int HY = g.ty + 2, P = bwdw_pitch(g);
  const int row = P * XV, plane = HY * row;              // LDS bytes
  const int xbytes = bwdw_halo_bytes(g, XV), bytes = bwdw_buffer_bytes(g, XV, DV);
  const int octets_x = g.tx >> 3;
  for (int i = tid; i < 4 * g.steps * 12; i += 256) {
    const int o = i / 12, r = o / octets_x, z = r / g.ty;
    int v = (o - r * octets_x) * 8 + (i - o * 12);
    if (!g.stride) v = v == 0 ? P - 1 : (v > P ? v - P - 1 : v - 1);
    v += (z * HY + (r - z * g.ty)) * P;
    for (int k = 0; k < CT; ++k)
      xtab[k][i] = v * XV + (CT == 2 ? (k ^ ((v >> 1) & 1)) * 32 : 0);
  }

  // this lane's voxel and channel octet of a staging load
  constexpr int XG = 2 * CT, DG = 2 * RT;                // octets of a voxel
  constexpr int XL = 64 / XG, DL = 64 / DG;              // voxels per load
  const int xv = lane / XG, dv = lane / DG;
  auto octet_of = [](int slot, int v, int n) {           // swapped halves (above)
    return n == 4 ? (slot ^ (v & 2)) : slot;
  };
  const int xo = c0 + 8 * octet_of(lane % XG, xv, XG), od = o0 + 8 * octet_of(lane % DG, dv, DG);
  const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_address(Ls));
  const int dvox = g.tz * g.ty * g.tx;
  // (the loops below step through rows without divisions, whose instructions
  // would cost more than the loads)
  auto stage = [&](int t, int buf) {
    const long long m0 = (long long)t * dvox;              // (consecutive voxels)
    const int x0 = (t % g.ntx) * g.tx;
    t /= g.ntx;
    const int y0 = (t % g.nty) * g.ty;
    t /= g.nty;
    const int z0 = (t % g.ntz) * g.tz;
    const int bn_ = t / g.ntz;
    const uint32_t xl = lds + buf * bytes, dl = xl + xbytes;
    if (g.stride) {  // one load per row of 10 voxels
      int xx = x0 + xv - 1;
      xx = xx < 0 ? xx + s.w : (xx >= s.w ? xx - s.w : xx);
      const bool in = xv < g.tx + 2 && xo < ci;
      const uint16_t* xlane_src = x + (long long)xx * ci + xo;
      int hz = 0, hy = wv;                                 // (wavefront-uniform)
      uint32_t at = xl + wv * row;
      for (;; hy += NV, at += NV * row) {
        while (hy >= HY) {
          hy -= HY;
          ++hz;
        }
        if (hz >= g.tz + 2) break;
        int zz = z0 + hz - 1, yy = y0 + hy - 1;
        zz = zz < 0 ? zz + s.d : (zz >= s.d ? zz - s.d : zz);
        yy = yy < 0 ? yy + s.h : (yy >= s.h ? yy - s.h : yy);
        const long long v = (((long long)bn_ * s.d + zz) * s.h + yy) * s.w;
        if (in) load_to_lds_async(xlane_src + v * ci, at);
      }
    } else {         // whole rows of the box, 64 lanes of them per load
      for (int q = wv; q < xbytes >> 10; q += NV) {
        const uint32_t f = q * XL + xv, r = __umulhi(f, g.by_tx), hz = __umulhi(r, g.by_hy);
        int zz = z0 + (int)hz - 1, yy = y0 + (int)(r - hz * HY) - 1;
        zz = zz < 0 ? zz + s.d : (zz >= s.d ? zz - s.d : zz);
        yy = yy < 0 ? yy + s.h : (yy >= s.h ? yy - s.h : yy);
        const long long v =
            (((long long)bn_ * s.d + zz) * s.h + yy) * s.w + (long long)(f - r * g.tx);
        if ((int)hz < g.tz + 2 && xo < ci) load_to_lds_async(x + v * ci + xo, xl + q * 1024);
      }
    }
    for (int q = wv; q < dvox / DL; q += NV) {
      const int v = q * DL + dv;
      const long long m =
          g.stride ? (((long long)bn_ * s.d + z0 + (v >> 6)) * s.h + y0 + ((v >> 3) & 7)) * s.w +
                         x0 + (v & 7)
                   : m0 + v;
      if (od < co) load_to_lds_async(dy + m * co + od, dl + q * 1024);
    }
  };

  // LDS bytes of this lane's transposing reads: voxel i16 / 4 of an octet,
  // channels 4 (i16 % 4) of the 16-channel half
  const int half = (i16 >> 3) & 1;
  const int sub = (i16 & 3) * 8;
  const int dlane = (oct * 8 + (i16 >> 2)) * DV + sub;

  // the block's steps: [at, end) in steps of its tiles, `stride` tiles apart
  const int first = g.stride ? blockIdx.x : 0;
  const int total = g.tiles * g.steps;
  int at = g.stride ? 0 : blockIdx.x * g.split_steps;
  const int end = g.stride ? (first < g.tiles ? (g.tiles - first + g.stride - 1) / g.stride * g.steps : 0)
                           : (at + g.split_steps < total ? at + g.split_steps : total);
  const int hop = g.stride ? g.stride : 1;
  for_share<NW>(share, [&](auto index) {
    constexpr int U0 = U * decltype(index)::value / NW, U1 = U * (decltype(index)::value + 1) / NW;
    f32x4 acc[3 * (U1 - U0)];
#pragma unroll
    for (int j = 0; j < 3 * (U1 - U0); ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int buf = 0;
    if (g.buffers == 2 && at < end) stage(first + at / g.steps * hop, 0);
    while (at < end) {
      const int t = at / g.steps, s0 = at - t * g.steps;
      const int s1 = s0 + end - at < g.steps ? s0 + end - at : g.steps;
      if (g.buffers == 1) {
        __syncthreads();  // the previous tile's reads are done
        stage(first + t * hop, 0);
      }
      lds_loads_done();
      __syncthreads();  // (every share of the block passes the same barriers)
      if (g.buffers == 2 && at + s1 - s0 < end) stage(first + (t + 1) * hop, buf ^ 1);
      const unsigned char* xs = Ls + buf * bytes + sub;
      const unsigned char* ds = Ls + buf * bytes + xbytes + dlane;
      // this lane's voxels of a step: 0-3, 4-7 and 8-11 of its octet's row
      const int* tab = xtab[CT == 2 ? ct : 0] + oct * 12 + (i16 >> 2);
      int next[3] = {tab[48 * s0], tab[48 * s0 + 4], tab[48 * s0 + 8]};
#pragma unroll 1
      for (int k = s0; k < s1; ++k) {
        const int xoff[3] = {next[0], next[1], next[2]};
        const int n = 48 * (k + 1 < s1 ? k + 1 : k);
        next[0] = tab[n];
        next[1] = tab[n + 4];
        next[2] = tab[n + 8];
        bwdw_step<RT, U0, U1>(xs, xoff, ds + k * (32 * DV), DV, half, row, plane, acc);
      }
      at += s1 - s0;
      buf ^= g.buffers - 1;
    }
    // rows (co) 4 oct + e of the co tile, column (ci) lane & 15
    const long long base = (long long)blockIdx.x * co * 27 * ci;
    const int c = c0 + 16 * ct + i16;
#pragma unroll
    for (int u = U0; u < U1; ++u) {
      const int p = u / RT, o = o0 + 16 * (u % RT) + 4 * oct;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (o + e < co && c < ci)
            part[base + ((long long)(o + e) * 27 + 3 * p + dx) * ci + c] =
                acc[3 * (u - U0) + dx][e];
    }
  });
}

// wt[ci][tap][co] = w[co][26 - tap][ci]: the backward-data convolution is the
// forward convolution of dy with these weights (mirrored taps, swapped roles).
__global__ void flip_weights_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt,
                                    int ci, int co) {
  const long long n = 27LL * ci * co;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int o = (int)(i % co);
    const long long r = i / co;
    const int t = (int)(r % 27);
    const int c = (int)(r / 27);
    wt[i] = w[((long long)o * 27 + (26 - t)) * ci + c];
  }
}

// Packed weights (see k_steps above) of the forward convolution (FLIP false)
// or of its backward-data convolution, whose weights are flip_weights_kernel's
// (rows ci, K = 27 co); one thread per 16 bytes.  The convolution packed has
// ki input and ko output channels.
template <bool FLIP>
__device__ __forceinline__ void pack_weights_granule(const uint16_t* __restrict__ w,
                                                     uint4* __restrict__ out, int ki, int ko,
                                                     int i) {
  const int lane = i & 63, f = i >> 6, steps = k_steps(ki);
  const int row = (f / steps) * 16 + (lane & 15), o = (f % steps) * 4 + (lane >> 4);
  const int g8 = ki >> 3;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < ko && o < 27 * g8) {
    if constexpr (!FLIP) {
      v = *reinterpret_cast<const uint4*>(w + ((long long)row * 27 * g8 + o) * 8);
    } else {
      // value j: w[c][26 - tap][row], c = channel 8 (o % g8) + j of the tap o / g8
      const int tap = o / g8, c = 8 * (o - tap * g8);
      uint32_t h[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) h[j] = w[((long long)(c + j) * 27 + (26 - tap)) * ko + row];
      v = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                     h[6] | (h[7] << 16));
    }
  }
  out[i] = v;
}
template <bool FLIP>
__global__ __launch_bounds__(256) void pack_weights_kernel(const uint16_t* __restrict__ w,
                                                           uint4* __restrict__ out, int ki, int ko,
                                                           int total) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < total) pack_weights_granule<FLIP>(w, out, ki, ko, i);
}

// ------------------------------------------------------- backward weights
// dw[co][k] = sum_m dy[m][co] * x[m + off(tap(k))][ci(k)], split over voxel
// ranges: workgroup (tile of 64 co x 64 k, split s) writes its partial tile to
// part[s][co][k]; a second kernel folds the splits in order.  MFMA A operand =
// dy^T (co rows, m as the reduction), B operand = im2col(x) (m x k).
constexpr int kWM = 64;  // voxels per stage

// Voxel coordinates advanced by `step` voxels (row-major n, z, y, x).
__device__ __forceinline__ void advance_voxel(int& n, int& z, int& y, int& x, int step,
                                              const Shape& s) {
  x += step;
  while (x >= s.w) {
    x -= s.w;
    if (++y == s.h) {
      y = 0;
      if (++z == s.d) {
        z = 0;
        ++n;
      }
    }
  }
}

// 8 x 8 transpose of 16-bit values: in[v] holds 8 consecutive columns of
// voxel v (dword i = columns 2i, 2i+1); out[c] holds the 8 voxels of column
// c (dword p = voxels 2p, 2p+1).
__device__ __forceinline__ void transpose8x8(const uint4 (&in)[8], uint4 (&out)[8]) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    uint32_t o[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint32_t a = reinterpret_cast<const uint32_t*>(&in[2 * p])[c >> 1];
      const uint32_t b = reinterpret_cast<const uint32_t*>(&in[2 * p + 1])[c >> 1];
      o[p] = (c & 1) ? ((a >> 16) | (b & 0xFFFF0000u)) : ((a & 0xFFFFu) | (b << 16));
    }
    out[c] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// Weight gradient tile: TM output channels (32 or 64) x 64 im2col columns,
// reduced over a split's voxels in stages of 64.  A stage of each operand is
// cut into 8-column x 8-voxel blocks; thread t < TM loads dy block t, thread
// TM <= t < TM + 64 loads x block t - TM (8 gathered 16-byte loads, one per
// voxel: the 8 columns share one tap), transposes it in registers and writes
// 8 rows of 16 bytes to LDS ([column][voxel]), the layout the MFMA reduction
// over voxels needs.  With TM = 64 wavefront wv computes rows 16 wv..+15
// against four 16-column tiles; with TM = 32 it computes rows 16 (wv % 2)
// against tiles 2 (wv / 2), +1.  One stage of register prefetch.
template <int TM>
__global__ __launch_bounds__(256) void conv_bwdw_kernel(const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ dy,
                                                        float* __restrict__ part, Shape s, int ci,
                                                        int co, long long chunks_per_split) {
  constexpr int LDW = kWM + kPad;
  __shared__ __attribute__((aligned(16))) uint16_t Ds[TM][LDW];  // [co][m]
  __shared__ __attribute__((aligned(16))) uint16_t Xs[64][LDW];  // [k][m]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int K = 27 * ci;
  const int c0 = blockIdx.x * TM;   // co tile
  const int kt0 = blockIdx.y * 64;  // k tile
  const long long mbeg = (long long)blockIdx.z * chunks_per_split * kWM;
  const long long mend = std::min<long long>(s.m, mbeg + chunks_per_split * kWM);

  // this thread's block: columns 8 cb .. 8 cb + 7 of dy (is_dy) or of im2col(x),
  // voxels 8 vb .. 8 vb + 7 of the stage
  const bool is_dy = tid < TM;
  const bool has_block = tid < TM + 64;
  const int blk = is_dy ? tid : tid - TM;
  const int cb = blk >> 3, vb = blk & 7;
  const int col = is_dy ? c0 + 8 * cb : kt0 + 8 * cb;
  const bool col_ok = has_block && (is_dy ? col < co : col < K);
  const int tap = (!is_dy && col_ok) ? col / ci : 0;
  const int ch = is_dy ? 0 : col - tap * ci;
  const int dz = tap / 9 - 1, dyo = (tap / 3) % 3 - 1, dxo = tap % 3 - 1;
  int vn = 0, vz = 0, vy = 0, vx = 0;  // coordinates of the block's first voxel
  {
    const long long m = mbeg + 8 * vb;
    if (m < s.m) unflatten(m, s, vn, vz, vy, vx);
  }
  uint4 raw[8];
  auto gload = [&](long long mc) {
    int n = vn, z = vz, y = vy, xx = vx;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const long long m = mc + 8 * vb + j;
      raw[j] = make_uint4(0, 0, 0, 0);
      if (col_ok && m < mend) {
        if (is_dy) {
          raw[j] = *reinterpret_cast<const uint4*>(dy + m * co + col);
        } else {
          int zz = z + dz, yy = y + dyo, xq = xx + dxo;
          zz = zz < 0 ? zz + s.d : (zz >= s.d ? zz - s.d : zz);
          yy = yy < 0 ? yy + s.h : (yy >= s.h ? yy - s.h : yy);
          xq = xq < 0 ? xq + s.w : (xq >= s.w ? xq - s.w : xq);
          const long long v = (((long long)n * s.d + zz) * s.h + yy) * s.w + xq;
          raw[j] = *reinterpret_cast<const uint4*>(x + v * ci + ch);
        }
      }
      advance_voxel(n, z, y, xx, 1, s);
    }
  };
  constexpr int NT = TM == 64 ? 4 : 2;  // column tiles per wavefront
  const int row0 = TM == 64 ? 16 * wv : 16 * (wv & 1);
  const int tile0 = TM == 64 ? 0 : 2 * (wv >> 1);
  f32x4 acc[NT];
#pragma unroll
  for (int b = 0; b < NT; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (has_block) gload(mbeg);
  for (long long mc = mbeg; mc < mend; mc += kWM) {
    if (has_block) {
      uint4 tr[8];
      transpose8x8(raw, tr);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint16_t* dst = is_dy ? &Ds[8 * cb + e][8 * vb] : &Xs[8 * cb + e][8 * vb];
        *reinterpret_cast<uint4*>(dst) = tr[e];
      }
    }
    __syncthreads();
    if (has_block && mc + kWM < mend) {
      advance_voxel(vn, vz, vy, vx, kWM, s);
      gload(mc + kWM);
    }
    if (c0 + row0 < co) {
#pragma unroll
      for (int ks = 0; ks < kWM; ks += 32) {
        const int kk = ks + 8 * (lane >> 4);
        const bf16x8 a = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const uint4*>(&Ds[row0 + (lane & 15)][kk]));
#pragma unroll
        for (int b = 0; b < NT; ++b) {
          const bf16x8 bf = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const uint4*>(&Xs[(tile0 + b) * 16 + (lane & 15)][kk]));
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bf, acc[b], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  float* out = part + (long long)blockIdx.z * co * K;
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int k = kt0 + (tile0 + b) * 16 + (lane & 15);
    if (k >= K) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = c0 + row0 + (lane >> 4) * 4 + i;
      if (o < co) out[(long long)o * K + k] = acc[b][i];
    }
  }
}

// dw[i] = the splits' partials of i, added in order.  A thread's adds are a
// serial chain, but their loads are not: kFold of them are in flight (64^3 x 4
// training step, weight and bias folds together: 121 us, 188 with eight at a
// time; the bias folds have a kernel of their own since).
constexpr int kFold = 32;
__global__ __launch_bounds__(256) void fold_splits_kernel(const float* __restrict__ part,
                                                          float* __restrict__ dw, long long n,
                                                          int splits) {
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += gridDim.x * 256LL) {
    float a = 0.f;
    int s = 0;
    for (; s + kFold <= splits; s += kFold) {
      float v[kFold];
#pragma unroll
      for (int j = 0; j < kFold; ++j) v[j] = part[(long long)(s + j) * n + i];
#pragma unroll
      for (int j = 0; j < kFold; ++j) a += v[j];
    }
#pragma unroll 8
    for (; s < splits; ++s) a += part[(long long)s * n + i];
    dw[i] = a;
  }
}

// db[c] = sum_m dy[m][c], first pass: block b sums voxels [b per, (b+1) per)
// into part[b][c].  Thread (g, ch) of the G = 256 / c groups handles
// channel ch (consecutive threads read consecutive channels of a voxel) and
// voxels g, g + G, ...; the groups are folded in a fixed order in LDS, and
// fold_bias_kernel sums the blocks in order (deterministic).
__global__ __launch_bounds__(256) void bias_grad_part_kernel(const float* __restrict__ dy,
                                                             float* __restrict__ part,
                                                             long long m, int c,
                                                             long long per) {
  __shared__ float sh[256];
  const int G = c <= 256 ? 256 / c : 1;
  const long long beg = (long long)blockIdx.x * per;
  const long long end = beg + per < m ? beg + per : m;
  for (int cb = 0; cb < c; cb += 256) {
    const int tid = threadIdx.x;
    const int g = c <= 256 ? tid / c : 0;
    const int ch = c <= 256 ? tid % c : cb + tid;
    float a = 0.f;
    if (g < G && ch < c)
      for (long long v = beg + g; v < end; v += G) a += dy[v * c + ch];
    sh[tid] = a;
    __syncthreads();
    if (c <= 256) {
      if (tid < c) {
        float t = 0.f;
        for (int q = 0; q < G; ++q) t += sh[q * c + tid];
        part[(long long)blockIdx.x * c + tid] = t;
      }
    } else if (ch < c) {
      part[(long long)blockIdx.x * c + ch] = a;
    }
    __syncthreads();
    if (c <= 256) break;
  }
}

constexpr int kBiasSplits = 512;

// Bias-gradient partial sums with four consecutive channels per thread (c a
// multiple of 4, at most 1024): thread (g, q) of a block sums channels
// 4q..4q+3 over the block's voxels v = beg + g, beg + g + G, ... (G = 256 /
// (c / 4) voxel groups), then the block adds the G partial sums in order.
// Both nn_bias_grad (dz given, FUSED false) and nn_relu_backward_bias (dz =
// relu'(a) da, stored as BF16, FUSED true) sum in this order, so their db
// agree bit for bit.  vec selects 16-byte FP32 and 8-byte BF16 accesses when
// the pointers allow them (the order is the same either way).
//
// Bound by memory.  A thread's sum is a serial chain, so the loads of kBiasAhead
// voxels are issued before the first of them is added, and where the splits
// alone are too few blocks the channels are shared by blocks too (blockIdx.y:
// qs quads each).  All eight layers of a 64^3 x 4 training step: 202 us, 332 with
// the loads left to the compiler and 8 to 512 blocks; the largest layer's 268 MB
// in 48 us (73).
//
// With POOLED the gradient da is not stored: it is formed from the layers
// above, da[v] = 0.125 pooled[parent of v] + cat[v][ca + ch], the pooling's
// gradient plus the skip's slice of the concatenation's gradient (pooled
// float (n, d/2, h/2, w/2, c), cat float (m, ca + c)).
constexpr int kBiasAhead = 8;
struct PooledSource {
  const float* cat;
  int ca;
  int d, h, w;                 // fine box
  uint32_t by_w, by_h, by_d;   // ceil(2^32 / edge): divisions by __umulhi
};
template <bool FUSED, bool POOLED>
__global__ __launch_bounds__(256) void bias4_part_kernel(const float* __restrict__ da,
                                                         const uint16_t* __restrict__ a,
                                                         uint16_t* __restrict__ dzb,
                                                         float* __restrict__ part, long long m,
                                                         int c, int qs, long long per, int relu,
                                                         int vec, PooledSource src) {
  __shared__ float4 sh[256];
  const int G = 256 / (c >> 2);
  const int tid = threadIdx.x, g = tid / qs, ql = tid - g * qs;
  const int ch = 4 * ((int)blockIdx.y * qs + ql);
  const long long beg = (long long)blockIdx.x * per;
  const long long end = beg + per < m ? beg + per : m;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);

  auto gradient = [&](long long v, float4& z, float4& k) {
    if constexpr (POOLED) {
      const uint32_t r = __umulhi((uint32_t)v, src.by_w), x = (uint32_t)v - r * src.w;
      const uint32_t t = __umulhi(r, src.by_h), y = r - t * src.h;
      const uint32_t b = __umulhi(t, src.by_d), zz = t - b * src.d;
      const long long p = ((long long)(b * (src.d / 2) + zz / 2) * (src.h / 2) + y / 2) *
                              (src.w / 2) + x / 2;
      z = *reinterpret_cast<const float4*>(da + p * c + ch);
      k = *reinterpret_cast<const float4*>(src.cat + v * (src.ca + c) + src.ca + ch);
    } else if (vec) {
      z = *reinterpret_cast<const float4*>(da + v * c + ch);
    } else {
      const float* d = da + v * c + ch;
      z = make_float4(d[0], d[1], d[2], d[3]);
    }
  };
  auto activation = [&](long long v) {
    const uint16_t* h = a + v * c + ch;
    if (vec) return *reinterpret_cast<const uint2*>(h);
    return make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16),
                      (uint32_t)h[2] | ((uint32_t)h[3] << 16));
  };
  auto take = [&](long long v, float4 z, float4 k, uint2 h) {
    if constexpr (POOLED) {
      const float px = 0.125f * z.x, py = 0.125f * z.y, pz = 0.125f * z.z, pw = 0.125f * z.w;
      z = make_float4(px + k.x, py + k.y, pz + k.z, pw + k.w);
    }
    if constexpr (FUSED) {
      if (relu) {
        if (!(bf2f((uint16_t)h.x) > 0.f)) z.x = 0.f;
        if (!(bf2f((uint16_t)(h.x >> 16)) > 0.f)) z.y = 0.f;
        if (!(bf2f((uint16_t)h.y) > 0.f)) z.z = 0.f;
        if (!(bf2f((uint16_t)(h.y >> 16)) > 0.f)) z.w = 0.f;
      }
      const uint16_t o[4] = {f2bf(z.x), f2bf(z.y), f2bf(z.z), f2bf(z.w)};
      uint16_t* d = dzb + v * c + ch;
      if (vec)
        *reinterpret_cast<uint2*>(d) =
            make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
      else
        for (int j = 0; j < 4; ++j) d[j] = o[j];
    }
    s.x += z.x;
    s.y += z.y;
    s.z += z.z;
    s.w += z.w;
  };

  long long v = beg + g;
  for (; v + (kBiasAhead - 1) * G < end; v += kBiasAhead * G) {
    float4 z[kBiasAhead], k[kBiasAhead];
    uint2 h[kBiasAhead] = {};
    if (FUSED && relu)
#pragma unroll
      for (int j = 0; j < kBiasAhead; ++j) h[j] = activation(v + j * G);
#pragma unroll
    for (int j = 0; j < kBiasAhead; ++j) gradient(v + j * G, z[j], k[j]);
#pragma unroll
    for (int j = 0; j < kBiasAhead; ++j) take(v + j * G, z[j], k[j], h[j]);
  }
  for (; v < end; v += G) {
    float4 z, k;
    gradient(v, z, k);
    take(v, z, k, FUSED && relu ? activation(v) : make_uint2(0, 0));
  }
  sh[tid] = s;
  __syncthreads();
  if (tid < qs) {
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r = 0; r < G; ++r) {
      const float4 u = sh[r * qs + tid];
      t.x += u.x;
      t.y += u.y;
      t.z += u.z;
      t.w += u.w;
    }
    float* out = part + (long long)blockIdx.x * c + ch;
    out[0] = t.x;
    out[1] = t.y;
    out[2] = t.z;
    out[3] = t.w;
  }
}
bool bias4(int c) { return c % 4 == 0 && c <= 1024; }

// db[c] = the splits' partials of c (at most kBiasSplits), added in order.
// fold_splits_kernel's chains are as long as here but have only c of them, each
// waiting for sixteen rounds of loads (8.5 us for 512 splits of 32 channels);
// here a block's 16 groups of threads bring the partials of 32 channels to LDS
// in one round, and the chains run from there (6 us, of which 4.5 are the
// launch; the eight of a 64^3 x 4 training step 57 -> 45).
__global__ __launch_bounds__(512) void fold_bias_kernel(const float* __restrict__ part,
                                                        float* __restrict__ db, int c,
                                                        int splits) {
  __shared__ float sh[kBiasSplits * 32];
  const int l = threadIdx.x & 31, g = threadIdx.x >> 5, ch = blockIdx.x * 32 + l;
  const int cc = ch < c ? ch : c - 1;
  float v[kBiasSplits / 16];
#pragma unroll
  for (int j = 0; j < kBiasSplits / 16; ++j) {
    const int s = g + 16 * j;
    v[j] = part[(long long)(s < splits ? s : splits - 1) * c + cc];
  }
#pragma unroll
  for (int j = 0; j < kBiasSplits / 16; ++j) sh[(g + 16 * j) * 32 + l] = v[j];
  __syncthreads();
  if (g || ch >= c) return;
  float a = 0.f;
#pragma unroll 16
  for (int s = 0; s < splits; ++s) a += sh[s * 32 + l];
  db[ch] = a;
}

// Blocks of `splits` voxel ranges: the channels are halved among blocks until
// two of them per compute unit are there, in slices of at least 8 quads (128
// bytes of a row).
template <bool FUSED, bool POOLED>
void launch_bias4(const float* da, const void* a, void* dz, void* ws, long long m, int c,
                  long long splits, long long per, int relu, int vec, const PooledSource& src,
                  void* stream) {
  int slices = 1, qs = c / 4;
  const int groups = 256 / qs;
  while (splits * slices < 512 && qs % 2 == 0 && qs >= 16) slices *= 2, qs /= 2;
  bias4_part_kernel<FUSED, POOLED>
      <<<dim3((unsigned)splits, slices), groups * qs, 0, (hipStream_t)stream>>>(
          da, (const uint16_t*)a, (uint16_t*)dz, (float*)ws, m, c, qs, per, relu, vec, src);
}

// The backward of a layer's activation, fused with what the convolution's
// backward needs from it: dz = (relu ? (a > 0 ? da : 0) : da) stored as BF16
// (the MFMA operand of both convolution gradients), and the first pass of
// db = sum_m dz[m][c] over the FP32 dz, in bias_grad_part_kernel's order (so
// db is bit-identical to nn_bias_grad of the FP32 dz).
__global__ __launch_bounds__(256) void relu_bwd_bias_part_kernel(
    const float* __restrict__ da, const uint16_t* __restrict__ a, uint16_t* __restrict__ dzb,
    float* __restrict__ part, long long m, int c, long long per, int relu) {
  __shared__ float sh[256];
  const int G = c <= 256 ? 256 / c : 1;
  const long long beg = (long long)blockIdx.x * per;
  const long long end = beg + per < m ? beg + per : m;
  for (int cb = 0; cb < c; cb += 256) {
    const int tid = threadIdx.x;
    const int g = c <= 256 ? tid / c : 0;
    const int ch = c <= 256 ? tid % c : cb + tid;
    float s = 0.f;
    if (g < G && ch < c)
      for (long long v = beg + g; v < end; v += G) {
        const long long i = v * c + ch;
        float z = da[i];
        if (relu && !(bf2f(a[i]) > 0.f)) z = 0.f;
        dzb[i] = f2bf(z);
        s += z;
      }
    sh[tid] = s;
    __syncthreads();
    if (c <= 256) {
      if (tid < c) {
        float t = 0.f;
        for (int q = 0; q < G; ++q) t += sh[q * c + tid];
        part[(long long)blockIdx.x * c + tid] = t;
      }
    } else if (ch < c) {
      part[(long long)blockIdx.x * c + ch] = s;
    }
    __syncthreads();
    if (c <= 256) break;
  }
}

// --------------------------------------------------------------- elementwise

__global__ void relu_fwd_kernel(const float* __restrict__ z, uint16_t* __restrict__ a,
                                long long n, int relu) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    a[i] = f2bf(relu ? fmaxf(z[i], 0.f) : z[i]);
}

// dz = da where the stored activation is positive
__global__ void relu_bwd_kernel(const float* __restrict__ da, const uint16_t* __restrict__ a,
                                float* __restrict__ dz, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    dz[i] = bf2f(a[i]) > 0.f ? da[i] : 0.f;
}

__global__ void cast_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y,
                                 long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    y[i] = f2bf(x[i]);
}

// Four-element forms of the activation, its gradient and the cast (16-byte
// FP32 words, 8-byte BF16 words), for counts that are multiples of 4 and
// aligned pointers.
__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
  return make_uint2((uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16),
                    (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16));
}

__global__ void relu_fwd_vec_kernel(const float4* __restrict__ z, uint2* __restrict__ a,
                                    long long n4, int relu) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
       i += (long long)gridDim.x * blockDim.x) {
    float4 v = z[i];
    if (relu) {
      v.x = fmaxf(v.x, 0.f);
      v.y = fmaxf(v.y, 0.f);
      v.z = fmaxf(v.z, 0.f);
      v.w = fmaxf(v.w, 0.f);
    }
    a[i] = pack_bf16x4(v.x, v.y, v.z, v.w);
  }
}

__global__ void relu_bwd_vec_kernel(const float4* __restrict__ da, const uint2* __restrict__ a,
                                    float4* __restrict__ dz, long long n4) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
       i += (long long)gridDim.x * blockDim.x) {
    const float4 g = da[i];
    const uint2 h = a[i];
    dz[i] = make_float4(bf2f((uint16_t)h.x) > 0.f ? g.x : 0.f,
                        bf2f((uint16_t)(h.x >> 16)) > 0.f ? g.y : 0.f,
                        bf2f((uint16_t)h.y) > 0.f ? g.z : 0.f,
                        bf2f((uint16_t)(h.y >> 16)) > 0.f ? g.w : 0.f);
  }
}

__global__ void cast_bf16_vec_kernel(const float4* __restrict__ x, uint2* __restrict__ y,
                                     long long n4) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
       i += (long long)gridDim.x * blockDim.x) {
    const float4 v = x[i];
    y[i] = pack_bf16x4(v.x, v.y, v.z, v.w);
  }
}

// 2x2x2 average pooling (fine shape s, coarse = halves), bf16 in/out
__global__ void pool_fwd_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, Shape s,
                                int c) {
  const Shape q{s.n, s.d / 2, s.h / 2, s.w / 2, s.m / 8};
  const long long n = q.m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % c);
    int vn, vz, vy, vx;
    unflatten(i / c, q, vn, vz, vy, vx);
    float a = 0.f;
    for (int o = 0; o < 8; ++o) {
      const long long f = (((long long)vn * s.d + 2 * vz + (o >> 2)) * s.h + 2 * vy + ((o >> 1) & 1)) *
                              s.w + 2 * vx + (o & 1);
      a += bf2f(x[f * c + ch]);
    }
    y[i] = f2bf(0.125f * a);
  }
}

// gradient of the average pooling: each fine voxel gets 1/8 of its parent
__global__ void pool_bwd_kernel(const float* __restrict__ dy, float* __restrict__ dx, Shape s,
                                int c) {
  const Shape q{s.n, s.d / 2, s.h / 2, s.w / 2, s.m / 8};
  const long long n = s.m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % c);
    int vn, vz, vy, vx;
    unflatten(i / c, s, vn, vz, vy, vx);
    const long long p = (((long long)vn * q.d + vz / 2) * q.h + vy / 2) * q.w + vx / 2;
    dx[i] = 0.125f * dy[p * c + ch];
  }
}

// nearest-neighbour upsampling x2 (coarse shape q -> fine), bf16 in/out
__global__ void up_fwd_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, Shape q,
                              int c) {
  const Shape s{q.n, q.d * 2, q.h * 2, q.w * 2, q.m * 8};
  const long long n = s.m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % c);
    int vn, vz, vy, vx;
    unflatten(i / c, s, vn, vz, vy, vx);
    const long long p = (((long long)vn * q.d + vz / 2) * q.h + vy / 2) * q.w + vx / 2;
    y[i] = x[p * c + ch];
  }
}

// gradient of the upsampling: sum over the 8 fine children
__global__ void up_bwd_kernel(const float* __restrict__ dy, float* __restrict__ dx, Shape q,
                              int c) {
  const Shape s{q.n, q.d * 2, q.h * 2, q.w * 2, q.m * 8};
  const long long n = q.m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % c);
    int vn, vz, vy, vx;
    unflatten(i / c, q, vn, vz, vy, vx);
    float a = 0.f;
    for (int o = 0; o < 8; ++o) {
      const long long f = (((long long)vn * s.d + 2 * vz + (o >> 2)) * s.h + 2 * vy + ((o >> 1) & 1)) *
                              s.w + 2 * vx + (o & 1);
      a += dy[f * c + ch];
    }
    dx[i] = a;
  }
}

// y = [a | b] along channels (bf16)
__global__ void concat_kernel(const uint16_t* __restrict__ a, const uint16_t* __restrict__ b,
                              uint16_t* __restrict__ y, long long m, int ca, int cb) {
  const int c = ca + cb;
  const long long n = m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const long long v = i / c;
    const int ch = (int)(i % c);
    y[i] = ch < ca ? a[v * ca + ch] : b[v * cb + ch - ca];
  }
}

// da, db = split of dy along channels (fp32); either output may be null
__global__ void split_kernel(const float* __restrict__ dy, float* __restrict__ da,
                             float* __restrict__ db, long long m, int ca, int cb) {
  const int c = ca + cb;
  const long long n = m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const long long v = i / c;
    const int ch = (int)(i % c);
    if (ch < ca) {
      if (da) da[v * ca + ch] = dy[i];
    } else if (db) {
      db[v * cb + ch - ca] = dy[i];
    }
  }
}

__global__ void add_kernel(float* __restrict__ y, const float* __restrict__ x, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    y[i] += x[i];
}

// Masked mean-squared error over the first `used` of c channels at voxels
// with weight[m] > 0: loss partials per block (fixed tree), gradient
// 2 (pred - target) weight / norm.
__global__ __launch_bounds__(256) void mse_kernel(const float* __restrict__ pred,
                                                  const float* __restrict__ target,
                                                  const float* __restrict__ weight,
                                                  float* __restrict__ grad,
                                                  double* __restrict__ partial, long long m, int c,
                                                  int used, double inv_norm) {
  __shared__ double sh[256];
  double a = 0.0;
  const long long n = m * c;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const long long v = i / c;
    const int ch = (int)(i % c);
    float g = 0.f;
    if (ch < used && weight[v] > 0.f) {
      const float d = pred[i] - target[v * used + ch];
      a += (double)d * d * weight[v];
      g = (float)(2.0 * d * weight[v] * inv_norm);
    }
    grad[i] = g;
  }
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = sh[0] * inv_norm;
}

__device__ __forceinline__ void adam_one(float* __restrict__ w, const float* __restrict__ g,
                                         float* __restrict__ m1, float* __restrict__ m2,
                                         uint16_t* __restrict__ wb, long long i, float lr, float b1,
                                         float b2, float eps, float c1, float c2) {
  const float gi = g[i];
  const float a = b1 * m1[i] + (1.f - b1) * gi;
  const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
  m1[i] = a;
  m2[i] = b;
  const float wi = w[i] - lr * (a * c1) / (sqrtf(b * c2) + eps);
  w[i] = wi;
  if (wb) wb[i] = f2bf(wi);
}

// Adam update of FP32 master weights, refreshing the BF16 copy.
__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g,
                            float* __restrict__ m1, float* __restrict__ m2,
                            uint16_t* __restrict__ wb, long long n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    adam_one(w, g, m1, m2, wb, i, lr, b1, b2, eps, c1, c2);
}

// Many tensors in one launch, described by the kernel's arguments: a network's
// optimizer step is tens of tensors of a few hundred KB at most, each of which
// takes less time than its launch (the sixteen updates and sixteen packings of
// a 64^3 x 4 training step: 26 us in two launches, about 90 in 32).  A block does kItemSpan elements of one
// item; items start at the blocks `first` and are in order.
constexpr int kItems = 24, kItemSpan = 1024;
template <typename T>
struct ItemList {
  T item[kItems];
  int first[kItems + 1];
  int n;
};
template <typename T>
__device__ __forceinline__ int item_of(const ItemList<T>& l, int block) {
  int k = 0;
  while (k + 1 < l.n && block >= l.first[k + 1]) ++k;
  return k;
}
__global__ __launch_bounds__(256) void adam_many_kernel(const ItemList<nn_adam_tensor> l, float lr,
                                                        float b1, float b2, float eps, float c1,
                                                        float c2) {
  const int k = item_of(l, blockIdx.x);
  const nn_adam_tensor t = l.item[k];
  const long long beg = (long long)(blockIdx.x - l.first[k]) * kItemSpan;
#pragma unroll
  for (int j = 0; j < kItemSpan; j += 256) {
    const long long i = beg + j + threadIdx.x;
    if (i < t.n)
      adam_one(t.w, t.g, t.m1, t.m2, (uint16_t*)t.w_bf16, i, lr, b1, b2, eps, c1, c2);
  }
}
__global__ __launch_bounds__(256) void pack_many_kernel(const ItemList<nn_pack_item> l) {
  const int k = item_of(l, blockIdx.x);
  const nn_pack_item t = l.item[k];
  const int ki = t.flip ? t.co : t.ci, ko = t.flip ? t.ci : t.co;
  const int total = (ko + 15) / 16 * k_steps(ki) * 64;
#pragma unroll
  for (int j = 0; j < kItemSpan; j += 256) {
    const int i = (blockIdx.x - l.first[k]) * kItemSpan + j + (int)threadIdx.x;
    if (i >= total) continue;
    if (t.flip)
      pack_weights_granule<true>((const uint16_t*)t.w, (uint4*)t.packed, ki, ko, i);
    else
      pack_weights_granule<false>((const uint16_t*)t.w, (uint4*)t.packed, ki, ko, i);
  }
}

int grid_for(long long n) { return (int)std::min<long long>((n + 255) / 256, 8192); }

lbm_status check_launch() {
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_ERR_DEVICE;
}

Shape shape_of(int n, int d, int h, int w) {
  return Shape{n, d, h, w, (long long)n * d * h * w};
}

bool bad_shape(int n, int d, int h, int w) { return n < 1 || d < 1 || h < 1 || w < 1; }

// Granule forms of the pooling, upsampling, concatenation and split kernels:
// one thread moves 8 BF16 (or 4 FP32) channels of a voxel as one 16-byte
// word, with 32-bit index arithmetic.  Used when the channel counts are
// multiples of the granule, the pointers 16-byte aligned and the element
// count below 2^31; the element forms above cover the rest.
bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

__device__ __forceinline__ void voxel_of(int v, int d, int h, int w, int& n, int& z, int& y,
                                         int& x) {
  x = v % w;
  v /= w;
  y = v % h;
  v /= h;
  z = v % d;
  n = v / d;
}

__global__ void pool_fwd_vec_kernel(const uint4* __restrict__ x, uint4* __restrict__ y, int n_,
                                    int d, int h, int w, int g) {
  const int qd = d / 2, qh = h / 2, qw = w / 2;
  const int total = n_ * qd * qh * qw * g;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int gi = i % g;
    int vn, vz, vy, vx;
    voxel_of(i / g, qd, qh, qw, vn, vz, vy, vx);
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int o = 0; o < 8; ++o) {
      const int f = ((vn * d + 2 * vz + (o >> 2)) * h + 2 * vy + ((o >> 1) & 1)) * w + 2 * vx + (o & 1);
      const uint4 u = x[f * g + gi];
      const uint32_t q[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a[2 * k] += bf2f((uint16_t)q[k]);
        a[2 * k + 1] += bf2f((uint16_t)(q[k] >> 16));
      }
    }
    uint32_t r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      r[k] = (uint32_t)f2bf(0.125f * a[2 * k]) | ((uint32_t)f2bf(0.125f * a[2 * k + 1]) << 16);
    y[i] = make_uint4(r[0], r[1], r[2], r[3]);
  }
}

__global__ void pool_bwd_vec_kernel(const float4* __restrict__ dy, float4* __restrict__ dx,
                                    int n_, int d, int h, int w, int g) {
  const int total = n_ * d * h * w * g;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int gi = i % g;
    int vn, vz, vy, vx;
    voxel_of(i / g, d, h, w, vn, vz, vy, vx);
    const int p = ((vn * (d / 2) + vz / 2) * (h / 2) + vy / 2) * (w / 2) + vx / 2;
    const float4 v = dy[p * g + gi];
    dx[i] = make_float4(0.125f * v.x, 0.125f * v.y, 0.125f * v.z, 0.125f * v.w);
  }
}

// coarse (n, d, h, w) -> fine (n, 2d, 2h, 2w)
__global__ void up_fwd_vec_kernel(const uint4* __restrict__ x, uint4* __restrict__ y, int n_,
                                  int d, int h, int w, int g) {
  const int total = n_ * 8 * d * h * w * g;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int gi = i % g;
    int vn, vz, vy, vx;
    voxel_of(i / g, 2 * d, 2 * h, 2 * w, vn, vz, vy, vx);
    const int p = ((vn * d + vz / 2) * h + vy / 2) * w + vx / 2;
    y[i] = x[p * g + gi];
  }
}

// Fine rows of dy are gs granules apart: gs > g reads the first channels of the
// concatenation's gradient in place, which spares splitting it (three levels of
// a 64^3 x 4 training step: 78 us, 275 with the split).
__global__ void up_bwd_vec_kernel(const float4* __restrict__ dy, float4* __restrict__ dx, int n_,
                                  int d, int h, int w, int g, int gs) {
  const int total = n_ * d * h * w * g;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int gi = i % g;
    int vn, vz, vy, vx;
    voxel_of(i / g, d, h, w, vn, vz, vy, vx);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int o = 0; o < 8; ++o) {
      const int f = ((vn * 2 * d + 2 * vz + (o >> 2)) * 2 * h + 2 * vy + ((o >> 1) & 1)) * 2 * w +
                    2 * vx + (o & 1);
      const float4 v = dy[(long long)f * gs + gi];
      a.x += v.x;
      a.y += v.y;
      a.z += v.z;
      a.w += v.w;
    }
    dx[i] = a;
  }
}

// granules of 8 bf16 channels: ga + gb per voxel
__global__ void concat_vec_kernel(const uint4* __restrict__ a, const uint4* __restrict__ b,
                                  uint4* __restrict__ y, int m, int ga, int gb) {
  const int g = ga + gb, total = m * g;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int v = i / g, k = i % g;
    y[i] = k < ga ? a[v * ga + k] : b[v * gb + k - ga];
  }
}

// y = [upsampled a | b]: granules ga of the coarse a (n, d, h, w) and gb of the
// fine b.  Bound by memory: the upsampled tensor is neither written nor read
// again (the three levels of a 64^3 x 4 network: 76 us, 140 in two kernels).
__global__ __launch_bounds__(256) void upsample_concat_kernel(const uint4* __restrict__ a,
                                                              const uint4* __restrict__ b,
                                                              uint4* __restrict__ y, int n_, int d,
                                                              int h, int w, int ga, int gb) {
  const int g = ga + gb, total = n_ * 8 * d * h * w * g;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int v = i / g, k = i - v * g;
    if (k < ga) {
      int vn, vz, vy, vx;
      voxel_of(v, 2 * d, 2 * h, 2 * w, vn, vz, vy, vx);
      y[i] = a[(((vn * d + vz / 2) * h + vy / 2) * w + vx / 2) * ga + k];
    } else {
      y[i] = b[(long long)v * gb + k - ga];
    }
  }
}

// granules of 4 fp32 channels
__global__ void split_vec_kernel(const float4* __restrict__ dy, float4* __restrict__ da,
                                 float4* __restrict__ db, int m, int ga, int gb) {
  const int g = ga + gb, total = m * g;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int v = i / g, k = i % g;
    if (k < ga) {
      if (da) da[v * ga + k] = dy[i];
    } else if (db) {
      db[v * gb + k - ga] = dy[i];
    }
  }
}

}  // namespace

// ------------------------------------------------------------------ C ABI

namespace {

template <bool ACT>
int vector_stores(const void* y, int co) {
  return co % 4 == 0 && ((uintptr_t)y & (ACT ? 7 : 15)) == 0;
}

// Spatially tiled forward convolution: x rows of 16 where the box allows, and
// as many rows per wavefront as still leave about one block per CU (fewer
// operand reads per MFMA with more rows; measured at 64^3 x 4, 96 -> 32
// channels, 8 / 4 / 2 rows: 215 / 314 / 477 us; 16^3 x 4, 384 -> 128, with
// 128 / 256 / 512 blocks: 117 / 96 / 154 us).
template <int TX, int MT, int NT, int WC, bool PK, bool ACT>
void launch_fwd_tile(const uint16_t* x, const uint16_t* w, const float* bias, void* y,
                     const Shape& s, int ci, int co, int relu, hipStream_t st) {
  constexpr int voxels = (4 / WC) * 16 * MT;
  const int cgs = (co + 16 * NT * WC - 1) / (16 * NT * WC);
  conv_fwd_spatial_kernel<TX, MT, NT, WC, PK, ACT><<<(unsigned)(s.m / voxels * cgs), 256, 0, st>>>(
      x, w, bias, y, s, ci, co, relu, vector_stores<ACT>(y, co));
}
constexpr int kFillBlocks = 200;  // enough blocks for the 256 CUs
template <int NT, int WC, bool PK, bool ACT>
void launch_fwd_rows_of(const uint16_t* x, const uint16_t* w, const float* bias, void* y,
                        const Shape& s, int ci, int co, int relu, hipStream_t st) {
  const long long cgs = (co + 16 * NT * WC - 1) / (16 * NT * WC);
  const long long tiles = s.m / ((4 / WC) * 16) * cgs;  // blocks with one tile per wavefront
  if (s.w % 16) {
    launch_fwd_tile<8, 4, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  } else if (tiles >= 8 * kFillBlocks) {
    launch_fwd_tile<16, 8, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  } else if (WC > 1 || tiles >= 4 * kFillBlocks) {
    // (two groups of channels: always so many tiles)
    launch_fwd_tile<16, 4, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  } else {
    if constexpr (WC == 1)
      launch_fwd_tile<16, 2, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  }
}
// Channel groups of 32 per wavefront (16 for few channels); pairs of groups
// share a block's halo where their count is even (96 channels: 257 us with
// one group per block against 293 us with two, a quarter of them empty).
// Multiples of 96 channels are pairs of groups of 48 where two layers a block
// still are two blocks per CU: a fragment serves three weight tiles, the halo
// all channels (32 -> 96 channels at 64^3 x 4, packed, FP32 output 308 -> 287
// us, BF16 221 -> 207; 64 -> 96 at 32^3 x 4: 52 -> 48).
template <bool PK, bool ACT>
void launch_fwd_spatial(const uint16_t* x, const uint16_t* w, const float* bias, void* y,
                        const Shape& s, int ci, int co, int relu, hipStream_t st) {
  if (co <= 16)
    launch_fwd_rows_of<1, 1, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  else if (co % 96 == 0 && s.w % 16 == 0 && s.m / 256 * (co / 96) >= 2 * kFillBlocks)
    launch_fwd_tile<16, 8, 3, 2, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  else if ((co + 31) / 32 % 2)
    launch_fwd_rows_of<2, 1, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  else
    launch_fwd_rows_of<2, 2, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
}

constexpr size_t kLdsBytes = 160 * 1024;  // of a CU

template <int MT, int WC>
long long rows_blocks(const Shape& s, int groups) {
  return (long long)s.n * ((s.d + 4 / WC - 1) / (4 / WC)) * ((s.h + 2 * MT - 1) / (2 * MT)) *
         ((s.w + kRX - 1) / kRX) * groups;
}
template <int MT, int NT, int WC, bool PK, bool ACT>
void launch_rows(const uint16_t* x, const uint16_t* w, const float* bias, void* y, const Shape& s,
                 int ci, int co, int relu, hipStream_t st) {
  const int cgs = (co + 16 * NT * WC - 1) / (16 * NT * WC);
  conv_fwd_rows_kernel<MT, NT, WC, PK, ACT>
      <<<(unsigned)rows_blocks<MT, WC>(s, cgs), 256, rows_lds<MT, WC>(ci), st>>>(
          x, w, bias, y, s, ci, co, relu, vector_stores<ACT>(y, co));
}
// Which of the kernel above with 1, 2 or 4 row pairs a wavefront and the gathered
// tiles takes a box: the least of four estimated times, us.  A launch is whole
// rounds of the blocks that the 256 CUs hold and the last round's fullest CU;
// block(k) is the time of k blocks together on a CU, the larger of a block's own
// latency and what k of them ask of the CU (MFMAs, weights, LDS).  The constants
// are fits to launches of 1400 random boxes (edges 1 to 96, 8 to 512 channels,
// thin and half-empty boxes among them), which they give to 8% (gathered tiles
// 5%).  Halo tiles are taken where they are estimated a fifth ahead: of those
// 1400 boxes, from packed weights, 10 are then 4 to 9% slower than gathered tiles
// from unpacked ones, the mean takes 0.46 of their time.  (Limits on the block
// count in place of the estimates: 75 slower, up to 3.9 times where the edges
// leave the 8-wide tiles empty: 20 x 51 x 1 x 12, 8 -> 512 channels, 50 against
// 20 us.)
//
// Unpacked weights of 32 channels and more are scattered rows that bound the
// launch: there the fewest row pairs whose blocks run at once, one per CU, and
// gathered tiles beyond (20^3 x 3, 64 -> 128: 47 against 42 us).
template <typename F>
double launch_time(long long blocks, long long resident, F block) {
  const long long per = (blocks + 255) / 256, last = per % resident;
  return (double)(per / resident) * block((double)resident) + (last ? block((double)last) : 0.0);
}
template <int MT, int NT, int WC, bool PK>
double rows_time(const Shape& s, int ci, int co) {
  const size_t lds = rows_lds<MT, WC>(ci);
  if (lds > kLdsBytes) return HUGE_VAL;
  const long long blocks = rows_blocks<MT, WC>(s, (co + 16 * NT * WC - 1) / (16 * NT * WC));
  if (!PK && ci >= 32) return blocks <= 256 ? MT : HUGE_VAL;  // (an order, not a time)
  const double steps = k_steps(ci), kb = (double)lds / 1024;
  const double own = PK ? 0.029 + 0.038 * MT : 0.05 * MT;
  const double shared = NT * (PK ? 0.0088 * MT + 0.0187 : 0.0187 * MT + 0.0424);
  const double stage = (PK ? 0.029 : 0.005) * kb, start = PK ? 1.4 : 0.9;
  return (PK ? 3.1 : 3.9) +
         launch_time(blocks, std::min<long long>(4, (long long)(kLdsBytes / lds)),
                     [&](double k) { return start + stage * k + steps * std::max(own, k * shared); });
}
double gathered_time(const Shape& s, int ci, int co) {
  const int nt = co <= 16 ? 1 : (co <= 32 ? 2 : 4);
  const double stages = (27 * ci + 63) / 64;
  return 5.6 + launch_time((s.m + 127) / 128 * ((co + 16 * nt - 1) / (16 * nt)), nt == 4 ? 3 : 4,
                           [&](double k) {
                             return 4.6 + stages * std::max(0.455 + 0.097 * nt,
                                                            k * (0.059 * nt + 0.261));
                           });
}
// False where gathered tiles are the better kernel.
template <int NT, int WC, bool PK, bool ACT>
bool launch_rows_of(const uint16_t* x, const uint16_t* w, const float* bias, void* y,
                    const Shape& s, int ci, int co, int relu, hipStream_t st) {
  const double t1 = rows_time<1, NT, WC, PK>(s, ci, co), t2 = rows_time<2, NT, WC, PK>(s, ci, co),
               t4 = rows_time<4, NT, WC, PK>(s, ci, co);
  const double t = std::min(t1, std::min(t2, t4));
  const double limit = !PK && ci >= 32 ? HUGE_VAL : 0.8 * gathered_time(s, ci, co);
  if (!(t < limit)) return false;
  if (t == t1)
    launch_rows<1, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  else if (t == t2)
    launch_rows<2, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  else
    launch_rows<4, NT, WC, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  return true;
}
template <bool PK, bool ACT>
bool launch_fwd_halo(const uint16_t* x, const uint16_t* w, const float* bias, void* y,
                     const Shape& s, int ci, int co, int relu, hipStream_t st) {
  if (co <= 16) return launch_rows_of<1, 1, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  if (co <= 32) return launch_rows_of<2, 1, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  if (co <= 64) return launch_rows_of<2, 2, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
  return launch_rows_of<2, 4, PK, ACT>(x, w, bias, y, s, ci, co, relu, st);
}

template <bool PK, bool ACT>
lbm_status conv_forward(const void* x, const void* w, const float* bias, void* y, int n, int d,
                        int h, int wd, int ci, int co, int relu, void* stream) {
  if (!x || !w || !y || bad_shape(n, d, h, wd) || ci < 8 || ci % 8 || co < 1)
    return LBM_ERR_INVALID_ARG;
  const Shape s = shape_of(n, d, h, wd);
  if (s.m >= (1LL << 31)) return LBM_ERR_INVALID_ARG;  // voxel indices are 32-bit in the tables
  const int bn = co <= 16 ? 16 : (co <= 32 ? 32 : 64);
  const hipStream_t st = (hipStream_t)stream;
  const uint16_t* xx = (const uint16_t*)x;
  const uint16_t* ww = (const uint16_t*)w;
  // spatial tiles where the box and channels allow and the grid is not tiny
  const long long tiles = s.m / (kTZ * kTY * kTX);
  if (ci % kCC == 0 && d % kTZ == 0 && h % kTY == 0 && wd % kTX == 0 &&
      tiles * ((co + bn - 1) / bn) >= 128 && aligned16(x) && aligned16(w) &&
      s.m * (ci / 8) < (1LL << 31)) {
    launch_fwd_spatial<PK, ACT>(xx, ww, bias, y, s, ci, co, relu, st);
    return check_launch();
  }
  dim3 grid((unsigned)((s.m + 127) / 128), (unsigned)((co + bn - 1) / bn));
  if (aligned16(x) && launch_fwd_halo<PK, ACT>(xx, ww, bias, y, s, ci, co, relu, st))
    return check_launch();
  if (bn == 16)
    conv_fwd_tiled_kernel<16, PK, ACT><<<grid, 256, 0, st>>>(xx, ww, bias, y, s, ci, co, relu);
  else if (bn == 32)
    conv_fwd_tiled_kernel<32, PK, ACT><<<grid, 256, 0, st>>>(xx, ww, bias, y, s, ci, co, relu);
  else
    conv_fwd_tiled_kernel<64, PK, ACT><<<grid, 256, 0, st>>>(xx, ww, bias, y, s, ci, co, relu);
  return check_launch();
}

}  // namespace

NN_API lbm_status nn_conv3d_forward(const void* x, const void* w, const float* bias, float* y,
                                    int n, int d, int h, int wd, int ci, int co, void* stream) {
  return conv_forward<false, false>(x, w, bias, y, n, d, h, wd, ci, co, 0, stream);
}

NN_API lbm_status nn_conv3d_forward_act(const void* x, const void* w, const float* bias, void* a,
                                        int n, int d, int h, int wd, int ci, int co, int relu,
                                        void* stream) {
  if (relu != 0 && relu != 1) return LBM_ERR_INVALID_ARG;
  return conv_forward<false, true>(x, w, bias, a, n, d, h, wd, ci, co, relu, stream);
}

NN_API lbm_status nn_conv3d_flip_weights(const void* w, void* wt, int ci, int co, void* stream) {
  if (!w || !wt || ci < 1 || co < 1) return LBM_ERR_INVALID_ARG;
  flip_weights_kernel<<<grid_for(27LL * ci * co), 256, 0, (hipStream_t)stream>>>(
      (const uint16_t*)w, (uint16_t*)wt, ci, co);
  return check_launch();
}

NN_API lbm_status nn_conv3d_packed_bytes(int ci, int co, size_t* bytes) {
  if (!bytes || ci < 8 || ci % 8 || co < 1) return LBM_ERR_INVALID_ARG;
  *bytes = (size_t)((co + 15) / 16) * k_steps(ci) * 1024;
  return LBM_OK;
}

NN_API lbm_status nn_conv3d_pack_weights(const void* w, void* packed, int ci, int co, int flip,
                                         void* stream) {
  if (!w || !packed || ci < 1 || co < 1 || (flip != 0 && flip != 1)) return LBM_ERR_INVALID_ARG;
  // channels of the convolution that reads them
  const int ki = flip ? co : ci, ko = flip ? ci : co;
  size_t bytes = 0;
  if (nn_conv3d_packed_bytes(ki, ko, &bytes) != LBM_OK || bytes / 16 >= (1ULL << 31) - 256)
    return LBM_ERR_INVALID_ARG;
  const int total = (int)(bytes / 16);
  const unsigned blocks = (unsigned)((total + 255) / 256);
  if (flip)
    pack_weights_kernel<true><<<blocks, 256, 0, (hipStream_t)stream>>>(
        (const uint16_t*)w, (uint4*)packed, ki, ko, total);
  else
    pack_weights_kernel<false><<<blocks, 256, 0, (hipStream_t)stream>>>(
        (const uint16_t*)w, (uint4*)packed, ki, ko, total);
  return check_launch();
}

NN_API lbm_status nn_conv3d_forward_packed(const void* x, const void* packed, const float* bias,
                                           void* out, int out_kind, int n, int d, int h, int wd,
                                           int ci, int co, void* stream) {
  if (!aligned16(packed) || out_kind < 0 || out_kind > 2) return LBM_ERR_INVALID_ARG;
  if (out_kind == 0)
    return conv_forward<true, false>(x, packed, bias, out, n, d, h, wd, ci, co, 0, stream);
  return conv_forward<true, true>(x, packed, bias, out, n, d, h, wd, ci, co, out_kind - 1, stream);
}

NN_API lbm_status nn_conv3d_backward_data(const void* dy, const void* wt, float* dx, int n, int d,
                                          int h, int wd, int ci, int co, void* stream) {
  // forward convolution of dy (co channels) with the flipped weights (ci outputs)
  return nn_conv3d_forward(dy, wt, nullptr, dx, n, d, h, wd, co, ci, stream);
}

// How the weight gradient of a layer is split: its partial sums, and the
// tiles of conv_bwdw_tile_kernel (steps 0: the general kernel).  The splits and
// the order of the voxels within them depend on the shape alone and not on the
// kernel: 4 x 8 x 8 tiles strided over about 512 blocks for boxes of at least
// 256 of them, else ranges of consecutive 64-voxel chunks.
struct BwdwPlan {
  int splits;
  long long chunks_per_split;  // consecutive voxels: chunks of 64
  BwdwTiles tiles;
};
constexpr int kTileVox = kTZ * kTY * kTX;
constexpr int kBwdwLds = 153 * 1024;  // of a CU, less the octet tables

static BwdwPlan bwdw_plan(int n, int d, int h, int w, int ci, int co) {
  BwdwPlan p{};
  const long long m = (long long)n * d * h * w;
  const int ct = ci % 32 == 0 ? 32 : 16, rt = co % 32 == 0 ? 32 : 16;
  const long long chan_tiles = (long long)((ci + ct - 1) / ct) * ((co + rt - 1) / rt);
  BwdwTiles& g = p.tiles;
  const long long tiles = m / kTileVox;
  if (d % kTZ == 0 && h % kTY == 0 && w % kTX == 0 && tiles >= 256 && m < (1LL << 31)) {
    p.splits = (int)std::max<long long>(
        1, std::min<long long>({256, tiles / 2, 512 / std::max<long long>(chan_tiles, 1)}));
    g.tz = kTZ;
    g.ty = kTY;
    g.tx = kTX;
    g.stride = p.splits;
  } else {
    const int tm = co <= 32 ? 32 : 64;
    const long long ktiles = (long long)((co + tm - 1) / tm) * ((27 * ci + 63) / 64);
    const long long chunks = (m + kWM - 1) / kWM;
    long long sp = std::max<long long>(
        1, std::min<long long>(chunks, 2048 / std::max<long long>(ktiles, 1)));
    sp = std::min<long long>(sp, 256);
    p.splits = (int)sp;
    p.chunks_per_split = (chunks + sp - 1) / sp;
    if (w % 8 || m >= (1LL << 31) || p.chunks_per_split < 2) return p;
    // tiles of whole rows that follow each other in memory (rows of a plane,
    // or whole planes), a multiple of 64 voxels: the largest of 128 to 256
    // whose buffer leaves room for a second block on the CU (single rows of 64
    // are slower than the general kernel, 18 against 15 us: their halo is nine
    // times the tile).  Splits of one chunk take the general kernel: they would
    // bring a tile of two chunks or more to LDS and use one (138 random boxes: 11%
    // slower in the median, 8 x 8 x 8 x 3, 64 -> 32: 15.4 against 10.9 us; of two
    // chunks 12% faster, of more up to 3 times).
    g.tx = w;
    int vox = 0;
    for (int ty = 1; ty <= h && (long long)ty * w <= 256; ++ty) {
      if (h % ty) continue;
      for (int tz = 1; tz <= (ty == h ? d : 1) && (long long)tz * ty * w <= 256; ++tz) {
        BwdwTiles q = g;
        q.tz = tz;
        q.ty = ty;
        const int v = tz * ty * w;
        if (d % tz || v % kWM || v < 128 || v <= vox || bwdw_buffer_bytes(q, ct * 2, rt * 2) > kBwdwLds / 2)
          continue;
        g = q;
        vox = v;
      }
    }
    if (vox == 0) return p;
    g.split_steps = (int)(2 * p.chunks_per_split);
  }
  const int vox = g.tz * g.ty * g.tx;
  g.ntx = w / g.tx;
  g.nty = h / g.ty;
  g.ntz = d / g.tz;
  g.tiles = (int)(m / vox);
  // two LDS buffers where two blocks of a CU, or the only one, have room
  const int bytes = bwdw_buffer_bytes(g, ct * 2, rt * 2);
  const long long blocks = chan_tiles * p.splits;
  g.buffers = 2 * bytes <= (blocks > 256 ? kBwdwLds / 2 : kBwdwLds) ? 2 : 1;
  g.steps = vox / 32;
  // exact for the halo's few thousand voxels
  g.by_tx = (uint32_t)(((1ULL << 32) + g.tx - 1) / g.tx);
  g.by_hy = (uint32_t)(((1ULL << 32) + g.ty + 1) / (g.ty + 2));
  return p;
}

NN_API lbm_status nn_conv3d_backward_weight_workspace(int n, int d, int h, int wd, int ci, int co,
                                                      size_t* bytes, int* splits) {
  if (!bytes || bad_shape(n, d, h, wd) || ci < 8 || ci % 8 || co < 8 || co % 8)
    return LBM_ERR_INVALID_ARG;
  const BwdwPlan p = bwdw_plan(n, d, h, wd, ci, co);
  *bytes = (size_t)p.splits * co * 27 * ci * sizeof(float);
  if (splits) *splits = p.splits;
  return LBM_OK;
}

template <int RT, int CT>
static void launch_bwdw_tiles(const uint16_t* x, const uint16_t* dy, float* part, const Shape& s,
                              int ci, int co, const BwdwPlan& p, hipStream_t st) {
  const dim3 grid((unsigned)p.splits, (unsigned)((ci + 16 * CT - 1) / (16 * CT)),
                  (unsigned)((co + 16 * RT - 1) / (16 * RT)));
  const size_t lds = (size_t)p.tiles.buffers * bwdw_buffer_bytes(p.tiles, 32 * CT, 32 * RT);
  conv_bwdw_tile_kernel<RT, CT><<<grid, 256, lds, st>>>(x, dy, part, s, ci, co, p.tiles);
}

NN_API lbm_status nn_conv3d_backward_weight(const void* x, const void* dy, float* dw, void* ws,
                                            size_t ws_bytes, int n, int d, int h, int wd, int ci,
                                            int co, void* stream) {
  size_t need = 0;
  int sp = 0;
  lbm_status status = nn_conv3d_backward_weight_workspace(n, d, h, wd, ci, co, &need, &sp);
  if (status != LBM_OK) return status;
  if (!x || !dy || !dw || !ws || ws_bytes < need) return LBM_ERR_WORKSPACE;
  const Shape s = shape_of(n, d, h, wd);
  const long long nw = (long long)co * 27 * ci;
  const BwdwPlan p = bwdw_plan(n, d, h, wd, ci, co);
  const uint16_t* xx = (const uint16_t*)x;
  const uint16_t* dd = (const uint16_t*)dy;
  float* pp = (float*)ws;
  const hipStream_t st = (hipStream_t)stream;
  if (p.tiles.steps && aligned16(x) && aligned16(dy)) {
    // channel tiles: 32 where the count is a multiple of 32, else 16 (zero padded)
    const bool c2 = ci % 32 == 0, r2 = co % 32 == 0;
    if (r2 && c2)
      launch_bwdw_tiles<2, 2>(xx, dd, pp, s, ci, co, p, st);
    else if (r2)
      launch_bwdw_tiles<2, 1>(xx, dd, pp, s, ci, co, p, st);
    else if (c2)
      launch_bwdw_tiles<1, 2>(xx, dd, pp, s, ci, co, p, st);
    else
      launch_bwdw_tiles<1, 1>(xx, dd, pp, s, ci, co, p, st);
  } else {
    const long long chunks = (s.m + kWM - 1) / kWM;
    const long long per = (chunks + sp - 1) / sp;
    const int tm = co <= 32 ? 32 : 64;
    const dim3 grid((unsigned)((co + tm - 1) / tm), (unsigned)((27 * ci + 63) / 64), (unsigned)sp);
    if (tm == 32)
      conv_bwdw_kernel<32><<<grid, 256, 0, st>>>(xx, dd, pp, s, ci, co, per);
    else
      conv_bwdw_kernel<64><<<grid, 256, 0, st>>>(xx, dd, pp, s, ci, co, per);
  }
  fold_splits_kernel<<<grid_for(nw), 256, 0, st>>>((const float*)ws, dw, nw, sp);
  return check_launch();
}

NN_API lbm_status nn_bias_grad_workspace(long long m, int c, size_t* bytes) {
  if (!bytes || m < 1 || c < 1) return LBM_ERR_INVALID_ARG;
  const long long splits = std::min<long long>(kBiasSplits, (m + 255) / 256);
  *bytes = (size_t)splits * c * sizeof(float);
  return LBM_OK;
}

NN_API lbm_status nn_bias_grad(const float* dy, float* db, void* ws, size_t ws_bytes, long long m,
                               int c, void* stream) {
  size_t need = 0;
  lbm_status st = nn_bias_grad_workspace(m, c, &need);
  if (st != LBM_OK || !dy || !db) return LBM_ERR_INVALID_ARG;
  if (!ws || ws_bytes < need) return LBM_ERR_WORKSPACE;
  const long long splits = need / ((size_t)c * sizeof(float));
  const long long per = (m + splits - 1) / splits;
  if (bias4(c))
    launch_bias4<false, false>(dy, nullptr, nullptr, ws, m, c, splits, per, 0,
                               aligned16(dy) ? 1 : 0, PooledSource{}, stream);
  else
    bias_grad_part_kernel<<<(unsigned)splits, 256, 0, (hipStream_t)stream>>>(dy, (float*)ws, m,
                                                                            c, per);
  fold_bias_kernel<<<(c - 1) / 32 + 1, 512, 0, (hipStream_t)stream>>>((const float*)ws, db, c,
                                                                  (int)splits);
  return check_launch();
}

NN_API lbm_status nn_relu_backward_bias(const float* da, const void* a, void* dz, float* db,
                                       void* ws, size_t ws_bytes, long long m, int c, int relu,
                                       void* stream) {
  size_t need = 0;
  lbm_status st = nn_bias_grad_workspace(m, c, &need);
  if (st != LBM_OK || !da || !dz || !db || (relu != 0 && relu != 1) || (relu && !a))
    return LBM_ERR_INVALID_ARG;
  if (!ws || ws_bytes < need) return LBM_ERR_WORKSPACE;
  const long long splits = need / ((size_t)c * sizeof(float));
  const long long per = (m + splits - 1) / splits;
  if (bias4(c)) {
    const bool vec = aligned16(da) && ((uintptr_t)dz & 7) == 0 && (!relu || ((uintptr_t)a & 7) == 0);
    launch_bias4<true, false>(da, a, dz, ws, m, c, splits, per, relu, vec ? 1 : 0,
                              PooledSource{}, stream);
  } else {
    relu_bwd_bias_part_kernel<<<(unsigned)splits, 256, 0, (hipStream_t)stream>>>(
        da, (const uint16_t*)a, (uint16_t*)dz, (float*)ws, m, c, per, relu);
  }
  fold_bias_kernel<<<(c - 1) / 32 + 1, 512, 0, (hipStream_t)stream>>>((const float*)ws, db, c,
                                                                  (int)splits);
  return check_launch();
}

NN_API lbm_status nn_activation_forward(const float* z, void* a, long long n, int relu,
                                        void* stream) {
  if (!z || !a || n < 0) return LBM_ERR_INVALID_ARG;
  if (n % 4 == 0 && aligned16(z) && ((uintptr_t)a & 7) == 0) {
    relu_fwd_vec_kernel<<<grid_for(n / 4), 256, 0, (hipStream_t)stream>>>(
        (const float4*)z, (uint2*)a, n / 4, relu);
    return check_launch();
  }
  relu_fwd_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(z, (uint16_t*)a, n, relu);
  return check_launch();
}

NN_API lbm_status nn_relu_backward(const float* da, const void* a, float* dz, long long n,
                                   void* stream) {
  if (!da || !a || !dz || n < 0) return LBM_ERR_INVALID_ARG;
  if (n % 4 == 0 && aligned16(da) && aligned16(dz) && ((uintptr_t)a & 7) == 0) {
    relu_bwd_vec_kernel<<<grid_for(n / 4), 256, 0, (hipStream_t)stream>>>(
        (const float4*)da, (const uint2*)a, (float4*)dz, n / 4);
    return check_launch();
  }
  relu_bwd_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(da, (const uint16_t*)a, dz, n);
  return check_launch();
}

NN_API lbm_status nn_cast_bf16(const float* x, void* y, long long n, void* stream) {
  if (!x || !y || n < 0) return LBM_ERR_INVALID_ARG;
  if (n % 4 == 0 && aligned16(x) && ((uintptr_t)y & 7) == 0) {
    cast_bf16_vec_kernel<<<grid_for(n / 4), 256, 0, (hipStream_t)stream>>>(
        (const float4*)x, (uint2*)y, n / 4);
    return check_launch();
  }
  cast_bf16_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(x, (uint16_t*)y, n);
  return check_launch();
}

NN_API lbm_status nn_pool2_forward(const void* x, void* y, int n, int d, int h, int w, int c,
                                   void* stream) {
  if (!x || !y || bad_shape(n, d, h, w) || d % 2 || h % 2 || w % 2 || c < 1)
    return LBM_ERR_INVALID_ARG;
  const Shape s = shape_of(n, d, h, w);
  if (c % 8 == 0 && aligned16(x) && aligned16(y) && s.m * c < (1LL << 31)) {
    pool_fwd_vec_kernel<<<grid_for(s.m / 8 * (c / 8)), 256, 0, (hipStream_t)stream>>>(
        (const uint4*)x, (uint4*)y, n, d, h, w, c / 8);
    return check_launch();
  }
  pool_fwd_kernel<<<grid_for(s.m / 8 * c), 256, 0, (hipStream_t)stream>>>(
      (const uint16_t*)x, (uint16_t*)y, s, c);
  return check_launch();
}

NN_API lbm_status nn_pool2_backward(const float* dy, float* dx, int n, int d, int h, int w, int c,
                                    void* stream) {
  if (!dy || !dx || bad_shape(n, d, h, w) || d % 2 || h % 2 || w % 2 || c < 1)
    return LBM_ERR_INVALID_ARG;
  const Shape s = shape_of(n, d, h, w);
  if (c % 4 == 0 && aligned16(dy) && aligned16(dx) && s.m * c < (1LL << 31)) {
    pool_bwd_vec_kernel<<<grid_for(s.m * (c / 4)), 256, 0, (hipStream_t)stream>>>(
        (const float4*)dy, (float4*)dx, n, d, h, w, c / 4);
    return check_launch();
  }
  pool_bwd_kernel<<<grid_for(s.m * c), 256, 0, (hipStream_t)stream>>>(dy, dx, s, c);
  return check_launch();
}

// Periodic trilinear prolongation by 2 (the two-grid warm start): fine node
// i of an axis sits between coarse nodes, 3/4 from the nearer one m = i / 2
// and 1/4 from the farther (m - 1 for even i, m + 1 for odd i), so it takes
// 0.75 x[m] + 0.25 x[far].  The three axes are applied in the order z, y, x,
// then the channel scale.
__device__ __forceinline__ float prolong_value(const float (&v)[2][2][2]) {  // [x][y][z] near, far
  float a[2];  // the y-then-z interpolated values at the near and far x
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float bn = 0.75f * v[q][0][0] + 0.25f * v[q][0][1];
    const float bf = 0.75f * v[q][1][0] + 0.25f * v[q][1][1];
    a[q] = 0.75f * bn + 0.25f * bf;
  }
  return 0.75f * a[0] + 0.25f * a[1];
}
__device__ __forceinline__ int prolong_far(int i, int m, int n) {
  return (i & 1) ? (m + 1 == n ? 0 : m + 1) : (m == 0 ? n - 1 : m - 1);
}

__global__ void prolong2_kernel(const float* __restrict__ x, float* __restrict__ y, int n, int d,
                                int h, int w, int cx, int c, const float* __restrict__ scale,
                                long long total) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % c);
    long long r = i / c;
    const int X = (int)(r % (2 * w));
    r /= 2 * w;
    const int Y = (int)(r % (2 * h));
    r /= 2 * h;
    const int Z = (int)(r % (2 * d));
    const int b = (int)(r / (2 * d));
    const int xs[2] = {X >> 1, prolong_far(X, X >> 1, w)},
              ys[2] = {Y >> 1, prolong_far(Y, Y >> 1, h)},
              zs[2] = {Z >> 1, prolong_far(Z, Z >> 1, d)};
    float v[2][2][2];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      v[q >> 2][(q >> 1) & 1][q & 1] =
          x[((((long long)b * d + zs[q & 1]) * h + ys[(q >> 1) & 1]) * w + xs[q >> 2]) * cx + ch];
    const float u = prolong_value(v);
    y[i] = scale ? u * scale[ch] : u;
  }
}

// The same for 4 channels (of cx, a multiple of 4) as 16-byte words, one
// thread per fine voxel and 32-bit index arithmetic: write bound (64^3 -> 128^3:
// 14 us against the element form's 59 us).
__global__ __launch_bounds__(256) void prolong2_vec_kernel(const float4* __restrict__ x,
                                                           float4* __restrict__ y, int d, int h,
                                                           int w, int g,
                                                           const float* __restrict__ scale,
                                                           int total) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  int b, Z, Y, X;
  voxel_of(i, 2 * d, 2 * h, 2 * w, b, Z, Y, X);
  const int xs[2] = {X >> 1, prolong_far(X, X >> 1, w)},
            ys[2] = {Y >> 1, prolong_far(Y, Y >> 1, h)},
            zs[2] = {Z >> 1, prolong_far(Z, Z >> 1, d)};
  float v[4][2][2][2];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float4 t =
        x[(((b * d + zs[q & 1]) * h + ys[(q >> 1) & 1]) * w + xs[q >> 2]) * g];
    v[0][q >> 2][(q >> 1) & 1][q & 1] = t.x;
    v[1][q >> 2][(q >> 1) & 1][q & 1] = t.y;
    v[2][q >> 2][(q >> 1) & 1][q & 1] = t.z;
    v[3][q >> 2][(q >> 1) & 1][q & 1] = t.w;
  }
  float o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o[k] = prolong_value(v[k]);
    if (scale) o[k] *= scale[k];
  }
  y[i] = make_float4(o[0], o[1], o[2], o[3]);
}

NN_API lbm_status nn_prolongate2(const float* x, float* y, int n, int d, int h, int w, int cx,
                                 int c, const float* scale, void* stream) {
  if (!x || !y || bad_shape(n, d, h, w) || cx < 1 || c < 1 || c > cx)
    return LBM_ERR_INVALID_ARG;
  const long long voxels = 8LL * n * d * h * w, total = voxels * c;
  if (c == 4 && cx % 4 == 0 && aligned16(x) && aligned16(y) &&
      std::max<long long>(voxels, voxels / 8 * (cx / 4)) < (1LL << 31) - 256) {
    prolong2_vec_kernel<<<(unsigned)((voxels + 255) / 256), 256, 0, (hipStream_t)stream>>>(
        (const float4*)x, (float4*)y, d, h, w, cx / 4, scale, (int)voxels);
    return check_launch();
  }
  prolong2_kernel<<<grid_for(total), 256, 0, (hipStream_t)stream>>>(x, y, n, d, h, w, cx, c, scale,
                                                                    total);
  return check_launch();
}

// Start fields of a warm start, for lbm_init_equilibrium_device, from
// predicted targets t (n boxes of d x h x w, cx channels; velocity targets in
// channels 0-2) and the fluid mask: drho = -(delta_rho / w)(x - (w - 1)/2) on
// fluid cells (the linear profile of the pressure drop), u = factor * t on
// fluid cells none of whose 18 lattice neighbours (periodic in the box) is
// solid, 0 elsewhere.  fields: [drho | u_x | u_y | u_z], n d h w values each.
// Write bound: a thread per cell, neighbours by conditional wraps (128^3:
// 25 us against 31 us with 64-bit divisions and a modulo per neighbour).
template <typename I>  // index type: unsigned for fewer than 2^31 cells in all
__global__ __launch_bounds__(256) void warm_fields_kernel(const float* __restrict__ t, int cx,
                                                          const uint8_t* __restrict__ fluid,
                                                          double* __restrict__ fields, int d,
                                                          int h, int w, long long total,
                                                          double factor, double delta_rho) {
  const long long plane = (long long)h * w;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < total; i += gridDim.x * 256LL) {
    const I row = (I)i / (I)w, slab = row / (I)h, bx = slab / (I)d;
    const int x = (int)((I)i - row * (I)w);
    const int y = (int)(row - slab * (I)h);
    const int z = (int)(slab - bx * (I)d);
    const long long box = (long long)bx * d * plane;
    const bool f = fluid[i] != 0;
    bool wall = false;
    if (f) {
      const long long zs[3] = {(z == 0 ? d - 1 : z - 1) * plane, z * plane,
                               (z == d - 1 ? 0 : z + 1) * plane};
      const int ys[3] = {(y == 0 ? h - 1 : y - 1) * w, y * w, (y == h - 1 ? 0 : y + 1) * w};
      const int xs[3] = {x == 0 ? w - 1 : x - 1, x, x == w - 1 ? 0 : x + 1};
#pragma unroll
      for (int q = 0; q < 27; ++q) {
        const int a = q / 9, b = (q / 3) % 3, c = q % 3;
        const int away = (a != 1) + (b != 1) + (c != 1);
        if (away == 0 || away == 3) continue;  // the 18 moving D3Q19 directions
        wall |= fluid[box + zs[a] + ys[b] + xs[c]] == 0;
      }
    }
    const double xc = x - (w - 1) / 2.0;
    fields[i] = f ? -(delta_rho / w) * xc : 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      fields[(1 + k) * total + i] = (f && !wall) ? (double)t[i * cx + k] * factor : 0.0;
  }
}

NN_API lbm_status nn_warm_start_fields(const float* t, int cx, const void* fluid, double* fields,
                                       int n, int d, int h, int w, double factor,
                                       double delta_rho, void* stream) {
  if (!t || !fluid || !fields || bad_shape(n, d, h, w) || cx < 3) return LBM_ERR_INVALID_ARG;
  const long long total = (long long)n * d * h * w;
  if (total < (1LL << 31))
    warm_fields_kernel<uint32_t><<<grid_for(total), 256, 0, (hipStream_t)stream>>>(
        t, cx, (const uint8_t*)fluid, fields, d, h, w, total, factor, delta_rho);
  else
    warm_fields_kernel<unsigned long long><<<grid_for(total), 256, 0, (hipStream_t)stream>>>(
        t, cx, (const uint8_t*)fluid, fields, d, h, w, total, factor, delta_rho);
  return check_launch();
}

// Network input of a pack on the half-resolution grid (nn_coarse_pack_input).
// The spheres travel as kernel arguments, 64 per launch; a thread takes one
// coarse node.  The squared periodic distances are formed and added as the
// host form (warmstart.coarse_fluid) does, in FP64 without fused operations,
// so that the masks are equal.  64^3 nodes, up to 27 spheres: 8 us, against about
// 2 ms for the mask in numpy and its upload.
constexpr int kPackSpheres = 64;
struct PackSpheres {
  double c[kPackSpheres][4];
};
__global__ __launch_bounds__(256) void coarse_pack_kernel(PackSpheres sp, int n, int ec, int first,
                                                          uint4* __restrict__ x) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= ec * ec * ec) return;
  const int X = i % ec, r = i / ec, Y = r % ec, Z = r / ec;
  const double edge = 2.0 * ec;
  const double pos[3] = {2.0 * X + 0.5, 2.0 * Y + 0.5, 2.0 * Z + 0.5};
  bool solid = false;
  for (int s = 0; s < n; ++s) {
    double sq[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double a = fabs(pos[k] - sp.c[s][k]);
      const double m = fmin(a, edge - a);
      sq[k] = m * m;
    }
    const double zy = sq[2] + sq[1];
    const double d2 = zy + sq[0];
    const double rr = sp.c[s][3] * sp.c[s][3];
    solid |= d2 < rr;
  }
  // bf16 1.0 in channel 0 of a fluid node; later launches only add solid nodes
  if (first)
    x[i] = make_uint4(solid ? 0u : 0x3f80u, 0u, 0u, 0u);
  else if (solid)
    x[i] = make_uint4(0u, 0u, 0u, 0u);
}

namespace {
// Launches `kernel` over the items in lists of at most kItems; work(t) is the
// elements of item t.
template <typename T, typename Work, typename Launch>
lbm_status launch_items(const T* items, int count, Work work, Launch launch) {
  for (int beg = 0; beg < count;) {
    ItemList<T> l{};
    long long blocks = 0;
    while (beg < count && l.n < kItems) {
      const long long b = (work(items[beg]) + kItemSpan - 1) / kItemSpan;
      if (l.n && blocks + b >= (1LL << 31)) break;
      if (b >= (1LL << 31)) return LBM_ERR_INVALID_ARG;
      if (b) {  // (an empty item has no block)
        l.item[l.n] = items[beg];
        l.first[l.n++] = (int)blocks;
        blocks += b;
      }
      ++beg;
    }
    if (!l.n) continue;
    l.first[l.n] = (int)blocks;
    launch(l, (unsigned)blocks);
    if (hipGetLastError() != hipSuccess) return LBM_ERR_DEVICE;
  }
  return LBM_OK;
}
}  // namespace

NN_API lbm_status nn_adam_many(const nn_adam_tensor* tensors, int count, float lr, float b1,
                               float b2, float eps, int step, void* stream) {
  if (!tensors || count < 1 || step < 1) return LBM_ERR_INVALID_ARG;
  for (int i = 0; i < count; ++i) {
    const nn_adam_tensor& t = tensors[i];
    if (!t.w || !t.g || !t.m1 || !t.m2 || t.n < 0) return LBM_ERR_INVALID_ARG;
  }
  const float c1 = 1.f / (1.f - powf(b1, (float)step)), c2 = 1.f / (1.f - powf(b2, (float)step));
  return launch_items(
      tensors, count, [](const nn_adam_tensor& t) { return t.n; },
      [&](const ItemList<nn_adam_tensor>& l, unsigned blocks) {
        adam_many_kernel<<<blocks, 256, 0, (hipStream_t)stream>>>(l, lr, b1, b2, eps, c1, c2);
      });
}

NN_API lbm_status nn_conv3d_pack_weights_many(const nn_pack_item* items, int count, void* stream) {
  if (!items || count < 1) return LBM_ERR_INVALID_ARG;
  for (int i = 0; i < count; ++i) {
    const nn_pack_item& t = items[i];
    size_t bytes = 0;
    if (!t.w || !t.packed || t.ci < 1 || t.co < 1 || (t.flip != 0 && t.flip != 1) ||
        nn_conv3d_packed_bytes(t.flip ? t.co : t.ci, t.flip ? t.ci : t.co, &bytes) != LBM_OK ||
        bytes / 16 >= (1ULL << 31) - 256)
      return LBM_ERR_INVALID_ARG;
  }
  return launch_items(
      items, count,
      [](const nn_pack_item& t) {
        size_t bytes = 0;
        nn_conv3d_packed_bytes(t.flip ? t.co : t.ci, t.flip ? t.ci : t.co, &bytes);
        return (long long)(bytes / 16);
      },
      [&](const ItemList<nn_pack_item>& l, unsigned blocks) {
        pack_many_kernel<<<blocks, 256, 0, (hipStream_t)stream>>>(l);
      });
}

NN_API lbm_status nn_coarse_pack_input(const double* spheres, int n, int edge, void* x,
                                       void* stream) {
  if (n < 0 || (n > 0 && !spheres) || !x || edge < 2 || edge % 2 || edge > 2048)
    return LBM_ERR_INVALID_ARG;
  const int ec = edge / 2;
  const unsigned blocks = (unsigned)((ec * (long long)ec * ec + 255) / 256);
  int at = 0;
  do {
    PackSpheres sp;
    const int m = std::min(n - at, kPackSpheres);
    std::memset(&sp, 0, sizeof(sp));
    if (m > 0) std::memcpy(sp.c, spheres + 4 * (size_t)at, (size_t)m * 4 * sizeof(double));
    coarse_pack_kernel<<<blocks, 256, 0, (hipStream_t)stream>>>(sp, m, ec, at == 0, (uint4*)x);
    at += m;
  } while (at < n);
  return check_launch();
}

NN_API lbm_status nn_upsample2_forward(const void* x, void* y, int n, int d, int h, int w, int c,
                                       void* stream) {
  if (!x || !y || bad_shape(n, d, h, w) || c < 1) return LBM_ERR_INVALID_ARG;
  const Shape q = shape_of(n, d, h, w);
  if (c % 8 == 0 && aligned16(x) && aligned16(y) && q.m * 8 * c < (1LL << 31)) {
    up_fwd_vec_kernel<<<grid_for(q.m * 8 * (c / 8)), 256, 0, (hipStream_t)stream>>>(
        (const uint4*)x, (uint4*)y, n, d, h, w, c / 8);
    return check_launch();
  }
  up_fwd_kernel<<<grid_for(q.m * 8 * c), 256, 0, (hipStream_t)stream>>>(
      (const uint16_t*)x, (uint16_t*)y, q, c);
  return check_launch();
}

NN_API lbm_status nn_upsample2_backward(const float* dy, float* dx, int n, int d, int h, int w,
                                        int c, void* stream) {
  if (!dy || !dx || bad_shape(n, d, h, w) || c < 1) return LBM_ERR_INVALID_ARG;
  const Shape q = shape_of(n, d, h, w);
  if (c % 4 == 0 && aligned16(dy) && aligned16(dx) && q.m * 8 * c < (1LL << 31)) {
    up_bwd_vec_kernel<<<grid_for(q.m * (c / 4)), 256, 0, (hipStream_t)stream>>>(
        (const float4*)dy, (float4*)dx, n, d, h, w, c / 4, c / 4);
    return check_launch();
  }
  up_bwd_kernel<<<grid_for(q.m * c), 256, 0, (hipStream_t)stream>>>(dy, dx, q, c);
  return check_launch();
}

NN_API lbm_status nn_concat_channels(const void* a, const void* b, void* y, long long m, int ca,
                                     int cb, void* stream) {
  if (!a || !b || !y || m < 1 || ca < 1 || cb < 1) return LBM_ERR_INVALID_ARG;
  if (ca % 8 == 0 && cb % 8 == 0 && aligned16(a) && aligned16(b) && aligned16(y) &&
      m * (ca + cb) < (1LL << 31)) {
    concat_vec_kernel<<<grid_for(m * ((ca + cb) / 8)), 256, 0, (hipStream_t)stream>>>(
        (const uint4*)a, (const uint4*)b, (uint4*)y, (int)m, ca / 8, cb / 8);
    return check_launch();
  }
  concat_kernel<<<grid_for(m * (ca + cb)), 256, 0, (hipStream_t)stream>>>(
      (const uint16_t*)a, (const uint16_t*)b, (uint16_t*)y, m, ca, cb);
  return check_launch();
}

NN_API lbm_status nn_split_channels(const float* dy, float* da, float* db, long long m, int ca,
                                    int cb, void* stream) {
  if (!dy || m < 1 || ca < 1 || cb < 1) return LBM_ERR_INVALID_ARG;
  if (ca % 4 == 0 && cb % 4 == 0 && aligned16(dy) && aligned16(da) && aligned16(db) &&
      m * (ca + cb) < (1LL << 31)) {
    split_vec_kernel<<<grid_for(m * ((ca + cb) / 4)), 256, 0, (hipStream_t)stream>>>(
        (const float4*)dy, (float4*)da, (float4*)db, (int)m, ca / 4, cb / 4);
    return check_launch();
  }
  split_kernel<<<grid_for(m * (ca + cb)), 256, 0, (hipStream_t)stream>>>(dy, da, db, m, ca, cb);
  return check_launch();
}

NN_API lbm_status nn_upsample_concat(const void* a, const void* b, void* y, int n, int d, int h,
                                     int w, int ca, int cb, void* stream) {
  if (!a || !b || !y || bad_shape(n, d, h, w) || ca < 8 || ca % 8 || cb < 8 || cb % 8 ||
      !aligned16(a) || !aligned16(b) || !aligned16(y) ||
      8LL * n * d * h * w * (ca + cb) >= (1LL << 31))
    return LBM_ERR_INVALID_ARG;
  upsample_concat_kernel<<<grid_for(8LL * n * d * h * w * ((ca + cb) / 8)), 256, 0,
                           (hipStream_t)stream>>>((const uint4*)a, (const uint4*)b, (uint4*)y, n,
                                                  d, h, w, ca / 8, cb / 8);
  return check_launch();
}

NN_API lbm_status nn_concat_upsample_backward(const float* dcat, float* da, int n, int d, int h,
                                              int w, int ca, int cb, void* stream) {
  if (!dcat || !da || bad_shape(n, d, h, w) || ca < 4 || ca % 4 || cb < 4 || cb % 4 ||
      !aligned16(dcat) || !aligned16(da) || 8LL * n * d * h * w * (ca + cb) >= (1LL << 31))
    return LBM_ERR_INVALID_ARG;
  up_bwd_vec_kernel<<<grid_for((long long)n * d * h * w * (ca / 4)), 256, 0, (hipStream_t)stream>>>(
      (const float4*)dcat, (float4*)da, n, d, h, w, ca / 4, (ca + cb) / 4);
  return check_launch();
}

NN_API lbm_status nn_pooled_backward_bias(const float* pooled, const float* cat, int ca,
                                          const void* a, void* dz, float* db, void* ws,
                                          size_t ws_bytes, int n, int d, int h, int w, int c,
                                          int relu, void* stream) {
  size_t need = 0;
  if (bad_shape(n, d, h, w) || d % 2 || h % 2 || w % 2) return LBM_ERR_INVALID_ARG;
  const long long m = (long long)n * d * h * w;
  lbm_status st = nn_bias_grad_workspace(m, c, &need);
  // v e < 2^32 for every voxel v and edge e: the divisions by __umulhi are exact
  const int edge = d > h ? (d > w ? d : w) : (h > w ? h : w);
  if (st != LBM_OK || !pooled || !cat || !dz || !db || (relu != 0 && relu != 1) || (relu && !a) ||
      ca < 4 || ca % 4 || !bias4(c) || m * (ca + c) >= (1LL << 31) || m > (1LL << 32) / edge ||
      !aligned16(pooled) || !aligned16(cat) || ((uintptr_t)dz & 7) ||
      (relu && ((uintptr_t)a & 7)))
    return LBM_ERR_INVALID_ARG;
  if (!ws || ws_bytes < need) return LBM_ERR_WORKSPACE;
  const long long splits = need / ((size_t)c * sizeof(float));
  const long long per = (m + splits - 1) / splits;
  auto by = [](int e) { return (uint32_t)(((1ULL << 32) + e - 1) / e); };
  const PooledSource src{cat, ca, d, h, w, by(w), by(h), by(d)};
  launch_bias4<true, true>(pooled, a, dz, ws, m, c, splits, per, relu, 1, src, stream);
  fold_bias_kernel<<<(c - 1) / 32 + 1, 512, 0, (hipStream_t)stream>>>((const float*)ws, db, c,
                                                                  (int)splits);
  return check_launch();
}

NN_API lbm_status nn_add(float* y, const float* x, long long n, void* stream) {
  if (!y || !x || n < 0) return LBM_ERR_INVALID_ARG;
  add_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(y, x, n);
  return check_launch();
}

NN_API lbm_status nn_masked_mse(const float* pred, const float* target, const float* weight,
                                float* grad, double* partial, int n_partial, long long m, int c,
                                int used, double norm, void* stream) {
  if (!pred || !target || !weight || !grad || !partial || n_partial < 1 || m < 1 || used > c ||
      !(norm > 0))
    return LBM_ERR_INVALID_ARG;
  mse_kernel<<<n_partial, 256, 0, (hipStream_t)stream>>>(pred, target, weight, grad, partial, m, c,
                                                         used, 1.0 / norm);
  return check_launch();
}

NN_API lbm_status nn_adam(float* w, const float* g, float* m1, float* m2, void* w_bf16, long long n,
                          float lr, float b1, float b2, float eps, int step, void* stream) {
  if (!w || !g || !m1 || !m2 || n < 0 || step < 1) return LBM_ERR_INVALID_ARG;
  const float c1 = 1.f / (1.f - powf(b1, (float)step)), c2 = 1.f / (1.f - powf(b2, (float)step));
  adam_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(w, g, m1, m2, (uint16_t*)w_bf16, n, lr,
                                                            b1, b2, eps, c1, c2);
  return check_launch();
}
