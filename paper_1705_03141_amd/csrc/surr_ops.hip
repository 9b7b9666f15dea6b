// surr_ops.hip -- operators of the learned surrogate (include/surrogate.h): 3x3x3
// convolutions as implicit GEMMs on the matrix cores, their data and weight gradients, and
// the small element-wise operators of the encoder-decoder and its training.
//
// Convolution.  out[v][co] = sum_tap sum_ci in[v + off(tap)][ci] w[tap][co][ci] is a GEMM with
// M = voxels, N = cout, K = 27 cin.  The kernels that carry the network (conv_slide_kernel;
// conv_box_kernel for the 8-channel input; wgrad_kernel) stage their operands through LDS and
// issue v_mfma_f32_32x32x16_bf16; conv_staged_kernel takes small volumes of 64 channels, and planes
// of 2^31 and more elements with 32 or 64, too large for the sliding kernel's 32-bit offsets;
// conv_fwd_kernel, the direct form with one wave per 32 voxels x 32 output channels and
// v_mfma_f32_32x32x8_bf16 fed from global memory, takes 128 channels.  Tensors and weights may have any
// alignment that their values have.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "surrogate.h"

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x4_any __attribute__((ext_vector_type(4), aligned(2), may_alias));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// v_mfma_f32_32x32x16_bf16: lane l supplies A[l % 32][8 (l / 32) + j] and B[8 (l / 32) + j][l % 32],
// j = 0..7, and holds D rows 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32, in accumulator r.
__device__ __forceinline__ floatx16 mfma16(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// 16 bytes of global memory at any address a BF16 (or FP32) value may have: one instruction all the
// same, the hardware takes wide accesses at every alignment.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2), may_alias));
__device__ __forceinline__ uint4 load16(const uint16_t* p) {
  const u32x4_any v = *reinterpret_cast<const u32x4_any*>(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <typename T>
__device__ __forceinline__ void store16(T* p, uint4 v) {
  *reinterpret_cast<u32x4_any*>(p) = u32x4_any{v.x, v.y, v.z, v.w};
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ void unpack8(uint4 u, float (&f)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = (uint32_t)f2bf(f[2 * i]) | ((uint32_t)f2bf(f[2 * i + 1]) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// Two values rounded to BF16 (to nearest even), the first in the low half.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{a, b}), bf16x2));
}

// All ones in the halves of a dword of two BF16 values that are positive.
__device__ __forceinline__ uint32_t positive_mask(uint32_t y) {
  return (__uint_as_float(y << 16) > 0.0f ? 0x0000FFFFu : 0u) | (__uint_as_float(y & 0xFFFF0000u) > 0.0f ? 0xFFFF0000u : 0u);
}

constexpr int kTapOff[27][3] = {
    {-1, -1, -1}, {-1, -1, 0}, {-1, -1, 1}, {-1, 0, -1}, {-1, 0, 0}, {-1, 0, 1}, {-1, 1, -1}, {-1, 1, 0}, {-1, 1, 1},
    {0, -1, -1},  {0, -1, 0},  {0, -1, 1},  {0, 0, -1},  {0, 0, 0},  {0, 0, 1},  {0, 1, -1},  {0, 1, 0},  {0, 1, 1},
    {1, -1, -1},  {1, -1, 0},  {1, -1, 1},  {1, 0, -1},  {1, 0, 0},  {1, 0, 1},  {1, 1, -1},  {1, 1, 0},  {1, 1, 1}};

// ---------------------------------------------------------------- forward convolution, direct
// v_mfma_f32_32x32x8_bf16: lane l holds the 4 input channels kq..kq+3 (kq = 4 (l / 32)) of
// voxel l % 32 as the A fragment and the same 4 channels of weight row co = l % 32 as the B
// fragment (8-byte loads in the channels-last layout); the 16 accumulators of lane l are rows
// 8 (r / 4) + kq + r % 4, column l % 32, of the tile.
// grid (ceil(nvox / 128), cout / (32 NT)), 256 threads: wave w of block b owns voxels
// [(4 b + w) 32, +32) and output channels [32 NT blockIdx.y, +32 NT).  CIN is the input
// channel count (a template constant, so the loads of a tap are issued ahead of its MFMAs);
// the A fragment of a tap is reused for the NT output-channel tiles.
template <int CIN, int NT>
__global__ void __launch_bounds__(256) conv_fwd_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ w,
                                                       const float* __restrict__ bias, uint16_t* __restrict__ out,
                                                       float* __restrict__ out_f32, int D, int H, int W, int cout,
                                                       int relu, long long nvox) {
  constexpr int KS = CIN / 8;  // MFMA K steps per tap
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long v0 = ((long long)blockIdx.x * 4 + wave) * 32;
  if (v0 >= nvox) return;  // the whole wave leaves; the kernel has no barrier
  const int co0 = blockIdx.y * 32 * NT;
  const long long va = v0 + (lane & 31);
  const bool valid = va < nvox;
  int x = 0, y = 0, z = 0;
  long long nb = 0;
  if (valid) {
    long long t = va;
    x = (int)(t % W);
    t /= W;
    y = (int)(t % H);
    t /= H;
    z = (int)(t % D);
    nb = t / D;
  }
  const int kq = (lane >> 5) * 4;
  floatx16 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = floatx16{};
  for (int tap = 0; tap < 27; ++tap) {
    const int zz = z + kTapOff[tap][0], yy = y + kTapOff[tap][1], xx = x + kTapOff[tap][2];
    const bool inb = valid && zz >= 0 && zz < D && yy >= 0 && yy < H && xx >= 0 && xx < W;
    const long long src = inb ? ((nb * D + zz) * H + yy) * (long long)W + xx : 0;
    const uint16_t* arow = in + src * CIN + kq;
    bf16x4 a[KS], b[NT][KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      a[k] = bf16x4{0, 0, 0, 0};
      if (inb) a[k] = *reinterpret_cast<const bf16x4_any*>(arow + 8 * k);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const uint16_t* brow = w + ((long long)tap * cout + co0 + 32 * j + (lane & 31)) * CIN + kq;
#pragma unroll
      for (int k = 0; k < KS; ++k) b[j][k] = *reinterpret_cast<const bf16x4_any*>(brow + 8 * k);
    }
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[k], b[j][k], acc[j], 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = co0 + 32 * j + (lane & 31);
    const float bb = bias ? bias[col] : 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const long long v = v0 + (r / 4) * 8 + kq + (r & 3);
      if (v < nvox) {
        float val = acc[j][r] + bb;
        if (relu) val = fmaxf(val, 0.0f);
        if (out_f32)
          out_f32[v * cout + col] = val;
        else
          out[v * cout + col] = f2bf(val);
      }
    }
  }
}

template <int CIN>
void launch_conv(const uint16_t* in, const uint16_t* w, const float* bias, uint16_t* out, float* out_f32, int d, int h,
                 int wd, int cout, int relu, long long nvox, hipStream_t s) {
  if (cout % 64 == 0)
    hipLaunchKernelGGL((conv_fwd_kernel<CIN, 2>), dim3((unsigned)((nvox + 127) / 128), cout / 64), dim3(256), 0, s, in,
                       w, bias, out, out_f32, d, h, wd, cout, relu, nvox);
  else
    hipLaunchKernelGGL((conv_fwd_kernel<CIN, 1>), dim3((unsigned)((nvox + 127) / 128), cout / 32), dim3(256), 0, s, in,
                       w, bias, out, out_f32, d, h, wd, cout, relu, nvox);
}

// ---------------------------------------------------------------- forward convolution, staged
// For cin in {32, 64}: a block of NW waves owns a co tile of 32 and walks tiles of two
// output rows x SEG voxels (grid-stride).  Per tile it stages into LDS every input voxel the
// tile reads -- 3 z-planes x 4 rows x (SEG + 2) voxels, all cin channels, zeros outside the
// volume -- with a voxel stride of cin + 8 elements (4 x an odd number of dwords, so each
// group of 8 lanes reading 16 bytes covers all banks once).  The K dimension of the GEMM,
// 27 cin / 16 steps of v_mfma_f32_32x32x16_bf16 over (tap, 16 input channels), is split
// evenly over the waves; each wave
// holds the weight fragments of its steps in registers for the whole kernel and accumulates
// every M-tile of the output tile over them.  The NW partial sums of an M-tile are added in
// wave order through LDS by the wave that finalizes it (m % NW).  NW = 8 for 64 channels
// keeps a wave's weight fragments at 56 registers.
template <int CIN>
struct StagedConv {
  static constexpr int SEG = CIN == 64 ? 32 : 64;  // voxels of an output row in a tile
  static constexpr int XT = SEG / 32;              // M-tiles per output row
  static constexpr int MT = 2 * XT;                // M-tiles per tile
  static constexpr int RV = SEG + 2;               // staged voxels per row
  static constexpr int VS = CIN + 8;               // staged voxel stride (elements)
  static constexpr int SL = CIN / 16;              // 16-channel slices (MFMA K-steps per tap)
  static constexpr int NW = CIN == 64 ? 8 : 4;     // waves per block
  static constexpr int KSTEPS = 27 * SL;
  static constexpr int IPW = (KSTEPS + NW - 1) / NW;  // K-steps of a wave, at most
  static constexpr int STAGE_BYTES = 12 * RV * VS * 2;
  static constexpr int RED_BYTES = (NW - 1) * MT * 4096;
  static constexpr int LDS_BYTES = STAGE_BYTES > RED_BYTES ? STAGE_BYTES : RED_BYTES;
  static_assert(LDS_BYTES <= 65536, "staged tile exceeds LDS");
};

template <int CIN>
__global__ void __launch_bounds__(64 * StagedConv<CIN>::NW, 2) conv_staged_kernel(const uint16_t* __restrict__ in,
                                                             const uint16_t* __restrict__ w,
                                                             const float* __restrict__ bias, uint16_t* __restrict__ out,
                                                             float* __restrict__ out_f32, int D, int H, int W, int cout,
                                                             int relu, long long ntiles) {
  using P = StagedConv<CIN>;
  __shared__ __align__(16) unsigned char lds[P::LDS_BYTES];
  uint16_t* st = reinterpret_cast<uint16_t*>(lds);
  float* red = reinterpret_cast<float*>(lds);
  const int t = threadIdx.x, lane = t & 63, h = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int co0 = blockIdx.y * 32;
  const int k0 = P::KSTEPS * wave / P::NW, nk = P::KSTEPS * (wave + 1) / P::NW - k0;

  uint4 wb[P::IPW];
#pragma unroll
  for (int i = 0; i < P::IPW; ++i) {
    wb[i] = make_uint4(0, 0, 0, 0);
    if (i < nk) {
      const int k = k0 + i, tap = k / P::SL, sl = k % P::SL;
      wb[i] = load16(w + ((long long)tap * cout + co0 + c) * CIN + sl * 16 + 8 * h);
    }
  }
  const float bb = bias ? bias[co0 + c] : 0.0f;
  const int lane_off = c * P::VS + 8 * h;
  const int nseg = (W + P::SEG - 1) / P::SEG, nyp = (H + 1) / 2;

  for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int yp = (int)(tile % nyp);
    const long long col = tile / nyp;  // (n D + z) nseg + seg
    const int seg = (int)(col % nseg);
    const long long nz = col / nseg;
    const int z = (int)(nz % D);
    const int x0 = seg * P::SEG, y0 = 2 * yp;

    __syncthreads();  // the previous tile's reads of LDS are done
    constexpr int Q = CIN / 8;  // 16-byte chunks of a voxel
    for (int it = t; it < 12 * P::RV * Q; it += 64 * P::NW) {
      const int q = it % Q, v = (it / Q) % P::RV, row = it / (Q * P::RV);
      const int dz = row / 4 - 1, ys = y0 + row % 4 - 1, zs = z + dz, x = x0 + v - 1;
      uint4 val = make_uint4(0, 0, 0, 0);
      if (zs >= 0 && zs < D && ys >= 0 && ys < H && x >= 0 && x < W)
        val = load16(in + (((nz + dz) * H + ys) * (long long)W + x) * CIN + 8 * q);
      *reinterpret_cast<uint4*>(st + (row * P::RV + v) * P::VS + 8 * q) = val;
    }
    __syncthreads();

    floatx16 acc[P::MT];
#pragma unroll
    for (int m = 0; m < P::MT; ++m) acc[m] = floatx16{};
#pragma unroll
    for (int i = 0; i < P::IPW; ++i) {
      if (i < nk) {
        const int k = k0 + i, tap = k / P::SL, sl = k % P::SL;
        const int dz = tap / 9, dy = (tap / 3) % 3, dx = tap % 3;  // each offset + 1
        const uint16_t* a0 = st + ((dz * 4 + dy) * P::RV + dx) * P::VS + sl * 16 + lane_off;
#pragma unroll
        for (int m = 0; m < P::MT; ++m) {
          const int moff = (m / P::XT) * P::RV * P::VS + (m % P::XT) * 32 * P::VS;
          acc[m] = mfma16(*reinterpret_cast<const uint4*>(a0 + moff), wb[i], acc[m]);
        }
      }
    }

    __syncthreads();  // every wave is done with the staged rows; LDS now holds partial sums
#pragma unroll
    for (int m = 0; m < P::MT; ++m) {
      const int f = m % P::NW;
      if (wave != f) {
        float* slot = red + (m * (P::NW - 1) + (wave < f ? wave : wave - 1)) * 1024;
#pragma unroll
        for (int r = 0; r < 16; ++r) slot[r * 64 + lane] = acc[m][r];
      }
    }
    __syncthreads();
    if (wave < P::MT) {  // wave m finalizes tile m (MT <= NW): its partial plus the others' in wave order
      floatx16 mine = acc[0];
#pragma unroll
      for (int m = 1; m < P::MT; ++m)
        if (wave == m) mine = acc[m];
      const int m = wave;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        float sum = 0.0f;
#pragma unroll
        for (int ww = 0; ww < P::NW; ++ww)
          sum += ww == m ? mine[e] : red[(m * (P::NW - 1) + (ww < m ? ww : ww - 1)) * 1024 + e * 64 + lane];
        mine[e] = sum;
      }
      const int y = y0 + m / P::XT;
      if (y < H) {
        int co = cout;
        asm volatile("" : "+s"(co));  // keeps the per-element offsets from being hoisted as addresses
        const int xb = x0 + (m % P::XT) * 32 + 4 * h;
        const long long obase = ((nz * H + y) * (long long)W + xb) * co + co0 + c;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (xb + (e / 4) * 8 + (e & 3) < W) {
            float val = mine[e] + bb;
            if (relu) val = fmaxf(val, 0.0f);
            const long long o = obase + ((e / 4) * 8 + (e & 3)) * co;
            if (out_f32)
              out_f32[o] = val;
            else
              out[o] = f2bf(val);
          }
        }
      }
    }
  }
}

template <int CIN>
void launch_staged(const uint16_t* in, const uint16_t* w, const float* bias, uint16_t* out, float* out_f32, int n,
                   int d, int h, int wd, int cout, int relu, hipStream_t s) {
  using P = StagedConv<CIN>;
  const long long ntiles = (long long)n * d * ((wd + P::SEG - 1) / P::SEG) * ((h + 1) / 2);
  const int ctiles = cout / 32;
  const long long want = (512 + ctiles - 1) / ctiles;  // two resident blocks on each of 256 CUs
  const unsigned gx = (unsigned)(ntiles < want ? ntiles : want);
  hipLaunchKernelGGL(conv_staged_kernel<CIN>, dim3(gx, ctiles), dim3(64 * P::NW), 0, s, in, w, bias, out, out_f32, d, h, wd,
                     cout, relu, ntiles);
}

// A wave's 32 x 32 result with channels as rows: lane (h, c) holds voxel c, register 4 g + k channel
// 8 g + 4 h + k.
__device__ __forceinline__ void add_bias_relu(floatx16& v, const float* sb, int h, int relu) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float4 b4 = *reinterpret_cast<const float4*>(sb + 8 * g + 4 * h);
    const float bb[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float f = v[4 * g + k] + bb[k];
      v[4 * g + k] = relu ? fmaxf(f, 0.0f) : f;
    }
  }
}

// As BF16 with 16 consecutive channels per lane, 16 h + 8 g of u[g]: the halves of the wave
// exchange groups (v_permlane32_swap: the first operand's upper half and the second's lower half
// change places), so that a lane stores 16 bytes at a time.
__device__ __forceinline__ void pack_halves(const floatx16& v, uint4 (&u)[2]) {
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const auto x = __builtin_amdgcn_permlane32_swap(pack2(v[4 * g], v[4 * g + 1]), pack2(v[4 * g + 8], v[4 * g + 9]),
                                                    false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(pack2(v[4 * g + 2], v[4 * g + 3]),
                                                    pack2(v[4 * g + 10], v[4 * g + 11]), false, false);
    u[g] = make_uint4(x[0], y[0], x[1], y[1]);
  }
}

__device__ __forceinline__ void store_f32x16(float* o, const floatx16& v, int h) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
    store16(o + 8 * g + 4 * h, make_uint4(__float_as_uint(v[4 * g]), __float_as_uint(v[4 * g + 1]),
                                          __float_as_uint(v[4 * g + 2]), __float_as_uint(v[4 * g + 3])));
}

// ---------------------------------------------------------------- convolution, sliding
// For cin in {32, 64}: activations, FP32 results and data gradients.  A block of eight waves owns a
// co tile of 32, a tile of ROWS x SEG output columns and a range of z, and sweeps the input planes of
// that range.  Each staged plane is used once, for all the outputs it contributes to: a wave (one
// row of 32 voxels) keeps the accumulators of three output planes (z - 1, z, z + 1) in registers,
// and a fragment of voxels read from LDS feeds three MFMAs.  No partial sums pass between waves.
//
// The sums are in the order of kernels that split the taps over the waves of a block, with 64 channels
// that of conv_staged_kernel, so that small and large volumes agree bitwise and results stay what they
// have been: another order moves one BF16 activation in 10^4 by an ulp, which the network carries to
// 5e-4 of its prediction.  The K-steps
// k = tap * SL + slice fall into NCHAIN chains of consecutive k, each summed from zero; with 64
// channels the 8 chains are added in order, with 32 the 4 chains c as ((c_w + c_w-1) + c_w-2) +
// c_w-3, indices modulo 4, w = 2 (y % 2) + x / 32 % 2; the bias comes last.  So the taps of a plane
// are walked in order, and unfinished chains travel with their output: two accumulators per output
// with 64 channels (sum and chain), up to four with 32, nine for the three planes, which leaves
// room for one row per wave (with 64 channels still 256 registers and 24 to 60 B per lane of scratch).
//
// The weights of the co tile stay in LDS in fragment order (1 KB per tap and 16 channels, read
// without conflicts); the plane of voxels has a voxel stride of CIN + 8 elements (4 x an odd number
// of dwords, so that groups of 8 lanes reading 16 bytes cover all banks once).  The weights are the
// first operand, so a lane holds 4 x 4 consecutive output channels of one voxel, and stores 16 bytes
// at a time (in BF16 after an exchange between the halves of the wave); a data gradient's ReLU mask
// is applied there.  The next plane's global
// loads are issued before the MFMAs of the present one.
//
// What bounds it is the rate the card sustains on the matrix cores: an 8192^3 BF16 product reaches
// 1180 TFLOP/s, a form of this kernel without its stores 1160.  One layer repeated by itself, against
// kernels that split the taps over the waves (and their separate mask pass): 32 -> 32 on 1x256x64x64 97 -> 58 us (1000 TFLOP/s),
// FP32 result 95 -> 64, masked data gradient 123 -> 70; 1x128x32x32: 32 -> 64 49 -> 20 us, 64 -> 32
// 63 -> 21; 64 -> 64 on 1x64x16x16 31 -> 15 us.  With 8-byte stores (no exchange between the halves)
// the first three took 62, 65 and 81 us.  In a training step, where the inputs come from HBM, 32 -> 32
// takes 67 us (865 TFLOP/s) and the masked data gradient 74 (788).
//
// CIN: input channels; XT x WY waves, each 32 voxels of a row; NBUF staged planes (two where they
// fit beside the weights: one barrier per plane instead of two).
template <int CIN_, int XT_, int WY_, int NBUF_>
struct SlideConv {
  static constexpr int CIN = CIN_, XT = XT_, WY = WY_, NBUF = NBUF_;
  static constexpr int NCHAIN = CIN == 64 ? 8 : 4;
  static constexpr int NA = CIN == 64 ? 2 : 4;  // accumulators per output
  static constexpr int NW = XT * WY, NT = 64 * NW;
  static constexpr int SEG = 32 * XT, ROWS = WY;
  static constexpr int RV = SEG + 2, SR = ROWS + 2;  // staged voxels per row, rows
  static constexpr int VS = CIN + 8;                 // staged voxel stride (elements)
  static constexpr int SL = CIN / 16;                // 16-channel slices
  static constexpr int Q = CIN / 8;                  // 16-byte chunks of a voxel
  static constexpr int PLANE = SR * RV * VS;         // elements of a staged plane
  static constexpr int CHUNKS = SR * RV * Q;
  static constexpr int PF = (CHUNKS + NT - 1) / NT;  // chunks per thread
  static constexpr int WELEMS = 27 * SL * 512;       // elements of the weights' fragments
  static constexpr int LDS = 2 * (WELEMS + NBUF * PLANE) + 128;
  static_assert(LDS <= 163840, "tile exceeds LDS");
};

template <typename P, bool MASKED>
__global__ void __launch_bounds__(P::NT, P::NW / 4) conv_slide_kernel(
    const uint16_t* __restrict__ in, const uint16_t* __restrict__ w, const float* __restrict__ bias,
    const uint16_t* __restrict__ relu_y, uint16_t* __restrict__ out, float* __restrict__ out_f32, int D, int H, int W,
    int cout, int relu, int nzc, int zlen, unsigned item0) {
  constexpr int SL = P::SL, Q = P::Q;
  __shared__ __align__(16) uint16_t sw[P::WELEMS];
  __shared__ __align__(16) uint16_t sv[P::NBUF * P::PLANE];
  __shared__ __align__(16) float sb[32];
  const int t = threadIdx.x, lane = t & 63, h = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), xt = wave % P::XT, wy = wave / P::XT;
  const int co0 = blockIdx.y * 32;

  // the blocks of one XCD (ids congruent modulo 8) take neighbouring items, which share halos
  unsigned item = blockIdx.x;
  if ((gridDim.x & 7) == 0) item = (item & 7) * (gridDim.x >> 3) + (item >> 3);
  item += item0;
  const unsigned nseg = (W + P::SEG - 1) / P::SEG, nyb = (H + P::ROWS - 1) / P::ROWS;
  const int zc = (int)(item % (unsigned)nzc);
  unsigned col = item / (unsigned)nzc;
  const int seg = (int)(col % nseg);
  col /= nseg;
  const int yb = (int)(col % nyb);
  const long long nb = col / nyb;
  const int x0 = seg * P::SEG, y0 = yb * P::ROWS, za = zc * zlen, zb = min(D, za + zlen);
  const long long plane_elems = (long long)H * W * P::CIN;
  const uint16_t* in_n = in + nb * D * plane_elems;

  // the staged chunks this thread moves: offset within an input plane, -1 outside of it
  int src[P::PF], dst[P::PF];
#pragma unroll
  for (int k = 0; k < P::PF; ++k) {
    const int it = t + P::NT * k, q = it % Q, v = (it / Q) % P::RV, r = it / (Q * P::RV);
    const int ys = y0 + r - 1, x = x0 + v - 1;
    src[k] = it < P::CHUNKS && ys >= 0 && ys < H && x >= 0 && x < W ? (ys * W + x) * P::CIN + 8 * q : -1;
    dst[k] = (r * P::RV + v) * P::VS + 8 * q;
  }
  uint4 pf[P::PF];
  auto load = [&](int p) {
    const uint16_t* base = in_n + (long long)p * plane_elems;
#pragma unroll
    for (int k = 0; k < P::PF; ++k) {
      pf[k] = make_uint4(0, 0, 0, 0);
      if (src[k] >= 0) pf[k] = load16(base + src[k]);
    }
  };
  auto store = [&](int p) {
    uint16_t* d = sv + (P::NBUF == 2 ? (p & 1) * P::PLANE : 0);
#pragma unroll
    for (int k = 0; k < P::PF; ++k)
      if (P::CHUNKS % P::NT == 0 || k < P::PF - 1 || t + P::NT * k < P::CHUNKS)
        *reinterpret_cast<uint4*>(d + dst[k]) = pf[k];
  };

  if (za > 0) load(za - 1);
  // weights and bias of the co tile (after the loads of the first plane: all are in flight together)
  {
    constexpr int WCH = 27 * 32 * Q, WPT = (WCH + P::NT - 1) / P::NT;
    uint4 wr[WPT];
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
      const int i = min(t + P::NT * k, WCH - 1), q = i % Q, co = (i / Q) % 32, tap = i / (Q * 32);
      wr[k] = load16(w + ((long long)tap * cout + co0 + co) * P::CIN + 8 * q);
    }
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
      const int i = min(t + P::NT * k, WCH - 1), q = i % Q, co = (i / Q) % 32, tap = i / (Q * 32);
      *reinterpret_cast<uint4*>(sw + (tap * SL + q / 2) * 512 + ((q & 1) * 32 + co) * 8) = wr[k];
    }
  }
  if (t < 32) sb[t] = bias ? bias[co0 + t] : 0.0f;

  constexpr int NA = P::NA;
  floatx16 acc[3][NA];  // outputs p + 1, p, p - 1 of the staged plane p
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[d][a] = floatx16{};

  // every MFMA of plane p towards the output planes in MASK (bit dz: output p + 1 - dz)
  auto plane_mfmas = [&](auto M, int p) {
    constexpr int MASK = decltype(M)::value;
    int b0 = (P::NBUF == 2 ? (p & 1) * P::PLANE : 0) + (wy * P::RV + xt * 32 + c) * P::VS + 8 * h, w0 = lane * 8;
    asm volatile("" : "+v"(b0), "+v"(w0));
    auto chain = [](int k) {  // of K-step k
      int ch = 0;
      for (int w = 1; w < P::NCHAIN; ++w) ch += k >= 27 * SL * w / P::NCHAIN;
      return ch;
    };
#pragma unroll
    for (int tp = 0; tp < 9; ++tp)
#pragma unroll
      for (int sl = 0; sl < SL; ++sl) {
        const uint4 vf =
            *reinterpret_cast<const uint4*>(sv + b0 + ((tp / 3) * P::RV + tp % 3) * P::VS + sl * 16);
        uint4 wf[3];
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
          if ((MASK >> dz) & 1) wf[dz] = *reinterpret_cast<const uint4*>(sw + w0 + ((dz * 9 + tp) * SL + sl) * 512);
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
          if ((MASK >> dz) & 1) {
            const int k = (dz * 9 + tp) * SL + sl, ch = chain(k), a = NA == 2 ? 1 : ch;
            const bool begins = k == 0 || chain(k - 1) != ch;
            if (NA == 2 && begins && k > 0) acc[dz][0] += acc[dz][1];
            acc[dz][a] = mfma16(wf[dz], vf, begins ? floatx16{} : acc[dz][a]);
          }
        if (tp % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // bounds the reads in flight
      }
  };

  if (za > 0) store(za - 1);
  __syncthreads();
#pragma unroll 1
  for (int p = za - 1; p <= zb; ++p) {
    const bool more = p + 1 <= zb && p + 1 < D;
    if (more) load(p + 1);
    // the chains that no earlier plane has begun
    acc[0][0] = acc[0][1] = floatx16{};
    if constexpr (NA == 4) acc[1][2] = acc[2][3] = floatx16{};
    if (p >= 0 && p < D) {
      const int mask = (p + 1 < zb ? 1 : 0) | (p >= za && p < zb ? 2 : 0) | (p > za ? 4 : 0);
      switch (mask) {
        case 7: plane_mfmas(std::integral_constant<int, 7>{}, p); break;
        case 1: plane_mfmas(std::integral_constant<int, 1>{}, p); break;
        case 2: plane_mfmas(std::integral_constant<int, 2>{}, p); break;
        case 3: plane_mfmas(std::integral_constant<int, 3>{}, p); break;
        case 4: plane_mfmas(std::integral_constant<int, 4>{}, p); break;
        case 6: plane_mfmas(std::integral_constant<int, 6>{}, p); break;
      }
    }
    const int x = x0 + xt * 32 + c, y = y0 + wy;
    const bool put = p > za && y < H && x < W;  // output plane p - 1 is complete
    const long long o = (((nb * D + p - 1) * H + y) * (long long)W + x) * cout + co0;
    uint4 m[2];
    if (MASKED && put) {  // in flight while the next plane goes to LDS
#pragma unroll
      for (int g = 0; g < 2; ++g) m[g] = load16(relu_y + o + 16 * h + 8 * g);
    }
    if constexpr (P::NBUF == 1) __syncthreads();  // every wave is done with the plane
    if (more) store(p + 1);
    if (p > za && y < H) {  // (uniform over the wave)
      floatx16 v;
      if constexpr (NA == 2) {
        v = acc[2][0] + acc[2][1];
      } else {
        const floatx16 c0 = acc[2][0], c1 = acc[2][1], c2 = acc[2][2], c3 = acc[2][3];
        const int half = ((x0 >> 5) + xt) & 1;
        if ((wy & 1) == 0)  // (y0 is even)
          v = half ? ((c1 + c0) + c3) + c2 : ((c0 + c3) + c2) + c1;
        else
          v = half ? ((c3 + c2) + c1) + c0 : ((c2 + c1) + c0) + c3;
      }
      add_bias_relu(v, sb, h, relu);
      if (out_f32) {
        if (put) store_f32x16(out_f32 + o, v, h);
      } else {
        uint4 u[2];
        pack_halves(v, u);
        if (put)
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            if (MASKED) {  // the gradient of the pre-activation: 0 where the ReLU output is not positive
              u[g].x &= positive_mask(m[g].x);
              u[g].y &= positive_mask(m[g].y);
              u[g].z &= positive_mask(m[g].z);
              u[g].w &= positive_mask(m[g].w);
            }
            store16(out + o + 16 * h + 8 * g, u[g]);
          }
      }
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      acc[2][a] = acc[1][a];
      acc[1][a] = acc[0][a];
    }
    __syncthreads();
  }
}

// Blocks of one launch of the kernels that take one item a block, along x: a launch may hold less than
// 2^32 threads along it, and 512 x 2^22 do (many volumes of one voxel have an item each).  All items of a
// call are below 2^32, for each has at least one voxel of 80 bytes and more: 32-bit divisions (16
// channels on 1x16x16x16 5.5 us with 64-bit ones, 5.2 with these).
constexpr long long kMaxItems = 1LL << 22;

template <typename P>
void launch_slide(const uint16_t* in, const uint16_t* w, const float* bias, const uint16_t* relu_y, uint16_t* out,
                  float* out_f32, int n, int d, int h, int wd, int cout, int relu, hipStream_t s) {
  const int ctiles = cout / 32;
  const long long ncols = (long long)n * ((h + P::ROWS - 1) / P::ROWS) * ((wd + P::SEG - 1) / P::SEG);
  // One block fills a compute unit's LDS: the number of z ranges that minimises the rounds of 256
  // blocks times the planes of a block, its halo and its start-up (about 1.5 planes) included, here
  // in half planes.  k ranges cost at least (2 d + 3 k) c / 256, which grows with k: the search ends
  // where that reaches the best so far (at k = 17 of 256 for 1x256x64x64; over every k it cost the host
  // 1.4 us a call there and 22 us with d = 4096).
  int nzc = 1;
  long long best = -1;
  const long long c = ncols * ctiles;
  for (int k = 1; k <= d; ++k) {
    if (best >= 0 && c * (2LL * d + 3LL * k) >= 256 * best) break;
    const int zl = (d + k - 1) / k;
    if ((d + zl - 1) / zl != k) continue;
    const long long cost = (c * k + 255) / 256 * (2LL * zl + 3);
    if (best < 0 || cost < best) {
      best = cost;
      nzc = k;
    }
  }
  const int zlen = (d + nzc - 1) / nzc;
  const long long nitems = ncols * nzc;
  for (long long i = 0; i < nitems; i += kMaxItems) {
    const dim3 grid((unsigned)(nitems - i < kMaxItems ? nitems - i : kMaxItems), ctiles), block(P::NT);
    if (relu_y)
      hipLaunchKernelGGL((conv_slide_kernel<P, true>), grid, block, 0, s, in, w, bias, relu_y, out, out_f32, d, h, wd,
                         cout, relu, nzc, zlen, (unsigned)i);
    else
      hipLaunchKernelGGL((conv_slide_kernel<P, false>), grid, block, 0, s, in, w, bias, relu_y, out, out_f32, d, h, wd,
                         cout, relu, nzc, zlen, (unsigned)i);
  }
}

// 32 channels: tiles of 4 rows x 64 voxels or 8 rows x 32, whichever covers the plane with less
// padding.
inline void launch_slide32(const uint16_t* in, const uint16_t* w, const float* bias, const uint16_t* relu_y,
                           uint16_t* out, float* out_f32, int n, int d, int h, int wd, int cout, int relu,
                           hipStream_t s) {
  const long long wide = (long long)((wd + 63) / 64 * 64) * ((h + 3) / 4 * 4);
  const long long tall = (long long)((wd + 31) / 32 * 32) * ((h + 7) / 8 * 8);
  if (wide <= tall)
    launch_slide<SlideConv<32, 2, 4, 2>>(in, w, bias, relu_y, out, out_f32, n, d, h, wd, cout, relu, s);
  else
    launch_slide<SlideConv<32, 1, 8, 2>>(in, w, bias, relu_y, out, out_f32, n, d, h, wd, cout, relu, s);
}

// ---------------------------------------------------------------- convolution, few channels
// For cin in {8, 16}.  A block of four waves stages a box of the input -- ZT + 2 planes, 6 rows and 66
// voxels, every load in flight at once and one barrier -- and forms ZT planes of 4 x 64 outputs from
// it, one row per wave, 32 voxels at a time, with the weights of its 32 output channels in registers.
//
// The sums have a fixed order, that of the sliding kernel with 32 channels: the K-steps (tap pairs with 8 channels,
// tap 2 k in lanes 0-31 and 2 k + 1 in the rest; taps with 16) fall into four chains of consecutive
// steps, each summed from zero, and chain c of the tile w = 2 (y % 2) + x / 32 % 2 comes in the order
// w, w - 1, w - 2, w - 3 modulo 4; the bias last.  With the order known per row parity and half, a
// tile needs two accumulators.
//
// What bounds it is memory: 8 -> 32 on 1x256x64x64 moves 84 MB, 18 us at the rate of a large copy,
// and takes 26 (FP32 result 31), where a kernel whose waves passed partial sums to each other for
// every 128 voxels took 57; 16 -> 64 on 1x128x64x64 72 -> 42, 8 -> 32 on 128x32x32 17 -> 8 us.
template <int CIN_, int ZT_>
struct BoxConv {
  static constexpr int CIN = CIN_, ZT = ZT_;
  static constexpr int SEG = 64, ROWS = 4, NT = 256;
  static constexpr int RV = SEG + 2, SR = ROWS + 2;  // staged voxels per row, rows per plane
  static constexpr int VS = CIN == 8 ? 8 : CIN + 8;  // staged voxel stride: 4 x an odd number of dwords
  static constexpr int Q = CIN / 8;                  // 16-byte chunks of a voxel
  static constexpr int PLANE = SR * RV * VS;
  static constexpr int CHUNKS = (ZT + 2) * SR * RV * Q;
  static constexpr int PF = (CHUNKS + NT - 1) / NT;
  static constexpr int KSTEPS = CIN == 8 ? 14 : 27;
};

template <typename P>
__global__ void __launch_bounds__(P::NT, P::CIN == 8 ? 4 : 2) conv_box_kernel(
    const uint16_t* __restrict__ in, const uint16_t* __restrict__ w, const float* __restrict__ bias,
    uint16_t* __restrict__ out, float* __restrict__ out_f32, int D, int H, int W, int cout, int relu, unsigned item0) {
  constexpr int Q = P::Q, CIN = P::CIN, VS = P::VS, RV = P::RV;
  __shared__ __align__(16) uint16_t sv[(P::ZT + 2) * P::PLANE];
  __shared__ __align__(16) float sb[32];
  const int t = threadIdx.x, lane = t & 63, h = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int co0 = blockIdx.y * 32;

  // the blocks of one XCD (ids congruent modulo 8) take neighbouring boxes, which share halos
  unsigned item = blockIdx.x;
  if ((gridDim.x & 7) == 0) item = (item & 7) * (gridDim.x >> 3) + (item >> 3);
  item += item0;
  const unsigned nseg = (W + P::SEG - 1) / P::SEG, nyb = (H + P::ROWS - 1) / P::ROWS, nzb = (D + P::ZT - 1) / P::ZT;
  const int z0 = (int)(item % nzb) * P::ZT;
  unsigned col = item / nzb;
  const int x0 = (int)(col % nseg) * P::SEG;
  col /= nseg;
  const int y0 = (int)(col % nyb) * P::ROWS;
  const long long nb = col / nyb;

  uint4 pf[P::PF];
#pragma unroll
  for (int k = 0; k < P::PF; ++k) {
    const int it = t + P::NT * k, q = it % Q, v = (it / Q) % RV, r = (it / (Q * RV)) % P::SR, pz = it / (Q * RV * P::SR);
    const int x = x0 + v - 1, y = y0 + r - 1, z = z0 + pz - 1;
    pf[k] = make_uint4(0, 0, 0, 0);
    if (it < P::CHUNKS && x >= 0 && x < W && y >= 0 && y < H && z >= 0 && z < D)
      pf[k] = load16(in + (((nb * D + z) * H + y) * (long long)W + x) * CIN + 8 * q);
  }
  uint4 wb[P::KSTEPS];
#pragma unroll
  for (int k = 0; k < P::KSTEPS; ++k) {
    wb[k] = make_uint4(0, 0, 0, 0);
    const int tap = CIN == 8 ? 2 * k + h : k;
    if (tap < 27)
      wb[k] = load16(w + ((long long)tap * cout + co0 + c) * CIN + (CIN == 8 ? 0 : 8 * h));
  }
  if (t < 32) sb[t] = bias ? bias[co0 + t] : 0.0f;
#pragma unroll
  for (int k = 0; k < P::PF; ++k) {
    const int it = t + P::NT * k, q = it % Q, v = it / Q;
    if (it < P::CHUNKS) *reinterpret_cast<uint4*>(sv + v * VS + 8 * q) = pf[k];
  }
  __syncthreads();
  const int y = y0 + wave;
  if (y >= H) return;

  // With 8 channels lanes 32-63 read the tap after that of lanes 0-31: the next voxel, or the
  // first of the next row or plane (the zero weight of the last step reads tap 26 again).
  const int b0 = (wave * RV + c) * VS + (CIN == 8 ? 0 : 8 * h);
  const int b1 = CIN == 8 ? b0 + h * VS : b0, b2 = CIN == 8 ? b0 + h * (RV - 2) * VS : b0,
            b3 = CIN == 8 ? b0 + h * (P::PLANE - (2 * RV + 2) * VS) : b0;
  auto rows = [&](auto par) {  // par: y % 2
#pragma unroll 1
    for (int zz = 0; zz < P::ZT; ++zz) {
      if (z0 + zz >= D) break;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (x0 + 32 * half >= W) break;
        const uint16_t* base = sv + zz * P::PLANE + half * 32 * VS;
        floatx16 sum = {};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int ch = (2 * decltype(par)::value + half + 4 - j) % 4;
          floatx16 chain = {};
#pragma unroll
          for (int k = P::KSTEPS * ch / 4; k < P::KSTEPS * (ch + 1) / 4; ++k) {
            const int tap = CIN == 8 ? 2 * k : k, dz = tap / 9, dy = (tap / 3) % 3, dx = tap % 3;  // each offset + 1
            const int b = tap == 26 ? b0 : dx < 2 ? b1 : dy < 2 ? b2 : b3;
            const uint4 vf = *reinterpret_cast<const uint4*>(base + b + dz * P::PLANE + (dy * RV + dx) * VS);
            chain = mfma16(wb[k], vf, chain);
          }
          sum = j == 0 ? chain : sum + chain;
        }
        const int x = x0 + 32 * half + c;
        add_bias_relu(sum, sb, h, relu);
        const long long o = (((nb * D + z0 + zz) * H + y) * (long long)W + x) * cout + co0;
        if (out_f32) {
          if (x < W) store_f32x16(out_f32 + o, sum, h);
        } else {
          uint4 u[2];
          pack_halves(sum, u);
          if (x < W)
#pragma unroll
            for (int g = 0; g < 2; ++g) store16(out + o + 16 * h + 8 * g, u[g]);
        }
      }
    }
  };
  if (wave & 1)
    rows(std::integral_constant<int, 1>{});
  else
    rows(std::integral_constant<int, 0>{});
}

template <typename P>
void launch_boxes(const uint16_t* in, const uint16_t* w, const float* bias, uint16_t* out, float* out_f32, int n, int d,
                  int h, int wd, int cout, int relu, hipStream_t s) {
  const long long items = (long long)n * ((d + P::ZT - 1) / P::ZT) * ((h + P::ROWS - 1) / P::ROWS) *
                          ((wd + P::SEG - 1) / P::SEG);
  for (long long i = 0; i < items; i += kMaxItems)
    hipLaunchKernelGGL(conv_box_kernel<P>, dim3((unsigned)(items - i < kMaxItems ? items - i : kMaxItems), cout / 32),
                       dim3(P::NT), 0, s, in, w, bias, out, out_f32, d, h, wd, cout, relu, (unsigned)i);
}

// Boxes of two planes, or of one where those would leave compute units without a block (8 -> 64 on
// 9x17x40, 50 boxes x 2: 6.3 against 7.5 us; 8 -> 32 on 256x64x64, 2048: 28.7 against 27.7; four
// planes are no better there, and 68 against 45 us for three planes with 16 channels).
template <int CIN>
void launch_box(const uint16_t* in, const uint16_t* w, const float* bias, uint16_t* out, float* out_f32, int n, int d,
                int h, int wd, int cout, int relu, hipStream_t s) {
  if ((long long)n * ((d + 1) / 2) * ((h + 3) / 4) * ((wd + 63) / 64) * (cout / 32) > 256)
    launch_boxes<BoxConv<CIN, 2>>(in, w, bias, out, out_f32, n, d, h, wd, cout, relu, s);
  else
    launch_boxes<BoxConv<CIN, 1>>(in, w, bias, out, out_f32, n, d, h, wd, cout, relu, s);
}

// w_t[tap'][ci][co] = w[26 - tap'][co][ci]
__global__ void flip_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt, int cin, int cout) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = 27LL * cin * cout;
  if (i >= total) return;
  const int co = (int)(i % cout);
  const int ci = (int)((i / cout) % cin);
  const int tap = (int)(i / ((long long)cout * cin));
  wt[i] = w[((long long)(26 - tap) * cout + co) * cin + ci];
}

// ---------------------------------------------------------------- weight gradient
// dw[tap][co][ci] = sum_v dout[v][co] in[v + off(tap)][ci]: per tap a GEMM with M = cout,
// N = cin, K = voxels.  A block of eight waves owns a 32 x 32 (co, ci) tile and walks, along z, tiles
// of 16 rows x 32 voxels of `in`: per step one plane z of `in` (with the voxels left and right of
// it) and the planes z - 1, z, z + 1 of dout (with a row above and below; a ring of three, so a
// step stages one) lie in LDS as they lie in memory, and are read with ds_read_b64_tr_b16, which
// transposes 4 voxels x 16 channels on the way to registers: lane l gets 4 voxels of channel l % 16
// of its group, so two reads make an MFMA operand and a shift in x is a shift of the address.
//
// An operand of `in` (a row, a shift dx, 16 voxels) meets the 9 rows (z - dz, y - dy) of dout, and an
// operand of dout stays in registers for the three rows of `in` it meets while y advances.  The 27
// taps are split over four waves so that each keeps 7 accumulators (112 registers) and shares
// operands: wave dx of the first three takes 7 of the 9 (dz, dy), the fourth the other two for
// every dx, and the bias (dout against ones).  Two such groups take 8 rows each.  Per 7 MFMAs of
// 32 cycles a wave reads 4 KB of LDS, 0.6 of its rate over the block.
//
// With 8 input channels (PACK8) one MFMA takes all three dx: rows of voxels are 16 bytes apart, so
// 32 consecutive elements of a row are the channels of the voxels x - 1, x, x + 1 (and one unused),
// and each wave keeps all 9 (dz, dy) for its rows.
//
// One block per compute unit: 256 partial sums in all, a third of the time of a full-resolution
// layer at 512.  The next step's planes are loaded during the present one's MFMAs.  Measured
// (with the sum of the partials), 32 -> 32 channels on 1x256x64x64 79 us, 730 TFLOP/s, against 114 us
// for the kernel before (transposes while staging, three waves, 512 partial sums); 8 -> 32 50
// against 121, 32 -> 64 on 1x128x32x32 33 against 64, 64 -> 64 on 1x64x16x16 29 against 45.  Rows and
// half-rows of a tile beyond the lattice are passed over, which is what small volumes spend their
// time on otherwise: 32 -> 64 on 1x3x100 14.1 us with them, 10.2 without (12 before).
constexpr int kWgX = 32, kWgY = 16;               // voxels and rows of a tile
constexpr int kWgThreads = 512, kWgBlocks = 256;  // one resident block on each of 256 compute units
constexpr int kWgRow = kWgX * 32, kWgPlane = (kWgY + 2) * kWgRow;  // elements of a staged dout row, plane

constexpr int kSeg = 64;  // voxels of a row segment of wgrad_row_kernel

struct WgradPlan {
  long long steps;  // (column, plane) pairs
  int nxb, nyb;     // tiles of a plane
  int nchunks, ci_tiles, tiles;
  bool rows;        // a block per row segment (wgrad_row_kernel)
};

inline WgradPlan wgrad_plan(int n, int d, int h, int wd, int cin, int cout) {
  WgradPlan p;
  p.nxb = (wd + kWgX - 1) / kWgX;
  p.nyb = (h + kWgY - 1) / kWgY;
  p.steps = (long long)n * p.nyb * p.nxb * d;
  p.ci_tiles = (cin + 31) / 32;
  p.tiles = (cout / 32) * p.ci_tiles;
  const long long want = (kWgBlocks + p.tiles - 1) / p.tiles;
  p.nchunks = (int)(want < p.steps ? want : p.steps);
  // Few rows: tiles of 16 rows leave the device to a handful of blocks, each of which walks through its
  // rows and adds up two groups, where a block per row segment is done after one (us, rows against tiles:
  // 8 -> 32 on 3x17x33 9.9 and 15.0, 12x9x33 10.9 and 14.0; 32 -> 32 on 3x17x33 11.6 and 15.2).  Each
  // leaves a partial sum, so that only so many pay (28x9x33, 8 -> 32 14.3 and 14.6), and fewer where a tile
  // has at most 8 rows or 16 voxels and is done sooner itself (8x10x10, 16 -> 32 11.0 and 11.8, but
  // 16x16x16, 8 -> 32 13.8 and 13.4; 3x5x5, 32 -> 32 9.5 and 10.1, but 40x5x5, 8 -> 32 12.8 and 10.8).
  const long long rows = (long long)n * d * h * ((wd + kSeg - 1) / kSeg);
  p.rows = cin <= 32 && rows * cin * cout <= (16384 << ((h > 8) + (wd > 16)));
  if (p.rows) p.nchunks = (int)rows;
  return p;
}

// Small volumes (WgradPlan::rows): block (row segment, tile) of three waves owns a row of 64 voxels (x0 ..) and
// the (co, ci) tile of 32 x 32; wave k accumulates the nine taps with dz = k - 1.  The block stages the
// transposed row of dout, [co][x], into LDS, and each wave its three source rows (z + dz, y - 1 .. y + 1),
// [ci][x] over x0 - 8 .. x0 + kSeg + 7.  The K order of an MFMA is free: lane half h takes voxels
// x0 + 32 h + 8 s + j at step s, so that each lane walks its 32 voxels eight at a time and the dx = -1, +1
// operands are its 16-byte words shifted by one element, the word before or after coming from the
// previous or the next step.  Bound by the latency of one round of loads and of two launches.
constexpr int kRsA = kSeg + 8;      // LDS row stride of the row of dout (elements; 36 dwords)
constexpr int kRowB = kSeg + 16;    // staged source row
constexpr int kRsB = kRowB + 8;     // LDS row stride of a source row (44 dwords)
// Channel row r of a staged tile starts at r * stride + (r / 8) * 16 elements: the 8-dword shift per group
// of 8 rows spreads the transposing stores of the four 8-channel groups over distinct banks.
__host__ __device__ constexpr int trow(int r, int stride) { return r * stride + (r >> 3) * 16; }
constexpr int kTileA = 32 * kRsA + 4 * 16, kTileB = 32 * kRsB + 4 * 16;  // elements

// [p.e7, c.e0 .. c.e6] and [c.e1 .. c.e7, n.e0] of 8-element BF16 words (element 2i in the low half of
// dword i)
__device__ __forceinline__ uint4 shift_in_prev(uint4 p, uint4 c) {
  return make_uint4((c.x << 16) | (p.w >> 16), (c.y << 16) | (c.x >> 16), (c.z << 16) | (c.y >> 16),
                    (c.w << 16) | (c.z >> 16));
}
__device__ __forceinline__ uint4 shift_in_next(uint4 c, uint4 n) {
  return make_uint4((c.x >> 16) | (c.y << 16), (c.y >> 16) | (c.z << 16), (c.z >> 16) | (c.w << 16),
                    (c.w >> 16) | (n.x << 16));
}

__global__ void __launch_bounds__(192, 2) wgrad_row_kernel(const uint16_t* __restrict__ in,
                                                           const uint16_t* __restrict__ dout, float* __restrict__ part,
                                                           float* __restrict__ bpart, int D, int H, int W, int cin,
                                                           int cout) {
  __shared__ __align__(16) uint16_t sA[kTileA];
  __shared__ __align__(16) uint16_t sB[3][3][kTileB];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, dz = wave - 1;
  const int chunk = blockIdx.x, co0 = blockIdx.y * 32;  // one ci tile (cin <= 32)
  const int nseg = (W + kSeg - 1) / kSeg;
  const int y = chunk % H, x0 = chunk / H % nseg * kSeg, nz = chunk / H / nseg, z = nz % D;  // nz: n D + z

  // 16-byte chunks two voxels at a time, so that the transposed stores are whole dwords (one channel of
  // both voxels, paired by v_perm)
  auto pair_store = [&](uint16_t* base, int stride, int q, int xi, const uint4& A, const uint4& B) {
    const uint32_t a4[4] = {A.x, A.y, A.z, A.w}, b4[4] = {B.x, B.y, B.z, B.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      *reinterpret_cast<uint32_t*>(base + trow(8 * q + 2 * k, stride) + xi) = __builtin_amdgcn_perm(b4[k], a4[k], 0x05040100u);
      *reinterpret_cast<uint32_t*>(base + trow(8 * q + 2 * k + 1, stride) + xi) =
          __builtin_amdgcn_perm(b4[k], a4[k], 0x07060302u);
    }
  };
  if (t < 128) {
    const int q = t & 3, x = x0 + 2 * (t >> 2);
    const uint16_t* src = dout + (((long long)nz * H + y) * W + x) * cout + co0 + 8 * q;
    const uint4 none = make_uint4(0, 0, 0, 0), a = x < W ? load16(src) : none, b = x + 1 < W ? load16(src + cout) : none;
    pair_store(sA, kRsA, q, 2 * (t >> 2), a, b);
  }
  constexpr int PB = (2 * kRowB + 63) / 64;  // voxel pairs per lane of a source row
  for (int r = 0; r < 3; ++r) {
    const int zz = z + dz, yy = y + r - 1;
    const bool row_ok = zz >= 0 && zz < D && yy >= 0 && yy < H;
    const long long base = ((long long)(nz + dz) * H + yy) * W;
    uint4 buf[PB][2];
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      const int it = lane + 64 * k, q = it & 3, x = x0 - 8 + 2 * (it >> 2);
      buf[k][0] = buf[k][1] = make_uint4(0, 0, 0, 0);
      if (it < 2 * kRowB && row_ok && 8 * q < cin) {
        const uint16_t* src = in + (base + x) * cin + 8 * q;
        if (x >= 0 && x < W) buf[k][0] = load16(src);
        if (x + 1 >= 0 && x + 1 < W) buf[k][1] = load16(src + cin);
      }
    }
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      const int it = lane + 64 * k;
      if (it < 2 * kRowB) pair_store(sB[wave][r], kRsB, it & 3, 2 * (it >> 2), buf[k][0], buf[k][1]);
    }
  }
  __syncthreads();

  const int h = lane >> 5, c = lane & 31;
  const uint16_t* pa = sA + trow(c, kRsA) + 32 * h;
  float bsum = 0.0f;  // wave 0, lane (h, c): channel co0 + c over voxels x0 + 32 h .. + 31
  if (bpart && wave == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float f[8];
      unpack8(*reinterpret_cast<const uint4*>(pa + 8 * j), f);
#pragma unroll
      for (int i = 0; i < 8; ++i) bsum += f[i];
    }
  }
  floatx16 acc[9];
  const uint16_t* pb[3];
  uint4 prv[3], cur[3];
#pragma unroll
  for (int dy = 0; dy < 3; ++dy) {
    pb[dy] = sB[wave][dy] + trow(c, kRsB) + 32 * h;  // element 8 + 32 h is voxel x0 + 32 h
    prv[dy] = *reinterpret_cast<const uint4*>(pb[dy]);
    cur[dy] = *reinterpret_cast<const uint4*>(pb[dy] + 8);
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[3 * dy + k] = floatx16{};
  }
#pragma unroll
  for (int st = 0; st < kSeg / 16; ++st) {
    const uint4 a = *reinterpret_cast<const uint4*>(pa + 8 * st);
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
      const uint4 nxt = *reinterpret_cast<const uint4*>(pb[dy] + 16 + 8 * st);
      acc[3 * dy + 0] = mfma16(a, shift_in_prev(prv[dy], cur[dy]), acc[3 * dy + 0]);  // voxels x - 1 ..
      acc[3 * dy + 1] = mfma16(a, cur[dy], acc[3 * dy + 1]);
      acc[3 * dy + 2] = mfma16(a, shift_in_next(cur[dy], nxt), acc[3 * dy + 2]);      // voxels x + 1 ..
      prv[dy] = cur[dy];
      cur[dy] = nxt;
    }
  }
  // acc[3 dy + dx] row m = 8 (r / 4) + 4 h + r % 4 (co0 + m), column c
  if (c < cin) {
    float* dst = part + ((long long)chunk * 27 + 9 * wave) * cout * cin;
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        dst[((long long)k * cout + co0 + (r / 4) * 8 + 4 * h + (r & 3)) * cin + c] = acc[k][r];
  }
  if (bpart) {
    __syncthreads();
    float* red = reinterpret_cast<float*>(&sB[0][0][0]);
    if (t < 64) red[t] = bsum;
    __syncthreads();
    if (t < 32) bpart[(long long)chunk * cout + co0 + t] = red[t] + red[t + 32];
  }
}

// Two transposing reads: the operand of 16 voxels x 32 channels that begins at `p` + this lane's
// offset, rows of voxels `stride` elements apart.
__device__ __forceinline__ uint4 read_tr(const uint16_t* p, int stride) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * stride));
  const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
  return make_uint4(a.x, a.y, b.x, b.y);
}

template <bool PACK8>
__global__ void __launch_bounds__(kWgThreads, 2) wgrad_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ dout,
                                                              float* __restrict__ part, float* __restrict__ bpart, int D, int H,
                                                              int W, int cin, int cout, WgradPlan P) {
  constexpr int IC = PACK8 ? 8 : 32;                // channels of a staged voxel of `in`
  constexpr int IRV = PACK8 ? kWgX + 4 : kWgX + 2;  // staged voxels of a row of `in`
  constexpr int NACC = PACK8 ? 9 : 7;
  constexpr int IN0 = 3 * kWgPlane;                 // where `in` begins
  constexpr int STAGE = IN0 + kWgY * IRV * IC, REDUCE = 4 * NACC * 2048;
  __shared__ __align__(16) uint16_t lds[STAGE > REDUCE ? STAGE : REDUCE];
  const int t = threadIdx.x, lane = t & 63, h = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int chunk = blockIdx.x;
  const int co0 = (blockIdx.y / P.ci_tiles) * 32, ci0 = (blockIdx.y % P.ci_tiles) * 32;
  const long long p0 = P.steps * chunk / P.nchunks, p1 = P.steps * (chunk + 1) / P.nchunks;
  const bool do_bias = bpart != nullptr && ci0 == 0;
  // lane offsets of the transposing reads: voxel 8 h + (l % 16) / 4, channel 16 (l / 16 % 2) + 4 (l % 4)
  const int vox = 8 * h + ((lane & 15) >> 2), chan = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const int offA = vox * 32 + chan, offB = vox * IC + chan;

  const uint4 ones = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);

  // the chunks of 16 bytes this thread moves per plane
  constexpr int DCH = (kWgY + 2) * kWgX * 4, ICH = kWgY * IRV * (IC / 8);
  constexpr int DPF = (DCH + kWgThreads - 1) / kWgThreads, IPF = (ICH + kWgThreads - 1) / kWgThreads;
  uint4 pd[DPF], pi[IPF];
  auto load_dout = [&](long long nb, int z, int y0, int x0) {
    const uint16_t* base = dout + (nb * D + z) * H * (long long)W * cout + co0;
#pragma unroll
    for (int k = 0; k < DPF; ++k) {
      int it = t + kWgThreads * k;
      asm volatile("" : "+v"(it));  // the addresses are formed per step, not kept
      const int q = it & 3, v = (it >> 2) % kWgX, r = (it >> 2) / kWgX;
      const int y = y0 + r - 1, x = x0 + v;
      pd[k] = make_uint4(0, 0, 0, 0);
      if (it < DCH && z >= 0 && z < D && y >= 0 && y < H && x < W)
        pd[k] = load16(base + ((long long)y * W + x) * cout + 8 * q);
    }
  };
  auto store_dout = [&](int z) {
    uint16_t* dst = lds + ((z + 3) % 3) * kWgPlane;
#pragma unroll
    for (int k = 0; k < DPF; ++k)
      if (t + kWgThreads * k < DCH) *reinterpret_cast<uint4*>(dst + 8 * (t + kWgThreads * k)) = pd[k];
  };
  auto load_in = [&](long long nb, int z, int y0, int x0) {
    const uint16_t* base = in + (nb * D + z) * H * (long long)W * cin + ci0;
#pragma unroll
    for (int k = 0; k < IPF; ++k) {
      int it = t + kWgThreads * k;
      asm volatile("" : "+v"(it));
      const int q = PACK8 ? 0 : it & 3, v = (PACK8 ? it : it >> 2) % IRV, r = (PACK8 ? it : it >> 2) / IRV;
      const int y = y0 + r, x = x0 + v - 1;
      pi[k] = make_uint4(0, 0, 0, 0);
      if (it < ICH && y < H && x >= 0 && x < W && ci0 + 8 * q < cin)
        pi[k] = load16(base + ((long long)y * W + x) * cin + 8 * q);
    }
  };
  auto store_in = [&]() {
#pragma unroll
    for (int k = 0; k < IPF; ++k)
      if (t + kWgThreads * k < ICH) *reinterpret_cast<uint4*>(lds + IN0 + 8 * (t + kWgThreads * k)) = pi[k];
  };

  // The whole walk for one role.  LAST: the fourth wave of a group.  The two instances run side by
  // side and meet at the same barriers, two per step and two per round of the reduction: every barrier
  // stands in code that both have, outside of what depends on LAST, and under conditions that hold for
  // the whole block.  Each instance has its own accumulators (one code path for both kept them twice,
  // and spilled).
  auto walk = [&](auto last) {
  constexpr bool LAST = decltype(last)::value;
  floatx16 acc[NACC], accb = floatx16{};
#pragma unroll
  for (int k = 0; k < NACC; ++k) acc[k] = floatx16{};
  for (long long p = p0; p < p1; ++p) {
    const int z = (int)(p % D);
    const long long col = p / D;
    const int xb = (int)(col % P.nxb), yb = (int)((col / P.nxb) % P.nyb);
    const long long nb = col / ((long long)P.nxb * P.nyb);
    const int x0 = xb * kWgX, y0 = yb * kWgY;
    __syncthreads();  // the previous step's reads are done
    if (p > p0 && z > 0) {
      store_dout(z + 1);
      store_in();
    } else {  // a new column: all three planes
#pragma unroll 1
      for (int dz = -1; dz <= 1; ++dz) {
        load_dout(nb, z + dz, y0, x0);
        store_dout(z + dz);
      }
      load_in(nb, z, y0, x0);
      store_in();
    }
    __syncthreads();
    if (p + 1 < p1 && z + 1 < D) {  // the next step continues the column
      load_dout(nb, z + 2, y0, x0);
      load_in(nb, z + 1, y0, x0);
    }

    // the planes z + 1, z, z - 1 (dz = -1, 0, +1); staged row r is row y0 - 1 + r
    const uint16_t* d1 = lds + ((z + 4) % 3) * kWgPlane + offA;
    const uint16_t* d0 = lds + ((z + 3) % 3) * kWgPlane + offA;
    const uint16_t* dm = lds + ((z + 2) % 3) * kWgPlane + offA;
    auto rowA = [&](const uint16_t* plane, int r, int s) { return read_tr(plane + (r * kWgX + 16 * s) * 32, 32); };
    auto rowB = [&](int r, int v) { return read_tr(lds + IN0 + offB + (r * IRV + v) * IC, IC); };
    if constexpr (PACK8) {
      const int s = wave & 1, ya = 4 * (wave >> 1);
      const int rows = 16 * s < W - x0 ? H - y0 - ya : 0;
      uint4 a1[3], a0[3], am[3];  // rows y + 1, y, y - 1
      a1[1] = rowA(d1, ya + 1, s), a1[2] = rowA(d1, ya, s);
      a0[1] = rowA(d0, ya + 1, s), a0[2] = rowA(d0, ya, s);
      am[1] = rowA(dm, ya + 1, s), am[2] = rowA(dm, ya, s);
#pragma unroll
      for (int yy = 0; yy < 4; ++yy) {
        if (yy >= rows) break;
        const uint4 b = rowB(ya + yy, 16 * s);
        a1[0] = rowA(d1, ya + yy + 2, s);
        a0[0] = rowA(d0, ya + yy + 2, s);
        am[0] = rowA(dm, ya + yy + 2, s);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          acc[k] = mfma16(a1[k], b, acc[k]);
          acc[3 + k] = mfma16(a0[k], b, acc[3 + k]);
          acc[6 + k] = mfma16(am[k], b, acc[6 + k]);
        }
        if (do_bias) accb = mfma16(a0[1], ones, accb);
        a1[2] = a1[1], a1[1] = a1[0], a0[2] = a0[1], a0[1] = a0[0], am[2] = am[1], am[1] = am[0];
      }
    } else {
      const int role = wave & 3, ya = 8 * (wave >> 2);
      const int rows = H - y0 - ya, halves = W - x0 > 16 ? 2 : 1;  // the rest of the tile is 0
      if constexpr (!LAST) {  // dx = role - 1
#pragma unroll 1
        for (int s = 0; s < halves; ++s) {
          uint4 a1[3], a0[3];
          a1[1] = rowA(d1, ya + 1, s), a1[2] = rowA(d1, ya, s);
          a0[1] = rowA(d0, ya + 1, s), a0[2] = rowA(d0, ya, s);
#pragma unroll
          for (int yy = 0; yy < 8; ++yy) {
            if (yy >= rows) break;
            const uint4 b = rowB(ya + yy, 16 * s + role);
            a1[0] = rowA(d1, ya + yy + 2, s);
            a0[0] = rowA(d0, ya + yy + 2, s);
            const uint4 am = rowA(dm, ya + yy + 2, s);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              acc[k] = mfma16(a1[k], b, acc[k]);
              acc[3 + k] = mfma16(a0[k], b, acc[3 + k]);
            }
            acc[6] = mfma16(am, b, acc[6]);
            a1[2] = a1[1], a1[1] = a1[0], a0[2] = a0[1], a0[1] = a0[0];
            __builtin_amdgcn_sched_barrier(0);  // not every row's reads at once
          }
        }
      } else {  // (dz, dy) = (1, 0) and (1, 1) for every dx, and the bias
#pragma unroll 1
        for (int s = 0; s < halves; ++s) {
          uint4 am1, am2 = rowA(dm, ya, s);
#pragma unroll
          for (int yy = 0; yy < 8; ++yy) {
            if (yy >= rows) break;
            am1 = rowA(dm, ya + yy + 1, s);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const uint4 b = rowB(ya + yy, 16 * s + k);
              acc[k] = mfma16(am1, b, acc[k]);
              acc[3 + k] = mfma16(am2, b, acc[3 + k]);
            }
            if (do_bias) acc[6] = mfma16(rowA(d0, ya + yy + 1, s), ones, acc[6]);
            am2 = am1;
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  }

  // the waves' sums together, in a fixed order: PACK8 8 -> 4 -> 2 -> 1, else 8 -> 4 (the groups);
  // waves whose rows all lie beyond the lattice hold zeros and are left out
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll 1
  for (int half = H > 8 ? 4 : PACK8 ? (H > 4 ? 2 : 1) : 0; half >= (PACK8 ? 1 : 4); half /= 2) {
    __syncthreads();
    if (wave >= half && wave < 2 * half) {
      float* slot = red + (wave - half) * NACC * 1024 + lane;
#pragma unroll
      for (int k = 0; k < NACC; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) slot[(k * 16 + r) * 64] = acc[k][r];
    }
    __syncthreads();
    if (wave < half) {
      const float* slot = red + wave * NACC * 1024 + lane;
#pragma unroll
      for (int k = 0; k < NACC; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] += slot[(k * 16 + r) * 64];
    }
  }
  if (PACK8 && do_bias) {  // (every column of accb holds the sum)
    __syncthreads();
    if (c == 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[wave * 32 + (r / 4) * 8 + 4 * h + (r & 3)] = accb[r];
    __syncthreads();
    if (t < 32) {
      float sum = red[t];
      for (int w = 1; w < 8; ++w) sum += red[w * 32 + t];
      bpart[(long long)chunk * cout + co0 + t] = sum;
    }
  }

  // accumulator row m = 8 (r / 4) + 4 h + r % 4 (channel co0 + m), column c
  float* dst = part + (long long)chunk * 27 * cout * cin;
  if constexpr (PACK8) {
    if (wave == 0 && c < 24) {
#pragma unroll
      for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          dst[((long long)(3 * k + (c >> 3)) * cout + co0 + (r / 4) * 8 + 4 * h + (r & 3)) * cin + (c & 7)] = acc[k][r];
    }
  } else if (wave < 4) {
    const int ci = ci0 + c;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      const int tap = LAST ? 21 + k : 3 * k + wave;
      if (LAST && k == 6) {
        if (do_bias && c == 0)
#pragma unroll
          for (int r = 0; r < 16; ++r) bpart[(long long)chunk * cout + co0 + (r / 4) * 8 + 4 * h + (r & 3)] = acc[k][r];
      } else if (ci < cin) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          dst[((long long)tap * cout + co0 + (r / 4) * 8 + 4 * h + (r & 3)) * cin + ci] = acc[k][r];
      }
    }
  }
  };
  if constexpr (PACK8) {
    walk(std::false_type{});
  } else {
    if ((wave & 3) == 3)
      walk(std::true_type{});
    else
      walk(std::false_type{});
  }
}

// out[i] = sum over k of part[k][i], i < len.  A block of 256 threads covers OPB outputs with
// G = 256 / OPB groups; group g adds chunks g, g + G, ... in order, and the G group sums are
// added in group order, so the result does not depend on scheduling.
// Two sums share the launch: blocks [0, nb1) cover (part1, out1, len1), the rest (part2,
// out2, len2).
__global__ void __launch_bounds__(256) chunk_sum_kernel(const float* __restrict__ part1, float* __restrict__ out1,
                                                        long long len1, const float* __restrict__ part2,
                                                        float* __restrict__ out2, long long len2, long long nb1,
                                                        int nchunks, int opb) {
  __shared__ float sred[256];
  const bool first = blockIdx.x < nb1;
  const float* __restrict__ part = first ? part1 : part2;
  float* __restrict__ out = first ? out1 : out2;
  const long long len = first ? len1 : len2;
  const int t = threadIdx.x, o = t % opb, g = t / opb, G = 256 / opb;
  const long long i = (first ? (long long)blockIdx.x : (long long)blockIdx.x - nb1) * opb + o;
  float s = 0.0f;
  if (i < len) {
#pragma unroll 4
    for (int k = g; k < nchunks; k += G) s += part[(long long)k * len + i];
  }
  sred[t] = s;
  __syncthreads();
  if (g == 0 && i < len) {
    float sum = 0.0f;
    for (int q = 0; q < G; ++q) sum += sred[q * opb + o];
    out[i] = sum;
  }
}

// out1 = chunk sums of part1 (len1 >= 32), and of part2 into out2 when out2 is not null
inline void launch_chunk_sums(const float* part1, float* out1, long long len1, const float* part2, float* out2,
                              long long len2, int nchunks, hipStream_t s) {
  const int opb = 32;
  const long long nb1 = (len1 + opb - 1) / opb, nb2 = out2 ? (len2 + opb - 1) / opb : 0;
  hipLaunchKernelGGL(chunk_sum_kernel, dim3((unsigned)(nb1 + nb2)), dim3(256), 0, s, part1, out1, len1, part2, out2,
                     len2, nb1, nchunks, opb);
}

// ---------------------------------------------------------------- element-wise operators
// The element-wise operators move 8 channels (16 bytes) per thread; channel counts are
// multiples of 8 wherever they are called with voxel layouts, and the flat operators take a
// scalar tail.
// dx may alias dy: each thread reads its 8 elements before writing them
__global__ void relu_bwd_kernel(const uint16_t* __restrict__ y, const uint16_t* dy, uint16_t* dx, long long count,
                                int vec) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long e = 8 * i;
  if (vec && e + 8 <= count) {
    const uint4 yv = *reinterpret_cast<const uint4*>(y + e), gv = *reinterpret_cast<const uint4*>(dy + e);
    const uint32_t yw[4] = {yv.x, yv.y, yv.z, yv.w}, gw[4] = {gv.x, gv.y, gv.z, gv.w};
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = gw[k] & positive_mask(yw[k]);
    *reinterpret_cast<uint4*>(dx + e) = make_uint4(o[0], o[1], o[2], o[3]);
  } else {
    for (long long j = e; j < count && j < e + 8; ++j) dx[j] = bf2f(y[j]) > 0.0f ? dy[j] : (uint16_t)0;
  }
}

// (d, h, w): dimensions of the fine lattice; thread = (coarse voxel, 8 channels)
__global__ void pool_fwd_kernel(const uint16_t* __restrict__ in, uint16_t* __restrict__ out, int d, int h, int w, int c,
                                long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int c8 = c / 8, ch = 8 * (int)(i % c8);
  long long t = i / c8;
  const int x = (int)(t % (w / 2));
  t /= (w / 2);
  const int y = (int)(t % (h / 2));
  t /= (h / 2);
  const int z = (int)(t % (d / 2));
  const long long n = t / (d / 2);
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int k = 0; k < 8; ++k) {
    const int zz = 2 * z + (k >> 2), yy = 2 * y + ((k >> 1) & 1), xx = 2 * x + (k & 1);
    float f[8];
    unpack8(*reinterpret_cast<const uint4*>(in + (((n * d + zz) * h + yy) * (long long)w + xx) * c + ch), f);
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] += f[j];
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) s[j] *= 0.125f;
  *reinterpret_cast<uint4*>(out + (i / c8) * c + ch) = pack8(s);
}

// thread = (fine voxel, 8 channels)
__global__ void pool_bwd_kernel(const uint16_t* __restrict__ dout, uint16_t* __restrict__ din, int d, int h, int w,
                                int c, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int c8 = c / 8, ch = 8 * (int)(i % c8);
  long long t = i / c8;
  const long long vf = t;
  const int x = (int)(t % w);
  t /= w;
  const int y = (int)(t % h);
  t /= h;
  const int z = (int)(t % d);
  const long long n = t / d;
  float f[8];
  unpack8(*reinterpret_cast<const uint4*>(dout + (((n * (d / 2) + z / 2) * (h / 2) + y / 2) * (long long)(w / 2) + x / 2) *
                                                     c +
                                                 ch),
          f);
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] *= 0.125f;
  *reinterpret_cast<uint4*>(din + vf * c + ch) = pack8(f);
}

// (d, h, w): dimensions of the coarse input; out and skip are 2d x 2h x 2w; thread = (fine
// voxel, 8 channels)
__global__ void up_add_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ skip,
                              uint16_t* __restrict__ out, int d, int h, int w, int c, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int c8 = c / 8, ch = 8 * (int)(i % c8);
  long long t = i / c8;
  const long long vf = t;
  const int x = (int)(t % (2 * w));
  t /= (2 * w);
  const int y = (int)(t % (2 * h));
  t /= (2 * h);
  const int z = (int)(t % (2 * d));
  const long long n = t / (2 * d);
  float a[8], b[8];
  unpack8(*reinterpret_cast<const uint4*>(in + (((n * d + z / 2) * h + y / 2) * (long long)w + x / 2) * c + ch), a);
  unpack8(*reinterpret_cast<const uint4*>(skip + vf * c + ch), b);
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] += b[j];
  *reinterpret_cast<uint4*>(out + vf * c + ch) = pack8(a);
}

// thread = (coarse voxel, 8 channels); where mask (a ReLU output) is not positive the
// gradient is 0
__global__ void up_bwd_kernel(const uint16_t* __restrict__ dout, const uint16_t* __restrict__ mask,
                              uint16_t* __restrict__ din, int d, int h, int w, int c, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int c8 = c / 8, ch = 8 * (int)(i % c8);
  long long t = i / c8;
  const long long vc = t;
  const int x = (int)(t % w);
  t /= w;
  const int y = (int)(t % h);
  t /= h;
  const int z = (int)(t % d);
  const long long n = t / d;
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int k = 0; k < 8; ++k) {
    const int zz = 2 * z + (k >> 2), yy = 2 * y + ((k >> 1) & 1), xx = 2 * x + (k & 1);
    float f[8];
    unpack8(*reinterpret_cast<const uint4*>(dout + (((n * 2 * d + zz) * (2 * h) + yy) * (long long)(2 * w) + xx) * c + ch),
            f);
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] += f[j];
  }
  if (mask) {
    float mv[8];
    unpack8(*reinterpret_cast<const uint4*>(mask + vc * c + ch), mv);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (!(mv[j] > 0.0f)) s[j] = 0.0f;
  }
  *reinterpret_cast<uint4*>(din + vc * c + ch) = pack8(s);
}

// A block covers 256 voxels: each thread forms the errors of one, and the block then writes the
// gradient's 16-byte words in memory order (used <= 8; a thread that wrote its voxel's row by
// itself scattered them 2 stride bytes apart: 69 us for 2^20 voxels of 32 channels, 61 us now, of which 134 MB of pred lines are the most).
__global__ void __launch_bounds__(256) mse_kernel(const float* __restrict__ pred, const float* __restrict__ target,
                                                  uint16_t* __restrict__ dpred, float* __restrict__ loss_part,
                                                  long long count, int stride, int used) {
  __shared__ float s[256];
  __shared__ uint4 first[256];  // the first 8 channels of each voxel's gradient
  const long long v = (long long)blockIdx.x * 256 + threadIdx.x;
  float e2 = 0.0f;
  if (v < count) {
    const float scale = 2.0f / ((float)count * (float)used);
    for (int k0 = 0; k0 < (used > 8 ? stride : 8); k0 += 8) {
      float g[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        g[j] = 0.0f;
        if (k0 + j < used) {
          const float e = pred[v * stride + k0 + j] - target[v * used + k0 + j];
          e2 += e * e;
          g[j] = scale * e;
        }
      }
      if (used > 8)
        *reinterpret_cast<uint4*>(dpred + v * stride + k0) = pack8(g);
      else
        first[threadIdx.x] = pack8(g);
    }
  }
  s[threadIdx.x] = e2;
  __syncthreads();
  if (used <= 8) {
    const int words = stride / 8;
    const long long left = count - (long long)blockIdx.x * 256;
    const int n = (int)(left < 256 ? left : 256) * words;
    uint4* dst = reinterpret_cast<uint4*>(dpred) + (long long)blockIdx.x * 256 * words;
    for (int i = threadIdx.x; i < n; i += 256)
      dst[i] = i % words == 0 ? first[i / words] : make_uint4(0, 0, 0, 0);
  }
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_part[blockIdx.x] = s[0];
}

__global__ void adam_kernel(float* __restrict__ w, uint16_t* __restrict__ wb, const float* __restrict__ g,
                            float* __restrict__ m, float* __restrict__ v, long long count, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi, vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float wi = w[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  w[i] = wi;
  wb[i] = f2bf(wi);
}

// out may alias a or b: each thread reads its 8 elements before writing them.  Where mask (a
// ReLU output) is given and not positive the sum is 0.
__global__ void add_kernel(const uint16_t* a, const uint16_t* b, const uint16_t* mask, uint16_t* out, long long count,
                           int vec) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long e = 8 * i;
  if (vec && e + 8 <= count) {
    float fa[8], fb[8];
    unpack8(*reinterpret_cast<const uint4*>(a + e), fa);
    unpack8(*reinterpret_cast<const uint4*>(b + e), fb);
#pragma unroll
    for (int j = 0; j < 8; ++j) fa[j] += fb[j];
    if (mask) {
      float mv[8];
      unpack8(*reinterpret_cast<const uint4*>(mask + e), mv);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (!(mv[j] > 0.0f)) fa[j] = 0.0f;
    }
    *reinterpret_cast<uint4*>(out + e) = pack8(fa);
  } else {
    for (long long j = e; j < count && j < e + 8; ++j) {
      const float v = bf2f(a[j]) + bf2f(b[j]);
      out[j] = (mask && !(bf2f(mask[j]) > 0.0f)) ? (uint16_t)0 : f2bf(v);
    }
  }
}

__global__ void to_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) y[i] = f2bf(x[i]);
}

// y[v][c] = bf16(x[v][c]) for c < c_src, 0 for c_src <= c < c_dst; thread = (voxel, 8
// output channels), with 16-byte stores when c_dst is a multiple of 8 and y is aligned
__global__ void pack_input_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, long long nvox, int c_src,
                                  int c_dst, int vec) {
  const int g8 = (c_dst + 7) / 8;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvox * g8) return;
  const long long v = i / g8;
  const int c0 = 8 * (int)(i % g8);
  float f[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = c0 + j < c_src ? x[v * c_src + c0 + j] : 0.0f;
  if (vec) {
    *reinterpret_cast<uint4*>(y + v * c_dst + c0) = pack8(f);
  } else {
    for (int j = 0; j < 8 && c0 + j < c_dst; ++j) y[v * c_dst + c0 + j] = f2bf(f[j]);
  }
}

__global__ void to_f32_kernel(const uint16_t* __restrict__ x, float* __restrict__ y, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) y[i] = bf2f(x[i]);
}

inline hipStream_t S(void* s) { return static_cast<hipStream_t>(s); }
inline unsigned blocks(long long count, int per) { return (unsigned)((count + per - 1) / per); }
inline bool aligned16(const void* p) { return p && ((uintptr_t)p & 15) == 0; }
inline int done() { return hipGetLastError() == hipSuccess ? 0 : -2; }

}  // namespace

namespace {
// relu_y: the result is 0 where it is not positive (BF16 output)
int conv_dispatch(const uint16_t* in, const uint16_t* w, const float* bias, const uint16_t* relu_y, uint16_t* out,
                  float* out_f32, int n, int d, int h, int wd, int cin, int cout, int relu, void* stream) {
  if (n < 1 || d < 1 || h < 1 || wd < 1 || cin < 8 || cin % 8 || cout < 32 || cout % 32 || !in || !w ||
      (!out && !out_f32))
    return -1;
  const long long nvox = (long long)n * d * h * wd;
  hipStream_t s = S(stream);
  const bool small_plane = (long long)h * wd * cin < (1LL << 31);  // 32-bit offsets within an input plane
  switch (cin) {
    // (the box kernel applies no mask: the pass below does)
    case 8: launch_box<8>(in, w, bias, out, out_f32, n, d, h, wd, cout, relu, s); break;
    case 16: launch_box<16>(in, w, bias, out, out_f32, n, d, h, wd, cout, relu, s); break;
    case 32:
      if (small_plane) {
        launch_slide32(in, w, bias, relu_y, out, out_f32, n, d, h, wd, cout, relu, s);
        return done();
      }
      launch_staged<32>(in, w, bias, out, out_f32, n, d, h, wd, cout, relu, s);
      break;
    case 64:
      // few tiles: the staged kernel, whose blocks load no more than their own tile's share of the
      // weights and all three planes at once (1x5x9x33, 50 tiles x 2: 11 against 15 us; 1x64x16x16,
      // 512 x 2: 31 against 17)
      if (small_plane && (long long)n * d * ((wd + 31) / 32) * ((h + 1) / 2) * (cout / 32) > 256) {
        launch_slide<SlideConv<64, 1, 8, 1>>(in, w, bias, relu_y, out, out_f32, n, d, h, wd, cout, relu, s);
        return done();
      }
      launch_staged<64>(in, w, bias, out, out_f32, n, d, h, wd, cout, relu, s);
      break;
    case 128: launch_conv<128>(in, w, bias, out, out_f32, d, h, wd, cout, relu, nvox, s); break;
    default: return -1;
  }
  const int rc = done();
  return rc != 0 || !relu_y ? rc : surr_relu_bwd(relu_y, out, out, nvox * cout, stream);
}
}  // namespace

extern "C" int surr_conv3d_fwd(const uint16_t* in, const uint16_t* w, const float* bias, uint16_t* out, float* out_f32,
                               int n, int d, int h, int wd, int cin, int cout, int relu, void* stream) {
  return conv_dispatch(in, w, bias, nullptr, out, out_f32, n, d, h, wd, cin, cout, relu, stream);
}

extern "C" int surr_conv3d_flip_weights(const uint16_t* w, uint16_t* w_t, int cin, int cout, void* stream) {
  if (cin < 1 || cout < 1 || !w || !w_t) return -1;
  const long long total = 27LL * cin * cout;
  hipLaunchKernelGGL(flip_kernel, dim3(blocks(total, 256)), dim3(256), 0, S(stream), w, w_t, cin, cout);
  return done();
}

extern "C" int surr_conv3d_dgrad(const uint16_t* dout, const uint16_t* w_t, const uint16_t* relu_y, uint16_t* din, int n,
                                 int d, int h, int wd, int cin, int cout, void* stream) {
  // the forward convolution of dout (cout channels) with w_t gives din (cin channels)
  if (!din) return -1;
  return conv_dispatch(dout, w_t, nullptr, relu_y, din, nullptr, n, d, h, wd, cout, cin, 0, stream);
}

extern "C" size_t surr_conv3d_wgrad_scratch_bytes(int n, int d, int h, int wd, int cin, int cout) {
  if (n < 1 || d < 1 || h < 1 || wd < 1 || cin < 8 || cout < 32) return 0;
  const WgradPlan p = wgrad_plan(n, d, h, wd, cin, cout);
  return (size_t)p.nchunks * ((size_t)27 * cout * cin + (size_t)cout) * sizeof(float);
}

extern "C" int surr_conv3d_wgrad(const uint16_t* in, const uint16_t* dout, float* dw, float* dbias, void* scratch, int n,
                                 int d, int h, int wd, int cin, int cout, void* stream) {
  if (n < 1 || d < 1 || h < 1 || wd < 1 || cin < 8 || cin % 8 || cout < 32 || cout % 32 || !in || !dout || !dw ||
      !scratch)
    return -1;
  if ((long long)n * d * h * wd >= (1LL << 40)) return -1;
  const WgradPlan p = wgrad_plan(n, d, h, wd, cin, cout);
  float* part = static_cast<float*>(scratch);
  float* bpart = part + (size_t)p.nchunks * 27 * cout * cin;
  const dim3 grid(p.nchunks, p.tiles), block(kWgThreads);
  // PACK8 has a third of the MFMAs but adds up eight waves' sums at the end, not two.  With one step
  // per block that is no gain: 8 -> 32 channels on 3x5x5 voxels 12.1 us with it and 9.7 without, on
  // 256x16x32 (256 steps) 21.1 and 21.0, on 256x16x64 24.8 and 28.0.
  if (p.rows)
    hipLaunchKernelGGL(wgrad_row_kernel, grid, dim3(192), 0, S(stream), in, dout, part, dbias ? bpart : nullptr, d, h,
                       wd, cin, cout);
  else if (cin == 8 && p.steps > kWgBlocks)
    hipLaunchKernelGGL(wgrad_kernel<true>, grid, block, 0, S(stream), in, dout, part, dbias ? bpart : nullptr, d, h, wd,
                       cin, cout, p);
  else
    hipLaunchKernelGGL(wgrad_kernel<false>, grid, block, 0, S(stream), in, dout, part, dbias ? bpart : nullptr, d, h, wd,
                       cin, cout, p);
  launch_chunk_sums(part, dw, 27LL * cout * cin, bpart, dbias, (long long)cout, p.nchunks, S(stream));
  return done();
}

extern "C" int surr_relu_bwd(const uint16_t* y, const uint16_t* dy, uint16_t* dx, long long count, void* stream) {
  if (count < 0 || !y || !dy || !dx) return -1;
  if (count == 0) return 0;
  const int vec = aligned16(y) && aligned16(dy) && aligned16(dx);
  hipLaunchKernelGGL(relu_bwd_kernel, dim3(blocks(count, 8 * 256)), dim3(256), 0, S(stream), y, dy, dx, count, vec);
  return done();
}

extern "C" int surr_pool_fwd(const uint16_t* in, uint16_t* out, int n, int d, int h, int wd, int c, void* stream) {
  if (n < 1 || d < 2 || h < 2 || wd < 2 || (d | h | wd) & 1 || c < 8 || c % 8 || !aligned16(in) || !aligned16(out))
    return -1;
  const long long count = (long long)n * (d / 2) * (h / 2) * (wd / 2) * (c / 8);
  hipLaunchKernelGGL(pool_fwd_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), in, out, d, h, wd, c, count);
  return done();
}

extern "C" int surr_pool_bwd(const uint16_t* dout, uint16_t* din, int n, int d, int h, int wd, int c, void* stream) {
  if (n < 1 || d < 2 || h < 2 || wd < 2 || (d | h | wd) & 1 || c < 8 || c % 8 || !aligned16(dout) || !aligned16(din))
    return -1;
  const long long count = (long long)n * d * h * wd * (c / 8);
  hipLaunchKernelGGL(pool_bwd_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), dout, din, d, h, wd, c, count);
  return done();
}

extern "C" int surr_up_add_fwd(const uint16_t* in, const uint16_t* skip, uint16_t* out, int n, int d, int h, int wd,
                               int c, void* stream) {
  if (n < 1 || d < 1 || h < 1 || wd < 1 || c < 8 || c % 8 || !aligned16(in) || !aligned16(skip) || !aligned16(out))
    return -1;
  const long long count = (long long)n * 8 * d * h * wd * (c / 8);
  hipLaunchKernelGGL(up_add_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), in, skip, out, d, h, wd, c,
                     count);
  return done();
}

extern "C" int surr_up_bwd(const uint16_t* dout, const uint16_t* relu_y, uint16_t* din, int n, int d, int h, int wd, int c,
                           void* stream) {
  if (n < 1 || d < 1 || h < 1 || wd < 1 || c < 8 || c % 8 || !aligned16(dout) || !aligned16(din) ||
      (relu_y && !aligned16(relu_y)))
    return -1;
  const long long count = (long long)n * d * h * wd * (c / 8);
  hipLaunchKernelGGL(up_bwd_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), dout, relu_y, din, d, h, wd, c,
                     count);
  return done();
}

extern "C" int surr_mse(const float* pred, const float* target, uint16_t* dpred, float* loss_part, long long count,
                        int stride, int used, void* stream) {
  if (count < 1 || stride < 8 || stride % 8 || used < 1 || used > stride || !pred || !target || !aligned16(dpred) ||
      !loss_part)
    return -1;
  hipLaunchKernelGGL(mse_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), pred, target, dpred, loss_part,
                     count, stride, used);
  return done();
}

extern "C" int surr_adam(float* w, uint16_t* w_bf16, const float* g, float* m, float* v, long long count, float lr,
                         float beta1, float beta2, float eps, int t, void* stream) {
  if (count < 0 || t < 1 || !w || !w_bf16 || !g || !m || !v) return -1;
  const float c1 = 1.0f / (1.0f - powf(beta1, (float)t)), c2 = 1.0f / (1.0f - powf(beta2, (float)t));
  hipLaunchKernelGGL(adam_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), w, w_bf16, g, m, v, count, lr,
                     beta1, beta2, eps, c1, c2);
  return done();
}

extern "C" int surr_add(const uint16_t* a, const uint16_t* b, const uint16_t* relu_y, uint16_t* out, long long count,
                        void* stream) {
  if (count < 0 || !a || !b || !out) return -1;
  if (count == 0) return 0;
  const int vec = aligned16(a) && aligned16(b) && aligned16(out) && (!relu_y || aligned16(relu_y));
  hipLaunchKernelGGL(add_kernel, dim3(blocks(count, 8 * 256)), dim3(256), 0, S(stream), a, b, relu_y, out, count, vec);
  return done();
}

extern "C" int surr_to_bf16(const float* x, uint16_t* y, long long count, void* stream) {
  if (count < 0 || !x || !y) return -1;
  hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), x, y, count);
  return done();
}

extern "C" int surr_to_f32(const uint16_t* x, float* y, long long count, void* stream) {
  if (count < 0 || !x || !y) return -1;
  hipLaunchKernelGGL(to_f32_kernel, dim3(blocks(count, 256)), dim3(256), 0, S(stream), x, y, count);
  return done();
}

extern "C" int surr_pack_input(const float* x, uint16_t* y, long long nvox, int c_src, int c_dst, void* stream) {
  if (nvox < 0 || c_src < 1 || c_dst < c_src || !x || !y) return -1;
  if (nvox == 0) return 0;
  const int vec = c_dst % 8 == 0 && aligned16(y);
  hipLaunchKernelGGL(pack_input_kernel, dim3(blocks(nvox * ((c_dst + 7) / 8), 256)), dim3(256), 0, S(stream), x, y, nvox,
                     c_src, c_dst, vec);
  return done();
}
