// Learned-start network kernels (not part of the paper's method): three periodic
// 3x3x3 convolutions, channels-last bfloat16 activations, FP32 accumulation.
//
//   x0 = [delta_s, S_U u_p, r_x, r_y, r_z, 0, 0, 0]     (assembled on the fly)
//   a1 = relu(conv(x0; W1, b1))      8 -> 16   BF16 MFMA
//   a2 = relu(conv(a1; W2, b2))     16 -> 16   BF16 MFMA
//   y  =      conv(a2; W3, b3)      16 -> 1    BF16 MFMA (k_conv_out_mfma)
//   Delta u = y / S_U
//
// Parameter vector (FP32, device): W1 [16][27][8], b1 [16], W2 [16][27][16], b2 [16],
// W3 [1][27][16], b3 [1]; tap t = (dz+1)*9 + (dy+1)*3 + (dx+1), offset (dx, dy, dz).
//
// The forward convolutions and the data gradient of layer 2 (k_conv_fwd, k_conv_out_mfma) are implicit
// GEMMs on v_mfma_f32_16x16x32_bf16 over 16 x 8 x 8 output tiles (see there); the weight gradients
// (k_wgrad) run on the same instruction with positions as K, the output layer's backward
// (k_conv_out_bwd) on v_mfma_f32_16x16x4_f32.
#pragma once

#include "recon_kernels.hpp"

namespace recon {
namespace cnn {

constexpr int CIN = 8, CH = 16;
constexpr float S_U = 0.1f;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + CH * 27 * CIN, OFF_W2 = OFF_B1 + CH, OFF_B2 = OFF_W2 + CH * 27 * CH,
              OFF_W3 = OFF_B2 + CH, OFF_B3 = OFF_W3 + 27 * CH, NPARAM = OFF_B3 + 1;
constexpr int K1 = 27 * CIN, K1P = 224;      // layer-1 K padded to a multiple of 16
constexpr int K2 = 27 * CH;                  // 432
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float from_bf16(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

struct Geo3 {
  int n;
  float hs;
  float ds[3];
};

// ---------------------------------------------------------------------------
// Forward convolution on v_mfma_f32_16x16x32_bf16 (inference and the training forward).
//
// Block tile 16 (x) x 8 (y) x 8 (z) output cells, halo 18 x 10 x 10 cells staged once in LDS;
// each wave owns 16 x 4 x 4 outputs (16 output rows of 16 cells).  The wave walks the 6 x 6 input
// rows of its halo: an input row's A fragment (16 cells x K = 32) is loaded from LDS once and
// multiplied into every output row that uses it (up to 9), so one LDS read feeds up to 9 MFMAs.
// K = 32 of one fragment: C = 16: half 0 = taps dx = -1, 0 (16 channels each), half 1 = dx = +1
// and 16 zero columns;  C = 8: dx = -1, 0, +1 and 8 zero columns.
// Operand layout of that instruction: lane l holds A[l%16][8(l/16)+0..7], B[8(l/16)+0..7][l%16],
// and the result D[4(l/16)+0..3][l%16].
constexpr int FX = 16, FY = 8, FZ = 8, GX = FX + 2, GY = FY + 2, GZ = FZ + 2, GCELLS = GX * GY * GZ;
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// Byte offset of the 16-byte half h of halo cell c (C = 16: halves swapped on every other group of
// four cells so that 8 consecutive lanes reading one half hit distinct banks).
template <int C>
__device__ __forceinline__ int frag_off(int c, int h) {
  if (C == 16) return c * 32 + ((h ^ ((c >> 2) & 1)) << 4);
  return c * 16;
}

// Weight fragments: C = 16: wf[(g * 2 + h) * 64 + lane], C = 8: wf[g * 64 + lane], with
// g = (dz+1)*3 + (dy+1); 8 bf16 per lane in the B layout above.  wf2t: layer 2 with its taps flipped and
// its channels transposed (the data gradient of layer 2 as a forward convolution).
__global__ void __launch_bounds__(256) k_prep_frag(const float* __restrict__ th, uint4* __restrict__ wf1,
                                                   uint4* __restrict__ wf2, uint4* __restrict__ wf2t) {
  constexpr int F1 = 9 * 64, F2 = 9 * 2 * 64;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= F1 + 2 * F2) return;
  unsigned short v[8];
  if (e < F1) {
    const int g = e / 64, lane = e % 64, o = lane % 16, q = lane / 16;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int t = g * 3 + q;                     // dx = q - 1
      v[j] = q < 3 ? to_bf16(th[OFF_W1 + (o * 27 + t) * CIN + j]) : (unsigned short)0;
    }
  } else {
    const bool flip = e >= F1 + F2;
    const int f = e - F1 - (flip ? F2 : 0), g = f / 128, h = (f / 64) % 2, lane = f % 64, o = lane % 16, q = lane / 16;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 8 * q + j, ch = k % 16;
      const int t = g * 3 + (h == 0 ? (k < 16 ? 0 : 1) : 2);
      const bool zero = h == 1 && k >= 16;
      const int w = flip ? (ch * 27 + 26 - t) * CH + o : (o * 27 + t) * CH + ch;
      v[j] = zero ? (unsigned short)0 : to_bf16(th[OFF_W2 + w]);
    }
  }
  uint4* dst = e < F1 ? wf1 + e : (e < F1 + F2 ? wf2 + (e - F1) : wf2t + (e - F1 - F2));
  *dst = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}

// One cell of the assembled 8-channel input x0 = [delta, S_U u_p, r_hat, 0, 0, 0] (bf16) at node (x, y, z).
__device__ __forceinline__ uint4 x0_cell(const Geo3& g, int x, int y, int z, float delta, float up) {
  const float rx = fmaf(g.hs, (float)x, g.ds[0]), ry = fmaf(g.hs, (float)y, g.ds[1]),
              rz = fmaf(g.hs, (float)z, g.ds[2]);
  const float r2 = rx * rx + ry * ry + rz * rz;
  const float ir = r2 > 0.f ? rsqrtf(r2) : 0.f;
  const unsigned a0 = to_bf16(delta), a1 = to_bf16(S_U * up);
  const unsigned a2 = to_bf16(rx * ir), a3 = to_bf16(ry * ir), a4 = to_bf16(rz * ir);
  return make_uint4(a0 | (a1 << 16), a2 | (a3 << 16), a4, 0u);
}

// Stage the 18 x 10 x 10 halo of a channels-last bf16 tensor into LDS: every thread issues all of
// its 16-byte loads before the first LDS store so the loads are in flight together.
template <int C>
__device__ __forceinline__ void stage_halo(unsigned char* lds, const unsigned short* __restrict__ src, int n, int x0,
                                           int y0, int z0) {
  constexpr int CPC = C / 8, TOTAL = GCELLS * CPC, PER = (TOTAL + 255) / 256;
  const int msk = n - 1;
  uint4 v[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int e0 = threadIdx.x + k * 256;
    const int e = e0 < TOTAL ? e0 : TOTAL - 1;        // tail lanes reload the last chunk
    const int c = e / CPC, h = e % CPC;
    const int hx = c % GX, hy = (c / GX) % GY, hz = c / (GX * GY);
    const long long gc = ((long long)((z0 - 1 + hz) & msk) * n + ((y0 - 1 + hy) & msk)) * n + ((x0 - 1 + hx) & msk);
    v[k] = *(const uint4*)(src + gc * C + 8 * h);
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int e = threadIdx.x + k * 256;
    if (e < TOTAL) *(uint4*)(lds + frag_off<C>(e / CPC, e % CPC)) = v[k];
  }
}

//   SRC 0: input is a bf16 tensor [n^3][C];  SRC 1: input is x0 assembled from (delta, u_p), C = 8.
//   EPI 0: out = bf16(relu(acc + bias));     EPI 1: out = bf16(acc) where gate > 0, else 0 (data gradient).
//   out and gate: channels-last [n^3][16].
template <int C, int SRC, int EPI = 0>
__global__ void __launch_bounds__(256) k_conv_fwd(const unsigned short* __restrict__ in,
                                                     const float* __restrict__ delta, const float* __restrict__ up,
                                                     Geo3 g, const uint4* __restrict__ wf,
                                                     const float* __restrict__ bias, unsigned short* __restrict__ out,
                                                     const unsigned short* __restrict__ gate = nullptr) {
  constexpr int NH = C == 16 ? 2 : 1;
  // halo of the input (bf16 channels) during the products, then the output tile (16 channels, bf16)
  constexpr int LDS_IN = GCELLS * C * 2, LDS_OUT = FX * FY * FZ * 32;
  __shared__ __align__(16) unsigned char lds[LDS_IN > LDS_OUT ? LDS_IN : LDS_OUT];
  const long long n3 = (long long)g.n * g.n * g.n;
  const int b = blockIdx.y, msk = g.n - 1;
  const int nbx = g.n / FX, nby = g.n / FY;
  const int x0 = (blockIdx.x % nbx) * FX, y0 = ((blockIdx.x / nbx) % nby) * FY, z0 = (blockIdx.x / (nbx * nby)) * FZ;
  if (SRC == 0) {
    stage_halo<C>(lds, in + b * n3 * C, g.n, x0, y0, z0);
  } else {
    const float* dl = delta + b * n3;
    const float* ul = up + b * n3;
    constexpr int PER = (GCELLS + 255) / 256;
    float dv[PER], uv[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int c = threadIdx.x + k * 256;
      if (c < GCELLS) {
        const int hx = c % GX, hy = (c / GX) % GY, hz = c / (GX * GY);
        const long long gc = ((long long)((z0 - 1 + hz) & msk) * g.n + ((y0 - 1 + hy) & msk)) * g.n + ((x0 - 1 + hx) & msk);
        dv[k] = dl[gc];
        uv[k] = ul[gc];
      }
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int c = threadIdx.x + k * 256;
      if (c < GCELLS) {
        const int hx = c % GX, hy = (c / GX) % GY, hz = c / (GX * GY);
        const int x = (x0 - 1 + hx) & msk, y = (y0 - 1 + hy) & msk, z = (z0 - 1 + hz) & msk;
        *(uint4*)(lds + c * 16) = x0_cell(g, x, y, z, dv[k], uv[k]);
      }
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 15, q = lane >> 4;
  bf8 bw[9][NH];
#pragma unroll
  for (int gi = 0; gi < 9; ++gi)
#pragma unroll
    for (int h = 0; h < NH; ++h) bw[gi][h] = __builtin_bit_cast(bf8, wf[(gi * NH + h) * 64 + lane]);
  __syncthreads();
  const int wy0 = 4 * (wave & 1), wz0 = 4 * (wave >> 1);
  f4 acc[4][4];
#pragma unroll
  for (int oz = 0; oz < 4; ++oz)
#pragma unroll
    for (int oy = 0; oy < 4; ++oy) acc[oz][oy] = f4{0.f, 0.f, 0.f, 0.f};
  const bf8 zero8 = __builtin_bit_cast(bf8, make_uint4(0u, 0u, 0u, 0u));
#pragma unroll
  for (int iz = 0; iz < 6; ++iz) {
#pragma unroll
    for (int iy = 0; iy < 6; ++iy) {
      const int rowc = ((wz0 + iz) * GY + (wy0 + iy)) * GX;
      bf8 a[NH];
      if (C == 16) {
        a[0] = __builtin_bit_cast(bf8, *(const uint4*)(lds + frag_off<C>(rowc + m + (q >> 1), q & 1)));
        const bf8 t1 = __builtin_bit_cast(bf8, *(const uint4*)(lds + frag_off<C>(rowc + m + 2, q & 1)));
        a[NH - 1] = q < 2 ? t1 : zero8;
      } else {
        const bf8 t0 = __builtin_bit_cast(bf8, *(const uint4*)(lds + frag_off<C>(rowc + m + (q < 3 ? q : 2), 0)));
        a[0] = q < 3 ? t0 : zero8;
      }
#pragma unroll
      for (int oz = 0; oz < 4; ++oz) {
        const int dz = iz - 1 - oz;
        if (dz < -1 || dz > 1) continue;
#pragma unroll
        for (int oy = 0; oy < 4; ++oy) {
          const int dy = iy - 1 - oy;
          if (dy < -1 || dy > 1) continue;
          const int gi = (dz + 1) * 3 + (dy + 1);
#pragma unroll
          for (int h = 0; h < NH; ++h)
            acc[oz][oy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[h], bw[gi][h], acc[oz][oy], 0, 0, 0);
        }
      }
    }
  }
  // epilogue: lane (m, q) holds channel m of cells 4q..4q+3 of each output row; channel pairs are
  // exchanged with the neighbouring lane and the packed words go to the output tile in LDS
  // ([cell][16 channels]), from which every lane stores whole 16-byte halves of cells
  const float bm = EPI == 0 ? bias[m] : 0.f;
  const bool even = (m & 1) == 0;
  __syncthreads();                                  // every wave is done with the halo
  unsigned* t32 = (unsigned*)lds;
#pragma unroll
  for (int oz = 0; oz < 4; ++oz) {
#pragma unroll
    for (int oy = 0; oy < 4; ++oy) {
      unsigned mine[4], other[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) mine[i] = to_bf16(EPI == 0 ? fmaxf(acc[oz][oy][i] + bm, 0.f) : acc[oz][oy][i]);
#pragma unroll
      for (int i = 0; i < 4; ++i) other[i] = (unsigned)__shfl_xor((int)mine[i], 1);
      const int cell0 = ((wz0 + oz) * FY + (wy0 + oy)) * FX + 4 * q;
      const int ch2 = m >> 1;                       // channel pair
      if (even) {
        t32[(cell0 + 0) * 8 + ch2] = mine[0] | (other[0] << 16);
        t32[(cell0 + 1) * 8 + ch2] = mine[1] | (other[1] << 16);
      } else {
        t32[(cell0 + 2) * 8 + ch2] = other[2] | (mine[2] << 16);
        t32[(cell0 + 3) * 8 + ch2] = other[3] | (mine[3] << 16);
      }
    }
  }
  __syncthreads();
  const uint4* t128 = (const uint4*)lds;
  uint4* o128 = (uint4*)out;
#pragma unroll
  for (int k = 0; k < FX * FY * FZ * 2 / 256; ++k) {
    const int e = threadIdx.x + k * 256;           // 16-byte half e % 2 of tile cell e / 2
    const int cell = e >> 1, lx = cell % FX, ly = (cell / FX) % FY, lz = cell / (FX * FY);
    const long long row = b * n3 + ((long long)(z0 + lz) * g.n + (y0 + ly)) * g.n + x0 + lx;
    uint4 v = t128[e];
    if constexpr (EPI == 1) {
      const uint4 gt = ((const uint4*)gate)[row * 2 + (e & 1)];
      auto open = [](unsigned w, unsigned gw) {
        return (from_bf16((unsigned short)(gw & 0xFFFFu)) > 0.f ? (w & 0xFFFFu) : 0u) |
               (from_bf16((unsigned short)(gw >> 16)) > 0.f ? (w & 0xFFFF0000u) : 0u);
      };
      v = make_uint4(open(v.x, gt.x), open(v.y, gt.y), open(v.z, gt.z), open(v.w, gt.w));
    }
    o128[row * 2 + (e & 1)] = v;
  }
}

// Output layer (16 -> 1) on MFMA for the forward pass: with one output channel the N dimension of
// the instruction runs over the wave's 16 output rows instead.  For input row (iz, iy) the B
// fragment column n = output row (oz, oy) = (n / 4, n % 4) holds W3 of tap (iz - 1 - oz, iy - 1 - oy, dx)
// (zero when that row is out of reach), so each A fragment is used once for all 16 output rows.
__global__ void __launch_bounds__(256) k_conv_out_mfma(const unsigned short* __restrict__ a2, Geo3 g,
                                                       const float* __restrict__ w3f, const float* __restrict__ b3,
                                                       float scale, float* __restrict__ y_out) {
  __shared__ __align__(16) unsigned char lds[GCELLS * CH * 2];
  __shared__ __align__(16) unsigned short w3b[27 * CH];
  const long long n3 = (long long)g.n * g.n * g.n;
  const int b = blockIdx.y, msk = g.n - 1;
  const int nbx = g.n / FX, nby = g.n / FY;
  const int x0 = (blockIdx.x % nbx) * FX, y0 = ((blockIdx.x / nbx) % nby) * FY, z0 = (blockIdx.x / (nbx * nby)) * FZ;
  stage_halo<CH>(lds, a2 + b * n3 * CH, g.n, x0, y0, z0);
  for (int i = threadIdx.x; i < 27 * CH; i += 256) w3b[i] = to_bf16(w3f[i]);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 15, q = lane >> 4;
  const int wy0 = 4 * (wave & 1), wz0 = 4 * (wave >> 1);
  const int oz = m >> 2, oy = m & 3;                  // output row of B / D column m
  const bf8 zero8 = __builtin_bit_cast(bf8, make_uint4(0u, 0u, 0u, 0u));
  f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int iz = 0; iz < 6; ++iz) {
#pragma unroll
    for (int iy = 0; iy < 6; ++iy) {
      const int rowc = ((wz0 + iz) * GY + (wy0 + iy)) * GX;
      const bf8 a0 = __builtin_bit_cast(bf8, *(const uint4*)(lds + frag_off<CH>(rowc + m + (q >> 1), q & 1)));
      const bf8 t1 = __builtin_bit_cast(bf8, *(const uint4*)(lds + frag_off<CH>(rowc + m + 2, q & 1)));
      const bf8 a1 = q < 2 ? t1 : zero8;
      const int dz = iz - 1 - oz, dy = iy - 1 - oy;
      const bool ok = dz >= -1 && dz <= 1 && dy >= -1 && dy <= 1;
      const int tb = ok ? (dz + 1) * 9 + (dy + 1) * 3 : 0;   // tap of dx = -1
      // half 0: q < 2 -> dx = -1, q >= 2 -> dx = 0;  half 1: q < 2 -> dx = +1, else zero
      const bf8 w0 = __builtin_bit_cast(bf8, *(const uint4*)(w3b + (tb + (q >> 1)) * CH + 8 * (q & 1)));
      const bf8 w1 = __builtin_bit_cast(bf8, *(const uint4*)(w3b + (tb + 2) * CH + 8 * (q & 1)));
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, ok ? w0 : zero8, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, (ok && q < 2) ? w1 : zero8, acc, 0, 0, 0);
    }
  }
  // lane (m, q) holds output row m, cells 4q .. 4q+3
  const float bb = b3[0];
  const long long row = b * n3 + ((long long)(z0 + wz0 + oz) * g.n + (y0 + wy0 + oy)) * g.n + x0 + 4 * q;
  *(float4*)(y_out + row) = make_float4((acc[0] + bb) * scale, (acc[1] + bb) * scale, (acc[2] + bb) * scale,
                                        (acc[3] + bb) * scale);
}

// Loss residual: r = y - S_U target; dy = 2 r / count; per-block partial of sum r^2.
__global__ void __launch_bounds__(256) k_loss(const float* __restrict__ y, const float* __restrict__ target,
                                              long long count, float* __restrict__ dy, double* __restrict__ partial) {
  double acc = 0.0;
  const float inv = 2.0f / (float)count;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < count; i += (long long)gridDim.x * 256) {
    const float r = y[i] - S_U * target[i];
    dy[i] = inv * r;
    acc += (double)r * (double)r;
  }
  double t1, t2;
  block_sum2<256>(acc, 0.0, &t1, &t2);
  if (threadIdx.x == 0) partial[blockIdx.x] = t1;
}

// ---------------------------------------------------------------------------
// Backward of the training step.  Every block takes its tiles in a fixed order and leaves one row of partial
// sums; k_reduce_parts adds the rows in FP64 in a fixed order, so a step is deterministic for a given grid and
// batch.  What is added up in FP32 does not grow with the batch: 256 positions in the output layer's backward
// (wgrad_rows for the other two).
// ---------------------------------------------------------------------------
// 16 bytes as a vector: arrays of the struct uint4 held across a barrier are put in scratch memory (the weight
// gradients took 120 and 52 us with it, 58 and 35 us as below).
typedef unsigned u4 __attribute__((ext_vector_type(4)));

// Output-layer backward: d2[p][i] = bf16((sum_t W3[t][i] dy[p - d_t]) * [a2[p][i] > 0]),
// and per-block partials of dW3[t][i] = sum_p dy[p - d_t] a2[p][i] (the same sum as over dy[p] a2[p + d_t]:
// the grid is periodic) and db3 = sum_p dy[p].
//
// Both sums are contractions with FP32 operands (dy is never rounded) on v_mfma_f32_16x16x4_f32, tile
// 16 x 8 x 8 cells, four waves of 16 rows: d2 with M = 16 cells of a row, N = 16 channels, K = 27 taps
// padded to 28; dW3 with M = taps (two tiles), N = channels, K = 4 cells per instruction.  Only dy needs
// a halo.  One tile per block: each wave adds up its 256 positions in FP32, the four waves' sums meet in FP64.
// Operand layout: lane l holds A[l%16][l/16], B[l/16][l%16], D[4(l/16)+0..3][l%16].
// 63 us on a 128^3 network grid (0.14 GB, 240 products of 32 cycles per wave and tile; 72 with several tiles per
// block, whose loads then wait for the last tile's stores), against 200 us
// with one FMA and two LDS reads per (tap, channel, cell).
__global__ void __launch_bounds__(256) k_conv_out_bwd(const float* __restrict__ dy, const unsigned short* __restrict__ a2,
                                                      Geo3 g, const float* __restrict__ w3f,
                                                      unsigned short* __restrict__ dpre2, float* __restrict__ part) {
  constexpr int ROWW = 27 * CH + 1, CELLS = FX * FY * FZ;
  __shared__ float dyt[GCELLS];
  __shared__ __align__(16) unsigned short tile[CELLS * CH];   // a2, then d2 in place; at the end the wave sums
  static_assert(sizeof(double) * 4 * ROWW <= sizeof(tile), "the wave sums reuse the tile");
  const long long n3 = (long long)g.n * g.n * g.n;
  const int n = g.n, msk = n - 1, nbx = n / FX, nby = n / FY, per = nbx * nby * (n / FZ);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, q = lane >> 4;
  const int wy0 = 4 * (wave & 1), wz0 = 4 * (wave >> 1);
  auto tap_off = [](int t) { return (t % 3 - 1) + ((t / 3) % 3 - 1) * GX + (t / 9 - 1) * GX * GY; };
  float w[7];
  int da[7], dt[2];
#pragma unroll
  for (int s = 0; s < 7; ++s) {
    const int t = 4 * s + q;
    w[s] = t < 27 ? from_bf16(to_bf16(w3f[t * CH + m])) : 0.f;
    da[s] = m - tap_off(t < 27 ? t : 26);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int t = 16 * a + m;
    dt[a] = q - tap_off(t < 27 ? t : 26);                  // rows 27..31 of the product are not used
  }
  f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
  float bacc = 0.f;
  const int b = blockIdx.x / per, tt = blockIdx.x % per;
  const int x0 = (tt % nbx) * FX, y0 = ((tt / nbx) % nby) * FY, z0 = (tt / (nbx * nby)) * FZ;
  constexpr int PD = (GCELLS + 255) / 256, PA = CELLS * 2 / 256;
  float dv[PD];
  u4 av[PA];
#pragma unroll
  for (int k = 0; k < PD; ++k) {
    const int c0 = threadIdx.x + k * 256, c = c0 < GCELLS ? c0 : GCELLS - 1;
    const int hx = c % GX, hy = (c / GX) % GY, hz = c / (GX * GY);
    dv[k] = dy[b * n3 + ((long long)((z0 - 1 + hz) & msk) * n + ((y0 - 1 + hy) & msk)) * n + ((x0 - 1 + hx) & msk)];
  }
  const u4* a128 = (const u4*)a2;
#pragma unroll
  for (int k = 0; k < PA; ++k) {
    const int e = threadIdx.x + k * 256, cell = e >> 1;
    const int lx = cell % FX, ly = (cell / FX) % FY, lz = cell / (FX * FY);
    av[k] = a128[(b * n3 + ((long long)(z0 + lz) * n + (y0 + ly)) * n + x0 + lx) * 2 + (e & 1)];
  }
#pragma unroll
  for (int k = 0; k < PD; ++k)
    if (threadIdx.x + k * 256 < GCELLS) dyt[threadIdx.x + k * 256] = dv[k];
#pragma unroll
  for (int k = 0; k < PA; ++k) ((u4*)tile)[threadIdx.x + k * 256] = av[k];
  __syncthreads();
  for (int c = threadIdx.x; c < CELLS; c += 256)
    bacc += dyt[((c / (FX * FY) + 1) * GY + (c / FX) % FY + 1) * GX + c % FX + 1];
#pragma unroll 2
  for (int row = 0; row < 16; ++row) {
    const int lz = wz0 + (row >> 2), ly = wy0 + (row & 3);
    const int hrow = ((lz + 1) * GY + ly + 1) * GX + 1;  // halo cell of the row's first cell
    unsigned short* cells = tile + (lz * FY + ly) * FX * CH;
    f4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 7; ++s) d = __builtin_amdgcn_mfma_f32_16x16x4f32(dyt[hrow + da[s]], w[s], d, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float bv = from_bf16(cells[(4 * k + q) * CH + m]);
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(dyt[hrow + 4 * k + dt[0]], bv, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(dyt[hrow + 4 * k + dt[1]], bv, acc[1], 0, 0, 0);
    }
    // the wave alone reads and writes this row: its reads above are issued before these writes
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      unsigned short* c = cells + (4 * q + i) * CH + m;
      *c = from_bf16(*c) > 0.f ? to_bf16(d[i]) : (unsigned short)0;
    }
  }
  __syncthreads();
  uint4* o128 = (uint4*)dpre2;
#pragma unroll
  for (int k = 0; k < PA; ++k) {
    const int e = threadIdx.x + k * 256, cell = e >> 1;
    const int lx = cell % FX, ly = (cell / FX) % FY, lz = cell / (FX * FY);
    o128[(b * n3 + ((long long)(z0 + lz) * n + (y0 + ly)) * n + x0 + lx) * 2 + (e & 1)] = ((const uint4*)tile)[e];
  }
  __syncthreads();
  double* red = (double*)tile;                             // [4 waves][ROWW]
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = 16 * a + 4 * q + i;
      if (t < 27) red[wave * ROWW + t * CH + m] = (double)acc[a][i];
    }
  double bsum = (double)bacc;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) bsum += __shfl_xor(bsum, o, 64);
  if (lane == 0) red[wave * ROWW + ROWW - 1] = bsum;
  __syncthreads();
  for (int e = threadIdx.x; e < ROWW; e += 256)
    part[(long long)blockIdx.x * ROWW + e] =
        (float)((red[e] + red[ROWW + e]) + (red[2 * ROWW + e] + red[3 * ROWW + e]));
}

// Weight gradient of a 16-output convolution:
//   dW[o][t C + i] = sum_p dpre[p][o] x[p + d_t][i],  db[o] = sum_p dpre[p][o]
// on v_mfma_f32_16x16x32_bf16 with M = 16 output channels, N = 16 columns (C = 16: the channels of one
// tap; C = 8: two taps) and K = 32 positions (two x rows).  Both operands are channels-last in LDS and
// are needed position-fastest: ds_read_b64_tr_b16 transposes on the way (in each group of 16 lanes, lane
// 4 r + c reads channels 4c..4c+3 of position r, and lane i receives channel i of positions 0..3), so a
// tap is only an address offset and nothing is gathered element by element.  A group of lanes reads 128
// contiguous bytes, free of bank conflicts.  The four waves split the column tiles; a block takes the tiles of
// 16 x 4 x 8 positions that wgrad_rows gives it, adds their products up in FP32 and writes one partial [16][KP + 1]
// (bias in the last column).  HALVES (16^3): the FP32 sums end with each half of a tile.
// Bound by the staging of a tile before its products (with a wave taking two z planes and all taps, a third
// of the LDS reads, 56 us instead of 58).  On a 128^3 network grid 57 us (layer 2) and 35 us (layer 1); with
// element-by-element gathers of the operand, 225 and 201 us.
constexpr int VX = 16, VY = 4, VZ = 8, UX = VX + 2, UY = VY + 2, UZ = VZ + 2, UCELLS = UX * UY * UZ;
constexpr int VCELLS = VX * VY * VZ;

// Blocks of k_wgrad, and so rows of partial sums (42 KB each, both layers): 16 n positions a row, which is what is
// added up in FP32 (256 at 16^3, where a block's tile of 512 is summed in halves), or one tile.  1,024 rows at
// 128^3, 4,096 at 256^3.
inline long long wgrad_rows(long long n, long long batch) {
  const long long tiles = batch * n * n * n / VCELLS, rows = batch * n * n / 16;
  return tiles < rows ? tiles : rows;
}

__device__ __forceinline__ bf8 tr_pair(const unsigned short* p0, const unsigned short* p1) {
  typedef __attribute__((address_space(3))) s4 lds4;
  const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)p0);
  const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)p1);
  typedef short s8 __attribute__((ext_vector_type(8)));
  return __builtin_bit_cast(bf8, s8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]});
}

//   SRC 0: x is a bf16 tensor [n^3][C];  SRC 1: x is x0 assembled from (delta, u_p), C = 8
template <int C, int KP, int SRC, bool HALVES>
__global__ void __launch_bounds__(256) k_wgrad(const unsigned short* __restrict__ dpre,
                                               const unsigned short* __restrict__ in, const float* __restrict__ delta,
                                               const float* __restrict__ up, Geo3 g, int tiles,
                                               float* __restrict__ part) {
  constexpr int NT = KP / 16;                 // column tiles: C = 16 -> 27 taps, C = 8 -> 14 tap pairs
  constexpr int TPW = (NT + 3) / 4;           // column tiles per wave
  __shared__ __align__(16) unsigned short xt[UCELLS * C];
  __shared__ __align__(16) unsigned short dt[VCELLS * CH];
  const long long n3 = (long long)g.n * g.n * g.n;
  const int n = g.n, msk = n - 1, nbx = n / VX, nby = n / VY, per = nbx * nby * (n / VZ);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, q = lane >> 4;
  const int r = m >> 2, c = m & 3;            // position and channel quarter this lane reads for its group
  int off[TPW];                               // element offset of column tile wave + 4k from the row's first halo cell
#pragma unroll
  for (int k = 0; k < TPW; ++k) {
    int t = C == 16 ? wave + 4 * k : 2 * (wave + 4 * k) + (c >> 1);
    if (t > 26) t = 26;                       // padded columns: computed and not used
    const int cell = 1 + (t % 3 - 1) + ((t / 3) % 3 - 1) * UX + (t / 9 - 1) * UX * UY + 4 * q + r;
    off[k] = cell * C + (C == 16 ? 4 * c : 4 * (c & 1));
  }
  const bf8 ones = __builtin_bit_cast(bf8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
  f4 acc[TPW], bacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < TPW; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
  double sum[TPW][4] = {}, bsum[4] = {};      // HALVES
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int b = t / per, tt = t % per;
    const int x0 = (tt % nbx) * VX, y0 = ((tt / nbx) % nby) * VY, z0 = (tt / (nbx * nby)) * VZ;
    auto halo = [&](int cell) {
      const int hx = cell % UX, hy = (cell / UX) % UY, hz = cell / (UX * UY);
      return b * n3 + ((long long)((z0 - 1 + hz) & msk) * n + ((y0 - 1 + hy) & msk)) * n + ((x0 - 1 + hx) & msk);
    };
    constexpr int PD = VCELLS * 2 / 256;
    u4 dv[PD];
#pragma unroll
    for (int k = 0; k < PD; ++k) {
      const int e = threadIdx.x + k * 256, cell = e >> 1;
      const int lx = cell % VX, ly = (cell / VX) % VY, lz = cell / (VX * VY);
      dv[k] = ((const u4*)dpre)[(b * n3 + ((long long)(z0 + lz) * n + (y0 + ly)) * n + x0 + lx) * 2 + (e & 1)];
    }
    if constexpr (SRC == 0) {
      constexpr int CPC = C / 8, TOTAL = UCELLS * CPC, PER = (TOTAL + 255) / 256;
      u4 v[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e0 = threadIdx.x + k * 256, e = e0 < TOTAL ? e0 : TOTAL - 1;
        v[k] = *(const u4*)(in + halo(e / CPC) * C + 8 * (e % CPC));
      }
      __syncthreads();                        // every wave is done with the last tile
#pragma unroll
      for (int k = 0; k < PER; ++k)
        if (threadIdx.x + k * 256 < TOTAL) ((u4*)xt)[threadIdx.x + k * 256] = v[k];
    } else {
      constexpr int PER = (UCELLS + 255) / 256;
      float fd[PER], fu[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e0 = threadIdx.x + k * 256;
        const long long s = halo(e0 < UCELLS ? e0 : UCELLS - 1);
        fd[k] = delta[s];
        fu[k] = up[s];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + k * 256;
        if (e < UCELLS) {
          const int hx = e % UX, hy = (e / UX) % UY, hz = e / (UX * UY);
          ((uint4*)xt)[e] = x0_cell(g, (x0 - 1 + hx) & msk, (y0 - 1 + hy) & msk, (z0 - 1 + hz) & msk, fd[k], fu[k]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < PD; ++k) ((u4*)dt)[threadIdx.x + k * 256] = dv[k];
    __syncthreads();
    const int da = (4 * q + r) * CH + 4 * c;  // dpre element of this lane in a row
#pragma unroll 2
    for (int s = 0; s < VY * VZ / 2; ++s) {   // rows 2s and 2s + 1: the same z, y = 2 (s % 2) and the next
      const int lz = s / (VY / 2), ly = 2 * (s % (VY / 2));
      const unsigned short* dr = dt + (lz * VY + ly) * VX * CH + da;
      const bf8 a = tr_pair(dr, dr + VX * CH);
      const unsigned short* xr = xt + ((lz + 1) * UY + ly + 1) * UX * C;
      // every wave runs all TPW products and the bias, without branches between them (a wave past the
      // last column tile repeats the last tap, and only wave 3 stores its bias)
      bf8 x[TPW];
#pragma unroll
      for (int k = 0; k < TPW; ++k) x[k] = tr_pair(xr + off[k], xr + off[k] + UX * C);
#pragma unroll
      for (int k = 0; k < TPW; ++k) acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x[k], acc[k], 0, 0, 0);
      bacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, bacc, 0, 0, 0);
      if (HALVES && (s + 1) % (VY * VZ / 4) == 0) {
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
#pragma unroll
          for (int i = 0; i < 4; ++i) sum[k][i] += (double)acc[k][i];
          acc[k] = f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) bsum[i] += (double)bacc[i];
        bacc = f4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
  // D[o = 4q + i][col = m] for each column tile
  float* pb = part + (long long)blockIdx.x * (CH * (KP + 1));
#pragma unroll
  for (int k = 0; k < TPW; ++k) {
    const int nt = wave + 4 * k;
    if (nt < NT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) pb[(4 * q + i) * (KP + 1) + nt * 16 + m] = HALVES ? (float)sum[k][i] : acc[k][i];
    }
  }
  if (wave == 3 && m == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) pb[(4 * q + i) * (KP + 1) + KP] = HALVES ? (float)bsum[i] : bacc[i];
  }
}

// Sums of the partial rows in FP64, all three layers in one launch: out[slice][column] = sum over the
// slice's rows, columns in the order layer 3 [433], layer 2 [16][433], layer 1 [16][225].  A block takes
// 64 columns; its four waves take every fourth row of the slice with four loads in flight each: 14 us
// at 128^3.  (One thread per column over all rows, 8,192 of them in layer 3, was 3.87 of a 4.84 ms
// training step: three launches of 2 to 28 blocks, one dependent FP64 add after another.)  The last
// column block's first slice sums the loss.
constexpr int kRedSlices = 16;   // at most; one per 64 rows
constexpr int COL3 = K2 + 1, COL2 = CH * (K2 + 1), COL1 = CH * (K1P + 1), NCOLS = COL3 + COL2 + COL1;
constexpr int RB3 = (COL3 + 63) / 64, RB2 = (COL2 + 63) / 64, RB1 = (COL1 + 63) / 64;
__global__ void __launch_bounds__(256) k_reduce_parts(const float* __restrict__ p3, long long n3r,
                                                      const float* __restrict__ p2, const float* __restrict__ p1,
                                                      long long nwr, double* __restrict__ out,
                                                      const double* __restrict__ lossp, int nloss,
                                                      double* __restrict__ losst) {
  if (blockIdx.x == RB3 + RB2 + RB1) {
    if (blockIdx.y != 0) return;
    double a = 0.0;
    for (int i = threadIdx.x; i < nloss; i += 256) a += lossp[i];
    double t1, t2;
    block_sum2<256>(a, 0.0, &t1, &t2);
    if (threadIdx.x == 0) losst[0] = t1;
    return;
  }
  __shared__ double sh[4][64];
  int cb = blockIdx.x, ncols = COL3, base = 0;
  const float* p = p3;
  long long rows = n3r;
  if (cb >= RB3) { cb -= RB3; p = p2; rows = nwr; ncols = COL2; base = COL3; }
  if (base && cb >= RB2) { cb -= RB2; p = p1; ncols = COL1; base = COL3 + COL2; }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = cb * 64 + lane;
  const long long lo = rows * blockIdx.y / gridDim.y, hi = rows * (blockIdx.y + 1) / gridDim.y;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  if (col < ncols) {
    long long i = lo + wave;
    for (; i + 12 < hi; i += 16) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] += (double)p[(i + 4 * k) * ncols + col];
    }
    for (; i < hi; i += 4) s[0] += (double)p[i * ncols + col];
  }
  sh[wave][lane] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (wave == 0 && col < ncols)
    out[(long long)blockIdx.y * NCOLS + base + col] = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
}

// Gradient in the parameter layout from the sliced sums and, with lr > 0, the Adam update (Kingma & Ba
// 2015) with bias correction, step counted from 1 (c1 = 1 - beta1^step, c2 = 1 - beta2^step).
__global__ void __launch_bounds__(64) k_grad_adam(const double* __restrict__ red, int slices, float* __restrict__ grad,
                                                  float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
                                                  float lr, float b1, float b2, float eps, float c1, float c2) {
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= NPARAM) return;
  int col;
  if (e < OFF_B1) col = COL3 + COL2 + (e / K1) * (K1P + 1) + e % K1;
  else if (e < OFF_W2) col = COL3 + COL2 + (e - OFF_B1) * (K1P + 1) + K1P;
  else if (e < OFF_B2) col = COL3 + ((e - OFF_W2) / K2) * (K2 + 1) + (e - OFF_W2) % K2;
  else if (e < OFF_W3) col = COL3 + (e - OFF_B2) * (K2 + 1) + K2;
  else col = e - OFF_W3;                                   // W3 (432) then b3 (entry 432)
  double s4[4] = {0.0, 0.0, 0.0, 0.0};                     // four loads in flight
  for (int k = 0; k < slices; k += 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i < slices) s4[i] += red[(long long)(k + i) * NCOLS + col];
  }
  const double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
  const float gr = (float)s;
  grad[e] = gr;
  if (lr > 0.f) {
    const float mm = b1 * m[e] + (1.f - b1) * gr;
    const float vv = b2 * v[e] + (1.f - b2) * gr * gr;
    m[e] = mm;
    v[e] = vv;
    th[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  }
}

// u = Psi . r_hat from the displacement (planar [b][3][N^3]).
__global__ void __launch_bounds__(256) k_radial(const float* __restrict__ psi, Geo3 g, int batch,
                                                float* __restrict__ u) {
  const long long n3 = (long long)g.n * g.n * g.n;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n3 * batch; i += (long long)gridDim.x * 256) {
    const long long c = i % n3;
    const int x = (int)(c % g.n), y = (int)((c / g.n) % g.n), z = (int)(c / ((long long)g.n * g.n));
    const float rx = fmaf(g.hs, (float)x, g.ds[0]), ry = fmaf(g.hs, (float)y, g.ds[1]),
                rz = fmaf(g.hs, (float)z, g.ds[2]);
    const float r2 = rx * rx + ry * ry + rz * rz;
    const float ir = r2 > 0.f ? rsqrtf(r2) : 0.f;
    const float* p = psi + 3 * (i - c);
    u[i] = (rx * p[c] + ry * p[n3 + c] + rz * p[2 * n3 + c]) * ir;
  }
}

// Full-weighting restriction of periodic n^3 node fields to (n/2)^3: coarse node J sits on fine
// node 2J, weights 1/4, 1/2, 1/4 per axis on fine nodes 2J-1, 2J, 2J+1.  One thread per coarse
// node restricts NF fields, blockIdx.y = realisation.
template <int NF>
__global__ void __launch_bounds__(256) k_restrict(const float* __restrict__ fa, const float* __restrict__ fb, int n,
                                                  float* __restrict__ ca, float* __restrict__ cb) {
  const int m = n >> 1, msk = n - 1;
  const long long mc = (long long)m * m * m;
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= mc) return;
  const int X = (int)(i % m), Y = (int)((i / m) % m), Z = (int)(i / ((long long)m * m));
  const long long off = (long long)blockIdx.y * n * n * n;
  const float w[3] = {0.25f, 0.5f, 0.25f};
  float acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = 0.f;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const long long z = (2 * Z + c - 1) & msk;
#pragma unroll
    for (int bb = 0; bb < 3; ++bb) {
      const long long row = off + (z * n + ((2 * Y + bb - 1) & msk)) * n;
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const float* src = f == 0 ? fa : fb;
        float r = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) r = fmaf(w[a], src[row + ((2 * X + a - 1) & msk)], r);
        acc[f] = fmaf(w[c] * w[bb], r, acc[f]);
      }
    }
  }
  const long long o = (long long)blockIdx.y * mc + i;
  ca[o] = acc[0];
  if (NF > 1) cb[o] = acc[NF - 1];
}

// The same restriction for n/2 >= 64: a block covers 64 (x) by 4 (y) coarse nodes and marches over
// 16 coarse z planes, so each fine z plane is filtered once in x and y and shared by the two coarse
// planes it feeds (the filtered plane 2Z+1 is carried in registers to the next coarse plane).
template <int NF>
__global__ void __launch_bounds__(256) k_restrict_slab(const float* __restrict__ fa, const float* __restrict__ fb, int n,
                                                       float* __restrict__ ca, float* __restrict__ cb) {
  constexpr int TXW = 64, TYH = 4, ZB = 16;
  const int m = n >> 1, msk = n - 1;
  const int nbx = m / TXW, nby = m / TYH;
  int t = blockIdx.x;
  const int X = (t % nbx) * TXW + (threadIdx.x % TXW);
  t /= nbx;
  const int Y = (t % nby) * TYH + threadIdx.x / TXW;
  const int Z0 = (t / nby) * ZB;
  const long long off = (long long)blockIdx.y * n * n * n, mc = (long long)m * m * m;
  const int xs0 = (2 * X - 1) & msk, xs1 = 2 * X, xs2 = 2 * X + 1;
  const int ys[3] = {(2 * Y - 1) & msk, 2 * Y, 2 * Y + 1};
  auto plane = [&](const float* __restrict__ f, int z) {
    float p = 0.f;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const float* r = f + off + ((long long)z * n + ys[b]) * n;
      const float v = fmaf(0.25f, r[xs0], fmaf(0.5f, r[xs1], 0.25f * r[xs2]));
      p = fmaf(b == 1 ? 0.5f : 0.25f, v, p);
    }
    return p;
  };
  float prev[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) prev[f] = plane(f == 0 ? fa : fb, (2 * Z0 - 1) & msk);
  for (int k = 0; k < ZB; ++k) {
    const int Z = Z0 + k;
    const long long o = (long long)blockIdx.y * mc + ((long long)Z * m + Y) * m + X;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const float* src = f == 0 ? fa : fb;
      const float p0 = plane(src, 2 * Z), p1 = plane(src, 2 * Z + 1);
      const float v = fmaf(0.25f, prev[f], fmaf(0.5f, p0, 0.25f * p1));
      prev[f] = p1;
      (f == 0 ? ca : cb)[o] = v;
    }
  }
}

// Linear prolongation of a periodic (n/2)^3 node field to n^3, times scale: fine node 2J copies
// coarse node J, fine node 2J+1 takes the mean of coarse J and J+1, axis by axis.  One thread per
// coarse node writes its 2 x 2 x 2 block of fine nodes.
__global__ void __launch_bounds__(256) k_prolong(const float* __restrict__ coarse, int n, float scale,
                                                 float* __restrict__ fine) {
  const int m = n >> 1, mm = m - 1;
  const long long mc = (long long)m * m * m;
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= mc) return;
  const int X = (int)(i % m), Y = (int)((i / m) % m), Z = (int)(i / ((long long)m * m));
  const float* c = coarse + (long long)blockIdx.y * mc;
  const int X1 = (X + 1) & mm, Y1 = (Y + 1) & mm, Z1 = (Z + 1) & mm;
  float v[2][2][2];                                   // [z][y][x] corners J, J+1
  const long long zr[2] = {(long long)Z * m, (long long)Z1 * m};
  const int yr[2] = {Y, Y1};
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      const long long r = (zr[a] + yr[bb]) * m;
      v[a][bb][0] = c[r + X];
      v[a][bb][1] = c[r + X1];
    }
  // x, then y, then z halves
  float hx[2][2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      hx[a][bb][0] = v[a][bb][0];
      hx[a][bb][1] = 0.5f * (v[a][bb][0] + v[a][bb][1]);
    }
  float hy[2][2][2];                                  // [z corner][ey][ex]
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int ex = 0; ex < 2; ++ex) {
      hy[a][0][ex] = hx[a][0][ex];
      hy[a][1][ex] = 0.5f * (hx[a][0][ex] + hx[a][1][ex]);
    }
  float* out = fine + (long long)blockIdx.y * n * n * n;
#pragma unroll
  for (int ez = 0; ez < 2; ++ez)
#pragma unroll
    for (int ey = 0; ey < 2; ++ey) {
      float o[2];
#pragma unroll
      for (int ex = 0; ex < 2; ++ex) o[ex] = scale * (ez ? 0.5f * (hy[0][ey][ex] + hy[1][ey][ex]) : hy[0][ey][ex]);
      const long long fi = (((long long)(2 * Z + ez) * n) + (2 * Y + ey)) * n + 2 * X;
      *(float2*)(out + fi) = make_float2(o[0], o[1]);
    }
}

// Linear prolongation twice = trilinear interpolation at four fine nodes per coarse cell: fine node
// 4J + q takes (1 - q/4) of coarse J and q/4 of coarse J+1 per axis (periodic), times scale.  One
// thread per coarse node writes its 4 x 4 x 4 block of fine nodes, one 16-byte row at a time.
__global__ void __launch_bounds__(256) k_prolong4(const float* __restrict__ coarse, int n, float scale,
                                                  float* __restrict__ fine) {
  const int m = n >> 2, mm = m - 1;
  const long long mc = (long long)m * m * m;
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= mc) return;
  const int X = (int)(i % m), Y = (int)((i / m) % m), Z = (int)(i / ((long long)m * m));
  const float* c = coarse + (long long)blockIdx.y * mc;
  const int X1 = (X + 1) & mm, Y1 = (Y + 1) & mm, Z1 = (Z + 1) & mm;
  float v[2][2][2];                                   // [z][y][x] corners J, J+1
  const long long zr[2] = {(long long)Z * m, (long long)Z1 * m};
  const int yr[2] = {Y, Y1};
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      const long long r = (zr[a] + yr[bb]) * m;
      v[a][bb][0] = c[r + X];
      v[a][bb][1] = c[r + X1];
    }
  const float wq[4] = {0.f, 0.25f, 0.5f, 0.75f};
  float* out = fine + (long long)blockIdx.y * n * n * n;
#pragma unroll
  for (int qz = 0; qz < 4; ++qz)
#pragma unroll
    for (int qy = 0; qy < 4; ++qy) {
      float row[2];
#pragma unroll
      for (int ex = 0; ex < 2; ++ex) {
        const float y0 = fmaf(wq[qy], v[0][1][ex] - v[0][0][ex], v[0][0][ex]);
        const float y1 = fmaf(wq[qy], v[1][1][ex] - v[1][0][ex], v[1][0][ex]);
        row[ex] = fmaf(wq[qz], y1 - y0, y0);
      }
      float4 o;
      o.x = scale * row[0];
      o.y = scale * fmaf(0.25f, row[1] - row[0], row[0]);
      o.z = scale * fmaf(0.5f, row[1] - row[0], row[0]);
      o.w = scale * fmaf(0.75f, row[1] - row[0], row[0]);
      const long long fi = (((long long)(4 * Z + qz) * n) + (4 * Y + qy)) * n + 4 * X;
      *(float4*)(out + fi) = o;
    }
}

}  // namespace cnn
}  // namespace recon
