// Device helpers for the reconstruction kernels (gfx950, wave64).
//
// The 3D transforms are built from one block-level primitive: a length-N
// complex FFT of W independent columns, computed by self-sorting Stockham
// passes on register fragments that exchange through an LDS tile (see the
// fragment engine below).  Twiddles come from an FP32 table of exp(-2 pi i m/N)
// rounded once from FP64 on the host and staged into LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "recon_tuning.h"

namespace recon {

constexpr int kThreads = 256;

// Bounds checks of the debug build (-DRECON_DEBUG): an index outside [0, n) of the array it addresses
// is counted in recon_debug_count and the access is skipped; the release build compiles the checks
// out (in_bounds is the constant true).  recon_debug_violations() reads the count.
#ifdef RECON_DEBUG
__device__ unsigned long long recon_debug_count;
__device__ __forceinline__ bool in_bounds(long long i, long long n) {
  if (i >= 0 && i < n) return true;
  atomicAdd(&recon_debug_count, 1ull);
  return false;
}
#else
__device__ __forceinline__ constexpr bool in_bounds(long long, long long) { return true; }
#endif

// Streaming accesses of the transform passes.  Each pass reads and writes its spectra once, and a
// spectrum (539 MB at 512^3) may be far larger than the caches, so the accesses may carry the
// non-temporal hint: RECON_STREAM bit 0 for stores, bit 1 for loads (the staging loads of the z
// passes included); 0 keeps plain accesses.  H is what a kernel uses: stream_of<N>() unless its launch
// chooses (SizeOps::hinted).
template <int N> constexpr int stream_of() { return N <= 64 ? 0 : RECON_STREAM; }
typedef float recon_v2f __attribute__((ext_vector_type(2)));
template <int H>
__device__ __forceinline__ void st_stream(float2* p, float2 v) {
  if constexpr (H & 1) __builtin_nontemporal_store(recon_v2f{v.x, v.y}, reinterpret_cast<recon_v2f*>(p));
  else *p = v;
}
template <int H>
__device__ __forceinline__ float2 ld_stream(const float2* p) {
  if constexpr (H & 2) {
    const recon_v2f t = __builtin_nontemporal_load(reinterpret_cast<const recon_v2f*>(p));
    return make_float2(t.x, t.y);
  } else {
    return *p;
  }
}
// One plane of a spectrum as a buffer: an element is addressed by a lane offset (one VGPR for all of a
// thread's elements) and a wave-uniform one (an SGPR or a constant), where a flat pointer would take two
// VGPRs per element in flight; accesses past the plane's end are dropped by the hardware.
struct PlaneBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ PlaneBuf(const float2* a, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(a), 0, bytes, 0x00027000)) {}
  template <bool HINT>
  __device__ __forceinline__ float2 load(unsigned lane_bytes, unsigned bytes) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 t = __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, bytes, HINT ? 2 : 0);
    return make_float2(__uint_as_float(t[0]), __uint_as_float(t[1]));
  }
  template <bool HINT>
  __device__ __forceinline__ void store(float2 v, unsigned lane_bytes, unsigned bytes) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u2{__float_as_uint(v.x), __float_as_uint(v.y)}, r, lane_bytes, bytes,
                                          HINT ? 2 : 0);
  }
};


__host__ __device__ constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }

__device__ __forceinline__ float2 operator+(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 operator-(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 operator*(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }
// i * a
__device__ __forceinline__ float2 mul_i(float2 a) { return make_float2(-a.y, a.x); }

// Multiply by the quarter-turn root: -i for the forward transform, +i for the inverse.
template <bool INV>
__device__ __forceinline__ float2 quarter(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

template <bool INV>
__device__ __forceinline__ void dft2(float2* v) {
  float2 t = v[0];
  v[0] = t + v[1];
  v[1] = t - v[1];
}

template <bool INV>
__device__ __forceinline__ void dft4(float2& y0, float2& y1, float2& y2, float2& y3) {
  float2 t0 = y0 + y2, t1 = y0 - y2, t2 = y1 + y3, t3 = quarter<INV>(y1 - y3);
  y0 = t0 + t2;
  y2 = t0 - t2;
  y1 = t1 + t3;
  y3 = t1 - t3;
}

template <bool INV>
__device__ __forceinline__ void dft4v(float2* v) { dft4<INV>(v[0], v[1], v[2], v[3]); }

// 8-point DFT, one decimation-in-frequency radix-2 stage followed by two 4-point DFTs.
template <bool INV>
__device__ __forceinline__ void dft8(float2* v) {
  const float r = 0.70710678118654752440f;
  float2 a0 = v[0] + v[4], a1 = v[1] + v[5], a2 = v[2] + v[6], a3 = v[3] + v[7];
  float2 b0 = v[0] - v[4], b1 = v[1] - v[5], b2 = v[2] - v[6], b3 = v[3] - v[7];
  if (INV) {
    b1 = make_float2((b1.x - b1.y) * r, (b1.x + b1.y) * r);
    b3 = make_float2((-b3.x - b3.y) * r, (b3.x - b3.y) * r);
  } else {
    b1 = make_float2((b1.x + b1.y) * r, (b1.y - b1.x) * r);
    b3 = make_float2((b3.y - b3.x) * r, (-b3.x - b3.y) * r);
  }
  b2 = quarter<INV>(b2);
  dft4<INV>(a0, a1, a2, a3);
  dft4<INV>(b0, b1, b2, b3);
  v[0] = a0; v[2] = a1; v[4] = a2; v[6] = a3;
  v[1] = b0; v[3] = b1; v[5] = b2; v[7] = b3;
}

template <int R, bool INV>
__device__ __forceinline__ void dftR(float2* v) {
  if constexpr (R == 2) dft2<INV>(v);
  else if constexpr (R == 4) dft4v<INV>(v);
  else dft8<INV>(v);
}

// ---------------------------------------------------------------------------
// Register-fragment FFT engine.
//
// A tile holds W independent length-N columns.  Each of the (N/8) W fragment
// threads owns one radix-8 butterfly: element r of its fragment v[8] is row
// i = j + r N/8 of column c.  Two thread layouts exist:
//   column-fast (JF = false): c = t % W, j = t / W   (tiles whose columns are contiguous in memory)
//   row-fast    (JF = true):  j = t % (N/8), c = t / (N/8)   (tiles whose rows are contiguous)
// so that global loads and stores in fragment layout are coalesced either way.
// The first radix-8 pass (sub-transform length NS = 1) consumes the fragment from
// registers, the middle passes run LDS to LDS, and the last radix-8 pass
// (NS = N/8) leaves the result in the same fragment layout in registers, so an
// N = 512 transform costs two LDS exchanges.  Radix-2/4 passes (log2 N not a
// multiple of 3) sit in the middle; each fragment thread then handles 8/R of them.
// LDS layouts: column-fast [N][W+1]; row-fast [W][N + N/8] with one pad slot per 8 rows.  In the
// row-fast layout a wave holds one column, so its lanes write rows 8 j + r (first pass) and read
// rows j + (N/8) r: with the pad the first pattern lands on word offsets 18 j, distinct modulo the
// 64 banks over 32 lanes, and the second is contiguous.
// ---------------------------------------------------------------------------
template <int N, int W, bool JF>
struct Lay {
  static constexpr int LDC = W + 1;
  static constexpr int LDJ = N + N / 8;
  static constexpr int SIZE = JF ? W * LDJ : N * LDC;
  static constexpr int NTF = (N / 8) * W;   // fragment threads
  __device__ __forceinline__ static int at(int i, int c) { return JF ? c * LDJ + i + (i >> 3) : i * LDC + c; }
};

// Block size that runs one fragment per thread (at least one wave).
template <int N, int W>
constexpr int frag_threads() { return (N / 8) * W < 64 ? 64 : (N / 8) * W; }

template <int N, int W, int R, bool JF>
__device__ __forceinline__ void bfly_coords(int b, int& c, int& j) {
  if (JF) { j = b % (N / R); c = b / (N / R); }
  else { c = b % W; j = b / W; }
}

// Fragment coordinates of this thread (valid when t < NTF).  Here and below, t is the thread's index among
// those of its tile: the block's own, unless a block holds several tiles; threads with t >= NTF take part in
// the barriers only.
template <int N, int W, bool JF>
__device__ __forceinline__ void frag_coords(int& c, int& j, int t = threadIdx.x) { bfly_coords<N, W, 8, JF>(t, c, j); }

// Generic LDS-to-LDS Stockham pass (radix R, completed sub-transform length NS).
template <int N, int W, int R, int NS, bool INV, bool JF>
__device__ __forceinline__ void lds_pass(float2* buf, const float2* tw, int t = threadIdx.x) {
  using L = Lay<N, W, JF>;
  constexpr int Q = 8 / R;
  float2 v[Q][R];
  if (t < L::NTF) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      int c, j;
      bfly_coords<N, W, R, JF>(t + q * L::NTF, c, j);
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = buf[L::at(j + r * (N / R), c)];
    }
  }
  __syncthreads();
  if (t < L::NTF) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      int c, j;
      bfly_coords<N, W, R, JF>(t + q * L::NTF, c, j);
      const int k = j % NS;
      if constexpr (NS > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) {
          float2 w = tw[r * k * (N / (NS * R))];
          if (INV) w.y = -w.y;
          v[q][r] = cmul(v[q][r], w);
        }
      }
      dftR<R, INV>(v[q]);
      const int idx = (j / NS) * NS * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[L::at(idx + r * NS, c)] = v[q][r];
    }
  }
  __syncthreads();
}

// First radix-8 pass from the register fragment into LDS (preceded by a barrier that
// protects earlier readers of the tile).
template <int N, int W, bool INV, bool JF>
__device__ __forceinline__ void first_pass(float2* v, float2* buf, int t = threadIdx.x) {
  using L = Lay<N, W, JF>;
  __syncthreads();
  if (t < L::NTF) {
    int c, j;
    frag_coords<N, W, JF>(c, j, t);
    dft8<INV>(v);
#pragma unroll
    for (int r = 0; r < 8; ++r) buf[L::at(j * 8 + r, c)] = v[r];
  }
  __syncthreads();
}

// Last radix-8 pass (NS = N/8) from LDS into the register fragment.
template <int N, int W, bool INV, bool JF>
__device__ __forceinline__ void last_pass(float2* v, const float2* buf, const float2* tw, int t = threadIdx.x) {
  using L = Lay<N, W, JF>;
  if (t < L::NTF) {
    int c, j;
    frag_coords<N, W, JF>(c, j, t);
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = buf[L::at(j + r * (N / 8), c)];
#pragma unroll
    for (int r = 1; r < 8; ++r) {
      float2 w = tw[r * j];
      if (INV) w.y = -w.y;
      v[r] = cmul(v[r], w);
    }
    dft8<INV>(v);
  }
}

// Middle passes between NS = 8 and NS = N/8 (factor N/64).  The split of the factor for 512 and
// 1024 is a tuning knob (RECON_MID_512: 0 = 8, 1 = 2 x 4, 2 = 4 x 2; RECON_MID_1024: 0 = 4 x 4,
// 1 = 2 x 8, 2 = 8 x 2), chosen by the autotuner (autotune.py).
template <int N, int W, bool INV, bool JF>
__device__ __forceinline__ void middle_passes(float2* buf, const float2* tw, int t = threadIdx.x) {
  if constexpr (N == 128) lds_pass<N, W, 2, 8, INV, JF>(buf, tw, t);
  else if constexpr (N == 256) lds_pass<N, W, 4, 8, INV, JF>(buf, tw, t);
  else if constexpr (N == 512) {
    if constexpr (RECON_MID_512 == 1) {
      lds_pass<N, W, 2, 8, INV, JF>(buf, tw, t);
      lds_pass<N, W, 4, 16, INV, JF>(buf, tw, t);
    } else if constexpr (RECON_MID_512 == 2) {
      lds_pass<N, W, 4, 8, INV, JF>(buf, tw, t);
      lds_pass<N, W, 2, 32, INV, JF>(buf, tw, t);
    } else {
      lds_pass<N, W, 8, 8, INV, JF>(buf, tw, t);
    }
  } else if constexpr (N == 1024) {
    if constexpr (RECON_MID_1024 == 1) {
      lds_pass<N, W, 2, 8, INV, JF>(buf, tw, t);
      lds_pass<N, W, 8, 16, INV, JF>(buf, tw, t);
    } else if constexpr (RECON_MID_1024 == 2) {
      lds_pass<N, W, 8, 8, INV, JF>(buf, tw, t);
      lds_pass<N, W, 2, 64, INV, JF>(buf, tw, t);
    } else {
      lds_pass<N, W, 4, 8, INV, JF>(buf, tw, t);
      lds_pass<N, W, 4, 32, INV, JF>(buf, tw, t);
    }
  }
}

// ---------------------------------------------------------------------------
// Optional radix-8 stage on the matrix cores with split-bfloat16 compensated products (the
// precision study's DFT-as-GEMM variant; the default transforms are FP32 throughout).
//
// A radix-8 butterfly is the product of the 8-point DFT matrix (in real form, 16 x 16) with the 16
// real inputs of the butterfly after their twiddle factors.  Sixteen butterflies form the 16
// columns of one v_mfma_f32_16x16x16bf16_1k product.  Operands are split into bfloat16 terms,
// x = x_1 + x_2 (+ x_3), x_1 = bf16(x), x_2 = bf16(x - x_1), x_3 = bf16(x - x_1 - x_2), and the
// products whose terms are not both of the smallest order are accumulated in FP32 (TERMS = 2: three
// products, relative error about 2^-16; TERMS = 3: six products, about 2^-24).
// Operand layout: lane l holds A[l%16][4(l/16) + 0..3] and B[4(l/16) + 0..3][l%16]; the result is
// D[4(l/16) + 0..3][l%16].  Lane l therefore feeds complex inputs 2(l/16), 2(l/16) + 1 of butterfly
// l%16 and receives the complex outputs of the same indices.
// ---------------------------------------------------------------------------
typedef short mf_s4 __attribute__((ext_vector_type(4)));
typedef float mf_f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short bf16_rne(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_val(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

// Split four values into TERMS bfloat16 operand vectors.
template <int TERMS>
__device__ __forceinline__ void bf16_split4(const float* x, mf_s4* t) {
  float r[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
  for (int k = 0; k < TERMS; ++k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned short h = bf16_rne(r[i]);
      t[k][i] = (short)h;
      r[i] -= bf16_val(h);
    }
  }
}

// Real form of the 8-point DFT, element (m, kk): output (m/2, re|im), input (kk/2, re|im).
template <bool INV>
__device__ __forceinline__ float dft8_real(int m, int kk) {
  const float s = 0.70710678118654752440f;
  const float c8[8] = {1.f, s, 0.f, -s, -1.f, -s, 0.f, s};
  const float s8[8] = {0.f, s, 1.f, s, 0.f, -s, -1.f, -s};
  const int a = ((m >> 1) * (kk >> 1)) & 7;
  const float wr = c8[a], wi = INV ? s8[a] : -s8[a];    // omega^(p r), omega = exp(-+ 2 pi i / 8)
  if ((m & 1) == 0) return (kk & 1) ? -wi : wr;
  return (kk & 1) ? wr : wi;
}

// LDS-to-LDS radix-8 Stockham pass (completed sub-transform length NS) on the matrix cores.  Every
// wave handles the 64 butterflies of its 64 fragment threads, 16 per product.  Needs (N/8) W to be a
// multiple of 64 (whole waves).
template <int N, int W, int NS, bool INV, bool JF, int TERMS>
__device__ __forceinline__ void lds_pass_r8_mfma(float2* buf, const float2* tw) {
  using L = Lay<N, W, JF>;
  static_assert(L::NTF % 64 == 0, "the matrix-core radix-8 pass runs whole waves");
  const int t = threadIdx.x, lane = t & 63, wbase = t - lane, n = lane & 15, q = lane >> 4;
  float x[4][4];
  if (t < L::NTF) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      int c, j;
      bfly_coords<N, W, 8, JF>(wbase + 16 * g + n, c, j);
      const int k = j % NS;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = 2 * q + h;
        float2 v = buf[L::at(j + r * (N / 8), c)];
        if constexpr (NS > 1) {
          float2 w = tw[r * k * (N / (NS * 8))];
          if (INV) w.y = -w.y;
          v = cmul(v, w);
        }
        x[g][2 * h] = v.x;
        x[g][2 * h + 1] = v.y;
      }
    }
  }
  __syncthreads();
  if (t < L::NTF) {
    float a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = dft8_real<INV>(n, 4 * q + i);
    mf_s4 at[TERMS];
    bf16_split4<TERMS>(a, at);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      mf_s4 bt[TERMS];
      bf16_split4<TERMS>(x[g], bt);
      mf_f4 acc = {0.f, 0.f, 0.f, 0.f};
      // smallest products first
      if constexpr (TERMS == 3) {
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(at[1], bt[1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(at[2], bt[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(at[0], bt[2], acc, 0, 0, 0);
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(at[1], bt[0], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(at[0], bt[1], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(at[0], bt[0], acc, 0, 0, 0);
      int c, j;
      bfly_coords<N, W, 8, JF>(wbase + 16 * g + n, c, j);
      const int k = j % NS;
      const int idx = (j / NS) * NS * 8 + k;
      buf[L::at(idx + (2 * q) * NS, c)] = make_float2(acc[0], acc[1]);
      buf[L::at(idx + (2 * q + 1) * NS, c)] = make_float2(acc[2], acc[3]);
    }
  }
  __syncthreads();
}

// Eight values as they are in registers here: nothing is contracted across this point.
__device__ __forceinline__ void hold8(float2* v) {
#pragma unroll
  for (int r = 0; r < 8; ++r) asm volatile("" : "+v"(v[r].x), "+v"(v[r].y));
}

// Length-N FFT of the tile, register fragment in and out.  The caller must place a
// barrier before its next write to the tile.  SPLIT > 0 (N >= 64): the last radix-8 stage runs on
// the matrix cores with SPLIT bfloat16 terms per operand (lds_pass_r8_mfma).
template <int N, int W, bool INV, bool JF, int SPLIT = 0>
__device__ __forceinline__ void fft_rr(float2* v, float2* buf, const float2* tw, int t = threadIdx.x) {
  using L = Lay<N, W, JF>;
  if constexpr (N == 8) {
    // The caller's products are rounded before the transform and its sums after it: with no exchange between
    // them the compiler would contract the two differently in each kernel, and a result would depend on which
    // kernels a pass ran in.
    if (t < L::NTF) {
      hold8(v);
      dft8<INV>(v);
      hold8(v);
    }
  } else if constexpr (N < 64) {
    first_pass<N, W, INV, JF>(v, buf, t);
    lds_pass<N, W, N / 8, 8, INV, JF>(buf, tw, t);
    if (t < L::NTF) {
      int c, j;
      frag_coords<N, W, JF>(c, j, t);
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = buf[L::at(j + r * (N / 8), c)];
    }
  } else if constexpr (SPLIT > 0) {
    first_pass<N, W, INV, JF>(v, buf, t);
    middle_passes<N, W, INV, JF>(buf, tw, t);
    lds_pass_r8_mfma<N, W, N / 8, INV, JF, SPLIT>(buf, tw);
    if (t < L::NTF) {
      int c, j;
      frag_coords<N, W, JF>(c, j, t);
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = buf[L::at(j + r * (N / 8), c)];
    }
  } else {
    first_pass<N, W, INV, JF>(v, buf, t);
    middle_passes<N, W, INV, JF>(buf, tw, t);
    last_pass<N, W, INV, JF>(v, buf, tw, t);
  }
}

// Length-N FFT of the tile, register fragment in, natural order in LDS out (ends with a barrier).
// SPLIT as in fft_rr.
template <int N, int W, bool INV, bool JF, int SPLIT = 0>
__device__ __forceinline__ void fft_rl(float2* v, float2* buf, const float2* tw) {
  using L = Lay<N, W, JF>;
  if constexpr (N == 8) {
    __syncthreads();
    if (threadIdx.x < L::NTF) {
      int c, j;
      frag_coords<N, W, JF>(c, j);
      dft8<INV>(v);
#pragma unroll
      for (int r = 0; r < 8; ++r) buf[L::at(r, c)] = v[r];
    }
    __syncthreads();
  } else if constexpr (N < 64) {
    first_pass<N, W, INV, JF>(v, buf);
    lds_pass<N, W, N / 8, 8, INV, JF>(buf, tw);
  } else {
    first_pass<N, W, INV, JF>(v, buf);
    middle_passes<N, W, INV, JF>(buf, tw);
    if constexpr (SPLIT > 0) lds_pass_r8_mfma<N, W, N / 8, INV, JF, SPLIT>(buf, tw);
    else lds_pass<N, W, 8, N / 8, INV, JF>(buf, tw);
  }
}

// ---------------------------------------------------------------------------
// Column engine for N = 256, 512, 1024: 16 elements per thread, tiles of 16 columns, one LDS exchange.
//
// N = 16 x (16 X), X = N / 256.  Thread (j, c) of the N threads of a tile owns rows j + r N/16 of column
// c, before and after a transform.  First pass: a 16-point DFT in registers, exchanged through LDS to
// position 16 j + r.  Second pass, radix 16 X over positions k + 16 r (k = j mod 16): its factor X runs
// across the lanes 32 (and 16) apart that hold the same k, as radix-2 decimation-in-frequency stages whose
// operands meet by lane swaps, its factor 16 in registers; the outputs fall on rows j + r N/16 again.
// Against the radix-8 engine above (8 elements per thread, two or three exchanges, up to 1024 threads a
// block): half the LDS traffic and barriers, and blocks of 256 or 512 threads, so that at 512^3 two blocks
// share a CU and one's loads and stores run under the other's transforms; at 1024^3 a tile is 16 columns
// (128-byte rows) instead of 8, which alone is worth a factor 1.8 (plain pass 3.28 -> 1.79 ms).
// ---------------------------------------------------------------------------
template <int N>
struct Col {
  static_assert(N == 256 || N == 512 || N == 1024, "column engine sizes");
  static constexpr int W = 16, E = 16, T = N / E, NT = T * W, X = T / 16, LDC = W + 1;
  static constexpr int SIZE = N * LDC + (X == 4 ? 32 : 0);
  // one pad slot per row; at N = 1024 lanes that meet rows 256 or 512 apart are kept on other banks
  __device__ __forceinline__ static int at(int i, int c) {
    return i * LDC + c + (X == 4 ? (((i >> 8) & 1) + (i >> 9)) * 16 : 0);
  }
  // column and first row of this thread
  __device__ __forceinline__ static void coords(int& c, int& j) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    c = t & 15;
    if constexpr (X == 1) j = t >> 4;
    else if constexpr (X == 2) j = 2 * wave + ((lane >> 4) & 1) + 16 * (lane >> 5);
    else j = wave + 16 * ((lane >> 5) + 2 * ((lane >> 4) & 1));
  }
};

// a exp(-+2 pi i M / 32), compile-time M
template <int M, bool INV>
__device__ __forceinline__ float2 rot32(float2 a) {
  constexpr float c[9] = {1.f, 0.98078528040323044913f, 0.92387953251128675613f, 0.83146961230254523708f,
                          0.70710678118654752440f, 0.55557023301960222474f, 0.38268343236508977173f,
                          0.19509032201612826785f, 0.f};
  constexpr int m = M & 31, q = m / 8, k = m % 8;
  if constexpr (k == 4) {
    a = INV ? make_float2((a.x - a.y) * c[4], (a.x + a.y) * c[4]) : make_float2((a.x + a.y) * c[4], (a.y - a.x) * c[4]);
  } else if constexpr (k != 0) {
    a = INV ? make_float2(a.x * c[k] - a.y * c[8 - k], a.x * c[8 - k] + a.y * c[k])
            : make_float2(a.x * c[k] + a.y * c[8 - k], a.y * c[k] - a.x * c[8 - k]);
  }
  if constexpr (q == 1) return quarter<INV>(a);
  else if constexpr (q == 2) return make_float2(-a.x, -a.y);
  else if constexpr (q == 3) return quarter<!INV>(a);
  else return a;
}

// 16-point DFT in natural order: 4 x 4.
template <bool INV>
__device__ __forceinline__ void dft16(float2* v) {
  float2 t[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int b = 0; b < 4; ++b) t[a][b] = v[a + 4 * b];
    dft4<INV>(t[a][0], t[a][1], t[a][2], t[a][3]);
  }
  t[1][1] = rot32<2, INV>(t[1][1]); t[1][2] = rot32<4, INV>(t[1][2]); t[1][3] = rot32<6, INV>(t[1][3]);
  t[2][1] = rot32<4, INV>(t[2][1]); t[2][2] = rot32<8, INV>(t[2][2]); t[2][3] = rot32<12, INV>(t[2][3]);
  t[3][1] = rot32<6, INV>(t[3][1]); t[3][2] = rot32<12, INV>(t[3][2]); t[3][3] = rot32<18, INV>(t[3][3]);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    dft4<INV>(t[0][k], t[1][k], t[2][k], t[3][k]);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[k + 4 * q] = t[q][k];
  }
}

// Exchanges a of the upper lane group with b of the lower one (groups of D = 32 or 16 lanes).
template <int D>
__device__ __forceinline__ void lane_swap(float& a, float& b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 r;
  if constexpr (D == 32) r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  else r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// One decimation-in-frequency radix-2 stage between lanes D apart: the lower lane holds x[r], the upper
// x[r + half] for the same 16 r; afterwards the lower holds the sums, the upper the differences (not yet
// multiplied by their twiddle factors).  Two registers at a time: after a swap each lane holds both
// operands of one of the two butterflies.
template <int D>
__device__ __forceinline__ void cross_stage(float2* v) {
#pragma unroll
  for (int i = 0; i < 16; i += 2) {
    float2 p = v[i], q = v[i + 1];
    lane_swap<D>(p.x, q.x);
    lane_swap<D>(p.y, q.y);
    float2 s = p + q, d = p - q;
    lane_swap<D>(s.x, d.x);
    lane_swap<D>(s.y, d.y);
    v[i] = s;
    v[i + 1] = d;
  }
}

// v[r] *= tw[i0 + r st] (conjugate for the inverse) for r < 16; index 0 is a factor 1
template <bool INV>
__device__ __forceinline__ void twiddle16(float2* v, const float2* tw, int i0, int st) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float2 w = tw[i0 + r * st];
    if (INV) w.y = -w.y;
    v[r] = cmul(v[r], w);
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // few factors in registers at a time
  }
}

// Length-N FFT of the tile's 16 columns, rows j + r N/16 in registers in and out.  Its first barrier
// ends the caller's earlier reads of the tile; the caller places a barrier before its next write to it.
template <int N, bool INV>
__device__ __forceinline__ void col_fft(float2* v, float2* buf, const float2* tw, int c, int j) {
  using G = Col<N>;
  // the lane's indices are taken afresh in every transform: the addresses derived from them (16 table
  // entries a stage) are recomputed instead of being held, and spilled, across the kernel's transforms
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane), "+v"(j));
  const int k = j & 15;
  const int hr = G::X == 1 ? 0 : (G::X == 2 ? lane >> 5 : lane >> 4);   // first of the thread's 16 r, over 16
  __builtin_amdgcn_sched_barrier(0);
  dft16<INV>(v);
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) buf[G::at(16 * j + r, c)] = v[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = buf[G::at(k + 16 * (16 * hr + r), c)];
  __builtin_amdgcn_sched_barrier(0);
  twiddle16<INV>(v, tw, 16 * hr * k, k);
  if constexpr (G::X == 2) {
    cross_stage<32>(v);                        // differences times w_32^r
    twiddle16<INV>(v, tw, 0, (lane >> 5) * (N / 32));
  }
  if constexpr (G::X == 4) {
    // radix 4: the quarter turn between its two stages, then the factors w_64^(r q) of both at once
    const int h1 = lane >> 5, h0 = (lane >> 4) & 1;
    cross_stage<32>(v);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float2 q = quarter<INV>(v[r]);
      v[r] = h1 & h0 ? q : v[r];
    }
    cross_stage<16>(v);
    twiddle16<INV>(v, tw, 0, (h1 + 2 * h0) * (N / 64));
  }
  dft16<INV>(v);
  __builtin_amdgcn_sched_barrier(0);
}

// The same with the result in natural order in the tile (ends with a barrier).
template <int N, bool INV>
__device__ __forceinline__ void col_fft_lds(float2* v, float2* buf, const float2* tw, int c, int j) {
  col_fft<N, INV>(v, buf, tw, c, j);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) buf[Col<N>::at(j + r * Col<N>::T, c)] = v[r];
  __syncthreads();
}

template <int N, int NT>
__device__ __forceinline__ void stage_twiddles(float2* tw_lds, const float2* __restrict__ tw) {
  for (int i = threadIdx.x; i < N; i += NT) tw_lds[i] = tw[i];
}

// Wavenumber index m in [0, N) -> signed mode m' (Nyquist as -N/2).
template <int N>
__device__ __forceinline__ float signed_mode(int m) { return (float)(m < N / 2 ? m : m - N); }
// Derivative mode: zero at the Nyquist index.
template <int N>
__device__ __forceinline__ float deriv_mode(int m) { return m == N / 2 ? 0.f : signed_mode<N>(m); }

// Deterministic block reduction of two doubles (fixed shuffle tree, then fixed LDS order).
template <int NT>
__device__ __forceinline__ void block_sum2(double a, double b, double* out_a, double* out_b) {
  __shared__ double red[2][NT / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  if (lane == 0) { red[0][wave] = a; red[1][wave] = b; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sa = 0.0, sb = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) { sa += red[0][w]; sb += red[1][w]; }
    *out_a = sa;
    *out_b = sb;
  }
}

}  // namespace recon
