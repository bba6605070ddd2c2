// Kernels of the reconstruction hot path.
//
// Memory layout (per realisation, b-th block of each buffer):
//   real field      [z][y][x]              N^3 float, x fastest
//   int64 grid      [z][y][x]              N^3 int64 (units of 2^-32 weight)
//   spectrum C      [kz][ky][kx]           (N/2+1) N N float2; kz is the halved axis
// Forward 3D transforms run z (real-to-complex, two real columns packed per
// complex column), then y, then x; inverse transforms run x, y, z.  Every
// k-space multiplier is applied inside the pass where its wavenumber index is
// known, so the fan-out Psi_j = i k'_j P and the fan-in div = sum_j i k'_j V_j
// are staged across passes instead of transforming three fields end to end.
#pragma once

#include "recon_device.hpp"

namespace recon {

// Geometry and physics constants shared by the transform kernels.
struct Geo {
  float kf;          // fundamental wavenumber 2 pi / L
  float hs;          // cell size divided by the line-of-sight scale R0 (a power of two)
  float ds[3];       // (box origin - observer) / R0, per axis
  float growth;      // f
  float inv_bn3;     // 1 / (b N^3): Zel'dovich solve including the inverse-transform factor
  float smooth_c;    // R^2 / 2
  float inv_n3;      // 1 / N^3
  float start_scale; // u_0 = start_scale * u_p for the FFTA starts
};

// Per-realisation scalars of the overdensity step.
struct DeltaScal {
  float alpha;       // W_g / W_r
  float inv_rhobar;  // N^3 / W_g (mean-density mode)
};

// Cloud-in-cell frame: u = fl32(fl32(x - o) * s), s = fl32(N / L).
struct CicGeo {
  int n;
  float s;
  float o[3];
};

enum ZIterMode { ZI_PLAIN = 0, ZI_FFTA = 1, ZI_LEARNED = 2, ZI_CROSS = 3 };

// The displacement buffer is planar, [b][3][N^3] floats with x fastest (the layout recon_get_psi
// hands out): the final z pass then writes whole 128-byte lines (a tile's 32 consecutive x of one
// component), 12 bytes per node, and the shift reads each component's rows.

// Tile shapes (compile-time tuning knobs from recon_tuning.h): packed z columns, y-pass columns,
// x-pass rows.  A block of the radix-8 engine runs one fragment per thread, (N/8) * tile threads.
constexpr int cmin(int a, int b) { return a < b ? a : b; }
template <int N> constexpr int tile_x() {
  return N == 256 ? RECON_TILE_X_256 : (N == 1024 ? RECON_TILE_X_1024 : RECON_TILE_X);
}
// The z and y passes run on the column engine from 256 on: tiles of 16 columns (packed, in z) and one block
// of N threads per tile, 16 elements each.  Below 256 there is no such engine (its second pass is of radix 16
// and more), and the radix-8 engine with its tile knobs stays, for a single grid and for a batch; so it does for
// the matrix-core variants of the z iteration at every size, with 8 columns at 1024 (more would not fit the LDS).
// Both sides on a batch of eight 256^3 (where the engine gives least; ms): z iteration 0.404 against 0.523, y
// passes 0.412 against 0.440; one 512^3: 0.462 / 0.556 and 0.473 / 0.488; one 1024^3: 6.3 / 8.4 and 4.0 / 5.9.
template <int N> constexpr bool z_col() { return N >= 256; }
template <int N> constexpr int wz() { return z_col<N>() ? 16 : cmin(N / 2, RECON_TILE_Z); }
template <int N, int SPLIT> constexpr int wzs() { return SPLIT > 0 && N >= 1024 ? 8 : wz<N>(); }
template <int N> constexpr int wy() { return N >= 256 ? 16 : cmin(N, RECON_TILE_Y); }
template <int N> constexpr int wx() { return tile_x<N>(); }
// y passes: engine, elements per thread, rows between them
template <int N> constexpr bool y_col() { return N >= 256; }
template <int N> constexpr int y_el() { return y_col<N>() ? 16 : 8; }
template <int N> constexpr int y_st() { return N / y_el<N>(); }
// (the plain y passes at 512: the radix-8 engine, whose 1024-thread blocks put 32 waves on a CU and whose
// transform has no cross-lane stages: two arrays forward / inverse 344 / 307 us against 369 / 354)
template <int N> constexpr bool yp_col() { return y_col<N>() && N != 512; }
// The grids' forward z pass takes the column engine at 1024 (4.5 against 5.9 ms with the radix-8 engine,
// whose tile would be 8 packed columns there) and for two grids of 256 (77 against 90 us).  One grid of 256
// and grids of 512 want the 32 waves per CU of the radix-8 engine's 512- and 1024-thread blocks on their
// 16-byte row segments (47 against 56 us, and 431 against 549 us for two).
template <int N, int NA> constexpr bool zg_col() { return N == 1024 || (N == 256 && NA == 2); }
// Grids up to this size run the y and x steps of a plane in one kernel (k_plane_*).
constexpr int kPlaneN = 64;
// z tiles (one y row, 2 wz consecutive x) and tiles per block of the z iteration
template <int N, int SPLIT = 0> constexpr int ztiles() { return N * (N / (2 * wzs<N, SPLIT>())); }
// (the start and cross modes and the matrix-core radix variants, which hold more live state, take one
// tile per block)
template <int N, int MODE, int SPLIT = 0> constexpr int ztpb() {
  return MODE == ZI_PLAIN && SPLIT == 0 && !z_col<N>() ? cmin(RECON_Z_TPB, ztiles<N>()) : 1;
}


__device__ __forceinline__ long long ceil_div_ll(long long a, long long b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// Fill, deposit, totals, mask
// ---------------------------------------------------------------------------
// (zero_too: one more int to clear, or null)
__global__ void k_fill_u64(unsigned long long* p, long long count, int* zero_too = nullptr) {
  if (zero_too && blockIdx.x == 0 && threadIdx.x == 0) *zero_too = 0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = 0ull;
}

__global__ void k_fill_i32(int* p, long long count, int v) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}

__device__ __forceinline__ int find_realisation(const long long* __restrict__ off, int batch, long long i) {
  int lo = 0, hi = batch - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Integer CIC shares of one object: corner k = (dx, dy, dz) gets floor(W_Q c_k / 2^48) with
// c_k = a_x a_y a_z, a = 2^16 - tau or tau per axis, for the first seven corners, and corner (1,1,1)
// the remainder, so the eight shares add up to W_Q exactly.  For a unit weight (W_Q = 2^32) the share
// is floor(c_k / 2^16); c_k <= 2^48 is formed exactly in FP64 at full rate instead of with 64-bit
// integer products (the same integers either way).
__device__ __forceinline__ void cic_shares(unsigned long long wq, const unsigned long long tau[3],
                                           unsigned long long share[8]) {
  unsigned long long sum = 0;
  if (wq == (1ull << 32)) {
    const double ax[2] = {(double)(65536u - (unsigned)tau[0]), (double)(unsigned)tau[0]};
    const double ay[2] = {(double)(65536u - (unsigned)tau[1]), (double)(unsigned)tau[1]};
    const double az[2] = {(double)(65536u - (unsigned)tau[2]), (double)(unsigned)tau[2]};
#pragma unroll
    for (int cnr = 0; cnr < 7; ++cnr) {
      const double c = ax[cnr & 1] * ay[(cnr >> 1) & 1] * az[cnr >> 2];
      const double f = floor(c * 0x1p-16);
      share[cnr] = f >= 0x1p32 ? (1ull << 32) : (unsigned long long)(unsigned)f;
      sum += share[cnr];
    }
  } else {
#pragma unroll
    for (int cnr = 0; cnr < 7; ++cnr) {
      const int dx = cnr & 1, dy = (cnr >> 1) & 1, dz = cnr >> 2;
      const unsigned long long ax = dx ? tau[0] : 65536ull - tau[0];
      const unsigned long long ay = dy ? tau[1] : 65536ull - tau[1];
      const unsigned long long az = dz ? tau[2] : 65536ull - tau[2];
      const unsigned long long c = ax * ay * az;
      const unsigned long long chi = c >> 24, clo = c & 0xFFFFFFull;
      share[cnr] = (wq * chi + ((wq * clo) >> 24)) >> 24;
      sum += share[cnr];
    }
  }
  share[7] = wq - sum;
}

// The rounded value itself, opaque to the compiler: u = fl(fl(x - o) s) stays one rounding, so the
// fraction t = u - floor(u) is formed from it and never fused into fma(s, x - o, -floor(u)) (which the
// backend otherwise does in some kernels and not in others).  No instruction is emitted.
__device__ __forceinline__ float keep_rounded(float v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Nearest-grid-point deposit in the same fixed point: the whole W_Q goes to node i + 1 when the
// FP32 fraction is at least 1/2, else to node i (per axis, periodic).
__global__ void __launch_bounds__(256) k_paint_ngp(const float* __restrict__ pos, const float* __restrict__ w,
                                                   long long n, const long long* __restrict__ off, int batch,
                                                   unsigned long long* __restrict__ grid, CicGeo g,
                                                   int* __restrict__ err) {
  const long long n3 = (long long)g.n * g.n * g.n;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    bool ok = true;
    float uu[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float d = __fsub_rn(pos[3 * i + a], g.o[a]);
      uu[a] = keep_rounded(__fmul_rn(d, g.s));
      ok = ok && (fabsf(uu[a]) < 1073741824.0f);
    }
    const float wv = w ? w[i] : 1.0f;
    ok = ok && (wv >= 0.0f) && (wv < 64.0f);
    if (!ok) { atomicAdd(err, 1); continue; }
    long long ii[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float fl = floorf(uu[a]);
      const float t = __fsub_rn(uu[a], fl);
      ii[a] = ((int)fl + (t >= 0.5f ? 1 : 0)) & (g.n - 1);
    }
    const unsigned long long wq = w ? (unsigned long long)__double2ll_rn((double)wv * 4294967296.0)
                                    : (1ull << 32);
    const int b = off ? find_realisation(off, batch, i) : 0;
    const long long cell = (ii[2] * g.n + ii[1]) * g.n + ii[0];
    if (wq && in_bounds(cell, n3)) atomicAdd(grid + (long long)b * n3 + cell, wq);
  }
}

// Integer fixed-point CIC deposit.  Seven corners get floor(W_Q c / 2^48) and
// corner (1,1,1) the remainder, so every object deposits exactly W_Q; integer
// atomics make the grid independent of the order of the objects.
__global__ void __launch_bounds__(256) k_paint(const float* __restrict__ pos, const float* __restrict__ w,
                                               long long n, const long long* __restrict__ off, int batch,
                                               unsigned long long* __restrict__ grid, CicGeo g,
                                               int* __restrict__ err) {
  const long long n3 = (long long)g.n * g.n * g.n;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    bool ok = true;
    float uu[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float d = __fsub_rn(pos[3 * i + a], g.o[a]);
      uu[a] = keep_rounded(__fmul_rn(d, g.s));
      ok = ok && (fabsf(uu[a]) < 1073741824.0f);   // false for NaN / inf too
    }
    float wv = w ? w[i] : 1.0f;
    ok = ok && (wv >= 0.0f) && (wv < 64.0f);
    if (!ok) { atomicAdd(err, 1); continue; }
    int ii[3];
    unsigned long long tau[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float fl = floorf(uu[a]);
      float t = __fsub_rn(uu[a], fl);
      tau[a] = (unsigned long long)floorf(t * 65536.0f);
      ii[a] = ((int)fl) & (g.n - 1);
    }
    const unsigned long long wq = w ? (unsigned long long)__double2ll_rn((double)wv * 4294967296.0)
                                    : (1ull << 32);
    const int b = off ? find_realisation(off, batch, i) : 0;
    unsigned long long* gb = grid + (long long)b * n3;
    unsigned long long share[8];
    cic_shares(wq, tau, share);
#pragma unroll
    for (int cnr = 0; cnr < 8; ++cnr) {
      const int dx = cnr & 1, dy = (cnr >> 1) & 1, dz = cnr >> 2;
      const long long ix = (ii[0] + dx) & (g.n - 1);
      const long long iy = (ii[1] + dy) & (g.n - 1);
      const long long iz = (ii[2] + dz) & (g.n - 1);
      const long long cell = (iz * g.n + iy) * g.n + ix;
      if (share[cnr] && in_bounds(cell, n3)) atomicAdd(gb + cell, share[cnr]);
    }
  }
}

// ---------------------------------------------------------------------------
// Brick-binned deposit: objects are counted per BS^3 brick of their base cell,
// scattered into brick order, and each brick is accumulated in LDS before a
// coalesced flush.  Same integer shares as k_paint, so the grid is identical.
// ---------------------------------------------------------------------------
constexpr int kBrick = 16;

// Brick of this block in a launch of one block per brick: each XCD (workgroups are dealt to the 8
// XCDs round robin) takes a contiguous range of bricks, so x-adjacent bricks, which share halo and
// output lines, run together on one L2 (identity when the brick count is not a multiple of 8).
__device__ __forceinline__ long long brick_of_block() {
  const long long nblk = gridDim.x;
  return (nblk & 7) ? (long long)blockIdx.x : (long long)(blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
}
constexpr int kLdsBins = 32768;   // most bins a block histograms in LDS (128 KB)

// Cell coordinate of an object; false for a non-finite / far position or a bad weight.
__device__ __forceinline__ bool cic_locate(float px, float py, float pz, float wv, const CicGeo& g, int ii[3],
                                           unsigned long long tau[3]) {
  const float pp[3] = {px, py, pz};
  float uu[3];
  bool ok = (wv >= 0.0f) && (wv < 64.0f);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float d = __fsub_rn(pp[a], g.o[a]);
    uu[a] = keep_rounded(__fmul_rn(d, g.s));
    ok = ok && (fabsf(uu[a]) < 1073741824.0f);
  }
  if (!ok) return false;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float fl = floorf(uu[a]);
    float t = __fsub_rn(uu[a], fl);
    tau[a] = (unsigned long long)floorf(t * 65536.0f);
    ii[a] = ((int)fl) & (g.n - 1);
  }
  return true;
}

__device__ __forceinline__ long long brick_key(const int ii[3], int n, int b) {
  const int nbs = (n + kBrick - 1) / kBrick;
  return (long long)b * nbs * nbs * nbs + ((long long)(ii[2] / kBrick) * nbs + ii[1] / kBrick) * nbs + ii[0] / kBrick;
}

// Objects handled per loop trip by the deposit and shift loops: their loads are issued together so that
// their latencies overlap (each thread still takes the same objects in the same order).
constexpr int kObjBatch = RECON_OBJ_BATCH;

// Positions and weights of objects i0 + u * stride, u < U; an index at or past hi loads object hi - 1
// instead (in bounds; the caller skips it).  Requires i0 < hi.
template <int U>
__device__ __forceinline__ void load_objects(const float* __restrict__ pos, const float* __restrict__ w, long long i0,
                                             long long stride, long long hi, float px[U], float py[U], float pz[U],
                                             float wv[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    long long i = i0 + (long long)u * stride;
    if (i >= hi) i = hi - 1;
    px[u] = pos[3 * i];
    py[u] = pos[3 * i + 1];
    pz[u] = pos[3 * i + 2];
    wv[u] = w ? w[i] : 1.0f;
  }
}

// Count with a per-block LDS histogram over the bins of the realisation that owns the
// chunk's first object; one global atomic per (block, non-empty bin).  Objects whose bin
// lies outside that window (a chunk crossing realisations) use a direct global atomic.
// The invalid objects of the block go to errblk[block], which the scan adds up; with ordblk (not null),
// ordblk[block] says whether the catalogue is in spatial order (count_near: a quarter of the neighbours or more),
// and *occupied is cleared for the scan, which counts the bricks that hold objects.
// The block's histogram is also stored in bhist[block][bin], so that the scatter,
// which splits the catalogue into the same chunks, need not count again.
// First brick key of the LDS window of the binning block that takes objects [lo, ...): the block's
// realisation when all of its bricks fit (every size up to 512^3); above that, kBins bricks centred
// on the brick of the chunk's first object, inside its realisation, so that a catalogue stored in
// spatial order (a lattice formed plane by plane) keeps each block's objects in its window.  Objects
// outside the window go to global atomics; the count and the scatter take the same window.
template <int kBins>
__device__ __forceinline__ long long bin_window(const float* __restrict__ pos, long long lo,
                                                const long long* __restrict__ off, int batch, const CicGeo& g) {
  const int nbs = (g.n + kBrick - 1) / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const int b = off ? find_realisation(off, batch, lo) : 0;
  const long long rb = (long long)b * per;
  if (per <= kBins) return rb;
  int ii[3];
  unsigned long long tau[3];
  if (!cic_locate(pos[3 * lo], pos[3 * lo + 1], pos[3 * lo + 2], 1.0f, g, ii, tau)) return rb;
  long long base = brick_key(ii, g.n, b) - kBins / 2;
  if (base < rb) base = rb;
  if (base > rb + per - kBins) base = rb + per - kBins;
  return base;
}

// How many neighbours in a catalogue lie in the same or in touching bricks, from the block's first NT objects
// (votes[1] of votes[0]; LDS, zero before; every thread of the block takes part).  Nearly all do where the
// catalogue is stored in spatial order (a lattice plane by plane) or fills a few bricks only, 1 in 28 where it is
// sorted along one axis of 256^3, 1 in 150 in random order there.
template <int NT>
__device__ __forceinline__ void count_near(const float* __restrict__ pos, long long lo, long long hi, const CicGeo& g,
                                           unsigned* votes) {
  const long long i = lo + threadIdx.x;
  int ii[3] = {0, 0, 0};
  unsigned long long tau[3];
  const bool ok = i < hi && cic_locate(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], 1.0f, g, ii, tau);
  bool pair = (threadIdx.x & 63) && ok, near = true;
  pair = __shfl_up((int)ok, 1, 64) && pair;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int k = ii[a] / kBrick, d = k - __shfl_up(k, 1, 64);
    near = near && d >= -1 && d <= 1;
  }
  const int n0 = __popcll(__ballot(pair)), n1 = __popcll(__ballot(pair && near));
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(votes, (unsigned)n0);
    atomicAdd(votes + 1, (unsigned)n1);
  }
}

template <int NT, int kBins>
__global__ void __launch_bounds__(NT) k_bin_count_lds(const float* __restrict__ pos, const float* __restrict__ w,
                                                       long long n, long long chunk,
                                                       const long long* __restrict__ off, int batch, CicGeo g,
                                                       unsigned* __restrict__ counts, int* __restrict__ errblk,
                                                       unsigned* __restrict__ bhist, int* __restrict__ ordblk,
                                                       int* __restrict__ occupied) {
  __shared__ unsigned hist[kBins];
  __shared__ int bad;
  __shared__ unsigned votes[2];
  if (ordblk && blockIdx.x == 0 && threadIdx.x == 0) *occupied = 0;
  const long long lo = blockIdx.x * chunk;
  if (lo >= n) {                                         // (whole block)
    if (threadIdx.x == 0) {
      errblk[blockIdx.x] = 0;
      if (ordblk) ordblk[blockIdx.x] = 0;
    }
    return;
  }
  const long long hi = lo + chunk < n ? lo + chunk : n;
  const int nbs = (g.n + kBrick - 1) / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const long long base = bin_window<kBins>(pos, lo, off, batch, g);
  for (int i = threadIdx.x; i < kBins; i += NT) hist[i] = 0u;
  if (threadIdx.x == 0) bad = 0;
  if (threadIdx.x < 2) votes[threadIdx.x] = 0u;
  __syncthreads();
  if (ordblk) count_near<NT>(pos, lo, hi, g, votes);
  constexpr int U = kObjBatch;
  for (long long i0 = lo + threadIdx.x; i0 < hi; i0 += (long long)NT * U) {
    float px[U], py[U], pz[U], wv[U];
    load_objects<U>(pos, w, i0, NT, hi, px, py, pz, wv);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = i0 + (long long)u * NT;
      if (i >= hi) break;
      int ii[3];
      unsigned long long tau[3];
      if (!cic_locate(px[u], py[u], pz[u], wv[u], g, ii, tau)) {
        atomicAdd(&bad, 1);
        continue;
      }
      const int b = off ? find_realisation(off, batch, i) : 0;
      const long long key = brick_key(ii, g.n, b);
      const long long rel = key - base;
      if (rel >= 0 && rel < kBins) atomicAdd(&hist[rel], 1u);
      else atomicAdd(counts + key, 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    errblk[blockIdx.x] = bad;
    if (ordblk) ordblk[blockIdx.x] = 4 * votes[1] > votes[0] ? 1 : 0;
  }
  const long long nb_total = per * batch;
  for (int i = threadIdx.x; i < kBins; i += NT) {
    const unsigned c = hist[i];
    if (c && base + i < nb_total) atomicAdd(counts + base + i, c);
    bhist[(long long)blockIdx.x * kBins + i] = c;
  }
}

// Scatter into brick order: each block reserves one contiguous slot range per non-empty
// bin of its window, then ranks its objects inside the range with LDS atomics.
template <int NT, int kBins>
__global__ void __launch_bounds__(NT) k_bin_scatter_lds(const float* __restrict__ pos, const float* __restrict__ w,
                                                         long long n, long long chunk,
                                                         const long long* __restrict__ off, int batch, CicGeo g,
                                                         unsigned* __restrict__ cursor, float4* __restrict__ sorted,
                                                         unsigned* __restrict__ slot_of,
                                                         const unsigned* __restrict__ bhist,
                                                         unsigned* __restrict__ counts, long long ncounts) {
  __shared__ unsigned hist[kBins];
  // the counts are used up (the scan has read them): cleared for the next deposit
  for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < ncounts; i += (long long)gridDim.x * NT) counts[i] = 0u;
  const long long lo = blockIdx.x * chunk;
  if (lo >= n) return;
  const long long hi = lo + chunk < n ? lo + chunk : n;
  const int nbs = (g.n + kBrick - 1) / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const long long base = bin_window<kBins>(pos, lo, off, batch, g);
  const long long nb_total = per * batch;
  // the count kernel's histogram of this very chunk
  for (int i = threadIdx.x; i < kBins; i += NT) hist[i] = bhist[(long long)blockIdx.x * kBins + i];
  __syncthreads();
  for (int i = threadIdx.x; i < kBins; i += NT) {
    const unsigned c = hist[i];
    if (c && base + i < nb_total) hist[i] = atomicAdd(cursor + base + i, c);
  }
  __syncthreads();
  constexpr int U = kObjBatch;
  for (long long i0 = lo + threadIdx.x; i0 < hi; i0 += (long long)NT * U) {
    float px[U], py[U], pz[U], wv[U];
    load_objects<U>(pos, w, i0, NT, hi, px, py, pz, wv);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = i0 + (long long)u * NT;
      if (i >= hi) break;
      int ii[3];
      unsigned long long tau[3];
      if (!cic_locate(px[u], py[u], pz[u], wv[u], g, ii, tau)) {
        slot_of[i] = 0xFFFFFFFFu;   // not in the sorted copy
        continue;
      }
      const int b = off ? find_realisation(off, batch, i) : 0;
      const long long key = brick_key(ii, g.n, b);
      const long long rel = key - base;
      const unsigned slot = (rel >= 0 && rel < kBins) ? atomicAdd(&hist[rel], 1u) : atomicAdd(cursor + key, 1u);
      sorted[slot] = make_float4(px[u], py[u], pz[u], wv[u]);
      slot_of[i] = slot;
    }
  }
}

// Totals of runs of 256 * kScanItems counts (only where there are more than kScanDirect of them).
constexpr int kScanItems = 16;
constexpr long long kScanDirect = 65536;
__global__ void __launch_bounds__(256) k_scan_blocks(const unsigned* __restrict__ in, long long n,
                                                     unsigned* __restrict__ bsum) {
  const long long base = (long long)blockIdx.x * 256 * kScanItems;
  unsigned s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    const long long i = base + (long long)k * 256 + threadIdx.x;
    if (i < n) s += in[i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  __shared__ unsigned ws[4];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// Exclusive scan of the counts by one block of 256 threads per run of 256 * kScanItems: out[i] = sum of
// in[0..i) (n + 1 entries; out[n] = total), cursor = copy of out[0..n).  What comes before the run is
// added up by the block itself, from the counts (bsum null; at most kScanDirect of them, a few loads per
// thread) or from the runs' totals.  Each thread scans kScanItems consecutive counts, the threads' sums
// are scanned with lane shuffles: 3 us, where three launches with a 256-wide scan in LDS (16 barriers) for
// every 256 counts took 20 us at any size.
__device__ __forceinline__ void scan_run(const unsigned* __restrict__ in, long long n,
                                         const unsigned* __restrict__ bsum, long long run,
                                         unsigned* __restrict__ out, unsigned* __restrict__ cursor,
                                         int* __restrict__ occupied) {
  __shared__ unsigned ws[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long first = run * 256 * kScanItems;
  unsigned before = 0;
  if (bsum) {
    for (long long i = threadIdx.x; i < run; i += 256) before += bsum[i];
  } else {
    for (long long i = threadIdx.x; i < first; i += 256) before += in[i];
  }
  const long long i0 = first + (long long)threadIdx.x * kScanItems;
  unsigned v[kScanItems], sum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = i0 + k < n ? in[i0 + k] : 0u;
    sum += v[k];
  }
  if (occupied) {                                        // (not null: how many of the counts are not zero)
    int held = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) held += v[k] != 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) held += __shfl_xor(held, o, 64);
    if (lane == 0 && held) atomicAdd(occupied, held);
  }
  unsigned inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  if (lane == 63) { ws[0][wave] = inc; ws[1][wave] = before; }
  __syncthreads();
  unsigned ex = ws[1][0] + ws[1][1] + ws[1][2] + ws[1][3] + inc - sum;
  for (int w = 0; w < wave; ++w) ex += ws[0][w];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (i0 + k < n) {
      out[i0 + k] = ex;
      cursor[i0 + k] = ex;
      ex += v[k];
      if (i0 + k == n - 1) out[n] = ex;
    }
  }
}

// Part blockIdx.y of a brick's objects [lo, hi): the launch has gridDim.y blocks per brick, of which a
// brick uses one per `least` objects it holds.  False for a block with no part.
__device__ __forceinline__ bool brick_part(unsigned& lo, unsigned& hi, unsigned least) {
  const unsigned cnt = hi - lo;
  if (cnt == 0) return false;
  if (gridDim.y > 1) {
    unsigned parts = (cnt - 1) / least + 1;
    if (parts > gridDim.y) parts = gridDim.y;
    if (blockIdx.y >= parts) return false;
    const unsigned first = lo;
    lo = first + (unsigned)((unsigned long long)cnt * blockIdx.y / parts);
    hi = first + (unsigned)((unsigned long long)cnt * (blockIdx.y + 1) / parts);
  }
  return true;
}

// One block per brick (or several, brick_part): LDS accumulation of the (BS+1)^3 footprint, then a flush with
// 64-bit atomics (bricks overlap by one cell on their upper faces).  NT threads walk the brick's
// objects side by side (a brick of the survey's randoms holds about 8,700 of them).
// NGP: the whole weight on the nearest node (k_paint_ngp's rule), which lies in the same footprint.
template <int NT, bool NGP>
__global__ void __launch_bounds__(NT) k_brick_deposit(const float4* __restrict__ sorted,
                                                      const unsigned* __restrict__ start, CicGeo g,
                                                      unsigned long long* __restrict__ grid, unsigned least) {
  constexpr int T = kBrick + 1;
  __shared__ unsigned long long acc[T * T * T];
  const long long key = brick_of_block();
  unsigned lo = start[key], hi = start[key + 1];
  if (!brick_part(lo, hi, least)) return;
  const int nbs = (g.n + kBrick - 1) / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const int b = (int)(key / per);
  const long long kk = key - (long long)b * per;
  const int bx = (int)(kk % nbs), by = (int)((kk / nbs) % nbs), bz = (int)(kk / ((long long)nbs * nbs));
  for (int i = threadIdx.x; i < T * T * T; i += NT) acc[i] = 0ull;
  __syncthreads();
  constexpr int U = kObjBatch;
  for (long long j0 = (long long)lo + threadIdx.x; j0 < hi; j0 += (long long)NT * U) {
    float4 rr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long j = j0 + (long long)u * NT;
      rr[u] = sorted[j < hi ? j : hi - 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j0 + (long long)u * NT >= hi) break;
      const float4 r = rr[u];
      int ii[3];
      unsigned long long tau[3];
      cic_locate(r.x, r.y, r.z, r.w, g, ii, tau);
      const unsigned long long wq = (unsigned long long)__double2ll_rn((double)r.w * 4294967296.0);
      const int lx = ii[0] - bx * kBrick, ly = ii[1] - by * kBrick, lz = ii[2] - bz * kBrick;
      if constexpr (NGP) {
        // the fraction t is at least 1/2 exactly when floor(2^16 t) is at least 2^15
        const int ux = lx + (tau[0] >= 32768u), uy = ly + (tau[1] >= 32768u), uz = lz + (tau[2] >= 32768u);
        if (wq) atomicAdd(&acc[(uz * T + uy) * T + ux], wq);
        continue;
      }
      unsigned long long share[8];
      cic_shares(wq, tau, share);
#pragma unroll
      for (int cnr = 0; cnr < 8; ++cnr) {
        const int dx = cnr & 1, dy = (cnr >> 1) & 1, dz = cnr >> 2;
        if (share[cnr]) atomicAdd(&acc[((lz + dz) * T + (ly + dy)) * T + (lx + dx)], share[cnr]);
      }
    }
  }
  __syncthreads();
  unsigned long long* gb = grid + (long long)b * g.n * g.n * g.n;
  for (int i = threadIdx.x; i < T * T * T; i += NT) {
    const unsigned long long v = acc[i];
    if (!v) continue;
    const int lx = i % T, ly = (i / T) % T, lz = i / (T * T);
    const long long x = (bx * kBrick + lx) & (g.n - 1), y = (by * kBrick + ly) & (g.n - 1),
                    z = (bz * kBrick + lz) & (g.n - 1);
    const long long cell = ((long long)z * g.n + y) * g.n + x;
    if (in_bounds(cell, (long long)g.n * g.n * g.n)) atomicAdd(gb + cell, v);
  }
}

// Brick-sparse integer grids.  valid[key] (one byte per 16^3 brick) marks the bricks whose cells are
// held in memory; every other brick is zero and is neither cleared nor read.  A deposit through the
// bricks touches brick B when B or one of its seven lower neighbours holds objects (a brick's
// footprint reaches one cell into its upper neighbours).  Modes, one block per brick:
//   0 (new grid):   clear the touched bricks, valid = touched
//   1 (accumulate): clear the touched bricks that are not valid yet, valid |= touched
//   2 (densify):    clear every brick that is not valid, valid = 1 (before a deposit that does not go
//                   through the bricks)
// Requires n to be a multiple of the brick size.
__device__ __forceinline__ void brick_prepare(const unsigned* __restrict__ count, int n, int mode, long long key,
                                              unsigned char* __restrict__ valid,
                                              unsigned long long* __restrict__ grid) {
  const int nbs = n / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const int b = (int)(key / per);
  const long long kk = key - (long long)b * per;
  const int bx = (int)(kk % nbs), by = (int)((kk / nbs) % nbs), bz = (int)(kk / ((long long)nbs * nbs));
  bool touched = true;
  if (mode != 2) {
    touched = false;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      const int x = (bx - (d & 1) + nbs) % nbs, y = (by - ((d >> 1) & 1) + nbs) % nbs,
                z = (bz - (d >> 2) + nbs) % nbs;
      touched = touched || count[(long long)b * per + ((long long)z * nbs + y) * nbs + x] != 0u;
    }
  }
  const bool was = valid[key] != 0;
  __syncthreads();                                       // every thread has read the flag that thread 0 replaces
  const bool clear = mode == 0 ? touched : (mode == 1 ? (touched && !was) : !was);
  if (clear) {
    // 16-byte stores, two cells each (a brick row starts at an even cell, the grid on 16 bytes)
    unsigned long long* gb = grid + (long long)b * n * n * n;
    constexpr int H = kBrick / 2;
    for (int i = threadIdx.x; i < H * kBrick * kBrick; i += 256) {
      const long long x = bx * kBrick + 2 * (i % H), y = by * kBrick + (i / H) % kBrick,
                      z = bz * kBrick + i / (H * kBrick);
      *reinterpret_cast<uint4*>(gb + (z * n + y) * n + x) = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  if (threadIdx.x == 0) valid[key] = (unsigned char)(mode == 0 ? touched : (mode == 1 ? (was || touched) : 1));
}

__global__ void __launch_bounds__(256) k_brick_prepare(const unsigned* __restrict__ count, int n, int mode,
                                                       unsigned char* __restrict__ valid,
                                                       unsigned long long* __restrict__ grid) {
  brick_prepare(count, n, mode, blockIdx.x, valid, grid);
}

// The scan of the brick counts (the first `runs` blocks) and, when valid is given, the preparation of the
// grid's bricks (one block each after those), which both only read the counts, in one launch.
__global__ void __launch_bounds__(256) k_scan_prepare(const unsigned* __restrict__ count, long long nbins,
                                                      const unsigned* __restrict__ bsum, int runs,
                                                      unsigned* __restrict__ out, unsigned* __restrict__ cursor, int n,
                                                      int mode, unsigned char* __restrict__ valid,
                                                      unsigned long long* __restrict__ grid,
                                                      const int* __restrict__ errblk, int nerr, int* __restrict__ err,
                                                      int fresh, const int* __restrict__ ordblk,
                                                      int* __restrict__ order, int* __restrict__ occupied) {
  if (blockIdx.x == 0) {
    // invalid objects of this deposit: replace the grid's count (new grid) or add to it; and whether most of
    // the binning blocks found the catalogue in spatial order
    __shared__ int bad, inorder;
    if (threadIdx.x == 0) bad = inorder = 0;
    __syncthreads();
    int mine = 0, ord = 0;
    for (int i = threadIdx.x; i < nerr; i += 256) {
      mine += errblk[i];
      if (ordblk) ord += ordblk[i];
    }
    if (mine) atomicAdd(&bad, mine);
    if (ord) atomicAdd(&inorder, ord);
    __syncthreads();
    if (threadIdx.x == 0) {
      *err = (fresh ? 0 : *err) + bad;
      if (ordblk) *order = 2 * inorder > nerr ? 1 : 0;
    }
  }
  if ((int)blockIdx.x < runs) scan_run(count, nbins, bsum, blockIdx.x, out, cursor, ordblk ? occupied : nullptr);
  else brick_prepare(count, n, mode, (long long)blockIdx.x - runs, valid, grid);
}

// Validity of the brick holding cell (x, y, z) of realisation b (null: every brick is valid).
__device__ __forceinline__ bool brick_valid(const unsigned char* __restrict__ valid, int n, int b, int x, int y,
                                            int z) {
  if (!valid) return true;
  const int nbs = n / kBrick;
  return valid[(((long long)b * nbs + z / kBrick) * nbs + y / kBrick) * nbs + x / kBrick] != 0;
}

// Dense copy of a brick-sparse grid (zeros in the bricks that are not valid).
__global__ void __launch_bounds__(256) k_grid_export(const long long* __restrict__ grid,
                                                     const unsigned char* __restrict__ valid, int n, int batch,
                                                     long long* __restrict__ out) {
  const long long n3 = (long long)n * n * n, total = n3 * batch;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const int b = (int)(i / n3);
    const long long c = i - b * n3;
    const int x = (int)(c % n), y = (int)((c / n) % n), z = (int)(c / ((long long)n * n));
    out[i] = brick_valid(valid, n, b, x, y, z) ? grid[i] : 0;
  }
}

// Binary survey mask with a sliding window: each wave owns one y row and 64 consecutive x
// (62 outputs plus one halo lane each side); per z it sums the three y rows, adds the two
// x neighbours through lane shuffles, and keeps a running three-plane window along z.
// Sums are exact int64; a cell is inside when the 27-cell sum exceeds thr[b].
__global__ void __launch_bounds__(256) k_mask_win(const long long* __restrict__ gr, int n,
                                                  const long long* __restrict__ thr,
                                                  unsigned char* __restrict__ mask) {
  const int b = blockIdx.y;
  const int nseg = (n + 61) / 62;
  const int seg = blockIdx.x % nseg;
  const int y = (blockIdx.x / nseg) * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (y >= n) return;                                   // whole wave leaves together
  const long long n2 = (long long)n * n;
  const long long* g = gr + (long long)b * n2 * n;
  unsigned char* m = mask + (long long)b * n2 * n;
  const long long t = thr[b];
  const int xs = seg * 62 + lane - 1;                   // may be -1 or >= n: wrapped below
  const int x = xs & (n - 1);
  const long long ym = (long long)((y - 1) & (n - 1)) * n, y0 = (long long)y * n,
                  yp = (long long)((y + 1) & (n - 1)) * n;
  const bool out = lane >= 1 && lane <= 62 && xs < n;
  auto plane = [&](int z) -> long long {
    const long long* gz = g + (long long)z * n2 + x;
    const long long r = gz[ym] + gz[y0] + gz[yp];
    const long long l = __shfl(r, (lane + 63) & 63, 64);
    const long long h = __shfl(r, (lane + 1) & 63, 64);
    return l + r + h;
  };
  const long long first = plane(0);
  long long prev = plane(n - 1), cur = first;
  for (int z = 0; z < n; ++z) {
    const long long next = z + 1 < n ? plane(z + 1) : first;
    if (out) m[(long long)z * n2 + y0 + xs] = (prev + cur + next) > t ? 1 : 0;
    prev = cur;
    cur = next;
  }
}

// The same mask on a brick-sparse random grid, one block per 16^3 brick: the 18^3 neighbourhood is
// staged in LDS (bricks that are not valid read as zero and are not loaded), each thread owns one
// (x, y) column of the brick and keeps the 3 x 3 sums of the 18 planes in registers, then slides
// along z.  A brick whose 27 neighbours are all not valid has every window sum 0.  Bricks are
// taken in XCD ranges (brick_of_block): the one-cell halo reads of x-adjacent bricks and the 16-byte
// pieces of the 128-byte mask lines they write meet in one L2 instead of in HBM.  With mflag (zeroed
// before the launch), a row of the brick with any cell inside the mask sets the flag of its z tile
// (one y row, tw consecutive x, every z; tw a multiple of the brick size).
__global__ void __launch_bounds__(256) k_mask_brick(const long long* __restrict__ gr, int n,
                                                    const long long* __restrict__ thr,
                                                    const unsigned char* __restrict__ valid,
                                                    unsigned char* __restrict__ mask,
                                                    unsigned char* __restrict__ mflag = nullptr, int tw = 0) {
  constexpr int H = kBrick + 2, H3 = H * H * H, PER = (H3 + 255) / 256;
  __shared__ __align__(16) long long h[H3];
  __shared__ int nv[27];
  __shared__ int any;
  const int nbs = n / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const long long key = brick_of_block();
  const int b = (int)(key / per);
  const long long kk = key - (long long)b * per;
  const int bx = (int)(kk % nbs), by = (int)((kk / nbs) % nbs), bz = (int)(kk / ((long long)nbs * nbs));
  const long long n2 = (long long)n * n;
  const long long* g = gr + (long long)b * n2 * n;
  unsigned char* m = mask + (long long)b * n2 * n;
  const long long t = thr[b];
  if (threadIdx.x == 0) any = 0;
  __syncthreads();
  if (threadIdx.x < 27) {
    const int dx = threadIdx.x % 3 - 1, dy = (threadIdx.x / 3) % 3 - 1, dz = threadIdx.x / 9 - 1;
    const int x = (bx + dx + nbs) % nbs, y = (by + dy + nbs) % nbs, z = (bz + dz + nbs) % nbs;
    nv[threadIdx.x] = valid[(long long)b * per + ((long long)z * nbs + y) * nbs + x] != 0;
    if (nv[threadIdx.x]) atomicOr(&any, 1);
  }
  __syncthreads();
  // thread t writes mask row (z, y) = (t / 16, t % 16) of the brick: 16 bytes along x
  const int rz = threadIdx.x / kBrick, ry = threadIdx.x % kBrick;
  uint4* row = (uint4*)(m + (long long)(bz * kBrick + rz) * n2 + (long long)(by * kBrick + ry) * n + bx * kBrick);
  unsigned char* fl = mflag ? mflag + (long long)b * n * (n / tw) + (long long)(by * kBrick + ry) * (n / tw) +
                                    bx * kBrick / tw
                            : nullptr;
  if (!any) {
    const unsigned v = 0 > t ? 0x01010101u : 0u;
    *row = make_uint4(v, v, v, v);
    if (fl && v) *fl = 1;
    return;
  }
  long long vals[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = threadIdx.x + 256 * k;
    vals[k] = 0;
    if (i < H3) {
      const int lx = i % H, ly = (i / H) % H, lz = i / (H * H);
      // neighbour brick of this halo cell: -1, 0 or +1 per axis
      const int ox = lx == 0 ? 0 : (lx == H - 1 ? 2 : 1), oy = ly == 0 ? 0 : (ly == H - 1 ? 2 : 1),
                oz = lz == 0 ? 0 : (lz == H - 1 ? 2 : 1);
      if (nv[(oz * 3 + oy) * 3 + ox]) {
        const long long x = (bx * kBrick + lx - 1 + n) & (n - 1), y = (by * kBrick + ly - 1 + n) & (n - 1),
                        z = (bz * kBrick + lz - 1 + n) & (n - 1);
        vals[k] = g[z * n2 + y * n + x];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (threadIdx.x + 256 * k < H3) h[threadIdx.x + 256 * k] = vals[k];
  __syncthreads();
  // thread (tx, ty) owns one (x, y) column: 3 x 3 sums of the 18 planes, then the z window
  const int tx = threadIdx.x % kBrick, ty = threadIdx.x / kBrick;
  long long sxy[H];
#pragma unroll
  for (int lz = 0; lz < H; ++lz) {
    long long a = 0;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) a += h[(lz * H + ty + dy) * H + tx + dx];
    sxy[lz] = a;
  }
  __syncthreads();                                       // h is reused for the mask bytes below
  unsigned char* mb = (unsigned char*)h;                 // [z][y][x], 16^3 bytes
#pragma unroll
  for (int z = 0; z < kBrick; ++z)
    mb[(z * kBrick + ty) * kBrick + tx] = (sxy[z] + sxy[z + 1] + sxy[z + 2]) > t ? 1 : 0;
  __syncthreads();
  const uint4 w4 = ((const uint4*)mb)[threadIdx.x];
  *row = w4;
  if (fl && (w4.x | w4.y | w4.z | w4.w)) *fl = 1;      // every writer stores the same value
}

constexpr int kOrderAt = 4, kOccupiedAt = 6;
// Per-realisation scalars from the exact totals {W_g, W_r, n_occ}:
//   alpha = W_g / W_r, 1/rho_bar = N^3 / (W_g 2^-32), mask threshold floor(tau 27 W_r / n_occ);
// status[b] bit 0: galaxy total is zero, bit 1: random total is zero.  err: invalid objects of the two grids
// and of their last deposits, from err[kOrderAt] whether in spatial order and from err[kOccupiedAt] the bricks
// with objects.  host (pinned host memory, or null): these six, then the status of every realisation.
// One block per realisation: sums the per-tile integer partials (exact, any order), then derives
// the scalars; tot[b] keeps the totals.
__global__ void __launch_bounds__(256) k_scalars(const unsigned long long* __restrict__ tpart, int nblk, long long n3,
                                                 double tau, int randoms, unsigned long long* __restrict__ tot,
                                                 DeltaScal* __restrict__ sc, long long* __restrict__ thr,
                                                 int* __restrict__ status, const int* __restrict__ err,
                                                 double* __restrict__ host) {
  const int b = blockIdx.x;
  unsigned long long acc[3] = {0ull, 0ull, 0ull};
  for (int i = threadIdx.x; i < nblk; i += 256) {
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[k] += tpart[3 * ((long long)b * nblk + i) + k];
  }
  __shared__ unsigned long long red[3][4];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) red[k][threadIdx.x >> 6] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const long long wg = (long long)(red[0][0] + red[0][1] + red[0][2] + red[0][3]);
    const long long wr = (long long)(red[1][0] + red[1][1] + red[1][2] + red[1][3]);
    const long long occ = (long long)(red[2][0] + red[2][1] + red[2][2] + red[2][3]);
    tot[3 * b] = (unsigned long long)wg;
    tot[3 * b + 1] = (unsigned long long)wr;
    tot[3 * b + 2] = (unsigned long long)occ;
    int st = 0;
    DeltaScal d;
    d.inv_rhobar = wg > 0 ? (float)((double)n3 / ((double)wg * 2.3283064365386963e-10)) : 0.f;
    d.alpha = 0.f;
    long long th = 0;
    if (wg <= 0) st |= 1;
    if (randoms) {
      if (wr <= 0 || occ <= 0) st |= 2;
      else {
        d.alpha = (float)((double)wg / (double)wr);
        th = (long long)floor(tau * 27.0 * (double)wr / (double)occ);
      }
    }
    sc[b] = d;
    thr[b] = th;
    status[b] = st;
    if (host) {
      host[6 + b] = (double)st;
      if (b == 0) {
        for (int k = 0; k < 2; ++k) {
          host[k] = (double)err[k];
          host[2 + k] = (double)err[kOrderAt + k];
          host[4 + k] = (double)err[kOccupiedAt + k];
        }
      }
    }
  }
}

// Mask-tile flags: mflag[b][tile] = 1 when any cell of z tile `tile` (one y row, tw consecutive x,
// every z) lies inside the survey mask.  One block per tile; 16-byte words when the tile row is a
// multiple of 16 bytes, bytes otherwise.
__global__ void __launch_bounds__(256) k_mask_tiles(const unsigned char* __restrict__ mask, int n, int tw,
                                                    unsigned char* __restrict__ mflag) {
  const long long n3 = (long long)n * n * n;
  const int b = blockIdx.y, tpr = n / tw;
  const int y = blockIdx.x / tpr, x0 = (blockIdx.x % tpr) * tw;
  const unsigned char* m = mask + b * n3;
  int mine = 0;
  if (tw % 16 == 0) {
    const int row16 = tw / 16;
    for (int i = threadIdx.x; i < n * row16; i += 256) {
      const long long e = ((long long)(i / row16) * n + y) * n + x0 + 16 * (i % row16);
      if (in_bounds(e + 15, n3)) {
        const uint4 w4 = *(const uint4*)(m + e);
        mine |= (w4.x | w4.y | w4.z | w4.w) != 0u;
      }
    }
  } else {
    for (int i = threadIdx.x; i < n * tw; i += 256) {
      const long long e = ((long long)(i / tw) * n + y) * n + x0 + i % tw;
      if (in_bounds(e, n3)) mine |= m[e] != 0;
    }
  }
  mine = __syncthreads_or(mine);
  if (threadIdx.x == 0) mflag[(long long)b * gridDim.x + blockIdx.x] = mine ? 1 : 0;
}

// ---------------------------------------------------------------------------
// z passes (real <-> half spectrum along z, two real columns packed per complex
// column).  Tile: one y row and 2*WP consecutive x; fragment threads are column-fast
// over the WP packed columns.
// ---------------------------------------------------------------------------
template <int N, int WP>
__device__ __forceinline__ void z_tile_at(int tile, int& y, int& x0) {
  constexpr int TPR = N / (2 * WP);
  y = tile / TPR;
  x0 = (tile % TPR) * 2 * WP;
}

template <int N, int WP>
__device__ __forceinline__ void z_tile_coords(int& y, int& x0) { z_tile_at<N, WP>(blockIdx.x, y, x0); }

// Packed full-length column element k of the half spectra A (column x0+c) and B
// (column x0+c+WP): Z(k) = A(k) + i B(k), extended Hermitian-wise for k > N/2; the
// imaginary parts at k = 0 and N/2 are dropped as for a real inverse transform.
template <int N, int WP>
__device__ __forceinline__ void z_pack_frag(float2* v, const float2* __restrict__ a, int y, int x0, int c, int j) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int k = j + r * (N / 8);
    const int m = k <= N / 2 ? k : N - k;
    const long long base = ((long long)m * N + y) * N + x0 + c;
    constexpr long long CN = (long long)(N / 2 + 1) * N * N;
    const float2 A = in_bounds(base, CN) ? a[base] : float2{}, B = in_bounds(base + WP, CN) ? a[base + WP] : float2{};
    if (k == 0 || k == N / 2) v[r] = make_float2(A.x, B.x);
    else if (k < N / 2) v[r] = make_float2(A.x - B.y, A.y + B.x);
    else v[r] = make_float2(A.x + B.y, B.x - A.y);
  }
}

// LDS-direct staging of a z tile: rows kz = 0..N/2 of columns x0 .. x0 + 2 WP - 1 at plane row y
// land in `stage` as [kz][2 WP] float2 without passing through registers, so the loads of the next
// array run while the current one is transformed.  Each lane moves 16 bytes; one wave instruction
// fills one 1 KB chunk (its LDS base is wave-uniform).  Completion: s_waitcnt vmcnt(0), then a barrier.
template <int N, int WP>
struct ZStage {
  static constexpr int ROWB = 2 * WP * 8;             // bytes per kz row
  static constexpr int LPR = ROWB / 16;               // lanes per row
  static constexpr int RPC = 64 / LPR;                // rows per 1 KB chunk
  static constexpr int ROWS = N / 2 + 1;
  static constexpr int NCH = (ROWS + RPC - 1) / RPC;
  static constexpr int SIZE = NCH * 128;              // float2 elements
};

template <int N, int WP, int NT, int H = stream_of<N>()>
__device__ __forceinline__ void z_stage_issue(float2* stage, const float2* __restrict__ a, int y, int x0) {
  using S = ZStage<N, WP>;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int q = wave; q < S::NCH; q += NT / 64) {
    const int m = q * S::RPC + lane / S::LPR;
    const long long e = ((long long)m * N + y) * N + x0 + 2 * (lane % S::LPR);
    if (m < S::ROWS && in_bounds(e + 1, (long long)(N / 2 + 1) * N * N)) {
      const float2* g = a + e;
      __builtin_amdgcn_global_load_lds((const void*)g, (__attribute__((address_space(3))) void*)(stage + q * 128),
                                       16, 0, (H & 2) ? 2 : 0 /* the nt bit */);
    }
  }
}

__device__ __forceinline__ void z_stage_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// z_pack_frag from a staged tile.
template <int N, int WP>
__device__ __forceinline__ void z_pack_stage(float2* v, const float2* stage, int c, int j) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int k = j + r * (N / 8);
    const int m = k <= N / 2 ? k : N - k;
    const float2 A = stage[m * 2 * WP + c], B = stage[m * 2 * WP + c + WP];
    if (k == 0 || k == N / 2) v[r] = make_float2(A.x, B.x);
    else if (k < N / 2) v[r] = make_float2(A.x - B.y, A.y + B.x);
    else v[r] = make_float2(A.x + B.y, B.x - A.y);
  }
}

// Split a transformed packed tile (natural order in LDS) into the half spectra of its
// two real columns and store them.  MULK: multiply by i k'_z.
template <int N, int WP, int NT, bool MULK, int H = stream_of<N>()>
__device__ __forceinline__ void z_unpack_store(const float2* buf, float2* __restrict__ out, int y, int x0, float kf) {
  using L = Lay<N, WP, false>;
  for (int e = threadIdx.x; e < (N / 2 + 1) * WP; e += NT) {
    const int p = e % WP, kz = e / WP;
    const float2 Z = buf[L::at(kz, p)];
    const float2 M = buf[L::at((N - kz) & (N - 1), p)];
    float2 A = make_float2(0.5f * (Z.x + M.x), 0.5f * (Z.y - M.y));
    float2 B = make_float2(0.5f * (Z.y + M.y), 0.5f * (M.x - Z.x));
    if (MULK) {
      const float k = kf * deriv_mode<N>(kz);
      A = mul_i(A) * k;
      B = mul_i(B) * k;
    }
    const long long base = ((long long)kz * N + y) * N + x0 + p;
    constexpr long long CN = (long long)(N / 2 + 1) * N * N;
    if (in_bounds(base, CN)) st_stream<H>(out + base, A);
    if (in_bounds(base + WP, CN)) st_stream<H>(out + base + WP, B);
  }
}

// Scaled line-of-sight vector of a node: r = (origin + H i - observer) / R0.
__device__ __forceinline__ float los_comp(const Geo& g, int a, int i) { return fmaf(g.hs, (float)i, g.ds[a]); }
// |r|^2 with a fixed rounding order, so that every z kernel (and every tiling of one) forms the same
// value whatever the compiler hoists or contracts
__device__ __forceinline__ float los_r2(float rx, float ry, float rz) { return fmaf(rz, rz, fmaf(ry, ry, rx * rx)); }

template <int N> constexpr int ntz() { return z_col<N>() ? N : frag_threads<N, wz<N>()>(); }
template <int N, int SPLIT> constexpr int ntzs() { return SPLIT > 0 ? frag_threads<N, wzs<N, SPLIT>()>() : ntz<N>(); }
template <int N> constexpr int nty() { return y_col<N>() ? N : frag_threads<N, wy<N>()>(); }
template <int N> constexpr int ntx() { return frag_threads<N, wx<N>()>(); }

// Column-engine z tile (one y row, 32 consecutive x as 16 packed columns, every z).
template <int N>
struct ZCol {
  using G = Col<N>;
  static constexpr int WP = 16, RT = N / 16, RL = 8;      // rows a load step apart, load steps (kz < N/2)
  // whether column x of row (kz, y) lies in the spectrum (debug build), from its own index: a buffer access
  // that leaves its rows would be dropped without a trace
  __device__ __forceinline__ static bool inside(int kz, int y, int x) {
    return in_bounds(((long long)kz * N + y) * N + x, (long long)(N / 2 + 1) * N * N);
  }
  // half-spectrum rows kz = m + i RT (i < 8) of columns p and p + 16 of an array, and of row N/2 in the
  // first 16 threads: loads that stay in flight while another array is transformed
  struct Half {
    float2 a[RL], b[RL], na, nb;
  };
  // the rows of load step i as a buffer: kz planes lie N^2 elements apart
  __device__ __forceinline__ static PlaneBuf rows(const float2* arr, int kz, int y, int x0) {
    return PlaneBuf(arr + ((long long)kz * N + y) * N + x0, (unsigned)((RT - 1) * N * N + 2 * WP) * 8u);
  }
  __device__ __forceinline__ static unsigned lane() {
    return ((unsigned)(threadIdx.x >> 4) * (unsigned)(N * N) + (threadIdx.x & 15)) * 8u;
  }
  template <int H = stream_of<N>()>
  __device__ __forceinline__ static void fetch(Half& h, const float2* arr, int y, int x0) {
    constexpr bool HINT = (H & 2) != 0;
    const unsigned l = lane();
    const int m0 = threadIdx.x >> 4, x = x0 + (threadIdx.x & 15);
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      const PlaneBuf pb = rows(arr, i * RT, y, x0);
      h.a[i] = inside(m0 + i * RT, y, x) ? pb.template load<HINT>(l, 0) : float2{};
      h.b[i] = inside(m0 + i * RT, y, x + WP) ? pb.template load<HINT>(l, WP * 8) : float2{};
    }
    if (threadIdx.x < 16) {
      const PlaneBuf pb = rows(arr, N / 2, y, x0);
      h.na = inside(N / 2, y, x) ? pb.template load<HINT>(l, 0) : float2{};
      h.nb = inside(N / 2, y, x + WP) ? pb.template load<HINT>(l, WP * 8) : float2{};
    }
  }
  // the packed full-length columns Z = A + i B, extended Hermitian-wise, in natural order in the tile
  // (the imaginary parts at k = 0 and N/2 are dropped as for a real inverse transform)
  __device__ __forceinline__ static void put(const Half& h, float2* buf) {
    const int m0 = threadIdx.x >> 4, p = threadIdx.x & 15;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      const int m = m0 + i * RT;
      const float2 A = h.a[i], B = h.b[i];
      if (i == 0 && m == 0) {
        buf[G::at(0, p)] = make_float2(A.x, B.x);
      } else {
        buf[G::at(m, p)] = make_float2(A.x - B.y, A.y + B.x);
        buf[G::at(N - m, p)] = make_float2(A.x + B.y, B.x - A.y);
      }
    }
    if (threadIdx.x < 16) buf[G::at(N / 2, p)] = make_float2(h.na.x, h.nb.x);
  }
  // this thread's fragment, rows j + r N/16 of column c
  __device__ __forceinline__ static void frag(float2* v, const float2* buf, int c, int j) {
#pragma unroll
    for (int r = 0; r < G::E; ++r) v[r] = buf[G::at(j + r * G::T, c)];
  }
  // Half spectra of the two real columns of each packed column (natural order in the tile) to memory;
  // MULK: times i k'_z.
  template <bool MULK, int H = stream_of<N>()>
  __device__ __forceinline__ static void unpack(const float2* buf, float2* out, int y, int x0, float kf) {
    constexpr bool HINT = (H & 1) != 0;
    const int m0 = threadIdx.x >> 4, p = threadIdx.x & 15;
    const unsigned l = lane();
    auto one = [&](int kz, const PlaneBuf& pb) {
      const float2 Z = buf[G::at(kz, p)], M = buf[G::at((N - kz) & (N - 1), p)];
      float2 A = make_float2(0.5f * (Z.x + M.x), 0.5f * (Z.y - M.y));
      float2 B = make_float2(0.5f * (Z.y + M.y), 0.5f * (M.x - Z.x));
      if (MULK) {
        const float k = kf * deriv_mode<N>(kz);
        A = mul_i(A) * k;
        B = mul_i(B) * k;
      }
      if (inside(kz, y, x0 + p)) pb.template store<HINT>(A, l, 0);
      if (inside(kz, y, x0 + p + WP)) pb.template store<HINT>(B, l, WP * 8);
    };
#pragma unroll
    for (int i = 0; i < RL; ++i) one(m0 + i * RT, rows(out, i * RT, y, x0));
    if (threadIdx.x < 16) one(N / 2, rows(out, N / 2, y, x0));
  }
};

// The column engine's in-flight half spectra (nothing on the radix-8 engine).
struct ZNone {};
template <int N, bool COL = z_col<N>()>
struct ZHalf {
  using type = ZNone;
};
template <int N>
struct ZHalf<N, true> {
  using type = typename ZCol<N>::Half;
};

// Fragment coordinates, transforms and stores of a z tile, on the engine of its size (COL: the column
// engine; the tile is the same on both from 256 on).
template <int N, bool COL = z_col<N>()>
struct ZTile {
  static constexpr int WP = wz<N>(), NT = COL ? N : frag_threads<N, WP>(), E = COL ? 16 : 8, ST = N / E;
  static constexpr int SIZE = [] {
    if constexpr (COL) return Col<N>::SIZE;
    else return Lay<N, WP, false>::SIZE;
  }();
  __device__ __forceinline__ static void coords(int& c, int& j) {
    if constexpr (COL) Col<N>::coords(c, j);
    else frag_coords<N, WP, false>(c, j);
  }
  __device__ __forceinline__ static bool active() { return COL || threadIdx.x < Lay<N, WP, false>::NTF; }
  template <bool INV>
  __device__ __forceinline__ static void fft(float2* v, float2* buf, const float2* tw, int c, int j) {
    if constexpr (COL) col_fft<N, INV>(v, buf, tw, c, j);
    else fft_rr<N, WP, INV, false>(v, buf, tw);
  }
  template <bool INV>
  __device__ __forceinline__ static void fft_lds(float2* v, float2* buf, const float2* tw, int c, int j) {
    if constexpr (COL) col_fft_lds<N, INV>(v, buf, tw, c, j);
    else fft_rl<N, WP, INV, false>(v, buf, tw);
  }
  template <bool MULK>
  __device__ __forceinline__ static void unpack(const float2* buf, float2* out, int y, int x0, float kf) {
    if constexpr (COL) ZCol<N>::template unpack<MULK>(buf, out, y, x0, kf);
    else z_unpack_store<N, WP, NT, MULK>(buf, out, y, x0, kf);
  }
};

// Rows z = j + r ST of a real field (elements of BYTES bytes, x fastest) at one z tile: element h (0: column
// x0 + c, 1: x0 + c + wz) of row r, addressed as a buffer per r, so that a thread's 2 E elements share one
// lane offset.  skip: the access is dropped (a load gives 0).
template <int N, int BYTES, bool COL = z_col<N>()>
struct ZField {
  static constexpr int ST = ZTile<N, COL>::ST, WP = wz<N>();
  const char* base;
  unsigned lane;
  long long first;                                       // element (r, h) = (0, 0), in the field
  __device__ __forceinline__ ZField(const void* f, int y, int x0, int c, int j)
      : base((const char*)f + ((long long)y * N + x0) * BYTES), lane(((unsigned)j * (unsigned)(N * N) + c) * BYTES),
        first(((long long)j * N + y) * N + x0 + c) {}
  // whether element (r, h) lies in the field (debug build)
  __device__ __forceinline__ bool inside(int r, int h) const {
    return in_bounds(first + (long long)r * ST * N * N + h * WP, (long long)N * N * N);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows(int r) const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base) + (long long)r * ST * N * N * BYTES, 0,
                                             ((unsigned)(ST - 1) * (unsigned)(N * N) + 2 * WP) * BYTES, 0x00027000);
  }
  __device__ __forceinline__ unsigned off(bool skip) const { return skip ? 0x80000000u : lane; }
  __device__ __forceinline__ float load(int r, int h) const {
    if (!inside(r, h)) return 0.f;
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows(r), lane, h * WP * BYTES, 0));
  }
  __device__ __forceinline__ void store(float v, int r, int h) const {
    if (!inside(r, h)) return;
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rows(r), lane, h * WP * BYTES, 0);
  }
  __device__ __forceinline__ unsigned char load_byte(int r, int h) const {
    if (!inside(r, h)) return 0;
    return __builtin_amdgcn_raw_buffer_load_b8(rows(r), lane, h * WP * BYTES, 0);
  }
  __device__ __forceinline__ long long load64(int r, int h, bool skip) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 t = __builtin_amdgcn_raw_buffer_load_b64(rows(r), off(skip || !inside(r, h)), h * WP * BYTES, 0);
    return (long long)(((unsigned long long)t[1] << 32) | t[0]);
  }
};

// (float)q, rounded once as by the plain conversion, without its 64-bit shift by a register: gfx950 reads the
// shift amount wrongly when it sits in the last VGPR of the wave's allocation (seen on a build of the 128^3
// grid pass with 40 VGPRs: v39 read as v0 in some waves), and the compiler does not avoid that register.
// The two words meet in FP64, exact below 2^53; above, the low 12 bits are folded into one sticky bit first,
// far below the 24 bits that remain.
__device__ __forceinline__ float float_of(long long q) {
  const int hi = (int)(q >> 32);
  unsigned lo = (unsigned)q;
  if (hi >= (1 << 21) || hi < -(1 << 21)) lo = (lo & ~0xfffu) | ((lo & 0xfffu) ? 0x800u : 0u);
  return (float)fma((double)hi, 4294967296.0, (double)lo);
}

// Forward z transform of int64 grids (units 2^-32) into half spectra.
// Also writes the exact totals {sum g0, sum g1, #(g1 != 0)} of the tile to tpart[b][block].
// With tile flags (zflag != null, [NA][batch][z tiles]): a tile whose bricks are all not valid gets
// flag 0 and its zero half spectra are not written (the forward y pass reads such rows as zeros);
// every other tile gets flag 1.
template <int N, int NA>
__global__ void __launch_bounds__((ZTile<N, zg_col<N, NA>()>::NT), N < 256 ? 4 : 8) k_z_fwd_grid(const long long* __restrict__ g0,
                                                         const long long* __restrict__ g1, float2* __restrict__ o0,
                                                         float2* __restrict__ o1, unsigned long long* __restrict__ tpart,
                                                         const float2* __restrict__ twg,
                                                         const unsigned char* __restrict__ v0 = nullptr,
                                                         const unsigned char* __restrict__ v1 = nullptr,
                                                         unsigned char* __restrict__ zflag = nullptr) {
  constexpr int NT = ZTile<N, zg_col<N, NA>()>::NT, WP = wz<N>();
  using Z = ZTile<N, zg_col<N, NA>()>;
  __shared__ float2 buf[Z::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int y, x0, c, j;
  z_tile_coords<N, WP>(y, x0);
  Z::coords(c, j);
  const bool act = Z::active();
  const long long n3 = (long long)N * N * N, cn = (long long)(N / 2 + 1) * N * N;
  const int b = blockIdx.y;
  const float unit = 2.3283064365386963e-10f;   // 2^-32
  unsigned long long sums[3] = {0ull, 0ull, 0ull};
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const long long* gsrc = (a == 0 ? g0 : g1) + b * n3;
    // brick-validity of the two columns' bricks along z (brick-sparse grids; null: all valid)
    const unsigned char* vg = a == 0 ? v0 : v1;
    constexpr int NBS = N / kBrick;
    const unsigned char* vb = vg ? vg + (long long)b * NBS * NBS * NBS + (y / kBrick) * NBS : nullptr;
    if (vb) {
      // a tile whose bricks are all not valid holds zeros: its half spectra are zero, no transform
      constexpr int XB = (2 * WP + kBrick - 1) / kBrick;   // bricks across the tile's 2 WP columns
      int mine = 0;
      for (int i = threadIdx.x; i < NBS * XB; i += NT) mine |= vb[(i / XB) * NBS * NBS + x0 / kBrick + i % XB];
      if (!__syncthreads_or(mine)) {
        if (zflag) {
          if (threadIdx.x == 0) zflag[((long long)a * gridDim.y + b) * gridDim.x + blockIdx.x] = 0;
        } else {
          float2* out = (a == 0 ? o0 : o1) + b * cn;
          for (int e = threadIdx.x; e < (N / 2 + 1) * 2 * WP; e += NT)
            out[((long long)(e / (2 * WP)) * N + y) * N + x0 + e % (2 * WP)] = make_float2(0.f, 0.f);
        }
        continue;
      }
    }
    if (zflag && threadIdx.x == 0) zflag[((long long)a * gridDim.y + b) * gridDim.x + blockIdx.x] = 1;
    float2 v[Z::E];
    const ZField<N, 8, zg_col<N, NA>()> fld(gsrc, y, x0, c, j);
    if (act) {
#pragma unroll
      for (int r = 0; r < Z::E; ++r) {
        const int z = j + r * Z::ST;
        const unsigned char* vz = vb ? vb + (z / kBrick) * NBS * NBS : nullptr;
        const bool ok0 = !vz || vz[(x0 + c) / kBrick], ok1 = !vz || vz[(x0 + c + WP) / kBrick];
        const long long q0 = fld.load64(r, 0, !ok0), q1 = fld.load64(r, 1, !ok1);
        sums[a] += (unsigned long long)q0 + (unsigned long long)q1;
        if (a == 1) sums[2] += (q0 != 0) + (q1 != 0);
        v[r] = make_float2(float_of(q0) * unit, float_of(q1) * unit);
      }
    }
    Z::template fft_lds<false>(v, buf, tw, c, j);
    Z::template unpack<false>(buf, (a == 0 ? o0 : o1) + b * cn, y, x0, 0.f);
  }
  __shared__ unsigned long long red[3][NT / 64];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sums[k] += __shfl_xor(sums[k], o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) red[k][threadIdx.x >> 6] = sums[k];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    unsigned long long t = 0;
    for (int w = 0; w < NT / 64; ++w) t += red[threadIdx.x][w];
    tpart[3 * ((long long)b * gridDim.x + blockIdx.x) + threadIdx.x] = t;
  }
}

// Forward z transform of one real field.
template <int N>
__global__ void __launch_bounds__(ntz<N>()) k_z_fwd_real(const float* __restrict__ f, float2* __restrict__ o,
                                                         const float2* __restrict__ twg) {
  constexpr int NT = ntz<N>(), WP = wz<N>();
  using Z = ZTile<N>;
  __shared__ float2 buf[Z::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int y, x0, c, j;
  z_tile_coords<N, WP>(y, x0);
  Z::coords(c, j);
  const long long n3 = (long long)N * N * N, cn = (long long)(N / 2 + 1) * N * N;
  const int b = blockIdx.y;
  f += b * n3;
  float2 v[Z::E];
  const ZField<N, 4> fld(f, y, x0, c, j);
  if (Z::active()) {
#pragma unroll
    for (int r = 0; r < Z::E; ++r) v[r] = make_float2(fld.load(r, 0), fld.load(r, 1));
  }
  Z::template fft_lds<false>(v, buf, tw, c, j);
  Z::template unpack<false>(buf, o + b * cn, y, x0, 0.f);
}

// Inverse z transform of the smoothed galaxy (and random) densities, overdensity in
// configuration space, forward z transform of the overdensity (written over a0).
//   with randoms:  delta = m (G - alpha R) / (alpha R), 0 outside the mask or where R <= 0
//   mean density:  delta = G / rho_bar - 1
template <int N, int NA>
__global__ void __launch_bounds__(ntz<N>(), N == 512 ? 4 : 1) k_z_delta(float2* __restrict__ a0, const float2* __restrict__ a1,
                                                      const unsigned char* __restrict__ mask,
                                                      const DeltaScal* __restrict__ sc, float* __restrict__ delta_out,
                                                      float log_floor, double* __restrict__ partials,
                                                      const float2* __restrict__ twg,
                                                      const unsigned char* __restrict__ mflag = nullptr) {
  constexpr int NT = ntz<N>(), WP = wz<N>();
  using Z = ZTile<N>;
  __shared__ float2 buf[Z::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int y, x0, c, j;
  z_tile_coords<N, WP>(y, x0);
  Z::coords(c, j);
  const bool act = Z::active();
  const long long n3 = (long long)N * N * N, cn = (long long)(N / 2 + 1) * N * N;
  const int b = blockIdx.y;
  a0 += b * cn;
  const DeltaScal s = sc[b];
  double lsum = 0.0;
  float2 gv[Z::E], v[Z::E];
  if constexpr (NA == 2) {
    // a tile outside the survey mask (mask-tile flag 0) has delta_s = 0 in every cell (also after the
    // lognormal transform, ln 1 = 0): its spectrum is zero and no transform is needed; it is not
    // written either (the forward y pass reads such rows as zeros), nor were its inputs (the inverse
    // y pass skipped them).  Without flags every tile is transformed.
    if (mflag && !mflag[(long long)b * gridDim.x + blockIdx.x]) {
      if (delta_out)
        for (int e = threadIdx.x; e < N * 2 * WP; e += NT)
          delta_out[b * n3 + ((long long)(e / (2 * WP)) * N + y) * N + x0 + e % (2 * WP)] = 0.f;
      if (log_floor > 0.f && threadIdx.x == 0) {
        partials[2 * ((long long)b * gridDim.x + blockIdx.x)] = 0.0;
        partials[2 * ((long long)b * gridDim.x + blockIdx.x) + 1] = 0.0;
      }
      return;
    }
    if constexpr (z_col<N>()) {
      // the second array's loads run under the first one's transform
      using C = ZCol<N>;
      typename C::Half h;
      C::fetch(h, a0, y, x0);
      C::put(h, buf);
      C::fetch(h, a1 + b * cn, y, x0);
      __syncthreads();
      C::frag(gv, buf, c, j);
      Z::template fft<true>(gv, buf, tw, c, j);
      __syncthreads();
      C::put(h, buf);
      __syncthreads();
      C::frag(v, buf, c, j);
      Z::template fft<true>(v, buf, tw, c, j);
    } else {
      // the second array is staged in LDS by direct loads while the first is transformed
      __shared__ float2 stage[ZStage<N, WP>::SIZE];
      z_stage_issue<N, WP, NT>(stage, a0, y, x0);
      z_stage_wait();
      __syncthreads();
      if (act) z_pack_stage<N, WP>(gv, stage, c, j);
      __syncthreads();
      z_stage_issue<N, WP, NT>(stage, a1 + b * cn, y, x0);
      fft_rr<N, WP, true, false>(gv, buf, tw);
      z_stage_wait();
      __syncthreads();
      if (act) z_pack_stage<N, WP>(v, stage, c, j);
      fft_rr<N, WP, true, false>(v, buf, tw);
    }
  } else if constexpr (z_col<N>()) {
    using C = ZCol<N>;
    typename C::Half h;
    C::fetch(h, a0, y, x0);
    C::put(h, buf);
    __syncthreads();
    C::frag(gv, buf, c, j);
    Z::template fft<true>(gv, buf, tw, c, j);
  } else {
    if (act) z_pack_frag<N, WP>(gv, a0, y, x0, c, j);
    fft_rr<N, WP, true, false>(gv, buf, tw);
  }
  if (act) {
    const ZField<N, 1> msk(mask + b * n3, y, x0, c, j);
    const ZField<N, 4> dout(delta_out + b * n3, y, x0, c, j);
#pragma unroll
    for (int r = 0; r < Z::E; ++r) {
      float d0, d1;
      if constexpr (NA == 2) {
        const float ar0 = s.alpha * v[r].x, ar1 = s.alpha * v[r].y;
        const bool in0 = (msk.load_byte(r, 0) != 0) & (ar0 > 0.f), in1 = (msk.load_byte(r, 1) != 0) & (ar1 > 0.f);
        const float q0 = (gv[r].x - ar0) / ar0, q1 = (gv[r].y - ar1) / ar1;
        d0 = in0 ? q0 : 0.f;
        d1 = in1 ? q1 : 0.f;
      } else {
        d0 = gv[r].x * s.inv_rhobar - 1.f;
        d1 = gv[r].y * s.inv_rhobar - 1.f;
      }
      if (log_floor > 0.f) {                           // lognormal option: ln(max(1 + delta, floor))
        d0 = logf(fmaxf(1.f + d0, log_floor));
        d1 = logf(fmaxf(1.f + d1, log_floor));
        lsum += (double)d0 + (double)d1;
      }
      v[r] = make_float2(d0, d1);
      if (delta_out) {
        dout.store(d0, r, 0);
        dout.store(d1, r, 1);
      }
      if (z_col<N>() && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (log_floor > 0.f) {
    double t1, t2;
    block_sum2<NT>(lsum, 0.0, &t1, &t2);
    if (threadIdx.x == 0) {
      partials[2 * ((long long)b * gridDim.x + blockIdx.x)] = t1;
      partials[2 * ((long long)b * gridDim.x + blockIdx.x) + 1] = 0.0;
    }
  }
  Z::template fft_lds<false>(v, buf, tw, c, j);
  Z::template unpack<false>(buf, a0, y, x0, 0.f);
}

// Lognormal option: add C = -<ln(max(1 + delta, floor))> (sums[2 b] = sum over the n^3 cells of
// realisation b) to the kept configuration-space field.  Only the k = 0 mode of the spectrum would
// change, and that mode does not enter Psi, so the spectrum is left alone.
__global__ void __launch_bounds__(256) k_log_shift(float* __restrict__ delta, long long n3, int batch,
                                                   const double* __restrict__ sums) {
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n3 * batch; i += (long long)gridDim.x * 256) {
    const long long b = i / n3;
    delta[i] += (float)(-sums[2 * b] / (double)n3);
  }
}

// One iteration's configuration-space step (step A tail + step B head), on the combined fan-out
// state a0 = transverse part r_x Psi_x + r_y Psi_y, a2 = Psi_z (z spectra; r the scaled line of sight):
//   inverse z of both -> s = Psi . r = Z^-1[a0] + r_z Z^-1[a2];  u_p = s / |r|
//   q = u_0 / |r| (V_j = u_0 r_hat_j = q r_j) -> a0 = Z[q], a1 = i k'_z Z[r_z q]
// Start modes (first pass only):
//   ZI_FFTA:    u_0 = start_scale * u_p, Delta = u_0 - u_p stored in corr
//   ZI_LEARNED: u_0 = u_p + corr (corr taken as 0 at the observer), with u_p read from up_in, the
//               start's own inverse z step (the same arithmetic), so no inverse transform is redone
// and both accumulate S1 = sum Delta u_p, S2 = sum Delta^2 into partials.  On the pass after such
// a start, ZI_CROSS iterates as ZI_PLAIN and accumulates S3 = sum Delta u_1 (second entry 0), the
// cross term of ||Psi_1 - Psi_0||^2.
template <int N, int MODE, int SPLIT = 0, int H = stream_of<N>()>
__global__ void __launch_bounds__((ntzs<N, SPLIT>())) k_z_iter(float2* __restrict__ a0, float2* __restrict__ a1,
                                                     const float2* __restrict__ a2, Geo g, float* __restrict__ corr,
                                                     double* __restrict__ partials, const int* __restrict__ active,
                                                     const float2* __restrict__ twg,
                                                     const float* __restrict__ up_in = nullptr) {
  constexpr int NT = ntzs<N, SPLIT>(), WP = wzs<N, SPLIT>(), TPB = ztpb<N, MODE, SPLIT>();
  using L = Lay<N, WP, false>;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[L::SIZE];
  __shared__ float2 tw[N];
  __shared__ float2 stage[ZStage<N, WP>::SIZE];
  stage_twiddles<N, NT>(tw, twg);
  const bool act = threadIdx.x < L::NTF;
  const long long n3 = (long long)N * N * N, cn = (long long)(N / 2 + 1) * N * N;
  a0 += b * cn; a1 += b * cn; a2 += b * cn;
  float acc1 = 0.f, acc2 = 0.f;          // 16 terms per thread and tile; block and grid sums in FP64
  // TPB tiles per block, strided by the grid; the next tile's transverse part is staged in LDS by
  // direct loads while the current tile is finished, and the z component while the transverse
  // part is transformed
  int tile = blockIdx.x, y, x0;
  z_tile_at<N, WP>(tile, y, x0);
  // With RECON_Z_DEFER the second output of a tile (still in the exchange tile after its transform)
  // is stored only after the next tile's first array has been packed, so that the stores drain while
  // the next inverse transform runs instead of delaying the wait for the next tile's staged input;
  // py < 0: nothing deferred
  constexpr bool DEFER = RECON_Z_DEFER && MODE != ZI_LEARNED;
  int py = -1, px0 = 0;
  if (MODE != ZI_LEARNED && tile < (ztiles<N, SPLIT>())) z_stage_issue<N, WP, NT, H>(stage, a0, y, x0);
#pragma unroll 1
  for (int t = 0; t < TPB && tile < (ztiles<N, SPLIT>()); ++t) {     // block-uniform bound
    int c, j;
    frag_coords<N, WP, false>(c, j);
    const float ry = los_comp(g, 1, y);
    const float rx0 = los_comp(g, 0, x0 + c), rx1 = los_comp(g, 0, x0 + c + WP);
    float2 s[8], v[8];
    const int next = tile + gridDim.x;
    int ny = y, nx0 = x0;
    if constexpr (MODE != ZI_LEARNED) {
      z_stage_wait();
      __syncthreads();
      if (act) z_pack_stage<N, WP>(s, stage, c, j);
      __syncthreads();                                // every thread has read the staged tile
      if (DEFER && py >= 0) z_unpack_store<N, WP, NT, true, H>(buf, a1, py, px0, g.kf);
      z_stage_issue<N, WP, NT, H>(stage, a2, y, x0);
      fft_rr<N, WP, true, false, SPLIT>(s, buf, tw);        // (its first barrier ends the reads of buf above)
      z_stage_wait();
      __syncthreads();
      if (act) z_pack_stage<N, WP>(v, stage, c, j);
      if (t + 1 < TPB && next < (ztiles<N, SPLIT>())) {
        __syncthreads();
        z_tile_at<N, WP>(next, ny, nx0);
        z_stage_issue<N, WP, NT, H>(stage, a0, ny, nx0);
      }
      fft_rr<N, WP, true, false, SPLIT>(v, buf, tw);
    }
    // s = Psi . r (two columns packed as .x / .y) -> q = u_0 / |r|, so that V_j = q r_j
    if (act) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int z = j + r * (N / 8);
        const float rz = los_comp(g, 2, z);
        if (MODE != ZI_LEARNED) s[r] = make_float2(fmaf(rz, v[r].x, s[r].x), fmaf(rz, v[r].y, s[r].y));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float rx = h ? rx1 : rx0;
          const float r2 = los_r2(rx, ry, rz);
          const float ir = r2 > 0.f ? rsqrtf(r2) : 0.f;
          const long long cell = b * n3 + ((long long)z * N + y) * N + x0 + c + h * WP;
          // u_p = Psi . r_hat
          const float up = MODE == ZI_LEARNED ? up_in[cell] : (h ? s[r].y : s[r].x) * ir;
          float u0 = up;
          if (MODE != ZI_PLAIN) {
            float dlt;
            if (MODE == ZI_FFTA) {
              u0 = g.start_scale * up;
              dlt = u0 - up;
              corr[cell] = dlt;
            } else if (MODE == ZI_CROSS) {
              dlt = r2 > 0.f ? corr[cell] : 0.f;
            } else {
              dlt = r2 > 0.f ? corr[cell] : 0.f;
              u0 = up + dlt;
            }
            acc1 = fmaf(dlt, up, acc1);
            if (MODE != ZI_CROSS) acc2 = fmaf(dlt, dlt, acc2);
          }
          const float q = u0 * ir;
          if (h) s[r].y = q; else s[r].x = q;
        }
        v[r] = s[r] * rz;
      }
    }
    // Z[q] -> a0 and i k'_z Z[r_z q] -> a1; Z[V_x] = r_x Z[q] and Z[V_y] = r_y Z[q] are formed in
    // the y pass
    fft_rl<N, WP, false, false, SPLIT>(s, buf, tw);
    z_unpack_store<N, WP, NT, false, H>(buf, a0, y, x0, g.kf);
    fft_rl<N, WP, false, false, SPLIT>(v, buf, tw);
    if (DEFER) {
      py = y;
      px0 = x0;
    } else {
      z_unpack_store<N, WP, NT, true, H>(buf, a1, y, x0, g.kf);
    }
    tile = next; y = ny; x0 = nx0;
  }
  if (DEFER && py >= 0) z_unpack_store<N, WP, NT, true, H>(buf, a1, py, px0, g.kf);
  if (MODE != ZI_PLAIN) {
    double t1, t2;
    block_sum2<NT>((double)acc1, (double)acc2, &t1, &t2);
    if (threadIdx.x == 0) {
      const long long nb = gridDim.x;
      partials[2 * (b * nb + blockIdx.x) + 0] = t1;
      partials[2 * (b * nb + blockIdx.x) + 1] = t2;
    }
  }
}

// The z iteration of k_z_iter on the column engine, one tile per block.  It moves 4 spectrum passes (2.15 GB
// at 512^3, 0.34 ms at the chip's streaming rate) and issues 2,985 VALU instructions a wave, 64 waves per SIMD:
// 0.32 of its 0.44 ms.  Both come near what it takes, and a block's chain of loads, four transforms and stores
// runs one after the other, so the blocks are small (N threads) and two or more share a CU, one loading or
// storing while another transforms.  512^3 0.556 -> 0.44 ms (1024-thread blocks of the radix-8 engine with
// wave-local transforms before), 256^3 69 -> 56 us, 1024^3 8.4 -> 6.3 ms.
template <int N, int MODE, int H = stream_of<N>()>
__global__ void __launch_bounds__(N, N == 512 ? 4 : 1) k_z_iter_c(float2* __restrict__ a0, float2* __restrict__ a1,
                                                  const float2* __restrict__ a2, Geo g, float* __restrict__ corr,
                                                  double* __restrict__ partials, const int* __restrict__ active,
                                                  const float2* __restrict__ twg,
                                                  const float* __restrict__ up_in = nullptr) {
  using C = ZCol<N>;
  using G = Col<N>;
  constexpr int WP = C::WP;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[G::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, N>(tw, twg);
  const long long n3 = (long long)N * N * N, cn = (long long)(N / 2 + 1) * N * N;
  a0 += b * cn; a1 += b * cn; a2 += b * cn;
  int y, x0, c, j;
  z_tile_coords<N, WP>(y, x0);
  G::coords(c, j);
  float2 s[16], v[16];
  if constexpr (MODE != ZI_LEARNED) {
    // Psi_z's loads run under the transverse part's transform
    typename C::Half h;
    C::template fetch<H>(h, a0, y, x0);
    C::put(h, buf);
    C::template fetch<H>(h, a2, y, x0);
    __syncthreads();
    C::frag(s, buf, c, j);
    col_fft<N, true>(s, buf, tw, c, j);
    __syncthreads();
    C::put(h, buf);
    __syncthreads();
    C::frag(v, buf, c, j);
    col_fft<N, true>(v, buf, tw, c, j);
  } else {
    __syncthreads();                                    // the twiddle factors
  }
  // s = Psi . r (two columns packed as .x / .y) -> q = u_0 / |r|, so that V_j = q r_j
  float acc1 = 0.f, acc2 = 0.f;          // 16 terms of a thread; everything beyond in FP64
  double sum1 = 0.0, sum2 = 0.0;
  const float ry = los_comp(g, 1, y);
  const float rx0 = los_comp(g, 0, x0 + c), rx1 = los_comp(g, 0, x0 + c + WP);
  const ZField<N, 4> cf(corr + b * n3, y, x0, c, j), uf(up_in + b * n3, y, x0, c, j);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int z = j + r * G::T;
    const float rz = los_comp(g, 2, z);
    if (MODE != ZI_LEARNED) s[r] = make_float2(fmaf(rz, v[r].x, s[r].x), fmaf(rz, v[r].y, s[r].y));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float rx = h ? rx1 : rx0;
      const float r2 = los_r2(rx, ry, rz);
      const float ir = r2 > 0.f ? rsqrtf(r2) : 0.f;
      // u_p = Psi . r_hat
      const float up = MODE == ZI_LEARNED ? uf.load(r, h) : (h ? s[r].y : s[r].x) * ir;
      float u0 = up;
      if (MODE != ZI_PLAIN) {
        float dlt;
        if (MODE == ZI_FFTA) {
          u0 = g.start_scale * up;
          dlt = u0 - up;
          cf.store(dlt, r, h);
        } else {
          const float in = cf.load(r, h);
          dlt = r2 > 0.f ? in : 0.f;
          if (MODE == ZI_LEARNED) u0 = up + dlt;
        }
        acc1 = fmaf(dlt, up, acc1);
        if (MODE != ZI_CROSS) acc2 = fmaf(dlt, dlt, acc2);
      }
      const float q = u0 * ir;
      if (h) s[r].y = q; else s[r].x = q;
    }
    v[r] = s[r] * rz;
    if (MODE != ZI_PLAIN && r % 8 == 7) {
      sum1 += (double)acc1;
      sum2 += (double)acc2;
      acc1 = acc2 = 0.f;
    }
    if (MODE != ZI_PLAIN && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // few loads in flight at a time
  }
  // Z[q] -> a0 and i k'_z Z[r_z q] -> a1
  col_fft_lds<N, false>(s, buf, tw, c, j);
  C::template unpack<false, H>(buf, a0, y, x0, g.kf);
  col_fft_lds<N, false>(v, buf, tw, c, j);
  C::template unpack<true, H>(buf, a1, y, x0, g.kf);
  if (MODE != ZI_PLAIN) {
    double t1, t2;
    block_sum2<N>(sum1, sum2, &t1, &t2);
    if (threadIdx.x == 0) {
      const long long nb = gridDim.x;
      partials[2 * (b * nb + blockIdx.x) + 0] = t1;
      partials[2 * (b * nb + blockIdx.x) + 1] = t2;
    }
  }
}

// Inverse z of the displacement spectra.
//   ZF_PSI:   full state (a0..a2 = Psi_x, Psi_y, Psi_z): writes Psi (planar [b][3][N^3])
//   ZF_CROSS: the same, and the block's partial sum of corr * u with u = Psi . r_hat
//   ZF_U:     combined state (a0 = r_x Psi_x + r_y Psi_y, a2 = Psi_z): writes u to u_out
// One component is transformed and written at a time; only the running Psi . r is held beside it.
enum ZFinalKind { ZF_PSI = 0, ZF_CROSS = 1, ZF_U = 2 };
template <int N, int KIND>
__global__ void __launch_bounds__(ntz<N>(), N == 512 ? 4 : 1) k_z_final(const float2* __restrict__ a0, const float2* __restrict__ a1,
                                                      const float2* __restrict__ a2, Geo g, float* __restrict__ psi,
                                                      float* __restrict__ u_out, const float* __restrict__ corr,
                                                      double* __restrict__ partials, const int* __restrict__ active,
                                                      const float2* __restrict__ twg) {
  constexpr int NT = ntz<N>(), WP = wz<N>();
  using Z = ZTile<N>;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[Z::SIZE];
  __shared__ float2 tw[N];
  __shared__ float2 stage[z_col<N>() ? 1 : ZStage<N, WP>::SIZE];   // radix-8 engine only
  stage_twiddles<N, NT>(tw, twg);
  int y, x0, c, j;
  z_tile_coords<N, WP>(y, x0);
  Z::coords(c, j);
  const bool act = Z::active();
  const long long n3 = (long long)N * N * N, cn = (long long)(N / 2 + 1) * N * N;
  const float2* src[3] = {a0 + b * cn, (KIND == ZF_U ? a2 : a1) + b * cn, a2 + b * cn};
  constexpr int NC = KIND == ZF_U ? 2 : 3;
  const float ry = los_comp(g, 1, y);
  const float rx0 = los_comp(g, 0, x0 + c), rx1 = los_comp(g, 0, x0 + c + WP);
  typename ZHalf<N>::type h;
  if constexpr (z_col<N>()) ZCol<N>::fetch(h, src[0], y, x0);
  else z_stage_issue<N, WP, NT>(stage, src[0], y, x0);
  float2 v[Z::E], s[Z::E];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    // the next array's loads run under this one's transform
    if constexpr (z_col<N>()) {
      if (k) __syncthreads();
      ZCol<N>::put(h, buf);
      if (k + 1 < NC) ZCol<N>::fetch(h, src[k + 1], y, x0);
      __syncthreads();
      ZCol<N>::frag(v, buf, c, j);
    } else {
      z_stage_wait();
      __syncthreads();
      if (act) z_pack_stage<N, WP>(v, stage, c, j);
      __syncthreads();
      if (k + 1 < NC) z_stage_issue<N, WP, NT>(stage, src[k + 1], y, x0);
    }
    Z::template fft<true>(v, buf, tw, c, j);
    if (!act) continue;
    if (KIND != ZF_U) {
      const ZField<N, 4> f(psi + (3 * b + k) * n3, y, x0, c, j);
#pragma unroll
      for (int r = 0; r < Z::E; ++r) {
        f.store(v[r].x, r, 0);
        f.store(v[r].y, r, 1);
      }
    }
    if (KIND == ZF_PSI) continue;
#pragma unroll
    for (int r = 0; r < Z::E; ++r) {
      const float rz = los_comp(g, 2, j + r * Z::ST);
      if (k == 0) s[r] = KIND == ZF_U ? v[r] : make_float2(rx0 * v[r].x, rx1 * v[r].y);
      else if (KIND == ZF_CROSS && k == 1) s[r] = make_float2(fmaf(ry, v[r].x, s[r].x), fmaf(ry, v[r].y, s[r].y));
      else s[r] = make_float2(fmaf(rz, v[r].x, s[r].x), fmaf(rz, v[r].y, s[r].y));
    }
  }
  if (KIND == ZF_PSI) return;
  double acc = 0.0;
  if (act) {
    const ZField<N, 4> f(KIND == ZF_U ? u_out + b * n3 : corr + b * n3, y, x0, c, j);
#pragma unroll
    for (int r = 0; r < Z::E; ++r) {
      const float rz = los_comp(g, 2, j + r * Z::ST);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float r2 = los_r2(q ? rx1 : rx0, ry, rz);
        const float ir = r2 > 0.f ? rsqrtf(r2) : 0.f;
        const float u = (q ? s[r].y : s[r].x) * ir;
        if (KIND == ZF_U) f.store(u, r, q);
        else acc += (double)f.load(r, q) * (double)u;
      }
      if (z_col<N>() && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (KIND == ZF_CROSS) {
    double t1, t2;
    block_sum2<NT>(acc, 0.0, &t1, &t2);
    if (threadIdx.x == 0) {
      partials[2 * ((long long)b * gridDim.x + blockIdx.x)] = t1;
      partials[2 * ((long long)b * gridDim.x + blockIdx.x) + 1] = 0.0;
    }
  }
}

// Radial-ratio diagnostic (Sec. 4, Table 1): per cell q = (Psi_ref . r) / (Psi . r); cells with
// Psi . r != 0 and lo <= q <= hi contribute q and q^2 (FP64 block sums into part[2 blk..]) and
// one count (cnt[blk]).  psi_ref: planar [b][3][n^3]; blockIdx.y = realisation.
template <int NT>
__global__ void __launch_bounds__(NT) k_ratio_stats(const float* __restrict__ psi, const float* __restrict__ psi_ref,
                                                    Geo g, int n, double lo, double hi, double* __restrict__ part,
                                                    unsigned long long* __restrict__ cnt) {
  const long long n3 = (long long)n * n * n;
  const int b = blockIdx.y;
  double s1 = 0.0, s2 = 0.0;
  unsigned long long c = 0;
  for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < n3; i += (long long)gridDim.x * NT) {
    const int x = (int)(i % n), y = (int)((i / n) % n), z = (int)(i / ((long long)n * n));
    const float rx = los_comp(g, 0, x), ry = los_comp(g, 1, y), rz = los_comp(g, 2, z);
    const float* p = psi + b * 3 * n3;
    const float* q = psi_ref + b * 3 * n3;
    const double a = (double)rx * q[i] + (double)ry * q[n3 + i] + (double)rz * q[2 * n3 + i];
    const double d = (double)rx * p[i] + (double)ry * p[n3 + i] + (double)rz * p[2 * n3 + i];
    if (d != 0.0) {
      const double r = a / d;
      if (r >= lo && r <= hi) {
        s1 += r;
        s2 += r * r;
        ++c;
      }
    }
  }
  double t1, t2;
  block_sum2<NT>(s1, s2, &t1, &t2);
  __shared__ unsigned long long cs[NT / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((threadIdx.x & 63) == 0) cs[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tc = 0;
    for (int k = 0; k < NT / 64; ++k) tc += cs[k];
    const long long blk = (long long)b * gridDim.x + blockIdx.x;
    part[2 * blk] = t1;
    part[2 * blk + 1] = t2;
    cnt[blk] = tc;
  }
}

// ---------------------------------------------------------------------------
// y passes.  Tile: one kz plane, W consecutive x, all N rows; column-fast fragments.
// ---------------------------------------------------------------------------
template <int N, int W>
__device__ __forceinline__ void y_tile_coords(int& p, int& x0) {
  p = blockIdx.x / (N / W);
  x0 = (blockIdx.x % (N / W)) * W;
}

// Tile, fragment coordinates and transform of a y pass, on the engine of its size (COL: the column engine;
// the tile is the same on both).
template <int N, bool COL = y_col<N>()>
struct YTile {
  static constexpr int W = wy<N>(), E = COL ? 16 : 8, ST = N / E, NT = COL ? N : frag_threads<N, W>();
  static constexpr int SIZE = [] {
    if constexpr (COL) return Col<N>::SIZE;
    else return Lay<N, W, false>::SIZE;
  }();
  __device__ __forceinline__ static void coords(int& c, int& j) {
    if constexpr (COL) Col<N>::coords(c, j);
    else frag_coords<N, W, false>(c, j);
  }
  __device__ __forceinline__ static bool active() { return COL || threadIdx.x < Lay<N, W, false>::NTF; }
  template <bool INV>
  __device__ __forceinline__ static void fft(float2* v, float2* buf, const float2* tw, int c, int j) {
    if constexpr (COL) col_fft<N, INV>(v, buf, tw, c, j);
    else fft_rr<N, W, INV, false>(v, buf, tw);
  }
};

// Element r of a fragment is row j + r ST of plane p.
template <int N, int H = stream_of<N>()>
__device__ __forceinline__ void y_load(float2* v, const float2* __restrict__ a, int p, int x0, int c, int j) {
  const PlaneBuf pl(a + (long long)p * N * N, (unsigned)N * N * 8);
  const unsigned lane = ((unsigned)j * N + x0 + c) * 8;
#pragma unroll
  for (int r = 0; r < y_el<N>(); ++r)
    v[r] = in_bounds((long long)p * N * N + lane / 8 + r * y_st<N>() * N, (long long)(N / 2 + 1) * N * N)
               ? pl.template load<(H & 2) != 0>(lane, r * y_st<N>() * N * 8)
               : float2{};
}

template <int N, int H = stream_of<N>()>
__device__ __forceinline__ void y_store(const float2* v, float2* __restrict__ a, int p, int x0, int c, int j) {
  const PlaneBuf pl(a + (long long)p * N * N, (unsigned)N * N * 8);
  const unsigned lane = ((unsigned)j * N + x0 + c) * 8;
#pragma unroll
  for (int r = 0; r < y_el<N>(); ++r)
    if (in_bounds((long long)p * N * N + lane / 8 + r * y_st<N>() * N, (long long)(N / 2 + 1) * N * N))
      pl.template store<(H & 1) != 0>(v[r], lane, r * y_st<N>() * N * 8);
}

// Row flags (flag != null): one byte per z tile (one y row, 2 wz consecutive x), [NA][batch][z tiles]
// for the forward pass, [batch][z tiles] shared by both arrays for the inverse one.  Forward: rows
// (y, x) whose z tile has flag 0 were not written by the z pass and are read as zeros.  Inverse:
// such rows are not stored (the z pass that follows does not read them).

template <int N, int NA, bool INV>
__global__ void __launch_bounds__((YTile<N, yp_col<N>()>::NT)) k_y_plain(float2* __restrict__ a0, float2* __restrict__ a1,
                                                      const float2* __restrict__ twg,
                                                      const unsigned char* __restrict__ flag = nullptr) {
  using Y = YTile<N, yp_col<N>()>;
  constexpr int NT = Y::NT, W = Y::W, NZT = N / (2 * wz<N>());
  static_assert((2 * wz<N>()) % W == 0, "a y tile lies inside one z tile");
  constexpr int NF = INV ? 1 : NA;                     // flag sets: per array (forward) or shared (inverse)
  __shared__ float2 buf[Y::SIZE];
  __shared__ float2 tw[N];
  __shared__ unsigned char live[NF][N];                // the tile's row flags, staged with the twiddles
  stage_twiddles<N, NT>(tw, twg);
  int p, x0, c, j;
  y_tile_coords<N, W>(p, x0);
  Y::coords(c, j);
  const bool act = Y::active();
  const long long cn = (long long)(N / 2 + 1) * N * N;
  const int b = blockIdx.y;
  if (flag) {
    for (int i = threadIdx.x; i < NF * N; i += NT) {
      const int f = i / N, yy = i % N;
      live[f][yy] = flag[((long long)f * gridDim.y + b) * N * NZT + (long long)yy * NZT + x0 / (2 * wz<N>())];
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const PlaneBuf pl((a == 0 ? a0 : a1) + b * cn + (long long)p * N * N, (unsigned)N * N * 8);
    const unsigned char* lv = live[INV ? 0 : a];
    const unsigned lane = ((unsigned)j * N + x0 + c) * 8;
    // a row that is not live is read as zero (forward) or not stored (inverse): its lane offset lies past
    // the plane's end
    auto at = [&](int r, bool skip) {
      const bool out = (skip && flag && !lv[j + r * Y::ST]) ||
                       !in_bounds((long long)p * N * N + lane / 8 + r * Y::ST * N, cn);
      return out ? 0x80000000u : lane;
    };
    float2 v[Y::E];
    if (act) {
#pragma unroll
      for (int r = 0; r < Y::E; ++r) v[r] = pl.template load<(stream_of<N>() & 2) != 0>(at(r, !INV), r * Y::ST * N * 8);
    }
    Y::template fft<INV>(v, buf, tw, c, j);
    if (act) {
#pragma unroll
      for (int r = 0; r < Y::E; ++r) pl.template store<(stream_of<N>() & 1) != 0>(v[r], at(r, INV), r * Y::ST * N * 8);
    }
  }
}

// Inverse y with the displacement fan-out.  Full form (COMB = false), the three displacement
// components for the output:
//   a0 <- Y^-1[a0]                    (x component, i k'_x applied in the x pass)
//   a1 <- Y^-1[i k'_y a1]             (y component)
//   a2 <- i k'_z Y^-1[a1]             (z component)
// Combined form (COMB = true), what the z iteration needs: the scaled line-of-sight components r_x
// and r_y are constant along a z column, so the transverse part of Psi . r is formed here, before
// the z transform:
//   a0 <- r_x Y^-1[a0] + r_y Y^-1[i k'_y a1],   a2 <- i k'_z Y^-1[a1]   (a1 is left as it was)
template <int N, bool COMB, int H = stream_of<N>()>
__global__ void __launch_bounds__(nty<N>(), N == 512 ? 4 : 1) k_y_fanout(float2* __restrict__ a0, float2* __restrict__ a1,
                                                       float2* __restrict__ a2, Geo g, const int* __restrict__ active,
                                                       const float2* __restrict__ twg) {
  constexpr int NT = nty<N>(), W = wy<N>();
  using Y = YTile<N>;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[Y::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int p, x0, c, j;
  y_tile_coords<N, W>(p, x0);
  Y::coords(c, j);
  const bool act = Y::active();
  const long long cn = (long long)(N / 2 + 1) * N * N;
  a0 += b * cn; a1 += b * cn; a2 += b * cn;
  // a1 first: once its z component is stored only w is live, so a0 is loaded while w is transformed
  // and no transform runs with more than two arrays live (a third would not fit the registers)
  float2 v[Y::E], w[Y::E];
  {
    float2 keep[Y::E];
    if (act) {
      y_load<N, H>(keep, a1, p, x0, c, j);
#pragma unroll
      for (int r = 0; r < Y::E; ++r) w[r] = mul_i(keep[r]) * (g.kf * deriv_mode<N>(j + r * Y::ST));
    }
    Y::template fft<true>(keep, buf, tw, c, j);
    if (act) {
      const float kz = g.kf * deriv_mode<N>(p);     // p in [0, N/2]; N/2 is the Nyquist plane
#pragma unroll
      for (int r = 0; r < Y::E; ++r) keep[r] = mul_i(keep[r]) * kz;
      y_store<N, H>(keep, a2, p, x0, c, j);
      y_load<N, H>(v, a0, p, x0, c, j);               // in flight during the transform of w
    }
  }
  Y::template fft<true>(w, buf, tw, c, j);
  if (!COMB && act) y_store<N, H>(w, a1, p, x0, c, j);
  Y::template fft<true>(v, buf, tw, c, j);
  if (act) {
    if (COMB) {
      const float rx = los_comp(g, 0, x0 + c);
#pragma unroll
      for (int r = 0; r < Y::E; ++r) {
        const float ry = los_comp(g, 1, j + r * Y::ST);
        const float2 t = v[r] * rx;
        v[r] = make_float2(fmaf(ry, w[r].x, t.x), fmaf(ry, w[r].y, t.y));
      }
    }
    y_store<N, H>(v, a0, p, x0, c, j);
  }
}

// Full fan-out state -> combined state, in place: a0 <- r_x a0 + r_y a1 (the same arithmetic as the
// combined fan-out; a2 is shared by both states).  Element-wise over [kz][y][x] spectra.
template <int N>
__global__ void __launch_bounds__(256) k_y_combine(float2* __restrict__ a0, const float2* __restrict__ a1, Geo g,
                                                   const int* __restrict__ active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long cn = (long long)(N / 2 + 1) * N * N;
  a0 += b * cn; a1 += b * cn;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < cn; i += (long long)gridDim.x * 256) {
    const float rx = los_comp(g, 0, (int)(i % N)), ry = los_comp(g, 1, (int)((i / N) % N));
    const float2 t = a0[i] * rx, w = a1[i];
    a0[i] = make_float2(fmaf(ry, w.x, t.x), fmaf(ry, w.y, t.y));
  }
}

// Forward y with the divergence fan-in.  In: a0 = Z[q], a1 = i k'_z Z[r_z q] (z spectra of the
// iteration's q = u / |r| with r the scaled line of sight, so that V_j = q r_j):
//   a0 <- r_x Y[a0]                   (x component Y Z[V_x]; i k'_x applied in the x pass)
//   a1 <- i k'_y Y[r_y a0] + Y[a1]    (y component plus the z component)
template <int N, int H = stream_of<N>()>
__global__ void __launch_bounds__(nty<N>(), N == 512 ? 4 : 1) k_y_fanin(float2* __restrict__ a0, float2* __restrict__ a1, Geo g,
                                                      const int* __restrict__ active, const float2* __restrict__ twg) {
  constexpr int NT = nty<N>(), W = wy<N>();
  using Y = YTile<N>;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[Y::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int p, x0, c, j;
  y_tile_coords<N, W>(p, x0);
  Y::coords(c, j);
  const bool act = Y::active();
  const long long cn = (long long)(N / 2 + 1) * N * N;
  a0 += b * cn; a1 += b * cn;
  float2 v[Y::E], keep[Y::E];
  if (act) {
    y_load<N, H>(v, a0, p, x0, c, j);
#pragma unroll
    for (int r = 0; r < Y::E; ++r) keep[r] = v[r] * los_comp(g, 1, j + r * Y::ST);
  }
  Y::template fft<false>(v, buf, tw, c, j);
  if (act) {
    const float rx = los_comp(g, 0, x0 + c);
#pragma unroll
    for (int r = 0; r < Y::E; ++r) v[r] = v[r] * rx;
    y_store<N, H>(v, a0, p, x0, c, j);
    y_load<N, H>(v, a1, p, x0, c, j);                  // in flight during the next transform
  }
  Y::template fft<false>(keep, buf, tw, c, j);
  if (act) {
#pragma unroll
    for (int r = 0; r < Y::E; ++r) keep[r] = mul_i(keep[r]) * (g.kf * deriv_mode<N>(j + r * Y::ST));
  }
  Y::template fft<false>(v, buf, tw, c, j);
  if (act) {
#pragma unroll
    for (int r = 0; r < Y::E; ++r) v[r] = v[r] + keep[r];
    y_store<N, H>(v, a1, p, x0, c, j);
  }
}

// ---------------------------------------------------------------------------
// x passes.  Tile: W consecutive rows (row = kz * N + ky), all N x; row-fast fragments.
// ---------------------------------------------------------------------------
template <int N, int H = stream_of<N>()>
__device__ __forceinline__ void x_load(float2* v, const float2* __restrict__ a, long long row, int j) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const long long e = row * N + j + r * (N / 8);
    v[r] = in_bounds(e, (long long)(N / 2 + 1) * N * N) ? ld_stream<H>(a + e) : float2{};
  }
}

template <int N, int H = stream_of<N>()>
__device__ __forceinline__ void x_store(const float2* v, float2* __restrict__ a, long long row, int j) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const long long e = row * N + j + r * (N / 8);
    if (in_bounds(e, (long long)(N / 2 + 1) * N * N)) st_stream<H>(a + e, v[r]);
  }
}

// k^2 and the derivative components of element (row, kx).
template <int N>
__device__ __forceinline__ void x_wavenumbers(long long row, int kx, float kf, float& k2, float& dx, float& dy,
                                              float& dz, int& kzi) {
  const int ky = (int)row % N;
  kzi = (int)row / N;
  const float mx = signed_mode<N>(kx), my = signed_mode<N>(ky), mz = (float)kzi;
  k2 = kf * kf * (mx * mx + my * my + mz * mz);
  dx = kf * deriv_mode<N>(kx);
  dy = kf * deriv_mode<N>(ky);
  dz = kzi == N / 2 ? 0.f : kf * mz;
}

// Forward x, Gaussian smoothing S(k) = exp(-k^2 R^2 / 2) with the 1/N^3 of the inverse, inverse x.
template <int N, int NA>
__global__ void __launch_bounds__(ntx<N>()) k_x_smooth(float2* __restrict__ a0, float2* __restrict__ a1, Geo g,
                                                       const float2* __restrict__ twg) {
  constexpr int NT = ntx<N>(), W = wx<N>();
  using L = Lay<N, W, true>;
  __shared__ float2 buf[L::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int c, j;
  frag_coords<N, W, true>(c, j);
  const bool act = threadIdx.x < L::NTF;
  const long long cn = (long long)(N / 2 + 1) * N * N;
  const long long row = (long long)blockIdx.x * W + c;
  const int b = blockIdx.y;
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    float2* arr = (a == 0 ? a0 : a1) + b * cn;
    float2 v[8];
    if (act) x_load<N>(v, arr, row, j);
    fft_rr<N, W, false, true>(v, buf, tw);
    if (act) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float k2, dx, dy, dz;
        int kzi;
        x_wavenumbers<N>(row, j + r * (N / 8), g.kf, k2, dx, dy, dz, kzi);
        v[r] = v[r] * (expf(-k2 * g.smooth_c) * g.inv_n3);
      }
    }
    fft_rr<N, W, true, true>(v, buf, tw);
    if (act) x_store<N>(v, arr, row, j);
  }
}

// Forward x of the overdensity -> D_s (stored); P = D_s / (b k^2 N^3);
// a0 <- X^-1[i k'_x P], a1 <- X^-1[P].
// HELM: the transformed field F is first multiplied by i k'_x and P = i k'_x F / (k^2 N^3); the
// fan-out then yields IFFT[-k'_j k'_x F / k^2], minus the irrotational part of (F) x (Sec. 4.1).
template <int N, bool HELM = false>
__global__ void __launch_bounds__(ntx<N>()) k_x_start(float2* __restrict__ a0, float2* __restrict__ a1,
                                                      float2* __restrict__ ds, Geo g, const float2* __restrict__ twg) {
  constexpr int NT = ntx<N>(), W = wx<N>();
  using L = Lay<N, W, true>;
  __shared__ float2 buf[L::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int c, j;
  frag_coords<N, W, true>(c, j);
  const bool act = threadIdx.x < L::NTF;
  const long long cn = (long long)(N / 2 + 1) * N * N;
  const long long row = (long long)blockIdx.x * W + c;
  const int b = blockIdx.y;
  a0 += b * cn; a1 += b * cn; ds += b * cn;
  float2 v[8], pr[8];
  if (act) x_load<N>(v, a0, row, j);
  fft_rr<N, W, false, true>(v, buf, tw);
  if (act) {
    x_store<N>(v, ds, row, j);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float k2, dx, dy, dz;
      int kzi;
      x_wavenumbers<N>(row, j + r * (N / 8), g.kf, k2, dx, dy, dz, kzi);
      if (HELM) v[r] = mul_i(v[r]) * dx;
      pr[r] = k2 > 0.f ? v[r] * ((HELM ? g.inv_n3 : g.inv_bn3) / k2) : make_float2(0.f, 0.f);
      v[r] = mul_i(pr[r]) * dx;
    }
  }
  fft_rr<N, W, true, true>(v, buf, tw);
  if (act) x_store<N>(v, a0, row, j);
  fft_rr<N, W, true, true>(pr, buf, tw);
  if (act) x_store<N>(pr, a1, row, j);
}

// State X (a0 = X^-1[i k'_x P], a1 = X^-1[P], P = D / (b k^2 N^3)) rebuilt from a stored spectrum D;
// the tail of k_x_start without its forward transform.
template <int N>
__global__ void __launch_bounds__(ntx<N>()) k_x_refan(float2* __restrict__ a0, float2* __restrict__ a1,
                                                      const float2* __restrict__ d, Geo g,
                                                      const int* __restrict__ active, const float2* __restrict__ twg) {
  constexpr int NT = ntx<N>(), W = wx<N>();
  using L = Lay<N, W, true>;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[L::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int c, j;
  frag_coords<N, W, true>(c, j);
  const bool act = threadIdx.x < L::NTF;
  const long long cn = (long long)(N / 2 + 1) * N * N;
  const long long row = (long long)blockIdx.x * W + c;
  a0 += b * cn; a1 += b * cn; d += b * cn;
  float2 v[8], pr[8];
  if (act) {
    x_load<N>(v, d, row, j);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float k2, dx, dy, dz;
      int kzi;
      x_wavenumbers<N>(row, j + r * (N / 8), g.kf, k2, dx, dy, dz, kzi);
      pr[r] = k2 > 0.f ? v[r] * (g.inv_bn3 / k2) : make_float2(0.f, 0.f);
      v[r] = mul_i(pr[r]) * dx;
    }
  }
  fft_rr<N, W, true, true>(v, buf, tw);
  if (act) x_store<N>(v, a0, row, j);
  fft_rr<N, W, true, true>(pr, buf, tw);
  if (act) x_store<N>(pr, a1, row, j);
}

// Helmholtz split output: irrotational = -Psi (the fan-out of the HELM start), solenoidal =
// f x - irrotational; planar [b][3][n^3]; sol may be null.
__global__ void __launch_bounds__(256) k_helm_out(const float* __restrict__ psi, const float* __restrict__ f,
                                                  int n, int batch, float* __restrict__ irr,
                                                  float* __restrict__ sol) {
  const long long n3 = (long long)n * n * n;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n3 * batch; i += (long long)gridDim.x * 256) {
    const long long b = i / n3, c = i - b * n3;
    const float* p = psi + b * 3 * n3;
    const float ix = -p[c], iy = -p[n3 + c], iz = -p[2 * n3 + c];
    irr[(b * 3 + 0) * n3 + c] = ix;
    irr[(b * 3 + 1) * n3 + c] = iy;
    irr[(b * 3 + 2) * n3 + c] = iz;
    if (sol) {
      sol[(b * 3 + 0) * n3 + c] = f[i] - ix;
      sol[(b * 3 + 1) * n3 + c] = -iy;
      sol[(b * 3 + 2) * n3 + c] = -iz;
    }
  }
}

// One iteration's k-space step:
//   div = i k'_x X[a0] + X[a1];  D_{n+1} = D_s + f div  (stored to dnext); with a relaxation weight
//   omega != 1, D_{n+1} = D_n + omega (D_s + f div - D_n)
//   partial sums of  sum w k'^2 |D_{n+1} - D_n|^2 / k^4  and  sum w k'^2 |D_{n+1}|^2 / k^4
//   (w = 2 inside the halved kz axis) -> convergence norm by Parseval
//   P = D_{n+1} / (b k^2 N^3);  a0 <- X^-1[i k'_x P],  a1 <- X^-1[P]
// dprev and dnext may be the same buffer (element-wise in place).
// RECON_X_WAVES > 0: occupancy hint (waves per SIMD) for the x iteration, which bounds its registers
#if RECON_X_WAVES > 0
#define RECON_X_ITER_BOUNDS(N) __launch_bounds__(ntx<N>(), RECON_X_WAVES)
#else
#define RECON_X_ITER_BOUNDS(N) __launch_bounds__(ntx<N>())
#endif
template <int N, int H = stream_of<N>()>
__global__ void RECON_X_ITER_BOUNDS(N) k_x_iter(float2* __restrict__ a0, float2* __restrict__ a1,
                                                     const float2* __restrict__ ds, const float2* dprev,
                                                     float2* dnext, Geo g, double* __restrict__ partials,
                                                     const int* __restrict__ active, const float2* __restrict__ twg,
                                                     float omega) {
  constexpr int NT = ntx<N>(), W = wx<N>();
  using L = Lay<N, W, true>;
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  __shared__ float2 buf[L::SIZE];
  __shared__ float2 tw[N];
  stage_twiddles<N, NT>(tw, twg);
  int c, j;
  frag_coords<N, W, true>(c, j);
  const bool act = threadIdx.x < L::NTF;
  const long long cn = (long long)(N / 2 + 1) * N * N;
  const long long row = (long long)blockIdx.x * W + c;
  a0 += b * cn; a1 += b * cn; ds += b * cn; dprev += b * cn; dnext += b * cn;
  float2 xa[8], v[8];
  if (act) x_load<N, H>(xa, a0, row, j);
  fft_rr<N, W, false, true>(xa, buf, tw);
  if (act) x_load<N, H>(v, a1, row, j);
  fft_rr<N, W, false, true>(v, buf, tw);
  double num = 0.0, den = 0.0;
  if (act) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int kx = j + r * (N / 8);
      float k2, dx, dy, dz;
      int kzi;
      x_wavenumbers<N>(row, kx, g.kf, k2, dx, dy, dz, kzi);
      const float2 div = mul_i(xa[r]) * dx + v[r];
      const long long idx = row * N + kx;
      const float2 dsv = ds[idx];
      const float2 dp = dprev[idx];
      float2 dn = make_float2(fmaf(g.growth, div.x, dsv.x), fmaf(g.growth, div.y, dsv.y));
      if (omega != 1.f) dn = make_float2(fmaf(omega, dn.x - dp.x, dp.x), fmaf(omega, dn.y - dp.y, dp.y));
      dnext[idx] = dn;
      if (k2 > 0.f) {
        const float wgt = (kzi == 0 || kzi == N / 2) ? 1.f : 2.f;
        const float kd2 = dx * dx + dy * dy + dz * dz;
        const float f = wgt * kd2 / (k2 * k2);
        const float ex = dn.x - dp.x, ey = dn.y - dp.y;
        num += (double)(f * (ex * ex + ey * ey));
        den += (double)(f * (dn.x * dn.x + dn.y * dn.y));
        v[r] = dn * (g.inv_bn3 / k2);
      } else {
        v[r] = make_float2(0.f, 0.f);
      }
      xa[r] = mul_i(v[r]) * dx;
    }
  }
  {
    double t1, t2;
    block_sum2<NT>(num, den, &t1, &t2);
    if (threadIdx.x == 0) {
      partials[2 * ((long long)b * gridDim.x + blockIdx.x) + 0] = t1;
      partials[2 * ((long long)b * gridDim.x + blockIdx.x) + 1] = t2;
    }
  }
  fft_rr<N, W, true, true>(xa, buf, tw);
  if (act) x_store<N, H>(xa, a0, row, j);
  fft_rr<N, W, true, true>(v, buf, tw);
  if (act) x_store<N, H>(v, a1, row, j);
}

// ---------------------------------------------------------------------------
// Plane kernels (N <= kPlaneN): one block holds a whole kz plane of a spectrum, N x N, and runs the y and x
// transforms of a step back to back, so a step that was three launches over global memory is one.  What
// bounds these sizes is the latency of a launch's own chain (each of the three took 5 to 8 us at 32^3 and
// 64^3 for 0.1 to 1 us of memory traffic), not bandwidth; a larger plane's arrays do not fit the LDS.
// The chain is kept short: loads are issued before anything is waited for, and the two arrays of a step run
// side by side in two groups of N^2/8 threads, one exchange tile each.  Fan-in to fan-out at 32^3: 10.8 us
// (12.4 with one group; 4.8 + 8.1 + 4.9 as three launches), at 64^3 17.7 us (17.3; 5.1 + 8.5 + 5.4), where
// the transforms of a plane fill the vector units of its one CU.  Eight passes, us, three launches against
// one: 32^3 291 / 202, 64^3 310 / 267, 256 grids of 32^3 1814 / 1195, 128 of 64^3 4637 / 3678.
// Fragments: y form (column x = c, rows y = j + r N/8) and x form (row y = cx, columns x = jx + r N/8), turned
// into each other through the exchange tile.
// ---------------------------------------------------------------------------
// a or b, by value (?: of two array elements would select between addresses and put the array in memory)
__device__ __forceinline__ float2 pick(bool first, float2 a, float2 b) {
  return make_float2(first ? a.x : b.x, first ? a.y : b.y);
}

template <int N, int GROUPS>
struct Plane {
  using LY = Lay<N, N, false>;
  using LX = Lay<N, N, true>;
  static constexpr int NTF = N * N / 8, NT = GROUPS * NTF < 64 ? 64 : GROUPS * NTF;
  static constexpr int TILE = LY::SIZE > LX::SIZE ? LY::SIZE : LX::SIZE;
  static constexpr int SIZE = GROUPS == 1 ? TILE : 3 * TILE;   // (two groups: and a tile to hand values over)
  static_assert(TILE >= 8 * NTF, "a tile holds every fragment");
  float2 *buf, *mid;
  const float2* tw;
  int g, t, c, j, cx, jx;
  bool on;
  __device__ __forceinline__ Plane(float2* b, const float2* w) : tw(w) {
    const int i = threadIdx.x / NTF;
    on = i < GROUPS;
    g = on ? i : 0;
    t = on ? threadIdx.x - i * NTF : NTF;
    buf = b + g * TILE;
    mid = b + 2 * TILE;
    frag_coords<N, N, false>(c, j, t);
    frag_coords<N, N, true>(cx, jx, t);
  }
  __device__ __forceinline__ int row(int r) const { return j + r * (N / 8); }                // y of element r, y form
  __device__ __forceinline__ int at_y(int r) const { return row(r) * N + c; }                // element r, in the plane
  __device__ __forceinline__ int at_x(int r) const { return cx * N + jx + r * (N / 8); }
  // element `at` of plane p of a spectrum (debug build: checked against the whole spectrum, not read outside it)
  __device__ __forceinline__ static bool inside(int p, int at) {
    return in_bounds((long long)p * N * N + at, (long long)(N / 2 + 1) * N * N);
  }
  __device__ __forceinline__ static float2 get(const float2* a, int p, int at) {
    return inside(p, at) ? a[at] : make_float2(0.f, 0.f);
  }
  __device__ __forceinline__ static void set(float2* a, int p, int at, float2 v) {
    if (inside(p, at)) a[at] = v;
  }
  __device__ __forceinline__ void put_y(const float2* v, float2* b) const {                   // to a tile, by (y, x)
#pragma unroll
    for (int r = 0; r < 8; ++r) b[LX::at(c, row(r))] = v[r];
  }
  __device__ __forceinline__ void get_x(float2* v, const float2* b) const {
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = b[LX::at(jx + r * (N / 8), cx)];
  }
  __device__ __forceinline__ void y_to_x(float2* v) const {
    __syncthreads();
    if (on) put_y(v, buf);
    __syncthreads();
    if (on) get_x(v, buf);
  }
  __device__ __forceinline__ void x_to_y(float2* v) const {
    __syncthreads();
    if (on) {
#pragma unroll
      for (int r = 0; r < 8; ++r) buf[LX::at(jx + r * (N / 8), cx)] = v[r];
    }
    __syncthreads();
    if (on) {
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = buf[LX::at(c, row(r))];
    }
  }
  // transforms of the groups for which run is set
  template <bool INV>
  __device__ __forceinline__ void fft_y(float2* v, bool run = true) const {
    fft_rr<N, N, INV, false>(v, buf, tw, run ? t : NTF);
  }
  template <bool INV>
  __device__ __forceinline__ void fft_x(float2* v, bool run = true) const {
    fft_rr<N, N, INV, true>(v, buf, tw, run ? t : NTF);
  }
  // Two groups.  From P in x form to the fan-out, as k_y_fanout does it: group 0 takes v = i k'_x P, group 1
  // v = P.  STORE_X: state X, no fan-out.
  template <bool COMB>
  __device__ __forceinline__ void tail(float2* v, const Geo& geo, int p, bool state_x, float2* a0, float2* a1,
                                       float2* a2) const {
    fft_x<true>(v);
    if (state_x) {
      if (on) {
        float2* a = g == 0 ? a0 : a1;
#pragma unroll
        for (int r = 0; r < 8; ++r) set(a, p, at_x(r), v[r]);
      }
      return;
    }
    x_to_y(v);
    float2 w[8];                                       // what the first round transforms
#pragma unroll
    for (int r = 0; r < 8; ++r) w[r] = pick(g == 0, v[r], mul_i(v[r]) * (geo.kf * deriv_mode<N>(row(r))));
    fft_y<true>(w);
    if (COMB) {
      if (on && g == 1) {
#pragma unroll
        for (int r = 0; r < 8; ++r) mid[r * NTF + t] = w[r];
      }
      __syncthreads();
      if (on && g == 0) {
        const float rx = los_comp(geo, 0, c);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const float ry = los_comp(geo, 1, row(r));
          const float2 s = w[r] * rx, u = mid[r * NTF + t];
          set(a0, p, at_y(r), make_float2(fmaf(ry, u.x, s.x), fmaf(ry, u.y, s.y)));
        }
      }
    } else if (on) {
      float2* a = g == 0 ? a0 : a1;
#pragma unroll
      for (int r = 0; r < 8; ++r) set(a, p, at_y(r), w[r]);
    }
    fft_y<true>(v, g == 1);
    if (on && g == 1) {
      const float kz = geo.kf * deriv_mode<N>(p);
#pragma unroll
      for (int r = 0; r < 8; ++r) set(a2, p, at_y(r), mul_i(v[r]) * kz);
    }
  }
};

// y forward, x forward, smoothing, x inverse, y inverse of one array (blockIdx.z): k_y_plain, k_x_smooth and
// k_y_plain in one.  in_flag [arrays][batch][z tiles]: rows of z tiles flagged 0 are zero and are not read;
// out_flag [batch][z tiles]: such rows are not stored (null: every row).
template <int N>
__global__ void __launch_bounds__((Plane<N, 1>::NT)) k_plane_smooth(float2* __restrict__ a0, float2* __restrict__ a1,
                                                                    Geo g, const float2* __restrict__ twg,
                                                                    const unsigned char* __restrict__ in_flag,
                                                                    const unsigned char* __restrict__ out_flag) {
  using P = Plane<N, 1>;
  __shared__ float2 buf[P::SIZE];
  __shared__ float2 tw[N];
  const P pl(buf, tw);
  constexpr int NZT = N / (2 * wz<N>());
  const int p = blockIdx.x, b = blockIdx.y, a = blockIdx.z;
  float2* arr = (a == 0 ? a0 : a1) + ((long long)b * (N / 2 + 1) + p) * N * N;
  if (in_flag) in_flag += ((long long)a * gridDim.y + b) * N * NZT + pl.c / (2 * wz<N>());
  if (out_flag) out_flag += (long long)b * N * NZT + pl.c / (2 * wz<N>());
  float2 v[8];
  if (pl.on) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
      v[r] = !in_flag || in_flag[pl.row(r) * NZT] ? P::get(arr, p, pl.at_y(r)) : make_float2(0.f, 0.f);
  }
  stage_twiddles<N, P::NT>(tw, twg);
  pl.template fft_y<false>(v);
  pl.y_to_x(v);
  pl.template fft_x<false>(v);
  if (pl.on) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float k2, dx, dy, dz;
      int kzi;
      x_wavenumbers<N>((long long)p * N + pl.cx, pl.jx + r * (N / 8), g.kf, k2, dx, dy, dz, kzi);
      v[r] = v[r] * (expf(-k2 * g.smooth_c) * g.inv_n3);
    }
  }
  pl.template fft_x<true>(v);
  pl.x_to_y(v);
  pl.template fft_y<true>(v);
  if (pl.on) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (!out_flag || out_flag[pl.row(r) * NZT]) P::set(arr, p, pl.at_y(r), v[r]);
  }
}

// y forward and x forward of the overdensity, D_s, and the combined fan-out of the plain start: k_y_plain,
// k_x_start and k_y_fanout in one (state X is not stored).
template <int N>
__global__ void __launch_bounds__((Plane<N, 2>::NT)) k_plane_start(float2* __restrict__ a0, float2* __restrict__ a2,
                                                                   float2* __restrict__ ds, Geo g,
                                                                   const float2* __restrict__ twg,
                                                                   const unsigned char* __restrict__ in_flag) {
  using P = Plane<N, 2>;
  __shared__ float2 buf[P::SIZE];
  __shared__ float2 tw[N];
  const P pl(buf, tw);
  constexpr int NZT = N / (2 * wz<N>());
  const int p = blockIdx.x, b = blockIdx.y;
  const long long off = ((long long)b * (N / 2 + 1) + p) * N * N;
  a0 += off; a2 += off; ds += off;
  if (in_flag) in_flag += (long long)b * N * NZT + pl.c / (2 * wz<N>());
  float2 v[8];
  if (pl.on && pl.g == 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
      v[r] = !in_flag || in_flag[pl.row(r) * NZT] ? P::get(a0, p, pl.at_y(r)) : make_float2(0.f, 0.f);
  }
  stage_twiddles<N, P::NT>(tw, twg);
  pl.template fft_y<false>(v, pl.g == 0);
  pl.y_to_x(v);
  pl.template fft_x<false>(v, pl.g == 0);
  if (pl.on && pl.g == 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      P::set(ds, p, pl.at_x(r), v[r]);
      float k2, dx, dy, dz;
      int kzi;
      x_wavenumbers<N>((long long)p * N + pl.cx, pl.jx + r * (N / 8), g.kf, k2, dx, dy, dz, kzi);
      v[r] = k2 > 0.f ? v[r] * (g.inv_bn3 / k2) : make_float2(0.f, 0.f);
      pl.mid[r * P::NTF + pl.t] = v[r];
      v[r] = mul_i(v[r]) * dx;
    }
  }
  __syncthreads();
  if (pl.on && pl.g == 1) {
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = pl.mid[r * P::NTF + pl.t];
  }
  pl.template tail<true>(v, g, p, false, a0, nullptr, a2);
}

// A pass from the z step's output to the next fan-out: k_y_fanin, k_x_iter and k_y_fanout in one.  FAN: the
// fan-out of the realisations marked in fan (PF_COMB: combined, PF_FULL: full); the others' state X is stored.
// Group 0 carries a0, group 1 a1; each takes half of the k-space step's elements.
enum PlaneFan { PF_NONE = 0, PF_COMB = 1, PF_FULL = 2 };
template <int N, int FAN>
__global__ void __launch_bounds__((Plane<N, 2>::NT)) k_plane_iter(float2* __restrict__ a0, float2* __restrict__ a1,
                                                                  float2* __restrict__ a2,
                                                                  const float2* __restrict__ ds, const float2* dprev,
                                                                  float2* dnext, Geo g, double* __restrict__ partials,
                                                                  const int* __restrict__ active,
                                                                  const int* __restrict__ fan,
                                                                  const float2* __restrict__ twg, float omega) {
  using P = Plane<N, 2>;
  __shared__ float2 buf[P::SIZE];
  __shared__ float2 tw[N];
  const P pl(buf, tw);
  const int p = blockIdx.x, b = blockIdx.y;
  const long long off = ((long long)b * (N / 2 + 1) + p) * N * N;
  a0 += off; a1 += off; a2 += off; ds += off; dprev += off; dnext += off;
  float2 v[8], keep[8], dsv[4], dp[4];
  const int r0 = 4 * pl.g;                              // the k-space step's elements of this thread
  if (pl.on) {
    const float2* a = pl.g == 0 ? a0 : a1;
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = P::get(a, p, pl.at_y(r));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      dsv[r] = P::get(ds, p, pl.at_x(r0 + r));
      dp[r] = P::get(dprev, p, pl.at_x(r0 + r));
    }
  }
  if (!active[b]) return;
  stage_twiddles<N, P::NT>(tw, twg);
#pragma unroll
  for (int r = 0; r < 8; ++r) keep[r] = v[r] * los_comp(g, 1, pl.row(r));
  pl.template fft_y<false>(v);
  pl.template fft_y<false>(keep, pl.g == 0);
  if (pl.on && pl.g == 0) {
    const float rx = los_comp(g, 0, pl.c);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      v[r] = v[r] * rx;
      keep[r] = mul_i(keep[r]) * (g.kf * deriv_mode<N>(pl.row(r)));
    }
  }
  __syncthreads();
  if (pl.on) {
    pl.put_y(v, pl.buf);
    if (pl.g == 0) pl.put_y(keep, pl.mid);
  }
  __syncthreads();
  if (pl.on) {
    pl.get_x(v, pl.buf);
    if (pl.g == 1) {
      pl.get_x(keep, pl.mid);
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = v[r] + keep[r];
    }
  }
  pl.template fft_x<false>(v);
  // (a transform of 8 points has no barrier of its own between the reads of mid above and the writes below;
  // the two groups are one wave there, and this states the order without a cost)
  if constexpr (N == 8) __syncthreads();
  // the other group's value of this thread's elements; slot r holds element r of the thread pair
  if (pl.on) {
#pragma unroll
    for (int r = 0; r < 4; ++r) pl.mid[(4 - r0 + r) * P::NTF + pl.t] = pick(pl.g == 0, v[4 + r], v[r]);
  }
  __syncthreads();
  double num = 0.0, den = 0.0;
  if (pl.on) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float2 mine = pick(pl.g == 0, v[r], v[4 + r]), other = pl.mid[(r0 + r) * P::NTF + pl.t];
      const float2 xa = pick(pl.g == 0, mine, other), ya = pick(pl.g == 0, other, mine);
      float k2, dx, dy, dz;
      int kzi;
      x_wavenumbers<N>((long long)p * N + pl.cx, pl.jx + (r0 + r) * (N / 8), g.kf, k2, dx, dy, dz, kzi);
      const float2 div = mul_i(xa) * dx + ya;
      float2 dn = make_float2(fmaf(g.growth, div.x, dsv[r].x), fmaf(g.growth, div.y, dsv[r].y));
      if (omega != 1.f) dn = make_float2(fmaf(omega, dn.x - dp[r].x, dp[r].x), fmaf(omega, dn.y - dp[r].y, dp[r].y));
      P::set(dnext, p, pl.at_x(r0 + r), dn);
      float2 pot = make_float2(0.f, 0.f);
      if (k2 > 0.f) {
        const float wgt = (kzi == 0 || kzi == N / 2) ? 1.f : 2.f;
        const float kd2 = dx * dx + dy * dy + dz * dz;
        const float f = wgt * kd2 / (k2 * k2);
        const float ex = dn.x - dp[r].x, ey = dn.y - dp[r].y;
        num += (double)(f * (ex * ex + ey * ey));
        den += (double)(f * (dn.x * dn.x + dn.y * dn.y));
        pot = dn * (g.inv_bn3 / k2);
      }
      pl.mid[(r0 + r) * P::NTF + pl.t] = pot;          // (the slot this thread has just read)
    }
  }
  __syncthreads();
  if (pl.on) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      v[r] = pl.mid[r * P::NTF + pl.t];
      if (pl.g == 0) v[r] = mul_i(v[r]) * (g.kf * deriv_mode<N>(pl.jx + r * (N / 8)));
    }
  }
  {
    double t1, t2;
    block_sum2<P::NT>(num, den, &t1, &t2);
    if (threadIdx.x == 0) {
      partials[2 * ((long long)b * gridDim.x + p) + 0] = t1;
      partials[2 * ((long long)b * gridDim.x + p) + 1] = t2;
    }
  }
  pl.template tail<FAN == PF_COMB>(v, g, p, FAN == PF_NONE || !fan[b], a0, a1, a2);
}

// Fixed-order reduction of per-block partial pairs: out[b] = sum over blocks, also written to the host's
// pinned buffer (host, when not null), so that no copy has to follow.
__global__ void __launch_bounds__(1024) k_reduce_pairs(const double* __restrict__ partials, int nblk,
                                                       double* __restrict__ out, double* __restrict__ host) {
  // one block per realisation; four independent accumulators per thread keep many loads in flight
  constexpr int NT = 1024;
  const int b = blockIdx.x;
  const double2* p = (const double2*)partials + (long long)b * nblk;
  double s0[4] = {0.0, 0.0, 0.0, 0.0}, s1[4] = {0.0, 0.0, 0.0, 0.0};
  int i = threadIdx.x;
  for (; i + 3 * NT < nblk; i += 4 * NT) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 v = p[i + k * NT];
      s0[k] += v.x;
      s1[k] += v.y;
    }
  }
  for (; i < nblk; i += NT) {
    const double2 v = p[i];
    s0[0] += v.x;
    s1[0] += v.y;
  }
  double t0, t1;
  block_sum2<NT>((s0[0] + s0[1]) + (s0[2] + s0[3]), (s1[0] + s1[1]) + (s1[2] + s1[3]), &t0, &t1);
  if (threadIdx.x == 0) {
    out[2 * b] = t0;
    out[2 * b + 1] = t1;
    if (host) { host[2 * b] = t0; host[2 * b + 1] = t1; }
  }
}

// ---------------------------------------------------------------------------
// Shift: CIC interpolation of Psi at each object with the deposit's stencil.
//   galaxies: disp = -Psi - f (Psi . r_hat) r_hat;  randoms: disp = -Psi
// ---------------------------------------------------------------------------
// CIC interpolation of Psi at one valid position, with the deposit's cell index and fractions, and its
// displacement: galaxies -Psi - f (Psi . r_hat) r_hat, randoms -Psi.  fetch(ix, iy, iz, ii) returns
// Psi at the corner ix, iy, iz (wrapped) of base cell ii, from memory or from a staged footprint.
template <class Fetch>
__device__ __forceinline__ void shift_one_f(float px, float py, float pz, const float uu[3], Fetch fetch,
                                            const CicGeo& cg, float ox, float oy, float oz, float growth,
                                            int galaxies, float d[3]) {
  int ii[3];
  float t[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float fl = floorf(uu[a]);
    t[a] = __fsub_rn(uu[a], fl);
    ii[a] = ((int)fl) & (cg.n - 1);
  }
  // every rounding is spelled out and nothing is contracted, so that the direct and the brick-order
  // shift give the same bits
  float p0 = 0.f, p1 = 0.f, p2 = 0.f;
#pragma unroll
  for (int cnr = 0; cnr < 8; ++cnr) {
    const int dx = cnr & 1, dy = (cnr >> 1) & 1, dz = cnr >> 2;
    const float wx = dx ? t[0] : __fsub_rn(1.f, t[0]), wy = dy ? t[1] : __fsub_rn(1.f, t[1]),
                wz = dz ? t[2] : __fsub_rn(1.f, t[2]);
    const float wgt = __fmul_rn(__fmul_rn(wx, wy), wz);
    const float4 v = fetch(dx, dy, dz, ii);
    p0 = fmaf(wgt, v.x, p0);
    p1 = fmaf(wgt, v.y, p1);
    p2 = fmaf(wgt, v.z, p2);
  }
  float d0 = -p0, d1 = -p1, d2 = -p2;
  if (galaxies && growth != 0.f) {
    const float rx = __fsub_rn(px, ox), ry = __fsub_rn(py, oy), rz = __fsub_rn(pz, oz);
    const float r2 = fmaf(rz, rz, fmaf(ry, ry, __fmul_rn(rx, rx)));
    if (r2 > 0.f) {
      const float ir = rsqrtf(r2);
      const float hx = __fmul_rn(rx, ir), hy = __fmul_rn(ry, ir), hz = __fmul_rn(rz, ir);
      const float u = __fmul_rn(growth, fmaf(p2, hz, fmaf(p1, hy, __fmul_rn(p0, hx))));
      d0 = fmaf(-u, hx, d0);
      d1 = fmaf(-u, hy, d1);
      d2 = fmaf(-u, hz, d2);
    }
  }
  d[0] = d0;
  d[1] = d1;
  d[2] = d2;
}

// The same from the displacement in memory (planar, one realisation's [3][N^3]).
__device__ __forceinline__ void shift_one(float px, float py, float pz, const float uu[3], const float* __restrict__ pb,
                                          const CicGeo& cg, float ox, float oy, float oz, float growth,
                                          int galaxies, float d[3]) {
  const int m = cg.n - 1, n = cg.n;
  const long long n3 = (long long)n * n * n;
  shift_one_f(px, py, pz, uu,
              [&](int dx, int dy, int dz, const int ii[3]) {
                const long long c = (((long long)((ii[2] + dz) & m) * n + ((ii[1] + dy) & m)) * n) + ((ii[0] + dx) & m);
                return in_bounds(c, n3) ? make_float4(pb[c], pb[n3 + c], pb[2 * n3 + c], 0.f) : float4{};
              },
              cg, ox, oy, oz, growth, galaxies, d);
}

// Scaled grid coordinates of a position; false for a non-finite or far position.
__device__ __forceinline__ bool shift_coords(float px, float py, float pz, const CicGeo& cg, float uu[3]) {
  const float pp[3] = {px, py, pz};
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float d = __fsub_rn(pp[a], cg.o[a]);
    uu[a] = keep_rounded(__fmul_rn(d, cg.s));
    ok = ok && (fabsf(uu[a]) < 1073741824.0f);
  }
  return ok;
}

__global__ void __launch_bounds__(256) k_shift(const float* __restrict__ pos, long long n,
                                               const long long* __restrict__ off, int batch,
                                               const float* __restrict__ psi, CicGeo cg, float ox, float oy,
                                               float oz, float growth, int galaxies, float* __restrict__ disp,
                                               float* __restrict__ pos_out) {
  const long long n3 = (long long)cg.n * cg.n * cg.n;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const float px = pos[3 * i], py = pos[3 * i + 1], pz = pos[3 * i + 2];
    float uu[3];
    if (!shift_coords(px, py, pz, cg, uu)) {
#pragma unroll
      for (int a = 0; a < 3; ++a) disp[3 * i + a] = 0.f;
      if (pos_out) {                                         // where it was, as k_shift_unpermute leaves it
        pos_out[3 * i] = __fadd_rn(px, 0.f);
        pos_out[3 * i + 1] = __fadd_rn(py, 0.f);
        pos_out[3 * i + 2] = __fadd_rn(pz, 0.f);
      }
      continue;
    }
    const int b = off ? find_realisation(off, batch, i) : 0;
    float d[3];
    shift_one(px, py, pz, uu, psi + 3 * (long long)b * n3, cg, ox, oy, oz, growth, galaxies, d);
    disp[3 * i] = d[0];
    disp[3 * i + 1] = d[1];
    disp[3 * i + 2] = d[2];
    if (pos_out) {
      pos_out[3 * i] = __fadd_rn(px, d[0]);
      pos_out[3 * i + 1] = __fadd_rn(py, d[1]);
      pos_out[3 * i + 2] = __fadd_rn(pz, d[2]);
    }
  }
}

// The brick-order shift with one block per 16^3 brick: the block stages the displacement at the
// 17^3 nodes its objects' stencils can reach (base cells 0..15 of the brick and their upper corners;
// rows of 17 consecutive x per component) in LDS, then interpolates every object of the brick from
// LDS.  Same arithmetic as k_shift.
template <int NT>
__global__ void __launch_bounds__(NT) k_shift_brick(const float4* __restrict__ sorted,
                                                    const unsigned* __restrict__ start,
                                                    const float* __restrict__ psi, CicGeo cg, float ox, float oy,
                                                    float oz, float growth, int galaxies,
                                                    float4* __restrict__ tmp, unsigned least) {
  constexpr int F = kBrick + 1, F3 = F * F * F;
  __shared__ float px_[F3], py_[F3], pz_[F3];
  const long long key = brick_of_block();
  unsigned lo = start[key], hi = start[key + 1];
  if (!brick_part(lo, hi, least)) return;
  const int n = cg.n, m = n - 1;
  const int nbs = (n + kBrick - 1) / kBrick;
  const long long per = (long long)nbs * nbs * nbs;
  const int b = (int)(key / per);
  const long long kk = key - (long long)b * per;
  const int bx = (int)(kk % nbs) * kBrick, by = (int)((kk / nbs) % nbs) * kBrick,
            bz = (int)(kk / ((long long)nbs * nbs)) * kBrick;
  const long long n3 = (long long)n * n * n;
  const float* pb = psi + 3 * (long long)b * n3;
  // node (lx, ly, lz) of the footprint is grid node (bx + lx, by + ly, bz + lz), wrapped; consecutive
  // threads take consecutive x of one row
  for (int l = threadIdx.x; l < F3; l += NT) {
    const int lx = l % F, ly = (l / F) % F, lz = l / (F * F);
    const long long c = (((long long)((bz + lz) & m) * n + ((by + ly) & m)) * n) + ((bx + lx) & m);
    const bool ok = in_bounds(c, n3);
    px_[l] = ok ? pb[c] : 0.f;
    py_[l] = ok ? pb[n3 + c] : 0.f;
    pz_[l] = ok ? pb[2 * n3 + c] : 0.f;
  }
  __syncthreads();
  constexpr int U = kObjBatch;
  for (long long j0 = (long long)lo + threadIdx.x; j0 < hi; j0 += (long long)NT * U) {
    float4 rr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long j = j0 + (long long)u * NT;
      rr[u] = sorted[j < hi ? j : hi - 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long j = j0 + (long long)u * NT;
      if (j >= hi) break;
      const float4 r = rr[u];
      float uu[3], d[3];
      shift_coords(r.x, r.y, r.z, cg, uu);
      shift_one_f(r.x, r.y, r.z, uu,
                  [&](int dx, int dy, int dz, const int ii[3]) {
                    // the base cell lies in this brick (it decided the object's brick)
                    const int l = ((ii[2] - bz + dz) * F + (ii[1] - by + dy)) * F + (ii[0] - bx + dx);
                    return make_float4(px_[l], py_[l], pz_[l], 0.f);
                  },
                  cg, ox, oy, oz, growth, galaxies, d);
      tmp[j] = make_float4(d[0], d[1], d[2], 0.f);
    }
  }
}

// Back to the caller's order: object i takes the displacement of its slot (an object the deposit
// rejected has no slot: displacement 0, as in k_shift).  Consecutive objects of one
// scatter chunk have their slots in short runs per brick, so their staged results share lines; the
// 8 XCDs (workgroups are dealt to them round robin) each take a contiguous eighth of the objects,
// and a block takes U adjacent 256-object chunks, so that the chunks in flight on one XCD form a
// single window that moves forward in dispatch order and the lines it gathers are reused in that
// XCD's L2 (gridDim.x is a multiple of 8; the result does not depend on the dispatch order).
__global__ void __launch_bounds__(256) k_shift_unpermute(const unsigned* __restrict__ slot_of,
                                                         const float4* __restrict__ tmp, long long n,
                                                         const float* __restrict__ pos, float* __restrict__ disp,
                                                         float* __restrict__ pos_out) {
  const long long chunks = (n + 255) / 256, per_x = gridDim.x / 8;
  const int xcd = blockIdx.x % 8;
  const long long c_lo = chunks * xcd / 8, c_hi = chunks * (xcd + 1) / 8;
  constexpr int U = kObjBatch;
  for (long long c0 = c_lo + (long long)(blockIdx.x / 8) * U; c0 < c_hi; c0 += per_x * U) {
    // the U chunks' slot and staged-result loads are issued together
    unsigned sl[U];
    float4 dd[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = (c0 + u) * 256 + threadIdx.x;
      sl[u] = (c0 + u < c_hi && i < n) ? slot_of[i] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) dd[u] = sl[u] < n ? tmp[sl[u]] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long c = c0 + u;
      const long long i = c * 256 + threadIdx.x;
      if (c >= c_hi || i >= n) continue;
      const float4 d = dd[u];
      float q[3] = {0.f, 0.f, 0.f};
      if (pos_out) {                                         // (read before disp is written, which may be pos)
#pragma unroll
        for (int a = 0; a < 3; ++a) q[a] = pos[3 * i + a];
      }
      disp[3 * i] = d.x;
      disp[3 * i + 1] = d.y;
      disp[3 * i + 2] = d.z;
      if (pos_out) {
        pos_out[3 * i] = __fadd_rn(q[0], d.x);
        pos_out[3 * i + 1] = __fadd_rn(q[1], d.y);
        pos_out[3 * i + 2] = __fadd_rn(q[2], d.z);
      }
    }
  }
}

}  // namespace recon
