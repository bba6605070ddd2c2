// One kernel per kind of access of the transform passes (test_debug_build_checks.py): compiled with
// -DRECON_DEBUG, each must count its out-of-bounds indices.
#include "recon_kernels.hpp"

using namespace recon;

__global__ void probe_zcol_fetch(const float2* a, float2* o, int y, int x0) {
  ZCol<256>::Half h;
  ZCol<256>::fetch(h, a, y, x0);
  o[threadIdx.x] = h.a[0] + h.b[7] + h.na + h.nb;
}
__global__ void probe_zcol_unpack(const float2* b, float2* o, int y, int x0) {
  __shared__ float2 buf[Col<256>::SIZE];
  for (int i = threadIdx.x; i < Col<256>::SIZE; i += 256) buf[i] = b[i];
  __syncthreads();
  ZCol<256>::unpack<true>(buf, o, y, x0, 1.f);
}
__global__ void probe_zfield_load(const float* f, float* o, int y, int x0) {
  o[threadIdx.x] = ZField<256, 4>(f, y, x0, threadIdx.x & 15, threadIdx.x >> 4).load(3, 1);
}
__global__ void probe_zfield_store(float* f, int y, int x0) {
  ZField<256, 4>(f, y, x0, threadIdx.x & 15, threadIdx.x >> 4).store(1.f, 3, 1);
}
__global__ void probe_zfield_load_byte(const unsigned char* f, unsigned char* o, int y, int x0) {
  o[threadIdx.x] = ZField<256, 1>(f, y, x0, threadIdx.x & 15, threadIdx.x >> 4).load_byte(3, 1);
}
__global__ void probe_zfield_load64(const long long* f, long long* o, int y, int x0) {
  o[threadIdx.x] = ZField<256, 8>(f, y, x0, threadIdx.x & 15, threadIdx.x >> 4).load64(3, 1, false);
}
__global__ void probe_y_load(const float2* a, float2* o, int p, int x0) {
  float2 v[y_el<256>()];
  y_load<256>(v, a, p, x0, threadIdx.x & 15, threadIdx.x >> 4);
  for (int r = 0; r < y_el<256>(); ++r) o[threadIdx.x * y_el<256>() + r] = v[r];
}
__global__ void probe_y_store(const float2* b, float2* o, int p, int x0) {
  float2 v[y_el<256>()];
  for (int r = 0; r < y_el<256>(); ++r) v[r] = b[threadIdx.x * y_el<256>() + r];
  y_store<256>(v, o, p, x0, threadIdx.x & 15, threadIdx.x >> 4);
}
__global__ void probe_x_load(const float2* a, float2* o, long long row) {
  float2 v[8];
  x_load<256>(v, a, row, threadIdx.x);
  for (int r = 0; r < 8; ++r) o[threadIdx.x * 8 + r] = v[r];
}

template __global__ void recon::k_plane_smooth<32>(float2*, float2*, Geo, const float2*, const unsigned char*,
                                                   const unsigned char*);
template __global__ void recon::k_plane_start<32>(float2*, float2*, float2*, Geo, const float2*,
                                                  const unsigned char*);
template __global__ void recon::k_plane_iter<32, PF_NONE>(float2*, float2*, float2*, const float2*, const float2*,
                                                          float2*, Geo, double*, const int*, const int*, const float2*,
                                                          float);
template __global__ void recon::k_plane_iter<32, PF_COMB>(float2*, float2*, float2*, const float2*, const float2*,
                                                          float2*, Geo, double*, const int*, const int*, const float2*,
                                                          float);
template __global__ void recon::k_plane_iter<32, PF_FULL>(float2*, float2*, float2*, const float2*, const float2*,
                                                          float2*, Geo, double*, const int*, const int*, const float2*,
                                                          float);
