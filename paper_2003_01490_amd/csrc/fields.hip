// Domain initialisation, field read-out/write-in and a plain copy kernel.
#include "internal.hpp"

namespace lbmdem {

// fluid at rest (deviation 0), wall layers flagged, claims cleared
template <typename T>
__global__ void k_init(DevDomain d) {
  const size_t N = (size_t)d.N;
  T* a = (T*)d.pdf[0];
  T* b = (T*)d.pdf[1];
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < N;
       c += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(c % d.nx);
    const int j = (int)((c / d.nx) % d.ny);
    const int k = (int)(c / ((size_t)d.nx * d.ny));
    const bool wall = (d.walls[0] && (i == 0 || i == d.nx - 1)) ||
                      (d.walls[1] && (j == 0 || j == d.ny - 1)) ||
                      (d.walls[2] && (k == 0 || k == d.nz - 1));
    d.flags[c] = wall ? F_WALL : 0;
    d.owner[c] = -1;
    if (d.claim) {
      d.claim[c] = 0ull;
      d.shellstamp[c] = 0u;
    }
    if (d.cellw) d.cellw[c] = wall ? F_WALL : 0u;
    const size_t p = pidx(d, i, j, k);
    for (int q = 0; q < Q; ++q) {
      a[(size_t)q * d.nx + p] = T(0.0f);
      b[(size_t)q * d.nx + p] = T(0.0f);
    }
  }
}

template <typename T>
__device__ inline double to_d(T v) {
  return (double)v;
}
template <>
__device__ inline double to_d<__half>(__half v) {
  return (double)__half2float(v);
}

// Field read-out, one pass over the populations for all the planes asked for
// (bound by HBM: 19 values read per cell; a plane per launch through a staging
// copy read them once per plane: velocity and density of 512^3 FP32 18.4 ms,
// now 4.5 ms, 5.4 TB/s).
// Velocity component a of a cell, or (a = -1) its density.  With a body force
// the stored (post-collision) momentum holds the whole impulse; the velocity
// is half-way.
template <typename T>
__device__ __forceinline__ void load_cell(const DevDomain& d, const T* f, size_t p, double* g) {
#pragma unroll
  for (int q = 0; q < Q; ++q) g[q] = to_d<T>(f[(size_t)q * d.nx + p]);
}
__device__ __forceinline__ double cell_moment(const DevDomain& d, const double* g, int a) {
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < Q; ++q) s += g[q] * (a < 0 ? 1 : (a == 0 ? CX[q] : (a == 1 ? CY[q] : CZ[q])));
  return a < 0 ? 1.0 + s : s - 0.5 * d.force[a < 0 ? 0 : a];
}

// planes [first, first + count) of a field into dst (N doubles each)
template <typename T, int FIELD>
__global__ __launch_bounds__(256) void k_get_field(DevDomain d, int first, int count, double* __restrict__ dst) {
  const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x, N = (size_t)d.N;
  if (c >= N) return;
  const T* f = (const T*)(d.ctl->cur ? d.pdf[1] : d.pdf[0]);
  const bool fluid = !(d.flags[c] & (F_SOLID | F_WALL));
  const size_t p = pidx_of(d, c);
  if (FIELD == FIELD_RHO || FIELD == FIELD_VEL) {
    double g[Q];
    if (fluid) load_cell<T>(d, f, p, g);
    if (FIELD == FIELD_RHO) {
      dst[c] = fluid ? cell_moment(d, g, -1) : 0.0;
      return;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (a >= first && a < first + count) dst[(size_t)(a - first) * N + c] = fluid ? cell_moment(d, g, a) : 0.0;
  } else {
    for (int q = first; q < first + count; ++q)
      dst[(size_t)(q - first) * N + c] =
          fluid || FIELD == FIELD_PDF_RAW ? to_d<T>(f[(size_t)q * d.nx + p]) + WQ[q] : 0.0;
  }
}

// canonical flags (bytes) or owners (32-bit) of all cells
__global__ __launch_bounds__(256) void k_get_map(DevDomain d, uint8_t* __restrict__ flags, int32_t* __restrict__ owner) {
  const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= (size_t)d.N) return;
  const uint8_t fl = d.flags[c];
  if (flags) flags[c] = (fl & F_WALL) ? 3 : ((fl & F_SOLID) ? 2 : ((fl & F_SHELL) ? 1 : 0));
  if (owner) owner[c] = (fl & F_SOLID) ? d.owner[c] : -1;
}

template <typename T>
__device__ inline T from_d(double v) {
  return (T)v;
}
template <>
__device__ inline __half from_d<__half>(double v) {
  return __float2half_rn((float)v);
}

template <typename T>
__global__ void k_set_plane(DevDomain d, int q, const double* src) {
  const int cur = d.ctl->cur;
  const size_t N = (size_t)d.N;
  T* f = (T*)d.pdf[cur];
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < N;
       c += (size_t)gridDim.x * blockDim.x)
    f[(size_t)q * d.nx + pidx_of(d, c)] = from_d<T>(src[c] - WQ[q]);
}

// a PDF buffer as 19 plain planes of N cells, as stored (out: from the buffer
// into the planes, else back), for checkpoints
template <typename T>
__global__ void k_planes_copy(DevDomain d, int buf, T* planes, int out) {
  T* f = (T*)(buf ? d.pdf[1] : d.pdf[0]);
  const size_t N = (size_t)d.N;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < N; c += (size_t)gridDim.x * blockDim.x) {
    const size_t p = pidx_of(d, c);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (out)
        planes[(size_t)q * N + c] = f[(size_t)q * d.nx + p];
      else
        f[(size_t)q * d.nx + p] = planes[(size_t)q * N + c];
    }
  }
}

__global__ void k_copy16(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n16) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
       i += (size_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ void k_copy1(uint8_t* dst, const uint8_t* src, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// Density at points (xyz[3n], lattice units) by trilinear interpolation of
// the cell-centre densities of the current state (periodic axes wrap); NaN
// when one of the eight cells is not fluid or lies outside a walled axis.
// Buffer io: the 3n coordinates, then the n results.  Eight lanes per point,
// one per cell, added in cell order (256 points: one thread walking the eight
// cells of a point 82 us, 9 us so: latency).
template <typename T>
__global__ __launch_bounds__(256) void k_probe_density(DevDomain d, double* io, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x, k = t >> 3, c = t & 7;
  const bool in = k < n;
  const T* f = (const T*)(d.ctl->cur ? d.pdf[1] : d.pdf[0]);
  const int nn[3] = {d.nx, d.ny, d.nz};
  int ijk[3] = {0, 0, 0};
  double w = 1.0, rho = 1.0;
  bool ok = in;
  if (in) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double s = io[3 * (size_t)k + a] - 0.5;
      const double fl = floor(s);
      // (the range is checked before the conversion: a coordinate beyond the
      // integers must not wrap into it)
      const int i0 = (int)fmin(fmax(fl, -2147483648.0), 2147483646.0), o = (c >> a) & 1;
      const double fr = s - fl;
      if (d.walls[a]) ok = ok && i0 >= 0 && i0 + 1 < nn[a];
      ijk[a] = d.walls[a] ? i0 + o : wrapmod(i0 + o, nn[a]);
      w *= o ? fr : 1.0 - fr;
    }
  }
  if (ok) {
    if (d.flags[cidx(d, ijk[0], ijk[1], ijk[2])] & (F_SOLID | F_WALL)) ok = false;
    double g[Q];
    load_cell<T>(d, f, pidx(d, ijk[0], ijk[1], ijk[2]), g);
#pragma unroll
    for (int q = 0; q < Q; ++q) rho += g[q];
  }
  const int base = (threadIdx.x & 63) & ~7;
  const bool all = ((__ballot(ok) >> base) & 0xFFull) == 0xFFull;
  double r = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double we = __shfl(w, base + e, 64), re = __shfl(rho, base + e, 64);
    r += we * re;
  }
  if (in && c == 0) io[3 * (size_t)n + k] = all ? r : __builtin_nan("");
}

void launch_probe_density(const DevDomain& d, double* io, int n, hipStream_t s) {
  const dim3 g((unsigned)((8 * (long long)n + 255) / 256));
  if (d.storage == 0)
    hipLaunchKernelGGL(k_probe_density<double>, g, dim3(256), 0, s, d, io, n);
  else if (d.storage == 1)
    hipLaunchKernelGGL(k_probe_density<float>, g, dim3(256), 0, s, d, io, n);
  else
    hipLaunchKernelGGL(k_probe_density<__half>, g, dim3(256), 0, s, d, io, n);
}

// Health check of the fluid: the density 1 + sum_q g_q of up to
// DENSITY_SAMPLES fluid cells spread over the lattice by a multiplicative
// hash (the same cells on every call); one outside (0.5, 1.5), or not finite,
// raises ST_DENSITY.
constexpr int DENSITY_SAMPLES = 65536;
template <typename T>
__global__ void k_density_check(DevDomain d, int n) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const size_t N = (size_t)d.N;
  const size_t c = n == (int)N ? (size_t)k : (size_t)(((unsigned long long)k * 2654435761ull) % N);
  if (d.flags[c] & (F_SOLID | F_WALL)) return;
  const T* f = (const T*)(d.ctl->cur ? d.pdf[1] : d.pdf[0]);
  const size_t p = pidx_of(d, c);
  double rho = 1.0;
  for (int q = 0; q < Q; ++q) rho += to_d<T>(f[(size_t)q * d.nx + p]);
  if (!(rho > 0.5 && rho < 1.5)) atomicOr(d.status, ST_DENSITY);
}

void launch_density_check(const DevDomain& d, hipStream_t s) {
  const int n = d.N < (long long)DENSITY_SAMPLES ? (int)d.N : DENSITY_SAMPLES;
  const dim3 g((unsigned)((n + 255) / 256));
  if (d.storage == 0)
    hipLaunchKernelGGL(k_density_check<double>, g, dim3(256), 0, s, d, n);
  else if (d.storage == 1)
    hipLaunchKernelGGL(k_density_check<float>, g, dim3(256), 0, s, d, n);
  else
    hipLaunchKernelGGL(k_density_check<__half>, g, dim3(256), 0, s, d, n);
}

static dim3 grid_for(size_t n) {
  size_t b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return dim3((unsigned)b);
}

void launch_fill_claims(const DevDomain& d, hipStream_t s) {
  if (d.storage == 0)
    hipLaunchKernelGGL(k_init<double>, grid_for(d.N), dim3(256), 0, s, d);
  else if (d.storage == 1)
    hipLaunchKernelGGL(k_init<float>, grid_for(d.N), dim3(256), 0, s, d);
  else
    hipLaunchKernelGGL(k_init<__half>, grid_for(d.N), dim3(256), 0, s, d);
}

template <typename T>
static void launch_fields_t(const DevDomain& d, int field, int first, int count, double* dst, hipStream_t s) {
  const dim3 g((unsigned)((d.N + 255) / 256)), b(256);
  if (field == FIELD_RHO)
    hipLaunchKernelGGL((k_get_field<T, FIELD_RHO>), g, b, 0, s, d, first, count, dst);
  else if (field == FIELD_VEL)
    hipLaunchKernelGGL((k_get_field<T, FIELD_VEL>), g, b, 0, s, d, first, count, dst);
  else if (field == FIELD_PDF)
    hipLaunchKernelGGL((k_get_field<T, FIELD_PDF>), g, b, 0, s, d, first, count, dst);
  else
    hipLaunchKernelGGL((k_get_field<T, FIELD_PDF_RAW>), g, b, 0, s, d, first, count, dst);
}

void launch_fields(const DevDomain& d, int field, int first, int count, double* dst, hipStream_t s) {
  if (d.storage == 0)
    launch_fields_t<double>(d, field, first, count, dst, s);
  else if (d.storage == 1)
    launch_fields_t<float>(d, field, first, count, dst, s);
  else
    launch_fields_t<__half>(d, field, first, count, dst, s);
}

void launch_get_map(const DevDomain& d, uint8_t* flags, int32_t* owner, hipStream_t s) {
  hipLaunchKernelGGL(k_get_map, dim3((unsigned)((d.N + 255) / 256)), dim3(256), 0, s, d, flags, owner);
}

// src: the full distribution of direction q on every cell
void launch_set_pdf(const DevDomain& d, int q, const double* src, hipStream_t s) {
  if (d.storage == 0)
    hipLaunchKernelGGL(k_set_plane<double>, grid_for(d.N), dim3(256), 0, s, d, q, src);
  else if (d.storage == 1)
    hipLaunchKernelGGL(k_set_plane<float>, grid_for(d.N), dim3(256), 0, s, d, q, src);
  else
    hipLaunchKernelGGL(k_set_plane<__half>, grid_for(d.N), dim3(256), 0, s, d, q, src);
}

void launch_planes_copy(const DevDomain& d, int buf, void* planes, bool out, hipStream_t s) {
  if (d.storage == 0)
    hipLaunchKernelGGL(k_planes_copy<double>, grid_for(d.N), dim3(256), 0, s, d, buf, (double*)planes, out ? 1 : 0);
  else if (d.storage == 1)
    hipLaunchKernelGGL(k_planes_copy<float>, grid_for(d.N), dim3(256), 0, s, d, buf, (float*)planes, out ? 1 : 0);
  else
    hipLaunchKernelGGL(k_planes_copy<__half>, grid_for(d.N), dim3(256), 0, s, d, buf, (__half*)planes, out ? 1 : 0);
}

void launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  if (n16 > 0) {
    size_t b = (n16 + 255) / 256;
    if (b > 16384) b = 16384;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)b), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, n16);
  }
  const size_t tail = bytes - n16 * 16;
  if (tail)
    hipLaunchKernelGGL(k_copy1, dim3(1), dim3(256), 0, s, (uint8_t*)dst + n16 * 16,
                       (const uint8_t*)src + n16 * 16, tail);
}

}  // namespace lbmdem
