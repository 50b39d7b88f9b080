// Initial data on the device: seeded Gaussian field, particle sample, and the
// pre-initial-condition transform (sec. 2.1).
#include "fdf_device.h"
#include "fdf_internal.h"
#include "fdf_key.h"

namespace fdf {
namespace {

// BBKS transfer function, q = k / (Gamma h) with k in 1/Mpc.
__device__ __forceinline__ double bbks(double k, double gamma, double h) {
  const double q = k / (gamma * h);
  const double a = 3.89 * q, b = 16.1 * q, c = 5.46 * q, d = 6.71 * q;
  const double poly = 1.0 + a + b * b + c * c * c + (d * d) * (d * d);
  return log1p(2.34 * q) / (2.34 * q) * pow(poly, -0.25);
}

// One thread per stored mode (ix, iy, iz), iz in [0, G/2).  The Philox counter
// is the mode's index in the (G, G, G/2+1) half-complex array, so the draws
// do not depend on storage.  On the iz = 0 plane the mode with the larger
// index takes the conjugate of its partner (-nx, -ny, 0).
template <typename R>
__global__ void k_field_gen(FieldGenArgs a) {
  const int G = a.G, M = G / 2, H = G / 2 + 1;
  const size_t total = (size_t)G * G * M;
  const double V = a.box * a.box * a.box;
  const double kf = 2.0 * 3.14159265358979323846 / a.box;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x) {
    const int iz = (int)(e % M), iy = (int)((e / M) % G), ix = (int)(e / ((size_t)M * G));
    cplx<R> val = {(R)0, (R)0};
    const bool zero = ix == G / 2 || iy == G / 2 || (ix == 0 && iy == 0 && iz == 0);
    if (!zero) {
      int sx = ix, sy = iy;
      bool conj = false;
      if (iz == 0) {
        const int px = (G - ix) % G, py = (G - iy) % G;
        if ((long)ix * G + iy > (long)px * G + py) { sx = px; sy = py; conj = true; }
      }
      const uint64_t m = ((uint64_t)sx * G + sy) * H + iz;
      const u64x4 w = philox4x64(m, 0, 0, 0, a.seed, kStreamField);
      const double u1 = unit_open(w.v[0]), u2 = unit_open(w.v[1]);
      const double r = a.fixed_amp ? 1.0 : sqrt(-log(u1));
      const double ph = 2.0 * 3.14159265358979323846 * u2;
      const int nx = ix < G / 2 ? ix : ix - G, ny = iy < G / 2 ? iy : iy - G;
      const double k = sqrt((kf * nx) * (kf * nx) + (kf * ny) * (kf * ny) + (kf * iz) * (kf * iz));
      const double t = bbks(k, a.gamma, a.h);
      const double pk = a.amp * pow(k, a.ns) * (t * t);
      const double s = sqrt(pk / V) * r;
      double re = s * cos(ph), im = s * sin(ph);
      if (conj) im = -im;
      val = {(R)re, (R)im};
    }
    ((cplx<R>*)a.out)[e] = val;
  }
}

// Spatial order at creation.  Sampling is a function of seed and id, so the
// ids alone are ordered, by a counting sort over the tiles of the sampled
// positions, before any state is written: no particle is moved.  The positions
// are random, so a counting sort over all tiles at once sends every atomic and
// every id to a memory transaction of its own (134 M particles on 512^3: 6.9 ms
// for the ranks, 4.7 ms for the ids).  Two levels instead: the ids go to bins
// of consecutive tiles first, a block's share of a bin together, and each bin is
// then ordered by one block with its tile counts in LDS.
// 134 M particles on 512^3: 1.15 ms (tiles and counts), 0.94 (to the bins), 2.47
// (the bins), 4.6 ms for 11.6; 16.7 M on 256^3: 0.45 ms for 1.35.
constexpr int kPlaceThreads = 1024;
constexpr int kPlaceIds = 16384;         // ids of a scatter block, at most
constexpr int kPlaceBins = 4096;         // bins, at most
constexpr int kPlaceTiles = 16384;       // tiles of a bin, at most

__device__ __forceinline__ uint32_t place_key(const PlaceArgs& a, uint64_t id) {
  const u64x4 wp = philox4x64(id, 0, 0, 0, a.seed, kStreamPosition);
  uint32_t c[3];
  for (int d = 0; d < 3; ++d) c[d] = (uint32_t)(wp.v[d] >> 32) >> a.cell_shift;
  return sort_key::morton_key(c, a.fine_bits) >> (3 * a.fine_bits);
}

// In-place exclusive scan of v[0, n), n a multiple of 1024 or less than it, by
// a block of 1024 threads.
__device__ __forceinline__ void block_scan(uint32_t* v, int n) {
  __shared__ uint32_t wave[kPlaceThreads / 64];
  const int per = n > kPlaceThreads ? n / kPlaceThreads : 1, first = (int)threadIdx.x * per;
  uint32_t sum = 0;
  for (int k = 0; k < per && first + k < n; ++k) sum += v[first + k];
  uint32_t x = sum;   // inclusive over the wave
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if ((threadIdx.x & 63) >= (unsigned)off) x += y;
  }
  if ((threadIdx.x & 63) == 63) wave[threadIdx.x >> 6] = x;
  lds_barrier();
  uint32_t base = x - sum;
  for (unsigned w = 0; w < threadIdx.x >> 6; ++w) base += wave[w];
  for (int k = 0; k < per && first + k < n; ++k) {
    const uint32_t c = v[first + k];
    v[first + k] = base;
    base += c;
  }
  lds_barrier();
}

// Tile of every id, and the number of ids of each bin.
__global__ void __launch_bounds__(kPlaceThreads) k_place_count(PlaceArgs a) {
  __shared__ uint32_t count[kPlaceBins];
  for (int b = threadIdx.x; b < a.nbins; b += kPlaceThreads) count[b] = 0;
  lds_barrier();
  for (int64_t i = blockIdx.x * (int64_t)kPlaceThreads + threadIdx.x; i < a.seg.n;
       i += (int64_t)gridDim.x * kPlaceThreads) {
    const uint32_t k = place_key(a, (uint64_t)i);
    a.key[i] = k;
    atomicAdd(&count[k >> a.tile_bits], 1u);
  }
  lds_barrier();
  for (int b = threadIdx.x; b < a.nbins; b += kPlaceThreads)
    if (count[b]) atomicAdd(&a.count[b], count[b]);
}

// Ids to their bins: a block orders its ids by bin in LDS and reserves a range
// of every bin (a.count: the bins' starts, advanced to their ends).
__global__ void __launch_bounds__(kPlaceThreads) k_place_scatter(PlaceArgs a) {
  __shared__ uint32_t ids[kPlaceIds];
  __shared__ uint16_t bin[kPlaceIds];
  __shared__ uint32_t next[kPlaceBins];    // slot of the bin's next id
  __shared__ uint32_t shift[kPlaceBins];   // from the slot to the place in the bin
  const int64_t first = blockIdx.x * (int64_t)a.block_ids;
  const int n = (int)(a.seg.n - first < a.block_ids ? a.seg.n - first : a.block_ids);
  for (int b = threadIdx.x; b < a.nbins; b += kPlaceThreads) next[b] = 0;
  lds_barrier();
  for (int i = threadIdx.x; i < n; i += kPlaceThreads) atomicAdd(&next[a.key[first + i] >> a.tile_bits], 1u);
  lds_barrier();
  for (int b = threadIdx.x; b < a.nbins; b += kPlaceThreads)
    if (next[b]) shift[b] = atomicAdd(&a.count[b], next[b]);
  lds_barrier();
  block_scan(next, a.nbins);
  for (int b = threadIdx.x; b < a.nbins; b += kPlaceThreads) shift[b] -= next[b];
  lds_barrier();
  for (int i = threadIdx.x; i < n; i += kPlaceThreads) {
    const uint32_t b = a.key[first + i] >> a.tile_bits, s = atomicAdd(&next[b], 1u);
    ids[s] = (uint32_t)(first + i);
    bin[s] = (uint16_t)b;
  }
  lds_barrier();
  for (int s = threadIdx.x; s < n; s += kPlaceThreads) a.binned[(uint32_t)(shift[bin[s]] + s)] = ids[s];
}

// One block per bin: its ids in the order of their tiles.
__global__ void __launch_bounds__(kPlaceThreads) k_place_ids(PlaceArgs a) {
  __shared__ uint32_t next[kPlaceTiles];
  const int tiles = 1 << a.tile_bits;
  const int64_t start = blockIdx.x ? a.count[blockIdx.x - 1] : 0;
  const int64_t end = (int)blockIdx.x == a.nbins - 1 ? a.seg.n : (int64_t)a.count[blockIdx.x];
  for (int t = threadIdx.x; t < tiles; t += kPlaceThreads) next[t] = 0;
  lds_barrier();
  for (int64_t i = start + threadIdx.x; i < end; i += kPlaceThreads) {
    const uint32_t t = place_key(a, a.binned[i]) & (tiles - 1);
    a.key[i] = t;
    atomicAdd(&next[t], 1u);
  }
  lds_barrier();
  block_scan(next, tiles);
  for (int64_t i = start + threadIdx.x; i < end; i += kPlaceThreads)
    a.seg.id[start + atomicAdd(&next[a.key[i]], 1u)] = a.binned[i];
}

// Particle sample: uniform positions on the 2^-32 L lattice, |q| from
// q^2 fbar(q) by Gamma(3)-proposal rejection, isotropic directions; momentum
// components rounded once to binary32 (the canonical state of both forms).
__global__ void k_sample(SampleArgs a) {
  const int64_t n = a.seg.n;
  const double T = a.t_nu;
  const uint64_t seed = a.seed_at ? *a.seed_at : a.seed;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t id = a.by_id ? (uint64_t)a.seg.id[i] : (uint64_t)i;
    const u64x4 wp = philox4x64(id, 0, 0, 0, seed, kStreamPosition);
    uint32_t xu[3];
    for (int d = 0; d < 3; ++d) xu[d] = (uint32_t)(wp.v[d] >> 32);
    float qf[3];
    sample_momentum(seed, id, T, qf);
    if (a.fp64) {
      const double scale = a.box * 0x1p-32;
      for (int d = 0; d < 3; ++d) {
        a.seg.xd[d][i] = (double)xu[d] * scale;
        a.seg.qd[d][i] = (double)qf[d];
        a.seg.q0d[d][i] = (double)qf[d];
      }
    } else {
      for (int d = 0; d < 3; ++d) {
        a.seg.xu[d][i] = xu[d];
        a.seg.q0f[d][i] = qf[d];
        a.seg.dqf[d][i] = 0.0f;
      }
    }
    if (!a.by_id) a.seg.id[i] = (uint32_t)i;
  }
}

// Pre-initial conditions (sec. 2.1, eq. transform) with the super-horizon
// moments delta = -2 psi and theta_k = k^2 tau psi_k / 2, for which
// grad(nabla^-2 theta) = -(tau/2) grad psi; with nu = 4 and omega = 4/3:
//   q_i -> q_i (1 - psi/2) - (eps tau / 6) d_i psi,  eps = sqrt(q^2 + m^2 a^2).
// grid: [G^3][4] = (d psi/dx, d psi/dy, d psi/dz, psi), CIC-interpolated.
template <typename GR>
__global__ void k_pre_ic(PreIcArgs a) {
  const int64_t n = a.seg.n;
  const int G = a.G;
  const GR* grid = (const GR*)a.grid;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double x[3], q[3];
    for (int d = 0; d < 3; ++d) {
      if (a.fp64) { x[d] = a.seg.xd[d][i]; q[d] = a.seg.qd[d][i]; }
      else {
        x[d] = (double)a.seg.xu[d][i] * (a.box * 0x1p-32);
        q[d] = (double)a.seg.q0f[d][i] + (double)a.seg.dqf[d][i];
      }
    }
    int i0[3], i1[3];
    double t[3];
    for (int d = 0; d < 3; ++d) {
      const double u = x[d] * ((double)G / a.box);
      const double fl = floor(u);
      t[d] = u - fl;
      const int ii = ((int)fl % G + G) % G;
      i0[d] = ii; i1[d] = (ii + 1) % G;
    }
    double acc[4] = {0, 0, 0, 0};
    for (int c = 0; c < 8; ++c) {
      const int cx = c >> 2, cy = (c >> 1) & 1, cz = c & 1;
      const double w = (cx ? t[0] : 1 - t[0]) * (cy ? t[1] : 1 - t[1]) * (cz ? t[2] : 1 - t[2]);
      const size_t cell = (size_t)mesh_x(cx ? i1[0] : i0[0], G) + mesh_y(cy ? i1[1] : i0[1], G) +
                          mesh_z(cz ? i1[2] : i0[2]);
      for (int s = 0; s < 4; ++s) acc[s] += w * (double)grid[cell * 4 + s];
    }
    const double eps = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + (a.m * a.a) * (a.m * a.a));
    for (int d = 0; d < 3; ++d) {
      const float qn = (float)(q[d] * (1.0 - 0.5 * acc[3]) - (eps * a.tau / 6.0) * acc[d]);
      if (a.fp64) { a.seg.qd[d][i] = qn; a.seg.q0d[d][i] = qn; }
      else { a.seg.q0f[d][i] = qn; a.seg.dqf[d][i] = 0.0f; }
    }
  }
}

int grid_for(size_t n, int block) {
  size_t g = (n + block - 1) / block;
  return (int)(g > 65536 * 4 ? 65536 * 4 : (g ? g : 1));
}

}  // namespace

void launch_field_gen(const FieldGenArgs& a, hipStream_t s) {
  const size_t total = (size_t)a.G * a.G * (a.G / 2);
  if (a.fp64) hipLaunchKernelGGL(k_field_gen<double>, dim3(grid_for(total, 256)), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_field_gen<float>, dim3(grid_for(total, 256)), dim3(256), 0, s, a);
}

void launch_sample_species(const SampleArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_sample, dim3(grid_for((size_t)a.seg.n, 256)), dim3(256), 0, s, a);
}

void launch_place_species(const PlaceArgs& args, hipStream_t s) {
  PlaceArgs a = args;
  // Bins of no more tiles than a block counts and of about 4096 ids, fewer where
  // that leaves CUs without a bin (32 K ids: 17 us in bins of 4096, 6 in
  // bins of 512).
  int bins = (int)std::max<int64_t>(1, a.nkeys / kPlaceTiles);
  const int64_t per = std::min<int64_t>(4096, std::max<int64_t>(512, a.seg.n / 256));
  while (bins < kPlaceBins && bins < a.nkeys && bins * per < a.seg.n) bins *= 2;
  a.nbins = bins;
  a.tile_bits = 0;
  while (((int64_t)bins << a.tile_bits) < a.nkeys) ++a.tile_bits;
  // a block per CU at least
  const int64_t share = (a.seg.n / 256 + kPlaceThreads - 1) / kPlaceThreads * kPlaceThreads;
  a.block_ids = (int32_t)std::min<int64_t>(kPlaceIds, std::max<int64_t>(share, kPlaceThreads));
  launch_fill_zero(a.count, ((size_t)bins * 4 + 15) / 16 * 16, s);
  const int64_t blocks = (a.seg.n + kPlaceThreads - 1) / kPlaceThreads;
  hipLaunchKernelGGL(k_place_count, dim3((unsigned)std::min<int64_t>(blocks, 512)), dim3(kPlaceThreads), 0, s, a);
  launch_scan_exclusive(a.count, bins, a.scan_scratch, s);
  hipLaunchKernelGGL(k_place_scatter, dim3((unsigned)((a.seg.n + a.block_ids - 1) / a.block_ids)), dim3(kPlaceThreads),
                     0, s, a);
  hipLaunchKernelGGL(k_place_ids, dim3((unsigned)bins), dim3(kPlaceThreads), 0, s, a);
}

void launch_pre_ic(const PreIcArgs& a, hipStream_t s) {
  if (a.fp64) hipLaunchKernelGGL(k_pre_ic<double>, dim3(grid_for((size_t)a.seg.n, 256)), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_pre_ic<float>, dim3(grid_for((size_t)a.seg.n, 256)), dim3(256), 0, s, a);
}

}  // namespace fdf
