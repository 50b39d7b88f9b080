// Outputs of the push: delta-f weights (sec. 2.2) and the energy-density
// deposit of eq. empirical_rho, gfx950.
#include <algorithm>
#include <type_traits>

#include "fdf_device.h"
#include "fdf_internal.h"

namespace fdf {
namespace {

// Current momentum (binary64) and the sampled momentum p of particle i.
// PRE: the species has pre-initial conditions (a.pre_ic).
template <bool PRE>
__device__ __forceinline__ void momenta(const OutputArgs& a, int64_t i, uint32_t id,
                                        double* q, double* p) {
  if (a.fp64) {
#pragma unroll
    for (int d = 0; d < 3; ++d) { q[d] = a.seg.qd[d][i]; p[d] = a.seg.q0d[d][i]; }
  } else {
    // q = q0 + dq, exact in binary64
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      p[d] = (double)a.seg.q0f[d][i];
      q[d] = p[d] + (double)a.seg.dqf[d][i];
    }
  }
  if constexpr (PRE) {  // q0 carries the transformed momentum; p is the raw sample
    float pf[3];
    sample_momentum(a.seed, (uint64_t)id, a.t_nu, pf);
#pragma unroll
    for (int d = 0; d < 3; ++d) p[d] = (double)pf[d];
  }
}

// w = 1 - fbar(|q|)/fbar(|p|) = expm1(D/T) / (e^{-|p|/T} + e^{D/T}),
// D = |q| - |p| = (2 p.d + d.d) / (|q| + |p|), d = q - p: no cancellation.
__device__ __forceinline__ double deltaf_weight(const double* q, const double* p, double T) {
  double d[3], pd = 0.0, dd = 0.0, qq = 0.0, pp = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    d[k] = q[k] - p[k];
    pd += p[k] * d[k];
    dd += d[k] * d[k];
    qq += q[k] * q[k];
    pp += p[k] * p[k];
  }
  const double qn = sqrt(qq), pn = sqrt(pp);
  const double den = qn + pn;
  const double D = den > 0.0 ? (2.0 * pd + dd) / den : 0.0;
  return expm1(D / T) / (exp(-pn / T) + exp(D / T));
}

template <bool PRE>
__global__ void __launch_bounds__(256) k_weights(OutputArgs a) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.seg.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t id = a.seg.id[i];
    double q[3], p[3];
    momenta<PRE>(a, i, id, q, p);
    a.w_out[id] = deltaf_weight(q, p, a.t_nu);
  }
}

// Value deposited by particle i: w eps (energy density) or w q_axis = w eps
// v_axis (momentum density), times the per-half normalisation
// G^3 / (N_half <eps>); *half receives the half (even / odd id).
template <bool PRE>
__device__ __forceinline__ double deposit_value(const OutputArgs& a, int64_t i, int* half) {
  const uint32_t id = a.seg.id[i];
  double q[3], p[3];
  momenta<PRE>(a, i, id, q, p);
  const double w = deltaf_weight(q, p, a.t_nu);
  *half = a.auto_mode ? 0 : (int)(id & 1u);
  const double norm = *half ? a.norm[1] : a.norm[0];
  if (a.quantity >= 0) return (w * (a.quantity == 0 ? q[0] : a.quantity == 1 ? q[1] : q[2])) * norm;
  const double eps = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + (a.m * a.a) * (a.m * a.a));
  return (w * eps) * norm;
}

// CIC cell and weights of particle i on the G^3 deposit mesh (vertex-centred
// mesh points, periodic): x-major cell index, or (bricked) the 4^3-brick
// index of the gradient meshes, so that a wave of sorted particles adds into
// a few contiguous kilobytes (G <= 1024: cell indices fit 32 bits).
template <bool BRICKED>
__device__ __forceinline__ void deposit_cic(const OutputArgs& a, int64_t i, uint32_t* cell, double* wc) {
  const int G = a.G;
  const double ginv = (double)G / a.box;
  int i0[3], i1[3];
  double t[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double x = a.fp64 ? a.seg.xd[d][i] : (double)a.seg.xu[d][i] * (a.box * 0x1p-32);
    const double u = x * ginv;
    const double fl = floor(u);
    t[d] = u - fl;
    i0[d] = ((int)fl) & (G - 1);
    i1[d] = (i0[d] + 1) & (G - 1);
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int cx = c >> 2, cy = (c >> 1) & 1, cz = c & 1;
    wc[c] = (cx ? t[0] : 1 - t[0]) * (cy ? t[1] : 1 - t[1]) * (cz ? t[2] : 1 - t[2]);
    const int jx = cx ? i1[0] : i0[0], jy = cy ? i1[1] : i0[1], jz = cz ? i1[2] : i0[2];
    if constexpr (BRICKED)
      cell[c] = mesh_x((uint32_t)jx, (uint32_t)G) + mesh_y((uint32_t)jy, (uint32_t)G) + mesh_z((uint32_t)jz);
    else
      cell[c] = ((uint32_t)jx * (uint32_t)G + (uint32_t)jy) * (uint32_t)G + (uint32_t)jz;
  }
}

// Fixed-point deposit (FP32 form).  Every contribution wc * val is rounded
// to an integer multiple of a quantum Q = 2^(e - bits), where 2^e bounds the
// largest |val| of the spectrum's particles and bits leaves headroom for the
// sum over all of them in 63 bits; the integers are summed with 64-bit
// atomics, so the result does not depend on the order of the additions (bit
// for bit the same from run to run, whatever the launch shape or particle
// order).  Pass 1 finds the largest |val| (as binary32 bits, an order-free
// integer maximum); pass 2 deposits; pass 3 converts to binary32.
__device__ __forceinline__ double fixed_inv_quantum(uint32_t max_bits, int bits) {
  int e;
  frexpf(__uint_as_float(max_bits), &e);   // max |val| < 2^e (e = 0 when there is none)
  return ldexp(1.0, bits - e);
}

template <bool PRE>
__global__ void __launch_bounds__(256) k_deposit_max(OutputArgs a) {
  float m = 0.0f;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.seg.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    int half;
    const double v = fabs(deposit_value<PRE>(a, i, &half));
    m = fmaxf(m, __double2float_ru(v));
  }
  block_max_bits(m, a.max_bits);
}

// Deposit with the additions gathered first in a workgroup hash table of
// lines in LDS (a line: eight consecutive cells of the mesh, 64 bytes; key = 2
// line + half, linear probing), so that the sums of a block's particles reach
// the mesh with one global atomic per touched cell and half, eight lanes to a
// line.  Global atomics are carried out past the per-XCD L2 caches, one memory
// transaction per 64-byte line of an instruction: 19 G/s on scattered cells,
// 145 G/s when eight lanes share a line, which is why the table holds lines
// and not cells.  A contribution whose line finds no slot within kProbe probes
// goes to the mesh directly.  V = unsigned long long: the fixed-point form,
// whose integer sums do not depend on how the additions are grouped or
// ordered; V = double: the FP64 form.
// 134 M sorted particles, one per cell (cross spectrum): 22 ms with a table of
// cells and 256 threads of 4 particles, 13 ms with lines, 7.8 ms with barriers
// that do not wait for the mesh atomics, 6.4 ms with 1024 threads of one
// particle (8 waves per SIMD hide the binary64 weights' and the table's
// latencies; a bigger table with one block per CU: 7.9 ms).

template <typename V, bool PRE, int NT, int R, int LOGS>
__global__ void __launch_bounds__(NT, 4) k_deposit_lds(OutputArgs a) {
  constexpr uint32_t S = 1u << LOGS, kEmpty = 0xFFFFFFFFu;
  constexpr int kProbe = 16;
  constexpr bool kFixed = std::is_same<V, unsigned long long>::value;
  __shared__ uint32_t key[S];
  __shared__ V val[S * 8];
  for (uint32_t s = threadIdx.x; s < S; s += NT) key[s] = kEmpty;
  for (uint32_t s = threadIdx.x; s < S * 8; s += NT) val[s] = (V)0;
  const double scale = kFixed ? fixed_inv_quantum(*a.max_bits, a.fixed_bits) : 1.0;
  lds_barrier();
  auto to_mesh = [&](int half, size_t cell, V v) {
    V* const d = (V*)(half ? a.dens[1] : a.dens[0]) + cell;
    if constexpr (kFixed) atomicAdd(d, v);
    else unsafeAtomicAdd(d, v);
  };
  const int64_t i0 = a.first + (int64_t)blockIdx.x * (NT * R) + threadIdx.x;
#pragma unroll 1
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + r * NT;
    if (i >= a.seg.n) break;
    int half;
    const double v0 = deposit_value<PRE>(a, i, &half) * scale;
    uint32_t cell[8];
    double wc[8];
    deposit_cic<kFixed>(a, i, cell, wc);
    // the slots the lines hash to, read together; most hold their line
    uint32_t h[8], have[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      h[c] = (((cell[c] >> 3) * 2 + half) * 0x9E3779B1u) >> (32 - LOGS);
      have[c] = ((volatile uint32_t*)key)[h[c]];
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t k = (cell[c] >> 3) * 2 + half;
      V v;
      if constexpr (kFixed) v = (V)__double2ll_rn(wc[c] * v0);
      else v = wc[c] * v0;
      if (v == (V)0) continue;
      bool found = have[c] == k;
      if (!found) {
#pragma unroll 1
        for (int p = 0; p < kProbe; ++p) {
          const uint32_t prev = atomicCAS(&key[h[c]], kEmpty, k);
          found = prev == kEmpty || prev == k;
          if (found) break;
          h[c] = (h[c] + 1) & (S - 1);
        }
      }
      if (found) atomicAdd(&val[h[c] * 8 + (cell[c] & 7u)], v);
      else to_mesh(half, cell[c], v);
    }
  }
  lds_barrier();
  for (uint32_t s = threadIdx.x; s < S * 8; s += NT) {
    const uint32_t k = key[s >> 3];
    const V v = val[s];
    if (k != kEmpty && v != (V)0) to_mesh((int)(k & 1u), (size_t)(k >> 1) * 8 + (s & 7u), v);
  }
}

// Bricked fixed-point halves -> x-major binary32 meshes, four cells along z
// per thread: they are contiguous in both layouts (one 32-byte read of the
// brick's z-run, one 16-byte write).
__global__ void k_fixed_to_real(FixedToRealArgs a) {
  const double q = 1.0 / fixed_inv_quantum(*a.max_bits, a.fixed_bits);
  const uint32_t G = (uint32_t)a.G, lg = 31 - __clz(G);
  const size_t n4 = a.n / 4, h4 = a.n_half / 4;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n4;
       i += (size_t)gridDim.x * blockDim.x) {
    const int h = i >= h4;
    const size_t j = 4 * (i - (h ? h4 : 0));     // x-major cell (ix, iy, iz), iz = 0 mod 4
    const uint32_t iz = (uint32_t)(j & (G - 1)), iy = (uint32_t)((j >> lg) & (G - 1)), ix = (uint32_t)(j >> (2 * lg));
    const size_t b = (size_t)mesh_x(ix, G) + mesh_y(iy, G) + mesh_z(iz);
    const longlong2* src = (const longlong2*)(a.src[h] + b);
    const longlong2 v0 = src[0], v1 = src[1];
    *(float4*)(a.dst[h] + j) = make_float4((float)((double)v0.x * q), (float)((double)v0.y * q),
                                           (float)((double)v1.x * q), (float)((double)v1.y * q));
  }
}

// Squared magnitudes of -eps grad psi, -(q^2/eps) grad phi, q (q . grad phi)/eps
// and q phidot at the particle's CIC-interpolated mesh values, summed per
// block in LDS and added to a.out.
__device__ __forceinline__ double term_slot(const TermArgs& a, size_t cell, int slot) {
  if (a.fp64) return ((const double*)a.grid)[cell * a.nslot + slot];
  const uint16_t b = ((const uint16_t*)a.grid)[cell * a.nslot + slot];
  return (double)__uint_as_float((uint32_t)b << 16);
}

__global__ void __launch_bounds__(256) k_force_terms(TermArgs a) {
  __shared__ double red[4][256];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int G = a.G;
  const double ginv = (double)G / a.box;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.seg.n;
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
      const double u = x[d] * ginv;
      const double fl = floor(u);
      t[d] = u - fl;
      i0[d] = ((int)fl) & (G - 1);
      i1[d] = (i0[d] + 1) & (G - 1);
    }
    double gpsi[3] = {0, 0, 0}, gphi[3] = {0, 0, 0}, phidot = 0.0;
    for (int c = 0; c < 8; ++c) {
      const int cx = c >> 2, cy = (c >> 1) & 1, cz = c & 1;
      const double w = (cx ? t[0] : 1 - t[0]) * (cy ? t[1] : 1 - t[1]) * (cz ? t[2] : 1 - t[2]);
      const size_t cell = (size_t)mesh_x(cx ? i1[0] : i0[0], G) + mesh_y(cy ? i1[1] : i0[1], G) +
                          mesh_z(cz ? i1[2] : i0[2]);
      for (int d = 0; d < 3; ++d) {
        gpsi[d] += w * term_slot(a, cell, a.slot_gpsi + d);
        gphi[d] += w * term_slot(a, cell, a.slot_gphi + d);
      }
      if (a.slot_phidot >= 0) phidot += w * term_slot(a, cell, a.slot_phidot);
    }
    const double q2 = q[0] * q[0] + q[1] * q[1] + q[2] * q[2];
    const double eps = sqrt(q2 + a.ma * a.ma);
    const double qg = q[0] * gphi[0] + q[1] * gphi[1] + q[2] * gphi[2];
    const double g2psi = gpsi[0] * gpsi[0] + gpsi[1] * gpsi[1] + gpsi[2] * gpsi[2];
    const double g2phi = gphi[0] * gphi[0] + gphi[1] * gphi[1] + gphi[2] * gphi[2];
    acc[0] += eps * eps * g2psi;
    acc[1] += (q2 / eps) * (q2 / eps) * g2phi;
    acc[2] += q2 * (qg / eps) * (qg / eps);
    acc[3] += q2 * phidot * phidot;
  }
  for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < 4) atomicAdd(&a.out[threadIdx.x], red[threadIdx.x][0]);
}

__global__ void __launch_bounds__(256) k_read_state(ReadStateArgs a) {
  const double scale = a.box * 0x1p-32;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.seg.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = (int64_t)a.seg.id[i] - a.first;
    if (k < 0 || k >= a.count) continue;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double v;
      if (a.momenta) v = a.fp64 ? a.seg.qd[d][i] : (double)a.seg.q0f[d][i] + (double)a.seg.dqf[d][i];
      else v = a.fp64 ? a.seg.xd[d][i] : (double)a.seg.xu[d][i] * scale;
      a.out[3 * k + d] = v;
    }
  }
}

__global__ void k_store(StoreArgs a) {
  for (int i = threadIdx.x; i < a.n; i += blockDim.x) a.dst[i] = a.w[i];
}

__global__ void k_fill_zero(FillArgs a) {
#pragma unroll
  for (int b = 0; b < FillArgs::kBuffers; ++b)
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < a.bytes[b] / 16;
         i += (size_t)gridDim.x * blockDim.x)
      ((uint4*)a.ptr[b])[i] = make_uint4(0, 0, 0, 0);
}

int grid_for(size_t n, int block) {
  size_t g = (n + block - 1) / block;
  return (int)(g > 65536 * 4 ? 65536 * 4 : (g ? g : 1));
}

}  // namespace

void launch_weights(const OutputArgs& a, hipStream_t s) {
  const dim3 grid(grid_for((size_t)a.seg.n, 256));
  if (a.pre_ic) hipLaunchKernelGGL(k_weights<true>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_weights<false>, grid, dim3(256), 0, s, a);
}

void launch_force_terms(const TermArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_force_terms, dim3(std::min(grid_for((size_t)a.seg.n, 256), 4096)), dim3(256), 0, s, a);
}

template <typename V, int NT, int LOGS>
void deposit_nt(const OutputArgs& a, hipStream_t s) {
  OutputArgs p = a;
  for (p.first = 0; p.first < a.seg.n; p.first += kMaxGridThreads) {
    const dim3 grid((unsigned)((std::min(a.seg.n - p.first, kMaxGridThreads) + NT - 1) / NT));
    if (a.pre_ic) hipLaunchKernelGGL((k_deposit_lds<V, true, NT, 1, LOGS>), grid, dim3(NT), 0, s, p);
    else hipLaunchKernelGGL((k_deposit_lds<V, false, NT, 1, LOGS>), grid, dim3(NT), 0, s, p);
  }
}

// Below half a block of 1024 per CU the deposit is as long as one block takes:
// blocks of 256 use four times the CUs.  32 K particles: 23.8 us with 1024, 15.2
// with 256 (binary64 28 and 22); 128 K: 16.8 and 17.0; 2 M (binary64): 261 and
// 306; 16.7 M: 817 and 1135.
template <typename V>
void deposit(const OutputArgs& a, hipStream_t s) {
  if (a.seg.n < 128 * 1024) deposit_nt<V, 256, 9>(a, s);
  else deposit_nt<V, 1024, 10>(a, s);
}

void launch_deposit(const OutputArgs& a, hipStream_t s) {
  // grid_n <= 1024 (checked at creation): the keys 2 line + half stay below
  // the empty key in 32 bits
  if (a.fp64) deposit<double>(a, s);
  else deposit<unsigned long long>(a, s);
}

void launch_deposit_max(const OutputArgs& a, hipStream_t s) {
  const dim3 grid(std::min(grid_for((size_t)a.seg.n, 256), 4096));
  if (a.pre_ic) hipLaunchKernelGGL(k_deposit_max<true>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_deposit_max<false>, grid, dim3(256), 0, s, a);
}

void launch_fixed_to_real(const FixedToRealArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_fixed_to_real, dim3(grid_for(a.n / 4, 256)), dim3(256), 0, s, a);
}

void launch_read_state(const ReadStateArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_read_state, dim3(grid_for((size_t)a.seg.n, 256)), dim3(256), 0, s, a);
}

void launch_store(const StoreArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_store, dim3(1), dim3(128), 0, s, a);
}

// Zero 16-byte aligned buffers whose sizes are multiples of 16 with a plain
// kernel (no memset node, so the work may be captured in a graph).
void launch_fill_zero(const FillArgs& a, hipStream_t s) {
  size_t most = 0;
  for (size_t b : a.bytes) most = std::max(most, b);
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(most / 16, 256)), dim3(256), 0, s, a);
}

}  // namespace fdf
