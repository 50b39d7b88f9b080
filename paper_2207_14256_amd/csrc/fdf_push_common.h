// Pieces shared by the push kernels: block size, segment lookup, stencils and
// non-temporal particle-state access.
#pragma once
#include "fdf_device.h"
#include "fdf_internal.h"

namespace fdf {
namespace push_detail {

constexpr int kBlock = kPushBlock, kWideBlock = kPushWideBlock;

// The species (its segment in the copy that holds its state), job and
// block-sized chunk of block b of a launch; false: a block without work.
__device__ __forceinline__ bool block_chunk(const PushArgs& a, int64_t b, const Segment** sg, int* job,
                                            int64_t* chunk) {
  const int j = batch_block(a.batch, b, chunk);
  if (j < 0) return false;
  *job = j;
  *sg = a.batch.tables[a.batch.job_cur[j]] + a.batch.job_species[j];
  return true;
}

// The state arrays live in device global memory.  Their pointers come from a
// device-side segment table, so the compiler cannot infer the address space
// and would emit flat instructions; naming the global space gives global
// loads/stores with a scalar base and a 32-bit lane offset.
// (The host pass parses device code too; HIP's vector classes cannot bind
// address-space-qualified references there, and no code is emitted for it.)
#if defined(__HIP_DEVICE_COMPILE__)
#define FDF_GLOBAL __attribute__((address_space(1)))
#else
#define FDF_GLOBAL
#endif
template <typename T> __device__ __forceinline__ const FDF_GLOBAL T* gptr(const T* p) {
  return (const FDF_GLOBAL T*)p;
}
template <typename T> __device__ __forceinline__ T ldnt(const T* p) { return __builtin_nontemporal_load(gptr(p)); }
template <typename T> __device__ __forceinline__ void stnt(T v, T* p) {
  __builtin_nontemporal_store(v, (FDF_GLOBAL T*)p);
}

// Interpolation stencil of the force: CIC (r = 1, 8 points) or TSC (r = 2,
// 27 points).  Every operation is explicit so that each copy of the code is
// instruction-identical (bitwise results whatever slot a particle lands in).
template <bool TSC> struct Stencil { static constexpr int N = TSC ? 27 : 8; };

// FP32 form: x is a 32-bit fixed-point fraction of the box per axis.
template <bool TSC, typename I>
__device__ __forceinline__ void stencil_u32(const uint32_t* xu, int shift, uint32_t gmask, float finv,
                                            I G, I* cell, float* w) {
#pragma clang fp contract(off)
  const uint32_t fmask = (1u << shift) - 1u;
  if constexpr (!TSC) {
    uint32_t i0[3], i1[3];
    float t[3], u[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      i0[d] = xu[d] >> shift;
      i1[d] = (i0[d] + 1u) & gmask;
      t[d] = (float)(xu[d] & fmask) * finv;
      u[d] = 1.0f - t[d];
    }
    const I ax[2] = {(I)mesh_x(i0[0], (uint32_t)G), (I)mesh_x(i1[0], (uint32_t)G)};
    const I ay[2] = {(I)mesh_y(i0[1], (uint32_t)G), (I)mesh_y(i1[1], (uint32_t)G)};
    const I az[2] = {(I)mesh_z(i0[2]), (I)mesh_z(i1[2])};
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
      const int cx = cc >> 2, cy = (cc >> 1) & 1, cz = cc & 1;
      cell[cc] = ax[cx] + ay[cy] + az[cz];
      w[cc] = ((cx ? t[0] : u[0]) * (cy ? t[1] : u[1])) * (cz ? t[2] : u[2]);
    }
  } else {
    // nearest point i = floor(u + 1/2); f = u + 1/2 - i = d + 1/2 in [0, 1)
    uint32_t idx[3][3];
    float wt[3][3];
    const uint32_t half = 1u << (shift - 1);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const uint32_t xs = xu[d] + half;                 // wraps with the box
      const uint32_t i = xs >> shift;
      const float f = (float)(xs & fmask) * finv;
      const float g = 1.0f - f, h = f - 0.5f;
      idx[d][0] = (i - 1u) & gmask;
      idx[d][1] = i;
      idx[d][2] = (i + 1u) & gmask;
      wt[d][0] = 0.5f * (g * g);                        // (1/2 - d)^2 / 2
      wt[d][1] = 0.75f - h * h;                         // 3/4 - d^2
      wt[d][2] = 0.5f * (f * f);                        // (1/2 + d)^2 / 2
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          cell[9 * a + 3 * b + c] =
              (I)mesh_x(idx[0][a], (uint32_t)G) + (I)mesh_y(idx[1][b], (uint32_t)G) + (I)mesh_z(idx[2][c]);
          w[9 * a + 3 * b + c] = (wt[0][a] * wt[1][b]) * wt[2][c];
        }
  }
}

// CIC stencil of the FP32 form as byte offsets into a mesh of CB-byte cells
// (the same corners and weights as stencil_u32<false>): the per-axis terms
// of the brick layout scaled by CB with 24-bit multiplies and shifts (full
// rate), instead of a 32-bit multiplication of every corner's cell index.
template <uint32_t CB>
__device__ __forceinline__ void stencil_u32_bytes(const uint32_t* xu, int shift, uint32_t gmask, float finv,
                                                  uint32_t lg, uint32_t* off, float* w) {
#pragma clang fp contract(off)
  const uint32_t fmask = (1u << shift) - 1u;
  uint32_t i0[3], i1[3];
  float t[3], u[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    i0[d] = xu[d] >> shift;
    i1[d] = (i0[d] + 1u) & gmask;
    t[d] = (float)(xu[d] & fmask) * finv;
    u[d] = 1.0f - t[d];
  }
  // bytes of mesh_x(i) * CB, mesh_y(i) * CB, mesh_z(i) * CB
  auto mul24 = [](uint32_t a, uint32_t b) { return (uint32_t)__umul24(a, b); };
  auto bx = [&](uint32_t i) { return (mul24(i >> 2, CB) << (2u * lg + 2u)) + mul24(i & 3u, 16u * CB); };
  auto by = [&](uint32_t i) { return (mul24(i >> 2, CB) << (lg + 4u)) + mul24(i & 3u, 4u * CB); };
  auto bz = [&](uint32_t i) { return mul24(i >> 2, 64u * CB) + mul24(i & 3u, CB); };
  const uint32_t ax[2] = {bx(i0[0]), bx(i1[0])};
  const uint32_t ay[2] = {by(i0[1]), by(i1[1])};
  const uint32_t az[2] = {bz(i0[2]), bz(i1[2])};
#pragma unroll
  for (int cc = 0; cc < 8; ++cc) {
    const int cx = cc >> 2, cy = (cc >> 1) & 1, cz = cc & 1;
    off[cc] = ax[cx] + ay[cy] + az[cz];
    w[cc] = ((cx ? t[0] : u[0]) * (cy ? t[1] : u[1])) * (cz ? t[2] : u[2]);
  }
}

// FP64 form: x in [0, L) Mpc.
template <bool TSC, typename I>
__device__ __forceinline__ void stencil_f64(const double* x, double ginv, int gm, I G,
                                            I* cell, double* w) {
#pragma clang fp contract(off)
  if constexpr (!TSC) {
    int i0[3], i1[3];
    double t[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = x[d] * ginv;
      const double fl = floor(u);
      t[d] = u - fl;
      i0[d] = ((int)fl) & gm;
      i1[d] = (i0[d] + 1) & gm;
    }
    const I ax[2] = {(I)mesh_x((uint32_t)i0[0], (uint32_t)G), (I)mesh_x((uint32_t)i1[0], (uint32_t)G)};
    const I ay[2] = {(I)mesh_y((uint32_t)i0[1], (uint32_t)G), (I)mesh_y((uint32_t)i1[1], (uint32_t)G)};
    const I az[2] = {(I)mesh_z((uint32_t)i0[2]), (I)mesh_z((uint32_t)i1[2])};
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
      const int cx = cc >> 2, cy = (cc >> 1) & 1, cz = cc & 1;
      cell[cc] = ax[cx] + ay[cy] + az[cz];
      w[cc] = ((cx ? t[0] : 1.0 - t[0]) * (cy ? t[1] : 1.0 - t[1])) * (cz ? t[2] : 1.0 - t[2]);
    }
  } else {
    int idx[3][3];
    double wt[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = x[d] * ginv;
      const double fl = floor(u + 0.5);
      const double dd = u - fl;                         // in [-1/2, 1/2)
      const int i = ((int)fl) & gm;
      idx[d][0] = (i - 1) & gm;
      idx[d][1] = i;
      idx[d][2] = (i + 1) & gm;
      wt[d][0] = 0.5 * ((0.5 - dd) * (0.5 - dd));
      wt[d][1] = 0.75 - dd * dd;
      wt[d][2] = 0.5 * ((0.5 + dd) * (0.5 + dd));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          cell[9 * a + 3 * b + c] = (I)mesh_x((uint32_t)idx[0][a], (uint32_t)G) +
                                    (I)mesh_y((uint32_t)idx[1][b], (uint32_t)G) + (I)mesh_z((uint32_t)idx[2][c]);
          w[9 * a + 3 * b + c] = (wt[0][a] * wt[1][b]) * wt[2][c];
        }
  }
}

// x in [0, L) after a drift of less than L, as numpy.mod(x, L) (floor-mod):
// fmod(x, L) is x below L and the exact difference x - L from L to 2 L.
__device__ __forceinline__ double wrap_box(double x, double L) {
  double r = fabs(x) < L ? x : x - L;
  if (!(x > -L && x < 2.0 * L)) r = fmod(x, L);
  return r < 0.0 ? r + L : r;
}

}  // namespace push_detail
}  // namespace fdf
